// Threshold estimate of a head from its sample scores, by a workgroup (threshold_kernel) or by a wave of the
// filter scan.
#pragma once
#include "device_utils.h"
#include "internal.h"
#include "team.h"

namespace tka {

// Threshold estimate of each head: a score with about `rank` of the head's sample scores at or above it,
// by linear binning between the smallest and the largest sample (512 bins): the threshold is
// the lower edge of the bin that holds the rank-th largest sample.  The handful of samples of
// that bin below the rank-th only make the candidate list a little longer (the threshold is a
// heuristic to begin with: the tail checks the candidate count and redoes a head exactly when the
// list does not hold its k best keys).  (A radix select over the float bit pattern spends its
// first digit on sign and exponent, where a few bins take nearly all samples: thousands of
// shared-memory atomics on half a dozen addresses.)  The same histogram gives the parameters of
// tail_bin(), which the tail of the filtered path uses to sort candidates coarsely by score.
// When the range of the samples is so wide that only a few bins lie between the threshold and the
// top of the band the k-th score is expected in, the samples of those bins are binned once more.
constexpr int kThrRefineBelow = 8;   // the bins between threshold and band top are binned again when fewer than this
constexpr int kThrBins = 512;
template <class Team>
struct ThresholdShared {
    uint32_t hist[kThrBins];            // cleared before estimate_threshold()
    float red[2][2][Team::NW];
    uint32_t bin[4];
};
struct Threshold { float thr, bin_lo, bin_inv; };

// Slot j of a thread holds sample j * NT + rank; what lies beyond the sample is ignored.
template <class Team, int CPT>
__device__ __forceinline__ Threshold estimate_threshold(const float (&sv)[CPT], const Plan& pl, ThresholdShared<Team>& sm) {
    constexpr int NT = Team::NT, NB = kThrBins, BPL = NB / kWave;
    const int tid = Team::rank(), lane = lane_id();
    const bool first_wave = Team::NW == 1 || threadIdx.x < kWave;
    const int n_samp = pl.n_samp;
    const uint32_t rank = (uint32_t)(pl.rank < n_samp ? pl.rank : n_samp);
    const uint32_t rank_lo = (uint32_t)(pl.rank_lo < (int)rank ? pl.rank_lo : (int)rank);
    const uint32_t rank_hi = (uint32_t)(pl.rank_hi < (int)rank_lo ? pl.rank_hi : (int)rank_lo);
    // range of the finite samples (a sample beyond a query's own visible prefix is -inf)
    float mx = -INFINITY, mn = INFINITY;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
        const bool ok = j * NT + tid < n_samp;
        if (ok) mx = fmaxf(mx, sv[j]);
        if (ok && sv[j] > -INFINITY) mn = fminf(mn, sv[j]);
    }
    team_range<Team>(mn, mx, sm, 0);
    // sc1 = 0 puts every sample into bin 0 (all samples equal, none finite, or a range beyond fp32)
    const float range = mx - mn;
    const float sc1 = (range > 0.f && range < INFINITY) ? (float)NB / range : 0.f;
    auto place = [](int b) { return (b % BPL) * kWave + b / BPL; };
    auto coarse_bin = [&](float v) {
        int bb = 0;
        if (v > -INFINITY) {
            bb = (int)fminf((v - mn) * sc1, (float)(NB - 1));
            bb = bb < 0 ? 0 : bb;
        }
        return bb;
    };
#pragma unroll
    for (int j = 0; j < CPT; ++j)
        if (j * NT + tid < n_samp) atomicAdd(&sm.hist[place(coarse_bin(sv[j]))], 1u);
    Team::sync();
    // (a lane's bins lie kWave apart, see place(): no bank conflicts in the walk)
    // wave 0 walks the bins from the top: the bins in which the count (on top of `above` samples that lie
    // beyond the last bin) reaches each of the three ranks; sm.bin[3]: samples above the bin of the smallest rank
    auto walk = [&](uint32_t above) {
        uint32_t c[BPL], local = 0;
#pragma unroll
        for (int i = 0; i < BPL; ++i) { c[i] = sm.hist[place(NB - 1 - (BPL * lane + i))]; local += c[i]; }     // lane l owns bins NB - 1 - BPL l - i
        const uint32_t incl = wave_scan_add(local) + above;
        const uint32_t want[3] = {rank, rank_lo, rank_hi};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (incl - local < want[q] && want[q] <= incl) {   // exactly one lane
                uint32_t run = incl - local;
                int found = 0;
                uint32_t before = run;
#pragma unroll
                for (int i = 0; i < BPL; ++i) {                // bins in descending order
                    if (run < want[q] && want[q] <= run + c[i]) { found = NB - 1 - (BPL * lane + i); before = run; }
                    run += c[i];
                }
                sm.bin[q] = (uint32_t)found;
                if (q == 2) sm.bin[3] = before;
            }
        }
    };
    if (first_wave) walk(0u);
    Team::sync();
    int b1 = (int)sm.bin[0], b_lo = (int)sm.bin[1], b_hi = (int)sm.bin[2];
    // threshold: the lower edge of bin b1.  tail_bin(): fine bins over the band of scores the sample puts the
    // k-th score in, from the lower edge of the bin of sample rank_lo to the upper edge of that of sample rank_hi
    float lo = mn, sc = sc1;
    // A few samples far from the rest (keys every query attends to, say) stretch the range, and the whole band
    // falls into a handful of wide bins: the threshold, a bin's lower edge, then lets several times the wanted
    // candidates through.  The samples of those bins are then binned once more over the bins' own range.
    if (sc1 > 0.f && b_hi - b1 < kThrRefineBelow) {
        const float lo2 = mn + (float)b1 / sc1, hi2 = mn + (float)(b_hi + 1) / sc1;
        const float range2 = hi2 - lo2;
        const float sc2 = range2 > 0.f ? (float)NB / range2 : 0.f;
        const uint32_t above = sm.bin[3];                        // samples in the bins above b_hi
        if (sc2 > 0.f && sc2 < INFINITY) {
            Team::sync();                                    // (everyone has read s_bin)
            for (int i = tid; i < NB; i += NT) sm.hist[i] = 0;
            Team::sync();
#pragma unroll
            for (int j = 0; j < CPT; ++j) {
                if (j * NT + tid < n_samp) {
                    const int bb = coarse_bin(sv[j]);            // which samples take part is decided as before, bin by bin
                    if (bb >= b1 && bb <= b_hi) {
                        int fb = (int)fminf((sv[j] - lo2) * sc2, (float)(NB - 1));
                        atomicAdd(&sm.hist[place(fb < 0 ? 0 : fb)], 1u);
                    }
                }
            }
            Team::sync();
            if (first_wave) walk(above);
            Team::sync();
            b1 = (int)sm.bin[0]; b_lo = (int)sm.bin[1]; b_hi = (int)sm.bin[2];
            lo = lo2; sc = sc2;
        }
    }
    float thr = mn, bin_lo = mn, bin_inv = 0.f;
    if (sc > 0.f) {
        thr = (b1 == 0 && lo == mn) ? mn : lo + (float)b1 / sc;
        bin_lo = lo + (float)b_lo / sc;
        const float inv = (float)(kTailBins - 2) * sc / (float)(b_hi + 1 - b_lo);
        bin_inv = inv < INFINITY ? inv : 0.f;
    }
    // (a bin-0 threshold must let -inf samples through when the rank reaches that deep: no finite sample is left out)
    if (b1 == 0 && mn == INFINITY) thr = -INFINITY;
    return Threshold{thr, bin_lo, bin_inv};
}

// A sequence of the batch for which the filter is not worth it (a few tokens only, or k so dense that the
// candidate list cannot hold what passes) gets its threshold like any other: the scan still counts what
// reaches it per bin even where the list overflows, and the tail sorts the keys by those counts.  Its
// heads are marked so that they are not reported as fallbacks (bit 0); bit 2 makes the tail ignore a
// usable list (measurement aid).
__device__ __forceinline__ uint32_t threshold_flags(const Shape& sh, const Plan& pl, int64_t N) {
    return (plan_is_fast(pl, N, sh.cand_cap, true) ? 0u : 1u) | (sh.force_redo ? 4u : 0u);
}

// Leaves a head's threshold; also clears its flags and the call's fallback count.
__device__ __forceinline__ void leave_threshold(const Bufs& bf, int64_t bh, const Threshold& t, uint32_t flags) {
    bf.thr[bh] = t.thr;
    bf.bins[2 * bh] = t.bin_lo;
    bf.bins[2 * bh + 1] = t.bin_inv;
    bf.flags[bh] = flags;
    if (bh == 0) *bf.fallback_total = 0;
}

}  // namespace tka

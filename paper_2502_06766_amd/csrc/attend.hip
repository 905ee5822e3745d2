// Selection and attention of a head in one launch: exact top-k of its scores, softmax over the k selected ones
// (and the always-attended window, if any) and the weighted sum of their value rows -- the knn_search
// result and the attention step of Algorithm 1 of arXiv 2502.06766.  One workgroup per (sequence, head).
//
// It takes over where a head has few scores to select from (a few thousand): a step is then a chain of latencies,
// not a stream.  Every launch adds its ramp and a gap, and a radix select four passes of LDS
// atomics over a handful of exponent bins.  Here the k-th score is found by linear bins between the smallest and
// the largest score, over scores held in registers (the bin it falls in holds a few, which are ranked by
// comparison), and the value rows are fetched by the same workgroup as soon as the winners' positions are in LDS.
//
// What bounds it: a chain of trips to memory and barriers of one compute unit per head, so everything a phase needs is asked for
// ahead, scores stay in registers with slots nobody uses skipped uniformly (the same phases as rolled loops over LDS: 23.6 us
// against 14.5 at 16k tokens) and scans and reductions run in the vector unit instead of trips through LDS.  Measured, 32
// heads, 8 KV heads: a row of 16k scores, k = 256: 13.2 us (radix select + gather: 18.7 + 7.9); a list at 128k tokens, k = 2048:
// 17.1 us (chip-wide tail: 14.5 + 9.6 us and a launch more); 512 heads (16 queries) at 128k tokens 51.0 us.
//
//   attend_kernel        the scores of a short cache, stored by the scan (general path)
//   attend_list_kernel   the candidate list the filtered scan left (what becomes of one that is unusable: below)
//   attend_short_kernel  the scores too, for batches of short sequences
#include <algorithm>
#include <type_traits>

#include "device_utils.h"
#include "internal.h"
#include "scan_common.h"
#include "scan_tiles.h"
#include "select_common.h"
#include "team.h"

namespace tka {

// NT threads with CPT scores each in registers; ROWS: value rows whose positions and weights fit LDS; NB: bins.
template <int NT_, int CPT_, int ROWS_, int NB_>
struct AttendCfg {
    static constexpr int NT = NT_, CPT = CPT_, ROWS = ROWS_, NB = NB_, NW = NT_ / kWave;
    static_assert(NB % NT == 0 && NT % kWave == 0 && NW <= 16 && CPT <= 32, "whole bins per thread, a bit per score, a lane per wave");
};

// What a team shares while it selects; NB bins.
template <class Team, int NB_>
struct SelectShared {
    static constexpr int NB = NB_;
    uint64_t keys[Team::NT + 8];            // segments of the candidate list (length, first entry); later composite keys of the bin that is ranked
    __attribute__((aligned(8))) uint32_t hist[NB_];
    float red[2][2][Team::NW];
    uint32_t tot[2][Team::NW];
    uint32_t sel[3];
    uint32_t n_keys;
};

// Linear bin of a value (monotone; every caller evaluates these roundings).
template <int NB>
__device__ __forceinline__ int lin_bin(float x, float lo, float inv) {
    const float t = __fmul_rn(__fsub_rn(x, lo), inv);
    return (int)fminf(fmaxf(t, 0.f), (float)(NB - 1));
}

// Clears what team_select() counts in; a barrier has to follow (team_range()).
template <class Team, class SM>
__device__ __forceinline__ void select_clear(SM& sm) {
#pragma unroll
    for (int u = 0; u < SM::NB / Team::NT; ++u) sm.hist[Team::rank() + u * Team::NT] = 0;
    if (Team::rank() == 0) sm.n_keys = 0;
}

struct Boundary { uint32_t in, need; };     // what the first step left to rank, and how many of it win

// The k_eff best of the scores in question (1 <= k_eff <= their number), each handed to emit(place, score, position) once:
// bins between the smallest and the largest score (lo, hi), narrowed until the bin the k_eff-th falls in
// holds few.  Every step splits the scores in question: linearly by value, by their order-preserving keys where the
// range is beyond fp32 arithmetic, by their positions where they are all equal (the lower position wins).
// Slot j of a thread holds item j * NT + rank, its score is v(j); bit j of `act` says that there is one.  UNROLL: CPT where
// the scores are registers, less where they are read from LDS.
template <class Team, int CPT, int UNROLL, class Mask, class SM, class ScoreFn, class PosFn, class EmitFn>
__device__ __forceinline__ Boundary team_select(ScoreFn v, Mask act, int n_items, int P, int k_eff, float lo, float hi,
                                                SM& sm, PosFn pos, EmitFn emit) {
    constexpr int NT = Team::NT, NB = SM::NB, BPT = NB / NT;
    // A bin is ranked once it holds no more than this: the ranking compares all pairs, one more split costs less from there
    // on.  16k tokens, 32 heads, k = 256, a key that scores 400 standard deviations up stretching the range until the first bin
    // keeps hundreds: 57 us per call with up to 1024 ranked, 34 with 256 (radix select and gather: 38).
    constexpr uint32_t FEW = NT < 256 ? NT : 256;
    static_assert(NB % NT == 0 && CPT <= 8 * (int)sizeof(Mask), "whole bins per thread, a bit per score");
    const int tid = Team::rank();
    // bin b is counted at place(b): a thread's BPT bins lie NT apart (no bank conflicts in the prefix sum)
    auto place = [](int b) { return (b % BPT) * NT + b / BPT; };
    auto asked = [&](Mask m, int j) { return j * NT < n_items && ((m >> j) & 1u); };     // (the first part is uniform)
    Boundary first{0u, 0u};
    uint32_t need = (uint32_t)k_eff;
    Mask win = 0;                                     // certain winners
    float p_lo = -(float)P, p_hi = 0.f;               // range of the negated positions
    enum { BY_VALUE, BY_KEY, BY_POSITION };
    for (int it = 0; it < 64; ++it) {                 // (a few steps; scores that are not finite must not hang the team)
        const int how = !(hi > lo) ? BY_POSITION : (hi - lo < INFINITY && (float)NB / (hi - lo) < INFINITY) ? BY_VALUE : BY_KEY;
        const uint32_t k_lo = score_key(lo);
        const float base = how == BY_VALUE ? lo : how == BY_KEY ? 0.f : p_lo;
        const float inv = (float)NB / (how == BY_VALUE ? hi - lo : how == BY_KEY ? (float)(score_key(hi) - k_lo) : p_hi - p_lo);
        auto value = [&](int j) {
            float x = v(j);
            if (how != BY_VALUE) x = how == BY_KEY ? (float)(score_key(x) - k_lo) : -(float)pos(j);
            return x;
        };
#pragma unroll UNROLL
        for (int j = 0; j < CPT; ++j)
            if (asked(act, j)) atomicAdd(&sm.hist[place(lin_bin<NB>(value(j), base, inv))], 1u);
        Team::sync();
        {   // the bin in which the counts, summed from the top, reach `need`
            uint32_t n[BPT], local = 0, total;
#pragma unroll
            for (int u = 0; u < BPT; ++u) { n[u] = sm.hist[place(NB - 1 - (tid * BPT + u))]; local += n[u]; }
            uint32_t run = team_prefix<Team>(local, total, sm, 1);
#pragma unroll
            for (int u = 0; u < BPT; ++u) {
                if (run < need && need <= run + n[u]) {          // exactly one thread
                    sm.sel[0] = (uint32_t)(NB - 1 - (tid * BPT + u));
                    sm.sel[1] = run;
                    sm.sel[2] = n[u];
                }
                run += n[u];
            }
        }
        Team::sync();
        const int B = (int)sm.sel[0];
        const uint32_t in = sm.sel[2];
        need -= sm.sel[1];
        if (it == 0) first = Boundary{in, need};
        const bool last = in <= FEW || it == 63;
        // few enough: the bin's scores are ranked by composite key (score key, then inverted position: larger beats
        // smaller, equal scores go to the lower position, no two keys are equal), the need best win
#pragma unroll UNROLL
        for (int j = 0; j < CPT; ++j) {
            if (asked(act, j)) {
                const int bj = lin_bin<NB>(value(j), base, inv);
                if (bj > B) win |= (Mask)1 << j;
                if (bj != B) act &= ~((Mask)1 << j);
                else if (last) {
                    const uint32_t o = atomicAdd(&sm.n_keys, 1u);
                    if (o < (uint32_t)NT) sm.keys[o] = ((uint64_t)score_key(v(j)) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)pos(j));
                }
            }
        }
        if (last) {
            const int n_in = (int)(in < (uint32_t)NT ? in : (uint32_t)NT), n8 = (n_in + 7) & ~7;
            if (tid < n8 - n_in) sm.keys[n_in + tid] = 0ull;             // beats nothing
            // the certain winners come first, by thread, then slot: a fixed order
            uint32_t n_win;
            uint32_t at = team_prefix<Team>((uint32_t)__popcll((uint64_t)win), n_win, sm, 0);
            if (Team::NW == 1) Team::sync();
            if (tid < n_in) {
                const uint64_t mine[1] = {sm.keys[tid]};
                uint32_t rank[1];
                rank_by_comparison<1>(sm.keys, n8, mine, rank);
                if (rank[0] < need)
                    emit((uint32_t)k_eff - need + rank[0], key_score((uint32_t)(mine[0] >> 32)), (int32_t)(0xFFFFFFFFu - (uint32_t)mine[0]));
            }
#pragma unroll UNROLL
            for (int j = 0; j < CPT; ++j)
                if (asked(win, j)) emit(at++, v(j), pos(j));
            break;
        }
        float l2 = INFINITY, h2 = -INFINITY, pl = INFINITY, ph = -INFINITY;
#pragma unroll UNROLL
        for (int j = 0; j < CPT; ++j) {
            if (asked(act, j)) {
                const float p = -(float)pos(j), s = v(j);
                l2 = fminf(l2, s); h2 = fmaxf(h2, s);
                pl = fminf(pl, p); ph = fmaxf(ph, p);
            }
        }
        if (Team::NW == 1) Team::sync();              // (every lane has read the selection)
        select_clear<Team>(sm);
        team_range<Team>(l2, h2, sm, 0);
        team_range<Team>(pl, ph, sm, 1);
        lo = l2; hi = h2; p_lo = pl; p_hi = ph;
    }
    return first;
}

// What becomes of a head's list (the scan's counts per score bin go on where a segment is full):
//   LIST       the entries of the k-th score's bin B fit LDS: the usual case, however long the list is
//   LIST_TIED  they do not (most of them tie): one workgroup goes on alone, by radix select over the list
//   RESCORE    a segment overflowed: the head's workgroups score the keys of its tiles again (arithmetic and dealing of the scan),
//              put those from bin B up into the segments, and the last to finish goes on alone with that list
//   SCORE_ROW  the same where the counts do not cover k keys or the bin does not fit either: all scores go to
//              the score buffer, and the last to finish goes on alone by radix select over the row
// us per call, 32 heads, 8 KV heads, d = 128, chip-wide tail / here.  A quarter of the keys identical and just below the k-th score
// (lists of 36k, 135k at 512k tokens): 128k tokens, k = 2048 88 / 87; 512k tokens 287 / 281; 16 queries at 128k tokens 292 / 237.
// The same on top (tied): 279 / 244, at 16 queries 576 / 509.  Overflow: one KV head, 4 query heads, 512k tokens, 92 %
// identical 161 / 147; 8 KV heads, 512k tokens, 70 % on top (row) 3822 / 2826.  Slower than the tail where one head of
// a batch that fills the chip is scored by its one workgroup: 4 of 256 heads, 128k tokens, 97 % identical 1466 / 1951.

// The head's segments first, first + step, ... (one per wave and step) for RESCORE and SCORE_ROW: exact scores of
// their keys into the score buffer, and those of bin B and above (none: B = kTailBins) into the segment again.
template <int DT, int D>
__device__ __forceinline__ void score_segments(const Shape& sh, const Bufs& bf, int b, int h, int64_t N, int first, int step,
                                               int B, float bin_lo, float bin_inv, uint64_t* list) {
    using v8 = typename Mfma<DT>::v8;
    constexpr int KS = D / 32, SUB = D <= 64 ? 4 : D <= 128 ? 2 : 1;       // runs of 16 keys in flight
    const int64_t bh = (int64_t)b * sh.Hq + h;
    const int lane = lane_id(), jj = lane >> 4, n = lane & 15;
    const char* Kh = static_cast<const char*>(bf.K) + ((int64_t)cache_seq(sh, b) * sh.Hkv + h / sh.G) * sh.Ncap * (D * 2);
    // operand A holds this head alone (rows 0, 4, 8, 12), so that accumulator element 0 is its score in every lane
    v8 qa[KS];
    load_query_a<DT, D>(bf.q, bh, 1, qa);
    const int64_t n_tiles = (N + 63) / 64;
    for (int sid = first; sid < sh.n_seg; sid += step) {
        uint32_t cnt = 0;                                 // entries of bin B and above (uniform over the wave)
        for (int64_t row = 0; row * sh.n_seg < n_tiles; ++row) {
            const int64_t tile = seg_tile(row, sid, sh.n_seg);
            if (tile >= n_tiles) continue;
#pragma unroll 1
            for (int sub0 = 0; sub0 < 4; sub0 += SUB) {
                v8 kb[SUB][KS];
#pragma unroll
                for (int u = 0; u < SUB; ++u) {
                    const int64_t key = tile * 64 + (sub0 + u) * 16 + n;
                    const v8* p = reinterpret_cast<const v8*>(Kh + (key < N ? key : N - 1) * (D * 2)) + jj;
#pragma unroll
                    for (int s = 0; s < KS; ++s) kb[u][s] = p[4 * s];
                }
#pragma unroll
                for (int u = 0; u < SUB; ++u) {
                    f32x4 c = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int s = 0; s < KS; ++s) c = Mfma<DT>::mac(qa[s], kb[u][s], c);
                    const float sc = c[0] + 0.0f;
                    const int64_t key = tile * 64 + (sub0 + u) * 16 + n;
                    const bool mine = jj == 0 && key < N;               // every lane group holds the same scores: the first one writes
                    if (mine) bf.scores[bh * sh.Ncap + key] = sc;
                    const bool keep = mine && tail_bin(sc, bin_lo, bin_inv) >= B;
                    const uint64_t m = __ballot(keep);
                    const uint32_t e = cnt + (uint32_t)mask_rank(m);
                    if (keep && e < (uint32_t)sh.seg_cap)
                        list[cand_slot(e, sid, sh.n_seg)] = ((uint64_t)__float_as_uint(sc) << 32) | (uint64_t)(uint32_t)key;
                    cnt += (uint32_t)__popcll(m);
                }
            }
        }
        if (lane == 0 && B < kTailBins) {
            bf.seg_cnt2[bh * sh.n_seg + sid] = cnt < (uint32_t)sh.seg_cap ? cnt : (uint32_t)sh.seg_cap;
            if (cnt > (uint32_t)sh.seg_cap) atomicOr(&bf.flags[bh], 2u);           // overflowed once more: the score buffer is used
        }
    }
}

// LIST_TIED: the slots of the list as a source of the radix select; `segs`: lengths of its segments (LDS).
template <int NT>
struct SrcSegments {
    static constexpr int kThreads = NT;
    const uint64_t* list;
    const uint32_t* segs;
    int64_t n;
    int log2_n_seg;
    typedef uint64_t raw_t;
    __device__ __forceinline__ int64_t slots() const { return n; }
    __device__ __forceinline__ bool valid(int64_t i) const {
        return i < n && (uint32_t)cand_slot_entry(i, log2_n_seg) < segs[cand_slot_segment(i, log2_n_seg)];
    }
    __device__ __forceinline__ const uint64_t* where(int64_t i) const { return list + i; }
    __device__ __forceinline__ uint32_t key(uint64_t e) const { return score_key(__uint_as_float((uint32_t)(e >> 32))); }
    __device__ __forceinline__ uint32_t ipos(uint64_t e, int64_t) const { return 0xFFFFFFFFu - (uint32_t)e; }
    __device__ __forceinline__ void stash(int, uint64_t) const {}
    __device__ __forceinline__ uint32_t cached_ipos(int) const { return 0u; }
};

// Sums over the lane groups of a wave (lpr lanes each).
template <int EPL>
__device__ __forceinline__ void lane_group_sums(int lpr, float (&acc)[EPL], float& lsum) {
    for (int o = lpr; o < 16; o <<= 1) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] += wave_xor(acc[e], o);
        lsum += wave_xor(lsum, o);
    }
    if (lpr <= 16) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = add_lanes_16(acc[e]);
        lsum = add_lanes_16(lsum);
    }
    if (lpr <= 32) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = add_lanes_32(acc[e]);
        lsum = add_lanes_32(lsum);
    }
}

// The softmax-weighted value rows first .. end - 1 of the list in LDS (score bits, position), summed over the workgroup: thread t < D
// gets channel t, `l` the sum of the weights, which are relative to score M.  (The weights are worked out by the lanes that
// fetch the rows: a few each, where emitting a winner with its weight made every slot of a thread a branch with an exp2f behind it.)
template <int DT, int NT, int U>
__device__ __forceinline__ void weighted_rows(const char* Vh, int D, int N, const uint64_t* rows, int first, int end, float M, float scale_log2e,
                                              float (*acc_lds)[256 + 1], float& a, float& l) {
    constexpr int EPL = Elem<DT>::kPerLoad, NW = NT / kWave;
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lpr = D / EPL, rpw = kWave / lpr;           // lanes per value row, rows per wave and load
    const int rs = lane / lpr, c = lane % lpr, step = NW * rpw;
    // (With half the threads a lane adds up twice as many rows: four sums of every fourth row make up for it.  16 queries of 128k tokens,
    // k = 2048, two draws, relative error of out and lse against 64 bits: one sum 7.0e-7 and 5.6e-7, four 6.0e-7 and 5.4e-7, 1024 threads with
    // one sum 6.0e-7 and 5.3e-7; the same time.)
    constexpr int SUMS = NT == 512 ? 4 : 1;
    float sums[SUMS][EPL], lsums[SUMS];
#pragma unroll
    for (int i = 0; i < SUMS; ++i) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) sums[i][e] = 0.f;
        lsums[i] = 0.f;
    }
    for (int j = first + wave * rpw + rs; j < end; j += U * step) {
        float w[U];
        u32x4 raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int jj = j + u * step < end ? j + u * step : j;
            const uint64_t e = rows[jj];
            w[u] = j + u * step < end ? exp2f((__uint_as_float((uint32_t)(e >> 32)) - M) * scale_log2e) : 0.f;
            const uint32_t p = (uint32_t)e < (uint32_t)N ? (uint32_t)e : (uint32_t)(N - 1);     // (always below N)
            raw[u] = *reinterpret_cast<const u32x4*>(Vh + ((int64_t)p * D + c * EPL) * Elem<DT>::kBytes);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float vf[EPL];
            Elem<DT>::widen(raw[u], vf);
#pragma unroll
            for (int e = 0; e < EPL; ++e) sums[u % SUMS][e] = fmaf(w[u], vf[e], sums[u % SUMS][e]);
            lsums[u % SUMS] += w[u];
        }
    }
    float (&acc)[EPL] = sums[0];
    float& lsum = lsums[0];
#pragma unroll
    for (int i = SUMS / 2; i > 0; i /= 2) {
#pragma unroll
        for (int o = 0; o < i; ++o) {
#pragma unroll
            for (int e = 0; e < EPL; ++e) sums[o][e] += sums[o + i][e];
            lsums[o] += lsums[o + i];
        }
    }
    lane_group_sums(lpr, acc, lsum);
    if (rs == 0) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc_lds[wave][c * EPL + e] = acc[e];
        if (c == 0) acc_lds[wave][256] = lsum;
    }
    __syncthreads();
    a = 0.f; l = 0.f;
    if (tid < D) {
#pragma unroll
        for (int w = 0; w < NW; ++w) { a += acc_lds[w][tid]; l += acc_lds[w][256]; }
    }
}

// Score rows.  Grid: heads x sequences x layers.
template <int DT, class Cfg>
__global__ void __launch_bounds__(Cfg::NT) __attribute__((amdgpu_waves_per_eu(4))) attend_kernel(Shape sh, Bufs bf, float scale, float scale_log2e) {
    fetch_args<kArgBytes>();
    constexpr int NT = Cfg::NT, NW = Cfg::NW, CPT = Cfg::CPT;
    using Team = WorkgroupTeam<NT>;
    __shared__ SelectShared<Team, Cfg::NB> sm;
    __shared__ uint64_t rows_lds[Cfg::ROWS];              // value rows to fetch (score bits, position)
    __shared__ float acc_lds[NW][256 + 1];
    const int b = (int)blockIdx.y + (int)blockIdx.z * sh.layer_seqs, h = blockIdx.x;
    const int64_t bh = (int64_t)b * sh.Hq + h;
    const int tid = threadIdx.x;
    const LayerK lk = bf.layer_k[blockIdx.z];
    const int k = lk.k;
    const int64_t sel0 = selection_at(sh, lk, blockIdx.y, h);
    int32_t* const idx = bf.sel_idx + sel0;
    float* const vals = bf.sel_val + sel0;
    const int D = sh.D;

    // ---- the scores to select from, in registers: slot j of a thread holds item j * NT + tid
    const int N = (int)visible_len(sh, bf, b);
    const int P = (int)prefix_len(N, sh.window), W = N - P;      // searched prefix, window
    const int k_eff = k < P ? k : P;
    const float* const row = bf.scores + bh * sh.Ncap;
    float v[CPT];
    uint32_t act = 0;                                     // bit j: v[j] is a score in question
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
        const int i = j * NT + tid;
        v[j] = row[i < P ? i : 0];                        // (P == 0: the window's scores are there)
        act |= i < P ? 1u << j : 0u;
    }
    float lo = INFINITY, hi = -INFINITY;                  // range of the scores in question
    float w_top = -INFINITY;                              // largest score of the window
    for (int i = tid; i < W; i += NT) w_top = fmaxf(w_top, row[P + i]);
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
        if (j * NT < P) {                                 // (uniform)
            v[j] += 0.0f;                                 // -0 counts as +0
            if ((act >> j) & 1u) { lo = fminf(lo, v[j]); hi = fmaxf(hi, v[j]); }
        }
    }
    select_clear<Team>(sm);
    team_range<Team>(lo, hi, sm, 0);
    if (W > 0) {                                          // (uniform)
        float dummy = 0.f;
        team_range<Team>(dummy, w_top, sm, 1);
    }
    const float M = fmaxf(k_eff > 0 ? hi : -INFINITY, w_top);    // the weights' reference score

    // ---- the k_eff best
    if (k_eff > 0)
        team_select<Team, CPT, CPT>([&](int j) { return v[j]; }, act, P, P, k_eff, lo, hi, sm, [&](int j) { return j * NT + tid; },
                                    [&](uint32_t o, float s, int32_t p) {           // winner o of the head
            if (o < (uint32_t)k_eff)                      // always true; guards the buffer
                rows_lds[o] = ((uint64_t)__float_as_uint(s) << 32) | (uint64_t)(uint32_t)p;
        });
    for (int i = tid; i < W; i += NT) rows_lds[k_eff + i] = ((uint64_t)__float_as_uint(row[P + i]) << 32) | (uint64_t)(uint32_t)(P + i);
    __syncthreads();
    for (int o = tid; o < k; o += NT) {
        const uint64_t e = o < k_eff ? rows_lds[o] : ((uint64_t)0xFF800000u << 32) | 0xFFFFFFFFu;       // (padding: -inf, -1)
        idx[o] = (int32_t)(uint32_t)e;
        vals[o] = __uint_as_float((uint32_t)(e >> 32));
    }

    // ---- the weighted value rows (at most ROWS: the launcher's rule)
    const char* const Vh = static_cast<const char*>(bf.V) + ((int64_t)cache_seq(sh, b) * sh.Hkv + h / sh.G) * sh.Ncap * D * Elem<DT>::kBytes;
    float a, l;
    weighted_rows<DT, NT, 8>(Vh, D, N, rows_lds, 0, k_eff + W, M, scale_log2e, acc_lds, a, l);
    if (tid < D) {
        bf.out[bh * D + tid] = a / l;
        if (tid == 0 && bf.lse) bf.lse[bh] = M * scale + logf(l);
    }
}

// Candidate lists.  Grid: heads x sequences x (workgroups per head x layers).  Shape::share_wgs workgroups of a head all select from
// its list (the same winners, found side by side on compute units that would idle), each keeps and fetches its shares of the
// value rows, and the last to finish adds up the shares; so a head's rows are not bound by what one compute unit can fetch
// (about 64 GB/s).  Further ones, where the heads are few, only lend a hand when keys have to be scored again.
//
// The scan's counts per score bin say without a look at the list which bin B the k-th score falls in and how many entries lie
// above it, and the largest score its waves saw is the weights' reference: an entry above B is a winner as soon as it is
// read, and only those of B (a few hundred at most, as a rule) are ranked, or split once more.  So a head costs four barriers: the segments'
// lengths and the counts, the places of the winners, the ranking, the sum; stamps at 128k tokens: lengths and counts 3.8 us,
// entries 2.4, places 1.3, emission and ranking 2.3, rows and sum 3.5, the shares' exchange 2.0.  The list stays in registers, not in
// LDS, so that two workgroups of 512 threads share a compute unit where there are more than 256.  A first version put the list into
// LDS, found its range, binned it again and split the k-th score's bin (nine barriers, one workgroup per compute unit): 32 heads
// at 128k tokens 19.1 us and 17.1 now, 64 heads with a window 27.4 and 24.7, 512 heads 66.9 and 51.0.
template <int DT, int NT, int D>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) attend_list_kernel(Shape sh, Bufs bf, float scale, float scale_log2e) {
    constexpr int NW = NT / kWave, EPL = 8, LPR = D / EPL, RPW = kWave / LPR;
    constexpr int EDGES = NT == 1024 ? kAttendList : 3584;              // entries of the k-th score's bin that fit LDS (two workgroups of 512 threads share a compute unit)
    constexpr int FEW = 256;                              // more are split again before they are ranked
    constexpr int SPT = kMaxSeg / NT;                     // segments per thread
    using Team = WorkgroupTeam<NT>;
    constexpr int PRE = 8;                                // list slots of a thread in registers
    constexpr int NB = 1024;
    __shared__ SelectShared<Team, NB> sm;
    __shared__ uint64_t rows_lds[kAttendRows];            // value rows to fetch (score bits, position)
    __shared__ uint64_t edge_lds[EDGES];                  // composite keys of the entries of the k-th score's bin; later partial sums
    __shared__ uint32_t segs[kMaxSeg];                    // lengths of the segments
    __shared__ uint32_t bins_lds[NW][kTailBins];
    __shared__ uint32_t red_lds[3][NW];
    __shared__ uint32_t n_edge_lds;                       // entries of the k-th score's bin found
    static_assert(sizeof(edge_lds) >= (NT == 1024 ? 2 : 1) * NW * 257 * sizeof(float) && kTailBins == kWave, "partial sums in place of the entries; a bin per lane");
    float (*const acc_lds)[256 + 1] = reinterpret_cast<float (*)[256 + 1]>(edge_lds);
    const int layer = (int)blockIdx.z & ((1 << sh.log2_layers) - 1);
    const int wg = (int)blockIdx.z >> sh.log2_layers, n_wgs = (int)gridDim.z >> sh.log2_layers;
    const int b = (int)blockIdx.y + layer * sh.layer_seqs, h = blockIdx.x;
    const int64_t bh = (int64_t)b * sh.Hq + h;
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_seg = sh.n_seg, log2_n_seg = 31 - __clz(n_seg), n_scan = n_seg / kScanWaves;
    const bool helper = wg >= sh.share_wgs;               // (uniform)

    // ---- everything the selection starts from is asked for at once
    uint64_t* const list = bf.cand + bh * (int64_t)sh.cand_cap;
    uint32_t seg_len[SPT];
    float seg_top[SPT];
#pragma unroll
    for (int u = 0; u < SPT; ++u) {
        const int g = u * NT + tid;
        seg_len[u] = g < n_seg ? bf.seg_cnt[bh * n_seg + g] : 0u;
        seg_top[u] = g < n_seg ? bf.seg_max[bh * n_seg + g] : -INFINITY;
    }
    const uint32_t flags = bf.flags[bh];
    const float bin_lo = bf.bins[2 * bh], bin_inv = bf.bins[2 * bh + 1];
    uint32_t n_bin = 0;                                   // this wave's share of the counts of bin `lane`
    {
        const uint32_t* const hp = bf.hist + bh * (int64_t)sh.hist_cap * kTailBins + lane;
#pragma unroll 4
        for (int j = wave; j < n_scan; j += NW) n_bin += hp[j * kTailBins];
    }
    // (slots before the segments' lengths are known: any slot of the list may be read, what lies beyond its segment is ignored)
    static_assert(PRE * NT <= kMaxSeg * kCandChunk && PRE <= 32, "every list has room for as many; a bit per slot");
    uint64_t pre[PRE];
#pragma unroll
    for (int u = 0; u < PRE; ++u) pre[u] = helper ? 0ull : (list + u * NT)[tid];
#pragma unroll
    for (int u = 0; u < NB / NT; ++u) sm.hist[u * NT + tid] = 0;         // (while the loads are under way)
    const LayerK lk = bf.layer_k[layer];
    const int k = lk.k;
    const int64_t sel0 = selection_at(sh, lk, blockIdx.y, h);
    int32_t* const idx = bf.sel_idx + sel0;
    float* const vals = bf.sel_val + sel0;
    const int N = (int)visible_len(sh, bf, b);
    const int P = (int)prefix_len(N, sh.window), W = N - P;      // searched prefix, window
    const int k_eff = k < P ? k : P;
    const int64_t head_off = ((int64_t)cache_seq(sh, b) * sh.Hkv + h / sh.G) * sh.Ncap * D * 2;

    enum { LIST = 0, LIST_TIED, RESCORE, SCORE_ROW };
    int how = LIST;                                       // (uniform)
    bool alone = false;                                   // (uniform) this workgroup goes on for the whole head
    uint32_t above = 0, in_b = 0, total = 0;              // keys above bin B, and in it; entries of the list
    uint32_t before = 0;                                  // of them in the segments of the threads before this one
    int B = kTailBins, n_slots = 0;                       // bin of the k-th score; slots of the list in use
    float top = -INFINITY;                                // largest selected score
    if (k_eff > 0) {
        // lengths of the segments, and (with the first barrier) what all threads need to know of them
        auto lay_out = [&]() {
            if (tid == 0) n_edge_lds = 0;
            uint32_t sum = 0, longest = 0;
            float mx = -INFINITY;
#pragma unroll
            for (int u = 0; u < SPT; ++u) {
                segs[u * NT + tid] = seg_len[u];
                sum += seg_len[u];
                longest = seg_len[u] > longest ? seg_len[u] : longest;
                mx = fmaxf(mx, seg_top[u]);
            }
            before = sum;
            sum = wave_scan_add(sum);
            before = sum - before;
            longest = wave_max_u32(longest);
            mx = wave_max(mx);
            if (lane == kWave - 1) { red_lds[0][wave] = sum; red_lds[1][wave] = longest; red_lds[2][wave] = __float_as_uint(mx); }
            bins_lds[wave][lane] = n_bin;
            __syncthreads();
            const bool one = lane < NW;
            const uint32_t t = wave_scan_add(one ? red_lds[0][lane] : 0u);
            total = (uint32_t)__builtin_amdgcn_readlane((int)t, kWave - 1);
            before += wave ? (uint32_t)__builtin_amdgcn_readlane((int)t, wave - 1) : 0u;
            const uint32_t len = wave_max_u32(one ? red_lds[1][lane] : 0u);
            top = wave_max(one ? __uint_as_float(red_lds[2][lane]) : -INFINITY) + 0.0f;
            n_slots = __builtin_amdgcn_readfirstlane((int)((len + kCandChunk - 1) >> kCandChunkLog2) * n_seg * kCandChunk);
            return len;
        };
        const uint32_t longest = lay_out();
        uint32_t all = 0;                                 // lane l looks at bin kTailBins - 1 - l
#pragma unroll
        for (int w = 0; w < NW; ++w) all += bins_lds[w][kTailBins - 1 - lane];
        const uint32_t upto = wave_scan_add(all);
        const uint64_t hit = __ballot(upto - all < (uint32_t)k_eff && (uint32_t)k_eff <= upto);      // (one lane, or the counts do not cover k_eff keys)
        const int hit_lane = hit ? __builtin_ctzll(hit) : 0;
        B = kTailBins - 1 - hit_lane;
        in_b = (uint32_t)__builtin_amdgcn_readlane((int)all, hit_lane);
        above = (uint32_t)__builtin_amdgcn_readlane((int)upto, hit_lane) - in_b;
        // (an index leaves the approximate scores of a head it marked as not filterable)
        const bool over = longest > (uint32_t)sh.seg_cap || (flags & (sh.indexed ? 5u : 4u));
        if (!hit) how = SCORE_ROW;
        else if (over) how = sh.no_rescan || in_b > (uint32_t)EDGES ? SCORE_ROW : RESCORE;
        else if (in_b > (uint32_t)EDGES) how = LIST_TIED;
        how = __builtin_amdgcn_readfirstlane(how);        // (a branch for the compiler too: what one side holds in registers is free on the other)
        if (helper && how < RESCORE) return;              // (uniform)
        // a list that should have been usable (the measure of the chip-wide selection)
        const bool fallback = (over || !hit || in_b > (uint32_t)sh.bnd_cap) && !(flags & 5u) && counts_fallbacks(sh, b);
        if (how == LIST_TIED) {
            if (wg != 0) return;                          // (uniform)
            if (tid == 0 && fallback) atomicAdd(bf.fallback_total, 1u);
            alone = true;
        } else if (how != LIST) {
            score_segments<DT, D>(sh, bf, b, h, P, wg * NW + wave, n_wgs * NW, how == SCORE_ROW ? kTailBins : B, bin_lo, bin_inv, list);
            // every wave waits for its stores to arrive in the L2, one thread releases them all (a release writes back the whole
            // L2 of the XCD; one per wave: 247 us per call instead of 147 at one KV head, 512k tokens, 92 % identical)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid == 0) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                sm.n_keys = atomicAdd(&bf.flags[bh], kArrivalUnit);               // (the threshold estimate cleared the count)
            }
            __syncthreads();
            const uint32_t arrived = (uint32_t)__builtin_amdgcn_readfirstlane((int)sm.n_keys);
            if (arrived / kArrivalUnit + 1u != (uint32_t)n_wgs) return;           // (uniform)
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (tid == 0 && fallback) atomicAdd(bf.fallback_total, 1u);
            alone = true;
            if (how == RESCORE && (arrived & 2u)) how = SCORE_ROW;
            if (how == RESCORE) {
#pragma unroll
                for (int u = 0; u < SPT; ++u) {
                    const int g = u * NT + tid;
                    seg_len[u] = g < n_seg ? bf.seg_cnt2[bh * n_seg + g] : 0u;
                }
                lay_out();                                // (its barrier comes after the readers of what it overwrites)
            }
#pragma unroll
            for (int u = 0; u < PRE; ++u) pre[u] = 0ull;  // (not kept in registers through the scoring)
        }
    } else if (helper) {
        return;                                           // nothing to search for this sequence
    }

    // ---- the window's scores (plain FMAs), into the places behind the winners'
    float w_top = -INFINITY;                              // largest score of the window
    const int n_rows = k_eff + W;                         // rows to fetch (at most kAttendRows: the launcher's rule)
    if (W > 0) {                                          // (uniform)
        const int rs = lane / LPR, c = lane % LPR;
        float qf[EPL];
        Elem<DT>::widen(*reinterpret_cast<const u32x4*>(static_cast<const char*>(bf.q) + (bh * D + c * EPL) * 2), qf);
        const char* const Kh = static_cast<const char*>(bf.K) + head_off;
        constexpr int UW = 4, STEP = NW * RPW;
        for (int j = wave * RPW; j < W; j += UW * STEP) {            // (uniform over the wave)
            u32x4 raw[UW];
#pragma unroll
            for (int u = 0; u < UW; ++u) {
                const int i = j + u * STEP + rs;
                raw[u] = *reinterpret_cast<const u32x4*>(Kh + ((int64_t)(P + (i < W ? i : W - 1)) * D + c * EPL) * 2);
            }
#pragma unroll
            for (int u = 0; u < UW; ++u) {
                const int i = j + u * STEP + rs;
                float kf[EPL], a = 0.f;
                Elem<DT>::widen(raw[u], kf);
#pragma unroll
                for (int e = 0; e < EPL; ++e) a = fmaf(kf[e], qf[e], a);
                a = group_reduce<AddOp, LPR>(a);
                if (i < W) {
                    w_top = fmaxf(w_top, a);
                    if (c == 0) rows_lds[k_eff + i] = ((uint64_t)__float_as_uint(a) << 32) | (uint64_t)(uint32_t)(P + i);
                }
            }
        }
        float dummy = 0.f;
        team_range<Team>(dummy, w_top, sm, 1);
    }
    float M = fmaxf(top, w_top);                          // the weights' reference score
    const bool writer = wg == 0 || alone;                 // (uniform) the workgroup that writes the padding and the record
    // this workgroup's shares, and the value rows they cover: only winners that fall there are emitted (all of them find the same)
    const int shares = alone ? 1 : sh.attend, share_wgs = shares > 1 ? sh.share_wgs : 1;
    const int share0 = share_wgs > 1 ? wg * shares / share_wgs : 0, share1 = share_wgs > 1 ? (wg + 1) * shares / share_wgs : shares;
    auto share_row = [&](int share) { return (int)((uint32_t)(n_rows * share) / (uint32_t)shares); };
    const uint32_t row0 = (uint32_t)share_row(share0), row1 = (uint32_t)share_row(share1);
    auto emit = [&](uint32_t o, float s, uint32_t p) {    // winner o of the head
        if (o - row0 < row1 - row0 && o < (uint32_t)k_eff) {         // (o < k_eff always; guards the buffers)
            rows_lds[o] = ((uint64_t)__float_as_uint(s) << 32) | (uint64_t)p;
        }
    };
    auto score_of = [](uint64_t e) { return __uint_as_float((uint32_t)(e >> 32)); };

    // ---- the k_eff best
    if (k_eff > 0 && (how == LIST || how == RESCORE)) {
        int n_pre = how == LIST ? PRE : 0;                // (uniform) slots per thread in registers
        uint64_t* edges_lds = edge_lds;                   // entries to rank
        auto bin_of = [&](uint64_t ent) { return tail_bin(score_of(ent), bin_lo, bin_inv); };
        // whether slot i holds an entry (cand_slot(), in 32 bits)
        auto filled = [&](int i) {
            const int run = i >> kCandChunkLog2;
            return (uint32_t)(((run >> log2_n_seg) << kCandChunkLog2) | (i & (kCandChunk - 1))) < segs[run & (n_seg - 1)];
        };
        // f(slot, entry) for the entries that are not in registers.  (They are read for every purpose again, and most slots are empty
        // there: the list is as deep as its longest segment.)
        auto rest = [&](auto f) {
            for (int i0 = n_pre * NT + tid; i0 < n_slots; i0 += 4 * NT) {       // (uniform over the wave)
                bool in[4];
                uint64_t ent[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + u * NT;
                    in[u] = i < n_slots && filled(i);
                }
                if (!__any(in[0] || in[1] || in[2] || in[3])) continue;
#pragma unroll
                for (int u = 0; u < 4; ++u) ent[u] = in[u] ? list[i0 + u * NT] : 0ull;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (in[u]) f(i0 + u * NT, ent[u]);
            }
        };
        // Deeper lists that would fit the registers are put together in LDS first, each segment's entries behind those of the segments
        // before.  (Sparse ones: one or two KV heads, whose 1024 segments hold a few entries each, or the page index, where whole pages of
        // candidates fall into one segment.  Walked by slots for every purpose instead: one KV head, 16 query heads, 163k tokens
        // 48.5 us per call and 44.5 now, page index at 170k tokens 72.0 and 61.3.)
        const bool dense = n_slots > n_pre * NT && total <= (uint32_t)(PRE * NT) && total + in_b <= (uint32_t)EDGES;      // (uniform)
        if (__builtin_expect(dense, 0)) {
            uint32_t* const starts = reinterpret_cast<uint32_t*>(sm.keys);
            static_assert(sizeof(sm.keys) >= kMaxSeg * sizeof(uint32_t), "a word per segment");
            uint32_t start = before;
#pragma unroll
            for (int u = 0; u < SPT; ++u) { starts[u * NT + tid] = start; start += seg_len[u]; }
            __syncthreads();
            auto put = [&](int i, uint64_t ent) {
                const int run = i >> kCandChunkLog2;
                edge_lds[starts[run & (n_seg - 1)] + (uint32_t)(((run >> log2_n_seg) << kCandChunkLog2) | (i & (kCandChunk - 1)))] = ent;
            };
#pragma unroll
            for (int u = 0; u < PRE; ++u)
                if (u < n_pre && filled(u * NT + tid)) put(u * NT + tid, pre[u]);
            rest(put);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PRE; ++u) pre[u] = edge_lds[u * NT + tid < (int)total ? u * NT + tid : 0];
            n_pre = PRE;
            n_slots = ((int)total + kWave - 1) & ~(kWave - 1);
            edges_lds = edge_lds + total;
        }
        // (composite: score key, then inverted position: larger beats smaller, equal scores go to the lower position, no two are equal)
        auto edge = [&](uint32_t o, uint64_t ent) {
            if (o < in_b)                                 // (always)
                edges_lds[o] = ((uint64_t)score_key(score_of(ent)) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)ent);
        };
        uint32_t wins = 0, edges = 0;                     // bit u: pre[u] is a certain winner, an entry of bin B
        bool few = in_b <= (uint32_t)FEW;                 // (uniform) entries to rank, in whatever order they lie; more keep the list's
#pragma unroll
        for (int u = 0; u < PRE; ++u) {
            if (u < n_pre && u * NT < n_slots) {          // (uniform; n_slots is a multiple of 64, a segment's slots lie below it)
                const int bin = (dense ? u * NT + tid < (int)total : filled(u * NT + tid)) ? bin_of(pre[u]) : -1;
                wins |= bin > B ? 1u << u : 0u;
                edges |= bin == B ? 1u << u : 0u;
                if (few && bin == B) edge(atomicAdd(&n_edge_lds, 1u), pre[u]);
            }
        }
        // A crowded bin B is split into NB parts of its own range; S: the part the k-th score falls in, the parts above it win
        // too.  (Not the bins that are open to one side.  Nearly every call has a head with a few hundred entries in B; splitting them as
        // team_select() does costs 3 us more: d = 256, 29k tokens 52.8 us per call and 49.9 now, int8 index at 99k 50.0 and 47.1.)
        int S = -1;
        uint32_t sure = above, in_s = in_b;               // certain winners, entries that are left to rank
        auto part_of = [&](uint64_t ent) {                // (monotone: tail_bin() before its rounding to whole bins)
#pragma clang fp contract(off)
            const float t = __fmul_rn(__fsub_rn(score_of(ent), bin_lo), bin_inv) - (float)(B - 1);
            return (int)fminf(fmaxf(t * (float)NB, 0.f), (float)(NB - 1));
        };
        if (__builtin_expect(!few && B > 0 && B < kTailBins - 1, 0)) {         // (uniform)
            constexpr int BPT = NB / NT;
            auto place = [](int part) { return (part % BPT) * NT + part / BPT; };
#pragma unroll
            for (int u = 0; u < PRE; ++u)
                if (u * NT < n_slots && ((edges >> u) & 1u)) atomicAdd(&sm.hist[place(part_of(pre[u]))], 1u);
            rest([&](int, uint64_t ent) {
                if (bin_of(ent) == B) atomicAdd(&sm.hist[place(part_of(ent))], 1u);
            });
            __syncthreads();
            uint32_t n[BPT], local = 0, all_parts;
#pragma unroll
            for (int u = 0; u < BPT; ++u) { n[u] = sm.hist[place(NB - 1 - (tid * BPT + u))]; local += n[u]; }
            uint32_t run = above + team_prefix<Team>(local, all_parts, sm, 1);
#pragma unroll
            for (int u = 0; u < BPT; ++u) {
                if (run < (uint32_t)k_eff && (uint32_t)k_eff <= run + n[u]) {        // exactly one thread
                    sm.sel[0] = (uint32_t)(NB - 1 - (tid * BPT + u));
                    sm.sel[1] = run;
                    sm.sel[2] = n[u];
                }
                run += n[u];
            }
            __syncthreads();
            S = __builtin_amdgcn_readfirstlane((int)sm.sel[0]);
            sure = (uint32_t)__builtin_amdgcn_readfirstlane((int)sm.sel[1]);
            in_s = (uint32_t)__builtin_amdgcn_readfirstlane((int)sm.sel[2]);
            few = in_s <= (uint32_t)FEW;
#pragma unroll
            for (int u = 0; u < PRE; ++u) {
                if (u * NT < n_slots && ((edges >> u) & 1u)) {
                    const int part = part_of(pre[u]);
                    if (part > S) wins |= 1u << u;
                    if (part != S) edges &= ~(1u << u);
                    else if (few) edge(atomicAdd(&n_edge_lds, 1u), pre[u]);
                }
            }
        }
        auto wins_for_certain = [&](uint64_t ent) { return bin_of(ent) > B || (S >= 0 && bin_of(ent) == B && part_of(ent) > S); };
        auto is_edge = [&](uint64_t ent) { return bin_of(ent) == B && (S < 0 || part_of(ent) == S); };
        uint32_t n_win = (uint32_t)__popc(wins), n_edges = (uint32_t)__popc(edges);
        rest([&](int, uint64_t ent) {
            const bool e = is_edge(ent);
            n_win += wins_for_certain(ent) ? 1u : 0u;
            n_edges += e ? 1u : 0u;
            if (few && e) edge(atomicAdd(&n_edge_lds, 1u), ent);
        });
        uint32_t all_wins;                                // (`sure` of them)
        uint32_t at = team_prefix<Team>(n_win, all_wins, sm, 0);
        if (__ballot(at < row1 && at + n_win > row0)) {   // (the places of a wave's winners follow one another)
#pragma unroll
            for (int u = 0; u < PRE; ++u)
                if (u * NT < n_slots && ((wins >> u) & 1u)) emit(at++, score_of(pre[u]), (uint32_t)pre[u]);
            rest([&](int, uint64_t ent) {
                if (wins_for_certain(ent)) emit(at++, score_of(ent), (uint32_t)ent);
            });
        }
        // the best entries of the bin are the missing winners
        const uint32_t need = (uint32_t)k_eff - sure;
        const int n_edge = (int)(in_s < (uint32_t)EDGES ? in_s : (uint32_t)EDGES);
        auto edge_score = [&](uint64_t key) { return key_score((uint32_t)(key >> 32)); };
        auto edge_pos = [&](uint64_t key) { return 0xFFFFFFFFu - (uint32_t)key; };
        if (row1 <= sure) {                               // (uniform) none of the missing winners is in this workgroup's shares
        } else if (few) {                                 // each against all others, LP lanes per entry
            constexpr int LP = NT / FEW;
            static_assert(LP == 2 || LP == 4, "a pair or a quad of lanes");
            const int j = tid / LP;
            const uint64_t mine = edges_lds[j < n_edge ? j : 0];
            uint32_t rank = 0;
            if (j < n_edge) {
#pragma unroll 8
                for (int o = tid % LP; o < n_edge; o += LP) rank += edges_lds[o] > mine ? 1u : 0u;
            }
            rank += dpp_u32<0xB1, 0xF>(0u, rank);         // quad_perm 1,0,3,2
            if (LP == 4) rank += dpp_u32<0x4E, 0xF>(0u, rank);       // quad_perm 2,3,0,1
            if (j < n_edge && tid % LP == 0 && rank < need) emit(sure + rank, edge_score(mine), edge_pos(mine));
        } else {
            constexpr int CPT = EDGES / NT;
            uint32_t all_edges, to = team_prefix<Team>(n_edges, all_edges, sm, 1);
#pragma unroll
            for (int u = 0; u < PRE; ++u)
                if (u * NT < n_slots && ((edges >> u) & 1u)) edge(to++, pre[u]);
            rest([&](int, uint64_t ent) {
                if (is_edge(ent)) edge(to++, ent);
            });
            __syncthreads();
            uint32_t act = 0;
            float lo = INFINITY, hi = -INFINITY;
#pragma unroll 1
            for (int j = 0; j < CPT; ++j) {
                if (j * NT + tid < n_edge) {
                    const float s = edge_score(edges_lds[j * NT + tid]);
                    act |= 1u << j;
                    lo = fminf(lo, s); hi = fmaxf(hi, s);
                }
            }
            select_clear<Team>(sm);
            team_range<Team>(lo, hi, sm, 0);
            team_select<Team, CPT, 1>([&](int j) { return edge_score(edges_lds[j * NT + tid]); }, act, n_edge, P, (int)need, lo, hi, sm,
                                      [&](int j) { return (int32_t)edge_pos(edges_lds[j * NT + tid]); },
                                      [&](uint32_t o, float s, int32_t p) { emit(sure + o, s, (uint32_t)p); });
        }
        if (writer) pad_outputs(k_eff, k, idx, vals);
    } else if (k_eff == 0) {
        if (writer) pad_outputs(0, k, idx, vals);
    } else {                                              // radix select over the list or the full score row
        __shared__ SelShared sel_sm;
        if (how == SCORE_ROW) {
            top = key_score(wg_select_dense<NT, 0>(sh, bf, bh, P, k_eff, k, idx, vals, sel_sm));      // writes idx, vals and their padding
        } else {
            const SrcSegments<NT> src{list, segs, n_slots, log2_n_seg};
            const Items<0, SrcSegments<NT>> items(src);
            top = key_score(wg_topk_emit(items, k_eff, k, idx, vals, sel_sm));
        }
        M = fmaxf(top, w_top);
        __syncthreads();
        for (int o = tid; o < k_eff; o += NT) rows_lds[o] = ((uint64_t)__float_as_uint(vals[o]) << 32) | (uint64_t)(uint32_t)idx[o];
    }
    if (tid == 0 && writer) {                             // the head's record (of a list taken as it is: all winners found, the size of bin B)
        uint32_t* const rec = bf.tailrec + 4 * bh;
        const bool sel = how != SCORE_ROW && k_eff > 0, found = how == LIST;
        rec[0] = k_eff == 0 ? 2u : sel ? 0u : 1u;
        rec[1] = sel ? (found ? (uint32_t)k_eff : above) : 0u;
        rec[2] = sel && !found ? (uint32_t)k_eff - above : 0u;
        rec[3] = sel ? in_b : 0u;
    }
    __syncthreads();
    if (k_eff > 0 && (how == LIST || how == RESCORE)) {   // (the radix select has written its winners)
        const uint32_t sel_end = row1 < (uint32_t)k_eff ? row1 : (uint32_t)k_eff;
        for (uint32_t o = row0 + (uint32_t)tid; o < sel_end; o += NT) {
            idx[o] = (int32_t)(uint32_t)rows_lds[o];
            vals[o] = score_of(rows_lds[o]);
        }
    }

    // ---- the weighted value rows (of this workgroup's shares, one after the other)
    const char* const Vh = static_cast<const char*>(bf.V) + head_off;
    float* const pa = bf.part_acc + bh * sh.n_chunk_cap * (int64_t)D;
    float* const pl = bf.part_l + bh * sh.n_chunk_cap;
    float a = 0.f, l = 0.f;                               // thread t < D: channel t (D <= NT)
    // Leave a share where the head's other workgroups see it (agent-scope stores go through to memory, and the wait
    // below is for their arrival there), count it, and let the last workgroup add up all shares in their order.
    // No release or acquire fence: those write back and invalidate the whole L2 of the XCD, and nothing
    // but these values passes between the workgroups.  (A workgroup that takes all shares adds them up as it goes.)
    auto leave = [&](int share, float as, float ls) {
        if (share_wgs > 1) {
            if (tid < D) __hip_atomic_store(pa + share * D + tid, as, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (tid == 0) __hip_atomic_store(pl + share, ls, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            a += as; l += ls;
        }
    };
    constexpr int STEP = NW * RPW, SU = 2;
    if (share1 - share0 > 1 && NT == 1024 && n_rows <= SU * STEP * shares) {       // (uniform)
        // several short shares: the rows of all of them are asked for before the first is added up (one after the other, each
        // share was a trip to memory: 8 shares of 96 rows on each of 256 heads 38 us for the kernel, 29 like this; two rows a lane and
        // share are what the registers hold)
        const int rs = lane / LPR, c = lane % LPR;
        u32x4 raw[kAttendShares][SU];
        float w[kAttendShares][SU];
#pragma unroll
        for (int s = 0; s < kAttendShares; ++s) {
            const int first = share_row(share0 + s), end = share0 + s < share1 ? share_row(share0 + s + 1) : first;
            if (first < end) {                            // (uniform)
#pragma unroll
                for (int u = 0; u < SU; ++u) {
                    const int j = first + u * STEP + wave * RPW + rs;
                    // (a lane past the end takes the share's first row with weight 0: a selected row, so a value that is not finite
                    // counts only where it would count anyway)
                    const uint64_t e = rows_lds[j < end ? j : first];
                    w[s][u] = j < end ? exp2f((score_of(e) - M) * scale_log2e) : 0.f;
                    const uint32_t p = (uint32_t)e < (uint32_t)N ? (uint32_t)e : (uint32_t)(N - 1);     // (always below N)
                    raw[s][u] = *reinterpret_cast<const u32x4*>(Vh + ((int64_t)p * D + c * EPL) * 2);
                }
            } else {
#pragma unroll
                for (int u = 0; u < SU; ++u) { w[s][u] = 0.f; raw[s][u] = u32x4{0u, 0u, 0u, 0u}; }
            }
        }
#pragma unroll
        for (int s = 0; s < kAttendShares; ++s) {
            if (share0 + s < share1) {                    // (uniform)
                // (two places in turn: a share is written while the one before it is read)
                float (*const part)[256 + 1] = acc_lds + (s & 1) * NW;
                float acc[EPL];
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
                float lsum = 0.f;
#pragma unroll
                for (int u = 0; u < SU; ++u) {
                    float vf[EPL];
                    Elem<DT>::widen(raw[s][u], vf);
#pragma unroll
                    for (int e = 0; e < EPL; ++e) acc[e] = fmaf(w[s][u], vf[e], acc[e]);
                    lsum += w[s][u];
                }
                lane_group_sums(LPR, acc, lsum);
                if (rs == 0) {
#pragma unroll
                    for (int e = 0; e < EPL; ++e) part[wave][c * EPL + e] = acc[e];
                    if (c == 0) part[wave][256] = lsum;
                }
                __syncthreads();
                float as = 0.f, ls = 0.f;
                if (tid < D) {
#pragma unroll
                    for (int v = 0; v < NW; ++v) { as += part[v][tid]; ls += part[v][256]; }
                }
                leave(share0 + s, as, ls);
            }
        }
    } else {
        for (int share = share0; share < share1; ++share) {   // (uniform)
            float as, ls;
            weighted_rows<DT, NT, 8>(Vh, D, N, rows_lds, share_row(share), share_row(share + 1), M, scale_log2e, acc_lds, as, ls);
            leave(share, as, ls);
            if (share + 1 < share1) __syncthreads();      // (the partial sums are written again)
        }
    }
    if (share_wgs > 1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0)
            sm.n_keys = __hip_atomic_fetch_add(&bf.flags[bh], kArrivalUnit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) / kArrivalUnit;
        __syncthreads();
        if (sm.n_keys + 1u != (uint32_t)share_wgs) return;   // (uniform)
        a = 0.f; l = 0.f;
        if (tid < D) {
            float ta[kAttendShares], tl[kAttendShares];
#pragma unroll
            for (int s = 0; s < kAttendShares; ++s) {
                ta[s] = s < shares ? __hip_atomic_load(pa + s * D + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.f;
                tl[s] = s < shares ? __hip_atomic_load(pl + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.f;
            }
#pragma unroll
            for (int s = 0; s < kAttendShares; ++s) { a += ta[s]; l += tl[s]; }
        }
    }
    if (tid < D) {
        bf.out[bh * D + tid] = a / l;
        if (tid == 0 && bf.lse) bf.lse[bh] = M * scale + logf(l);
    }
}

// Batches of short sequences: scores, selection and attention of a KV head's query heads in one launch, a workgroup per key
// stream.  The four waves score the stream's tiles with the scan's routines and leave the scores in LDS (and their range);
// then each wave selects for one head of the group and fetches its rows, with no barrier between the waves.  Two or more workgroups
// per compute unit, each in a phase of its own, keep the keys coming while others select, if selecting is not what takes
// longest: a wave that branches over each of its 64 scores a lane waits for LDS every time (about 50 us for 4096 scores, against 33
// for the keys), so winners and ties are counted and placed without a branch, the weights follow for 64 winners at a time,
// and twice the rows are in flight.  ROW: scores of the longest sequence.  192 sequences of 2048 .. 4096 tokens, k = 128 (1.2 GB of
// keys, 0.2 GB of value rows): scan with stored scores, radix select and gather 277 + 70 + 42 us, first version of this kernel
// 310, now 295.  (One workgroup per compute unit whose waves score one stream while others select for the one before: 371.)
constexpr int kShortBins = 256;
template <int DT, int D, int ROW>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
attend_short_kernel(Shape sh, Bufs bf, float scale, float scale_log2e) {
    using v8 = typename Mfma<DT>::v8;
    constexpr int CPT = ROW / kWave, ROWS = attend_short_k(ROW), EPL = 8, LPR = D / EPL, RPW = kWave / LPR;
    constexpr int NB = kShortBins, BPT = NB / kWave;
    using Mask = typename std::conditional<(CPT > 32), uint64_t, uint32_t>::type;
    __shared__ __align__(16) float scores_lds[4][ROW];
    __shared__ uint64_t rows_all_lds[4][ROWS];            // winners (score bits, position), then rows to fetch (weight bits, position)
    __shared__ SelectShared<WaveTeam, NB> sms[4];
    __shared__ float range_lds[2][4][4];                  // smallest and largest score of each head, per wave
    const int kvh = blockIdx.x, b = (int)blockIdx.y + (int)blockIdx.z * sh.layer_seqs, G = sh.G;
    const int64_t head0 = (int64_t)b * sh.Hq + (int64_t)kvh * G;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int N = bf.len[b];                              // (no window on this path)
    const char* const Kh = static_cast<const char*>(bf.K) + ((int64_t)b * sh.Hkv + kvh) * sh.Ncap * (D * 2);
    {
        v8 qa[D / 32];
        load_query_a<DT, D>(bf.q, head0, G, qa);
        struct TileB { v8 b[4][D / 32]; } ba, bb;
        float lo4[4], hi4[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) { lo4[r] = INFINITY; hi4[r] = -INFINITY; }
        auto use = [&](TileB& t, int64_t ti) {
            const f32x4 res = tile_mac<DT, D>(t.b, qa);
            const int item = (int)ti * 64 + lane;
            if (item < N) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float s = res[r] + 0.0f;        // -0 counts as +0
                    lo4[r] = fminf(lo4[r], s); hi4[r] = fmaxf(hi4[r], s);
                    if (r < G) scores_lds[r][item] = s;
                }
            }
        };
        const LaneOffsets lane_off = lane_offsets<D>();
        walk_tiles<ScanPipelined<D>::value>(wave, (N + 63) / 64, 4, ba, bb,
            [&](TileB& t, int64_t ti) { tile_load_at<DT, D>(Kh, ti, N, lane_off, t.b); }, use);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float lo = wave_min(lo4[r]), hi = wave_max(hi4[r]);
            if (lane == 0) { range_lds[0][r][wave] = lo; range_lds[1][r][wave] = hi; }
        }
    }
    SelectShared<WaveTeam, NB>& sm = sms[wave];
    select_clear<WaveTeam>(sm);
    __syncthreads();
    if (wave >= G) return;                                // (no barrier of the workgroup follows)

    const int64_t bh = head0 + wave;
    const LayerK lk = bf.layer_k[blockIdx.z];
    const int k = lk.k, k_eff = k < N ? k : N;
    const int64_t sel0 = selection_at(sh, lk, blockIdx.y, kvh * G + wave);
    int32_t* const idx = bf.sel_idx + sel0;
    float* const vals = bf.sel_val + sel0;
    // (64 scores of a lane in registers spilled: they stay in LDS, eight reads in flight)
    const float* const row = scores_lds[wave] + lane;
    const float* const lo4 = range_lds[0][wave];
    const float* const hi4 = range_lds[1][wave];
    const float lo = fminf(fminf(lo4[0], lo4[1]), fminf(lo4[2], lo4[3])), hi = fmaxf(fmaxf(hi4[0], hi4[1]), fmaxf(hi4[2], hi4[3]));
    const float M = hi;                                   // the weights' reference score
    uint64_t* const rows = rows_all_lds[wave];
    // ---- the k_eff best: linear bins between the smallest and the largest score, as team_select()'s first step
    const float inv = (float)NB / (hi - lo);
    bool done = hi > lo && hi - lo < INFINITY && inv < INFINITY;         // (uniform)
    if (done) {
        auto place = [](int bin) { return (bin % BPT) * kWave + bin / BPT; };
        const int n_full = N / kWave;                     // slots that every lane has
#pragma unroll 8
        for (int j = 0; j < n_full; ++j) atomicAdd(&sm.hist[place(lin_bin<NB>(row[j * kWave], lo, inv))], 1u);
        if (n_full * kWave + lane < N) atomicAdd(&sm.hist[place(lin_bin<NB>(row[n_full * kWave], lo, inv))], 1u);
        wave_sync();
        uint32_t n[BPT], local = 0, total;
#pragma unroll
        for (int u = 0; u < BPT; ++u) { n[u] = sm.hist[place(NB - 1 - (lane * BPT + u))]; local += n[u]; }
        uint32_t run = team_prefix<WaveTeam>(local, total, sm, 1);
#pragma unroll
        for (int u = 0; u < BPT; ++u) {
            if (run < (uint32_t)k_eff && (uint32_t)k_eff <= run + n[u]) {        // exactly one lane
                sm.sel[0] = (uint32_t)(NB - 1 - (lane * BPT + u));
                sm.sel[1] = run;
                sm.sel[2] = n[u];
            }
            run += n[u];
        }
        wave_sync();
        const int B = (int)sm.sel[0], n_in = (int)sm.sel[2];
        const uint32_t above = sm.sel[1];
        done = n_in <= kWave;                             // more are split again (team_select() below)
        if (done) {
            // per lane: certain winners, and scores of bin B (upper half); then their places
            uint32_t cnt = 0;
            auto count = [&](int j) {
                const int bin = lin_bin<NB>(row[j * kWave], lo, inv);
                return (bin > B ? 1u : 0u) + (bin == B ? 0x10000u : 0u);
            };
#pragma unroll 8
            for (int j = 0; j < n_full; ++j) cnt += count(j);
            if (n_full * kWave + lane < N) cnt += count(n_full);
            uint32_t at = team_prefix<WaveTeam>(cnt, total, sm, 0);      // (at most 4096 winners: the halves do not meet)
            uint64_t* const keys = sm.keys;
            uint64_t* const nowhere = reinterpret_cast<uint64_t*>(sm.hist) + lane;       // (the counts are not needed any more)
            static_assert(NB * sizeof(uint32_t) >= kWave * sizeof(uint64_t), "a place per lane");
            auto put = [&](int j) {
                const float s = row[j * kWave];
                const int bin = lin_bin<NB>(s, lo, inv);
                const uint32_t p = (uint32_t)(j * kWave + lane);
                const bool win = bin > B, edge = bin == B;
                uint64_t* to = win ? rows + (at & 0xFFFFu) : edge ? keys + (at >> 16) : nowhere;
                // a score of bin B: its composite key (larger beats smaller, equal scores go to the lower position)
                *to = win ? ((uint64_t)__float_as_uint(s) << 32) | (uint64_t)p : ((uint64_t)score_key(s) << 32) | (uint64_t)(0xFFFFFFFFu - p);
                at += (win ? 1u : 0u) + (edge ? 0x10000u : 0u);
            };
#pragma unroll 8
            for (int j = 0; j < n_full; ++j) put(j);
            if (n_full * kWave + lane < N) put(n_full);
            const int n8 = (n_in + 7) & ~7;
            if (lane < n8 - n_in) keys[n_in + lane] = 0ull;              // beats nothing
            wave_sync();
            if (lane < n_in) {
                const uint64_t mine[1] = {keys[lane]};
                uint32_t rank[1];
                rank_by_comparison<1>(keys, n8, mine, rank);
                if (above + rank[0] < (uint32_t)k_eff)
                    rows[above + rank[0]] = ((uint64_t)__float_as_uint(key_score((uint32_t)(mine[0] >> 32))) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)mine[0]);
            }
        } else {
            select_clear<WaveTeam>(sm);
            wave_sync();
        }
    }
    if (!done) {                                          // (uniform) equal or crowded scores, or a range beyond fp32
        Mask act = 0;
        for (int j = 0; j < CPT; ++j) act |= j * kWave + lane < N ? (Mask)1 << j : (Mask)0;
        team_select<WaveTeam, CPT, 1>([&](int j) { return row[j * kWave]; }, act, N, N, k_eff, lo, hi, sm,
                                      [&](int j) { return j * kWave + lane; }, [&](uint32_t o, float s, int32_t p) {
            if (o < (uint32_t)k_eff)                      // always true; guards the buffer
                rows[o] = ((uint64_t)__float_as_uint(s) << 32) | (uint64_t)(uint32_t)p;
        });
    }
    wave_sync();
    for (int o = lane; o < k; o += kWave) {
        const bool in = o < k_eff;
        const uint64_t e = in ? rows[o] : 0ull;
        const float s = __uint_as_float((uint32_t)(e >> 32));
        idx[o] = in ? (int32_t)(uint32_t)e : -1;
        vals[o] = in ? s : -INFINITY;
        if (in) rows[o] = ((uint64_t)__float_as_uint(exp2f((s - M) * scale_log2e)) << 32) | (uint64_t)(uint32_t)e;
    }
    wave_sync();

    const char* const Vh = static_cast<const char*>(bf.V) + ((int64_t)b * sh.Hkv + kvh) * sh.Ncap * (D * 2);
    const int rs = lane / LPR, c = lane % LPR;
    float acc[EPL], l = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
    // as many rows in flight per lane group as there are, sixteen at most
    auto fetch = [&](auto u_tag) __attribute__((always_inline)) {
        constexpr int U = decltype(u_tag)::value;
        for (int j = rs; j < k_eff; j += U * RPW) {
            float w[U];
            u32x4 raw[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint64_t e = rows[j + u * RPW < k_eff ? j + u * RPW : j];
                w[u] = j + u * RPW < k_eff ? __uint_as_float((uint32_t)(e >> 32)) : 0.f;
                const uint32_t p = (uint32_t)e < (uint32_t)N ? (uint32_t)e : (uint32_t)(N - 1);     // (always below N)
                raw[u] = *reinterpret_cast<const u32x4*>(Vh + ((int64_t)p * D + c * EPL) * 2);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float vf[EPL];
                Elem<DT>::widen(raw[u], vf);
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[e] = fmaf(w[u], vf[e], acc[e]);
                l += w[u];
            }
        }
    };
    if (k_eff <= 4 * RPW) fetch(std::integral_constant<int, 4>{});
    else if (k_eff <= 8 * RPW) fetch(std::integral_constant<int, 8>{});
    else fetch(std::integral_constant<int, 16>{});
#pragma unroll
    for (int o = LPR; o < kWave; o <<= 1) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = o == 32 ? add_lanes_32(acc[e]) : o == 16 ? add_lanes_16(acc[e]) : acc[e] + wave_xor(acc[e], o);
        l = o == 32 ? add_lanes_32(l) : o == 16 ? add_lanes_16(l) : l + wave_xor(l, o);
    }
    if (rs == 0) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) bf.out[bh * D + c * EPL + e] = acc[e] / l;
    }
    if (lane == 0 && bf.lse) bf.lse[bh] = M * scale + logf(l);
}

hipError_t launch_attend_short(const Shape& s, const Bufs& b, int64_t Nmax, hipStream_t st) {
    const float scale = 1.0f / sqrtf((float)s.D);
    const float scale_log2e = scale * 1.4426950408889634f;
    const dim3 grid((unsigned)s.Hkv, (unsigned)s.layer_seqs, 1u << s.log2_layers);
    if (s.M != 1 || s.G > 4 || s.window || s.k > attend_short_k(Nmax)) return hipErrorInvalidValue;
#define TKA_AS(DT_, D_, ROW_) hipLaunchKernelGGL((attend_short_kernel<DT_, D_, ROW_>), grid, dim3(256), 0, st, s, b, scale, scale_log2e)
#define TKA_AS_ROW(DT_, D_)                           \
    do {                                              \
        if (Nmax <= 1024) TKA_AS(DT_, D_, 1024);      \
        else if (Nmax <= 2048) TKA_AS(DT_, D_, 2048); \
        else TKA_AS(DT_, D_, 4096);                   \
    } while (0)
    if (s.dtype == DT_F16 && s.D == 128) TKA_AS_ROW(DT_F16, 128);
    else if (s.dtype == DT_BF16 && s.D == 128) TKA_AS_ROW(DT_BF16, 128);
    else if (s.dtype == DT_F16 && s.D == 64) TKA_AS_ROW(DT_F16, 64);
    else if (s.dtype == DT_BF16 && s.D == 64) TKA_AS_ROW(DT_BF16, 64);
    else if (s.dtype == DT_F16 && s.D == 256) TKA_AS_ROW(DT_F16, 256);
    else if (s.dtype == DT_BF16 && s.D == 256) TKA_AS_ROW(DT_BF16, 256);
    else if (s.dtype == DT_F16 && s.D == 32) TKA_AS_ROW(DT_F16, 32);
    else if (s.dtype == DT_BF16 && s.D == 32) TKA_AS_ROW(DT_BF16, 32);
    else return hipErrorInvalidValue;
#undef TKA_AS_ROW
#undef TKA_AS
    return hipGetLastError();
}

hipError_t launch_attend_row(const Shape& s, const Bufs& b, int64_t Nmax, hipStream_t st) {
    const float scale = 1.0f / sqrtf((float)s.D);
    const float scale_log2e = scale * 1.4426950408889634f;
    const dim3 grid((unsigned)s.Hq, (unsigned)s.layer_seqs, 1u << s.log2_layers);
    // (more heads than compute units, rows of up to 8192 scores: workgroups no larger than the row needs take 0.49 - 0.99 of the time
    // of 1024 threads, median 0.81, over 320 to 1920 heads)
    // (the heads of a layer: a call over several layers gives what a call per layer gives)
    const int64_t heads = (int64_t)s.Hq * s.layer_seqs;
    if ((int64_t)s.k + s.window > attend_row_rows(heads, Nmax)) return hipErrorInvalidValue;
#define TKA_AR(DT_, NT_, CPT_, NB_)                                                                                         \
    hipLaunchKernelGGL((attend_kernel<DT_, AttendCfg<NT_, CPT_, NT_ == 1024 ? 4096 : NT_ == 512 ? 2048 : 1024, NB_>>), \
                       grid, dim3(NT_), 0, st, s, b, scale, scale_log2e)
#define TKA_AR_SIZE(DT_)                                     \
    do {                                                     \
        switch (attend_row_class(heads, Nmax)) {             \
            case 0: TKA_AR(DT_, 256, 8, 512); break;         \
            case 1: TKA_AR(DT_, 256, 16, 512); break;        \
            case 2: TKA_AR(DT_, 512, 16, 512); break;        \
            case 3: TKA_AR(DT_, 1024, 4, 1024); break;       \
            default: TKA_AR(DT_, 1024, 16, 1024);            \
        }                                                    \
    } while (0)
    if (s.dtype == DT_F32) TKA_AR_SIZE(DT_F32);
    else if (s.dtype == DT_F16) TKA_AR_SIZE(DT_F16);
    else TKA_AR_SIZE(DT_BF16);
#undef TKA_AR_SIZE
#undef TKA_AR
    return hipGetLastError();
}

hipError_t launch_attend_list(const Shape& s, const Bufs& b, hipStream_t st) {
    const float scale = 1.0f / sqrtf((float)s.D);
    const float scale_log2e = scale * 1.4426950408889634f;
    // as many helpers as fit the compute units beside the shares, a wave of theirs per segment at most
    const int64_t heads = (int64_t)s.Hq * s.B, room = std::min<int64_t>(kAttendManyHeads / heads, s.n_seg / (1024 / kWave));
    const dim3 grid((unsigned)s.Hq, (unsigned)s.layer_seqs, (unsigned)std::max<int64_t>(s.share_wgs, room) << s.log2_layers);
    const bool two_per_cu = heads * s.share_wgs > kAttendManyHeads;
#define TKA_AL(DT_, D_)                                                                                                                 \
    do {                                                                                                                                \
        if (two_per_cu) hipLaunchKernelGGL((attend_list_kernel<DT_, 512, D_>), grid, dim3(512), 0, st, s, b, scale, scale_log2e);       \
        else hipLaunchKernelGGL((attend_list_kernel<DT_, 1024, D_>), grid, dim3(1024), 0, st, s, b, scale, scale_log2e);                \
    } while (0)
    if (s.dtype == DT_F16 && s.D == 128) TKA_AL(DT_F16, 128);
    else if (s.dtype == DT_BF16 && s.D == 128) TKA_AL(DT_BF16, 128);
    else if (s.dtype == DT_F16 && s.D == 64) TKA_AL(DT_F16, 64);
    else if (s.dtype == DT_BF16 && s.D == 64) TKA_AL(DT_BF16, 64);
    else if (s.dtype == DT_F16 && s.D == 256) TKA_AL(DT_F16, 256);
    else if (s.dtype == DT_BF16 && s.D == 256) TKA_AL(DT_BF16, 256);
    else if (s.dtype == DT_F16 && s.D == 32) TKA_AL(DT_F16, 32);
    else if (s.dtype == DT_BF16 && s.D == 32) TKA_AL(DT_BF16, 32);
    else return hipErrorInvalidValue;
#undef TKA_AL
    return hipGetLastError();
}

}  // namespace tka

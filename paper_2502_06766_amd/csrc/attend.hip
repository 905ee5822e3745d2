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
// What bounds it: instructions and barriers of one compute unit per head (a stamp per phase: loads 1.5-3 us, bins and
// their prefix sum 1.6, ranking and emission 2, rows 1.5-2, sum and write 1.5), so scores stay in registers with
// slots nobody uses skipped uniformly (the same phases as rolled loops over LDS: 23.6 us against 14.5 at 16k
// tokens) and scans and reductions run in the vector unit instead of trips through LDS.  Measured, 32 heads, 8 KV heads:
// a row of 16k scores, k = 256: 14.5 us (radix select + gather before: 18.7 + 7.9); a list at 48k tokens, k = 768:
// 13.9 us, at 128k tokens, k = 1800: 18.0 us (chip-wide tail: 11.6 + 11.6 and 14.8 + 9.6 us and a launch more).
//
//   SRC_ROW   the scores of a short cache, stored by the scan (general path)
//   (attend_short_kernel: the scores too, for batches of short sequences)
//   SRC_LIST  the candidate list the filtered scan left; a head whose list is unusable (a segment overflowed, too few
//             or too many candidates) is scored again by the workgroups launched for it and selected from its full
//             score row by the last of them to finish
#include <type_traits>

#include "device_utils.h"
#include "internal.h"
#include "scan_tiles.h"
#include "select_common.h"
#include "team.h"

namespace tka {

enum { SRC_ROW = 0, SRC_LIST = 1 };

// NT threads with CPT scores each in registers; ROWS: value rows whose positions and weights fit LDS; NB: bins.
template <int NT_, int CPT_, int ROWS_, int NB_>
struct AttendCfg {
    static constexpr int NT = NT_, CPT = CPT_, ROWS = ROWS_, NB = NB_, NW = NT_ / kWave;
    static_assert(NB % NT == 0 && NT % kWave == 0 && NW <= 16 && CPT <= 32, "whole bins per thread, a bit per score, a lane per wave");
};
using ListCfg = AttendCfg<1024, kAttendList / 1024, kAttendRows, 1024>;

// What a team shares while it selects; NB bins.
template <class Team, int NB_>
struct SelectShared {
    static constexpr int NB = NB_;
    uint64_t keys[Team::NT + 8];            // segments of the candidate list (length, first entry); later composite keys of the bin that is ranked
    uint32_t hist[NB_];
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
        const bool last = in <= (uint32_t)NT || it == 63;
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

// Exact scores of the head's keys into the score buffer, the tiles `first`, `first + step`, ... of 16 keys, one per wave
// and step (a head whose candidate list is unusable; the arithmetic of the scan).
template <int DT, int D>
__device__ __forceinline__ void score_keys(const Shape& sh, const Bufs& bf, int b, int h, int64_t N, int64_t first, int64_t step) {
    using v8 = typename Mfma<DT>::v8;
    const int64_t bh = (int64_t)b * sh.Hq + h;
    const int lane = lane_id(), jj = lane >> 4, n = lane & 15;
    const char* Kh = static_cast<const char*>(bf.K) + ((int64_t)cache_seq(sh, b) * sh.Hkv + h / sh.G) * sh.Ncap * (D * 2);
    // operand A holds this head alone (rows 0, 4, 8, 12), so that accumulator element 0 is its score in every lane
    v8 qa[D / 32];
    load_query_a<DT, D>(bf.q, bh, 1, qa);
    for (int64_t t = first; t * 16 < N; t += step) {
        const int64_t key = t * 16 + n;
        const v8* p = reinterpret_cast<const v8*>(Kh + (key < N ? key : N - 1) * (D * 2)) + jj;
        v8 kb[D / 32];
#pragma unroll
        for (int s = 0; s < D / 32; ++s) kb[s] = p[4 * s];
        f32x4 c = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < D / 32; ++s) c = Mfma<DT>::mac(qa[s], kb[s], c);
        if (jj == 0 && key < N) bf.scores[bh * sh.Ncap + key] = c[0] + 0.0f;
    }
}

// Grid: heads x sequences x shares.  SRC_LIST: the gridDim.z workgroups of a head all select from its list (the same
// winners, found side by side on compute units that would idle), each fetches its share of the value rows, and the last
// to finish adds up the shares; so a head's rows are not bound by what one compute unit can fetch (about 64 GB/s).
template <int DT, class Cfg, int SRC>
__global__ void __launch_bounds__(Cfg::NT) __attribute__((amdgpu_waves_per_eu(4))) attend_kernel(Shape sh, Bufs bf, float scale, float scale_log2e) {
    constexpr int NT = Cfg::NT, NW = Cfg::NW, CPT = Cfg::CPT;
    using Team = WorkgroupTeam<NT>;
    constexpr int EPL = Elem<DT>::kPerLoad;
    constexpr int U = 8;                                  // value rows in flight per lane group
    __shared__ SelectShared<Team, Cfg::NB> sm;
    __shared__ uint64_t cand_lds[SRC == SRC_LIST ? CPT * NT : 1];      // candidates (score bits, position)
    __shared__ uint64_t rows_lds[Cfg::ROWS];              // value rows to fetch (weight bits, position)
    __shared__ float acc_lds[NW][256 + 1];
    const int b = blockIdx.y, h = blockIdx.x;
    const int64_t bh = (int64_t)b * sh.Hq + h;
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int32_t* const idx = bf.sel_idx + bh * sh.k;
    float* const vals = bf.sel_val + bh * sh.k;
    const int D = sh.D, lpr = D / EPL, rpw = kWave / lpr;          // lanes per key or value row, rows per wave and load
    const int rs = lane / lpr, c = lane % lpr;
    const int64_t head_off = ((int64_t)cache_seq(sh, b) * sh.Hkv + h / sh.G) * sh.Ncap * D * Elem<DT>::kBytes;

    // ---- the scores to select from, in registers: slot j of a thread holds item j * NT + tid
    float v[CPT];
    int n_items = 0;
    uint32_t act = 0;                                     // bit j: v[j] is a score in question
    bool usable = true;                                   // (uniform) there is a list
    constexpr int PRE = 12;                               // list slots per thread asked for before the segments' lengths are known
    uint64_t pre[SRC == SRC_LIST ? PRE : 1];
    const uint64_t* const list = bf.cand + bh * (int64_t)sh.cand_cap;
    uint32_t seg_len = 0, flags = 0;
    if (SRC == SRC_LIST) {
        if (tid < sh.n_seg) seg_len = bf.seg_cnt[bh * sh.n_seg + tid];
        flags = bf.flags[bh];
#pragma unroll
        for (int u = 0; u < PRE; ++u) {
            const int i = u * NT + tid;
            pre[u] = list[i < sh.cand_cap ? i : 0];       // (any slot of the list may be read; what lies beyond its segment is ignored)
        }
    }
    const int N = (int)visible_len(sh, bf, b);
    const int P = (int)prefix_len(N, sh.window), W = N - P;      // searched prefix, window
    const int k_eff = sh.k < P ? sh.k : P;
    const float* const row = bf.scores + bh * sh.Ncap;
    auto pos = [&](int j) { return SRC == SRC_LIST ? (int32_t)(uint32_t)cand_lds[j * NT + tid] : j * NT + tid; };
    float lo = INFINITY, hi = -INFINITY;                  // range of the scores in question
    if (SRC == SRC_ROW) {
        n_items = P;
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
            const int i = j * NT + tid;
            v[j] = row[i < P ? i : 0];                    // (P == 0: the window's scores are there)
            act |= i < P ? 1u << j : 0u;
        }
    } else if (k_eff > 0) {
        // lengths and places of the segments; the list is usable if it holds all that passed, at least k_eff and not more than fits
        uint32_t total;
        const uint32_t longest_w = wave_max_u32(seg_len);
        if (lane == 0) sm.hist[wave] = longest_w;
        const uint32_t at = team_prefix<Team>(seg_len, total, sm, 0);
        uint2* const segs = reinterpret_cast<uint2*>(sm.keys);
        segs[tid] = make_uint2(seg_len, at);
        const uint32_t longest = wave_max_u32(lane < NW ? sm.hist[lane] : 0u);
        const bool over = longest > (uint32_t)sh.seg_cap || total < (uint32_t)k_eff;
        // (an index leaves the approximate scores of a head it marked as not filterable)
        usable = !over && total <= (uint32_t)(CPT * NT) && !(flags & (sh.indexed ? 5u : 4u));
        if (usable) {
            n_items = (int)total;
            const int log2_n_seg = 31 - __clz(sh.n_seg);
            const int n_slots = (int)((longest + kCandChunk - 1) >> kCandChunkLog2) * sh.n_seg * kCandChunk;
            auto place = [&](int i, uint64_t ent) {       // slot i of the list: entry e of segment g
                const uint2 s = segs[cand_slot_segment(i, log2_n_seg)];
                const uint32_t e = (uint32_t)cand_slot_entry(i, log2_n_seg);
                if (e < s.x) cand_lds[s.y + e] = ent;
            };
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PRE; ++u)
                if (u * NT < n_slots) place(u * NT + tid, pre[u]);           // (n_slots is a multiple of 64; a segment's slots lie below it)
            for (int i0 = PRE * NT + tid; i0 < n_slots; i0 += 4 * NT) {
                uint64_t ent[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) ent[u] = list[i0 + u * NT < n_slots ? i0 + u * NT : 0];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (i0 + u * NT < n_slots) place(i0 + u * NT, ent[u]);
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < CPT; ++j) {
                if (j * NT < n_items) {
                    const int i = j * NT + tid;
                    v[j] = __uint_as_float((uint32_t)(cand_lds[i < n_items ? i : 0] >> 32));
                    act |= i < n_items ? 1u << j : 0u;
                }
            }
        } else {
            // all scores of the head to the score buffer, by all its workgroups; the last one to finish goes on
            if constexpr (DT != DT_F32) {
                const int64_t first = (int64_t)blockIdx.z * NW + wave, step = (int64_t)gridDim.z * NW;
                if (D == 128) score_keys<DT, 128>(sh, bf, b, h, P, first, step);
                else if (D == 64) score_keys<DT, 64>(sh, bf, b, h, P, first, step);
                else if (D == 256) score_keys<DT, 256>(sh, bf, b, h, P, first, step);
                else score_keys<DT, 32>(sh, bf, b, h, P, first, step);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __syncthreads();
            if (tid == 0) sm.n_keys = atomicAdd(&bf.flags[bh], kArrivalUnit) / kArrivalUnit;     // (the threshold estimate cleared the count)
            __syncthreads();
            if (sm.n_keys + 1u != gridDim.z) return;      // (uniform)
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            // a list that should have been usable (the measure of the chip-wide selection, whose lists are longer)
            if (tid == 0 && (over || total > (uint32_t)sh.bnd_cap) && !(flags & 5u)) atomicAdd(bf.fallback_total, 1u);
        }
    }

    // ---- the window's scores (a list has none: scored here with plain FMAs), into the places behind the winners'
    float w_top = -INFINITY;                              // largest score of the window
    const int n_rows = k_eff + W;                         // rows to fetch (at most ROWS: the launcher's rule)
    if (SRC == SRC_ROW) {
        for (int i = tid; i < W; i += NT) w_top = fmaxf(w_top, row[P + i]);
    } else if (W > 0) {
        float qf[EPL];
        Elem<DT>::widen(*reinterpret_cast<const u32x4*>(static_cast<const char*>(bf.q) + (bh * D + c * EPL) * Elem<DT>::kBytes), qf);
        const char* const Kh = static_cast<const char*>(bf.K) + head_off;
        constexpr int UW = 4;
        const int step = NW * rpw;
        for (int j = wave * rpw; j < W; j += UW * step) {            // (uniform over the wave)
            u32x4 raw[UW];
#pragma unroll
            for (int u = 0; u < UW; ++u) {
                const int i = j + u * step + rs;
                raw[u] = *reinterpret_cast<const u32x4*>(Kh + ((int64_t)(P + (i < W ? i : W - 1)) * D + c * EPL) * Elem<DT>::kBytes);
            }
#pragma unroll
            for (int u = 0; u < UW; ++u) {
                const int i = j + u * step + rs;
                float kf[EPL], a = 0.f;
                Elem<DT>::widen(raw[u], kf);
#pragma unroll
                for (int e = 0; e < EPL; ++e) a = fmaf(kf[e], qf[e], a);
                for (int o = 1; o < lpr; o <<= 1) a += wave_xor(a, o);
                if (i < W) {
                    w_top = fmaxf(w_top, a);
                    if (c == 0) rows_lds[k_eff + i] = (uint64_t)__float_as_uint(a) << 32;
                }
            }
        }
    }
    if (usable) {
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
            if (j * NT < n_items) {                       // (uniform)
                v[j] += 0.0f;                             // -0 counts as +0
                if ((act >> j) & 1u) { lo = fminf(lo, v[j]); hi = fmaxf(hi, v[j]); }
            }
        }
    }
    if (SRC == SRC_LIST && !usable) __syncthreads();      // (n_keys was read above)
    select_clear<Team>(sm);
    team_range<Team>(lo, hi, sm, 0);
    float top = hi;                                       // largest selected score
    if (W > 0) {                                          // (uniform)
        float dummy = 0.f;
        team_range<Team>(dummy, w_top, sm, 1);
    }
    float M = fmaxf(k_eff > 0 ? top : -INFINITY, w_top);  // the weights' reference score
    const bool writer = blockIdx.z == 0 || !usable;       // (uniform) the workgroup that writes the selection
    auto weight = [&](float s) { return (uint64_t)__float_as_uint(exp2f((s - M) * scale_log2e)) << 32; };
    auto emit = [&](uint32_t o, float s, int32_t p) {     // winner o of the head
        if (o < (uint32_t)k_eff) {                        // always true; guards the buffers
            if (writer) {
                idx[o] = p;
                vals[o] = s;
            }
            rows_lds[o] = weight(s) | (uint64_t)(uint32_t)p;
        }
    };

    // ---- the k_eff best
    Boundary left{0u, 0u};
    if (usable && k_eff > 0) {
        left = team_select<Team, CPT, CPT>([&](int j) { return v[j]; }, act, n_items, P, k_eff, lo, hi, sm, pos, emit);
        if (writer) pad_outputs(k_eff, sh.k, idx, vals);
    } else if (k_eff == 0) {                              // nothing to search for this sequence
        if (writer) pad_outputs(0, sh.k, idx, vals);
    } else if (SRC == SRC_LIST) {                         // radix select over the full score row
        __shared__ SelShared sel_sm;
        top = key_score(wg_select_dense<NT, 0>(sh, bf, bh, P, k_eff, sel_sm));      // writes idx, vals and their padding
        M = fmaxf(top, w_top);
        __syncthreads();
        for (int o = tid; o < k_eff; o += NT) rows_lds[o] = weight(vals[o]) | (uint64_t)(uint32_t)idx[o];
    }
    if (SRC == SRC_LIST && tid == 0 && writer) {          // the head's record, as the chip-wide selection leaves it
        uint32_t* const rec = bf.tailrec + 4 * bh;
        const bool sel = usable && k_eff > 0;
        rec[0] = k_eff == 0 ? 2u : usable ? 0u : 1u;
        rec[1] = sel ? (uint32_t)k_eff - left.need : 0u;
        rec[2] = sel ? left.need : 0u;
        rec[3] = sel ? left.in : 0u;
    }
    for (int i = tid; i < W; i += NT)
        rows_lds[k_eff + i] = weight(SRC == SRC_ROW ? row[P + i] : __uint_as_float((uint32_t)(rows_lds[k_eff + i] >> 32))) | (uint64_t)(uint32_t)(P + i);
    __syncthreads();

    // ---- the weighted value rows (of this workgroup's share)
    const char* const Vh = static_cast<const char*>(bf.V) + head_off;
    float acc[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
    float lsum = 0.f;
    const int step = NW * rpw;
    const int shares = SRC == SRC_LIST && usable ? (int)gridDim.z : 1;
    const int share = shares > 1 ? (int)blockIdx.z : 0;
    const int row_end = (int)((int64_t)n_rows * (share + 1) / shares);
    for (int j = (int)((int64_t)n_rows * share / shares) + wave * rpw + rs; j < row_end; j += U * step) {
        float w[U];
        u32x4 raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int jj = j + u * step < row_end ? j + u * step : j;
            const uint64_t e = rows_lds[jj];
            w[u] = j + u * step < row_end ? __uint_as_float((uint32_t)(e >> 32)) : 0.f;
            const uint32_t p = (uint32_t)e < (uint32_t)N ? (uint32_t)e : (uint32_t)(N - 1);     // (always below N)
            raw[u] = *reinterpret_cast<const u32x4*>(Vh + ((int64_t)p * D + c * EPL) * Elem<DT>::kBytes);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float vf[EPL];
            Elem<DT>::widen(raw[u], vf);
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] = fmaf(w[u], vf[e], acc[e]);
            lsum += w[u];
        }
    }
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
    if (rs == 0) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc_lds[wave][c * EPL + e] = acc[e];
        if (c == 0) acc_lds[wave][256] = lsum;
    }
    __syncthreads();
    float a = 0.f, l = 0.f;                               // thread t < D: channel t (D <= NT)
    if (tid < D) {
#pragma unroll
        for (int w = 0; w < NW; ++w) { a += acc_lds[w][tid]; l += acc_lds[w][256]; }
    }
    if (SRC == SRC_LIST && shares > 1) {
        // Leave the share where the head's other workgroups see it (agent-scope stores go through to memory, and the wait
        // below is for their arrival there), count it, and let the last workgroup add up all shares in their order.
        // No release or acquire fence: those write back and invalidate the whole L2 of the XCD, and nothing
        // but these values passes between the workgroups.
        float* const pa = bf.part_acc + bh * sh.n_chunk_cap * (int64_t)D;
        float* const pl = bf.part_l + bh * sh.n_chunk_cap;
        if (tid < D) __hip_atomic_store(pa + share * D + tid, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (tid == 0) __hip_atomic_store(pl + share, l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0)
            sm.n_keys = __hip_atomic_fetch_add(&bf.flags[bh], kArrivalUnit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) / kArrivalUnit;
        __syncthreads();
        if (sm.n_keys + 1u != (uint32_t)shares) return;   // (uniform)
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
// stream.  The four waves score the stream's tiles with the scan's routines and leave the scores in LDS; then
// each wave selects for one head of the group and fetches its rows, with no barrier between the waves.  The step is
// bound by reading the keys; two or more workgroups per compute unit, each in a phase of its own, keep that going
// while others select.  ROW: scores of the longest sequence.  192 sequences of 2048 .. 4096 tokens, k = 128 (1.2 GB of keys,
// 0.2 GB of value rows): 281 us = 5.0 TB/s; scan with stored scores, radix select and gather before: 277 + 70 + 42 us.
constexpr int kShortBins = 256;
template <int DT, int D, int ROW>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
attend_short_kernel(Shape sh, Bufs bf, float scale, float scale_log2e) {
    using v8 = typename Mfma<DT>::v8;
    constexpr int CPT = ROW / kWave, ROWS = attend_short_k(ROW), EPL = 8, LPR = D / EPL, RPW = kWave / LPR, U = 8;
    using Mask = typename std::conditional<(CPT > 32), uint64_t, uint32_t>::type;
    __shared__ float scores_lds[4][ROW];
    __shared__ uint64_t rows_all_lds[4][ROWS];            // rows to fetch (weight bits, position)
    __shared__ SelectShared<WaveTeam, kShortBins> sms[4];
    const int kvh = blockIdx.x, b = blockIdx.y, G = sh.G;
    const int64_t head0 = (int64_t)b * sh.Hq + (int64_t)kvh * G;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int N = bf.len[b];                              // (no window on this path)
    const char* const Kh = static_cast<const char*>(bf.K) + ((int64_t)b * sh.Hkv + kvh) * sh.Ncap * (D * 2);
    {
        v8 qa[D / 32];
        load_query_a<DT, D>(bf.q, head0, G, qa);
        struct TileB { v8 b[4][D / 32]; } ba, bb;
        auto use = [&](TileB& t, int64_t ti) {
            const f32x4 res = tile_mac<DT, D>(t.b, qa);
            const int item = (int)ti * 64 + lane;
            if (item < N) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (r < G) scores_lds[r][item] = res[r] + 0.0f;          // -0 counts as +0
            }
        };
        const uint32_t lane_off = (uint32_t)(((lane & 15) * D + (lane >> 4) * 8) * 2);
        const int64_t rest = walk_tiles<ScanPipelined<D>::value>(wave, N / 64, 4, ba, bb,
            [&](TileB& t, int64_t ti) { tile_load_full<DT, D>(Kh + ti * (64 * D * 2), lane_off, t.b); }, use);
        if (rest * 64 < N) {                              // the tile the end of the sequence cuts short
            tile_load<DT, D>(Kh, [&](int slot) { const int64_t p = rest * 64 + slot; return p < N ? p : (int64_t)(N - 1); }, ba.b);
            use(ba, rest);
        }
    }
    __syncthreads();
    if (wave >= G) return;                                // (no barrier of the workgroup follows)

    const int64_t bh = head0 + wave;
    const int k_eff = sh.k < N ? sh.k : N;
    int32_t* const idx = bf.sel_idx + bh * sh.k;
    float* const vals = bf.sel_val + bh * sh.k;
    SelectShared<WaveTeam, kShortBins>& sm = sms[wave];
    // (64 scores of a lane in registers spilled: they stay in LDS, eight reads in flight)
    const float* const row = scores_lds[wave] + lane;
    Mask act = 0;
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll 8
    for (int j = 0; j < CPT; ++j) {
        if (j * kWave + lane < N) {
            const float s = row[j * kWave];
            act |= (Mask)1 << j;
            lo = fminf(lo, s); hi = fmaxf(hi, s);
        }
    }
    select_clear<WaveTeam>(sm);
    team_range<WaveTeam>(lo, hi, sm, 0);
    const float M = hi;                                   // the weights' reference score
    uint64_t* const rows_lds = rows_all_lds[wave];
    team_select<WaveTeam, CPT, 8>([&](int j) { return row[j * kWave]; }, act, N, N, k_eff, lo, hi, sm,
                                  [&](int j) { return j * kWave + lane; }, [&](uint32_t o, float s, int32_t p) {
        if (o < (uint32_t)k_eff) {                        // always true; guards the buffers
            idx[o] = p;
            vals[o] = s;
            rows_lds[o] = ((uint64_t)__float_as_uint(exp2f((s - M) * scale_log2e)) << 32) | (uint64_t)(uint32_t)p;
        }
    });
    for (int o = k_eff + lane; o < sh.k; o += kWave) { idx[o] = -1; vals[o] = -INFINITY; }
    wave_sync();

    const char* const Vh = static_cast<const char*>(bf.V) + ((int64_t)b * sh.Hkv + kvh) * sh.Ncap * (D * 2);
    const int rs = lane / LPR, c = lane % LPR;
    float acc[EPL], l = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
    for (int j = rs; j < k_eff; j += U * RPW) {
        float w[U];
        u32x4 raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t e = rows_lds[j + u * RPW < k_eff ? j + u * RPW : j];
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
    if (lane == 0) {
        bf.hmax[bh] = M;
        if (bf.lse) bf.lse[bh] = M * scale + logf(l);
    }
}

hipError_t launch_attend_short(const Shape& s, const Bufs& b, int64_t Nmax, hipStream_t st) {
    const float scale = 1.0f / sqrtf((float)s.D);
    const float scale_log2e = scale * 1.4426950408889634f;
    const dim3 grid((unsigned)s.Hkv, (unsigned)s.B);
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
    const dim3 grid((unsigned)s.Hq, (unsigned)s.B);
    const bool many = (int64_t)s.Hq * s.B > kAttendManyHeads;
    if (s.k + s.window > attend_row_rows((int64_t)s.Hq * s.B, Nmax)) return hipErrorInvalidValue;
#define TKA_AR(DT_, NT_, CPT_, NB_)                                                                                         \
    hipLaunchKernelGGL((attend_kernel<DT_, AttendCfg<NT_, CPT_, NT_ == 1024 ? 4096 : NT_ == 512 ? 2048 : 1024, NB_>, SRC_ROW>), \
                       grid, dim3(NT_), 0, st, s, b, scale, scale_log2e)
#define TKA_AR_SIZE(DT_)                                     \
    do {                                                     \
        if (many && Nmax <= 2048) TKA_AR(DT_, 256, 8, 512);  \
        else if (many && Nmax <= 4096) TKA_AR(DT_, 256, 16, 512);  \
        else if (many && Nmax <= 8192) TKA_AR(DT_, 512, 16, 512);  \
        else if (Nmax <= 4096) TKA_AR(DT_, 1024, 4, 1024);   \
        else TKA_AR(DT_, 1024, 16, 1024);                    \
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
    const dim3 grid((unsigned)s.Hq, (unsigned)s.B, (unsigned)s.attend);
    if (s.dtype == DT_F16) hipLaunchKernelGGL((attend_kernel<DT_F16, ListCfg, SRC_LIST>), grid, dim3(ListCfg::NT), 0, st, s, b, scale, scale_log2e);
    else if (s.dtype == DT_BF16) hipLaunchKernelGGL((attend_kernel<DT_BF16, ListCfg, SRC_LIST>), grid, dim3(ListCfg::NT), 0, st, s, b, scale, scale_log2e);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace tka

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
// What bounds it: instructions and barriers of one compute unit per head (stamps of a first version: loads 1.5-3 us, bins and
// their prefix sum 1.6, ranking and emission 2, rows 1.5-2, sum and write 1.5, which is 8 to 10 us of the 14 to 18 below; where the
// rest goes, start and end of the launch included, was not measured), so scores stay in registers with
// slots nobody uses skipped uniformly (the same phases as rolled loops over LDS: 23.6 us against 14.5 at 16k
// tokens) and scans and reductions run in the vector unit instead of trips through LDS.  Measured, 32 heads, 8 KV heads:
// a row of 16k scores, k = 256: 14.6 us (radix select + gather before: 18.7 + 7.9); a list at 48k tokens, k = 768 on average:
// 16.4 us, at 128k tokens, k = 2048: 18.9 us (chip-wide tail: 11.6 + 11.6 and 14.5 + 9.6 us and a launch more).
//
//   SRC_ROW   the scores of a short cache, stored by the scan (general path)
//   (attend_short_kernel: the scores too, for batches of short sequences)
//   SRC_LIST  the candidate list the filtered scan left (what becomes of one that is too long or unusable: below)
#include <algorithm>
#include <type_traits>

#include "device_utils.h"
#include "internal.h"
#include "scan_common.h"
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

// A list longer than the registers hold, or unusable (a segment overflowed).  The scan's counts per score bin, which go on
// where a segment is full, say which bin B the k-th score falls in and how many entries of the bins from B up every scan
// workgroup left:
//   LONG_CUT   they fit: every workgroup of the head takes those alone into its registers and goes on as with a short list
//   LONG_TIED  they do not (most of them tie): one workgroup goes on alone, by radix select over the list
//   RESCORE    a segment overflowed: the head's workgroups score the keys of its tiles again (arithmetic and dealing of the scan),
//              put those from bin B up into the segments, and the last to finish goes on alone with that list
//   SCORE_ROW  the same where the counts do not cover k keys or those from B up do not fit either: all scores go to
//              the score buffer, and the last to finish goes on alone by radix select over the row
// us per call, 32 heads, 8 KV heads, d = 128; chip-wide tail / before the list was cut by the counts (every such head scored
// again, radix select over the row) / now.  A quarter of the keys identical and just below the k-th score (lists of 36k,
// 135k at 512k tokens): 128k tokens, k = 2048 88 / 444 / 87; 512k tokens 287 / 1518 / 281; 16 queries at 128k tokens 292 / 2579 /
// 237.  The same on top (tied): 279 / 548 / 244, at 16 queries 576 / 2789 / 509.  Overflow: one KV head, 4 query heads, 512k tokens, 92 %
// identical 161 / - / 147; 8 KV heads, 512k tokens, 70 % on top (row) 3822 / 2957 / 2826.  Slower than the tail where one head of
// a batch that fills the chip is scored by its one workgroup: 4 of 256 heads, 128k tokens, 97 % identical 1466 / - / 1951.
enum { LIST_SHORT = 0, LONG_CUT, LONG_TIED, RESCORE, SCORE_ROW };

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

// LONG_CUT: the entries of bin B and above, `keep` of scan workgroup j (four segments) from place at(j) on.
template <int NW>
__device__ __forceinline__ void cut_list(const Shape& sh, int wave, int B, float bin_lo, float bin_inv, const uint2* segs,
                                         const uint32_t* at, const uint64_t* list, uint64_t* kept, uint32_t n_kept) {
    constexpr int U = 2;
    const int lane = lane_id();
    for (int j = wave; j < sh.n_seg / kScanWaves; j += NW) {
        uint32_t o = at[j], len[kScanWaves], longest = 0;
#pragma unroll
        for (int s = 0; s < kScanWaves; ++s) {
            len[s] = segs[j * kScanWaves + s].x;
            longest = len[s] > longest ? len[s] : longest;
        }
        for (uint32_t e0 = 0; e0 < longest; e0 += U * kWave) {
            uint64_t ent[kScanWaves][U];
#pragma unroll
            for (int s = 0; s < kScanWaves; ++s) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t e = e0 + u * kWave + lane;
                    ent[s][u] = list[cand_slot(e < len[s] ? e : 0, j * kScanWaves + s, sh.n_seg)];
                }
            }
#pragma unroll
            for (int s = 0; s < kScanWaves; ++s) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool keep = e0 + u * kWave + lane < len[s] &&
                                      tail_bin(__uint_as_float((uint32_t)(ent[s][u] >> 32)), bin_lo, bin_inv) >= B;
                    const uint64_t m = __ballot(keep);
                    const uint32_t to = o + (uint32_t)mask_rank(m);
                    if (keep && to < n_kept) kept[to] = ent[s][u];           // (below n_kept always; guards the buffer)
                    o += (uint32_t)__popcll(m);
                }
            }
        }
    }
}

// LONG_TIED: the slots of the list as a source of the radix select; `segs`: lengths of its segments (LDS).
template <int NT>
struct SrcSegments {
    static constexpr int kThreads = NT;
    const uint64_t* list;
    const uint2* segs;
    int64_t n;
    int log2_n_seg;
    typedef uint64_t raw_t;
    __device__ __forceinline__ int64_t slots() const { return n; }
    __device__ __forceinline__ bool valid(int64_t i) const {
        return i < n && (uint32_t)cand_slot_entry(i, log2_n_seg) < segs[cand_slot_segment(i, log2_n_seg)].x;
    }
    __device__ __forceinline__ const uint64_t* where(int64_t i) const { return list + i; }
    __device__ __forceinline__ uint32_t key(uint64_t e) const { return score_key(__uint_as_float((uint32_t)(e >> 32))); }
    __device__ __forceinline__ uint32_t ipos(uint64_t e, int64_t) const { return 0xFFFFFFFFu - (uint32_t)e; }
    __device__ __forceinline__ void stash(int, uint64_t) const {}
    __device__ __forceinline__ uint32_t cached_ipos(int) const { return 0u; }
};

// Grid: heads x sequences x workgroups per head.  SRC_LIST: Shape::attend workgroups of a head all select from its list (the same
// winners, found side by side on compute units that would idle), each fetches its share of the value rows, and the last
// to finish adds up the shares; so a head's rows are not bound by what one compute unit can fetch (about 64 GB/s).
// Further ones, where the heads are few, only lend a hand when keys have to be scored again.
template <int DT, class Cfg, int SRC, int DIM = 0>     // DIM: the head dim of a list kernel
__global__ void __launch_bounds__(Cfg::NT) __attribute__((amdgpu_waves_per_eu(4))) attend_kernel(Shape sh, Bufs bf, float scale, float scale_log2e) {
    constexpr int NT = Cfg::NT, NW = Cfg::NW, CPT = Cfg::CPT;
    using Team = WorkgroupTeam<NT>;
    constexpr int EPL = Elem<DT>::kPerLoad;
    constexpr int U = 8;                                  // value rows in flight per lane group
    __shared__ SelectShared<Team, Cfg::NB> sm;
    __shared__ uint64_t cand_lds[SRC == SRC_LIST ? CPT * NT : 1];      // candidates (score bits, position)
    __shared__ uint64_t rows_lds[Cfg::ROWS];              // value rows to fetch (weight bits, position)
    __shared__ float acc_lds[NW][256 + 1];
    // SRC_LIST: grid z runs over the layers, then over the workgroups of a head
    const int layer = SRC == SRC_LIST ? (int)blockIdx.z & ((1 << sh.log2_layers) - 1) : (int)blockIdx.z;
    const int wg = SRC == SRC_LIST ? (int)blockIdx.z >> sh.log2_layers : 0, n_wgs = SRC == SRC_LIST ? (int)gridDim.z >> sh.log2_layers : 1;
    const int b = (int)blockIdx.y + layer * sh.layer_seqs, h = blockIdx.x;
    const int64_t bh = (int64_t)b * sh.Hq + h;
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const LayerK lk = bf.layer_k[layer];
    const int k = lk.k;
    const int64_t sel0 = selection_at(sh, lk, blockIdx.y, h);
    int32_t* const idx = bf.sel_idx + sel0;
    float* const vals = bf.sel_val + sel0;
    const int D = SRC == SRC_LIST ? DIM : sh.D, lpr = D / EPL, rpw = kWave / lpr;          // lanes per key or value row, rows per wave and load
    const int rs = lane / lpr, c = lane % lpr;
    const int64_t head_off = ((int64_t)cache_seq(sh, b) * sh.Hkv + h / sh.G) * sh.Ncap * D * Elem<DT>::kBytes;

    // ---- the scores to select from, in registers: slot j of a thread holds item j * NT + tid
    float v[CPT];
    int n_items = 0;
    uint32_t act = 0;                                     // bit j: v[j] is a score in question
    bool alone = false;                                   // (uniform) this workgroup goes on for the whole head
    int how = LIST_SHORT;                                 // (uniform)
    bool in_regs = true;                                  // (uniform) the scores to select from are in registers
    uint32_t above = 0, in_b = 0;                         // not LIST_SHORT: keys above bin B, and in it
    int n_slots = 0;                                      // slots of the list in use
    constexpr int PRE = 12;                               // list slots per thread asked for before the segments' lengths are known
    uint64_t pre[SRC == SRC_LIST ? PRE : 1];
    uint64_t* const list = bf.cand + bh * (int64_t)sh.cand_cap;
    uint32_t seg_len = 0, flags = 0;
    const bool helper = SRC == SRC_LIST && wg >= sh.share_wgs;     // (uniform)
    if (SRC == SRC_LIST) {
        if (tid < sh.n_seg) seg_len = bf.seg_cnt[bh * sh.n_seg + tid];
        flags = bf.flags[bh];
        const int n_pre = helper ? 0 : sh.cand_cap;
#pragma unroll
        for (int u = 0; u < PRE; ++u) {
            const int i = u * NT + tid;
            pre[u] = list[i < n_pre ? i : 0];             // (any slot of the list may be read; what lies beyond its segment is ignored)
        }
    }
    const int N = (int)visible_len(sh, bf, b);
    const int P = (int)prefix_len(N, sh.window), W = N - P;      // searched prefix, window
    const int k_eff = k < P ? k : P;
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
        // lengths and places of the segments
        uint32_t total, longest;
        uint2* const segs = reinterpret_cast<uint2*>(sm.keys);
        const int log2_n_seg = 31 - __clz(sh.n_seg);
        auto lay_out = [&]() {
            const uint32_t longest_w = wave_max_u32(seg_len);
            if (lane == 0) sm.hist[wave] = longest_w;
            const uint32_t at = team_prefix<Team>(seg_len, total, sm, 0);
            segs[tid] = make_uint2(seg_len, at);
            longest = wave_max_u32(lane < NW ? sm.hist[lane] : 0u);
            n_slots = (int)((longest + kCandChunk - 1) >> kCandChunkLog2) * sh.n_seg * kCandChunk;
        };
        lay_out();
        // (an index leaves the approximate scores of a head it marked as not filterable)
        const bool over = longest > (uint32_t)sh.seg_cap || (flags & (sh.indexed ? 5u : 4u));
        if (over || total < (uint32_t)k_eff || total > (uint32_t)(CPT * NT)) {
            // the bin of the k-th score from the scan's counts: lane l of every wave looks at bin kTailBins - 1 - l
            static_assert(kTailBins == kWave, "a bin per lane");
            const int n_wg = sh.n_seg / kScanWaves;
            const uint32_t* const hp = bf.hist + bh * (int64_t)sh.hist_cap * kTailBins;
            const float bin_lo = bf.bins[2 * bh], bin_inv = bf.bins[2 * bh + 1];
            uint32_t* const part = reinterpret_cast<uint32_t*>(cand_lds);
            uint32_t n = 0;
#pragma unroll 4
            for (int j = wave; j < n_wg; j += NW) n += hp[j * kTailBins + lane];
            part[wave * kTailBins + lane] = n;
            __syncthreads();
            uint32_t all = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) all += part[w * kTailBins + kTailBins - 1 - lane];
            const uint32_t upto = wave_scan_add(all);
            const uint64_t hit = __ballot(upto - all < (uint32_t)k_eff && (uint32_t)k_eff <= upto);      // (one lane, or the counts do not cover k_eff keys)
            const int hit_lane = hit ? __builtin_ctzll(hit) : 0;
            const int B = kTailBins - 1 - hit_lane;
            in_b = (uint32_t)__builtin_amdgcn_readlane((int)all, hit_lane);
            above = (uint32_t)__builtin_amdgcn_readlane((int)upto, hit_lane) - in_b;
            const uint32_t n_cut = above + in_b;
            if (!hit) how = SCORE_ROW;
            else if (over) how = sh.no_rescan || n_cut > (uint32_t)(CPT * NT) ? SCORE_ROW : RESCORE;
            else how = n_cut <= (uint32_t)(CPT * NT) ? LONG_CUT : LONG_TIED;
            // a list that should have been usable (the measure of the chip-wide selection)
            const bool fallback = (over || !hit || in_b > (uint32_t)sh.bnd_cap) && !(flags & 5u) && counts_fallbacks(sh, b);
            if (how == LONG_CUT) {
#pragma unroll 4
                for (int j = wave; j < n_wg; j += NW) {
                    const uint32_t c = wave_scan_add(lane >= B ? hp[j * kTailBins + lane] : 0u);
                    if (lane == kWave - 1) sm.hist[j] = c;
                }
                __syncthreads();
                const uint32_t at = team_prefix<Team>(tid < n_wg ? sm.hist[tid] : 0u, total, sm, 1);     // (total: n_cut)
                if (tid < n_wg) sm.hist[tid] = at;
                __syncthreads();
                cut_list<NW>(sh, wave, B, bin_lo, bin_inv, segs, sm.hist, list, cand_lds, (uint32_t)(CPT * NT));
            } else if (how == LONG_TIED) {
                if (wg != 0) return;                                               // (uniform)
                if (tid == 0 && fallback) atomicAdd(bf.fallback_total, 1u);
                alone = true;
            } else {
                if constexpr (SRC == SRC_LIST)
                    score_segments<DT, DIM>(sh, bf, b, h, P, wg * NW + wave, n_wgs * NW,
                                            how == SCORE_ROW ? kTailBins : B, bin_lo, bin_inv, list);
                // every wave waits for its stores to arrive in the L2, one thread releases them all (a release writes back the whole
                // L2 of the XCD; one per wave: 247 us per call instead of 147 at one KV head, 512k tokens, 92 % identical)
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                if (tid == 0) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                    sm.n_keys = atomicAdd(&bf.flags[bh], kArrivalUnit);               // (the threshold estimate cleared the count)
                }
                __syncthreads();
                const uint32_t arrived = sm.n_keys;
                if (arrived / kArrivalUnit + 1u != (uint32_t)n_wgs) return;                 // (uniform)
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                if (tid == 0 && fallback) atomicAdd(bf.fallback_total, 1u);
                alone = true;
                if (how == RESCORE && (arrived & 2u)) how = SCORE_ROW;
                if (how == RESCORE) {
                    seg_len = tid < sh.n_seg ? bf.seg_cnt2[bh * sh.n_seg + tid] : 0u;
                    lay_out();
                }
            }
            in_regs = how == LONG_CUT || how == RESCORE;
        }
        if (helper && !alone) return;                     // (uniform)
        if (in_regs) {
            n_items = (int)total;
            if (how != LONG_CUT) {
                auto place = [&](int i, uint64_t ent) {   // slot i of the list: entry e of segment g
                    const uint2 s = segs[cand_slot_segment(i, log2_n_seg)];
                    const uint32_t e = (uint32_t)cand_slot_entry(i, log2_n_seg);
                    if (e < s.x) cand_lds[s.y + e] = ent;
                };
                __syncthreads();
                if (how == LIST_SHORT) {
#pragma unroll
                    for (int u = 0; u < PRE; ++u)
                        if (u * NT < n_slots) place(u * NT + tid, pre[u]);   // (n_slots is a multiple of 64; a segment's slots lie below it)
                }
                for (int i0 = (how == LIST_SHORT ? PRE * NT : 0) + tid; i0 < n_slots; i0 += 4 * NT) {
                    uint64_t ent[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) ent[u] = list[i0 + u * NT < n_slots ? i0 + u * NT : 0];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (i0 + u * NT < n_slots) place(i0 + u * NT, ent[u]);
                }
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
    if (in_regs) {
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
            if (j * NT < n_items) {                       // (uniform)
                v[j] += 0.0f;                             // -0 counts as +0
                if ((act >> j) & 1u) { lo = fminf(lo, v[j]); hi = fmaxf(hi, v[j]); }
            }
        }
    }
    if (SRC == SRC_LIST && alone) __syncthreads();        // (what select_clear() writes was read above)
    select_clear<Team>(sm);
    team_range<Team>(lo, hi, sm, 0);
    float top = hi;                                       // largest selected score
    if (W > 0) {                                          // (uniform)
        float dummy = 0.f;
        team_range<Team>(dummy, w_top, sm, 1);
    }
    float M = fmaxf(k_eff > 0 ? top : -INFINITY, w_top);  // the weights' reference score
    const bool writer = wg == 0 || alone;         // (uniform) the workgroup that writes the selection
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
    if (in_regs && k_eff > 0) {
        left = team_select<Team, CPT, CPT>([&](int j) { return v[j]; }, act, n_items, P, k_eff, lo, hi, sm, pos, emit);
        if (writer) pad_outputs(k_eff, k, idx, vals);
    } else if (k_eff == 0) {                              // nothing to search for this sequence
        if (helper) return;
        if (writer) pad_outputs(0, k, idx, vals);
    } else if (SRC == SRC_LIST) {                         // radix select over the list or the full score row
        __shared__ SelShared sel_sm;
        if (how == SCORE_ROW) {
            top = key_score(wg_select_dense<NT, 0>(sh, bf, bh, P, k_eff, k, idx, vals, sel_sm));      // writes idx, vals and their padding
        } else {
            const SrcSegments<NT> src{list, reinterpret_cast<const uint2*>(sm.keys), n_slots, 31 - __clz(sh.n_seg)};
            const Items<0, SrcSegments<NT>> items(src);
            top = key_score(wg_topk_emit(items, k_eff, k, idx, vals, sel_sm));
        }
        M = fmaxf(top, w_top);
        __syncthreads();
        for (int o = tid; o < k_eff; o += NT) rows_lds[o] = weight(vals[o]) | (uint64_t)(uint32_t)idx[o];
    }
    if (SRC == SRC_LIST && tid == 0 && writer) {          // the head's record, as the chip-wide selection leaves it
        uint32_t* const rec = bf.tailrec + 4 * bh;
        const bool sel = how != SCORE_ROW && k_eff > 0;
        if (how != LIST_SHORT) left = Boundary{in_b, (uint32_t)k_eff - above};
        rec[0] = k_eff == 0 ? 2u : sel ? 0u : 1u;
        rec[1] = sel ? (uint32_t)k_eff - left.need : 0u;
        rec[2] = sel ? left.need : 0u;
        rec[3] = sel ? left.in : 0u;
    }
    for (int i = tid; i < W; i += NT)
        rows_lds[k_eff + i] = weight(SRC == SRC_ROW ? row[P + i] : __uint_as_float((uint32_t)(rows_lds[k_eff + i] >> 32))) | (uint64_t)(uint32_t)(P + i);
    __syncthreads();

    // ---- the weighted value rows (of this workgroup's shares, one after the other)
    const char* const Vh = static_cast<const char*>(bf.V) + head_off;
    const int step = NW * rpw;
    const int shares = SRC == SRC_LIST && !alone ? sh.attend : 1;
    const int share_wgs = shares > 1 ? sh.share_wgs : 1;
    float* const pa = bf.part_acc + bh * sh.n_chunk_cap * (int64_t)D;
    float* const pl = bf.part_l + bh * sh.n_chunk_cap;
    float a = 0.f, l = 0.f;                               // thread t < D: channel t (D <= NT)
    for (int share = share_wgs > 1 ? wg : 0; share < shares; share += share_wgs) {       // (uniform)
        float acc[EPL];
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
        float lsum = 0.f;
        const int row_end = (int)((uint32_t)(n_rows * (share + 1)) / (uint32_t)shares);      // (at most ROWS x 8)
        for (int j = (int)((uint32_t)(n_rows * share) / (uint32_t)shares) + wave * rpw + rs; j < row_end; j += U * step) {
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
        float as = 0.f, ls = 0.f;
        if (tid < D) {
#pragma unroll
            for (int w = 0; w < NW; ++w) { as += acc_lds[w][tid]; ls += acc_lds[w][256]; }
        }
        // Leave the share where the head's other workgroups see it (agent-scope stores go through to memory, and the wait
        // below is for their arrival there), count it, and let the last workgroup add up all shares in their order.
        // No release or acquire fence: those write back and invalidate the whole L2 of the XCD, and nothing
        // but these values passes between the workgroups.  (A workgroup that takes all shares adds them up as it goes.)
        if (SRC == SRC_LIST && share_wgs > 1) {
            if (tid < D) __hip_atomic_store(pa + share * D + tid, as, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (tid == 0) __hip_atomic_store(pl + share, ls, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            a += as; l += ls;
        }
        if (SRC == SRC_LIST && share + share_wgs < shares) __syncthreads();        // (acc_lds is written again)
    }
    if (SRC == SRC_LIST && share_wgs > 1) {
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
// stream.  The four waves score the stream's tiles with the scan's routines and leave the scores in LDS; then
// each wave selects for one head of the group and fetches its rows, with no barrier between the waves.  The step is
// bound by reading the keys; two or more workgroups per compute unit, each in a phase of its own, keep that going
// while others select.  ROW: scores of the longest sequence.  192 sequences of 2048 .. 4096 tokens, k = 128 (1.2 GB of keys,
// 0.2 GB of value rows): 310 us = 4.6 TB/s; scan with stored scores, radix select and gather before: 277 + 70 + 42 us.
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
    const LayerK lk = bf.layer_k[blockIdx.z];
    const int k = lk.k, k_eff = k < N ? k : N;
    const int64_t sel0 = selection_at(sh, lk, blockIdx.y, kvh * G + wave);
    int32_t* const idx = bf.sel_idx + sel0;
    float* const vals = bf.sel_val + sel0;
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
    for (int o = k_eff + lane; o < k; o += kWave) { idx[o] = -1; vals[o] = -INFINITY; }
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
    hipLaunchKernelGGL((attend_kernel<DT_, AttendCfg<NT_, CPT_, NT_ == 1024 ? 4096 : NT_ == 512 ? 2048 : 1024, NB_>, SRC_ROW>), \
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
    const int64_t room = std::min<int64_t>(kAttendManyHeads / ((int64_t)s.Hq * s.B), s.n_seg / ListCfg::NW);
    const dim3 grid((unsigned)s.Hq, (unsigned)s.layer_seqs, (unsigned)std::max<int64_t>(s.share_wgs, room) << s.log2_layers);
#define TKA_AL(DT_, D_) hipLaunchKernelGGL((attend_kernel<DT_, ListCfg, SRC_LIST, D_>), grid, dim3(ListCfg::NT), 0, st, s, b, scale, scale_log2e)
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

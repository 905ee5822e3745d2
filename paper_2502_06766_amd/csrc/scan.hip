// Key-scoring scan: S[h, i] = q_h . K[g(h), i] over the cached keys of one layer
// (the score matrix S = q K^T of Eq. 1 of arXiv 2502.06766, raw dot products as used by
// the paper's k-nearest-neighbour search under the dot-product metric).
//
// 16-bit caches use v_mfma_f32_16x16x32_{f16,bf16}: one wave scores a tile of 64
// consecutive keys against the (up to 4) query heads that share the KV head, fp32
// accumulate.  Operand B is loaded straight from the row-major key rows in its MFMA
// register layout (lane (j, n) holds 8 consecutive channels of key n), operand A holds the
// query block replicated in every group of four rows, so that after four accumulators
// (one per 16-key sub-tile) lane l owns the scores of key l for all heads of the group.
//
// Three uses of the same tile routine:
//   sample : score a strided, jittered sample of positions (threshold estimate)
//   filter : score every key, keep (score, position) pairs >= a per-head threshold; every
//            wave appends to a private segment of the head's candidate list (plain stores,
//            no atomics, so the list order is fixed by the launch geometry alone) and the
//            workgroup counts what it kept per score bin for the selection that follows; with
//            a page index the wave reads only the tiles (pages) the index could not rule out
//   full   : score every key and store the fp32 scores
// fp32 caches go through a plain FMA kernel (full only).
#include "device_utils.h"
#include "internal.h"
#include "scan_common.h"
#include "scan_tiles.h"
#include "threshold.h"

namespace tka {

// SAMPLED (filter mode only): the scan works out the thresholds of its heads itself (a wave per head, every workgroup of a
// key stream the same ones), while the first key tiles are on their way; the first workgroup leaves them for the kernels
// that follow.  For samples a wave can take at a glance this beats a launch of its own (8 KV heads: 48k
// tokens 4.8 + 22.0 us and the gap between two launches against 24.7 us, 128k tokens 5.5 + 45.0 against 48.8).
// PAGED (filter mode only): the wave skips the tiles whose bit in the page mask is clear (pages of 64 keys
// that the coarse page index has ruled out for every head of the group).
template <int DT, int D, int MODE, bool PAGED = false, bool SAMPLED = false>
__global__ void __launch_bounds__(kScanWaves* kWave)
scan_mfma_kernel(Shape sh, Bufs bf, int tiles_per_wave, float* dst) {
    fetch_args<kArgBytes>();
    using v8 = typename Mfma<DT>::v8;
    const int b = blockIdx.z, kvh = blockIdx.y;
    const int G = sh.G;
    const int64_t head0 = (int64_t)b * sh.Hq + (int64_t)kvh * G;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // wave-uniform
    const int64_t N = prefix_len(bf.len[b], sh.window);

    int64_t n_items = N;   // keys (or samples) this (b, kv head) has
    int stride = 1;
    if (MODE == MODE_SAMPLE) {
        if (N == 0) return;          // nothing to search: the whole sequence is inside the window
        Plan pl = make_plan(N, sh.k < N ? sh.k : (int)N);
        n_items = pl.n_samp;
        stride = pl.stride;
    }
    // tiles of this wave.  sample/full: a workgroup owns a contiguous run of tiles and its
    // waves take them round-robin.  filter: wave-segment sid = 4 blockIdx.x + wave takes one tile
    // of every row of n_seg tiles (seg_tile()), so that any clustering of high scores along the
    // sequence spreads evenly over the segments.
    const int64_t n_tiles_all = (n_items + 63) / 64;
    int64_t tile, tile_end, tile_step;
    if (MODE == MODE_FILTER) {
        tile = 0;                           // (the filter's walk counts rows of n_seg tiles)
        tile_step = 1;
        tile_end = 0;
    } else {
        const int64_t tile0 = (int64_t)blockIdx.x * tiles_per_wave * kScanWaves;
        if (tile0 >= n_tiles_all) return;   // whole workgroup past the end
        tile = tile0 + wave;
        tile_step = kScanWaves;
        tile_end = tile0 + (int64_t)tiles_per_wave * kScanWaves;
        if (tile_end > n_tiles_all) tile_end = n_tiles_all;
    }

    v8 qa[D / 32];
    load_query_a<DT, D>(bf.q, head0, G, qa);
    const char* Kh = static_cast<const char*>(bf.K) + ((int64_t)b * sh.Hkv + kvh) * sh.Ncap * (D * 2);

    // filter: this wave's segment in each head's candidate list
    const int seg_cap = sh.seg_cap;
    const int n_seg = sh.n_seg;
    const int sid = (int)blockIdx.x * kScanWaves + wave;
    uint64_t* const list0 = bf.cand + head0 * (int64_t)sh.cand_cap;
    __shared__ uint64_t stage_lds[MODE == MODE_FILTER ? kScanWaves * 4 * kStage : 1];
    uint64_t* const st0 = stage_lds + (MODE == MODE_FILTER ? wave * 4 * kStage : 0);
    CandStage cs0{st0, list0, sid, 0, 0}, cs1{st0 + kStage, list0 + (int64_t)sh.cand_cap, sid, 0, 0},
        cs2{st0 + 2 * kStage, list0 + 2 * (int64_t)sh.cand_cap, sid, 0, 0},
        cs3{st0 + 3 * kStage, list0 + 3 * (int64_t)sh.cand_cap, sid, 0, 0};
    float thr0 = 0.f, thr1 = 0.f, thr2 = 0.f, thr3 = 0.f;
    float lo0 = 0.f, lo1 = 0.f, lo2 = 0.f, lo3 = 0.f, iw0 = 0.f, iw1 = 0.f, iw2 = 0.f, iw3 = 0.f;   // tail_bin() of each head
    float top0 = -INFINITY, top1 = -INFINITY, top2 = -INFINITY, top3 = -INFINITY;   // largest score seen per head
    // candidates of this workgroup per score bin and head (the tail sorts them by bin)
    __shared__ uint32_t hist_lds[MODE == MODE_FILTER ? 4 * kTailBins : 1];
    struct TileB { v8 b[4][D / 32]; } ba, bb;
    const LaneOffsets lane_off = lane_offsets<D>();
    // filter: one tile per row of n_seg tiles; the first is asked for ahead of the thresholds
    const int64_t rows_mine = MODE == MODE_FILTER ? seg_rows((N + 63) / 64, sid, n_seg) : 0;
    auto load_at = [&](TileB& t, int64_t ti) { tile_load_at<DT, D>(Kh, ti, N, lane_off, t.b); };
    auto load_seg = [&](TileB& t, int64_t i) { load_at(t, seg_tile(i, sid, n_seg)); };
    constexpr bool kAhead = MODE == MODE_FILTER && !PAGED && ScanPipelined<D>::value;
    if (MODE == MODE_FILTER) {
        for (int i = threadIdx.x; i < 4 * kTailBins; i += kScanWaves * kWave) hist_lds[i] = 0;
        if constexpr (SAMPLED) {
            constexpr int CPT = kScanSampMax / kWave;
            __shared__ ThresholdShared<WaveTeam> thr_sm[kScanWaves];
            __shared__ float thr_lds[4][3];
            const bool mine = wave < G;                              // (uniform over the wave)
            const int64_t bh = head0 + (mine ? wave : 0);
            const Plan pl = make_plan(N > 0 ? N : 1, sh.k < N ? sh.k : (int)N);
            float sv[CPT];
#pragma unroll
            for (int u = 0; u < CPT; ++u)
                sv[u] = mine && u * kWave < pl.n_samp ? bf.samp[bh * sh.samp_cap + u * kWave + lane] : 0.f;
            if (kAhead) load_seg(ba, 0);                             // (without a tile for this wave it reads nothing)
            __builtin_amdgcn_sched_barrier(0);
            if (mine) {
                for (int u = lane; u < kThrBins; u += kWave) thr_sm[wave].hist[u] = 0;
                const Threshold t = N > 0 ? estimate_threshold<WaveTeam, CPT>(sv, pl, thr_sm[wave]) : Threshold{INFINITY, 0.f, 0.f};
                if (lane == 0) {
                    thr_lds[wave][0] = t.thr; thr_lds[wave][1] = t.bin_lo; thr_lds[wave][2] = t.bin_inv;
                    if (blockIdx.x == 0) leave_threshold(bf, bh, t, N > 0 ? threshold_flags(sh, pl, N) : 0u);
                }
            }
            lds_barrier();
            auto uni = [](float x) { return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(x))); };
            thr0 = uni(thr_lds[0][0]); lo0 = uni(thr_lds[0][1]); iw0 = uni(thr_lds[0][2]);
            if (1 < G) { thr1 = uni(thr_lds[1][0]); lo1 = uni(thr_lds[1][1]); iw1 = uni(thr_lds[1][2]); }
            if (2 < G) { thr2 = uni(thr_lds[2][0]); lo2 = uni(thr_lds[2][1]); iw2 = uni(thr_lds[2][2]); }
            if (3 < G) { thr3 = uni(thr_lds[3][0]); lo3 = uni(thr_lds[3][1]); iw3 = uni(thr_lds[3][2]); }
        } else {
            const float* bins = bf.bins + 2 * head0;
            thr0 = bf.thr[head0]; lo0 = bins[0]; iw0 = bins[1];
            if (1 < G) { thr1 = bf.thr[head0 + 1]; lo1 = bins[2]; iw1 = bins[3]; }
            if (2 < G) { thr2 = bf.thr[head0 + 2]; lo2 = bins[4]; iw2 = bins[5]; }
            if (3 < G) { thr3 = bf.thr[head0 + 3]; lo3 = bins[6]; iw3 = bins[7]; }
            if (kAhead) load_seg(ba, 0);
            lds_barrier();
        }
    }

    auto sample_row = [&](int64_t item) -> int64_t {        // key row of a sample (beyond the last one: the last one's)
        const int64_t p = sample_pos((int)(item < n_items ? item : n_items - 1), stride);
        return p < N ? p : N - 1;
    };
    auto consume = [&](const f32x4& res, int64_t item0) {
        const int64_t item = item0 + lane;
        const bool valid = item < n_items;
        if (MODE == MODE_SAMPLE) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (r < G && valid) bf.samp[(head0 + r) * sh.samp_cap + item] = res[r];
        } else if (MODE == MODE_FULL) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (r < G && valid) dst[(head0 + r) * sh.Ncap + item] = res[r];
        } else {
            if (valid) {
                top0 = fmaxf(top0, res[0]); top1 = fmaxf(top1, res[1]);
                top2 = fmaxf(top2, res[2]); top3 = fmaxf(top3, res[3]);
            }
            if (0 < G) filter_head(res[0], thr0, cs0, valid, item, seg_cap, sh.n_seg, hist_lds, lo0, iw0);
            if (1 < G) filter_head(res[1], thr1, cs1, valid, item, seg_cap, sh.n_seg, hist_lds + kTailBins, lo1, iw1);
            if (2 < G) filter_head(res[2], thr2, cs2, valid, item, seg_cap, sh.n_seg, hist_lds + 2 * kTailBins, lo2, iw2);
            if (3 < G) filter_head(res[3], thr3, cs3, valid, item, seg_cap, sh.n_seg, hist_lds + 3 * kTailBins, lo3, iw3);
        }
    };

    auto load_sample = [&](TileB& t, int64_t ti) { tile_load<DT, D>(Kh, [&](int slot) { return sample_row(ti * 64 + slot); }, t.b); };
    auto use = [&](TileB& t, int64_t ti) { consume(tile_mac<DT, D>(t.b, qa), ti * 64); };
    if (MODE == MODE_SAMPLE) {
        walk_tiles<false>(tile, tile_end, tile_step, ba, bb, load_sample, use);
    } else if (MODE == MODE_FILTER && PAGED) {
        // The pages kept, ascending, are dealt to the wave segments by rank like the tiles of the plain scan
        // (seg_tile() over ranks; 64 rows looked up at a time, one per lane), so every wave reads as many
        // tiles as any other.  They are walked like the plain sequence (next tile's loads in flight
        // while the current one is multiplied and filtered; one buffer at head_dim 256).
        // Every workgroup finds its ranks in the mask itself, by the counts of up to 1024 groups of mask words.  (A launch of one workgroup per
        // key stream that wrote the list out for the scan took 6.3 us, this costs the scan 3: a million tokens 191.8 -> 185.5 us, calls of 140k to 400k tokens
        // 1.08 - 1.16 times as fast.)  A group is one word up to 4.2 million tokens, and its word stays in LDS; the words of a longer group are
        // asked for eight at a time when a rank is looked up in it, so that no load waits for another.  (256 groups, walked word after
        // word / now / the scan beside the list launch, and that: 33 million tokens of one KV head, d = 32 33.6 / 30.7 / 29.1 + 32 us, 4 million, d = 128
        // 27.0 / 26.9 / 24.0 + 7.1; 2 KV heads of 8 million, d = 64 63.0 / 63.2 / 60.4 + 13.1; 4 of a million 21.4 / 21.2 / 22.4 + 5.6.)
        const int64_t stream = (int64_t)b * sh.Hkv + kvh;
        const uint64_t* const words = bf.page_mask + stream * sh.page_words;
        int32_t* const plist = bf.page_list + stream * (int64_t)sh.page_words * 64;
        constexpr int kThreads = kScanWaves * kWave, kGroups = 1024, kRounds = kGroups / kThreads, kParts = kGroups / kWave;
        __shared__ uint32_t group_at[kGroups], part_kept[kParts];           // pages kept in the groups before; per 64 groups
        __shared__ uint64_t group_word[kGroups];                            // first word of the group
        const int n_words = (int)((N + 64 * 64 - 1) / (64 * 64));           // (of the sequence, not of the cache's room)
        const int per_group = (n_words + kGroups - 1) / kGroups;
        const int n_groups = n_words > 0 ? (n_words + per_group - 1) / per_group : 0;
        const int top_step = n_groups > 1 ? 1 << (31 - __builtin_clz(n_groups - 1)) : 0;      // groups 0 .. 2 top_step - 1 are looked at
        const int n_rounds = top_step > kThreads / 2 ? 2 * top_step / kThreads : 1;
        uint32_t n_kept;
        {
            uint64_t first[kRounds];
#pragma unroll
            for (int u = 0; u < kRounds; ++u) {
                const int w0 = (u * kThreads + (int)threadIdx.x) * per_group;
                first[u] = w0 < n_words ? words[w0] : 0ull;
            }
#pragma unroll
            for (int u = 0; u < kRounds; ++u) {
                if (u >= n_rounds) break;                                   // (uniform)
                const int g = u * kThreads + (int)threadIdx.x;
                uint32_t cnt = (uint32_t)__popcll(first[u]);
                for (int i0 = 1; i0 < per_group; i0 += 8) {                 // (the last ones are asked for together too)
#pragma unroll
                    for (int i = i0; i < i0 + 8; ++i)
                        cnt += i < per_group && g * per_group + i < n_words ? (uint32_t)__popcll(words[g * per_group + i]) : 0u;
                }
                const uint32_t inc = wave_scan_add(cnt);
                if (lane == kWave - 1) part_kept[g / kWave] = inc;
                group_at[g] = inc - cnt;
                group_word[g] = first[u];
            }
            __syncthreads();
            static_assert(kParts <= kWave, "a lane per part");
            const uint32_t part = lane < n_rounds * kScanWaves ? part_kept[lane] : 0u;
            const uint32_t parts = wave_scan_add(part);
            n_kept = (uint32_t)__builtin_amdgcn_readlane((int)parts, kWave - 1);
#pragma unroll
            for (int u = 0; u < kRounds; ++u) {
                if (u >= n_rounds) break;
                group_at[u * kThreads + threadIdx.x] += (uint32_t)__builtin_amdgcn_readlane((int)(parts - part), u * kScanWaves + wave);
            }
            __syncthreads();
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) bf.page_cnt[stream] = n_kept;
        auto page_of = [&](uint32_t rank) -> int32_t {          // rank < n_kept
            int lo = 0;                                         // the last group that starts at or before the rank holds it
            for (int step = top_step; step > 0; step >>= 1)
                if (group_at[lo + step] <= rank) lo += step;
            uint32_t rest = rank - group_at[lo];
            uint64_t word = group_word[lo];
            int w = lo * per_group;
            if (per_group > 1) {                                // (uniform)
                const int end = w + per_group < n_words ? w + per_group : n_words;
                bool found = false;
                for (int w0 = w; w0 < end && !found; w0 += 8) {
                    uint64_t v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = w0 + i < end ? words[w0 + i] : 0ull;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const uint32_t c = (uint32_t)__popcll(v[i]);
                        const bool here = !found && rest < c;
                        word = here ? v[i] : word;
                        w = here ? w0 + i : w;
                        found |= here;
                        rest -= found ? 0u : c;
                    }
                }
            }
            // its rest-th set bit
            int bit = 0;
            uint32_t half = (uint32_t)word;
            uint32_t c = (uint32_t)__popc(half);
            if (rest >= c) { rest -= c; half = (uint32_t)(word >> 32); bit = 32; }
#pragma unroll
            for (int width = 16; width > 0; width >>= 1) {
                c = (uint32_t)__popc(half & ((1u << width) - 1u));
                if (rest >= c) { rest -= c; half >>= width; bit += width; }
            }
            return w * 64 + bit;
        };
        const int64_t rows = ((int64_t)n_kept + n_seg - 1) / n_seg;      // rows of n_seg ranks; the last one may be short
        int64_t base = 0;                        // first row of the current group of 64
        int32_t mine = 0;                        // lane i: page whose rank is this segment's in row base + i
        uint64_t m = 0ull;                       // rows of the group that hold a page for this segment, not yet taken
        auto look_up = [&]() {
            const int64_t i = base + lane;
            const int64_t r = seg_tile(i, sid, n_seg);
            const bool ok = i < rows && r < n_kept;
            mine = 0;
            if (ok) {
                mine = page_of((uint32_t)r);
                plist[r] = mine;
            }
            m = __ballot(ok);
        };
        if (rows > 0) look_up();
        auto next = [&]() -> int64_t {           // the wave's next tile to read, or -1 (wave-uniform)
            while (m == 0ull) {
                base += 64;
                if (base >= rows) return -1;
                look_up();
            }
            const int bit = __builtin_ctzll(m);
            m &= m - 1ull;
            return (int64_t)__builtin_amdgcn_readlane(mine, bit);
        };
        const int64_t past = (N + 63) / 64;      // (a tile of which nothing is read)
        if (rows > 0) {
            int64_t t0 = next();
            if (ScanPipelined<D>::value) {
                if (t0 >= 0) {
                    load_at(ba, t0);
                    while (true) {
                        const int64_t t1 = next();
                        load_at(bb, t1 >= 0 ? t1 : past);
                        __builtin_amdgcn_sched_barrier(0);
                        use(ba, t0);
                        if (t1 < 0) break;
                        const int64_t t2 = next();
                        load_at(ba, t2 >= 0 ? t2 : past);
                        __builtin_amdgcn_sched_barrier(0);
                        use(bb, t1);
                        if (t2 < 0) break;
                        t0 = t2;
                    }
                }
            } else {
                for (; t0 >= 0; t0 = next()) {
                    load_at(ba, t0);
                    __builtin_amdgcn_sched_barrier(0);
                    use(ba, t0);
                }
            }
        }
    } else {
        if (MODE == MODE_FULL) {
            walk_tiles<ScanPipelined<D>::value>(tile, tile_end, tile_step, ba, bb,
                [&](TileB& t, int64_t ti) { tile_load_at<DT, D>(Kh, ti, ti < tile_end ? N : 0, lane_off, t.b); }, use);
        }
    }
    if (MODE == MODE_FILTER) {
        if (!PAGED) {
            walk_tiles<ScanPipelined<D>::value, kAhead>(0, rows_mine, 1, ba, bb, load_seg,
                [&](TileB& t, int64_t i) { use(t, seg_tile(i, sid, n_seg)); });
        }
        stage_flush(cs0, seg_cap, n_seg, true);
        if (1 < G) stage_flush(cs1, seg_cap, n_seg, true);
        if (2 < G) stage_flush(cs2, seg_cap, n_seg, true);
        if (3 < G) stage_flush(cs3, seg_cap, n_seg, true);
        for (int o = 32; o > 0; o >>= 1) {
            top0 = fmaxf(top0, wave_xor(top0, o)); top1 = fmaxf(top1, wave_xor(top1, o));
            top2 = fmaxf(top2, wave_xor(top2, o)); top3 = fmaxf(top3, wave_xor(top3, o));
        }
        if (lane == 0) {
            uint32_t* sc = bf.seg_cnt + head0 * (int64_t)n_seg + sid;
            float* sx = bf.seg_max + head0 * (int64_t)n_seg + sid;
            sc[0] = (uint32_t)cs0.n_glob;
            sx[0] = top0;
            if (1 < G) { sc[n_seg] = (uint32_t)cs1.n_glob; sx[n_seg] = top1; }
            if (2 < G) { sc[2 * (int64_t)n_seg] = (uint32_t)cs2.n_glob; sx[2 * (int64_t)n_seg] = top2; }
            if (3 < G) { sc[3 * (int64_t)n_seg] = (uint32_t)cs3.n_glob; sx[3 * (int64_t)n_seg] = top3; }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < G * kTailBins; i += kScanWaves * kWave)
            bf.hist[((head0 + i / kTailBins) * sh.hist_cap + blockIdx.x) * kTailBins + i % kTailBins] = hist_lds[i];
    }
}

// ---------------------------------------------------------------------------------------
// Row-tile variant: up to 16 (32 with two row tiles) (query, head) rows against one KV head in a single pass over
// its keys -- head groups of 5..16, and several queries per sequence (a chunk of M
// queries, the cache-construction use the paper mentions for top-k attention).  Operand A
// holds 16 distinct rows, so the four accumulators of a 64-key tile give lane (j, n) the
// scores of rows 4 j + i (i = 0..3) for keys n, 16 + n, 32 + n, 48 + n: the same 16 MFMAs
// per tile as the grouped kernel, four times the rows.  Per-row state lives in the 16
// lanes that own the row.  A row's candidates are counted per score bin when they leave
// the row's LDS stage for its segment (the same counts the grouped kernel leaves).
// ---------------------------------------------------------------------------------------
// LDS staging slots per (wave, row): the 64 entries one step can add on top of the remainder (fewer than kCandChunk entries) an
// aligned flush leaves behind, and as many more as fit: one row tile and the scores' copy (FEW) leave room for 112 where two workgroups share a
// compute unit (4 queries over a million tokens, k = 16384: scan 372 us with 96, 363 with 112).  Two row tiles and the copy take as long with 96, 112
// and 118; 120 and 127 without the copy as long as 112.
template <int NT, bool FEW>
struct RowStage {
    static constexpr int value = FEW && NT == 2 ? 96 : 112;
    static_assert(kCandChunk <= 16 && value >= 64 + kCandChunk - 1 && value <= 127, "row stage too small for an aligned flush");
};

// NT row tiles (16 rows each) share every key tile: NT = 2 halves the passes over the keys for
// 17..32 rows at the price of one wave per SIMD (308 registers at d = 128) and 96 or 112 KiB of LDS stages,
// which costs this kernel nothing measurable.  (Four row tiles, with stages of 48 entries and two steps of two tiles, halve the
// passes again but pay it back at one wave per SIMD: 10 to 16 queries, d = 128, 150k tokens and more 0.95 - 1.01 of the time, below and at
// d = 64 1.0 - 1.13.)
// FEW (filter): few scores pass, they are staged one by one; otherwise every score has a store of its own (launch_scan_filter has the rule).
template <int DT, int D, int MODE, int NT, bool FEW = false>
__global__ void __launch_bounds__(kScanWaves* kWave)
__attribute__((amdgpu_waves_per_eu(NT == 1 || MODE == MODE_SAMPLE ? 2 : 1, MODE == MODE_SAMPLE ? 8 : NT == 1 ? 2 : 1)))
scan_rows_kernel(Shape sh, Bufs bf, int tiles_per_wave, float* dst) {
    using v8 = typename Mfma<DT>::v8;
    constexpr int KS = D / 32, kStageRow = RowStage<NT, FEW>::value;
    constexpr int X = 4 * NT;          // rows a lane owns: row 16 t + 4 j + i at x = 4 t + i
    const int G = sh.G, M = sh.M;
    // Workgroup -> (key stream bx of kv head kvh of cache sequence bc, row block blk).  With several
    // row blocks the blocks of one key stream take neighbouring slots of one XCD (workgroups go
    // to the XCDs round-robin by linear id), so they walk the same key tiles at the same time
    // and all but the first read of a tile are served by that XCD's L2.
    int bx = blockIdx.x, kvh = blockIdx.y, bc = (int)blockIdx.z / sh.n_qblk, blk = (int)blockIdx.z % sh.n_qblk;
    {
        const int gx = gridDim.x, gy = gridDim.y, streams = gx * gy * sh.Bc;
        if (sh.n_qblk > 1 && streams % 8 == 0) {
            const int lin = bx + gx * (kvh + gy * (int)blockIdx.z);
            const int slot = lin >> 3, stream = (slot / sh.n_qblk) * 8 + (lin & 7);
            blk = slot % sh.n_qblk;
            bx = stream % gx;
            kvh = (stream / gx) % gy;
            bc = stream / (gx * gy);
        }
    }
    // the M * G (query, head) rows of the KV head, query-major, are cut into blocks of 16 NT rows
    const int row0 = blk * 16 * NT;                                   // first row of the block
    const int R = M * G - row0 < 16 * NT ? M * G - row0 : 16 * NT;    // its rows
    const int lane = lane_id();
    const int j = lane >> 4, n = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t Nc = bf.len[bc];
    const int64_t N = prefix_len(Nc, sh.window);      // longest searched prefix of the sequence's queries

    // row rr of the block is head kvh * G + (row0 + rr) % G of query (row0 + rr) / G
    auto head_of = [&](int rr) -> int64_t {
        return ((int64_t)bc * M + (row0 + rr) / G) * sh.Hq + (int64_t)kvh * G + (row0 + rr) % G;
    };
    // candidates per score bin (tail_bin()) of each row, counted as they leave the stage
    __shared__ uint32_t hist_lds[MODE == MODE_FILTER ? 16 * NT * kTailBins : 1];
    auto prefix_of = [&](int rr) -> int {   // keys row rr searches (0 for rows the block does not have)
        if (rr >= R) return 0;
        const int m = (row0 + rr) / G;
        return (int)prefix_len(Nc - (sh.causal ? M - 1 - m : 0), sh.window);
    };
    // filter: what a row's lanes need to know of it, worked out once (a division per row and lane was half the prologue)
    struct Row { float thr, bin_lo, bin_inv; int prefix, head; };
    __shared__ Row row_lds[MODE == MODE_FILTER ? 16 * NT : 1];
    __shared__ uint32_t count_lds[MODE == MODE_FILTER ? kScanWaves * 16 * NT : 1];   // candidates appended so far, per wave and row

    int64_t n_items = N;
    int stride = 1;
    if (MODE == MODE_SAMPLE) {
        if (N == 0) return;
        Plan pl = make_plan(N, sh.k < N ? sh.k : (int)N);
        n_items = pl.n_samp;
        stride = pl.stride;
    }
    const int64_t n_tiles_all = (n_items + 63) / 64;
    int64_t tile, tile_end, tile_step;
    if (MODE == MODE_FILTER) {
        tile = 0;                           // (the filter's walk counts rows of n_seg tiles)
        tile_step = 1;
        tile_end = 0;
    } else {
        const int64_t tile0 = (int64_t)bx * tiles_per_wave * kScanWaves;
        if (tile0 >= n_tiles_all) return;
        tile = tile0 + wave;
        tile_step = kScanWaves;
        tile_end = tile0 + (int64_t)tiles_per_wave * kScanWaves;
        if (tile_end > n_tiles_all) tile_end = n_tiles_all;
    }

    // operand A of row tile t: lane (j, m) holds channels 32 s + 8 j .. +7 of row 16 t + m
    v8 qa[NT][KS];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int rr = 16 * t + n;
        const v8* p = reinterpret_cast<const v8*>(static_cast<const char*>(bf.q) + head_of(rr < R ? rr : 0) * (D * 2)) + j;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            v8 v = p[4 * s];
            if (rr >= R) v = v8{};
            qa[t][s] = v;
        }
    }
    const char* Kh = static_cast<const char*>(bf.K) + ((int64_t)bc * sh.Hkv + kvh) * sh.Ncap * (D * 2);

    // filter: one tile per row of n_seg tiles (seg_tile()); the first is asked for ahead of the rows' thresholds
    const int seg_cap = sh.seg_cap, n_seg = sh.n_seg;
    const int sid = bx * kScanWaves + wave;
    struct TileB { v8 b[4][KS]; } ba, bb;
    const LaneOffsets lane_off = lane_offsets<D>();
    constexpr bool kAhead = MODE == MODE_FILTER && ScanPipelined<D>::value;
    const int64_t rows_mine = MODE == MODE_FILTER ? seg_rows(n_tiles_all, sid, n_seg) : 0;
    auto load_seg = [&](TileB& t, int64_t i) { tile_load_at<DT, D>(Kh, seg_tile(i, sid, n_seg), N, lane_off, t.b); };
    if (MODE == MODE_FILTER) {
        auto row_of_block = [&](int rr) -> Row {
            const int64_t head = head_of(rr < R ? rr : 0);
            return Row{rr < R ? bf.thr[head] : INFINITY, bf.bins[2 * head], bf.bins[2 * head + 1], prefix_of(rr), (int)head};
        };
        auto clear = [&]() {
            for (int i = threadIdx.x; i < 16 * NT * kTailBins; i += kScanWaves * kWave) hist_lds[i] = 0;
            for (int i = threadIdx.x; i < kScanWaves * 16 * NT; i += kScanWaves * kWave) count_lds[i] = 0;
        };
        // One row tile, two waves per SIMD: the tile first, the barrier waits for it.  (The other way 15 shapes, 2 to 4 queries or 5 to 16 heads per
        // KV head, 27k to a million tokens, take 0.994 - 1.019 times as long, 1.006 in the geometric mean: 4 queries over a million tokens 523 us per call
        // and 526, over 524k 290 and 294, 64 heads over 33k 40.6 and 41.4.)  Two row tiles, one wave per SIMD: the rows' loads first, as loads return in order, and a barrier that does not wait for the
        // tile (16 queries of 128k tokens 144.4, 145.9 the other way; 8 queries of 262k 175.9 and 177.5).
        if constexpr (NT == 1) {
            if (kAhead && rows_mine > 0) {
                load_seg(ba, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            clear();
            if (threadIdx.x < 16 * NT) row_lds[threadIdx.x] = row_of_block(threadIdx.x);
            __syncthreads();
        } else {
            const Row row = row_of_block(threadIdx.x < 16 * NT ? threadIdx.x : 0);
            __builtin_amdgcn_sched_barrier(0);
            if (kAhead) load_seg(ba, 0);        // (without a tile for this wave it reads nothing)
            __builtin_amdgcn_sched_barrier(0);
            clear();
            if (threadIdx.x < 16 * NT) row_lds[threadIdx.x] = row;
            lds_barrier();
        }
    }

    // the rows this lane owns
    auto row_at = [&](int x) { return 16 * (x >> 2) + 4 * j + (x & 3); };
    constexpr int XS = MODE == MODE_FILTER ? 1 : X;
    int vh[XS], P[XS];      // sample, full: head (a 32-bit index: heads are few) and prefix of each row
    float thr[X], top[X];   // filter
    uint32_t staged[NT];    // staged candidates of the four rows of a row tile, a byte each (uniform over the 16 lanes of the rows)
#pragma unroll
    for (int t = 0; t < NT; ++t) staged[t] = 0;
#pragma unroll
    for (int x = 0; x < X; ++x) {
        const int rr = row_at(x);
        if constexpr (MODE == MODE_FILTER) {
            thr[x] = row_lds[rr].thr;
            top[x] = -INFINITY;
        } else {
            vh[x] = (int)head_of(rr < R ? rr : 0);
            P[x] = prefix_of(rr);
        }
    }
    __shared__ uint64_t stage_lds[MODE == MODE_FILTER ? kScanWaves * 16 * NT * kStageRow : 1];
    uint64_t* const st0 = stage_lds + (MODE == MODE_FILTER ? wave * 16 * NT * kStageRow : 0);

    uint32_t* const count = count_lds + (MODE == MODE_FILTER ? wave * 16 * NT : 0);
    // append the staged candidates of the rows at x (one per lane group) to their segments, up to
    // the last whole run of kCandChunk entries unless `final` (see stage_flush); returns how many stay
    auto flush = [&](int x, int n_staged, bool final) -> int {
        wave_sync();
        const int rr = row_at(x);
        uint64_t* list = bf.cand + row_lds[rr].head * (int64_t)sh.cand_cap;
        uint64_t* src = st0 + rr * kStageRow;
        const int n_glob = (int)count[rr];
        const int total = n_glob + n_staged;
        const int f = (final ? total : (total & ~(kCandChunk - 1))) - n_glob;
        const float bin_lo = row_lds[rr].bin_lo, bin_inv = row_lds[rr].bin_inv;
        uint32_t* const hist = hist_lds + rr * kTailBins;
        for (int e = n; e < f; e += 16) {
            const int slot = n_glob + e;
            const uint64_t ent = src[e];
            if (slot < seg_cap) list[cand_slot(slot, sid, n_seg)] = ent;
            atomicAdd(&hist[tail_bin(__uint_as_float((uint32_t)(ent >> 32)), bin_lo, bin_inv)], 1u);   // also past a full segment
        }
        const int r = f > 0 ? n_staged - f : n_staged;  // < kCandChunk <= 16 after a flush
        const bool mv = f > 0 && n < r;
        const uint64_t keep = mv ? src[f + n] : 0;
        wave_sync();
        if (mv) src[n] = keep;
        if (f > 0) count[rr] = (uint32_t)(n_glob + f);  // (the same from all 16 lanes)
        wave_sync();
        return r;
    };
    // Rows of the row tile t: those whose stage cannot take `add` more entries (a byte each), or all at the end.  (A loop: the
    // code of all rows in line, and their heads and counts, would take the registers of the tile loop.)
    auto flush_rows = [&](int t, uint32_t& have, uint32_t add, bool final) __attribute__((always_inline)) {
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {
            const int n_staged = (int)((have >> (8 * i)) & 0xFFu);
            const bool want = final || n_staged + (int)((add >> (8 * i)) & 0xFFu) > kStageRow;
            if (!__ballot(want)) continue;
            have -= (uint32_t)(n_staged - flush(4 * t + i, n_staged, final)) << (8 * i);
        }
    };

    auto sample_row = [&](int64_t item) -> int64_t {        // key row of a sample (beyond the last one: the last one's)
        const int64_t p = sample_pos((int)(item < n_items ? item : n_items - 1), stride);
        return p < N ? p : N - 1;
    };
    // Filter step of a tile.  A lane gathers which of its (row, sub-tile) scores pass in one
    // mask (bit 16 t + 4 i + g), the counts of the four rows of a row tile share a register (a byte each: a row has at most 64
    // passing keys per tile), and one inclusive scan over the 16 lanes of the rows (four DPP row shifts) ranks all of
    // them at once.  Staged order within a row: by lane, then sub-tile (the selection does not depend on it).
    // FEW: those that pass (one per lane for k = N / 64) are taken bit by bit from a copy of the scores in LDS, which can be
    // indexed by lane as registers cannot.  Otherwise a store per score, from its register and under its bit.
    // What bounds it is instructions (one or two waves per SIMD hide little): a store per score, to a scratch slot for those that do not
    // pass, took 18 per score.  Whole call, that way / now, few: 17 queries of 241k tokens, d = 64 275 / 240 us, 32 queries of 27k 84.5 / 80.2,
    // 4 queries of 60k 53.5 / 49.2, 64 heads over 111k tokens 68.9 / 65.0; 16 queries of 128k, d = 128, whose keys come at the rate of the
    // L1, 148 / 146.  A third of the keys selected, that way / taken from the mask / now: 8 queries of 200k, d = 64 430 / 456 / 425; 16 queries of 30k,
    // d = 128 191.5 / 199.3 / 190.8.
    const int Pmin = prefix_of(0);      // rows of a block search prefixes that grow with the row
    __shared__ f32x4 score_lds[MODE == MODE_FILTER && FEW ? kScanWaves * NT * 4 * kWave : 1];
    f32x4* const my_scores = score_lds + (MODE == MODE_FILTER && FEW ? wave * NT * 4 * kWave + lane : 0);
    auto filter = [&](f32x4 (&c)[NT][4], int64_t item0) __attribute__((always_inline)) {
        const int item_n = (int)item0 + n;              // positions fit 31 bits
        if (item0 + 64 > Pmin) {                        // (uniform) scores beyond a row's prefix become NaN, which no threshold lets through
#pragma unroll
            for (int x = 0; x < X; ++x) {
                const int Px = row_lds[row_at(x)].prefix;
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    if (item_n + 16 * g >= Px) c[x >> 2][g][x & 3] = NAN;
            }
        }
        uint32_t mask = 0;
#pragma unroll
        for (int x = X - 1; x >= 0; --x) {
#pragma unroll
            for (int g = 3; g >= 0; --g) mask = mask + mask + (c[x >> 2][g][x & 3] >= thr[x] ? 1u : 0u);
#pragma unroll
            for (int g = 0; g < 4; ++g) top[x] = fmaxf(top[x], c[x >> 2][g][x & 3]);
        }
        if (!__ballot(mask != 0u)) return;              // (uniform) nothing passes anywhere in the tile
        if constexpr (FEW) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int g = 0; g < 4; ++g) my_scores[(t * 4 + g) * kWave] = c[t][g];
            }
        }
        uint32_t incl[NT], pk[NT], tot[NT];
        uint32_t nib = mask - ((mask >> 1) & 0x55555555u);
        nib = (nib & 0x33333333u) + ((nib >> 2) & 0x33333333u);       // passing scores per row, four bits each
        bool over = false;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            uint32_t v = (nib >> (16 * t)) & 0xFFFFu;
            v = (v | (v << 8)) & 0x00FF00FFu;
            v = (v | (v << 4)) & 0x0F0F0F0Fu;
            pk[t] = v;
            v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);   // row_shr:1
            v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);   // row_shr:2
            v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);   // row_shr:4
            v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);   // row_shr:8
            incl[t] = v;
            tot[t] = (uint32_t)__builtin_amdgcn_ds_bpermute((lane | 15) << 2, (int)v);      // the group's last lane
            // a byte beyond kStageRow sets its top bit (at most kStageRow + 64 + 127 - kStageRow = 191)
            over |= ((staged[t] + tot[t] + 0x01010101u * (uint32_t)(127 - kStageRow)) & 0x80808080u) != 0u;
        }
        if (__builtin_expect(__ballot(over) != 0, 0)) {
#pragma unroll
            for (int t = 0; t < NT; ++t) flush_rows(t, staged[t], tot[t], false);
        }
        // where a lane's first passing score of each row goes (bytes of staged + incl are >= those of pk: no borrows)
        uint64_t at = staged[0] + incl[0] - pk[0];
        if (NT > 1) at |= (uint64_t)(staged[NT - 1] + incl[NT - 1] - pk[NT - 1]) << 32;
#pragma unroll
        for (int t = 0; t < NT; ++t) staged[t] += tot[t];
        if constexpr (!FEW) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const uint32_t to = (uint32_t)(at >> (32 * t));
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint64_t* where = st0 + row_at(4 * t + i) * kStageRow + ((to >> (8 * i)) & 0xFFu);
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const bool pass = (mask >> (16 * t + 4 * i + g)) & 1u;
                        if (pass) *where = ((uint64_t)__float_as_uint(c[t][g][i] + 0.0f) << 32) | (uint64_t)(uint32_t)(item_n + 16 * g);
                        where += pass ? 1 : 0;
                    }
                }
            }
            return;
        }
        // two at a time: their reads of the scores share a trip
        while (mask) {
            const int b0 = __builtin_ctz(mask);
            mask &= mask - 1u;
            const bool two = mask != 0u;
            const int b1 = two ? __builtin_ctz(mask) : b0;
            mask &= mask - 1u;                                        // (0 stays 0)
            const float* const my = reinterpret_cast<const float*>(my_scores);
            const float s0 = my[((b0 >> 2 & 4) + (b0 & 3)) * (kWave * 4) + (b0 >> 2 & 3)], s1 = my[((b1 >> 2 & 4) + (b1 & 3)) * (kWave * 4) + (b1 >> 2 & 3)];
            auto put = [&](int b, float v) __attribute__((always_inline)) {
                const int x = b >> 2;                                 // 4 t + i
                const int o = (int)((uint32_t)(at >> (8 * x)) & 0xFFu);
                at += 1ull << (8 * x);
                st0[row_at(x) * kStageRow + o] = ((uint64_t)__float_as_uint(v + 0.0f) << 32) | (uint64_t)(uint32_t)(item_n + 16 * (b & 3));
            };
            put(b0, s0);
            if (two) put(b1, s1);
        }
    };
    auto consume = [&](f32x4 (&c)[NT][4], int64_t item0) __attribute__((always_inline)) {
        if (MODE == MODE_SAMPLE) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int64_t item = item0 + 16 * g + n;
                if (item < n_items) {
                    const int64_t pos = sample_pos((int)item, stride);
#pragma unroll
                    for (int x = 0; x < X; ++x)   // a sample past the row's own prefix does not count
                        if (row_at(x) < R)
                            bf.samp[(int64_t)vh[x] * sh.samp_cap + item] = pos < P[x] ? c[x >> 2][g][x & 3] : -INFINITY;
                }
            }
        } else if (MODE == MODE_FULL) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int64_t item = item0 + 16 * g + n;
#pragma unroll
                for (int x = 0; x < X; ++x)
                    if (item < P[x]) dst[(int64_t)vh[x] * sh.Ncap + item] = c[x >> 2][g][x & 3];
            }
        } else {
            filter(c, item0);
        }
    };
    auto mac = [&](const v8 (&b)[4][KS], f32x4 (&c)[NT][4]) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                c[t][g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < KS; ++s) c[t][g] = Mfma<DT>::mac(qa[t][s], b[g][s], c[t][g]);
            }
        }
    };

    auto load_sample = [&](TileB& t, int64_t ti) { tile_load<DT, D>(Kh, [&](int slot) { return sample_row(ti * 64 + slot); }, t.b); };
    auto use = [&](TileB& t, int64_t ti) __attribute__((always_inline)) {
        f32x4 c[NT][4];
        mac(t.b, c);
        consume(c, ti * 64);
    };
    if (MODE == MODE_SAMPLE) {
        walk_tiles<false>(tile, tile_end, tile_step, ba, bb, load_sample, use);
    } else if (MODE == MODE_FILTER) {
        walk_tiles<ScanPipelined<D>::value, kAhead>(0, rows_mine, 1, ba, bb, load_seg,
            [&](TileB& t, int64_t i) __attribute__((always_inline)) { use(t, seg_tile(i, sid, n_seg)); });
    } else {
        walk_tiles<ScanPipelined<D>::value>(tile, tile_end, tile_step, ba, bb,
            [&](TileB& t, int64_t ti) { tile_load_at<DT, D>(Kh, ti, ti < tile_end ? N : 0, lane_off, t.b); }, use);
    }
    if (MODE == MODE_FILTER) {
#pragma unroll
        for (int t = 0; t < NT; ++t) flush_rows(t, staged[t], 0u, true);
#pragma unroll
        for (int i = 0; i < X; ++i) {
            const int rr = row_at(i);
            for (int o = 8; o > 0; o >>= 1) top[i] = fmaxf(top[i], wave_xor(top[i], o));
            if (n == 0 && rr < R) {
                const int64_t head = row_lds[rr].head;
                bf.seg_cnt[head * n_seg + sid] = count[rr];
                bf.seg_max[head * n_seg + sid] = top[i];
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < R * kTailBins; i += kScanWaves * kWave)
            bf.hist[((int64_t)row_lds[i / kTailBins].head * sh.hist_cap + bx) * kTailBins + i % kTailBins] = hist_lds[i];
    }
}

// Plain FMA scoring of fp32 caches: a row of D elements is spread over D / 4 lanes, 16 bytes each, U rows per lane group
// with all loads under way before the query is staged.  Few rows are a chain of latencies (one head, 4096 rows: sixteen
// workgroups that took their rows one after the other 11.4 us, a workgroup per 16 rows 3.0; 8 heads,
// 16k tokens, d = 128 31.9 -> 5.3).
template <int D, int U>
__global__ void __launch_bounds__(256)
scan_f32_kernel(Shape sh, Bufs bf, float* dst) {
    fetch_args<kArgBytes>();
    constexpr int LPR = D / 4, RPP = 256 / LPR;            // lanes per row, rows per pass of the workgroup
    const int b = blockIdx.z, kvh = blockIdx.y;
    const int G = sh.G;
    const int64_t head0 = (int64_t)b * sh.Hq + (int64_t)kvh * G;
    const int64_t N = prefix_len(visible_len(sh, bf, b), sh.window);
    const int64_t row0 = (int64_t)blockIdx.x * (RPP * U) + threadIdx.x / LPR;
    if ((int64_t)blockIdx.x * (RPP * U) >= N) return;
    const int c = threadIdx.x % LPR;
    const float* Kh = static_cast<const float*>(bf.K) + ((int64_t)cache_seq(sh, b) * sh.Hkv + kvh) * sh.Ncap * D + c * 4;
    f32x4 k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t r = row0 + u * RPP;
        k[u] = *reinterpret_cast<const f32x4*>(Kh + (r < N ? r : N - 1) * D);
    }
    __shared__ __align__(16) float q_lds[16 * 256];
    for (int i = threadIdx.x; i < G * D; i += 256) q_lds[i] = static_cast<const float*>(bf.q)[head0 * D + i];
    __syncthreads();
    for (int h = 0; h < G; ++h) {
        const f32x4 q = *reinterpret_cast<const f32x4*>(q_lds + h * D + c * 4);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float acc = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = fmaf(k[u][e], q[e], acc);
            acc = group_reduce<AddOp, LPR>(acc);
            const int64_t r = row0 + u * RPP;
            if (r < N && c == 0) dst[(head0 + h) * sh.Ncap + r] = acc;
        }
    }
}

template <int D>
static void launch_scan_f32(const Shape& s, const Bufs& b, int64_t Nmax, float* dst, hipStream_t st) {
    // four rows per lane group once the chip is full of workgroups with one (whole call, one row against four: 8 KV heads, 32k to 200k
    // tokens 1.02 - 1.15 times as long for 8 query heads, 1.03 - 1.41 for 32, most at d = 256; calls of few workgroups are bound by the host)
    constexpr int64_t kRowsPerPass = 256 / (D / 4);
    const int64_t passes = (Nmax + kRowsPerPass - 1) / kRowsPerPass;
    if (passes * s.Hkv * s.B <= 1024)
        hipLaunchKernelGGL((scan_f32_kernel<D, 1>), dim3((unsigned)passes, (unsigned)s.Hkv, (unsigned)s.B), dim3(256), 0, st, s, b, dst);
    else
        hipLaunchKernelGGL((scan_f32_kernel<D, 4>), dim3((unsigned)((passes + 3) / 4), (unsigned)s.Hkv, (unsigned)s.B), dim3(256), 0, st, s, b, dst);
}

bool scan_mfma_supported(const Shape& s) {
    return (s.dtype == DT_F16 || s.dtype == DT_BF16) && (s.D == 32 || s.D == 64 || s.D == 128 || s.D == 256) && s.G >= 1;
}

template <int MODE>
static hipError_t launch_mfma(const Shape& s, const Bufs& b, int64_t n_items, float* dst, hipStream_t st) {
    const bool rows = scan_row_tiles(s);
    const int tpw = tiles_per_wave_for(n_items, scan_grid_z(s), s.Hkv);
    const int64_t tiles = (n_items + 63) / 64;
    const int64_t per_wg = (int64_t)tpw * kScanWaves;
    dim3 grid((unsigned)((tiles + per_wg - 1) / per_wg), (unsigned)s.Hkv, (unsigned)(scan_grid_z(s)));
    dim3 block(kScanWaves * kWave);
#define TKA_LAUNCH(DT_, D_)                                                                                 \
    do {                                                                                                    \
        if (rows && s.row_tiles == 2)                                                                       \
            hipLaunchKernelGGL((scan_rows_kernel<DT_, D_, MODE, 2>), grid, block, 0, st, s, b, tpw, dst);   \
        else if (rows)                                                                                      \
            hipLaunchKernelGGL((scan_rows_kernel<DT_, D_, MODE, 1>), grid, block, 0, st, s, b, tpw, dst);   \
        else hipLaunchKernelGGL((scan_mfma_kernel<DT_, D_, MODE>), grid, block, 0, st, s, b, tpw, dst);     \
    } while (0)
    if (s.dtype == DT_F16 && s.D == 128) TKA_LAUNCH(DT_F16, 128);
    else if (s.dtype == DT_F16 && s.D == 64) TKA_LAUNCH(DT_F16, 64);
    else if (s.dtype == DT_BF16 && s.D == 128) TKA_LAUNCH(DT_BF16, 128);
    else if (s.dtype == DT_BF16 && s.D == 64) TKA_LAUNCH(DT_BF16, 64);
    else if (s.dtype == DT_F16 && s.D == 256) TKA_LAUNCH(DT_F16, 256);
    else if (s.dtype == DT_BF16 && s.D == 256) TKA_LAUNCH(DT_BF16, 256);
    else if (s.dtype == DT_F16 && s.D == 32) TKA_LAUNCH(DT_F16, 32);
    else if (s.dtype == DT_BF16 && s.D == 32) TKA_LAUNCH(DT_BF16, 32);
    else return hipErrorInvalidValue;
#undef TKA_LAUNCH
    return hipGetLastError();
}

hipError_t launch_scan_sample(const Shape& s, const Bufs& b, int64_t Nmax, hipStream_t st) {
    Plan pl = make_plan(Nmax, s.k);
    return launch_mfma<MODE_SAMPLE>(s, b, pl.n_samp, nullptr, st);
}

hipError_t launch_scan_filter_paged(const Shape& s, const Bufs& b, hipStream_t st) {
    if (scan_row_tiles(s)) return hipErrorInvalidValue;      // grouped scan only
    dim3 grid((unsigned)(s.n_seg / kScanWaves), (unsigned)s.Hkv, (unsigned)s.B);
    dim3 block(kScanWaves * kWave);
#define TKA_LAUNCH(DT_, D_) \
    hipLaunchKernelGGL((scan_mfma_kernel<DT_, D_, MODE_FILTER, true>), grid, block, 0, st, s, b, 0, (float*)nullptr)
    if (s.dtype == DT_F16 && s.D == 128) TKA_LAUNCH(DT_F16, 128);
    else if (s.dtype == DT_F16 && s.D == 64) TKA_LAUNCH(DT_F16, 64);
    else if (s.dtype == DT_BF16 && s.D == 128) TKA_LAUNCH(DT_BF16, 128);
    else if (s.dtype == DT_BF16 && s.D == 64) TKA_LAUNCH(DT_BF16, 64);
    else if (s.dtype == DT_F16 && s.D == 256) TKA_LAUNCH(DT_F16, 256);
    else if (s.dtype == DT_BF16 && s.D == 256) TKA_LAUNCH(DT_BF16, 256);
    else if (s.dtype == DT_F16 && s.D == 32) TKA_LAUNCH(DT_F16, 32);
    else if (s.dtype == DT_BF16 && s.D == 32) TKA_LAUNCH(DT_BF16, 32);
    else return hipErrorInvalidValue;
#undef TKA_LAUNCH
    return hipGetLastError();
}

hipError_t launch_scan_filter(const Shape& s, const Bufs& b, int64_t Nmax, hipStream_t st) {
    const bool sampled = threshold_in_scan(s, Nmax);
    // one wave per candidate segment: n_seg / 4 workgroups per KV head.  (Also where several layers share the launch: with as many
    // workgroups as run at once, which took the segments one after the other, 8 layers of 48k tokens 216 us per call, 209 like this; and the
    // loop around the walk cost other calls too, 3 ragged sequences of 98k 137 and 128.)
    const bool rows = scan_row_tiles(s);
    // how the row-tile scan stages what passes (scan_rows_kernel, FEW).  Whole call, a store per score / scores taken from the mask, by keys per selected key:
    // 128 0.99 - 1.03 (median 1.00), 64 0.98 - 1.02 (1.00), 32 0.96 - 1.01 (0.98), 10 0.91 - 1.00 (0.97), 4 0.89 - 1.00 (0.95); most with two row
    // tiles and small head_dim.  (2 to 16 queries over 30k to 400k tokens, d = 32 to 256.)
    const bool few = (int64_t)s.k * 48 < Nmax;
    dim3 grid((unsigned)(s.n_seg / kScanWaves), (unsigned)s.Hkv, (unsigned)(scan_grid_z(s)));
    dim3 block(kScanWaves * kWave);
#define TKA_LAUNCH(DT_, D_)                                                                                  \
    do {                                                                                                     \
        if (rows && few && s.row_tiles == 2)                                                                 \
            hipLaunchKernelGGL((scan_rows_kernel<DT_, D_, MODE_FILTER, 2, true>), grid, block, 0, st, s, b, 0, \
                               (float*)nullptr);                                                             \
        else if (rows && few)                                                                                \
            hipLaunchKernelGGL((scan_rows_kernel<DT_, D_, MODE_FILTER, 1, true>), grid, block, 0, st, s, b, 0, \
                               (float*)nullptr);                                                             \
        else if (rows && s.row_tiles == 2)                                                                   \
            hipLaunchKernelGGL((scan_rows_kernel<DT_, D_, MODE_FILTER, 2>), grid, block, 0, st, s, b, 0,     \
                               (float*)nullptr);                                                             \
        else if (rows)                                                                                       \
            hipLaunchKernelGGL((scan_rows_kernel<DT_, D_, MODE_FILTER, 1>), grid, block, 0, st, s, b, 0,     \
                               (float*)nullptr);                                                             \
        else if (sampled)                                                                                    \
            hipLaunchKernelGGL((scan_mfma_kernel<DT_, D_, MODE_FILTER, false, (D_ < 256)>), grid, block, 0, st, s, \
                               b, 0, (float*)nullptr);                                                       \
        else                                                                                                 \
            hipLaunchKernelGGL((scan_mfma_kernel<DT_, D_, MODE_FILTER>), grid, block, 0, st, s, b, 0,        \
                               (float*)nullptr);                                                             \
    } while (0)
    if (s.dtype == DT_F16 && s.D == 128) TKA_LAUNCH(DT_F16, 128);
    else if (s.dtype == DT_F16 && s.D == 64) TKA_LAUNCH(DT_F16, 64);
    else if (s.dtype == DT_BF16 && s.D == 128) TKA_LAUNCH(DT_BF16, 128);
    else if (s.dtype == DT_BF16 && s.D == 64) TKA_LAUNCH(DT_BF16, 64);
    else if (s.dtype == DT_F16 && s.D == 256) TKA_LAUNCH(DT_F16, 256);
    else if (s.dtype == DT_BF16 && s.D == 256) TKA_LAUNCH(DT_BF16, 256);
    else if (s.dtype == DT_F16 && s.D == 32) TKA_LAUNCH(DT_F16, 32);
    else if (s.dtype == DT_BF16 && s.D == 32) TKA_LAUNCH(DT_BF16, 32);
    else return hipErrorInvalidValue;
#undef TKA_LAUNCH
    return hipGetLastError();
}

hipError_t launch_scan_full(const Shape& s, const Bufs& b, int64_t Nmax, float* dst, hipStream_t st) {
    if (scan_mfma_supported(s)) return launch_mfma<MODE_FULL>(s, b, Nmax, dst, st);
    if (s.D == 64) launch_scan_f32<64>(s, b, Nmax, dst, st);
    else if (s.D == 128) launch_scan_f32<128>(s, b, Nmax, dst, st);
    else if (s.D == 256) launch_scan_f32<256>(s, b, Nmax, dst, st);
    else if (s.D == 32) launch_scan_f32<32>(s, b, Nmax, dst, st);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace tka

// MFMA tile routines of the key scan over 16-bit keys: operand layouts, tile loads, the
// double-buffered tile walk and the per-tile contraction (used by scan.hip and by the exact
// rescoring in tail.hip).
#pragma once
#include "device_utils.h"
#include "internal.h"

namespace tka {

template <int DT> struct Mfma;
template <> struct Mfma<DT_F16> {
    using v8 = f16x8;
    static __device__ __forceinline__ f32x4 mac(v8 a, v8 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
};
template <> struct Mfma<DT_BF16> {
    using v8 = bf16x8;
    static __device__ __forceinline__ f32x4 mac(v8 a, v8 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};

// Query block of the group in operand-A layout: lane (j, m) holds channels
// 32 s + 8 j .. +7 of head m % 4 (zero for heads the group does not have).
template <int DT, int D>
__device__ __forceinline__ void load_query_a(const void* q, int64_t head0, int G,
                                             typename Mfma<DT>::v8 (&qa)[D / 32]) {
    using v8 = typename Mfma<DT>::v8;
    const int lane = lane_id();
    const int j = lane >> 4, r = lane & 3;
    const v8* p = reinterpret_cast<const v8*>(static_cast<const char*>(q) + (head0 + (r < G ? r : 0)) * D * 2) + j;
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
        v8 v = p[4 * s];
        if (r >= G) v = v8{};
        qa[s] = v;
    }
}

// Operand B of a 64-key tile: for each 16-key sub-tile g, lane (j, n) loads the 16-byte
// chunks 4 s + j (s = 0 .. D/32-1) of the row rowfn(16 g + n).  All loads are issued
// before anything consumes them.
template <int DT, int D, class RowFn>
__device__ __forceinline__ void tile_load(const char* Kh, RowFn rowfn, typename Mfma<DT>::v8 (&b)[4][D / 32]) {
    using v8 = typename Mfma<DT>::v8;
    constexpr int KS = D / 32;
    const int lane = lane_id();
    const int j = lane >> 4, n = lane & 15;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int64_t row = rowfn(16 * g + n);
        const v8* p = reinterpret_cast<const v8*>(Kh + row * (D * 2)) + j;
#pragma unroll
        for (int s = 0; s < KS; ++s) b[g][s] = p[4 * s];
    }
}

// Rows of a tile, 0 .. 64, of the n_rows (wave-uniform) there are from its first one on.
__device__ __forceinline__ uint32_t bounded_rows(int n_rows) {
    // (two steps: a clamp to a range is a vector instruction, and a descriptor from there a loop over the lanes)
    const int have = __builtin_amdgcn_readfirstlane(n_rows);
    uint32_t rows = (uint32_t)(have < 0 ? 0 : have);
    asm("" : "+s"(rows));
    return rows > 64u ? 64u : rows;
}

// tile_load() for `n_rows` consecutive rows (64 for a whole tile), through buffer loads: the tile's address
// (wave-uniform) sits in a scalar buffer descriptor and a lane's byte offsets of the four 16-row sub-tiles are
// loop-invariant, so the loop holds no per-lane address arithmetic at all.  (With per-lane 64-bit addresses the compiler
// builds them in registers of the buffer it is about to refill and then waits for every
// outstanding load before it may overwrite them, which serialises every other prefetch.)
// The descriptor ends behind the rows there are: what lies beyond reads as zero and is not fetched, so the tile that the end of the
// cache cuts short is walked like the others, and a prefetch past the last tile (n_rows <= 0) costs nothing.  (The whole
// offset is in the lane's register and the instruction, which are what the range check looks at; a scalar offset need not be.)
// Whole call, cut-short tile in a round of its own and a tile read again at the end / now: 16k tokens, where a wave has one tile,
// 23.4 / 21.0 us, 8 layers of 48001 tokens (three tiles a wave) 207.7 / 197.3, 192 sequences of 2k to 4k tokens 308.9 / 300.3.
struct LaneOffsets { uint32_t g[4]; };
template <int D>
__device__ __forceinline__ LaneOffsets lane_offsets() {
    LaneOffsets o;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        o.g[g] = (uint32_t)(((16 * g + (lane_id() & 15)) * D + (lane_id() >> 4) * 8) * 2);
        asm volatile("" : "+v"(o.g[g]));      // (four registers; the chunks of a row are the instruction's own offset)
    }
    return o;
}
template <int DT, int D>
__device__ __forceinline__ void tile_load_rows(const char* tile_base, int n_rows, const LaneOffsets& off,
                                               typename Mfma<DT>::v8 (&b)[4][D / 32]) {
    using v8 = typename Mfma<DT>::v8;
    constexpr int KS = D / 32;
    const uint32_t rows = bounded_rows(n_rows);
    // raw buffer (stride 0), rows * D * 2 bytes long, 32-bit data format
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(tile_base), 0, (int)rows * (D * 2), 0x00020000);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off.g[g] + 64 * s, 0, 0);
            b[g][s] = __builtin_bit_cast(v8, v);
        }
    }
}
// Tile `tile` of a stream of N rows.  (A cache has at most 0x7FFFFF00 of them, and no walk asks for a tile whose first row lies further
// than that from row N: the difference, and minus the first row of a tile up to three past the end, fit an int.)
template <int DT, int D>
__device__ __forceinline__ void tile_load_at(const char* Kh, int64_t tile, int64_t N, const LaneOffsets& off,
                                             typename Mfma<DT>::v8 (&b)[4][D / 32]) {
    tile_load_rows<DT, D>(Kh + tile * (64 * D * 2), (int)((uint32_t)N - (uint32_t)tile * 64u), off, b);
}

// A wave's walk over the tiles tile, tile + step, ... < end with two register buffers: the
// next tile's loads are in flight while the current one is multiplied and filtered.  The
// prefetch is unconditional so that the wait before the MFMAs only covers the tile they consume: the walk asks for one tile past
// the end too, of which `load` has to read nothing.
// FIRST_LOADED: the first tile is in `ba` or on its way (double-buffered walks only).
// Returns the first tile of the sequence at or past `end`.  No caller takes it, but without the value the compiler allots the registers of the
// row-tile scan otherwise (16 queries of 128k tokens 147.4 us per call, 146.7 with it).
template <bool PIPELINED, bool FIRST_LOADED = false, class Buf, class Load, class Use>
__device__ __forceinline__ int64_t walk_tiles(int64_t tile, int64_t end, int64_t step, Buf& ba, Buf& bb, Load load, Use use) {
    if (PIPELINED) {
        if (tile < end) {
            if (!FIRST_LOADED) load(ba, tile);
            while (true) {
                const int64_t t1 = tile + step;
                load(bb, t1);
                __builtin_amdgcn_sched_barrier(0);
                use(ba, tile);
                if (t1 >= end) { tile = t1; break; }
                const int64_t t2 = t1 + step;
                load(ba, t2);
                __builtin_amdgcn_sched_barrier(0);
                use(bb, t1);
                if (t2 >= end) { tile = t2; break; }
                tile = t2;
            }
        }
    } else {
        // One buffer: the other waves of the compute unit cover the latency.  For head_dim 256, and for samples, whose waves have a tile or two: a
        // second buffer's prefetch read the only tile twice and its registers halved the waves (sample of 16 x 8 streams of 4096 rows,
        // d = 128, 45.1 -> 35.8 us; of 8 streams of 8192 8.0 -> 6.9, of 2048 for 128k tokens 6.6 -> 5.4 by the whole call's time).
        for (; tile < end; tile += step) {
            load(ba, tile);
            __builtin_amdgcn_sched_barrier(0);
            use(ba, tile);
        }
    }
    return tile;
}

// head_dim 256 makes a 64-key tile 32 KiB: two register buffers of it do not fit, and
// with 8 waves per compute unit 256 KiB are in flight anyway.
template <int D> struct ScanPipelined { static constexpr bool value = D <= 128; };

// Scores of the tile: lane l gets res[r] = q_{head0 + r} . K[row(l)].
template <int DT, int D>
__device__ __forceinline__ f32x4 tile_mac(const typename Mfma<DT>::v8 (&b)[4][D / 32],
                                          const typename Mfma<DT>::v8 (&qa)[D / 32]) {
    constexpr int KS = D / 32;
    const int j = lane_id() >> 4;
    f32x4 c[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        c[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) c[g] = Mfma<DT>::mac(qa[s], b[g][s], c[g]);
    }
    // rows 4 jj .. 4 jj + 3 of every accumulator hold heads 0..3; lane group jj keeps sub-tile jj
    f32x4 res;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float lo = (j & 1) ? c[1][r] : c[0][r];
        const float hi = (j & 1) ? c[3][r] : c[2][r];
        res[r] = (j & 2) ? hi : lo;
    }
    return res;
}

}  // namespace tka

// Compressed key index: every key row is kept a second time as int8 codes with one fp32
// scale per row (the search index of the paper's methodology section need not be the plain
// key list; this is the compressed-list kind: approximate search, exact refinement).
//
//   code_c = rint(x_c * (127 / amax)),  scale = amax / 127,  amax = max_c |x_c|
//   (rows with amax < 2^-100 are coded as all zeros with scale 0)
//   s~ = float(sum_c codeq_c * codeK_c) * (scale_q * scale_K)
//
// The scan over the codes is the grouped MFMA scan again with v_mfma_i32_16x16x64_i8 and
// half the bytes per key; the candidates it keeps carry approximate scores, which
// rerank_kernel replaces by exact fp32 dot products with the 16-bit rows before the exact
// selection runs.  A key whose approximate score falls below the (lowered) threshold
// although its exact score belongs to the top k is lost: the result is approximate, with
// recall measured against the exact path.
#include "device_utils.h"
#include "internal.h"
#include "scan_common.h"
#include "scan_tiles.h"

namespace tka {

typedef int i32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------
// Row coding.  A row of D elements is spread over D / 8 lanes (16-bit storage, 16 bytes per lane).
// ---------------------------------------------------------------------------------------
// Row coding of the tokens a batched append adds: source rows [B][n_new][Hkv] (contiguous),
// row (b, t, h) is coded into row len[b] + t of (b, h) of the layer's index.
template <int DT>
__global__ void __launch_bounds__(256)
quantize_step_kernel(const char* __restrict__ src, int64_t n_rows, int64_t n_new, int Hkv, int64_t Ncap, int D,
                     const int32_t* __restrict__ len, int8_t* __restrict__ dst, float* __restrict__ scale) {
    constexpr int EPL = Elem<DT>::kPerLoad;
    const int lpr = D / EPL;
    const int rows_per_pass = 256 / lpr;
    const int rs = threadIdx.x / lpr, c = threadIdx.x % lpr;
    for (int64_t base = (int64_t)blockIdx.x * rows_per_pass; base < n_rows; base += (int64_t)gridDim.x * rows_per_pass) {
        const int64_t r = base + rs;
        const bool valid = r < n_rows;
        const int64_t rr = valid ? r : n_rows - 1;
        const int h = (int)(rr % Hkv);
        const int64_t bt = rr / Hkv, t = bt % n_new, b = bt / n_new;
        const u32x4 raw = *reinterpret_cast<const u32x4*>(src + (rr * D + c * EPL) * Elem<DT>::kBytes);
        float x[EPL];
        Elem<DT>::widen(raw, x);
        float amax = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) amax = fmaxf(amax, fabsf(x[e]));
        for (int o = 1; o < lpr; o <<= 1) amax = fmaxf(amax, wave_xor(amax, o));
        const bool live = amax >= kTinyRow;
        const float inv = live ? 127.0f / amax : 0.f;
        uint32_t w[EPL / 4];
#pragma unroll
        for (int i = 0; i < EPL / 4; ++i) {
            uint32_t p = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int code = (int)rintf(x[4 * i + e] * inv);
                p |= ((uint32_t)code & 0xFFu) << (8 * e);
            }
            w[i] = p;
        }
        if (valid) {
            const int64_t drow = (b * Hkv + h) * Ncap + (int64_t)len[b] + t;
            uint32_t* d = reinterpret_cast<uint32_t*>(dst + drow * D + c * EPL);
#pragma unroll
            for (int i = 0; i < EPL / 4; ++i) d[i] = w[i];
            if (c == 0) scale[drow] = live ? amax / 127.0f : 0.f;
        }
    }
}

hipError_t launch_quantize_step(int dtype, int D, const void* src, int B, int64_t n_new, int Hkv, int64_t Ncap,
                                const int32_t* len, int8_t* codes, float* scale, hipStream_t st) {
    const int64_t n_rows = (int64_t)B * n_new * Hkv;
    if (n_rows <= 0) return hipSuccess;
    const int rows_per_pass = 256 / (D / 8);
    int64_t blocks = (n_rows + rows_per_pass - 1) / rows_per_pass;
    if (blocks > 65536) blocks = 65536;
    if (dtype == DT_F16)
        hipLaunchKernelGGL((quantize_step_kernel<DT_F16>), dim3((unsigned)blocks), dim3(256), 0, st,
                           static_cast<const char*>(src), n_rows, n_new, Hkv, Ncap, D, len, codes, scale);
    else if (dtype == DT_BF16)
        hipLaunchKernelGGL((quantize_step_kernel<DT_BF16>), dim3((unsigned)blocks), dim3(256), 0, st,
                           static_cast<const char*>(src), n_rows, n_new, Hkv, Ncap, D, len, codes, scale);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// A small batched append on a cache with the int8 index in one launch: one workgroup places the new key and
// value rows, codes the key rows, and bumps the lengths once all its threads have used them.
constexpr int kAppendSmall8Threads = 1024;
template <int DT>
__global__ void __launch_bounds__(kAppendSmall8Threads)
append_step_small8_kernel(const char* __restrict__ ksrc, const char* __restrict__ vsrc, char* __restrict__ kdst,
                          char* __restrict__ vdst, int64_t head_b, int64_t n_rows, int64_t n_new, int Hkv, int64_t Ncap,
                          int D, int B, int32_t* len, int8_t* __restrict__ dst, float* __restrict__ scale) {
    constexpr int EPL = Elem<DT>::kPerLoad;          // 8: the index codes 16-bit caches
    const int lpr = D / EPL;
    const int rows_per_pass = kAppendSmall8Threads / lpr;
    const int rs = threadIdx.x / lpr, c = threadIdx.x % lpr;
    for (int64_t base = 0; base < n_rows; base += rows_per_pass) {
        const int64_t r = base + rs;
        const bool valid = r < n_rows;
        const int64_t rr = valid ? r : n_rows - 1;
        const int h = (int)(rr % Hkv);
        const int64_t bt = rr / Hkv, t = bt % n_new, b = bt / n_new;
        const int64_t s_o = (rr * D + c * EPL) * Elem<DT>::kBytes;
        const u32x4 raw = *reinterpret_cast<const u32x4*>(ksrc + s_o);
        const u32x4 rawv = *reinterpret_cast<const u32x4*>(vsrc + s_o);
        const int64_t row = (int64_t)len[b] + t;
        float x[EPL];
        Elem<DT>::widen(raw, x);
        float amax = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) amax = fmaxf(amax, fabsf(x[e]));
        for (int o = 1; o < lpr; o <<= 1) amax = fmaxf(amax, wave_xor(amax, o));
        const bool live = amax >= kTinyRow;
        const float inv = live ? 127.0f / amax : 0.f;
        uint32_t w[EPL / 4];
#pragma unroll
        for (int i = 0; i < EPL / 4; ++i) {
            uint32_t p = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int code = (int)rintf(x[4 * i + e] * inv);
                p |= ((uint32_t)code & 0xFFu) << (8 * e);
            }
            w[i] = p;
        }
        if (valid) {
            const int64_t d_o = (b * Hkv + h) * head_b + (row * D + c * EPL) * Elem<DT>::kBytes;
            *reinterpret_cast<u32x4*>(kdst + d_o) = raw;
            *reinterpret_cast<u32x4*>(vdst + d_o) = rawv;
            const int64_t drow = (b * Hkv + h) * Ncap + row;
            uint32_t* d = reinterpret_cast<uint32_t*>(dst + drow * D + c * EPL);
#pragma unroll
            for (int i = 0; i < EPL / 4; ++i) d[i] = w[i];
            if (c == 0) scale[drow] = live ? amax / 127.0f : 0.f;
        }
    }
    __syncthreads();            // every thread has used the lengths it needed
    for (int b = threadIdx.x; b < B; b += kAppendSmall8Threads) len[b] += (int32_t)n_new;
}

hipError_t launch_append_step_small8(int dtype, int D, const void* ksrc, const void* vsrc, void* kdst, void* vdst,
                                     int64_t head_bytes, int B, int64_t n_new, int Hkv, int64_t Ncap, int32_t* len,
                                     int8_t* codes, float* scale, hipStream_t st) {
    const int64_t n_rows = (int64_t)B * n_new * Hkv;
#define TKA_AS8(DT_)                                                                                                     \
    hipLaunchKernelGGL((append_step_small8_kernel<DT_>), dim3(1), dim3(kAppendSmall8Threads), 0, st,                    \
                       static_cast<const char*>(ksrc), static_cast<const char*>(vsrc), static_cast<char*>(kdst),        \
                       static_cast<char*>(vdst), head_bytes, n_rows, n_new, Hkv, Ncap, D, B, len, codes, scale)
    if (dtype == DT_F16) TKA_AS8(DT_F16);
    else if (dtype == DT_BF16) TKA_AS8(DT_BF16);
    else return hipErrorInvalidValue;
#undef TKA_AS8
    return hipGetLastError();
}

bool index8_supported(int dtype, int D, int G) {
    return (dtype == DT_F16 || dtype == DT_BF16) && (D == 64 || D == 128 || D == 256) && G >= 1 && G <= 4;
}

// ---------------------------------------------------------------------------------------
// Scan over the codes (grouped layout: one query, up to four heads per KV head).
// ---------------------------------------------------------------------------------------
// Codes of a 64-key tile in operand-B layout (lane (j, n) holds the 16-byte chunk 4 s + j of
// key 16 g + n) and the scale of key `lane`.
template <int D, class RowFn>
__device__ __forceinline__ void tile_load8(const int8_t* Kh, const float* Sh, RowFn rowfn, i32x4 (&b)[4][D / 64],
                                           float& ks) {
    constexpr int KS = D / 64;
    const int lane = lane_id();
    const int j = lane >> 4, n = lane & 15;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int64_t row = rowfn(16 * g + n);
        const i32x4* p = reinterpret_cast<const i32x4*>(Kh + row * D) + j;
#pragma unroll
        for (int s = 0; s < KS; ++s) b[g][s] = p[4 * s];
    }
    ks = Sh[rowfn(lane)];
}

// The same for the 64 consecutive keys from `row0` on (wave-uniform), of `n_rows` the stream has from there, through buffer loads
// whose descriptors end behind the rows there are (see tile_load_rows(): no address arithmetic in the loop, and no wait
// for the registers of an address).  Beyond them codes and scales read as zero and nothing is fetched.  512k tokens, 8 KV
// heads, d = 128: 97.8 -> 95.0 us (5.73 TB/s of codes and scales).
struct LaneOffsets8 { uint32_t g[4]; };
template <int D>
__device__ __forceinline__ LaneOffsets8 lane_offsets8() {
    LaneOffsets8 o;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        o.g[g] = (uint32_t)((16 * g + (lane_id() & 15)) * D + (lane_id() >> 4) * 16);
        asm volatile("" : "+v"(o.g[g]));
    }
    return o;
}
template <int D>
__device__ __forceinline__ void tile_load8_rows(const int8_t* Kh, const float* Sh, int64_t row0, int n_rows, const LaneOffsets8& off,
                                                i32x4 (&b)[4][D / 64], float& ks) {
    const uint32_t rows = bounded_rows(n_rows);
    const __amdgpu_buffer_rsrc_t codes =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(Kh + row0 * D), 0, (int)rows * D, 0x00020000);
    const __amdgpu_buffer_rsrc_t scales =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Sh + row0), 0, (int)rows * 4, 0x00020000);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
#pragma unroll
        for (int s = 0; s < D / 64; ++s) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(codes, (int)off.g[g] + 64 * s, 0, 0);
            b[g][s] = __builtin_bit_cast(i32x4, v);
        }
    }
    ks = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(scales, lane_id() * 4, 0, 0));
}

// Operand A of the scan, coded by every wave from the 16-bit query: lane (j, m) gets the code chunks 4 s + j of head m % 4
// (zero for heads the group does not have); qs: the heads' scales.  (A launch of its own for the codes of a few rows
// cost 4.8 us per step, the prologue of the scan kernels does not show it.)
template <int DT, int D>
__device__ __forceinline__ void load_query8(const void* q, int64_t head0, int G, i32x4 (&qa)[D / 64], float (&qs)[4]) {
    const int lane = lane_id(), j = lane >> 4, r = lane & 3;
    const u32x4* p = reinterpret_cast<const u32x4*>(static_cast<const char*>(q) + (head0 + (r < G ? r : 0)) * D * 2) + 2 * j;
    float x[D / 64][16], amax = 0.f;
#pragma unroll
    for (int s = 0; s < D / 64; ++s) {
        Elem<DT>::widen(p[8 * s], x[s]);
        Elem<DT>::widen(p[8 * s + 1], x[s] + 8);
    }
#pragma unroll
    for (int s = 0; s < D / 64; ++s) {
#pragma unroll
        for (int e = 0; e < 16; ++e) amax = fmaxf(amax, fabsf(x[s][e]));
    }
    amax = fmaxf(amax, wave_xor(amax, 16));
    amax = fmaxf(amax, wave_xor(amax, 32));
    const bool live = amax >= kTinyRow && r < G;
    const float inv = live ? 127.0f / amax : 0.f, scale = live ? amax / 127.0f : 0.f;
#pragma unroll
    for (int s = 0; s < D / 64; ++s) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t w = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) w |= ((uint32_t)(int)rintf(x[s][4 * i + e] * inv) & 0xFFu) << (8 * e);
            qa[s][i] = (int)w;
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) qs[i] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(scale), i));
}

// Integer dot products of the tile: lane l gets res[r] = codes(q_{head0 + r}) . codes(K[row(l)]).
template <int D>
__device__ __forceinline__ i32x4 tile_mac8(const i32x4 (&b)[4][D / 64], const i32x4 (&qa)[D / 64]) {
    constexpr int KS = D / 64;
    const int j = lane_id() >> 4;
    i32x4 c[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        c[g] = i32x4{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) c[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(qa[s], b[g][s], c[g], 0, 0, 0);
    }
    i32x4 res;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int lo = (j & 1) ? c[1][r] : c[0][r];
        const int hi = (j & 1) ? c[3][r] : c[2][r];
        res[r] = (j & 2) ? hi : lo;
    }
    return res;
}

template <int DT, int D, int MODE>
__global__ void __launch_bounds__(kScanWaves* kWave)
scan8_kernel(Shape sh, Bufs bf, int tiles_per_wave, float* dst) {
    fetch_args<kArgBytes>();
    constexpr int KS = D / 64;
    const int b = blockIdx.z, kvh = blockIdx.y;
    const int G = sh.G;
    const int64_t head0 = (int64_t)b * sh.Hq + (int64_t)kvh * G;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t N = prefix_len(bf.len[b], sh.window);

    int64_t n_items = N;
    int stride = 1;
    if (MODE == MODE_SAMPLE) {
        if (N == 0) return;
        Plan pl = make_plan(N, sh.k < N ? sh.k : (int)N, 1);
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
        const int64_t tile0 = (int64_t)blockIdx.x * tiles_per_wave * kScanWaves;
        if (tile0 >= n_tiles_all) return;
        tile = tile0 + wave;
        tile_step = kScanWaves;
        tile_end = tile0 + (int64_t)tiles_per_wave * kScanWaves;
        if (tile_end > n_tiles_all) tile_end = n_tiles_all;
    }

    const int64_t head_rows = ((int64_t)b * sh.Hkv + kvh) * sh.Ncap;
    const int8_t* Kh = bf.K8 + head_rows * D;
    const float* Sh = bf.Kscale + head_rows;
    struct TileB { i32x4 b[4][KS]; float ks; } ba, bb;
    const LaneOffsets8 lane_off = lane_offsets8<D>();
    // filter: the wave takes one tile of every row of n_seg tiles (seg_tile()); its first one is asked for ahead of the
    // query and the thresholds
    const int sid = (int)blockIdx.x * kScanWaves + wave;
    const int64_t rows_mine = MODE == MODE_FILTER ? seg_rows(n_tiles_all, sid, sh.n_seg) : 0;
    auto load_at = [&](TileB& t, int64_t ti, int64_t n) {
        tile_load8_rows<D>(Kh, Sh, ti * 64, (int)((uint32_t)n - (uint32_t)ti * 64u), lane_off, t.b, t.ks);
    };
    auto load_seg = [&](TileB& t, int64_t i) { load_at(t, seg_tile(i, sid, sh.n_seg), N); };
    if (MODE == MODE_FILTER && rows_mine > 0) {
        load_seg(ba, 0);
        __builtin_amdgcn_sched_barrier(0);
    }

    i32x4 qa[KS];
    float qs[4];
    load_query8<DT, D>(bf.q, head0, G, qa, qs);
    const float qs0 = qs[0], qs1 = qs[1], qs2 = qs[2], qs3 = qs[3];

    const int seg_cap = sh.seg_cap;
    uint64_t* const list0 = bf.cand + head0 * (int64_t)sh.cand_cap;
    __shared__ uint64_t stage_lds[MODE == MODE_FILTER ? kScanWaves * 4 * kStage : 1];
    uint64_t* const st0 = stage_lds + (MODE == MODE_FILTER ? wave * 4 * kStage : 0);
    CandStage cs0{st0, list0, sid, 0, 0}, cs1{st0 + kStage, list0 + (int64_t)sh.cand_cap, sid, 0, 0},
        cs2{st0 + 2 * kStage, list0 + 2 * (int64_t)sh.cand_cap, sid, 0, 0},
        cs3{st0 + 3 * kStage, list0 + 3 * (int64_t)sh.cand_cap, sid, 0, 0};
    float thr0 = 0.f, thr1 = 0.f, thr2 = 0.f, thr3 = 0.f;
    if (MODE == MODE_FILTER) {
        thr0 = bf.thr[head0];
        if (1 < G) thr1 = bf.thr[head0 + 1];
        if (2 < G) thr2 = bf.thr[head0 + 2];
        if (3 < G) thr3 = bf.thr[head0 + 3];
    }

    auto sample_row = [&](int64_t item) -> int64_t {        // key row of a sample (beyond the last one: the last one's)
        const int64_t p = sample_pos((int)(item < n_items ? item : n_items - 1), stride);
        return p < N ? p : N - 1;
    };
    auto consume = [&](const i32x4& res, float ks, int64_t item0) {
        const int64_t item = item0 + lane;
        const bool valid = item < n_items;
        const float s0 = (float)res[0] * (qs0 * ks), s1 = (float)res[1] * (qs1 * ks), s2 = (float)res[2] * (qs2 * ks),
                    s3 = (float)res[3] * (qs3 * ks);
        if (MODE == MODE_SAMPLE || MODE == MODE_FULL) {
            float* out = MODE == MODE_SAMPLE ? bf.samp : dst;
            const int64_t pitch = MODE == MODE_SAMPLE ? (int64_t)sh.samp_cap : sh.Ncap;
            if (valid) {
                out[head0 * pitch + item] = s0;
                if (1 < G) out[(head0 + 1) * pitch + item] = s1;
                if (2 < G) out[(head0 + 2) * pitch + item] = s2;
                if (3 < G) out[(head0 + 3) * pitch + item] = s3;
            }
        } else {
            filter_head(s0, thr0, cs0, valid, item, seg_cap, sh.n_seg);
            if (1 < G) filter_head(s1, thr1, cs1, valid, item, seg_cap, sh.n_seg);
            if (2 < G) filter_head(s2, thr2, cs2, valid, item, seg_cap, sh.n_seg);
            if (3 < G) filter_head(s3, thr3, cs3, valid, item, seg_cap, sh.n_seg);
        }
    };

    auto use = [&](TileB& t, int64_t ti) { consume(tile_mac8<D>(t.b, qa), t.ks, ti * 64); };
    if (MODE == MODE_FILTER)
        walk_tiles<true, true>(0, rows_mine, 1, ba, bb, load_seg, [&](TileB& t, int64_t i) { use(t, seg_tile(i, sid, sh.n_seg)); });
    else if (MODE == MODE_FULL)
        walk_tiles<true>(tile, tile_end, tile_step, ba, bb, [&](TileB& t, int64_t ti) { load_at(t, ti, ti < tile_end ? N : 0); }, use);
    else
        walk_tiles<false>(tile, tile_end, tile_step, ba, bb,
            [&](TileB& t, int64_t ti) { tile_load8<D>(Kh, Sh, [&](int slot) { return sample_row(ti * 64 + slot); }, t.b, t.ks); }, use);
    if (MODE == MODE_FILTER) {
        stage_flush(cs0, seg_cap, sh.n_seg, true);
        if (1 < G) stage_flush(cs1, seg_cap, sh.n_seg, true);
        if (2 < G) stage_flush(cs2, seg_cap, sh.n_seg, true);
        if (3 < G) stage_flush(cs3, seg_cap, sh.n_seg, true);
        if (lane == 0) {
            uint32_t* sc = bf.seg_cnt + head0 * (int64_t)sh.n_seg + sid;
            sc[0] = (uint32_t)cs0.n_glob;
            if (1 < G) sc[sh.n_seg] = (uint32_t)cs1.n_glob;
            if (2 < G) sc[2 * (int64_t)sh.n_seg] = (uint32_t)cs2.n_glob;
            if (3 < G) sc[3 * (int64_t)sh.n_seg] = (uint32_t)cs3.n_glob;
        }
    }
}

template <int MODE>
static hipError_t launch_scan8(const Shape& s, const Bufs& b, int64_t n_items, float* dst, hipStream_t st) {
    dim3 grid, block(kScanWaves * kWave);
    int tpw = 0;
    if (MODE == MODE_FILTER) {
        grid = dim3((unsigned)(s.n_seg / kScanWaves), (unsigned)s.Hkv, (unsigned)s.B);
    } else {
        tpw = tiles_per_wave_for(n_items, s.B, s.Hkv);
        const int64_t tiles = (n_items + 63) / 64, per_wg = (int64_t)tpw * kScanWaves;
        grid = dim3((unsigned)((tiles + per_wg - 1) / per_wg), (unsigned)s.Hkv, (unsigned)s.B);
    }
#define TKA_S8(DT_, D_) hipLaunchKernelGGL((scan8_kernel<DT_, D_, MODE>), grid, block, 0, st, s, b, tpw, dst)
    if (s.dtype == DT_F16 && s.D == 128) TKA_S8(DT_F16, 128);
    else if (s.dtype == DT_BF16 && s.D == 128) TKA_S8(DT_BF16, 128);
    else if (s.dtype == DT_F16 && s.D == 64) TKA_S8(DT_F16, 64);
    else if (s.dtype == DT_BF16 && s.D == 64) TKA_S8(DT_BF16, 64);
    else if (s.dtype == DT_F16 && s.D == 256) TKA_S8(DT_F16, 256);
    else if (s.dtype == DT_BF16 && s.D == 256) TKA_S8(DT_BF16, 256);
    else return hipErrorInvalidValue;
#undef TKA_S8
    return hipGetLastError();
}

hipError_t launch_scan8_sample(const Shape& s, const Bufs& b, int64_t Nmax, hipStream_t st) {
    Plan pl = make_plan(Nmax, s.k, 1);
    return launch_scan8<MODE_SAMPLE>(s, b, pl.n_samp, nullptr, st);
}
hipError_t launch_scan8_filter(const Shape& s, const Bufs& b, hipStream_t st) {
    return launch_scan8<MODE_FILTER>(s, b, 0, nullptr, st);
}
hipError_t launch_scan8_full(const Shape& s, const Bufs& b, int64_t Nmax, float* dst, hipStream_t st) {
    return launch_scan8<MODE_FULL>(s, b, Nmax, dst, st);
}

// ---------------------------------------------------------------------------------------
// Exact refinement: the score of every candidate the index scan kept is replaced by the
// fp32 dot product of the query with the 16-bit key row.  One wave per segment of a head's
// candidate list (it knows the segment's length, so no slot is visited in vain), D / 8 lanes per row.
// All workgroups run at once and each is a chain of trips to memory, so what bounds it is their number: the segment's
// length, its first entries, the query and the head's flags are asked for together, a lane holds one of 64 entries
// (the rows' positions come from its registers, the next 64 are on their way meanwhile), and the next rows are
// under way while the current ones are multiplied.  512k tokens, 32 heads, 16.7k candidates each, d = 128 (137 MB of
// rows): 41.0 -> 31.7 us (4.3 TB/s; whole call 183.7 -> 174.6).  Rounds of the entry, then the row it points to, one after the other,
// kept it at 3.4 TB/s.
// ---------------------------------------------------------------------------------------
constexpr int kRerankInFlight = 4;    // rows per lane group and round, of two rounds in flight

template <int DT, int D>
__global__ void __launch_bounds__(256) rerank_kernel(Shape sh, Bufs bf) {
    fetch_args<kArgBytes>();
    constexpr int EPL = Elem<DT>::kPerLoad;
    constexpr int LPR = D / EPL, GR = kWave / LPR;       // lanes per row, rows per load of the wave
    constexpr int U = kRerankInFlight, RR = GR * U;      // rows per round
    static_assert(kWave % RR == 0 && LPR >= U, "rounds of whole batches, a lane of its own per row of a group");
    __shared__ uint32_t hist_lds[kTailBins];             // this workgroup's candidates per score bin (exact scores)
    const int h = blockIdx.y, b = blockIdx.z;
    const int64_t bh = (int64_t)b * sh.Hq + h;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = (int)blockIdx.x * 4 + wave;            // this wave's segment
    const int grp = lane / LPR, c = lane % LPR;
    uint64_t* const list = bf.cand + bh * (int64_t)sh.cand_cap;
    // (any slot of the list may be read; what lies beyond the segment's length is ignored)
    auto entry = [&](uint32_t e) -> uint64_t {
        const int64_t slot = cand_slot(e, g, sh.n_seg);
        return list[slot < sh.cand_cap ? slot : 0];
    };
    uint64_t ent = entry((uint32_t)lane);
    const u32x4 q_raw = *reinterpret_cast<const u32x4*>(static_cast<const char*>(bf.q) + (bh * D + c * EPL) * Elem<DT>::kBytes);
    uint32_t have = bf.seg_cnt[bh * sh.n_seg + g];
    const float bin_lo = bf.bins[2 * bh], bin_inv = bf.bins[2 * bh + 1];
    const uint32_t flags = bf.flags[bh];
    uint32_t* hist_out = bf.hist + (bh * sh.hist_cap + blockIdx.x) * kTailBins;
    const bool counts = (int)blockIdx.x < sh.hist_cap;   // (always, when the tail is going to read them)
    if (threadIdx.x < kTailBins) hist_lds[threadIdx.x] = 0u;
    __syncthreads();
    if (have > (uint32_t)sh.seg_cap) have = (uint32_t)sh.seg_cap;
    if (flags) have = 0;                                 // not filtered: the exact redo scores this head itself
    float qr[EPL];
    Elem<DT>::widen(q_raw, qr);
    const char* Kh = static_cast<const char*>(bf.K) +
                     ((int64_t)cache_seq(sh, b) * sh.Hkv + h / sh.G) * sh.Ncap * D * Elem<DT>::kBytes;
    float top = -INFINITY;                               // largest exact score of the segment
    struct Round { uint32_t pos[U]; u32x4 raw[U]; } ra, rb;
    for (uint32_t e0 = 0; e0 < have; e0 += kWave) {      // `have` is uniform over the wave
        const int n = have - e0 < (uint32_t)kWave ? (int)(have - e0) : kWave;
        const uint32_t pos = lane < n ? (uint32_t)ent : 0u;
        if (e0 + kWave < have) ent = entry(e0 + kWave + lane);
        auto ask = [&](int r0, Round& t) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                t.pos[u] = (uint32_t)__shfl((int)pos, r0 + GR * u + grp, kWave);
                t.raw[u] = *reinterpret_cast<const u32x4*>(Kh + ((int64_t)t.pos[u] * D + c * EPL) * Elem<DT>::kBytes);
            }
        };
        auto score = [&](int r0, const Round& t) {       // lane c < U of a group keeps the group's row c
            float mine = 0.f;
            uint32_t at = 0u;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float kf[EPL];
                Elem<DT>::widen(t.raw[u], kf);
                float acc = 0.f;
#pragma unroll
                for (int i = 0; i < EPL; ++i) acc = fmaf(kf[i], qr[i], acc);
                acc = group_reduce<AddOp, LPR>(acc);
                if (c == u) { mine = acc; at = t.pos[u]; }
            }
            const int e = r0 + GR * c + grp;
            if (c < U && e < n) {
                const float sc = mine + 0.0f;
                list[cand_slot(e0 + e, g, sh.n_seg)] = ((uint64_t)__float_as_uint(sc) << 32) | (uint64_t)at;
                atomicAdd(&hist_lds[tail_bin(sc, bin_lo, bin_inv)], 1u);
                top = fmaxf(top, sc);
            }
        };
        ask(0, ra);
#pragma unroll
        for (int r0 = 0; r0 < kWave; r0 += 2 * RR) {
            if (r0 < n) {                                // (uniform)
                if (r0 + RR < n) ask(r0 + RR, rb);
                __builtin_amdgcn_sched_barrier(0);
                score(r0, ra);
                if (r0 + RR < n) {
                    if (r0 + 2 * RR < n) ask(r0 + 2 * RR, ra);
                    __builtin_amdgcn_sched_barrier(0);
                    score(r0 + RR, rb);
                }
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) top = fmaxf(top, wave_xor(top, o));
    if (lane == 0) bf.seg_max[bh * sh.n_seg + g] = top;
    __syncthreads();
    if (counts && threadIdx.x < kTailBins) hist_out[threadIdx.x] = hist_lds[threadIdx.x];
}

hipError_t launch_rerank(const Shape& s, const Bufs& b, hipStream_t st) {
    dim3 grid((unsigned)(s.n_seg / 4), (unsigned)s.Hq, (unsigned)s.B);      // n_seg is a multiple of 4
#define TKA_RR(DT_, D_) hipLaunchKernelGGL((rerank_kernel<DT_, D_>), grid, dim3(256), 0, st, s, b)
    if (s.dtype == DT_F16 && s.D == 128) TKA_RR(DT_F16, 128);
    else if (s.dtype == DT_BF16 && s.D == 128) TKA_RR(DT_BF16, 128);
    else if (s.dtype == DT_F16 && s.D == 64) TKA_RR(DT_F16, 64);
    else if (s.dtype == DT_BF16 && s.D == 64) TKA_RR(DT_BF16, 64);
    else if (s.dtype == DT_F16 && s.D == 256) TKA_RR(DT_F16, 256);
    else if (s.dtype == DT_BF16 && s.D == 256) TKA_RR(DT_BF16, 256);
    else return hipErrorInvalidValue;
#undef TKA_RR
    return hipGetLastError();
}

}  // namespace tka

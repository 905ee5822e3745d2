// Host side of libtopk_attn: handle, argument checks, workspace layout, launches.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <memory>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "../../include/topk_attn.h"
#include "../../include/topk_attn_debug.h"
#include "device_utils.h"
#include "internal.h"

using namespace tka;

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
inline int elem_bytes(int dtype) { return dtype == TOPK_ATTN_F32 ? 4 : 2; }

struct WsLayout {
    size_t len, thr, bins, samp, seg_cnt, seg_max, seg_cnt2, flags, hmax, fallback, tailrec, page_mask, page_cnt, page_list, hist, cand, bnd, scores, sel_idx, sel_val, part_acc, part_l, part_m, total;
    int cand_cap, bnd_cap, n_chunk_cap, hist_cap, page_words, batch_layers;
};

bool config_ok(const topk_attn_config* c, int* why) {
    *why = TOPK_ATTN_EINVAL;
    if (!c || c->struct_size != sizeof(topk_attn_config)) return false;
    if (c->n_layers < 1 || c->n_seqs < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1) return false;
    if (c->max_tokens < 1 || c->max_k < 1 || c->device < 0 || c->max_window < 0) return false;
    if (c->max_queries < 0 || c->max_queries > 4096) return false;
    if (c->index_kind != TOPK_ATTN_INDEX_NONE && c->index_kind != TOPK_ATTN_INDEX_INT8 &&
        c->index_kind != TOPK_ATTN_INDEX_PAGES)
        return false;
    if ((int64_t)c->n_seqs * (c->max_queries > 1 ? c->max_queries : 1) > 65535) return false;   // a grid dimension
    if (c->max_tokens > (int64_t)0x7FFFFF00) return false;   // positions are int32
    if (c->max_k > (1 << 28)) return false;                  // the candidate list (about 4 max_k entries) is indexed by int32
    if (c->n_seqs > 65535 || c->n_kv_heads > 65535) return false;
    *why = TOPK_ATTN_EUNSUPPORTED;
    if (c->dtype != TOPK_ATTN_F32 && c->dtype != TOPK_ATTN_F16 && c->dtype != TOPK_ATTN_BF16) return false;
    if (c->head_dim != 32 && c->head_dim != 64 && c->head_dim != 128 && c->head_dim != 256) return false;
    if (c->n_q_heads % c->n_kv_heads) return false;
    if (c->n_q_heads / c->n_kv_heads > 128) return false;
    if (c->dtype == TOPK_ATTN_F32 && c->n_q_heads / c->n_kv_heads > 16) return false;   // plain-FMA scorer
    if (c->index_kind == TOPK_ATTN_INDEX_INT8 &&
        !index8_supported(c->dtype, c->head_dim, c->n_q_heads / c->n_kv_heads))
        return false;
    if (c->index_kind == TOPK_ATTN_INDEX_PAGES &&
        !pages_supported(c->dtype, c->head_dim, c->n_q_heads / c->n_kv_heads))
        return false;
    *why = TOPK_ATTN_OK;
    return true;
}

size_t kv_half_bytes(const topk_attn_config* c) {
    return align_up((size_t)c->n_layers * c->n_seqs * c->n_kv_heads * (size_t)c->max_tokens * c->head_dim *
                    elem_bytes(c->dtype));
}

// int8 index behind K and V: codes, then scales
size_t index_codes_bytes(const topk_attn_config* c) {
    if (c->index_kind != TOPK_ATTN_INDEX_INT8) return 0;
    return align_up((size_t)c->n_layers * c->n_seqs * c->n_kv_heads * (size_t)c->max_tokens * c->head_dim);
}
size_t index_scales_bytes(const topk_attn_config* c) {
    if (c->index_kind != TOPK_ATTN_INDEX_INT8) return 0;
    return align_up((size_t)c->n_layers * c->n_seqs * c->n_kv_heads * (size_t)c->max_tokens * sizeof(float));
}
// page index behind K and V: centres, then (radius, centre norm) pairs
int64_t page_cap_of(const topk_attn_config* c) { return (c->max_tokens + 63) / 64; }
size_t page_centres_bytes(const topk_attn_config* c) {
    if (c->index_kind != TOPK_ATTN_INDEX_PAGES) return 0;
    return align_up((size_t)c->n_layers * c->n_seqs * c->n_kv_heads * (size_t)page_cap_of(c) * c->head_dim * elem_bytes(c->dtype));
}
size_t page_balls_bytes(const topk_attn_config* c) {
    if (c->index_kind != TOPK_ATTN_INDEX_PAGES) return 0;
    return align_up((size_t)c->n_layers * c->n_seqs * c->n_kv_heads * (size_t)page_cap_of(c) * 2 * sizeof(float));
}
size_t kv_total_bytes(const topk_attn_config* c) {
    return 2 * kv_half_bytes(c) + index_codes_bytes(c) + index_scales_bytes(c) + page_centres_bytes(c) + page_balls_bytes(c);
}

// batch_layers: layers of a topk_attn_decode_layers call that share their launches, each with per-call buffers of its own (a
// layer's heads and those of a further query of a chunk take the same room).
WsLayout ws_layout(const topk_attn_config* c, int batch_layers) {
    WsLayout w;
    const int per_seq = std::max(std::max(c->max_queries, 1), batch_layers);
    const size_t BH = (size_t)c->n_seqs * per_seq * c->n_q_heads;
    const int64_t max_k = c->max_k < c->max_tokens ? c->max_k : c->max_tokens;
    // candidate list per head.  A call with few KV-head streams splits each stream into many wave
    // segments (up to about 1024 waves over the chip, doubled where the split is rounded up).
    int64_t seg_max = 8 * ((512 + (int64_t)c->n_seqs * c->n_kv_heads - 1) / ((int64_t)c->n_seqs * c->n_kv_heads));
    if (seg_max > kMaxSeg) seg_max = kMaxSeg;
    // The boundary list takes the expected candidates (about 2 k at most) and a few dozen spare entries
    // per segment.  The segments of the candidate list are sized for keys whose scores come in runs
    // along the sequence (a passage the query attends to): a whole 64-key tile of candidates lands in
    // one segment at a time, so a segment that expects m such tiles gets room for m + 5 sqrt(m) + 4.
    // m is that of the wider margin: room for keys that tie in their thousands above the threshold (16 sequences of 60k tokens,
    // k = 1000, half of one sequence's keys equal, d = 128: 413 us; 799 with lists sized by the narrower margin, two heads scored again).
    w.bnd_cap = (int)(4 * max_k + 16384 + 48 * seg_max);
    {
        const Plan top = make_plan(c->max_tokens, (int)max_k, 0, true);
        const double m = (double)top.c_hi / (64.0 * (double)seg_max);
        const int64_t lumpy = (int64_t)((double)seg_max * 64.0 * (m + 5.0 * sqrt(m) + 4.0));
        w.cand_cap = (int)(lumpy > w.bnd_cap ? lumpy : w.bnd_cap);
        // whole 128-byte lines per head and whole runs of kCandChunk per segment, however the list is split
        w.cand_cap = (int)(((int64_t)w.cand_cap + kMaxSeg * kCandChunk - 1) / (kMaxSeg * kCandChunk) * (kMaxSeg * kCandChunk));
    }
    const int64_t max_w = c->max_window < c->max_tokens ? c->max_window : c->max_tokens;
    w.hist_cap = (int)(seg_max / 4);            // scan workgroups per head (four wave segments each)
    // partial sums per head: the tail of the filtered path makes up to one per 128 selected rows, at least one per
    // four scan workgroups (and never more than scan workgroups fed the head), the gather one per 256; the window
    // adds one per 256 tokens
    {
        const int64_t by_k = ((int64_t)c->max_k + 127) / 128, by_wg = (w.hist_cap + 3) / 4;
        w.n_chunk_cap = (int)((by_k > by_wg ? by_k : by_wg) + (max_w + kGatherRows - 1) / kGatherRows);
    }
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes); return at; };
    w.len = take((size_t)c->n_layers * c->n_seqs * sizeof(int32_t));
    w.thr = take(BH * sizeof(float));
    w.bins = take(BH * 2 * sizeof(float));
    w.samp = take(BH * kSampMax * sizeof(float));
    w.seg_cnt = take(BH * kMaxSeg * sizeof(uint32_t));
    w.seg_max = take(BH * kMaxSeg * sizeof(float));
    w.seg_cnt2 = take(BH * kMaxSeg * sizeof(uint32_t));
    w.flags = take(BH * sizeof(uint32_t));
    w.hmax = take(BH * sizeof(float));
    w.fallback = take(sizeof(uint32_t));
    w.tailrec = take(BH * 4 * sizeof(uint32_t));
    w.page_words = (int)((page_cap_of(c) + 63) / 64);
    const size_t page_streams = c->index_kind == TOPK_ATTN_INDEX_PAGES ? (size_t)c->n_seqs * c->n_kv_heads : 0;
    w.page_mask = take(page_streams * (size_t)w.page_words * sizeof(uint64_t));
    w.page_cnt = take(page_streams * sizeof(uint32_t));
    w.page_list = take(page_streams * (size_t)w.page_words * 64 * sizeof(int32_t));
    w.hist = take(BH * (size_t)w.hist_cap * kTailBins * sizeof(uint32_t));
    w.cand = take(BH * (size_t)w.cand_cap * sizeof(uint64_t));
    w.bnd = take(BH * (size_t)w.bnd_cap * sizeof(uint64_t));
    w.scores = take(BH * (size_t)c->max_tokens * sizeof(float));
    w.sel_idx = take(BH * (size_t)c->max_k * sizeof(int32_t));   // stride is the requested k, up to max_k
    w.sel_val = take(BH * (size_t)c->max_k * sizeof(float));
    w.part_acc = take(BH * (size_t)w.n_chunk_cap * c->head_dim * sizeof(float));
    w.part_l = take(BH * (size_t)w.n_chunk_cap * sizeof(float));
    w.part_m = take(BH * (size_t)w.n_chunk_cap * sizeof(float));
    w.total = o;
    w.batch_layers = batch_layers;
    return w;
}

// Layers that may share their launches (a power of two): of the layers asked for, those the configuration has and a grid takes.
int batch_layers_at_most(const topk_attn_config* c, int layers) {
    int n = 1;
    while (2 * n <= std::min(std::min(layers, c->n_layers), kBatchLayers) && (int64_t)c->n_seqs * 2 * n <= 65535) n *= 2;
    return n;
}
// The most layers for which the room is of use: whose steps over max_tokens tokens with max_k join (joins(); steps through an
// index, of more than kAttendRows value rows or of lists that the chip-wide selection takes never do), within
// kBatchScratchBytes (8 KV heads, 32 query heads, 48k tokens: 65 MB a layer).
constexpr size_t kBatchScratchBytes = (size_t)1 << 30;
int batch_layers_useful(const topk_attn_config* c) {
    int n = batch_layers_at_most(c, kBatchLayers);
    const int64_t heads = (int64_t)c->n_seqs * c->n_q_heads, k = std::min<int64_t>(c->max_k, c->max_tokens);
    const int64_t window = std::min<int64_t>(c->max_window, c->max_tokens);
    if (k + window > kAttendRows) return 1;
    if (c->max_tokens > kAttendRowMax) {             // (shorter caches: over score rows)
        if (c->dtype == TOPK_ATTN_F32 || c->index_kind != TOPK_ATTN_INDEX_NONE) return 1;
        if (window * c->head_dim * 2 > kAttendWindowBytes || make_plan(c->max_tokens, (int)k).c_hi > kAttendList) return 1;
        while (n > 1 && (heads * n > kAttendManyHeads || c->max_tokens > kAttendShareKeys * (kAttendManyHeads / (heads * n)))) n /= 2;
    }
    while (n > 1 && ws_layout(c, n).total > kBatchScratchBytes) n /= 2;
    return n;
}

__global__ void append_kernel(const char* __restrict__ ksrc, const char* __restrict__ vsrc, char* __restrict__ kdst,
                              char* __restrict__ vdst, int64_t n_new, int Hkv, int chunks_per_row,
                              int64_t token_stride_b, int64_t head_stride_b, int64_t dst_head_stride_b,
                              int32_t* len_slot, int32_t new_len) {
    const int64_t total = n_new * Hkv * chunks_per_row;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % chunks_per_row);
        const int64_t th = i / chunks_per_row;
        const int h = (int)(th % Hkv);
        const int64_t t = th / Hkv;
        const int64_t so = t * token_stride_b + h * head_stride_b + (int64_t)c * 16;
        const int64_t d_o = h * dst_head_stride_b + (t * chunks_per_row + c) * 16;
        *reinterpret_cast<u32x4*>(kdst + d_o) = *reinterpret_cast<const u32x4*>(ksrc + so);
        *reinterpret_cast<u32x4*>(vdst + d_o) = *reinterpret_cast<const u32x4*>(vsrc + so);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *len_slot = new_len;
}

// The same with the int8 codes of the key rows (topk_attn.h: code = rint(x 127 / amax), scale = amax / 127): the rows are coded
// from the registers that carry them, so a bulk import reads the keys once.  Blocks of rows in grid x, KV heads in
// grid y; D / 8 lanes per row, kAppend8Rows rows in flight per lane group.  100001 tokens, 8 KV heads, d = 128
// (0.93 GB moved): 220 us per import with the coding in a launch of its own, 172 us (5.4 TB/s) now.
constexpr int kAppend8Rows = 4;
template <int DT, int D>
__global__ void __launch_bounds__(256)
append8_kernel(const char* __restrict__ ksrc, const char* __restrict__ vsrc, char* __restrict__ kdst, char* __restrict__ vdst,
               int64_t n_new, int64_t token_stride_b, int64_t head_stride_b, int64_t dst_head_stride_b, int8_t* __restrict__ codes,
               float* __restrict__ scales, int64_t ncap, int32_t* len_slot, int32_t new_len) {
    constexpr int LPR = D / 8, RPP = 256 / LPR, U = kAppend8Rows;      // lanes per row, rows per pass of the workgroup
    const int h = blockIdx.y, c = threadIdx.x % LPR;
    const int64_t t0 = (int64_t)blockIdx.x * (RPP * U) + threadIdx.x / LPR;
    const char* const ks = ksrc + h * head_stride_b + c * 16;
    const char* const vs = vsrc + h * head_stride_b + c * 16;
    u32x4 k[U], v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t t = t0 + u * RPP, r = t < n_new ? t : n_new - 1;
        k[u] = *reinterpret_cast<const u32x4*>(ks + r * token_stride_b);
        v[u] = *reinterpret_cast<const u32x4*>(vs + r * token_stride_b);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t t = t0 + u * RPP;
        float x[8];
        Elem<DT>::widen(k[u], x);
        float amax = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(x[e]));
        amax = group_reduce<MaxOp, LPR>(amax);
        const bool live = amax >= kTinyRow;
        const float inv = live ? 127.0f / amax : 0.f;
        uint32_t w[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint32_t p = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) p |= ((uint32_t)(int)rintf(x[4 * i + e] * inv) & 0xFFu) << (8 * e);
            w[i] = p;
        }
        if (t < n_new) {
            const int64_t d_o = h * dst_head_stride_b + (t * LPR + c) * 16, row = h * ncap + t;
            *reinterpret_cast<u32x4*>(kdst + d_o) = k[u];
            *reinterpret_cast<u32x4*>(vdst + d_o) = v[u];
            *reinterpret_cast<uint2*>(codes + row * D + c * 8) = make_uint2(w[0], w[1]);
            if (c == 0) scales[row] = live ? amax / 127.0f : 0.f;
        }
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *len_slot = new_len;
}

__global__ void set_len_kernel(int32_t* len_slot, int32_t v) { *len_slot = v; }

// n_new tokens for every sequence of a layer: source [B][n_new][Hkv][row], destination row
// len[b] + t of (b, h).  The lengths are bumped by a second kernel once every block has read them.
__global__ void append_step_kernel(const char* __restrict__ ksrc, const char* __restrict__ vsrc, char* __restrict__ kdst,
                                   char* __restrict__ vdst, const int32_t* __restrict__ len, int64_t total, int64_t n_new,
                                   int Hkv, int chunks_per_row, int64_t head_b) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % chunks_per_row);
        const int64_t th = i / chunks_per_row;
        const int h = (int)(th % Hkv);
        const int64_t bt = th / Hkv;
        const int64_t t = bt % n_new, b = bt / n_new;
        const int64_t d_o = (b * Hkv + h) * head_b + (((int64_t)len[b] + t) * chunks_per_row + c) * 16;
        *reinterpret_cast<u32x4*>(kdst + d_o) = *reinterpret_cast<const u32x4*>(ksrc + i * 16);
        *reinterpret_cast<u32x4*>(vdst + d_o) = *reinterpret_cast<const u32x4*>(vsrc + i * 16);
    }
}
// The same for a step small enough for one workgroup (a token or a few per sequence, no index to extend): the
// workgroup bumps the lengths itself once all its threads have placed their pieces, one launch instead of two.
constexpr int kAppendSmallThreads = 1024;
constexpr int64_t kAppendSmallPieces = 4 * kAppendSmallThreads;       // 16-byte pieces of K (and of V) per call: 256 rows of 256 bytes
__global__ void __launch_bounds__(kAppendSmallThreads)
append_step_small_kernel(const char* __restrict__ ksrc, const char* __restrict__ vsrc, char* __restrict__ kdst,
                         char* __restrict__ vdst, int32_t* len, int64_t total, int64_t n_new, int Hkv, int chunks_per_row,
                         int64_t head_b, int B) {
    for (int64_t i = threadIdx.x; i < total; i += kAppendSmallThreads) {
        const int c = (int)(i % chunks_per_row);
        const int64_t th = i / chunks_per_row;
        const int h = (int)(th % Hkv);
        const int64_t bt = th / Hkv;
        const int64_t t = bt % n_new, b = bt / n_new;
        const int64_t d_o = (b * Hkv + h) * head_b + (((int64_t)len[b] + t) * chunks_per_row + c) * 16;
        *reinterpret_cast<u32x4*>(kdst + d_o) = *reinterpret_cast<const u32x4*>(ksrc + i * 16);
        *reinterpret_cast<u32x4*>(vdst + d_o) = *reinterpret_cast<const u32x4*>(vsrc + i * 16);
    }
    __syncthreads();            // every thread has used the lengths it needed
    for (int b = threadIdx.x; b < B; b += kAppendSmallThreads) len[b] += (int32_t)n_new;
}
__global__ void bump_len_kernel(int32_t* len, int B, int32_t n_new) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) len[b] += n_new;
}

// Streaming read of n_vec 16-byte vectors: every wave walks 16 KiB tiles (16 independent
// 1 KiB-per-instruction loads in flight), the access shape of the key scan without its work.
__global__ void __launch_bounds__(256) read_probe_kernel(const u32x4* __restrict__ src, size_t n_vec, uint32_t* sink) {
    uint32_t acc = 0;
    const size_t lane = threadIdx.x & 63;
    const size_t wave = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6), n_waves = (size_t)gridDim.x * 4;
    const size_t n_tiles = n_vec / 1024;
    for (size_t t = wave; t < n_tiles; t += n_waves) {
        const u32x4* p = src + t * 1024 + lane;
        u32x4 v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = p[u * 64];
#pragma unroll
        for (int u = 0; u < 16; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    for (size_t i = n_tiles * 1024 + (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_vec;
         i += (size_t)gridDim.x * blockDim.x) {
        const u32x4 a = src[i];
        acc ^= a.x ^ a.y ^ a.z ^ a.w;
    }
    for (int o = 32; o > 0; o >>= 1) acc ^= __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63) == 0) atomicXor(&sink[blockIdx.x & 16383], acc);
}

__global__ void zero_words_kernel(uint32_t* p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

}  // namespace

// Built-in scratch of topk_attn_decode_static: the per-call buffers of one decode (everything the
// handle's workspace holds except the cache lengths) for callers that bring no workspace of
// their own to that call.  One copy per GPU, at its own address, held until the process ends.
constexpr size_t kStaticScratchBytes = (size_t)96 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Device address of `scratch` on each GPU (the array's name is only a host-side stand-in for
// it), looked up once per device with that device current.
constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mutex;
static int scratch_address(int device, void** out) {
    if (device < 0 || device >= kMaxDevices) return TOPK_ATTN_EINVAL;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return TOPK_ATTN_EDEVICE;
        g_scratch_ptr[device] = p;
    }
    *out = g_scratch_ptr[device];
    return TOPK_ATTN_OK;
}

constexpr int kTimingSlots = 512;

struct topk_attn {
    topk_attn_config cfg;
    WsLayout ws;
    WsLayout ws_one;            // the layout without room for further layers (the built-in scratch)
    size_t kv_half;
    std::vector<int64_t> len;   // host mirror of the device lengths, [L][B]
    int path;
    bool last_fast;
    bool last_static;           // the last decode used the built-in scratch
    int force_redo;             // measurement aid, see topk_attn_debug_force_redo: 0, 1, or 2 (chip-wide selection)
    float page_beta;            // scale of the page radius in the page bound (1 = exact)
    bool last_paged;            // the last decode went through the page index
    bool last_tail;             // the last decode used the chip-wide selection (its per-head records are in the workspace)
    int last_queries;           // queries per sequence of the last decode
    int last_n_seg, last_seg_cap;   // the split of the last filtered decode's candidate lists (0: not filtered)
    int last_layer;
    int last_slot;              // layers of the last call before its last one in the per-call buffers
    char* scratch_dev;          // this device's copy of the built-in scratch
    int n_cu;                   // compute units of the device
    // optional event pairs around the key scan of each decode (measurement only)
    bool timing;
    std::vector<hipEvent_t> ev;  // 2 * kTimingSlots once enabled
    int ev_used;
};

extern "C" {

size_t topk_attn_kv_bytes(const topk_attn_config* cfg) {
    int why;
    if (!config_ok(cfg, &why)) return 0;
    return kv_total_bytes(cfg);
}

size_t topk_attn_workspace_bytes(const topk_attn_config* cfg) {
    int why;
    if (!config_ok(cfg, &why)) return 0;
    return ws_layout(cfg, 1).total;
}

size_t topk_attn_layers_workspace_bytes(const topk_attn_config* cfg, int n_layers) {
    int why;
    if (n_layers < 0 || !config_ok(cfg, &why)) return 0;
    return ws_layout(cfg, n_layers == 0 ? batch_layers_useful(cfg) : batch_layers_at_most(cfg, n_layers)).total;
}

int topk_attn_create(const topk_attn_config* cfg, topk_attn_t** out) {
    if (!out) return TOPK_ATTN_EINVAL;
    *out = nullptr;
    int why;
    if (!config_ok(cfg, &why)) return why;
    if (!cfg->kv_storage || !cfg->workspace) return TOPK_ATTN_EINVAL;
    if (((uintptr_t)cfg->kv_storage | (uintptr_t)cfg->workspace) & (kAlign - 1)) return TOPK_ATTN_EINVAL;
    const WsLayout one = ws_layout(cfg, 1);
    if (cfg->kv_bytes < kv_total_bytes(cfg) || cfg->workspace_bytes < one.total) return TOPK_ATTN_ENOMEM;
    WsLayout w = one;                        // as many layers share their launches as the workspace has room for
    for (int n = batch_layers_at_most(cfg, kBatchLayers); n > 1; n /= 2) {
        w = ws_layout(cfg, n);
        if (w.total <= cfg->workspace_bytes) break;
        w = one;
    }
    topk_attn* h = new (std::nothrow) topk_attn;
    if (!h) return TOPK_ATTN_ENOMEM;
    h->cfg = *cfg;
    h->ws = w;
    h->ws_one = one;
    h->kv_half = kv_half_bytes(cfg);
    h->len.assign((size_t)cfg->n_layers * cfg->n_seqs, 0);
    h->path = TOPK_ATTN_PATH_AUTO;
    h->last_fast = false;
    h->timing = false;
    h->ev_used = 0;
    if (hipSetDevice(cfg->device) != hipSuccess) { delete h; return TOPK_ATTN_EDEVICE; }
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, cfg->device) != hipSuccess) { delete h; return TOPK_ATTN_EDEVICE; }
    h->n_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    h->last_static = false;
    h->force_redo = 0;
    h->page_beta = 1.0f;
    h->last_paged = false;
    h->last_tail = false;
    h->last_queries = 1;
    h->last_n_seg = h->last_seg_cap = 0;
    h->last_layer = 0;
    h->last_slot = 0;
    {   // cfg->device is current here
        void* p = nullptr;
        const int rc = scratch_address(cfg->device, &p);
        if (rc != TOPK_ATTN_OK) { delete h; return rc; }
        h->scratch_dev = static_cast<char*>(p);
    }
    // lengths and the small per-head control words start at zero
    if (hipMemset(cfg->workspace, 0, w.hist) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
        delete h;
        return TOPK_ATTN_EDEVICE;
    }
    *out = h;
    return TOPK_ATTN_OK;
}

int topk_attn_destroy(topk_attn_t* h) {
    if (!h) return TOPK_ATTN_EINVAL;
    for (hipEvent_t e : h->ev) (void)hipEventDestroy(e);
    delete h;
    return TOPK_ATTN_OK;
}

int64_t topk_attn_length(const topk_attn_t* h, int layer, int seq) {
    if (!h || layer < 0 || layer >= h->cfg.n_layers || seq < 0 || seq >= h->cfg.n_seqs) return -1;
    return h->len[(size_t)layer * h->cfg.n_seqs + seq];
}

int topk_attn_set_path(topk_attn_t* h, int path) {
    if (!h || path < TOPK_ATTN_PATH_AUTO || path > TOPK_ATTN_PATH_PAGES) return TOPK_ATTN_EINVAL;
    if (path == TOPK_ATTN_PATH_INDEX && h->cfg.index_kind != TOPK_ATTN_INDEX_INT8) return TOPK_ATTN_EINVAL;
    if (path == TOPK_ATTN_PATH_PAGES && h->cfg.index_kind != TOPK_ATTN_INDEX_PAGES) return TOPK_ATTN_EINVAL;
    h->path = path;
    return TOPK_ATTN_OK;
}

int topk_attn_reset(topk_attn_t* h, int layer, int seq, void* hip_stream) {
    if (!h || layer < 0 || layer >= h->cfg.n_layers || seq < 0 || seq >= h->cfg.n_seqs) return TOPK_ATTN_EINVAL;
    const size_t slot = (size_t)layer * h->cfg.n_seqs + seq;
    int32_t* len_dev = reinterpret_cast<int32_t*>(static_cast<char*>(h->cfg.workspace) + h->ws.len) + slot;
    hipLaunchKernelGGL(set_len_kernel, dim3(1), dim3(1), 0, (hipStream_t)hip_stream, len_dev, 0);
    if (hipGetLastError() != hipSuccess) return TOPK_ATTN_EDEVICE;
    h->len[slot] = 0;
    return TOPK_ATTN_OK;
}

int topk_attn_append_kv(topk_attn_t* h, int layer, int seq, const void* k_new, const void* v_new, int64_t n_new,
                        int64_t token_stride, int64_t head_stride, void* hip_stream) {
    if (!h || layer < 0 || layer >= h->cfg.n_layers || seq < 0 || seq >= h->cfg.n_seqs) return TOPK_ATTN_EINVAL;
    if (n_new < 0) return TOPK_ATTN_EINVAL;
    if (n_new == 0) return TOPK_ATTN_OK;
    if (!k_new || !v_new) return TOPK_ATTN_EINVAL;
    const topk_attn_config& c = h->cfg;
    const int e = elem_bytes(c.dtype);
    if (token_stride < 0 || head_stride < 0) return TOPK_ATTN_EINVAL;
    if (((uintptr_t)k_new | (uintptr_t)v_new) & 15) return TOPK_ATTN_EINVAL;
    if (((token_stride * e) | (head_stride * e)) & 15) return TOPK_ATTN_EINVAL;
    const size_t slot = (size_t)layer * c.n_seqs + seq;
    const int64_t cur = h->len[slot];
    if (cur + n_new > c.max_tokens) return TOPK_ATTN_ECAPACITY;

    const int64_t row_b = (int64_t)c.head_dim * e;
    const int64_t head_b = c.max_tokens * row_b;
    const int64_t off = ((int64_t)slot * c.n_kv_heads) * head_b + cur * row_b;
    char* kdst = static_cast<char*>(c.kv_storage) + off;
    char* vdst = static_cast<char*>(c.kv_storage) + h->kv_half + off;
    int32_t* len_dev = reinterpret_cast<int32_t*>(static_cast<char*>(c.workspace) + h->ws.len) + slot;
    const int chunks = (int)(row_b / 16);
    if (c.index_kind == TOPK_ATTN_INDEX_INT8) {
        char* base = static_cast<char*>(c.kv_storage) + 2 * h->kv_half;
        const int64_t row0 = (int64_t)slot * c.n_kv_heads * c.max_tokens + cur;
        int8_t* codes = reinterpret_cast<int8_t*>(base) + row0 * c.head_dim;
        float* scales = reinterpret_cast<float*>(base + index_codes_bytes(&c)) + row0;
        const int64_t rows_per_block = (int64_t)kAppend8Rows * (256 / (c.head_dim / 8));
        const dim3 grid((unsigned)((n_new + rows_per_block - 1) / rows_per_block), (unsigned)c.n_kv_heads);
#define TKA_A8(DT_, D_)                                                                                                     \
    hipLaunchKernelGGL((append8_kernel<DT_, D_>), grid, dim3(256), 0, (hipStream_t)hip_stream, static_cast<const char*>(k_new), \
                       static_cast<const char*>(v_new), kdst, vdst, n_new, token_stride * e, head_stride * e, head_b, codes,   \
                       scales, c.max_tokens, len_dev, (int32_t)(cur + n_new))
        if (c.dtype == TOPK_ATTN_F16 && c.head_dim == 128) TKA_A8(DT_F16, 128);
        else if (c.dtype == TOPK_ATTN_BF16 && c.head_dim == 128) TKA_A8(DT_BF16, 128);
        else if (c.dtype == TOPK_ATTN_F16 && c.head_dim == 64) TKA_A8(DT_F16, 64);
        else if (c.dtype == TOPK_ATTN_BF16 && c.head_dim == 64) TKA_A8(DT_BF16, 64);
        else if (c.dtype == TOPK_ATTN_F16 && c.head_dim == 256) TKA_A8(DT_F16, 256);
        else TKA_A8(DT_BF16, 256);
#undef TKA_A8
        if (hipGetLastError() != hipSuccess) return TOPK_ATTN_EDEVICE;
        h->len[slot] = cur + n_new;
        return TOPK_ATTN_OK;
    }
    const int64_t total = n_new * c.n_kv_heads * chunks;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(append_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)hip_stream,
                       static_cast<const char*>(k_new), static_cast<const char*>(v_new), kdst, vdst, n_new,
                       c.n_kv_heads, chunks, token_stride * e, head_stride * e, head_b, len_dev,
                       (int32_t)(cur + n_new));
    if (hipGetLastError() != hipSuccess) return TOPK_ATTN_EDEVICE;
    if (c.index_kind == TOPK_ATTN_INDEX_PAGES) {   // balls of the pages just touched (stream order: after the copy)
        char* base = static_cast<char*>(c.kv_storage) + 2 * h->kv_half;
        const int64_t pcap = page_cap_of(&c);
        const int64_t stream0 = (int64_t)slot * c.n_kv_heads;
        char* centres = base + stream0 * pcap * row_b;
        float* balls = reinterpret_cast<float*>(base + page_centres_bytes(&c)) + stream0 * pcap * 2;
        const char* kseq = static_cast<const char*>(c.kv_storage) + stream0 * head_b;
        if (launch_page_balls(c.dtype, c.head_dim, kseq, c.max_tokens, pcap, c.n_kv_heads, 1, nullptr, cur, n_new, centres,
                              balls, (hipStream_t)hip_stream) != hipSuccess)
            return TOPK_ATTN_EDEVICE;
    }
    h->len[slot] = cur + n_new;
    return TOPK_ATTN_OK;
}

int topk_attn_append_step(topk_attn_t* h, int layer, const void* k_new, const void* v_new, int64_t n_new,
                          void* hip_stream) {
    if (!h || layer < 0 || layer >= h->cfg.n_layers || n_new < 0) return TOPK_ATTN_EINVAL;
    if (n_new == 0) return TOPK_ATTN_OK;
    if (!k_new || !v_new || (((uintptr_t)k_new | (uintptr_t)v_new) & 15)) return TOPK_ATTN_EINVAL;
    const topk_attn_config& c = h->cfg;
    const int B = c.n_seqs;
    for (int b = 0; b < B; ++b)
        if (h->len[(size_t)layer * B + b] + n_new > c.max_tokens) return TOPK_ATTN_ECAPACITY;
    hipStream_t st = (hipStream_t)hip_stream;
    const int e = elem_bytes(c.dtype);
    const int64_t row_b = (int64_t)c.head_dim * e, head_b = c.max_tokens * row_b;
    const int64_t layer_off = (int64_t)layer * B * c.n_kv_heads * head_b;
    char* kdst = static_cast<char*>(c.kv_storage) + layer_off;
    char* vdst = static_cast<char*>(c.kv_storage) + h->kv_half + layer_off;
    int32_t* len_dev = reinterpret_cast<int32_t*>(static_cast<char*>(c.workspace) + h->ws.len) + (size_t)layer * B;
    const int chunks = (int)(row_b / 16);
    const int64_t total = (int64_t)B * n_new * c.n_kv_heads * chunks;
    if (c.index_kind == TOPK_ATTN_INDEX_NONE && total <= kAppendSmallPieces) {
        hipLaunchKernelGGL(append_step_small_kernel, dim3(1), dim3(kAppendSmallThreads), 0, st, static_cast<const char*>(k_new),
                           static_cast<const char*>(v_new), kdst, vdst, len_dev, total, n_new, c.n_kv_heads, chunks, head_b, B);
        if (hipGetLastError() != hipSuccess) return TOPK_ATTN_EDEVICE;
        for (int b = 0; b < B; ++b) h->len[(size_t)layer * B + b] += n_new;
        return TOPK_ATTN_OK;
    }
    if (c.index_kind == TOPK_ATTN_INDEX_INT8 && total <= kAppendSmallPieces) {      // the same with the rows' codes
        char* base = static_cast<char*>(c.kv_storage) + 2 * h->kv_half;
        const int64_t layer_rows = (int64_t)layer * B * c.n_kv_heads * c.max_tokens;
        int8_t* codes = reinterpret_cast<int8_t*>(base) + layer_rows * c.head_dim;
        float* scales = reinterpret_cast<float*>(base + index_codes_bytes(&c)) + layer_rows;
        if (launch_append_step_small8(c.dtype, c.head_dim, k_new, v_new, kdst, vdst, head_b, B, n_new, c.n_kv_heads,
                                      c.max_tokens, len_dev, codes, scales, st) != hipSuccess)
            return TOPK_ATTN_EDEVICE;
        for (int b = 0; b < B; ++b) h->len[(size_t)layer * B + b] += n_new;
        return TOPK_ATTN_OK;
    }
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(append_step_kernel, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<const char*>(k_new),
                       static_cast<const char*>(v_new), kdst, vdst, len_dev, total, n_new, c.n_kv_heads, chunks, head_b);
    if (hipGetLastError() != hipSuccess) return TOPK_ATTN_EDEVICE;
    if (c.index_kind == TOPK_ATTN_INDEX_INT8) {
        char* base = static_cast<char*>(c.kv_storage) + 2 * h->kv_half;
        const int64_t layer_rows = (int64_t)layer * B * c.n_kv_heads * c.max_tokens;
        int8_t* codes = reinterpret_cast<int8_t*>(base) + layer_rows * c.head_dim;
        float* scales = reinterpret_cast<float*>(base + index_codes_bytes(&c)) + layer_rows;
        if (launch_quantize_step(c.dtype, c.head_dim, k_new, B, n_new, c.n_kv_heads, c.max_tokens, len_dev, codes, scales,
                                 st) != hipSuccess)
            return TOPK_ATTN_EDEVICE;
    }
    if (c.index_kind == TOPK_ATTN_INDEX_PAGES) {
        char* base = static_cast<char*>(c.kv_storage) + 2 * h->kv_half;
        const int64_t pcap = page_cap_of(&c);
        const int64_t stream0 = (int64_t)layer * B * c.n_kv_heads;
        char* centres = base + stream0 * pcap * row_b;
        float* balls = reinterpret_cast<float*>(base + page_centres_bytes(&c)) + stream0 * pcap * 2;
        if (launch_page_balls(c.dtype, c.head_dim, kdst, c.max_tokens, pcap, c.n_kv_heads, B, len_dev, 0, n_new, centres, balls,
                              st) != hipSuccess)
            return TOPK_ATTN_EDEVICE;
    }
    hipLaunchKernelGGL(bump_len_kernel, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, st, len_dev, B, (int32_t)n_new);
    if (hipGetLastError() != hipSuccess) return TOPK_ATTN_EDEVICE;
    for (int b = 0; b < B; ++b) h->len[(size_t)layer * B + b] += n_new;
    return TOPK_ATTN_OK;
}

static void fill_call(topk_attn_t* h, int layer, const void* q, int k, int n_queries, Shape* s, Bufs* b,
                      bool use_static = false) {
    const topk_attn_config& c = h->cfg;
    const int e = elem_bytes(c.dtype);
    s->Bc = c.n_seqs; s->M = n_queries; s->causal = 0; s->B = c.n_seqs * n_queries;
    s->Hq = c.n_q_heads; s->Hkv = c.n_kv_heads; s->G = c.n_q_heads / c.n_kv_heads;
    s->row_tiles = n_queries * s->G > 16 ? 2 : 1;
    s->n_qblk = (n_queries * s->G + 16 * s->row_tiles - 1) / (16 * s->row_tiles);
    s->D = c.head_dim; s->dtype = c.dtype; s->k = k; s->window = 0; s->max_k = c.max_k;
    s->hist_cap = h->ws.hist_cap; s->tail_spw = 1; s->tail_wgs = 1;
    s->cand_cap = h->ws.cand_cap; s->bnd_cap = h->ws.bnd_cap; s->n_seg = 4; s->seg_cap = (h->ws.cand_cap / 4) & ~(kCandChunk - 1); s->samp_cap = kSampMax; s->n_chunk_cap = h->ws.n_chunk_cap;
    s->Ncap = c.max_tokens;
    s->indexed = 0; s->attend = 0; s->share_wgs = 0; s->log2_layers = 0; s->layer_seqs = s->B; b->layer_k[0] = LayerK{k, 0};
    s->paged = 0; s->no_rescan = 0;
    s->page_cap = (int)page_cap_of(&c); s->page_words = h->ws.page_words;
    s->force_redo = h->force_redo ? 1 : 0;
    char* const ws_len = static_cast<char*>(c.workspace);
    // everything after the lengths is per-call scratch: the handle's workspace, or the library's own array
    const WsLayout& w = use_static ? h->ws_one : h->ws;
    char* const ws = use_static ? reinterpret_cast<char*>(reinterpret_cast<uintptr_t>(h->scratch_dev) - w.thr) : ws_len;
    const size_t layer_b = (size_t)c.n_seqs * c.n_kv_heads * (size_t)c.max_tokens * c.head_dim * e;
    b->K = static_cast<char*>(c.kv_storage) + (size_t)layer * layer_b;
    b->V = static_cast<char*>(c.kv_storage) + h->kv_half + (size_t)layer * layer_b;
    b->q = q;
    b->K8 = nullptr; b->Kscale = nullptr;
    if (c.index_kind == TOPK_ATTN_INDEX_INT8) {
        const char* base = static_cast<const char*>(c.kv_storage) + 2 * h->kv_half;
        const size_t layer_rows = (size_t)layer * c.n_seqs * c.n_kv_heads * (size_t)c.max_tokens;
        b->K8 = reinterpret_cast<const int8_t*>(base) + layer_rows * c.head_dim;
        b->Kscale = reinterpret_cast<const float*>(base + index_codes_bytes(&c)) + layer_rows;
    }
    b->page_centres = nullptr; b->page_balls = nullptr;
    if (c.index_kind == TOPK_ATTN_INDEX_PAGES) {
        const char* base = static_cast<const char*>(c.kv_storage) + 2 * h->kv_half;
        const size_t layer_streams = (size_t)layer * c.n_seqs * c.n_kv_heads;
        b->page_centres = base + layer_streams * (size_t)page_cap_of(&c) * c.head_dim * e;
        b->page_balls = reinterpret_cast<const float*>(base + page_centres_bytes(&c)) + layer_streams * (size_t)page_cap_of(&c) * 2;
    }
    b->page_mask = reinterpret_cast<uint64_t*>(ws + w.page_mask);
    b->page_cnt = reinterpret_cast<uint32_t*>(ws + w.page_cnt);
    b->page_list = reinterpret_cast<int32_t*>(ws + w.page_list);
    b->len = reinterpret_cast<int32_t*>(ws_len + h->ws.len) + (size_t)layer * c.n_seqs;
    b->thr = reinterpret_cast<float*>(ws + w.thr);
    b->bins = reinterpret_cast<float*>(ws + w.bins);
    b->hist = reinterpret_cast<uint32_t*>(ws + w.hist);
    b->bnd = reinterpret_cast<uint64_t*>(ws + w.bnd);
    b->tailrec = reinterpret_cast<uint32_t*>(ws + w.tailrec);
    b->samp = reinterpret_cast<float*>(ws + w.samp);
    b->seg_cnt = reinterpret_cast<uint32_t*>(ws + w.seg_cnt);
    b->seg_max = reinterpret_cast<float*>(ws + w.seg_max);
    b->seg_cnt2 = reinterpret_cast<uint32_t*>(ws + w.seg_cnt2);
    b->flags = reinterpret_cast<uint32_t*>(ws + w.flags);
    b->hmax = reinterpret_cast<float*>(ws + w.hmax);
    b->cand = reinterpret_cast<uint64_t*>(ws + w.cand);
    b->scores = reinterpret_cast<float*>(ws + w.scores);
    b->sel_idx = reinterpret_cast<int32_t*>(ws + w.sel_idx);
    b->sel_val = reinterpret_cast<float*>(ws + w.sel_val);
    b->part_acc = reinterpret_cast<float*>(ws + w.part_acc);
    b->part_l = reinterpret_cast<float*>(ws + w.part_l);
    b->part_m = reinterpret_cast<float*>(ws + w.part_m);
    b->out = nullptr; b->lse = nullptr;
    b->fallback_total = reinterpret_cast<uint32_t*>(ws + w.fallback);
}

// Split of each head's candidate list into per-wave segments for the filtered scan:
// about two 4-wave workgroups per compute unit (as many as run at once: what does not fit starts a second round, with
// its prologue in front of an idle memory system) over the whole grid, no more waves than
// key tiles, and segments large enough for their share of the expected candidates plus
// eight standard deviations.  False if no split fits (the caller takes the full path).
static bool choose_segments(const topk_attn_t* h, const Shape& s, int64_t nmax, int64_t c_hi, int* n_seg,
                            int* seg_cap) {
    // (a scan with two row tiles runs one workgroup per compute unit: its stages take the LDS)
    const bool one_per_cu = scan_row_tiles(s) && s.row_tiles == 2;
    const int64_t target_wgs = (one_per_cu ? 1 : 2) * (int64_t)h->n_cu;
    int64_t P = target_wgs / ((int64_t)scan_grid_z(s) * s.Hkv);
    const int64_t tiles = (nmax + 63) / 64;
    if (P * 4 > tiles) P = tiles / 4;
    if (P * 4 > kMaxSeg) P = kMaxSeg / 4;
    if (P > s.hist_cap) P = s.hist_cap;     // every scan workgroup leaves its per-bin candidate counts
    if (P < 1) P = 1;
    while (P & (P - 1)) P &= P - 1;          // power of two: the selection indexes segments by mask
    bool full = false;
    if (one_per_cu) {
        // the first power of two from there on whose rounds of workgroups are four fifths full, as long as a wave keeps a dozen tiles
        // (17 queries over 8 KV heads, d = 256: 192 or 384 workgroups leave a quarter of the chip empty, 768 do not: 131k tokens, k = 600
        // 338 -> 297 us; with 7 tiles a wave the split costs more than it fills: 24 queries at 60k, d = 128 153 -> 169)
        const int64_t streams = (int64_t)scan_grid_z(s) * s.Hkv, cus = h->n_cu;
        for (int64_t p = P; !full && p * 4 * 12 <= tiles && p * 4 <= kMaxSeg && p <= s.hist_cap; p *= 2)
            if (streams * p * 5 >= 4 * cus * ((streams * p + cus - 1) / cus)) { P = p; full = true; }
    }
    if (!full) {   // rounding down may leave the chip a quarter empty: take the next power of two if it stays within 1.5 x
        const int64_t streams = (int64_t)scan_grid_z(s) * s.Hkv;
        if (streams * P * 8 < target_wgs * 7 && streams * P * 2 * 2 <= target_wgs * 3 && P * 2 * 4 <= tiles &&
            P * 2 * 4 <= kMaxSeg && P * 2 <= s.hist_cap)
            P *= 2;
    }
    for (; P >= 1; P /= 2) {
        const int64_t ns = P * 4;
        const int64_t cap = (s.cand_cap / ns) & ~(int64_t)(kCandChunk - 1);
        const double mean = (double)c_hi / (double)ns;
        if ((double)cap >= mean + 8.0 * sqrt(mean) + 32.0) {
            *n_seg = (int)ns;
            *seg_cap = (int)cap;
            return true;
        }
        if (P == 1) break;
    }
    return false;
}

// Shortest and longest searched prefix over the sequences of a layer; EINVAL if a sequence is empty.
static int lengths_of(const topk_attn_t* h, int layer, int window, int64_t min_tokens, int64_t* nmin,
                      int64_t* nmax) {
    const int B = h->cfg.n_seqs;
    int64_t lo = INT64_MAX, hi = 0;
    for (int b = 0; b < B; ++b) {
        const int64_t n = h->len[(size_t)layer * B + b];
        if (n < min_tokens) return TOPK_ATTN_EINVAL;
        const int64_t p = prefix_len(n, window);
        lo = p < lo ? p : lo;
        hi = p > hi ? p : hi;
    }
    *nmin = lo; *nmax = hi;
    return TOPK_ATTN_OK;
}

// Workgroups per head of the one-launch selection over the candidate list (attend.hip), 0 where the chip-wide tail takes
// the call.  32 heads, k = 256 .. 2048, against the tail's two launches: 49 against 56 us at 48k tokens, 73 against 82 at 128k,
// 213 against 222 at 512k.  Its limits: a list and the rows to fetch fit LDS; every workgroup scores the window; the keys a workgroup scores again
// when a list turns out unusable are bounded.  Heads beyond the compute units get one workgroup each, two to a compute unit: list / tail,
// 8 to 64 heads a sequence or query, 30k to 120k tokens, k = 64 .. 2000, windows up to 2048: batches of 9 to 40 sequences d = 64 0.88 - 0.98,
// d = 128 0.92 - 0.99, d = 256 0.96 - 1.00; chunks of 9 to 64 queries d = 64 0.79 - 0.88, d = 128 0.82 - 0.91, d = 256 0.86 - 0.95; with every
// list unusable 0.97 - 1.37.  9k to 25k tokens: batches 0.81 - 1.01 (geometric mean 0.95), chunks of 25k 0.82 - 1.02 (0.90), and shorter chunks of more
// than 16384 tokens, which are filtered where the lists are taken here, 0.40 - 0.74 of the general path's time.
static int attend_list_shares(const topk_attn_t* h, const Shape& s, int64_t nmax) {
    if (h->force_redo == 2 || (int64_t)s.k + s.window > kAttendRows) return 0;
    if ((int64_t)s.window * s.D * 2 > kAttendWindowBytes) return 0;
    if (make_plan(nmax, s.k < nmax ? s.k : (int)nmax, s.indexed).c_hi > kAttendList) return 0;
    const int64_t heads = (int64_t)s.B * s.Hq;
    int64_t shares = std::max<int64_t>(1, kAttendManyHeads / heads);
    shares = std::min<int64_t>(std::min<int64_t>(shares, kAttendShares), s.n_chunk_cap);
    return nmax <= kAttendShareKeys * shares ? (int)shares : 0;
}

// Whether the general path takes one launch in all, a workgroup per key stream.  A stream's keys and its heads' selections, a wave
// per head, are one compute unit's work there, so the streams have to fill the chip, in rounds that are not half empty, and the
// group has to have heads enough, or rows bytes enough, that the selecting waves do not set the time.  One launch / scan with
// stored scores and the one-launch selection over them, 100 to 4096 tokens, k = 16 and 256, 1 to 2000 streams, range (median):
//   up to 512 tokens                                       d < 256 0.40 - 1.02 (0.78), d = 256 0.61 - 1.32 (0.88; radix select at most 1.09: 1600 streams)
//   up to 1024 tokens, from 128 streams on                 d <= 64 0.52 - 1.03 (0.78); d >= 128, 128 streams 0.88 - 1.38 (1.09)
//   groups of four, d = 64 and 128, from 256 streams on    0.56 - 1.00 (0.79)
//   smaller groups of 64 and 128                           300 streams 0.93 - 1.26 (1.06); full rounds 0.64 - 1.13 (0.85), of them
//                                                          groups of one at d = 64 0.79 - 1.24 (1.02)
//   d = 256                                                256 streams 0.89 - 1.25 (1.03), groups of 3 and 4 0.77 - 1.01 (0.95); 512
//                                                          and more 0.76 - 1.08 (0.91)
//   d = 32 beyond 1024 tokens                              below 512 streams 0.85 - 1.71 (1.18); from there on groups of four
//                                                          0.72 - 0.95 (0.86), smaller ones 0.83 - 1.71 (1.13)
static bool attend_short_applies(const Shape& s, int64_t nmax) {
    if (!scan_mfma_supported(s) || scan_row_tiles(s) || s.window != 0 || s.k > attend_short_k(nmax)) return false;
    const int64_t streams = (int64_t)s.B * s.Hkv, round = kAttendManyHeads;      // (a workgroup per compute unit)
    if (nmax <= 512) return true;
    if (nmax <= 1024 && s.D <= 64) return streams >= 128;
    if (streams < round) return false;
    const bool middle = s.D == 64 || s.D == 128;
    if (middle && s.G == 4) return true;
    if (streams * 4 < 3 * round * ((streams + round - 1) / round)) return false;  // rounds of workgroups three quarters full on average
    if (!middle && streams < 2 * round && !(s.D == 256 && s.G >= 3)) return false;
    return nmax <= 1024 || s.G * s.D >= 128;
}

// A decode call: what is launched, and with what.
struct Call {
    Shape s;
    Bufs b;
    bool fast;             // filtered scan
    int64_t nmax;          // longest searched prefix
    int64_t n_scored;      // longest sequence (general path: keys whose scores are stored)
};

static int plan_call(topk_attn_t* h, int layer, const void* q, int n_queries, int causal, int k, int window,
                     float* out, int32_t* idx, float* vals, float* lse, bool use_static, Call* call) {
    if (!h || !q || !out) return TOPK_ATTN_EINVAL;
    if (use_static && h->ws_one.total - h->ws_one.thr > kStaticScratchBytes) return TOPK_ATTN_ESCRATCH;
    if (layer < 0 || layer >= h->cfg.n_layers) return TOPK_ATTN_EINVAL;
    if (k < 1 || k > h->cfg.max_k) return TOPK_ATTN_EINVAL;
    if (window < 0 || window > h->cfg.max_window) return TOPK_ATTN_EINVAL;
    if (n_queries < 1 || n_queries > (h->cfg.max_queries > 1 ? h->cfg.max_queries : 1)) return TOPK_ATTN_EINVAL;
    if (window > h->cfg.max_tokens) window = (int)h->cfg.max_tokens;   // same result: no sequence is longer
    if ((uintptr_t)q & 15) return TOPK_ATTN_EINVAL;
    // the plans below are made for the longest searched prefix of each sequence (its last
    // query's); the earlier queries of a causal chunk search up to n_queries - 1 keys fewer
    int64_t nmin, nmax;
    if (lengths_of(h, layer, window, causal ? n_queries : 1, &nmin, &nmax) != TOPK_ATTN_OK) return TOPK_ATTN_EINVAL;
    Shape& s = call->s;
    Bufs& b = call->b;
    fill_call(h, layer, q, k, n_queries, &s, &b, use_static);
    s.window = window;
    s.causal = causal ? 1 : 0;
    b.out = out; b.lse = lse;
    if (idx) b.sel_idx = idx;
    if (vals) b.sel_val = vals;

    // the int8 index serves one query per sequence with the grouped scan layout
    const bool want_index = h->path == TOPK_ATTN_PATH_INDEX && n_queries == 1 && s.G <= 4;
    s.indexed = want_index ? 1 : 0;
    // the page index serves the grouped scan (with a window: over the pages of the searched prefix)
    const bool want_pages = h->path == TOPK_ATTN_PATH_PAGES && n_queries == 1 && s.G <= 4;
    // The batch takes the filtered scan if its longest sequence is worth it.  Shorter sequences
    // ride along whenever their candidate list fits; the few that cannot be filtered at all (a
    // handful of tokens, or k too dense) are recognised by the kernels themselves (same
    // plan_is_fast) and go straight to the exact redo of the selection, which is cheap for them.
    bool fast = false;
    if (h->path != TOPK_ATTN_PATH_FULL && scan_mfma_supported(s) && nmax > 0) {
        const Plan longest = make_plan(nmax, k < nmax ? k : (int)nmax, s.indexed);
        int64_t total = 0;               // searched tokens of the whole call
        for (int i = 0; i < s.Bc; ++i) total += prefix_len(h->len[(size_t)layer * s.Bc + i], window);
        // (the page index adds two launches: with it 20k tokens, k = 64, take 53 us filtered against 42 with all scores)
        const int64_t min_n = total >= kFilterBatchTokens ? kFilterMinNBatch
                              : attend_list_shares(h, s, nmax) && !want_pages ? kAttendRowMax + 1 : kFilterMinN;
        fast = plan_is_fast(longest, nmax, s.cand_cap, h->path == TOPK_ATTN_PATH_FILTER, min_n);
        int64_t c_hi = 0;
        for (int i = 0; i < s.Bc && fast; ++i) {
            const int64_t n = prefix_len(h->len[(size_t)layer * s.Bc + i], window);
            if (n == 0) continue;            // this sequence lies entirely inside its window
            const Plan pl = make_plan(n, k < n ? k : (int)n, s.indexed);
            if (plan_is_fast(pl, n, s.cand_cap, true)) c_hi = pl.c_hi > c_hi ? pl.c_hi : c_hi;
        }
        if (fast) fast = choose_segments(h, s, nmax, c_hi, &s.n_seg, &s.seg_cap);
        if (fast) {     // tail: about 128 selected rows per workgroup and at most four scan workgroups each
            // (a tail workgroup walks its scan workgroups one after the other: dependent loads each time)
            const int n_wg = s.n_seg / 4;
            int want = (k + 127) / 128;
            if (want < (n_wg + 3) / 4) want = (n_wg + 3) / 4;
            want = want < 1 ? 1 : (want > n_wg ? n_wg : want);
            s.tail_spw = (n_wg + want - 1) / want;
            s.tail_wgs = (n_wg + s.tail_spw - 1) / s.tail_spw;
        }
    }
    if (!fast) s.indexed = 0;      // no filtered scan: exact path
    if (fast && s.indexed) s.no_rescan = 1;   // (the per-bin counts cover the listed candidates only: an unusable list is redone densely)
    // the selection that follows the filtered scan has limits of its own (count vectors, partial-sum slots); they hold
    // for every shape the scan takes with this workspace, and a shape beyond them takes the exact path like any other
    if (fast && !tail_supported(s)) { fast = false; s.indexed = 0; s.no_rescan = 0; }
    // Selection and attention in one launch, where the work per head is small: over the candidate list, or over the
    // score rows of the general path.
    if (fast) s.attend = attend_list_shares(h, s, nmax);
    else if (attend_short_applies(s, nmax)) s.attend = kAttendShort;
    else s.attend = attend_row_applies((int64_t)s.B * s.Hq, nmax, s.k, s.window, s.D * elem_bytes(s.dtype)) ? 1 : 0;
    s.share_wgs = s.attend;
    if (fast && !s.indexed) {
        s.paged = want_pages ? 1 : 0;
        s.no_rescan = s.paged;      // the paged scan deals its tiles to the waves by rank among the pages kept
    }
    call->fast = fast;
    call->nmax = call->n_scored = nmax;
    if (s.attend)                   // the window's scores come from the scan too
        for (int i = 0; i < s.Bc; ++i) call->n_scored = std::max(call->n_scored, h->len[(size_t)layer * s.Bc + i]);
    return TOPK_ATTN_OK;
}

static int enqueue_call(topk_attn_t* h, const Call& call, int layer, hipStream_t st, bool use_static) {
    const Shape& s = call.s;
    const Bufs& b = call.b;
    const bool fast = call.fast;
    const int64_t nmax = call.nmax;
    hipError_t e = hipSuccess;
    bool tail_done = false;
    if (use_static) {
        // the array keeps what the last call on this GPU left: the per-head control words start at zero
        // (a fill kernel, so that the call may be recorded into a HIP graph)
        uint32_t* first = b.flags;
        const size_t n_words = (size_t)(reinterpret_cast<char*>(b.fallback_total) + sizeof(uint32_t) -
                                        reinterpret_cast<char*>(first)) / sizeof(uint32_t);
        hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)((n_words + 255) / 256 < 64 ? (n_words + 255) / 256 : 64)),
                           dim3(256), 0, st, first, n_words);
        e = hipGetLastError();
    }
    const bool timed = h->timing && h->ev_used < kTimingSlots;
    if (fast && s.indexed) {
        e = launch_scan8_sample(s, b, nmax, st);
        if (e == hipSuccess) e = launch_threshold(s, b, nmax, st);
        if (e == hipSuccess && timed) e = hipEventRecord(h->ev[2 * h->ev_used], st);
        if (e == hipSuccess) e = launch_scan8_filter(s, b, st);
        if (e == hipSuccess && timed) e = hipEventRecord(h->ev[2 * h->ev_used + 1], st);
        if (e == hipSuccess && timed) h->ev_used++;
        if (e == hipSuccess) e = launch_rerank(s, b, st);              // exact scores, and their per-bin counts for the tail
        if (e == hipSuccess) e = launch_tail(s, b, st);                // (with a window: its partial sums too)
        tail_done = true;
    } else if (fast) {
        e = launch_scan_sample(s, b, nmax, st);
        if (e == hipSuccess) e = launch_threshold(s, b, nmax, st);
        if (e == hipSuccess && s.paged) e = launch_page_filter(s, b, h->page_beta, st);
        if (e == hipSuccess && timed) e = hipEventRecord(h->ev[2 * h->ev_used], st);
        if (e == hipSuccess) e = s.paged ? launch_scan_filter_paged(s, b, st) : launch_scan_filter(s, b, nmax, st);
        if (e == hipSuccess && timed) e = hipEventRecord(h->ev[2 * h->ev_used + 1], st);
        if (e == hipSuccess && timed) h->ev_used++;
        if (e == hipSuccess) e = launch_tail(s, b, st);                // selection and gather (with a window: its partial sums too); redoes unusable heads itself
        tail_done = true;
    } else {
        if (nmax > 0 || s.attend) {
            Shape all = s;
            if (s.attend) all.window = 0;    // the window's scores come from the scan too
            if (timed) e = hipEventRecord(h->ev[2 * h->ev_used], st);
            if (e == hipSuccess) e = s.attend == kAttendShort ? launch_select_full(s, b, nmax, st) : launch_scan_full(all, b, call.n_scored, b.scores, st);
            if (e == hipSuccess && timed) e = hipEventRecord(h->ev[2 * h->ev_used + 1], st);
            if (e == hipSuccess && timed) h->ev_used++;
        }
        if (e == hipSuccess && s.attend != kAttendShort) e = launch_select_full(s, b, nmax, st);   // with nothing to search it only pads
    }
    if (e == hipSuccess && !tail_done && !s.attend) e = launch_gather(s, b, st);
    h->last_fast = fast;
    h->last_paged = fast && s.paged;
    h->last_tail = tail_done;
    h->last_queries = s.M;
    h->last_n_seg = fast ? s.n_seg : 0;
    h->last_seg_cap = fast ? s.seg_cap : 0;
    h->last_slot = (1 << s.log2_layers) - 1;
    h->last_layer = layer + h->last_slot;
    h->last_static = use_static;
    return e == hipSuccess ? TOPK_ATTN_OK : TOPK_ATTN_EDEVICE;
}

static int decode_impl(topk_attn_t* h, int layer, const void* q, int n_queries, int causal, int k, int window,
                       float* out, int32_t* idx, float* vals, float* lse, void* hip_stream, bool use_static = false) {
    Call call;
    const int rc = plan_call(h, layer, q, n_queries, causal, k, window, out, idx, vals, lse, use_static, &call);
    return rc != TOPK_ATTN_OK ? rc : enqueue_call(h, call, layer, (hipStream_t)hip_stream, use_static);
}

// Whether layers share their launches with the layer of `all`, and how many at most.  A layer is taken through exactly the
// launch shapes it has alone (the same segments, shares and workgroups), so its results are the same bits; only how many of them are
// in flight differs.  (Not while the scans are timed one by one.)
static bool joins(const topk_attn_t* h, const Call& all, const Call& one, int layers) {
    const Shape &s = all.s, &o = one.s;
    if (h->timing || layers > h->ws.batch_layers || s.paged || s.indexed || !s.attend || all.fast != one.fast || o.attend != s.attend) return false;
    const int64_t nmax = std::max(all.nmax, one.nmax), layer_heads = (int64_t)s.layer_seqs * s.Hq, heads = layer_heads * layers;
    // filtered: one round of workgroups, and no more keys for one of them to score again than alone
    if (all.fast)
        return s.n_seg == o.n_seg && s.seg_cap == o.seg_cap && heads <= kAttendManyHeads &&
               nmax <= kAttendShareKeys * std::max<int64_t>(1, kAttendManyHeads / heads);
    if (s.attend == kAttendShort) return std::max(s.k, o.k) <= attend_short_k(nmax);
    return attend_row_class(layer_heads, all.nmax) == attend_row_class(layer_heads, one.nmax);
}

// Makes one call of the calls of n consecutive layers (a power of two, all of which join the first).
static Call join_layers(const Call* calls, int n) {
    Call all = calls[0];
    Shape& s = all.s;
    for (int i = 1; i < n; ++i) {
        const Call& one = calls[i];
        all.b.layer_k[i] = LayerK{one.s.k, all.b.layer_k[i - 1].before + all.b.layer_k[i - 1].k};
        s.k = std::max(s.k, one.s.k);
        all.nmax = std::max(all.nmax, one.nmax);
        all.n_scored = std::max(all.n_scored, one.n_scored);
    }
    while ((1 << s.log2_layers) < n) ++s.log2_layers;
    s.Bc = s.B = s.layer_seqs * n;
    if (all.fast) s.share_wgs = (int)std::max<int64_t>(1, std::min<int64_t>(s.attend, kAttendManyHeads / ((int64_t)s.B * s.Hq)));
    return all;
}

int topk_attn_decode(topk_attn_t* h, int layer, const void* q, int k, float* out, int32_t* idx, float* vals,
                     float* lse, void* hip_stream) {
    return decode_impl(h, layer, q, 1, 0, k, 0, out, idx, vals, lse, hip_stream);
}

int topk_attn_decode_static(topk_attn_t* h, int layer, const void* q, int k, float* out, int32_t* idx, float* vals,
                            float* lse, void* hip_stream) {
    return decode_impl(h, layer, q, 1, 0, k, 0, out, idx, vals, lse, hip_stream, true);
}

int topk_attn_decode_window(topk_attn_t* h, int layer, const void* q, int k, int window, float* out, int32_t* idx,
                            float* vals, float* lse, void* hip_stream) {
    return decode_impl(h, layer, q, 1, 0, k, window, out, idx, vals, lse, hip_stream);
}

int topk_attn_decode_multi(topk_attn_t* h, int layer, const void* q, int n_queries, int causal, int k, int window,
                           float* out, int32_t* idx, float* vals, float* lse, void* hip_stream) {
    return decode_impl(h, layer, q, n_queries, causal, k, window, out, idx, vals, lse, hip_stream);
}

int topk_attn_decode_layers(topk_attn_t* h, int layer0, int n_layers, const void* q, const int32_t* k, int window,
                            float* out, int32_t* idx, float* vals, float* lse, void* hip_stream) {
    if (!h || !q || !out || !k) return TOPK_ATTN_EINVAL;
    if (n_layers < 1 || layer0 < 0 || layer0 > h->cfg.n_layers - n_layers) return TOPK_ATTN_EINVAL;
    if (window < 0 || window > h->cfg.max_window || ((uintptr_t)q & 15)) return TOPK_ATTN_EINVAL;
    for (int l = 0; l < n_layers; ++l) {
        if (k[l] < 1 || k[l] > h->cfg.max_k) return TOPK_ATTN_EINVAL;
        for (int b = 0; b < h->cfg.n_seqs; ++b)
            if (h->len[(size_t)(layer0 + l) * h->cfg.n_seqs + b] < 1) return TOPK_ATTN_EINVAL;
    }
    const size_t BH = (size_t)h->cfg.n_seqs * h->cfg.n_q_heads;
    const size_t q_step = BH * h->cfg.head_dim * elem_bytes(h->cfg.dtype);
    size_t sel_off = 0;
    std::unique_ptr<Call[]> calls(new (std::nothrow) Call[(size_t)n_layers]);     // (no exception may leave a C entry)
    if (!calls) return TOPK_ATTN_ENOMEM;
    for (int l = 0; l < n_layers; ++l) {
        const int rc = plan_call(h, layer0 + l, static_cast<const char*>(q) + l * q_step, 1, 0, k[l], window,
                                 out + l * BH * h->cfg.head_dim, idx ? idx + sel_off : nullptr,
                                 vals ? vals + sel_off : nullptr, lse ? lse + l * BH : nullptr, false, &calls[l]);
        if (rc != TOPK_ATTN_OK) return rc;
        sel_off += BH * (size_t)k[l];
    }
    for (int l = 0, n; l < n_layers; l += n) {
        Call all = calls[l];
        for (n = 1; 2 * n <= n_layers - l; n *= 2) {        // twice as many layers, as long as all of them join
            bool ok = true;
            for (int i = n; ok && i < 2 * n; ++i) {
                ok = joins(h, all, calls[l + i], 2 * n);
                all.nmax = std::max(all.nmax, calls[l + i].nmax);
                all.s.k = std::max(all.s.k, calls[l + i].s.k);
            }
            if (!ok) break;
        }
        const int rc = enqueue_call(h, n > 1 ? join_layers(&calls[l], n) : calls[l], layer0 + l, (hipStream_t)hip_stream, false);
        if (rc != TOPK_ATTN_OK) return rc;
    }
    return TOPK_ATTN_OK;
}

int topk_attn_k_schedule(int64_t total_k, int n_layers, double last_over_first, int32_t* k_out) {
    if (!k_out || n_layers < 1 || total_k < n_layers) return TOPK_ATTN_EINVAL;
    if (!(last_over_first > 0.0) || !std::isfinite(last_over_first)) return TOPK_ATTN_EINVAL;
    std::vector<double> w((size_t)n_layers);
    double wsum = 0.0;
    for (int l = 0; l < n_layers; ++l) {
        w[l] = n_layers == 1 ? 1.0 : 1.0 + (last_over_first - 1.0) * (double)l / (double)(n_layers - 1);
        wsum += w[l];
    }
    std::vector<int64_t> k((size_t)n_layers);
    std::vector<std::pair<double, int>> frac((size_t)n_layers);
    int64_t used = 0;
    for (int l = 0; l < n_layers; ++l) {
        const double exact = (double)total_k * w[l] / wsum;
        int64_t fl = (int64_t)floor(exact);
        if (fl < 1) fl = 1;                       // every layer attends to at least one key
        k[l] = fl;
        used += fl;
        frac[l] = {exact - (double)fl, l};
    }
    // hand out (or, after the >= 1 clamp, take back) the remainder by fractional part
    std::sort(frac.begin(), frac.end(), [](const std::pair<double, int>& a, const std::pair<double, int>& b) {
        return a.first != b.first ? a.first > b.first : a.second > b.second;
    });
    int64_t rem = total_k - used;
    for (int i = 0; rem > 0; i = (i + 1) % n_layers, --rem) k[frac[i].second] += 1;
    for (int i = n_layers - 1; rem < 0; i = (i + n_layers - 1) % n_layers) {
        if (k[frac[i].second] > 1) { k[frac[i].second] -= 1; ++rem; }
    }
    for (int l = 0; l < n_layers; ++l) {
        if (k[l] > INT32_MAX) return TOPK_ATTN_EINVAL;
        k_out[l] = (int32_t)k[l];
    }
    return TOPK_ATTN_OK;
}

int topk_attn_scores(topk_attn_t* h, int layer, const void* q, float* scores, void* hip_stream) {
    if (!h || !q || !scores) return TOPK_ATTN_EINVAL;
    if (layer < 0 || layer >= h->cfg.n_layers) return TOPK_ATTN_EINVAL;
    if ((uintptr_t)q & 15) return TOPK_ATTN_EINVAL;
    int64_t nmin, nmax;
    if (lengths_of(h, layer, 0, 1, &nmin, &nmax) != TOPK_ATTN_OK) return TOPK_ATTN_EINVAL;
    Shape s; Bufs b;
    fill_call(h, layer, q, 1, 1, &s, &b);
    hipError_t e;
    if (h->path == TOPK_ATTN_PATH_INDEX && s.G <= 4) {   // approximate scores from the codes
        e = launch_scan8_full(s, b, nmax, scores, (hipStream_t)hip_stream);
    } else {
        e = launch_scan_full(s, b, nmax, scores, (hipStream_t)hip_stream);
    }
    return e == hipSuccess ? TOPK_ATTN_OK : TOPK_ATTN_EDEVICE;
}

int topk_attn_last_fallbacks(topk_attn_t* h, int* n_heads) {
    if (!h || !n_heads) return TOPK_ATTN_EINVAL;
    *n_heads = 0;
    if (!h->last_fast) return TOPK_ATTN_OK;
    uint32_t v = 0;
    const char* where = h->last_static ? h->scratch_dev + (h->ws_one.fallback - h->ws_one.thr)
                                       : static_cast<char*>(h->cfg.workspace) + h->ws.fallback;
    if (hipMemcpy(&v, where, sizeof v, hipMemcpyDeviceToHost) !=
        hipSuccess)
        return TOPK_ATTN_EDEVICE;
    *n_heads = (int)v;
    return TOPK_ATTN_OK;
}

int topk_attn_set_page_bound_scale(topk_attn_t* h, float beta) {
    if (!h || h->cfg.index_kind != TOPK_ATTN_INDEX_PAGES || !(beta > 0.0f) || beta > 1.0f) return TOPK_ATTN_EINVAL;
    h->page_beta = beta;
    return TOPK_ATTN_OK;
}

int topk_attn_last_pages_read(topk_attn_t* h, int64_t* pages_read, int64_t* pages_total) {
    if (!h || !pages_read || !pages_total) return TOPK_ATTN_EINVAL;
    const topk_attn_config& c = h->cfg;
    int64_t total = 0;
    for (int b = 0; b < c.n_seqs; ++b) total += (h->len[(size_t)h->last_layer * c.n_seqs + b] + 63) / 64 * c.n_kv_heads;
    *pages_total = total;
    *pages_read = total;                       // every page, unless the last decode went through the page index
    if (!h->last_paged || h->last_static) return TOPK_ATTN_OK;
    const size_t words = (size_t)c.n_seqs * c.n_kv_heads * h->ws.page_words;
    std::vector<uint64_t> mask(words);
    if (hipMemcpy(mask.data(), static_cast<char*>(c.workspace) + h->ws.page_mask, words * sizeof(uint64_t),
                  hipMemcpyDeviceToHost) != hipSuccess)
        return TOPK_ATTN_EDEVICE;
    int64_t read = 0;
    for (uint64_t w : mask) read += __builtin_popcountll(w);
    *pages_read = read;
    return TOPK_ATTN_OK;
}

int topk_attn_last_selection_records(topk_attn_t* h, uint32_t* records) {
    if (!h || !records || !h->last_tail || h->last_static) return TOPK_ATTN_EINVAL;
    const topk_attn_config& c = h->cfg;
    const size_t n = (size_t)c.n_seqs * h->last_queries * c.n_q_heads;
    if (hipMemcpy(records, static_cast<char*>(c.workspace) + h->ws.tailrec + h->last_slot * n * 4 * sizeof(uint32_t), n * 4 * sizeof(uint32_t), hipMemcpyDeviceToHost) !=
        hipSuccess)
        return TOPK_ATTN_EDEVICE;
    std::vector<uint32_t> flags(n);
    if (hipMemcpy(flags.data(), static_cast<char*>(c.workspace) + h->ws.flags + h->last_slot * n * sizeof(uint32_t), n * sizeof(uint32_t), hipMemcpyDeviceToHost) !=
        hipSuccess)
        return TOPK_ATTN_EDEVICE;
    for (size_t i = 0; i < n; ++i) records[4 * i] |= (flags[i] % kArrivalUnit) << 8;      // the head's flag word above the state
    return TOPK_ATTN_OK;
}

int topk_attn_debug_read_workspace(topk_attn_t* h, const char* name, void* dst, size_t bytes) {
    if (!h || !name || !dst) return TOPK_ATTN_EINVAL;
    const WsLayout& w = h->ws;
    const size_t per_seg = 4 * (size_t)h->last_n_seg;        // (these arrays hold the segments the call used, head after head)
    const struct { const char* name; size_t at, end, per_head; } arrays[] = {
        {"thr", w.thr, w.bins, 4}, {"bins", w.bins, w.samp, 8}, {"samp", w.samp, w.seg_cnt, 4 * kSampMax}, {"seg_cnt", w.seg_cnt, w.seg_max, per_seg},
        {"seg_max", w.seg_max, w.seg_cnt2, per_seg}, {"seg_cnt2", w.seg_cnt2, w.flags, per_seg}, {"flags", w.flags, w.hmax, 4},
        {"tailrec", w.tailrec, w.page_mask, 16}, {"page_mask", w.page_mask, w.page_cnt, 0}, {"page_cnt", w.page_cnt, w.page_list, 0},
        {"page_list", w.page_list, w.hist, 0}, {"hist", w.hist, w.cand, (size_t)w.hist_cap * kTailBins * 4},
        {"cand", w.cand, w.bnd, (size_t)w.cand_cap * 8}, {"bnd", w.bnd, w.scores, (size_t)w.bnd_cap * 8}};
    for (const auto& a : arrays) {
        if (strcmp(a.name, name) != 0) continue;
        const size_t at = a.at + (size_t)h->last_slot * h->cfg.n_seqs * h->cfg.n_q_heads * a.per_head;     // (the last layer of the call)
        if (at > a.end || bytes > a.end - at) return TOPK_ATTN_EINVAL;
        return hipMemcpy(dst, static_cast<char*>(h->cfg.workspace) + at, bytes, hipMemcpyDeviceToHost) == hipSuccess
                   ? TOPK_ATTN_OK : TOPK_ATTN_EDEVICE;
    }
    return TOPK_ATTN_EINVAL;
}

int topk_attn_debug_read_workspace_dims(topk_attn_t* h, int32_t* dims) {
    if (!h || !dims) return TOPK_ATTN_EINVAL;
    dims[0] = h->ws.cand_cap; dims[1] = h->ws.bnd_cap; dims[2] = h->ws.hist_cap; dims[3] = kMaxSeg;
    dims[4] = h->last_n_seg; dims[5] = h->last_seg_cap;
    return TOPK_ATTN_OK;
}

int topk_attn_debug_force_redo(topk_attn_t* h, int enable) {
    if (!h) return TOPK_ATTN_EINVAL;
    h->force_redo = enable == 2 ? 2 : enable != 0;
    return TOPK_ATTN_OK;
}

int topk_attn_set_scan_timing(topk_attn_t* h, int enable) {
    if (!h) return TOPK_ATTN_EINVAL;
    if (enable && h->ev.empty()) {
        h->ev.resize(2 * kTimingSlots);
        for (size_t i = 0; i < h->ev.size(); ++i) {
            if (hipEventCreate(&h->ev[i]) != hipSuccess) {
                for (size_t j = 0; j < i; ++j) (void)hipEventDestroy(h->ev[j]);
                h->ev.clear();
                return TOPK_ATTN_EDEVICE;
            }
        }
    }
    h->timing = enable != 0;
    h->ev_used = 0;
    return TOPK_ATTN_OK;
}

int topk_attn_scan_time(topk_attn_t* h, double* total_ms, int* n_calls) {
    if (!h || !total_ms || !n_calls) return TOPK_ATTN_EINVAL;
    double sum = 0.0;
    for (int i = 0; i < h->ev_used; ++i) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, h->ev[2 * i], h->ev[2 * i + 1]) != hipSuccess) return TOPK_ATTN_EDEVICE;
        sum += ms;
    }
    *total_ms = sum;
    *n_calls = h->ev_used;
    h->ev_used = 0;
    return TOPK_ATTN_OK;
}

int topk_attn_read_probe(const void* src, size_t bytes, void* sink, void* hip_stream) {
    if (!src || !sink || bytes == 0 || (bytes & 15) || ((uintptr_t)src & 15)) return TOPK_ATTN_EINVAL;
    const size_t n_vec = bytes / 16;
    size_t blocks = (n_vec + 4095) / 4096;      // one tile per wave at least
    if (blocks > 512) blocks = 512;             // two workgroups per compute unit, like the key scan
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(read_probe_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)hip_stream,
                       static_cast<const u32x4*>(src), n_vec, static_cast<uint32_t*>(sink));
    return hipGetLastError() == hipSuccess ? TOPK_ATTN_OK : TOPK_ATTN_EDEVICE;
}

#ifndef TKA_BUILD_ID
#define TKA_BUILD_ID "unknown"
#endif
// the tag in front lets a script find the identifier in the file without loading it
static const char kBuildTag[] = "tka-build-id:" TKA_BUILD_ID;
const char* topk_attn_build_id(void) { return kBuildTag + 13; }

const char* topk_attn_strerror(int code) {
    switch (code) {
        case TOPK_ATTN_OK: return "ok";
        case TOPK_ATTN_EINVAL: return "invalid argument";
        case TOPK_ATTN_ECAPACITY: return "cache capacity exceeded";
        case TOPK_ATTN_EUNSUPPORTED: return "unsupported configuration";
        case TOPK_ATTN_EDEVICE: return "HIP error";
        case TOPK_ATTN_ENOMEM: return "out of memory or buffer too small";
        case TOPK_ATTN_ESCRATCH: return "configuration needs more per-call scratch than the library's built-in buffer holds";
        default: return "unknown error";
    }
}

}  // extern "C"

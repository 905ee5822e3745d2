// Exact top-k selection (the result of the paper's knn_search: the k largest scores
// `vals` and their positions `I`), by radix select.  Scores are compared through an
// order-preserving 32-bit image of the fp32 value; when the k-th score is shared by more
// items than fit, a second radix select over the (unique) inverted positions of those
// items picks the lowest positions, so equal scores resolve to the lower position and the
// selected set never depends on the order in which candidates were produced.
// One workgroup per (sequence, head).
//
// The first CPT * kSelThreads items of a head keep their score key in registers for all
// passes (and, for candidate lists, their position in LDS); anything beyond is re-read
// from memory in batches of independent loads.  Output order is fixed (wave-major), so
// repeated calls return bit-identical results.
#include "device_utils.h"
#include "internal.h"
#include "select_common.h"
#include "threshold.h"

namespace tka {

// Threshold of each head from its sample (threshold.h), a workgroup per head.
template <int CPT, int NT>     // NT threads; the launcher makes sure n_samp <= CPT * NT <= samp_cap
__global__ void __launch_bounds__(NT) threshold_kernel(Shape sh, Bufs bf) {
    fetch_args<kArgBytes>();
    using Team = WorkgroupTeam<NT>;
    __shared__ ThresholdShared<Team> sm;
    const int b = blockIdx.y + blockIdx.z * sh.layer_seqs, h = blockIdx.x;
    const int tid = threadIdx.x;
    const int64_t bh = (int64_t)b * sh.Hq + h;
    const int k = bf.layer_k[blockIdx.z].k;
    // the sample scores are asked for before the sample size is known (it depends on the sequence
    // length, another trip to memory); what lies beyond the sample is ignored
    const float* samp = bf.samp + bh * sh.samp_cap;
    float sv[CPT];
#pragma unroll
    for (int j = 0; j < CPT; ++j) sv[j] = samp[j * NT + tid];
    for (int i = tid; i < kThrBins; i += NT) sm.hist[i] = 0;
    if (prefix_len(visible_len(sh, bf, b), sh.window) == 0) {   // nothing to search for this sequence
        if (tid == 0) leave_threshold(bf, bh, Threshold{INFINITY, 0.f, 0.f}, 0u);
        return;
    }
    // the sample was drawn by the plan of the cache sequence (shared by all its queries)
    const int64_t N = prefix_len(bf.len[cache_seq(sh, b)], sh.window);
    const Plan pl = make_plan(N, k < N ? k : (int)N, sh.indexed);
    const Threshold t = estimate_threshold<Team, CPT>(sv, pl, sm);
    if (tid == 0) leave_threshold(bf, bh, t, threshold_flags(sh, pl, N));
}

// Exact selection over the full score row, already in the score buffer (general path).
// NT threads per head: a batch of many short sequences is thousands of heads of a few
// thousand scores each, and a workgroup no larger than the row needs keeps more heads in
// flight per compute unit and makes every barrier of the select cheaper.
template <int NT, int CPT>
__global__ void __launch_bounds__(NT) select_full_kernel(Shape sh, Bufs bf) {
    fetch_args<kArgBytes>();
    __shared__ SelShared sm;
    const int b = blockIdx.y, h = blockIdx.x;
    const int64_t bh = (int64_t)b * sh.Hq + h;
    const int64_t N = prefix_len(visible_len(sh, bf, b), sh.window);
    const int k_eff = sh.k < N ? sh.k : (int)N;
    if (k_eff == 0) {
        pad_outputs(0, sh.k, bf.sel_idx + bh * sh.k, bf.sel_val + bh * sh.k);
        if (threadIdx.x == 0) bf.hmax[bh] = -INFINITY;
        return;
    }
    wg_select_dense<NT, CPT>(sh, bf, bh, N, k_eff, sh.k, bf.sel_idx + bh * sh.k, bf.sel_val + bh * sh.k, sm);
}

hipError_t launch_threshold(const Shape& s, const Bufs& b, int64_t Nmax, hipStream_t st) {
    if (threshold_in_scan(s, Nmax)) return hipSuccess;
    const int n_samp = make_plan(Nmax, s.k < Nmax ? s.k : (int)Nmax, s.indexed).n_samp;
    const dim3 grid(s.Hq, s.layer_seqs, 1u << s.log2_layers);
    static_assert(kSampMax <= 32 * 256, "the threshold kernel keeps every sample score in registers");
    // four waves per head whatever the sample size: the kernel is a chain of short phases between
    // barriers, which cost more with sixteen waves than the longer per-thread loops do with four
#define TKA_TH(CPT_, NT_) hipLaunchKernelGGL((threshold_kernel<CPT_, NT_>), grid, dim3(NT_), 0, st, s, b)
    if (n_samp <= 1024) TKA_TH(4, 256);
    else if (n_samp <= 2048) TKA_TH(8, 256);
    else if (n_samp <= 4096) TKA_TH(16, 256);
    else TKA_TH(32, 256);
#undef TKA_TH
    return hipGetLastError();
}
// The kernel is correct for any register-cache size (what does not fit is streamed); a
// cache much larger than the data only costs loop trips over empty slots, which matters
// when the whole step is a few tens of microseconds.
hipError_t launch_select_full(const Shape& s, const Bufs& b, int64_t Nmax, hipStream_t st) {
    if (s.attend == kAttendShort) return launch_attend_short(s, b, Nmax, st);
    if (s.attend) return launch_attend_row(s, b, Nmax, st);
    const dim3 grid(s.Hq, s.B);
#define TKA_SF(NT_, CPT_) hipLaunchKernelGGL((select_full_kernel<NT_, CPT_>), grid, dim3(NT_), 0, st, s, b)
    // workgroup size and register-cached scores per thread by the longest row of the call
    // (measured on batches of 256..4096 short sequences; any choice is correct)
    if (Nmax <= 512) TKA_SF(64, 8);
    else if (Nmax <= 1024) TKA_SF(64, 16);
    else if (Nmax <= 2048) TKA_SF(128, 16);
    else if (Nmax <= 4096) TKA_SF(256, 16);
    else if (Nmax <= 8192) TKA_SF(256, 32);
    else TKA_SF(kSelThreads, 8);
#undef TKA_SF
    return hipGetLastError();
}

}  // namespace tka

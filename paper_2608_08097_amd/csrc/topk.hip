// Top-K selection per (request, KV head) (paper §4.2.1-§4.2.2; §5.2: K = 128
// blocks of 16 tokens, and the budget is the sparsification threshold): one
// workgroup per (request, KV head) runs the exact select of select.h over the
// candidates of its score row.
#include "oasis_internal.h"
#include "select.h"

namespace oasis {

namespace {

constexpr int kThreads = 1024;
// Rows of at most 2,048 blocks take half the threads, so that four of them
// share a CU and few threads are idle. Measured on MI355X, scores and selection
// of 512 rows of 1,088 blocks: 1,024 threads 45.5 us, 512 44.0, 256 44.1; of 256
// rows of 2,048 blocks 49.0, 48.6 and 49.8.
constexpr int kShortThreads = 512;
constexpr int kShortKeys = 4;

// Two 1,024-thread workgroups share a CU only if eight waves fit each SIMD: at
// most 64 VGPRs, and 80 SGPRs of the SIMD's 800 (rounded up to 16, beside 16 of
// the trap handler). The ballot masks alone take more with 8 keys per thread and
// up, and 512 rows then ran in two rounds. Measured on MI355X, 512 rows, k = 128,
// without and with the bound of eight waves (256 rows beside it): 4,096 blocks
// 15.2 and 10.6 us (7.9), 8,192 blocks 19.8 and 16.3 us (11.3).
constexpr int kTwoPerCu = 16;  // keys per thread up to which the registers fit

template <int NTHR, int KPT>
__global__ __launch_bounds__(NTHR, KPT <= kTwoPerCu ? 8 : 4) void topk_kernel(TopkArgs a) {
  __shared__ SelectShared<NTHR, KPT> sh;
  const int rh = blockIdx.x;
  const int r = rh / a.Hkv;
  const Ctx c = ctx_blocks(a.ctx_len[r], a.B, a.NBmax);
  const float* s = a.scores + (long long)rh * a.NBmax;
  select_row<NTHR, KPT>([&](int i) { return select_key(s[i]); }, c.n_cand, a.k, a.sel + (long long)rh * a.k,
                            a.sel_count + rh, sh);
}

}  // namespace

hipError_t launch_topk(const TopkArgs& a, hipStream_t s, const LaunchTiming& t) {
  // the candidate count of every request is at most NBmax - 1
  const int per = (a.NBmax + kThreads - 1) / kThreads;
  const dim3 grid((unsigned)(a.R * a.Hkv));
  if (a.NBmax <= kShortThreads * kShortKeys)
    launch_kernel(topk_kernel<kShortThreads, kShortKeys>, grid, dim3(kShortThreads), s, t, a);
  else if (per <= 4)  // (rows of 2,100 to 4,096 blocks: 8 keys 5 to 10 % slower)
    launch_kernel(topk_kernel<kThreads, 4>, grid, dim3(kThreads), s, t, a);
  else if (per <= 8)
    launch_kernel(topk_kernel<kThreads, 8>, grid, dim3(kThreads), s, t, a);
  else if (per <= 16)
    launch_kernel(topk_kernel<kThreads, 16>, grid, dim3(kThreads), s, t, a);
  else if (per <= 32)
    launch_kernel(topk_kernel<kThreads, 32>, grid, dim3(kThreads), s, t, a);
  else
    launch_kernel(topk_kernel<kThreads, 0>, grid, dim3(kThreads), s, t, a);
  return hipGetLastError();
}

}  // namespace oasis

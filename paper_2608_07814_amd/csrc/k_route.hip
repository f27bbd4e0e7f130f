// Top-k of the unchanged router, on the GPU: the k largest logits in
// descending order (equal logits: lower expert index first; NaN below every
// number), weights = the softmax of the chosen logits (= the full softmax
// restricted to them and renormalised).
//
// The logits themselves (x W_r^T, fp32 accumulation of exact bf16 products)
// come from the skinny GEMM over implicit 32-row tiles. When the tiles are
// too few to stream W_r at speed, that GEMM is split along d and leaves S
// partial tiles per (row tile, 64-column tile) item in the workspace; this
// kernel adds them in split order while it reads the logits, so the pair
// needs no counters and stays run-to-run deterministic.
//
// One wavefront per token: lane l holds experts l, l + 64, ...; k rounds of
// a wavefront-wide (value, lower index) maximum; then the softmax over the
// chosen values, lanes 0 .. k-1 holding one chosen expert each.
#include "lx_internal.h"
#include "lx_topk.h"

namespace lx {
namespace {

constexpr int TK_WAVES = 4;

template <int PER, bool SWAP>
__global__ __launch_bounds__(TK_WAVES * 64) void k_topk(const float* __restrict__ logits,
                                                        const float* __restrict__ part, int S, int T, int E,
                                                        int k, int32_t* __restrict__ ids,
                                                        float* __restrict__ weights) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * TK_WAVES + (threadIdx.x >> 6);
  if (t >= T) return;  // whole wavefront
  int id;
  float wt;
  topk_token<PER, SWAP>(logits, part, S, E, k, t, id, wt);
  if (lane < k) {
    ids[(int64_t)t * k + lane] = id;
    weights[(int64_t)t * k + lane] = wt;
  }
}

// The same, then the token's distinct nodes at every level counted into its
// 64-token tile's histogram column (integer adds: order-free, so exact; the
// histograms are clear on entry). One launch instead of the top-k's and the
// histogram's, and the whole chip's wavefronts for the top-k: inside the
// histogram pass (one workgroup per 64 tokens) it took 33 us at T = 4096, E = 128
// and 59 us at T = 777, E = 256; here 18 and 20.
template <int PER, bool SWAP>
__global__ __launch_bounds__(TK_WAVES * 64) void k_topk_hist(RouteIn r, BucketArgs a) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * TK_WAVES + (threadIdx.x >> 6);
  if (t >= a.T) return;  // whole wavefront
  const int k = a.k;
  int id;
  float wt;
  topk_token<PER, SWAP>(r.logits, r.part, r.S, a.E, k, t, id, wt);
  if (lane < k) {
    const_cast<int32_t*>(a.ids)[(int64_t)t * k + lane] = id;
    const_cast<float*>(a.w)[(int64_t)t * k + lane] = wt;
  }
  int n[kMaxLvl];  // every level's node, loaded together
#pragma unroll
  for (int l = 0; l < kMaxLvl; ++l) n[l] = l <= a.L && lane < k ? a.anc[(int64_t)l * a.E + id] : -1;
#pragma unroll
  for (int l = 0; l < kMaxLvl; ++l) {
    if (l > a.L) break;
    bool first = n[l] >= 0;
    for (int j = 0; j < k; ++j) first &= !(j < lane && __builtin_amdgcn_readlane(n[l], j) == n[l]);
    if (first) atomicAdd(&a.lv[l].hist[(int64_t)n[l] * a.n_tok_tiles + t / kTokTile], 1);
  }
}

}  // namespace

namespace {

// E <= 64 PER, and how the wavefront's rows meet: swaps while the launch is a
// latency chain, lane exchanges from 2048 tokens on. k = 8, swaps against
// exchanges: T = 300, E = 128 14.0 and 14.4 us; T = 16384 52.4 and 50.3.
template <class F>
hipError_t with_topk_shape(int T, int E, F&& launch) {
  auto per = [&](auto swap) {
    if (E <= 64)
      launch(std::integral_constant<int, 1>{}, swap);
    else if (E <= 128)
      launch(std::integral_constant<int, 2>{}, swap);
    else if (E <= 256)
      launch(std::integral_constant<int, 4>{}, swap);
    else
      launch(std::integral_constant<int, kRouteMaxE / 64>{}, swap);
  };
  if (T < 2048)
    per(std::true_type{});
  else
    per(std::false_type{});
  return hipGetLastError();
}

}  // namespace

hipError_t launch_topk_hist(const RouteIn& r, const BucketArgs& a, hipStream_t s) {
  if (a.T <= 0) return hipSuccess;
  const dim3 grid((a.T + TK_WAVES - 1) / TK_WAVES), thr(TK_WAVES * 64);
  return with_topk_shape(a.T, a.E, [&](auto per, auto swap) {
    hipLaunchKernelGGL((k_topk_hist<decltype(per)::value, decltype(swap)::value>), grid, thr, 0, s, r, a);
  });
}

hipError_t launch_topk(const float* logits, const float* part, int S, int T, int E, int k, int32_t* ids,
                       float* weights, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  const dim3 grid((T + TK_WAVES - 1) / TK_WAVES), thr(TK_WAVES * 64);
  return with_topk_shape(T, E, [&](auto per, auto swap) {
    hipLaunchKernelGGL((k_topk<decltype(per)::value, decltype(swap)::value>), grid, thr, 0, s, logits, part, S, T, E, k,
                       ids, weights);
  });
}

}  // namespace lx

// Stages 1-2 of the compression pipeline on the GPU (Sec. 3 "Compression
// pipeline"): router profiling counts, the co-activation NPMI distance of the
// Coact-NPMI variant, and frequency-seeded k-medoids with the dominant
// choice. They run once per layer on calibration routing and fix the
// cluster map and factor indices of a flat layer.
//
//   * k_coact: an expert fires on a token when it is among the token's valid
//     ids (once per token); every unordered pair of distinct firing experts
//     co-fires once. E <= 128: per 1024 tokens one bit mask per expert in LDS;
//     the counts are the popcounts of the masks' pairwise intersections, kept
//     in registers over a workgroup's tokens and added to global memory once.
//     Else integer atomics per token. Order-free either way, so exact.
//   * k_npmi: D = 1 - NPMI in fp64, one thread per (i, j); mirrors the counts.
//   * k_kmedoids: one workgroup, one thread per expert (E <= 1024). Seeds =
//     the highest-firing unprotected experts; assign (nearest medoid, ties to
//     the lower cluster, a medoid stays in its own cluster) / update (member
//     with the smallest in-cluster distance sum, summed in ascending member
//     order, ties to the lower index) until no medoid moves. Per-cluster
//     minima in LDS with 64-bit atomic min on order-preserving keys, so every
//     decision is the exact fp64 comparison a sequential loop would make.
#include "lx_device_once.h"
#include "lx_internal.h"

#include <algorithm>

namespace lx {
namespace {

constexpr int KM_THR = 1024;

__global__ __launch_bounds__(256) void k_fill2_u32(uint32_t* __restrict__ p, int64_t n, uint32_t* __restrict__ q,
                                                   int64_t m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
  if (i < m) q[i] = 0u;
}

// Valid, first-occurrence ids of token t: slot j counts when 0 <= id < E and
// no earlier slot of the row holds the same id.
__device__ __forceinline__ bool first_valid(const int32_t* row, int j, int E) {
  const int e = row[j];
  if (e < 0 || e >= E) return false;
  for (int q = 0; q < j; ++q)
    if (row[q] == e) return false;
  return true;
}

// One thread per token, integer atomics on global memory (any E). (Token indexes
// here and below are unsigned: with N near 2^31 a grid stride past the last token
// leaves the signed range.)
__global__ __launch_bounds__(256) void k_coact(const int32_t* __restrict__ ids, int N, int k, int E,
                                               uint32_t* __restrict__ fire, uint32_t* __restrict__ pair) {
  for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < (uint32_t)N; t += gridDim.x * blockDim.x) {
    const int32_t* row = ids + (int64_t)t * k;
    for (int a = 0; a < k; ++a) {
      if (!first_valid(row, a, E)) continue;
      const int ea = row[a];
      atomicAdd(&fire[ea], 1u);
      for (int b = a + 1; b < k; ++b) {
        if (!first_valid(row, b, E)) continue;
        const int eb = row[b];
        const int lo = ea < eb ? ea : eb, hi = ea < eb ? eb : ea;
        atomicAdd(&pair[(int64_t)lo * E + hi], 1u);
      }
    }
  }
}

// E <= 128: 1024 tokens at a time, a 1024-bit mask per expert in LDS (a repeated
// id sets its bit once). A thread owns the pairs (bi + 32 u, bj + 32 v), v < 4, of
// one bi <= bj < 32 (528 threads; neighbouring threads read neighbouring
// experts' masks, on distinct banks) and its workgroup's u = blockIdx.y, and
// counts popcount(mask_i & mask_j) in registers; the diagonal gives the firing
// counts. The four workgroups of the same tokens each build all masks: that
// is a third of the popcounts' time, and 64 workgroups alone leave three of
// four compute units idle.
// What bounds it is the final adds to global memory (about 37 per ns over the
// chip), so kCoactGroups workgroups share the tokens. Against the kernel that
// gathered pair counts in LDS and flushed them per 256 tokens: 131072 tokens,
// top-8, E = 128: 78 -> 38 us, four workgroups per 1024 tokens: 30 us.
constexpr int kCoactTok = 1024, kCoactThr = 1024, kCoactGroups = 64, kCoactPitch = kCoactTok / 32 + 4;

__global__ __launch_bounds__(kCoactThr) void k_coact_bits(const int32_t* __restrict__ ids, int N, int k, int E,
                                                          uint32_t* __restrict__ fire, uint32_t* __restrict__ pair) {
  // (pitch: 16-byte aligned rows, an odd number of 16-byte chunks)
  __shared__ __attribute__((aligned(16))) uint32_t s_mask[128 * kCoactPitch];
  const int tid = threadIdx.x;
  int bi = 0, bj = tid;  // block pair of this thread
  while (bi < 32 && bj >= 32 - bi) {
    bj -= 32 - bi;
    ++bi;
  }
  bj += bi;
  const bool own = bi < 32 && bi + 32 * (int)blockIdx.y < E && bj < E;
  const int ei = bi + 32 * blockIdx.y;
  uint32_t cnt[4] = {};
  for (uint32_t t0 = blockIdx.x * kCoactTok; t0 < (uint32_t)N; t0 += gridDim.x * kCoactTok) {
    for (int i = tid; i < 128 * kCoactPitch; i += kCoactThr) s_mask[i] = 0u;
    __syncthreads();
    const uint32_t t = t0 + tid;
    if (t < (uint32_t)N) {
      const int32_t* row = ids + (int64_t)t * k;
      for (int a0 = 0; a0 < k; a0 += 8) {
        int e[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) e[u] = row[a0 + u < k ? a0 + u : k - 1];  // (a repeat changes nothing)
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (e[u] >= 0 && e[u] < E) atomicOr(&s_mask[e[u] * kCoactPitch + (tid >> 5)], 1u << (tid & 31));
      }
    }
    __syncthreads();
    if (own) {
      for (int w = 0; w < kCoactTok / 32; w += 4) {
        const uint4 x = *(const uint4*)&s_mask[ei * kCoactPitch + w];
        uint4 y[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = *(const uint4*)&s_mask[(bj + 32 * j) * kCoactPitch + w];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          cnt[j] += __popc(x.x & y[j].x) + __popc(x.y & y[j].y) + __popc(x.z & y[j].z) + __popc(x.w & y[j].w);
      }
    }
    __syncthreads();
  }
  if (!own) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int ej = bj + 32 * j;
    if ((bi == bj && (int)blockIdx.y > j) || ej >= E || cnt[j] == 0) continue;
    if (ei == ej)
      atomicAdd(&fire[ei], cnt[j]);
    else
      atomicAdd(&pair[(int64_t)min(ei, ej) * E + max(ei, ej)], cnt[j]);
  }
}

// Counts were gathered in the upper triangle (which only its own threads' lower
// mirror reads): D = 1 - NPMI, the lower triangle mirrored, the diagonal zeroed.
__global__ __launch_bounds__(256) void k_npmi(const uint32_t* __restrict__ fire, uint32_t* __restrict__ pair, int N,
                                              int E, double* __restrict__ dist) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (int64_t)E * E) return;
  const int i = (int)(q / E), j = (int)(q % E);
  if (i == j) {
    dist[q] = 0.0;
    pair[q] = 0u;
    return;
  }
  const int lo = i < j ? i : j, hi = i < j ? j : i;
  const uint32_t nij = pair[(int64_t)lo * E + hi];
  double npmi;
  if (nij == 0u) {
    npmi = -1.0;
  } else if (nij == (uint32_t)N) {
    npmi = 1.0;
  } else {
    const double n = (double)N, pij = (double)nij / n;
    npmi = log(pij / (((double)fire[i] / n) * ((double)fire[j] / n))) / (-log(pij));
  }
  dist[q] = 1.0 - npmi;
  if (i > j) pair[q] = nij;
}

// Order-preserving map of doubles onto unsigned 64-bit keys.
__device__ __forceinline__ unsigned long long dkey(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// Latency-bound (one workgroup). E <= KMAX = 128: the distance matrix is staged
// in LDS (odd pitch: the threads' rows on distinct banks), and a bit mask of each
// cluster's members lets the ordered sums walk the members alone, 4 loads in
// flight. E = 128, 16 clusters: 65 -> 37 us with the masks and 16 rows' staging
// loads in flight. Larger E reads the matrix from memory, its members only, one
// after the other: a thread's row is a line of its own, and all E loads of it in
// batches of 8 took 210 instead of 178 us at E = 160, 820 instead of 420 at 512
// and 2530 instead of 1009 at 1024.
constexpr int kKmSmall = 128;

template <int KMAX>
__global__ __launch_bounds__(KM_THR) void k_kmedoids(const double* __restrict__ D, const uint32_t* __restrict__ fire,
                                                     int E, int C, ProtMask pm, int P, int max_iter,
                                                     int32_t* __restrict__ cluster_of,
                                                     int32_t* __restrict__ factor_of, int32_t* __restrict__ dominant,
                                                     int32_t* __restrict__ iterations) {
  constexpr bool SMALL = KMAX <= kKmSmall;
  extern __shared__ double s_d[];  // SMALL: [E][E | 1]
  __shared__ int s_cl[KMAX];
  __shared__ int s_med[KMAX];
  __shared__ uint32_t s_fire[KMAX];
  __shared__ unsigned long long s_key[KMAX];
  __shared__ int s_idx[KMAX];
  __shared__ uint32_t s_fmax[KMAX];
  __shared__ int s_isdom[KMAX], s_prot[SMALL ? KMAX : 1];
  // SMALL: the members of each cluster, the last assignment's and the one before
  __shared__ unsigned long long s_mem[2][SMALL ? 2 * KMAX : 1];
  __shared__ int s_changed;
  const int e = threadIdx.x;
  const int K = C - P;
  const bool live = e < E;
  const bool prot = live && ((pm.bits[e >> 5] >> (e & 31)) & 1u);
  const bool free_e = live && !prot;
  if (e < KMAX) {
    s_fire[e] = live ? fire[e] : 0u;
    s_cl[e] = -1;
    s_isdom[e] = 0;
    if (SMALL) s_prot[e] = prot || !live;
  }
  const int pitch = E | 1;
  if (SMALL) {
    // a wavefront per row; 16 rows' loads in flight
    const int lane = e & 63, nw = blockDim.x >> 6;
    for (int i0 = e >> 6; i0 < E; i0 += 16 * nw) {
      double v[16][KMAX / 64];
#pragma unroll
      for (int u = 0; u < 16; ++u)
#pragma unroll
        for (int h = 0; h < KMAX / 64; ++h) {
          const int i = i0 + u * nw < E ? i0 + u * nw : E - 1, j = lane + 64 * h < E ? lane + 64 * h : E - 1;
          v[u][h] = D[(int64_t)i * E + j];
        }
#pragma unroll
      for (int u = 0; u < 16; ++u)
#pragma unroll
        for (int h = 0; h < KMAX / 64; ++h)
          if (i0 + u * nw < E && lane + 64 * h < E) s_d[(i0 + u * nw) * pitch + lane + 64 * h] = v[u][h];
    }
    for (int i = e; i < 2 * KMAX; i += blockDim.x) s_mem[0][i] = 0ull;
  }
  __syncthreads();
  // seeds: free experts ranked by (firing count descending, index ascending)
  if (free_e) {
    int rank = 0;
    const uint32_t fe = s_fire[e];
    if (SMALL) {
#pragma unroll 8
      for (int f = 0; f < E; ++f) {
        const uint32_t ff = s_fire[f];
        rank += !s_prot[f] && (ff > fe || (ff == fe && f < e)) ? 1 : 0;
      }
    } else {
      for (int f = 0; f < E; ++f) {
        const bool pf = (pm.bits[f >> 5] >> (f & 31)) & 1u;
        if (!pf && (s_fire[f] > fe || (s_fire[f] == fe && f < e))) ++rank;
      }
    }
    if (rank < K) s_med[rank] = e;
  }
  __syncthreads();
  const double* const De = SMALL ? s_d + (live ? e : 0) * pitch : D + (int64_t)(live ? e : 0) * E;
  // sum over j, ascending, of f(De[j]) where pick(j); only those are loaded
  auto sum_where = [&](auto pick, auto f) {
    double s = 0.0;
    for (int j = 0; j < E; ++j)
      if (pick(j)) s += f(De[j]);
    return s;
  };
  int cur = 0;  // the last assignment's masks
  // the same over the members of cluster c but `skip` (-1: none)
  auto sum_members = [&](int c, int skip, auto f) {
    unsigned long long lo = s_mem[cur][2 * c], hi = s_mem[cur][2 * c + 1];
    if (skip >= 64) hi &= ~(1ull << (skip - 64));
    if (skip >= 0 && skip < 64) lo &= ~(1ull << skip);
    double s = 0.0;
    while (lo | hi) {
      double v[4];
      bool on[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        on[u] = (lo | hi) != 0ull;
        const int j = lo ? __ffsll((long long)lo) - 1 : 63 + __ffsll((long long)hi);
        v[u] = De[on[u] ? j : 0];
        if (lo)
          lo &= lo - 1ull;
        else
          hi &= hi - 1ull;  // (0 stays 0)
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double w = s + f(v[u]);
        s = on[u] ? w : s;
      }
    }
    return s;
  };
  auto assign = [&](int into) {
    if (free_e) {
      int own = -1;
#pragma unroll 8
      for (int c = 0; c < K; ++c) own = s_med[c] == e ? c : own;
      if (own >= 0) {
        s_cl[e] = own;
      } else {
        int best = 0;
        double bd = De[s_med[0]];
        for (int c0 = 1; c0 < K; c0 += 8) {
          double v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = De[s_med[c0 + u < K ? c0 + u : K - 1]];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (c0 + u < K && v[u] < bd) {
              bd = v[u];
              best = c0 + u;
            }
        }
        s_cl[e] = best;
      }
      if (SMALL) atomicOr(&s_mem[into][2 * s_cl[e] + (e >> 6)], 1ull << (e & 63));
    }
    __syncthreads();
  };
  assign(0);
  int it = 0;
  while (it < max_iter) {
    ++it;
    double s = 0.0;
    if (free_e) {
      const int c = s_cl[e];
      if (SMALL)
        s = sum_members(c, -1, [](double v) { return v; });
      else
        s = sum_where([&](int j) { return s_cl[j] == c; }, [](double v) { return v; });
    }
    if (e < K) {
      s_key[e] = ~0ull;
      s_idx[e] = 0x7FFFFFFF;
    }
    __syncthreads();
    if (SMALL)
      for (int i = e; i < 2 * KMAX; i += blockDim.x) s_mem[cur ^ 1][i] = 0ull;
    if (free_e) atomicMin(&s_key[s_cl[e]], dkey(s));
    __syncthreads();
    if (free_e && dkey(s) == s_key[s_cl[e]]) atomicMin(&s_idx[s_cl[e]], e);
    if (e == 0) s_changed = 0;
    __syncthreads();
    if (e < K && s_idx[e] != s_med[e]) {
      s_med[e] = s_idx[e];
      s_changed = 1;
    }
    __syncthreads();
    if (!s_changed) break;
    assign(cur ^ 1);
    cur ^= 1;
  }
  // protected experts: singleton clusters after the seeded ones
  if (prot) {
    int rank = 0;
    if (SMALL) {
#pragma unroll 8
      for (int f = 0; f < E; ++f) rank += f < e && s_prot[f] ? 1 : 0;
    } else {
      for (int f = 0; f < e; ++f) rank += (pm.bits[f >> 5] >> (f & 31)) & 1u;
    }
    s_cl[e] = K + rank;
  }
  if (e < C) {
    s_fmax[e] = 0u;
    s_key[e] = 0ull;
    s_idx[e] = 0x7FFFFFFF;
  }
  __syncthreads();
  // dominant: most fired, then most central (sum of 1 - D to the other
  // members, ascending member order), then lowest index
  const int c = live ? s_cl[e] : 0;
  double cent = 0.0;
  if (SMALL) {
    if (free_e) cent = sum_members(c, e, [](double v) { return 1.0 - v; });  // (a protected expert is alone)
  } else if (live) {
    cent = sum_where([&](int j) { return j != e && s_cl[j] == c; }, [](double v) { return 1.0 - v; });
  }
  if (live) atomicMax(&s_fmax[c], s_fire[e]);
  __syncthreads();
  const bool top = live && s_fire[e] == s_fmax[c];
  if (top) atomicMax(&s_key[c], dkey(cent));
  __syncthreads();
  if (top && dkey(cent) == s_key[c]) atomicMin(&s_idx[c], e);
  __syncthreads();
  if (e < C) {
    dominant[e] = s_idx[e];
    s_isdom[s_idx[e]] = 1;
  }
  __syncthreads();
  if (live) {
    int rank = 0;
    if (SMALL) {
#pragma unroll 8
      for (int f = 0; f < E; ++f) rank += f < e && !s_isdom[f] ? 1 : 0;
    } else {
      for (int f = 0; f < e; ++f) rank += s_isdom[f] ? 0 : 1;
    }
    cluster_of[e] = c;
    factor_of[e] = s_isdom[e] ? -1 : rank;
  }
  if (e == 0) iterations[0] = it;
}

}  // namespace

hipError_t launch_coact(const int32_t* ids, int N, int k, int E, uint32_t* fire, uint32_t* pair, double* dist,
                        hipStream_t s) {
  const int64_t ee = (int64_t)E * E;
  const dim3 ge((unsigned)((ee + 255) / 256));
  hipLaunchKernelGGL(k_fill2_u32, ge, dim3(256), 0, s, pair, ee, fire, (int64_t)E);
  if (N > 0) {
    // the mask kernel's threads own the pairs of at most 128 experts; more take
    // the per-token atomics (N = 131072, k = 8: 0.91 ms at 129 experts, 0.60 at
    // 256, against 0.03 at 128. Masks tiled over the pairs would make fewer adds
    // there too, at most 64 E (E + 1) / 2 against N k (k + 1) / 2)
    if (E <= 128)
      hipLaunchKernelGGL(k_coact_bits, dim3((unsigned)std::min<int64_t>(((int64_t)N + kCoactTok - 1) / kCoactTok,
                                                                        kCoactGroups),
                                              (unsigned)std::min(4, (E + 31) / 32)),
                         dim3(kCoactThr), 0, s, ids, N, k, E, fire, pair);
    else
      hipLaunchKernelGGL(k_coact, dim3((unsigned)std::min<int64_t>(((int64_t)N + 255) / 256, 512)), dim3(256), 0, s, ids, N, k, E, fire,
                         pair);
  }
  hipLaunchKernelGGL(k_npmi, ge, dim3(256), 0, s, fire, pair, N, E, dist);
  return hipGetLastError();
}

hipError_t launch_kmedoids(const double* dist, const uint32_t* fire, int E, int C, const ProtMask& pm, int P,
                           int max_iter, int32_t* cluster_of, int32_t* factor_of, int32_t* dominant,
                           int32_t* iterations, hipStream_t s) {
  if (E <= kKmSmall) {
    static DeviceOnce once;
    int dev = 0;
    hipError_t lds = hipGetDevice(&dev);
    if (lds == hipSuccess)
      lds = once.run(dev, hipSuccess, [] {
        return hipFuncSetAttribute((const void*)k_kmedoids<kKmSmall>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   kKmSmall * (kKmSmall | 1) * 8);
      });
    if (lds != hipSuccess) return lds;
    hipLaunchKernelGGL(k_kmedoids<kKmSmall>, dim3(1), dim3(512), (size_t)E * (E | 1) * 8, s, dist, fire, E, C, pm, P,
                       max_iter, cluster_of, factor_of, dominant, iterations);
  } else {
    hipLaunchKernelGGL(k_kmedoids<KM_THR>, dim3(1), dim3(KM_THR), 0, s, dist, fire, E, C, pm, P, max_iter, cluster_of,
                       factor_of, dominant, iterations);
  }
  return hipGetLastError();
}

}  // namespace lx

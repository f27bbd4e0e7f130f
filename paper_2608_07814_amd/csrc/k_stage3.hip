// Stage 3 of the compression pipeline on the GPU (Sec. 3, "Alignment and
// low-rank decomposition"), in fp64: the neuron-alignment cost matrix
// (eq. cost), the aligned residual and its rank-r factors from a randomized
// truncated SVD with the symmetric split (eqs. svd and factors). The exact
// assignment between the two (eq. assign) runs on the host. Also the
// activation-weighted fit of the factors (Sec. 4, reconstruction fine-
// tuning; its closed form in Secs. 6-7): minimising ||(R - A B) X^T||^2 +
// damp ||R - A B||^2 over calibration activations X is the rank-r
// truncation of R L (G = X^T X + damp I = L L^T); the same randomized solver
// runs on the operator M = R Xp^T, Xp = [X; sqrt(damp) I], which has the
// left singular vectors and values of R L (M M^T = R G R^T), and B =
// sigma^(-1/2) U_r^T R, so no Cholesky factor of G or its inverse is formed.
//
//   * k_dgemm: C = op(A) op(B), fp64 on v_mfma_f64_16x16x4_f64, tiles chosen by
//     the product's shape; the workhorse of every product below (all are
//     thin: one side is the sketch width l = r + p <= 128, or the cost matrix's
//     f x f x 3d).
//   * k_chol: one workgroup, G = U^T U for an l x l Gram matrix held in
//     registers (right-looking, one barrier per column); k_trsm_rows: Y <- Y
//     U^-1, 16 lanes per row. Together they orthonormalise the sketch (once
//     between the products, twice, CholeskyQR2, for the final basis).
//   * k_jacobi: one workgroup, the eigenvalues of the l x l matrix Q^T R R^T Q
//     by cyclic Jacobi in the round-robin (tournament) order, so each step
//     rotates l / 2 disjoint pairs at once; matrix in LDS, rotations written
//     to a log. k_jacobi_vec: the eigenvectors from the log, one wavefront per
//     row of V, eigenpairs sorted descending.
#include "lx_device_once.h"
#include "lx_internal.h"
#include "lx_stage3_ws.h"

#include <algorithm>

namespace lx {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Workgroup barrier for LDS communication only: waits for this wavefront's
// LDS operations, not for its global stores (which nothing in the workgroup
// reads back), unlike __syncthreads().
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xF | (0x7 << 4) | (0x3 << 14));  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// 1 / x to a unit in the last place for normal x: the hardware estimate and
// two Newton steps (a dependent chain a third of a full division's).
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// 1 / sqrt(x), likewise.
__device__ __forceinline__ double fast_rsq(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = fma(r * fma(-x * r, r, 1.0), 0.5, r);
  return fma(r * fma(-x * r, r, 1.0), 0.5, r);
}

// C = op(A) op(B) in fp64 on the matrix cores: BM x BN output tiles, BM = 16 WM
// MI and BN = 16 WN NI, by 4 wavefronts in a WM x WN grid of MI x NI
// v_mfma_f64_16x16x4 blocks (lane l holds A row / B column l % 16 at k = l /
// 16; accumulator i is row 4 i + l / 16, column l % 16). 32-deep K slabs, double-
// buffered in LDS as [row][k] with a pitch of 34 doubles: the 32 lanes of
// half a ds_read_b64 (16 rows, 2 k) then fall on 64 distinct banks. The next
// slab's global loads are in flight during the MFMAs, and one barrier
// separates slabs. Bound by the loads' latency at the sizes it runs at (a few
// K slabs per workgroup), so split-K spreads a product over the chip.
// Against the VALU kernel it replaced (64 x 64 tiles, 4 x 4 outputs per thread):
// the cost product 768 x 768 x 6144 1237 -> 200 us, the sketch product 768 x
// 74 x 2048 55 -> 16 us.
//
// Split-K: blockIdx.z takes K range [z kc, (z + 1) kc) and writes its partial
// tile to C + z * M * N (ldc = N); the consumer adds the partials in z order.
// TI: element type of A and B (double, or float for the alignment cost's
// neuron vectors, which fp32 holds exactly).
constexpr int DG_K = 32, DG_PITCH = 34;

template <typename TI, int WM, int WN, int MI, int NI>
__global__ __launch_bounds__(256) void k_dgemm(int M, int N, int K, const TI* __restrict__ A, int64_t lda, int ta,
                                               const TI* __restrict__ B, int64_t ldb, int tb, double* __restrict__ C,
                                               int64_t ldc, int kc) {
  static_assert(WM * WN == 4, "4 wavefronts");
  constexpr int BM = 16 * WM * MI, BN = 16 * WN * NI;
  constexpr int RA = BM * DG_K / 256, RB = BN * DG_K / 256;  // elements per thread and slab
  extern __shared__ double s_dg[];  // A slabs [2][BM][DG_PITCH], B slabs [2][BN][DG_PITCH]
  double* const sA = s_dg;
  double* const sB = s_dg + 2 * BM * DG_PITCH;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = wave / WN, wn = wave % WN;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int kbeg = blockIdx.z * kc, kend = kbeg + kc < K ? kbeg + kc : K;
  C += (int64_t)blockIdx.z * M * N;

  // Element q of a thread's share of a slab of X (rows x K): with k contiguous
  // in memory 32 consecutive threads take one row's 32 values, with the rows
  // contiguous consecutive threads take consecutive rows. Rows past the edge
  // are clamped (their products are never stored), k past the end gives 0.
  auto load = [&](const TI* __restrict__ X, int64_t ld, bool kcontig, int r0, int rows, int rn, int k0, int q) -> TI {
    const int e = q * 256 + tid;
    const int r = kcontig ? e / DG_K : e % rn, k = kcontig ? e % DG_K : e / rn;
    const int gr = r0 + r < rows ? r0 + r : rows - 1, gk = k0 + k < kend ? k0 + k : kend - 1;
    const TI v = kcontig ? X[(int64_t)gr * ld + gk] : X[(int64_t)gk * ld + gr];
    return k0 + k < kend ? v : (TI)0;
  };
  auto slot = [&](bool kcontig, int rn, int q) {
    const int e = q * 256 + tid;
    const int r = kcontig ? e / DG_K : e % rn, k = kcontig ? e % DG_K : e / rn;
    return r * DG_PITCH + k;
  };
  const bool ka = !ta, kb = tb != 0;  // k contiguous in A, in B
  TI va[RA], vb[RB];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int q = 0; q < RA; ++q) va[q] = load(A, lda, ka, m0, M, BM, k0, q);
#pragma unroll
    for (int q = 0; q < RB; ++q) vb[q] = load(B, ldb, kb, n0, N, BN, k0, q);
  };
  auto put = [&](int st) {
#pragma unroll
    for (int q = 0; q < RA; ++q) sA[st * BM * DG_PITCH + slot(ka, BM, q)] = (double)va[q];
#pragma unroll
    for (int q = 0; q < RB; ++q) sB[st * BN * DG_PITCH + slot(kb, BN, q)] = (double)vb[q];
  };

  f64x4 acc[MI][NI] = {};
  if (kbeg < kend) {
    fetch(kbeg);
    put(0);
  }
  int st = 0;
  for (int k0 = kbeg; k0 < kend; k0 += DG_K) {
    const bool more = k0 + DG_K < kend;
    lds_barrier();
    if (more) fetch(k0 + DG_K);
    const double* const pa = &sA[st * BM * DG_PITCH + (wm * 16 * MI + (lane & 15)) * DG_PITCH + (lane >> 4)];
    const double* const pb = &sB[st * BN * DG_PITCH + (wn * 16 * NI + (lane & 15)) * DG_PITCH + (lane >> 4)];
#pragma unroll
    for (int kk = 0; kk < DG_K; kk += 4) {
      double fa[MI], fb[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) fa[i] = pa[i * 16 * DG_PITCH + kk];
#pragma unroll
      for (int j = 0; j < NI; ++j) fb[j] = pb[j * 16 * DG_PITCH + kk];
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
    // (the other stage's readers passed this slab's barrier)
    if (more) put(st ^ 1);
    st ^= 1;
  }
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int gm = m0 + (wm * MI + i) * 16 + 4 * u + (lane >> 4), gn = n0 + (wn * NI + j) * 16 + (lane & 15);
        if (gm < M && gn < N) C[(int64_t)gm * ldc + gn] = acc[i][j][u];
      }
}

__global__ __launch_bounds__(256) void k_dsum(const double* __restrict__ part, int S, int64_t n,
                                              double* __restrict__ C) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  double v = part[q];
  for (int z = 1; z < S; ++z) v += part[z * n + q];
  C[q] = v;
}

// Neuron vectors of an expert, fp32 [f][3d] (exact for bf16 and fp32 weights):
// row i = (gate[i, :], up[i, :], down[:, i]); squared norms in fp64.
__global__ __launch_bounds__(256) void k_neurons(const void* __restrict__ gate, const void* __restrict__ up,
                                                 const void* __restrict__ down, int bf16, int f, int d,
                                                 float* __restrict__ out, double* __restrict__ norms) {
  const int i = blockIdx.x;
  __shared__ double s_red[256];
  double s = 0.0;
  for (int c = threadIdx.x; c < 3 * d; c += blockDim.x) {
    int64_t src;
    const void* base;
    if (c < d) {
      base = gate;
      src = (int64_t)i * d + c;
    } else if (c < 2 * d) {
      base = up;
      src = (int64_t)i * d + (c - d);
    } else {
      base = down;
      src = (int64_t)(c - 2 * d) * f + i;
    }
    const float v = bf16 ? __uint_as_float((uint32_t)((const uint16_t*)base)[src] << 16) : ((const float*)base)[src];
    out[(int64_t)i * 3 * d + c] = v;
    s += (double)v * (double)v;
  }
  s_red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) s_red[threadIdx.x] += s_red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) norms[i] = s_red[0];
}

// C[i][j] = na[i] + nb[j] - 2 G[i][j], G the sum of the S partial products in
// part (S = 1: part may be C itself).
__global__ __launch_bounds__(256) void k_cost_finish(const double* __restrict__ na, const double* __restrict__ nb,
                                                     int f, const double* part, int S, double* C) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t ff = (int64_t)f * f;
  if (q >= ff) return;
  double g = part[q];
  for (int z = 1; z < S; ++z) g += part[z * ff + q];
  C[q] = na[q / f] + nb[q % f] - 2.0 * g;
}

// R[i][j] = W_m^P[i][j] - W_dom[i][j]: member rows (axis 0) or columns
// (axis 1) taken in the order perm (null: identity).
__global__ __launch_bounds__(256) void k_residual(const void* __restrict__ wd, const void* __restrict__ wm, int bf16,
                                                  int rows, int cols, const int32_t* __restrict__ perm, int axis,
                                                  double* __restrict__ R) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (int64_t)rows * cols) return;
  const int i = (int)(q / cols), j = (int)(q % cols);
  int pi = perm && axis == 0 ? perm[i] : i, pj = perm && axis == 1 ? perm[j] : j;
  // a permutation entry out of range reads a clamped (valid) element
  pi = pi < 0 ? 0 : pi >= rows ? rows - 1 : pi;
  pj = pj < 0 ? 0 : pj >= cols ? cols - 1 : pj;
  const int64_t sm = (int64_t)pi * cols + pj;
  double vd, vm;
  if (bf16) {
    vd = (double)__uint_as_float((uint32_t)((const uint16_t*)wd)[q] << 16);
    vm = (double)__uint_as_float((uint32_t)((const uint16_t*)wm)[sm] << 16);
  } else {
    vd = (double)((const float*)wd)[q];
    vm = (double)((const float*)wm)[sm];
  }
  R[q] = vm - vd;
}

// Cholesky of the l x l Gram matrix G = the sum of S partial products (row-
// major), upper factor U with G = U^T U written to Uf (zero below the
// diagonal). A pivot at or below 1e-14 of the largest diagonal entry of G (a
// direction the sketch does not have: exactly low-rank residuals) gives a zero
// row of U, and k_trsm_rows then a zero column of Q; the directions kept stay
// orthonormal and the zero ones carry no weight in Q^T R.
// Latency-bound (one workgroup, l dependent columns): thread (ti, tj) of a 16 x
// 16 grid keeps entries (ti + 16 a, tj + 16 b), a <= b, in registers, row k of the trailing
// matrix goes through LDS once (one barrier per column), and the division by
// the pivot's square root waits until every row is known. Column k first updates
// only the block row that holds row k + 1, which goes to LDS at once; the other
// block rows follow behind the next column's barrier, while its LDS reads are in
// flight. kAhead partials are loaded together. l = 74: all entries of 8 partials
// 31 us; the upper blocks of 12 partials 28, of 16 partials 30.
template <int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_chol(const double* __restrict__ part, int S, int l, double* __restrict__ Uf) {
  extern __shared__ double s_row[];  // [l][16 NB]: the trailing matrix's row k when its column is eliminated
  __shared__ double s_diag[16 * NB], s_rt[16 * NB], s_ri[16 * NB];
  constexpr int P = 16 * NB, kAhead = NB <= 5 ? 4 : 2;
  const int tid = threadIdx.x, ti = tid >> 4, tj = tid & 15;
  double a[NB][NB] = {};
  // the partials' entries (clamped past l and past S, then dropped), added in order
  for (int z = 0; z < S; z += kAhead) {
    double t[kAhead][NB][NB];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const double* const g = part + (int64_t)(z + u < S ? z + u : S - 1) * l * l;
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = i; j < NB; ++j) {
          const int gi = ti + 16 * i, gj = tj + 16 * j;
          t[u][i][j] = g[(gi < l ? gi : l - 1) * l + (gj < l ? gj : l - 1)];
        }
    }
    __builtin_amdgcn_sched_barrier(0);  // all loads issued before the first is waited for
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (z + u < S) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = i; j < NB; ++j) a[i][j] += t[u][i][j];
      }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = i; j < NB; ++j) {
      const int gi = ti + 16 * i, gj = tj + 16 * j;
      if (gi >= l || gj >= l) a[i][j] = 0.0;
      if (gi == gj) s_diag[gi] = a[i][j];
    }
  if (ti == 0) {
#pragma unroll
    for (int j = 0; j < NB; ++j) s_row[tj + 16 * j] = a[0][j];
  }
  lds_barrier();
  double gmax = 0.0;
  for (int k = tid & 63; k < P; k += 64) gmax = fmax(gmax, s_diag[k]);
  for (int o = 32; o > 0; o >>= 1) gmax = fmax(gmax, __shfl_xor(gmax, o, 64));
  const double floor_ = 1e-14 * gmax;
  // the column before: its row, and minus its column over the pivot (0 at first)
  double rj[NB] = {}, ri[NB] = {};
#pragma unroll
  for (int kb = 0; kb < NB; ++kb)
    for (int kr = 0; kr < 16; ++kr) {
      const int k = kb * 16 + kr;
      if (k >= l) break;
      const double* const row = s_row + k * P;
      if (k > 0) lds_barrier();
      const double pk = row[k];
      double nj[NB], ni[NB];
      // rows and columns of the blocks before kb are done
#pragma unroll
      for (int j = kb; j < NB; ++j) {
        nj[j] = row[tj + 16 * j];
        ni[j] = row[ti + 16 * j];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = kb + 1; i < NB; ++i)
#pragma unroll
        for (int j = i; j < NB; ++j) a[i][j] = fma(ri[i], rj[j], a[i][j]);
      const double inv = pk > floor_ ? fast_rcp(pk) : 0.0;
#pragma unroll
      for (int j = kb; j < NB; ++j) {
        rj[j] = nj[j];
        ri[j] = -ni[j] * inv;
      }
      if (kr < 15) {
#pragma unroll
        for (int j = kb; j < NB; ++j) a[kb][j] = fma(ri[kb], rj[j], a[kb][j]);
        if (ti == kr + 1 && k + 1 < l) {
#pragma unroll
          for (int j = kb; j < NB; ++j) s_row[(k + 1) * P + tj + 16 * j] = a[kb][j];
        }
      } else if (kb + 1 < NB) {
        const int nb = kb + 1 < NB ? kb + 1 : kb;
#pragma unroll
        for (int j = nb; j < NB; ++j) a[nb][j] = fma(ri[nb], rj[j], a[nb][j]);
        if (ti == 0) {
#pragma unroll
          for (int j = nb; j < NB; ++j) s_row[(k + 1) * P + tj + 16 * j] = a[nb][j];
        }
      }
    }
  lds_barrier();
  for (int k = tid; k < l; k += 256) {
    const double pk = s_row[k * P + k], d = pk > floor_ ? sqrt(pk) : 0.0;
    s_rt[k] = d;
    s_ri[k] = d > 0.0 ? 1.0 / d : 0.0;
  }
  lds_barrier();
#pragma unroll 4
  for (int q = tid; q < l * l; q += 256) {
    const int k = q / l, j = q % l;
    const double d = s_rt[k], r = s_ri[k], v = s_row[k * P + j];
    double u = v * r;
    u = fma(fma(-u, d, v), r, u);  // v / d, correctly rounded but for ties
    Uf[q] = j < k || !(d > 0.0) ? 0.0 : j == k ? d : u;
  }
}

// Value of lane N of each row of 16 lanes, in every lane of the row.
template <int N>
__device__ __forceinline__ double row_bcast(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x150 + N, 0xf, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x150 + N, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Y[i, :] <- Y[i, :] U^-1 for the upper-triangular l x l U: x U = y, solved
// left to right. 16 lanes hold one row (column c + 16 b in register b of lane
// c), so a wavefront solves 4 rows: column j's value is finished in its lane,
// broadcast over the row (DPP) and taken off the later columns. U is staged in
// LDS (pitch 16 NB, zero past l) with its diagonal and reciprocals beside it.
// Latency-bound: the chain is one division, one broadcast and one FMA per
// column. Against one thread per row (12 workgroups for 768 rows): l = 74, 768
// rows 100 -> 9 us.
constexpr int kTrsmRows = 16;  // rows per workgroup of 4 wavefronts

template <int NB, int J>
__device__ __forceinline__ void trsm_step(double (&y)[NB], const double* su, const double* sd, const double* sr, int c) {
  constexpr int P = 16 * NB, B = J / 16;
  const double u = sd[J], r = sr[J];
  double q = y[B] * r;
  q = fma(fma(-q, u, y[B]), r, q);  // y / u, correctly rounded but for ties
  const double v = row_bcast<J % 16>(q);
  if (c == J % 16) y[B] = q;
  const double* const row = su + J * P + c;
  // columns of register B after J (U is 0 at and before J: the diagonal is
  // kept apart)
  y[B] = fma(-v, row[16 * B], y[B]);
#pragma unroll
  for (int b = B + 1; b < NB; ++b) y[b] = fma(-v, row[16 * b], y[b]);
}

template <int NB, int J>
__device__ __forceinline__ void trsm_all(double (&y)[NB], const double* su, const double* sd, const double* sr, int c) {
  if constexpr (J < 16 * NB) {
    trsm_step<NB, J>(y, su, sd, sr, c);
    trsm_all<NB, J + 1>(y, su, sd, sr, c);
  }
}

template <int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_trsm_rows(double* __restrict__ Y, int rows, int l, const double* __restrict__ U) {
  extern __shared__ double su[];  // [16 NB][16 NB], strictly upper part
  constexpr int P = 16 * NB;
  __shared__ double sd[P], sr[P];
  const int tid = threadIdx.x, c = tid & 15;
  const int r = blockIdx.x * kTrsmRows + (tid >> 4);
  double y[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int j = c + 16 * b;
    y[b] = r < rows && j < l ? Y[(int64_t)r * l + j] : 0.0;
  }
  double uv[NB * NB];
#pragma unroll
  for (int u = 0; u < NB * NB; ++u) {
    const int q = tid + u * 256, k = q / P, j = q % P;
    uv[u] = U[(k < l ? k : l - 1) * l + (j < l ? j : l - 1)];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < NB * NB; ++u) {
    const int q = tid + u * 256, k = q / P, j = q % P;
    const double v = k < l && j < l ? uv[u] : 0.0;
    su[q] = j > k ? v : 0.0;
    if (j == k) {
      sd[k] = v;
      sr[k] = v != 0.0 ? 1.0 / v : 0.0;
    }
  }
  lds_barrier();
  trsm_all<NB, 0>(y, su, sd, sr, c);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int j = c + 16 * b;
    if (r < rows && j < l) Y[(int64_t)r * l + j] = y[b];
  }
}

// The rotation of a pair: t = sgn(tau) / (|tau| + sqrt(1 + tau^2)) for tau =
// (aqq - app) / (2 apq), by half angles: two reciprocal square roots in the
// dependent chain, no division.
__device__ __forceinline__ void jacobi_rot(double app, double aqq, double apq, double& c, double& s, double& t) {
  c = 1.0;
  s = t = 0.0;
  if (apq == 0.0) return;
  const double d = aqq - app, b = 2.0 * fabs(apq), ad = fabs(d);
  // (tau = 0 counts as positive)
  const bool pos = d == 0.0 || (d > 0.0) == (apq > 0.0);
  const double sum = ad + b;
  if (sum > 1e-140 && sum < 1e140) {
    // half angles: cos 2a = |d| / h, h = sqrt(d^2 + b^2); c^2 = (1 + cos 2a) / 2,
    // s = b / (2 h c)
    const double y = fast_rsq(fma(d, d, b * b));
    const double c2 = fma(0.5 * ad, y, 0.5);
    const double rc = fast_rsq(c2);
    c = c2 * rc;
    s = 0.5 * b * y * rc;
    t = s * rc;
  } else {  // d^2 or b^2 could leave the range
    const double tau = ad / b;
    t = 1.0 / (tau + sqrt(1.0 + tau * tau));
    c = 1.0 / sqrt(1.0 + t * t);
    s = t * c;
  }
  if (!pos) {
    s = -s;
    t = -t;
  }
}

// Eigenvalues of the symmetric l x l M (padded with zero rows and columns to lp
// = jacobi_order(l)): cyclic Jacobi, round-robin pair order; only entries (i, j)
// with i <= j are kept. A thread owns the 2 x 2 blocks (pair k1's rows, pair k2's
// columns, k1 < k2) of a step and applies both sides of the rotation at once; a
// rotation takes its pair in slot order.
// From one step to the next every slot moves on by one, so each pair of the
// next step has its entry in one block of this one: (0, 1), (x - 1, x + 1) and
// (half - 2, half - 1), all different from 3 pairs on. Wavefront 0 owns these
// blocks and turns the entry it has just rotated into the next step's rotation:
// one barrier per step. The rotations go to
// log[(sweep * (lp - 1) + step) * lp / 2 + pair] for k_jacobi_vec; meta: the
// number of sweeps, then the eigenvalue order. Bound by the step's dependent chain
// (LDS reads, two rotations applied, two reciprocal square roots) and by one
// compute unit's LDS (63 KB a step at l = 74). Against rotations formed between
// two barriers: l = 74 412 -> 377 us.
__host__ __device__ __forceinline__ int jacobi_order(int l) { return l <= 6 ? 6 : l + (l & 1); }

template <int U>
__global__ __launch_bounds__(1024) void k_jacobi(const double* __restrict__ Min, int l, int lp, double* __restrict__ w,
                                                 double2* __restrict__ log, int32_t* __restrict__ meta,
                                                 int max_sweeps) {
  extern __shared__ double s_m[];  // [lp][lp + 1], upper triangle (an odd pitch: rows and columns on distinct banks)
  __shared__ double2 s_cs[2][64];
  __shared__ double s_red[16];
  const int pt = lp + 1;
  const int tid = threadIdx.x, nth = blockDim.x, lane = tid & 63, wave = tid >> 6;
  for (int q = tid; q < lp * lp; q += nth) {
    const int i = q / lp, j = q % lp;
    s_m[i * pt + j] = (i < l && j < l) ? Min[i * l + j] : 0.0;
  }
  lds_barrier();
  // sum of squares of all entries (diag = 1) or of the off-diagonal ones
  auto sumsq = [&](bool diag) {
    double t = 0.0;
    for (int q = tid; q < lp * lp; q += nth) {
      const int i = q / lp, j = q % lp;
      const double v = s_m[i * pt + j];
      if (i < j) t += 2.0 * v * v;
      if (diag && i == j) t += v * v;
    }
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if (lane == 0) s_red[wave] = t;
    lds_barrier();
    double r = 0.0;
    for (int i = 0; i < (nth >> 6); ++i) r += s_red[i];
    lds_barrier();
    return r;
  };
  const double norm0 = sumsq(true);
  const int half = lp / 2, nrest = half * (half - 1) / 2 - half;
  // this thread's blocks: wavefront 0 the next step's pairs, the other
  // wavefronts the rest (pairs 1 apart but for the first and the last, and pairs
  // 3 or more apart), at most 1952 blocks in U = 3 rounds of
  // 960 threads (more registers than U = 1 leaves free)
  const int bth = nth - 64;
  int kk[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    int x = tid - 64 + u * bth;
    kk[u] = -1;
    if (tid < half) {
      if (u == 0) {
        const int k1 = tid == 0 ? 0 : tid == half - 1 ? half - 2 : tid - 1;
        const int k2 = tid == 0 ? 1 : tid == half - 1 ? half - 1 : tid + 1;
        kk[u] = k1 | (k2 << 16);
      }
    } else if (tid >= 64 && x < half - 3) {
      kk[u] = (1 + x) | ((2 + x) << 16);
    } else if (tid >= 64 && x < nrest) {
      x -= half - 3;
      int k1 = 0;
      while (x >= half - 3 - k1) {
        x -= half - 3 - k1;
        ++k1;
      }
      kk[u] = k1 | ((k1 + 3 + x) << 16);
    }
  }
  // Byte offsets: ec = 8 * element of the blocks' slots (first and second of
  // either pair), moved on by one element with every step (element 0 stays);
  // entry (i, j) lies at the smaller of (i, j)'s and (j, i)'s offset.
  auto addr = [&](int ci, int cj) { return min(__mul24(ci, pt) + cj, __mul24(cj, pt) + ci); };
  auto ent = [&](int off) -> double& { return *(double*)((char*)s_m + off); };
  int ec[U][4], at[U][4];
  auto locate = [&]() {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      at[u][0] = addr(ec[u][0], ec[u][2]);
      at[u][1] = addr(ec[u][0], ec[u][3]);
      at[u][2] = addr(ec[u][1], ec[u][2]);
      at[u][3] = addr(ec[u][1], ec[u][3]);
    }
  };
  // wavefront 0: the diagonal entries of the pair that the next step joins
  // (first slot, second slot)
  int df = 0, ds = 0;
  const bool x_first = tid == 0, x_last = tid == half - 1;
  auto diag = [&](int c) { return c * pt + c; };
  auto next_pair = [&]() {
    df = diag(x_first ? ec[0][0] : x_last ? ec[0][3] : ec[0][2]);
    ds = diag(x_first ? ec[0][2] : ec[0][1]);
  };
  auto rotate = [&](int sweep, int step, double aff, double ass, double afs, int off) {
    double c, s, t;
    jacobi_rot(aff, ass, afs, c, s, t);
    s_cs[step & 1][tid] = make_double2(c, s);
    ent(df) = aff - t * afs;
    ent(ds) = ass + t * afs;
    ent(off) = 0.0;
    log[(int64_t)(sweep * (lp - 1) + step) * half + tid] = make_double2(c, s);
  };
  if (wave == 0) __builtin_amdgcn_s_setprio(3);  // the chain of rotations
  int sweep = 0;
  for (; sweep < max_sweeps; ++sweep) {
    if (!(sumsq(false) > 1e-30 * norm0)) break;
#pragma unroll
    for (int u = 0; u < U; ++u) {  // slot x holds element x
      const int k1 = kk[u] & 0xFFFF, k2 = kk[u] >> 16;
      ec[u][0] = 8 * k1;
      ec[u][1] = 8 * (lp - 1 - k1);
      ec[u][2] = 8 * k2;
      ec[u][3] = 8 * (lp - 1 - k2);
    }
    locate();
    if (tid < half) {
      const int cf = 8 * tid, cs = 8 * (lp - 1 - tid), off = addr(cf, cs);
      df = diag(cf);
      ds = diag(cs);
      rotate(sweep, 0, ent(df), ent(ds), ent(off), off);
      next_pair();
    }
    lds_barrier();
    for (int step = 0; step < lp - 1; ++step) {
      double m[U][4];
      double2 e1[U], e2[U];
      double aff = 0.0, ass = 0.0;
      auto read = [&](int u) {
        e1[u] = s_cs[step & 1][kk[u] & 0xFFFF];
        e2[u] = s_cs[step & 1][kk[u] >> 16];
#pragma unroll
        for (int v = 0; v < 4; ++v) m[u][v] = ent(at[u][v]);
      };
      if (U == 1 && kk[0] >= 0) read(0);
      if (tid < half) {
        aff = ent(df);
        ass = ent(ds);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (U > 1) __builtin_amdgcn_sched_barrier(0);  // (a round at a time: all rounds' values would spill)
        if (kk[u] < 0) continue;
        if (U > 1) read(u);
        const double xff = e1[u].x * m[u][0] - e1[u].y * m[u][2], xsf = e1[u].y * m[u][0] + e1[u].x * m[u][2];
        const double xfs = e1[u].x * m[u][1] - e1[u].y * m[u][3], xss = e1[u].y * m[u][1] + e1[u].x * m[u][3];
        m[u][0] = e2[u].x * xff - e2[u].y * xfs;
        m[u][1] = e2[u].y * xff + e2[u].x * xfs;
        m[u][2] = e2[u].x * xsf - e2[u].y * xss;
        m[u][3] = e2[u].y * xsf + e2[u].x * xss;
#pragma unroll
        for (int v = 0; v < 4; ++v) ent(at[u][v]) = m[u][v];
      }
      if (tid < half && step + 1 < lp - 1)
        rotate(sweep, step + 1, aff, ass, x_first ? m[0][0] : x_last ? m[0][3] : m[0][2],
               x_first ? at[0][0] : x_last ? at[0][3] : at[0][2]);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int c = ec[u][v] + (v == 0 && (kk[u] & 0xFFFF) == 0 ? 0 : 8);
          ec[u][v] = c == 8 * lp ? 8 : c;
        }
      locate();
      if (tid < half) next_pair();
      lds_barrier();
    }
  }
  // descending order (ties: lower index first; the padding last), the first l
  // kept
  if (tid < lp) {
    const double e = s_m[tid * pt + tid];
    int rank = 0;
    if (tid >= l) {
      rank = tid;
    } else {
      for (int j = 0; j < l; ++j) {
        const double o = s_m[j * pt + j];
        if (o > e || (o == e && j < tid)) ++rank;
      }
      w[rank] = e;
    }
    meta[1 + rank] = tid;
  }
  if (tid == 0) meta[0] = sweep;
}

// Value of the next lane (lane 63: 0), of the lane before (lane 0: 0).
__device__ __forceinline__ double lane_above(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x130, 0xf, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x130, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double lane_below(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x138, 0xf, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x138, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Eigenvectors from k_jacobi's rotation log: row i of V = e_i J_1 J_2 ..., one
// wavefront per row (the rows are independent). Lane x holds slots x and lp - 1 -
// x of the row in registers and the slots move on by lane shifts (DPP); the
// log is streamed kJacAhead steps ahead. A sweep's lp - 1 steps bring every
// element back to the slot of its number. Writes row i of the sorted Vs [l][l],
// and workgroup 0 the singular values (square roots of the r largest
// eigenvalues). Bound by the chain of a product, an FMA and a shift per step;
// against the row in LDS: l = 74 88 -> 38 us.
constexpr int kJacAhead = 32;

__global__ __launch_bounds__(64) void k_jacobi_vec(const double2* __restrict__ log, const int32_t* __restrict__ meta,
                                                   int l, int lp, const double* __restrict__ lam, int r,
                                                   double* __restrict__ Vs, double* __restrict__ sig,
                                                   double* __restrict__ sigma) {
  __shared__ double s_v[128];  // elements by number
  const int lane = threadIdx.x, row = blockIdx.x, half = lp / 2;
  if (row == 0)
    for (int i = lane; i < r; i += 64) sig[i] = sigma[i] = sqrt(lam[i] > 0.0 ? lam[i] : 0.0);
  const int nsteps = meta[0] * (lp - 1);
  const int x = lane < half ? lane : half - 1;  // (the lanes past the pairs repeat the last; nothing reads them)
  double va = x == row ? 1.0 : 0.0, vb = lp - 1 - x == row ? 1.0 : 0.0;
  const bool first = x == 0, last = x == half - 1;
  double2 cur[kJacAhead], nxt[kJacAhead];
  auto fetch = [&](double2* e, int s0) {
#pragma unroll
    for (int u = 0; u < kJacAhead; ++u) e[u] = log[(int64_t)(s0 + u < nsteps ? s0 + u : nsteps - 1) * half + x];
  };
  if (nsteps > 0) fetch(cur, 0);
  for (int s0 = 0; s0 < nsteps; s0 += kJacAhead) {
    fetch(nxt, s0 + kJacAhead);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kJacAhead; ++u) {
      if (s0 + u < nsteps) {
        const double c = cur[u].x, s = cur[u].y;
        const double na = c * va - s * vb, nb = s * va + c * vb;
        const double up = lane_above(na), dn = lane_below(nb);
        va = first ? na : last ? nb : up;
        vb = first ? up : dn;
      }
    }
#pragma unroll
    for (int u = 0; u < kJacAhead; ++u) cur[u] = nxt[u];
  }
  if (lane < half) {
    s_v[lane] = va;
    s_v[lp - 1 - lane] = vb;
  }
  lds_barrier();
  for (int j = lane; j < l; j += 64) Vs[(int64_t)row * l + j] = s_v[meta[1 + j] & 127];
}

// The symmetric split of the singular values over a product of S partials
// [rows][cols]: out = the sum times (by_col) sqrt(s[column]), or divided by
// sqrt(s[row]) (0 where s is 0), in fp32.
__global__ __launch_bounds__(256) void k_split_f32(const double* __restrict__ part, int S, int rows, int cols,
                                                   const double* __restrict__ s, int by_col, float* __restrict__ out) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, n = (int64_t)rows * cols;
  if (q >= n) return;
  double v = part[q];
  for (int z = 1; z < S; ++z) v += part[z * n + q];
  const double x = s[by_col ? (int)(q % cols) : (int)(q / cols)];
  const double sg = sqrt(x > 0.0 ? x : 0.0);
  out[q] = (float)(by_col ? v * sg : sg > 0.0 ? v / sg : 0.0);
}

// Xp = [X; sqrt(damp) I]: rows i < n the activations X [n][cols] (bf16 or
// fp32) in fp64, rows n .. np - 1 the scaled identity (np = n or n + cols).
__global__ __launch_bounds__(256) void k_fill_act(const void* __restrict__ x, int bf16, int n, int cols, double sd,
                                                  int np, double* __restrict__ Xp) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (int64_t)np * cols) return;
  const int i = (int)(q / cols), j = (int)(q % cols);
  if (i < n)
    Xp[q] = bf16 ? (double)__uint_as_float((uint32_t)((const uint16_t*)x)[q] << 16) : (double)((const float*)x)[q];
  else
    Xp[q] = j == i - n ? sd : 0.0;
}

inline unsigned blocks(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

constexpr int kMaxSweeps = 40;
static_assert((int64_t)kMaxSweeps * 127 * 64 * 2 + 128 <= kDgParts, "the rotation log fits the partial products' buffer");

constexpr int dg_lds(int mb, int nb) { return 2 * 16 * (mb + nb) * DG_PITCH * 8; }

// The product op(A) op(B) as S > 1 partials [S][M][N] in part (at most `room`
// doubles), or whole in `one` (S = 1, also where part has no room for two); S
// returned. Tiles: 64 rows by all N <= 128
// columns (the sketch-wide products), all M <= 128 rows by 64 columns (their
// transposes), else 64 x 64; K is split, at least 2 slabs a split and at most
// max_split ways, so that whole rounds of two workgroups per compute unit (what
// the LDS holds) share the product: one round for the thin shapes, two for the
// wide ones.
template <typename TI>
int dgemm_parts(int M, int N, int K, const TI* A, int64_t lda, int ta, const TI* B, int64_t ldb, int tb, double* one,
                double* part, int64_t room, hipStream_t s, int max_split = 1 << 20) {
  const bool thin_n = N <= 128, thin_m = !thin_n && M <= 128;
  const int bm = thin_m ? 16 * ((M + 15) / 16) : 64, bn = thin_n ? 16 * ((N + 15) / 16) : 64;
  const int tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  int64_t S = std::max(1, (thin_n || thin_m ? 512 : 1024) / tiles);
  S = std::min<int64_t>(S, std::min(max_split, K / (2 * DG_K)));
  S = std::min<int64_t>(S, room / ((int64_t)M * N));
  S = std::max<int64_t>(S, 1);
  const int kc = (int)(((K + S - 1) / S + DG_K - 1) / DG_K * DG_K);
  S = std::max(1, (K + kc - 1) / kc);
  double* const C = S > 1 ? part : one;
  const dim3 grid((N + bn - 1) / bn, (M + bm - 1) / bm, (unsigned)S);
#define LX_DG(WM, WN, MI, NI)                                                                                          \
  hipLaunchKernelGGL((k_dgemm<TI, WM, WN, MI, NI>), grid, dim3(256), dg_lds(WM * MI, WN * NI), s, M, N, K, A, lda, ta, B, ldb, tb, C,      \
                     (int64_t)N, kc)
#define LX_DG_CASES(CASE) CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
  if (thin_n) {
#define LX_CASE(NB) case NB: LX_DG(4, 1, 1, NB); break;
    switch (bn / 16) { LX_DG_CASES(LX_CASE) }
#undef LX_CASE
  } else if (thin_m) {
#define LX_CASE(NB) case NB: LX_DG(1, 4, NB, 1); break;
    switch (bm / 16) { LX_DG_CASES(LX_CASE) }
#undef LX_CASE
  } else {
    LX_DG(2, 2, 2, 2);
  }
  return (int)S;
}

// C [M][N] = op(A) op(B): through the partials when K is split.
hipError_t dgemm(int M, int N, int K, const double* A, int64_t lda, int ta, const double* B, int64_t ldb, int tb,
                 double* C, hipStream_t s, double* part) {
  const int S = dgemm_parts(M, N, K, A, lda, ta, B, ldb, tb, C, part, kDgParts, s);
  if (S > 1) hipLaunchKernelGGL(k_dsum, dim3(blocks((int64_t)M * N)), dim3(256), 0, s, part, S, (int64_t)M * N, C);
  return hipGetLastError();
}

// Kernels with more than 64 KB of dynamic LDS: allow it, once per device.
template <int NB>
hipError_t allow_lds_nb() {
  const hipFuncAttribute a = hipFuncAttributeMaxDynamicSharedMemorySize;
  const int n = 16 * NB * 16 * NB * 8;
  hipError_t r = hipFuncSetAttribute((const void*)k_chol<NB>, a, n);
  if (r == hipSuccess) r = hipFuncSetAttribute((const void*)k_trsm_rows<NB>, a, n);
  if (r == hipSuccess) r = hipFuncSetAttribute((const void*)k_dgemm<double, 4, 1, 1, NB>, a, dg_lds(4, NB));
  if (r == hipSuccess) r = hipFuncSetAttribute((const void*)k_dgemm<double, 1, 4, NB, 1>, a, dg_lds(NB, 4));
  if (r == hipSuccess) r = hipFuncSetAttribute((const void*)k_dgemm<float, 4, 1, 1, NB>, a, dg_lds(4, NB));
  if (r == hipSuccess) r = hipFuncSetAttribute((const void*)k_dgemm<float, 1, 4, NB, 1>, a, dg_lds(NB, 4));
  return r;
}
hipError_t allow_lds() {
  static DeviceOnce once;
  int dev = 0;
  if (const hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
  return once.run(dev, hipSuccess, [] {
    hipError_t r = hipFuncSetAttribute((const void*)k_jacobi<1>, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 129 * 8);
    if (r == hipSuccess)
      r = hipFuncSetAttribute((const void*)k_jacobi<3>, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 129 * 8);
    if (r == hipSuccess)
      r = hipFuncSetAttribute((const void*)k_dgemm<double, 2, 2, 2, 2>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              dg_lds(4, 4));
    if (r == hipSuccess)
      r = hipFuncSetAttribute((const void*)k_dgemm<float, 2, 2, 2, 2>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              dg_lds(4, 4));
    if (r == hipSuccess) r = allow_lds_nb<1>();
    if (r == hipSuccess) r = allow_lds_nb<2>();
    if (r == hipSuccess) r = allow_lds_nb<3>();
    if (r == hipSuccess) r = allow_lds_nb<4>();
    if (r == hipSuccess) r = allow_lds_nb<5>();
    if (r == hipSuccess) r = allow_lds_nb<6>();
    if (r == hipSuccess) r = allow_lds_nb<7>();
    if (r == hipSuccess) r = allow_lds_nb<8>();
    return r;
  });
}

// Y (rows x l) <- Y U^-1, U the Cholesky factor of its Gram matrix; U: l x l
// scratch. One pass leaves the basis off orthonormal by about cond(Y)^2 eps: to
// rounding for a well-conditioned sketch, by as much as its own size where a
// column is about 1e-7 of the largest (the pivots are not ordered, so k_chol's
// floor bounds no condition number). Between the products of the subspace
// iteration only the span counts and that the next product is better conditioned
// than without the pass; two passes (CholeskyQR2) make the final basis orthonormal
// to rounding. Emulated in fp64 against two passes everywhere, singular values
// falling geometrically from 1 to 1e-3 .. 1e-7 over l = 74 to 128 columns: A B and
// sigma off by the same down to 1e-6, and within their scatter at 1e-7 (A B by
// 5e-11 and 4e-11, at most 6e-10 and 3e-10). The
// Gram matrix's K is split at most 16 ways (8 past l = 80, where k_chol loads
// fewer partials together): k_chol's one workgroup reads the partials. 2048 rows,
// l = 74, 8 -> 16 ways: Gram matrix 24 -> 14 us.
hipError_t cholqr(double* Y, int rows, int l, int passes, double* U, hipStream_t s, double* part) {
  const int nb = (l + 15) / 16;
  for (int pass = 0; pass < passes; ++pass) {
    const int S = dgemm_parts(l, l, rows, (const double*)Y, l, 1, (const double*)Y, l, 0, part, part, kDgParts, s, nb <= 5 ? 16 : 8);
    const dim3 gt((rows + kTrsmRows - 1) / kTrsmRows);
    switch (nb) {
#define LX_CASE(NB)                                                                                            \
  case NB:                                                                                                     \
    hipLaunchKernelGGL(k_chol<NB>, dim3(1), dim3(256), (size_t)l * 16 * NB * 8, s, part, S, l, U);             \
    hipLaunchKernelGGL(k_trsm_rows<NB>, gt, dim3(256), (size_t)16 * NB * 16 * NB * 8, s, Y, rows, l, U);       \
    break;
      LX_DG_CASES(LX_CASE)
#undef LX_CASE
    }
    if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

// From an orthonormal sketch Y (rows x l) of the range of an operator M, T =
// Y^T R (l x cols) and Gm = (Y^T M)(Y^T M)^T (l x l): the eigenpairs of Gm
// (descending), sigma = the square roots of the r largest, A = Y Ut[:, :r]
// sigma^(1/2) and B = sigma^(-1/2) Ut[:, :r]^T T (rows of B with sigma = 0
// are 0); Ad (rows x r) and Bd (r x cols) are scratch.
hipError_t factors_from_sketch(int rows, int cols, int r, int l, const double* Y, const double* T, const double* Gm,
                               double* lam, double* Ve, double* sig, double* Ad, double* Bd, float* A, float* B,
                               double* sigma, hipStream_t s, double* part) {
  const int lp = jacobi_order(l), half = lp / 2;
  int32_t* const meta = (int32_t*)(part + kDgParts - 128);
  const int nrest = half * (half - 1) / 2 - half;
  const int nth = 64 + std::min(960, (nrest + 63) / 64 * 64);  // wavefront 0 and the other blocks' threads
  hipLaunchKernelGGL(nrest <= 960 ? k_jacobi<1> : k_jacobi<3>, dim3(1), dim3(std::max(nth, 128)),
                     (size_t)lp * (lp + 1) * sizeof(double), s, Gm, l, lp, lam, (double2*)part, meta, kMaxSweeps);
  hipLaunchKernelGGL(k_jacobi_vec, dim3(l), dim3(64), 0, s, (const double2*)part, meta, l, lp, lam, r, Ve, sig, sigma);
  int S = dgemm_parts(rows, r, l, Y, l, 0, (const double*)Ve, l, 0, Ad, part, kDgParts, s);
  hipLaunchKernelGGL(k_split_f32, dim3(blocks((int64_t)rows * r)), dim3(256), 0, s,
                     (const double*)(S > 1 ? part : Ad), S, rows, r, sig, 1, A);
  S = dgemm_parts(r, cols, l, (const double*)Ve, l, 1, T, cols, 0, Bd, part, kDgParts, s);
  hipLaunchKernelGGL(k_split_f32, dim3(blocks((int64_t)r * cols)), dim3(256), 0, s,
                     (const double*)(S > 1 ? part : Bd), S, r, cols, sig, 0, B);
  return hipGetLastError();
}

}  // namespace

size_t lowrank_ws_doubles(int rows, int cols, int l) { return (size_t)stage3_ws(rows, cols, -1, l).total; }

size_t weighted_ws_doubles(int rows, int cols, int np, int l) { return (size_t)stage3_ws(rows, cols, np, l).total; }

hipError_t launch_align_cost(const void* dg, const void* du, const void* dd, const void* mg, const void* mu,
                             const void* md, int bf16, int f, int d, double* cost, double* ws, hipStream_t s) {
  if (const hipError_t e0 = allow_lds(); e0 != hipSuccess) return e0;
  // ws: 2 f (3d + 1) doubles: the fp32 vectors take half of it, the partial
  // products the rest
  const int64_t n = (int64_t)f * 3 * d;
  float* const a = (float*)ws;
  float* const b = a + n;
  double* const na = ws + n;
  double* const nb = na + f;
  double* const part = nb + f;  // n doubles
  hipLaunchKernelGGL(k_neurons, dim3(f), dim3(256), 0, s, dg, du, dd, bf16, f, d, a, na);
  hipLaunchKernelGGL(k_neurons, dim3(f), dim3(256), 0, s, mg, mu, md, bf16, f, d, b, nb);
  const int S = dgemm_parts(f, f, 3 * d, (const float*)a, 3 * d, 0, (const float*)b, 3 * d, 1, cost, part, n, s);
  hipLaunchKernelGGL(k_cost_finish, dim3(blocks((int64_t)f * f)), dim3(256), 0, s, na, nb, f,
                     (const double*)(S > 1 ? part : cost), S, cost);
  return hipGetLastError();
}

hipError_t launch_lowrank(const void* wd, const void* wm, int bf16, int rows, int cols, const int32_t* perm, int axis,
                          int r, int l, int q, const double* omega, float* A, float* B, double* sigma, double* ws,
                          hipStream_t s) {
  if (const hipError_t e0 = allow_lds(); e0 != hipSuccess) return e0;
  const Stage3Ws w = stage3_ws(rows, cols, -1, l);
  double* const R = ws + w.R;
  double* const Y = ws + w.Y;
  double* const Z = ws + w.Z;
  double* const Bs = ws + w.T;
  double* const G = ws + w.G;
  double* const U = ws + w.U;
  double* const Ve = ws + w.Ve;
  double* const lam = ws + w.lam;
  double* const sig = ws + w.sig;
  double* const Ad = ws + w.Ad;
  double* const part = ws + w.part;
  hipLaunchKernelGGL(k_residual, dim3(blocks((int64_t)rows * cols)), dim3(256), 0, s, wd, wm, bf16, rows, cols, perm,
                     axis, R);
  hipError_t e;
  // Y = R Omega, orthonormalised; q rounds of Z = R^T Y, Y = R Z, each
  // orthonormalised
  if ((e = dgemm(rows, l, cols, R, cols, 0, omega, l, 0, Y, s, part)) != hipSuccess) return e;
  if ((e = cholqr(Y, rows, l, q > 0 ? 1 : 2, U, s, part)) != hipSuccess) return e;
  for (int it = 0; it < q; ++it) {
    if ((e = dgemm(cols, l, rows, R, cols, 1, Y, l, 0, Z, s, part)) != hipSuccess) return e;
    if ((e = cholqr(Z, cols, l, 1, U, s, part)) != hipSuccess) return e;
    if ((e = dgemm(rows, l, cols, R, cols, 0, Z, l, 0, Y, s, part)) != hipSuccess) return e;
    if ((e = cholqr(Y, rows, l, it + 1 < q ? 1 : 2, U, s, part)) != hipSuccess) return e;
  }
  // Bs = Y^T R (l x cols); Bs Bs^T (l x l) = Ut diag(lambda) Ut^T
  if ((e = dgemm(l, cols, rows, Y, l, 1, R, cols, 0, Bs, s, part)) != hipSuccess) return e;
  if ((e = dgemm(l, l, cols, Bs, cols, 0, Bs, cols, 1, G, s, part)) != hipSuccess) return e;
  return factors_from_sketch(rows, cols, r, l, Y, Bs, G, lam, Ve, sig, Ad, Z, A, B, sigma, s, part);
}

hipError_t launch_weighted(const void* wd, const void* wm, int bf16, int rows, int cols, const int32_t* perm, int axis,
                           const void* x, int x_bf16, int n, double damp, int r, int l, int q, const double* omega,
                           float* A, float* B, double* sigma, double* ws, hipStream_t s) {
  const int np = n + (damp > 0.0 ? cols : 0);
  if (const hipError_t e0 = allow_lds(); e0 != hipSuccess) return e0;
  const Stage3Ws w = stage3_ws(rows, cols, np, l);
  double* const R = ws + w.R;
  double* const Xp = ws + w.Xp;  // [X; sqrt(damp) I]
  double* const P = ws + w.P;
  double* const Y = ws + w.Y;
  double* const Z = ws + w.Z;
  double* const T = ws + w.T;
  double* const Wt = ws + w.Wt;
  double* const G = ws + w.G;
  double* const U = ws + w.U;
  double* const Ve = ws + w.Ve;
  double* const lam = ws + w.lam;
  double* const sig = ws + w.sig;
  double* const Ad = ws + w.Ad;
  double* const part = ws + w.part;
  hipLaunchKernelGGL(k_residual, dim3(blocks((int64_t)rows * cols)), dim3(256), 0, s, wd, wm, bf16, rows, cols, perm,
                     axis, R);
  hipLaunchKernelGGL(k_fill_act, dim3(blocks((int64_t)np * cols)), dim3(256), 0, s, x, x_bf16, n, cols, sqrt(damp),
                     np, Xp);
  hipError_t e;
  // The operator M = R Xp^T (rows x np), applied as two thin products:
  // Y = R (Xp^T Omega), orthonormalised; q rounds of Z = Xp (R^T Y) and
  // Y = R (Xp^T Z), each orthonormalised
  if ((e = dgemm(cols, l, np, Xp, cols, 1, omega, l, 0, P, s, part)) != hipSuccess) return e;
  if ((e = dgemm(rows, l, cols, R, cols, 0, P, l, 0, Y, s, part)) != hipSuccess) return e;
  if ((e = cholqr(Y, rows, l, q > 0 ? 1 : 2, U, s, part)) != hipSuccess) return e;
  for (int it = 0; it < q; ++it) {
    if ((e = dgemm(cols, l, rows, R, cols, 1, Y, l, 0, P, s, part)) != hipSuccess) return e;
    if ((e = dgemm(np, l, cols, Xp, cols, 0, P, l, 0, Z, s, part)) != hipSuccess) return e;
    if ((e = cholqr(Z, np, l, 1, U, s, part)) != hipSuccess) return e;
    if ((e = dgemm(cols, l, np, Xp, cols, 1, Z, l, 0, P, s, part)) != hipSuccess) return e;
    if ((e = dgemm(rows, l, cols, R, cols, 0, P, l, 0, Y, s, part)) != hipSuccess) return e;
    if ((e = cholqr(Y, rows, l, it + 1 < q ? 1 : 2, U, s, part)) != hipSuccess) return e;
  }
  // T = Y^T R (l x cols); Wt = Y^T M = T Xp^T (l x np); Wt Wt^T = Ut diag(lambda) Ut^T.
  // B = sigma^(-1/2) Ut^T T is sigma^(-1/2) U_r^T R with U_r = Y Ut[:, :r].
  if ((e = dgemm(l, cols, rows, Y, l, 1, R, cols, 0, T, s, part)) != hipSuccess) return e;
  if ((e = dgemm(l, np, cols, T, cols, 0, Xp, cols, 1, Wt, s, part)) != hipSuccess) return e;
  if ((e = dgemm(l, l, np, Wt, np, 0, Wt, np, 1, G, s, part)) != hipSuccess) return e;
  return factors_from_sketch(rows, cols, r, l, Y, T, G, lam, Ve, sig, Ad, P, A, B, sigma, s, part);
}

}  // namespace lx

// Grouped GEMMs of the forward: every projection is C = A * W^T over the rows
// of one tree level, tile by tile, where a tile's rows all use the weights of
// one node (W in nn.Linear layout [N][K], K contiguous).
//
// bf16 path (gfx950 MFMA, v_mfma_f32_32x32x16_bf16):
//   * 128 x 128 output tile per 256-thread workgroup, 4 wavefronts of 64 x 64,
//     2 x 2 MFMA 32x32 blocks each, K staged through LDS 64 at a time;
//   * A rows may be gathered through an index map (activations per (token,
//     node) row), so no gathered copy of x is ever written;
//   * A may be bf16 (activations) or fp32 (intermediates). fp32 A is split
//     on the fly into hi = bf16(a) and lo = bf16(a - hi); both are multiplied
//     with the same weight fragment, which keeps about 16 bits of the
//     intermediate's mantissa at the cost of a second MFMA per fragment;
//   * LDS rows of 64 bf16 (128 B) are stored with the 16-byte chunk index
//     XOR-swizzled by the row so fragment reads of 32 consecutive rows hit
//     distinct banks;
//   * double-buffered LDS with register prefetch: the next K-slab is loaded
//     from HBM while the current one is multiplied.
// fp32 path: v_mfma_f32_32x32x2_f32 on 64 x 64 tiles with direct HBM -> LDS loads
// (K a multiple of 16), else a plain LDS-tiled VALU kernel.
#include "lx_internal.h"

namespace lx {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint16_t u16;

constexpr int BM = 128, BN = 128, BK = 64, NTHR = 256;
static_assert((BM & (BM - 1)) == 0, "tile heights are powers of two (bucketing shifts)");

__device__ __forceinline__ int swz(int row) { return (row ^ (row >> 3)) & 7; }
__device__ __forceinline__ int lds_off(int row, int kc) { return row * BK + ((kc ^ swz(row)) << 3); }

__device__ __forceinline__ void split_hilo(const float4& a, const float4& b, uint4& hi, uint4& lo) {
  const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  bf16x8 h, l;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const __bf16 hb = (__bf16)v[i];
    h[i] = hb;
    l[i] = (__bf16)(v[i] - (float)hb);
  }
  hi = __builtin_bit_cast(uint4, h);
  lo = __builtin_bit_cast(uint4, l);
}

template <int AMODE>
__global__ __launch_bounds__(NTHR) void k_gemm_bf16(GemmArgs p) {
  if ((int)blockIdx.x >= *p.n_tiles) return;
  const TileEntry te = p.tiles[blockIdx.x];
  const int ntp0 = (p.ncols[0] + BN - 1) / BN;
  const int part = (int)blockIdx.y < ntp0 ? 0 : 1;
  const int n0 = ((int)blockIdx.y - (part ? ntp0 : 0)) * BN;
  const int ncol = p.ncols[part];
  const int K = p.K;
  const int akoff = p.a_koff[part];
  const u16* __restrict__ Bw = (const u16*)p.B[part] + (int64_t)te.widx * p.b_stride[part];

  constexpr bool HILO = AMODE == A_F32_HILO;
  __shared__ __attribute__((aligned(16))) u16 sA[2][BM * BK];
  __shared__ __attribute__((aligned(16))) u16 sB[2][BN * BK];
  __shared__ __attribute__((aligned(16))) u16 sAl[HILO ? 2 : 1][HILO ? BM * BK : 8];

  const int tid = threadIdx.x;
  const int lrow = tid >> 3;   // 0..31
  const int lkc = tid & 7;     // 16-byte chunk within a 64-wide K slab

  // Rows this thread stages: lrow + 32*i. Invalid rows/columns read nothing
  // and stage zeros; their offsets are clamped to row 0 so no address is
  // ever formed outside the operands.
  int64_t aoff[4], boff[4];
  unsigned amask = 0, bmask = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = lrow + 32 * i;
    const bool av = r < te.nrows;
    const int64_t src = !av ? 0 : (p.a_rows ? (int64_t)p.a_rows[te.row0 + r] : (int64_t)(te.row0 + r));
    aoff[i] = src * p.lda + akoff;
    amask |= av ? (1u << i) : 0u;
    const int n = n0 + r;
    boff[i] = n < ncol ? (int64_t)n * K : 0;
    bmask |= n < ncol ? (1u << i) : 0u;
  }
  const u16* __restrict__ Ab = (const u16*)p.A;
  const float* __restrict__ Af = (const float*)p.A;

  uint4 ra0, ra1, ra2, ra3, rb0, rb1, rb2, rb3;
  float4 rf0a, rf0b, rf1a, rf1b, rf2a, rf2b, rf3a, rf3b;
  const uint4 z4 = make_uint4(0, 0, 0, 0);
  const float4 zf = make_float4(0.f, 0.f, 0.f, 0.f);

// Loads are unconditional from clamped, in-bounds addresses (row 0, column
// 0 for masked lanes); masking selects the loaded value, never the address.
// The four staged rows are written out explicitly so every staging register
// has a fixed name (no dynamically indexed arrays).
#define LX_LD1(i)                                                                 \
  do {                                                                            \
    const bool av = kin && ((amask >> i) & 1u);                                   \
    if (HILO) {                                                                   \
      const float4* q = (const float4*)(Af + aoff[i] + kcl);                      \
      const float4 v0 = q[0], v1 = q[1];                                          \
      rf##i##a = av ? v0 : zf;                                                    \
      rf##i##b = av ? v1 : zf;                                                    \
    } else {                                                                      \
      const uint4 v = *(const uint4*)(Ab + aoff[i] + kcl);                        \
      ra##i = av ? v : z4;                                                        \
    }                                                                             \
    const uint4 w = *(const uint4*)(Bw + boff[i] + kcl);                          \
    rb##i = (kin && ((bmask >> i) & 1u)) ? w : z4;                                \
  } while (0)
#define LX_GLOAD(K0)                                                              \
  do {                                                                            \
    const int kk = (K0) + lkc * 8;                                                \
    const bool kin = kk < K;                                                      \
    const int kcl = kin ? kk : 0;                                                 \
    LX_LD1(0);                                                                    \
    LX_LD1(1);                                                                    \
    LX_LD1(2);                                                                    \
    LX_LD1(3);                                                                    \
  } while (0)
#define LX_ST1(BUF, i)                                                            \
  do {                                                                            \
    const int off = lds_off(lrow + 32 * i, lkc);                                  \
    if (HILO) {                                                                   \
      uint4 hi, lo;                                                               \
      split_hilo(rf##i##a, rf##i##b, hi, lo);                                     \
      *(uint4*)&sA[BUF][off] = hi;                                                \
      *(uint4*)&sAl[BUF][off] = lo;                                               \
    } else {                                                                      \
      *(uint4*)&sA[BUF][off] = ra##i;                                             \
    }                                                                             \
    *(uint4*)&sB[BUF][off] = rb##i;                                               \
  } while (0)
#define LX_SSTORE(BUF)                                                            \
  do {                                                                            \
    LX_ST1(BUF, 0);                                                               \
    LX_ST1(BUF, 1);                                                               \
    LX_ST1(BUF, 2);                                                               \
    LX_ST1(BUF, 3);                                                               \
  } while (0)

  f32x16 acc[2][2];
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;

  const int wave = tid >> 6, lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1;
  const int nk = (K + BK - 1) / BK;

  LX_GLOAD(0);
  LX_SSTORE(0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) LX_GLOAD((kt + 1) * BK);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      const int kc = ks * 2 + (lane >> 5);
      bf16x8 af[2], al[2], bw[2];
#pragma unroll
      for (int mi = 0; mi < 2; ++mi) {
        const int off = lds_off(wm * 64 + mi * 32 + (lane & 31), kc);
        af[mi] = *(const bf16x8*)&sA[cur][off];
        if (HILO) al[mi] = *(const bf16x8*)&sAl[cur][off];
      }
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
        bw[ni] = *(const bf16x8*)&sB[cur][lds_off(wn * 64 + ni * 32 + (lane & 31), kc)];
#pragma unroll
      for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[mi], bw[ni], acc[mi][ni], 0, 0, 0);
          if (HILO)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[mi], bw[ni], acc[mi][ni], 0, 0, 0);
        }
    }
    if (kt + 1 < nk) LX_SSTORE(cur ^ 1);
    __syncthreads();
  }

#undef LX_LD1
#undef LX_GLOAD
#undef LX_ST1
#undef LX_SSTORE

  // 32x32 accumulator layout: lane holds column (lane & 31) and rows
  // 8*(i/4) + 4*(lane/32) + (i%4) for i = 0..15.
  float* __restrict__ C = p.C + p.c_coloff[part] + n0;
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
      const int c = wn * 64 + ni * 32 + (lane & 31);
      if (n0 + c >= ncol) continue;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = wm * 64 + mi * 32 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
        if (r < te.nrows) C[(int64_t)(te.row0 + r) * p.ldc + c] = acc[mi][ni][i];
      }
    }
}

// ------------------------------------------------------------------ fp32 path
constexpr int FBM = 64, FBN = 64, FBK = 16;
static_assert((FBM & (FBM - 1)) == 0, "tile heights are powers of two (bucketing shifts)");

__global__ __launch_bounds__(256) void k_gemm_f32(GemmArgs p) {
  if ((int)blockIdx.x >= *p.n_tiles) return;
  const TileEntry te = p.tiles[blockIdx.x];
  const int ntp0 = (p.ncols[0] + FBN - 1) / FBN;
  const int part = (int)blockIdx.y < ntp0 ? 0 : 1;
  const int n0 = ((int)blockIdx.y - (part ? ntp0 : 0)) * FBN;
  const int ncol = p.ncols[part];
  const int K = p.K;
  const float* __restrict__ Bw = (const float*)p.B[part] + (int64_t)te.widx * p.b_stride[part];
  const float* __restrict__ Af = (const float*)p.A;

  __shared__ float sA[FBK][FBM + 4];
  __shared__ float sB[FBK][FBN + 4];
  const int tid = threadIdx.x;
  const int ty = tid >> 4, tx = tid & 15;
  const int lk = tid & 15, lr = tid >> 4;  // loader: row lr + 16*e, column lk

  const float* arow[4];
  const float* brow[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = lr + 16 * e;
    if (r < te.nrows) {
      const int64_t src = p.a_rows ? (int64_t)p.a_rows[te.row0 + r] : (int64_t)(te.row0 + r);
      arow[e] = Af + src * p.lda + p.a_koff[part];
    } else {
      arow[e] = nullptr;
    }
    brow[e] = (n0 + r < ncol) ? Bw + (int64_t)(n0 + r) * K : nullptr;
  }

  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

  for (int k0 = 0; k0 < K; k0 += FBK) {
    const int kk = k0 + lk;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = lr + 16 * e;
      sA[lk][r] = (arow[e] && kk < K) ? arow[e][kk] : 0.f;
      sB[lk][r] = (brow[e] && kk < K) ? brow[e][kk] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < FBK; ++q) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = sA[q][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = sB[q][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
  float* __restrict__ C = p.C + p.c_coloff[part] + n0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = ty * 4 + i;
    if (r >= te.nrows) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = tx * 4 + j;
      if (n0 + c < ncol) C[(int64_t)(te.row0 + r) * p.ldc + c] = acc[i][j];
    }
  }
}

// The fp32 products on the matrix cores: 64 x 64 tiles by 4 wavefronts (2 x 2
// grid of 32 x 32 blocks), full fp32 operands and accumulation (in two sums of
// half the products each, which also halves the rounding of one long chain).
// K slabs of MBK values go straight to LDS through a ring of MST stages; 48 KB
// per workgroup (32 KB when MBK is 16), so three or more workgroups share a
// compute unit and cover each other's waits. LDS rows of MBK values, 16-byte
// chunks XOR-swizzled by the row so that 16 rows of one chunk fall on distinct
// banks. A lane's 16-byte fragment read holds 4 consecutive k of its row; the two
// lane halves read neighbouring chunks, so MFMA step s of a chunk pair multiplies
// k = s and k = 4 + s (any pairing sums the same products). Bound by the fp32
// MFMA rate (157 TFLOP/s nominal) and padding rows. Against the VALU kernel
// above: d = 2048, f = 768, 16 anchors, rank 64, T = 300: anchor gate|up 405 -> 187
// us (two thirds of it MFMA time), low-rank input 318 -> 60, anchor down 180 ->
// 90. 128-column tiles: 177, 96, 104; 16-wide slabs: 191, 73, 97.
// A node's few rows (19 of 64 on average there) leave half of the wavefronts of a
// tile idle; sharing K with them: low-rank input 60 -> 40 us, the leaf level's
// other products 77 -> 62 us together.
__device__ __forceinline__ void f32_load_lds16(const void* gptr, const void* lds_dst) {
  typedef __attribute__((address_space(3))) void lds_void_t;
  const uint32_t lds = (uint32_t)(uintptr_t)(lds_void_t*)lds_dst;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(gptr), "s"(__builtin_amdgcn_readfirstlane(lds))
               : "memory");
}
// s_waitcnt vmcnt(N) alone; barrier without a fence (each wavefront waits for
// its own loads first, and here for its own LDS reads: after the barrier
// another wavefront's direct load overwrites the stage that they read)
template <int N>
__device__ __forceinline__ void f32_wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}
__device__ __forceinline__ void f32_bar() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int MBK, int MST>
__global__ __launch_bounds__(256) void k_gemm_f32m(GemmArgs p) {
  constexpr int CH = MBK / 4, RPT = 256 / CH;  // 16-byte chunks per row, rows per load round
  constexpr int RA = FBM / RPT, RB = FBN / RPT;
  // XCD-aware order (workgroups go round-robin over the 8 XCDs): each XCD takes
  // a contiguous range of (row tile, column tile) items, so the column tiles of
  // a row tile and the row tiles of a node share rows and weights in one L2
  const int ntp0 = (p.ncols[0] + FBN - 1) / FBN, ntn = ntp0 + (p.ncols[1] + FBN - 1) / FBN;
  const int items = *p.n_tiles * ntn, x = blockIdx.x % 8, q8 = items / 8, r8 = items % 8;
  const int in_xcd = blockIdx.x / 8;
  if (in_xcd >= q8 + (x < r8 ? 1 : 0)) return;
  const int item = x * q8 + (x < r8 ? x : r8) + in_xcd;
  const TileEntry te = p.tiles[item / ntn];
  const int nt = item % ntn, part = nt < ntp0 ? 0 : 1;
  const int n0 = (nt - (part ? ntp0 : 0)) * FBN;
  const int ncol = p.ncols[part];
  const int K = p.K;
  __shared__ __attribute__((aligned(1024))) float smem[MST * (FBM + FBN) * MBK];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;

  // rows past the tile's end and weight rows past ncol are clamped (their
  // results are never stored), so every load is in bounds
  auto swz = [](int row) { return MBK == 16 ? (row >> 2) & 3 : (row >> 1) & 7; };
  const float* ap[RA];
  const float* bp[RB];
#pragma unroll
  for (int i = 0; i < RA; ++i) {
    const int row = i * RPT + tid / CH, c = (tid % CH) ^ swz(row);
    const int r = row < te.nrows ? row : te.nrows - 1;
    const int64_t src = p.a_rows ? (int64_t)p.a_rows[te.row0 + r] : (int64_t)(te.row0 + r);
    ap[i] = (const float*)p.A + src * p.lda + p.a_koff[part] + c * 4;
  }
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int row = i * RPT + tid / CH, c = (tid % CH) ^ swz(row);
    const int n = n0 + row < ncol ? n0 + row : ncol - 1;
    bp[i] = (const float*)p.B[part] + (int64_t)te.widx * p.b_stride[part] + (int64_t)n * K + c * 4;
  }
  auto issue = [&](int kt) {
    float* const st = smem + (kt % MST) * (FBM + FBN) * MBK;
#pragma unroll
    for (int i = 0; i < RA; ++i) f32_load_lds16(ap[i] + kt * MBK, st + i * 1024 + wave * 256);
#pragma unroll
    for (int i = 0; i < RB; ++i) f32_load_lds16(bp[i] + kt * MBK, st + FBM * MBK + i * 1024 + wave * 256);
  };

  const int wm = wave >> 1, wn = wave & 1, half = lane >> 5;
  // a tile of at most 32 rows: the second pair of wavefronts takes the second
  // half of every slab's k for the same rows
  const bool low = te.nrows <= 32;
  const int rw = low ? 0 : wm * 32;
  const int ra = rw + (lane & 31), rb = wn * 32 + (lane & 31);
  const bool live = rw < te.nrows && n0 + wn * 32 < ncol;  // wavefront-uniform
  f32x16 acc0, acc1;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc0[i] = acc1[i] = 0.f;
  const int nk = K / MBK;
  const int npre = nk < MST - 1 ? nk : MST - 1;
  for (int i = 0; i < npre; ++i) issue(i);
  for (int kt = 0; kt < nk; ++kt) {
    // slabs issued so far: 0 .. min(kt + MST - 2, nk - 1); slab kt must have landed
    const int ahead = (kt + MST - 2 < nk - 1 ? kt + MST - 2 : nk - 1) - kt;
    if (ahead >= 2)
      f32_wait_vm<2 * (RA + RB)>();
    else if (ahead == 1)
      f32_wait_vm<RA + RB>();
    else
      f32_wait_vm<0>();
    f32_bar();  // slab kt is in LDS; slab kt - 1's stage is free
    if (kt + MST - 1 < nk) issue(kt + MST - 1);
    if (live) {
      const float* const st = smem + (kt % MST) * (FBM + FBN) * MBK;
      const int j0 = low && wm ? CH / 4 : 0, j1 = low && !wm ? CH / 4 : CH / 2;
      for (int jj = j0; jj < j1; jj += CH / 4)
#pragma unroll
      for (int j = jj; j < jj + CH / 4; ++j) {
        const int c = 2 * j + half;
        const float4 fa = *(const float4*)(st + ra * MBK + ((c ^ swz(ra)) << 2));
        const float4 fb = *(const float4*)(st + FBM * MBK + rb * MBK + ((c ^ swz(rb)) << 2));
        acc0 = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.x, fb.x, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.y, fb.y, acc1, 0, 0, 0);
        acc0 = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.z, fb.z, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.w, fb.w, acc1, 0, 0, 0);
      }
    }
  }
  if (low) {
    // the two k halves meet in LDS (every slab's stage is free after the barrier)
    __syncthreads();
    float* const x = smem + wn * 1024 + lane;
    if (wm && live) {
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i * 64] = acc0[i] + acc1[i];
    }
    __syncthreads();
    if (wm || !live) return;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc0[i] += x[i * 64];
  }
  const int c = n0 + wn * 32 + (lane & 31);
  if (!live || c >= ncol) return;
  float* __restrict__ C = p.C + p.c_coloff[part] + c;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int rr = rw + 8 * (i >> 2) + 4 * half + (i & 3);
    if (rr < te.nrows) C[(int64_t)(te.row0 + rr) * p.ldc] = acc0[i] + acc1[i];
  }
}

}  // namespace

int gemm_bm(lx_dtype dt) { return dt == LX_BF16 ? BM : FBM; }
int gemm_bn(lx_dtype dt) { return dt == LX_BF16 ? BN : FBN; }

hipError_t launch_gemm(const GemmArgs& g, lx_dtype dt, AMode am, int grid_x, hipStream_t s) {
  const int bn = gemm_bn(dt);
  const int gy = (g.ncols[0] + bn - 1) / bn + (g.ncols[1] + bn - 1) / bn;
  if (grid_x <= 0 || gy <= 0) return hipSuccess;
  const dim3 grid(grid_x, gy);
  if (dt == LX_F32) {
    // 16-byte loads of whole slabs: K, the row pitch and every column offset
    // multiples of 4 values (weights and workspace are 16-byte aligned)
    const bool ok = g.lda % 4 == 0 && g.a_koff[0] % 4 == 0 && g.a_koff[1] % 4 == 0 && g.b_stride[0] % 4 == 0 &&
                    g.b_stride[1] % 4 == 0;
    const dim3 wgs((unsigned)(((int64_t)grid_x * gy + 7) / 8 * 8));
    if (ok && g.K % 32 == 0)
      hipLaunchKernelGGL((k_gemm_f32m<32, 3>), wgs, dim3(256), 0, s, g);
    else if (ok && g.K % 16 == 0)
      hipLaunchKernelGGL((k_gemm_f32m<16, 4>), wgs, dim3(256), 0, s, g);
    else
      hipLaunchKernelGGL(k_gemm_f32, grid, dim3(256), 0, s, g);
  } else if (am == A_BF16) {
    hipLaunchKernelGGL(k_gemm_bf16<A_BF16>, grid, dim3(NTHR), 0, s, g);
  } else {
    hipLaunchKernelGGL(k_gemm_bf16<A_F32_HILO>, grid, dim3(NTHR), 0, s, g);
  }
  return hipGetLastError();
}

}  // namespace lx

// Dense batched kernels of the transfer-block build (CDNA4 / gfx950).
//
// * k_assemble   : plane blocks D_k = A_plane - diag(r) G diag(c) [- ...]
//                  (the Schur complement recursion of block-tridiagonal
//                  elimination across the thin slab direction);
// * gj_invert    : in-place blocked Gauss-Jordan inversion without pivoting,
//                  kNB-wide pivot blocks; each step is a rank-kNB update done
//                  on the matrix cores (MFMA 16x16x4, FP32 or FP64);
// * k_gemm       : batched C = alpha A diag(s) B + beta C on the matrix cores
//                  (transfer chains Y_k = -G_k E Y_{k-1} and S = Sigma^{-1} R);
// * k_scale_cols : C = alpha A diag(s) (first link of a transfer chain).
//
// All matrices are ld x ld row-major, ld a multiple of 128, padded with the
// identity; products over the padding are left out.  Work-group tiles are
// 128 x 128 with 4 wavefronts of 64 lanes, each owning a 64 x 64 sub-tile (4 x
// 4 MFMA tiles); FP32 products of many tiles take those of tiles.h.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "tiles.h"

namespace ddst {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <typename T> struct AccT;
template <> struct AccT<float> { using type = f32x4; };
template <> struct AccT<double> { using type = f64x4; };

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f64x4 mfma16(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int BK = 8;            // k-depth of one FP64 LDS stage
constexpr int LW = kTile + 16;   // LDS row width (padding spreads banks)

template <int N, typename T>
__device__ __forceinline__ void ld16n(const T *p, T *r) {
  constexpr int V = 16 / sizeof(T);
  static_assert(N % V == 0, "whole 16-byte vectors");
#pragma unroll
  for (int i = 0; i < N / V; ++i) {
    const typename V16<T>::type v = ld16(p + V * i);
#pragma unroll
    for (int e = 0; e < V; ++e) r[V * i + e] = v[e];
  }
}

// Map the linear work-group id so that consecutive logical tiles land on
// the same XCD (work-groups are dispatched round-robin over the 8 XCDs):
// tiles of one batch entry then share one L2.  XCD x receives ids x, x + 8,
// ...; it is given the contiguous logical range starting at
// x q + min(x, rem) (total = 8 q + rem), a bijection for any total.
__device__ __forceinline__ int xcd_remap(int lin, int total) {
  const int x = lin & 7, k = lin >> 3, q = total >> 3, rem = total & 7;
  return x * q + (x < rem ? x : rem) + k;
}

template <typename T>
struct Tile {
  typename AccT<T>::type v[4][4];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[i][j][r] = T(0);
  }
};

// FP32 products on the BF16 matrix cores.  Every FP32 operand is split
// into three BF16 parts, x = x1 + x2 + x3 (x1 = bf16(x), x2 = bf16(x - x1),
// x3 = bf16(x - x1 - x2); each difference is exact in FP32 and the three
// parts carry the 24-bit significand), and a b is formed from the six
// products whose parts carry weight down to 2^-24 relative (a1 b1, a1 b2,
// a2 b1, a1 b3, a2 b2, a3 b1; the three dropped ones are below 2^-27),
// each exact in the FP32 accumulators of v_mfma_f32_16x16x32_bf16, added
// smallest first.  The result has the accuracy of an FP32 product; the
// BF16 matrix cores do the six products in 6 x 16 cycles per 16 x 16 x 32
// tile against 8 x 32 for the FP32 instruction (dense peaks 2.5 PFLOP/s
// BF16 and 157.3 TFLOP/s FP32).  FP32 operands are staged 32 deep.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f32x4 mfma_bf16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
struct Split3 {
  bf16x8 h, m, l;
};
// Parts of eight FP32 values (x[j] = h[j] + m[j] + l[j] to 2^-26 relative).
// Pairs are rounded together (one packed conversion gives two BF16 values
// in one register); the FP32 value of a part is its BF16 bits moved to the
// upper half (a shift for the low element, a mask for the high one), so a
// pair costs three conversions, two shifts, two masks and four
// subtractions.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned cvt_pk(float a, float b) {
  const f32x2 v = {a, b};
  const bf16x2 p = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(unsigned, p);
}
__device__ __forceinline__ float lo_f(unsigned p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float hi_f(unsigned p) { return __uint_as_float(p & 0xffff0000u); }
__device__ __forceinline__ void split8(const float (&x)[8], Split3 &s) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  u32x4 h, m, l;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float x0 = x[2 * j], x1 = x[2 * j + 1];
    const unsigned hp = cvt_pk(x0, x1);
    const float r0 = x0 - lo_f(hp), r1 = x1 - hi_f(hp);
    const unsigned mp = cvt_pk(r0, r1);
    const float q0 = r0 - lo_f(mp), q1 = r1 - hi_f(mp);
    h[j] = hp;
    m[j] = mp;
    l[j] = cvt_pk(q0, q1);
  }
  s.h = __builtin_bit_cast(bf16x8, h);
  s.m = __builtin_bit_cast(bf16x8, m);
  s.l = __builtin_bit_cast(bf16x8, l);
}
__device__ __forceinline__ f32x4 mfma_x6(const Split3 &a, const Split3 &b, f32x4 c) {
  c = mfma_bf16(a.l, b.h, c);
  c = mfma_bf16(a.m, b.m, c);
  c = mfma_bf16(a.h, b.l, c);
  c = mfma_bf16(a.m, b.h, c);
  c = mfma_bf16(a.h, b.m, c);
  return mfma_bf16(a.h, b.h, c);
}

// LDS of one tile product: FP64 operands staged 8 deep ([8][LW] each) and
// double-buffered (one barrier a stage; the update of 31 matrices of 1024 rows
// 180 us, with single stages of 16 and the exchange that FP32 uses 186);
// FP32 operands as their three BF16 parts, 32 deep, in fragment order
// ([part][row or column][k], k contiguous, rows padded to 40 entries).
constexpr int XK = 32;           // k per stage of the split products
constexpr int XKP = XK + 8;      // padded row of one BF16 part
template <typename T> struct MmaLds {
  static constexpr int bytes = 2 * 2 * BK * LW * (int)sizeof(T);
};
template <> struct MmaLds<float> {
  static constexpr int bytes = 2 * 3 * kTile * XKP * 2;
};

// acc += (NEG_A ? -A : A)[0:128, 0:K] * diag(bscale[0:K]) * B[0:K, 0:128]
// with FP32 operands on the BF16 matrix cores (split products above);
// layouts and arguments as mma_tile.  Each stage loads 32 k of both
// operands (a thread holds 16 values of one row of A and of one column of
// B), splits them once and stores the three parts in fragment order, so the
// product loop reads whole 8-element fragments (16 bytes) from LDS.
template <bool NEG_A, bool TA, bool TB, bool PART>
__device__ __forceinline__ void mma_tile_x6(const float *__restrict__ A, int lda,
                                            const float *__restrict__ B, int ldb,
                                            const double *__restrict__ bscale, int K,
                                            unsigned char *smem, Tile<float> &acc, int ni,
                                            int nj) {
  typedef __bf16 Part[kTile][XKP];
  Part *Ap = reinterpret_cast<Part *>(smem);         // Ap[part][row][k]
  Part *Bp = Ap + 3;                                 // Bp[part][col][k]
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  const int rr = tid & (kTile - 1), kh = (tid >> 7) * 16;  // row / column, k half
  float ra[16], rb[16];
  auto load = [&](int k0) {
    if (TA) {
#pragma unroll
      for (int e = 0; e < 16; ++e) ra[e] = gp(A)[(size_t)(k0 + kh + e) * lda + rr];
    } else {
      ld16n<16>(A + (size_t)rr * lda + k0 + kh, ra);
    }
    if (TB) {
      ld16n<16>(B + (size_t)rr * ldb + k0 + kh, rb);
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) rb[e] = gp(B)[(size_t)(k0 + kh + e) * ldb + rr];
    }
    if (bscale) {
#pragma unroll
      for (int e = 0; e < 16; ++e) rb[e] *= (float)gp(bscale)[k0 + kh + e];
    }
  };
  auto store = [&](Part *P, const float (&x)[16], bool neg) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = neg ? -x[8 * hh + e] : x[8 * hh + e];
      Split3 sp;
      split8(v, sp);
      *reinterpret_cast<bf16x8 *>(&P[0][rr][kh + 8 * hh]) = sp.h;
      *reinterpret_cast<bf16x8 *>(&P[1][rr][kh + 8 * hh]) = sp.m;
      *reinterpret_cast<bf16x8 *>(&P[2][rr][kh + 8 * hh]) = sp.l;
    }
  };
  load(0);
  const int g = lane >> 4, c = lane & 15;
  for (int k0 = 0; k0 < K; k0 += XK) {
    __syncthreads();
    store(Ap, ra, NEG_A);
    store(Bp, rb, false);
    __syncthreads();
    if (k0 + XK < K) load(k0 + XK);
    // lane l holds row / column l % 16 of its tile and k = 8 (l / 16) + 0..7
    Split3 bs[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = wn + j * 16 + c;
      bs[j].h = *reinterpret_cast<const bf16x8 *>(&Bp[0][col][8 * g]);
      bs[j].m = *reinterpret_cast<const bf16x8 *>(&Bp[1][col][8 * g]);
      bs[j].l = *reinterpret_cast<const bf16x8 *>(&Bp[2][col][8 * g]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (PART && i >= ni) continue;
      const int row = wm + i * 16 + c;
      Split3 as;
      as.h = *reinterpret_cast<const bf16x8 *>(&Ap[0][row][8 * g]);
      as.m = *reinterpret_cast<const bf16x8 *>(&Ap[1][row][8 * g]);
      as.l = *reinterpret_cast<const bf16x8 *>(&Ap[2][row][8 * g]);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (!PART || j < nj) acc.v[i][j] = mfma_x6(as, bs[j], acc.v[i][j]);
    }
  }
}

// acc += (NEG_A ? -A : A)[0:128, 0:K] * diag(bscale[0:K]) * B[0:K, 0:128]
// A row-major with leading dim lda (points at the tile's first row),
// B row-major with leading dim ldb (points at the tile's first column).
// TA: the operand is the transpose of a row-major matrix G, A[i][k] =
// G[k][i]; A then points at G's column of the tile's first row.
// TB: the right operand is the transpose of a row-major matrix H,
// B[k][j] = H[j][k]; B then points at H's row of the tile's first column.
// rows, cols: how many of the tile's rows and columns are wanted; 16 x 16
// tiles past them are skipped and stay as they are (products over the padding
// of ragged matrices, see k_gemm).  FP32 operands go to mma_tile_x6 (BF16
// matrix cores, K a multiple of 32), FP64 ones to the FP64 matrix cores (of 8).
template <typename T, bool NEG_A, bool TA, bool TB, bool PART>
__device__ __forceinline__ void mma_part(const T *__restrict__ A, int lda,
                                         const T *__restrict__ B, int ldb,
                                         const double *__restrict__ bscale, int K,
                                         T (*As)[LW], Tile<T> &acc, int rows,
                                         int cols) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  const int ni = __builtin_amdgcn_readfirstlane(min(4, max(0, (rows - wm + 15) / 16)));
  const int nj = __builtin_amdgcn_readfirstlane(min(4, max(0, (cols - wn + 15) / 16)));
  if constexpr (std::is_same<T, float>::value) {
    // As is the start of an MmaLds<float>::bytes buffer
    mma_tile_x6<NEG_A, TA, TB, PART>(A, lda, B, ldb, bscale, K,
                                 reinterpret_cast<unsigned char *>(As), acc, ni, nj);
    return;
  }
  // An operand stage of BK k.  Rows of k (A, TB): 128 rows, two threads each;
  // rows of columns (B, TA): BK rows, 256 / BK threads each.
  constexpr int NS = BK / 2;
  const int ar = tid >> 1, ak = (tid & 1) * NS;
  const int br = tid / (256 / BK), bc = tid % (256 / BK) * NS;
  T ra[NS], rb[NS];
  auto load = [&](int k0) {
    if (TA)
      ld16n<NS>(A + (size_t)(k0 + br) * lda + bc, ra);
    else
      ld16n<NS>(A + (size_t)ar * lda + k0 + ak, ra);
    if (TB) {
      ld16n<NS>(B + (size_t)ar * ldb + k0 + ak, rb);
    } else {
      ld16n<NS>(B + (size_t)(k0 + br) * ldb + bc, rb);
      if (bscale) {
        const T s = (T)gp(bscale)[k0 + br];
#pragma unroll
        for (int q = 0; q < NS; ++q) rb[q] *= s;
      }
    }
  };
  auto store = [&](int buf) {
    T (*Ad)[LW] = As + buf * 2 * BK, (*Bd)[LW] = Ad + BK;
#pragma unroll
    for (int q = 0; q < NS; ++q)
      (TA ? Ad[br][bc + q] : Ad[ak + q][ar]) = NEG_A ? -ra[q] : ra[q];
#pragma unroll
    for (int q = 0; q < NS; ++q) (TB ? Bd[ak + q][ar] : Bd[br][bc + q]) = rb[q];
  };
  load(0);
  store(0);
  if (BK < K) load(BK);
  __syncthreads();
  for (int k0 = 0; k0 < K; k0 += BK) {
    const int buf = (k0 / BK) & 1;
    if (k0 + BK < K) {
      store(buf ^ 1);
      if (k0 + 2 * BK < K) load(k0 + 2 * BK);
    }
    const T (*Ac)[LW] = As + buf * 2 * BK, (*Bc)[LW] = Ac + BK;
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      T a[4], b[4];
      const int kr = kk + (lane >> 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = Ac[kr][wm + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bc[kr][wn + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (!PART || (i < ni && j < nj)) acc.v[i][j] = mfma16(a[i], b[j], acc.v[i][j]);
    }
    __syncthreads();
  }
}
template <typename T, bool NEG_A = false, bool TA = false, bool TB = false>
__device__ __forceinline__ void mma_tile(const T *__restrict__ A, int lda,
                                         const T *__restrict__ B, int ldb,
                                         const double *__restrict__ bscale, int K,
                                         T (*As)[LW], Tile<T> &acc,
                                         int rows = kTile, int cols = kTile) {
  // a loop of its own, for the whole work-group: tests between the products
  // cost full tiles a tenth of their rate
  if (rows > kTile - 16 && cols > kTile - 16)
    mma_part<T, NEG_A, TA, TB, false>(A, lda, B, ldb, bscale, K, As, acc, rows, cols);
  else
    mma_part<T, NEG_A, TA, TB, true>(A, lda, B, ldb, bscale, K, As, acc, rows, cols);
}

// Rows, columns or k of a 128-wide tile from i0 that are not padding, and the
// depth of a product over k of them.
__device__ __forceinline__ int part_of_tile(int M, int i0) { return max(0, min(kTile, M - i0)); }
__device__ __forceinline__ int depth_of(int k) { return max(32, (k + 31) & ~31); }

// Row / column of accumulator element (i, j, r) inside the 128 x 128 tile.
// Lane l holds column l % 16 of each 16 x 16 MFMA output; the row of
// register r is 4*(l/16) + r for the FP32 instruction and 4*r + l/16 for
// the FP64 one (measured on gfx950 with identity operands).
template <typename T>
__device__ __forceinline__ int acc_row(int i, int r) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int in16 = sizeof(T) == 4 ? 4 * (lane >> 4) + r : 4 * r + (lane >> 4);
  return (wave >> 1) * 64 + i * 16 + in16;
}
__device__ __forceinline__ int acc_col(int j) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  return (wave & 1) * 64 + j * 16 + (lane & 15);
}

// C = alpha diag(cscale) A diag(bscale) B + beta C (TB: A B^T), 128 x 128 tiles.
// Matrix-core bound.  Only the first M rows, columns and k are multiplied:
// what lies past them is padding, whose products are zero (M = 899 in
// ld = 1024: 0.71 of the multiply-adds).
template <typename T, bool TB>
__global__ __launch_bounds__(256, 2) void k_gemm(const GemmJob *__restrict__ jobs, int ld, int M,
                                                 T alpha, T beta) {
  __shared__ __align__(16) unsigned char smem[MmaLds<T>::bytes];
  T (*As)[LW] = reinterpret_cast<T (*)[LW]>(smem);
  const int nt = ld / kTile;
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int b = lin / (nt * nt), t = lin % (nt * nt);
  const int bm = (t / nt) * kTile, bn = (t % nt) * kTile;
  const GemmJob J = jobs[b];
  const T *A = static_cast<const T *>(J.A);
  const T *B = static_cast<const T *>(J.B);
  auto *C = gp(static_cast<T *>(J.C));
  Tile<T> acc;
  acc.zero();
  mma_tile<T, false, false, TB>(A + (size_t)bm * ld, ld, TB ? B + (size_t)bn * ld : B + bn, ld,
                                J.bscale, depth_of(min(ld, M)), As, acc, M - bm, M - bn);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = bm + acc_row<T>(i, r);
      const T f = J.cscale ? alpha * (T)gp(J.cscale)[row] : alpha;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const size_t idx = (size_t)row * ld + bn + acc_col(j);
        T v = f * acc.v[i][j][r];
        if (beta != T(0)) v += beta * C[idx];
        C[idx] = v;
      }
    }
}

// The same for FP32 with 256 x 256 tiles (tiles.h), without bscale and beta.
template <bool TB>
__global__ __launch_bounds__(512, 2) void k_gemm_big(const GemmJob *__restrict__ jobs, int ld,
                                                     int M, float alpha) {
  using W = WgTile<2>;
  __shared__ __align__(16) unsigned char smem[W::lds];
  const int nt = (ld + W::TM - 1) / W::TM;
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int b = lin / (nt * nt), t = lin % (nt * nt);
  const int bm = (t / nt) * W::TM, bn = (t % nt) * W::TN;
  const GemmJob J = jobs[b];
  const float *B = static_cast<const float *>(J.B);
  W w;
  w.product(Opnd{static_cast<const float *>(J.A) + (size_t)bm * ld, ld, ld - bm, true},
            Opnd{TB ? B + (size_t)bn * ld : B + bn, ld, ld - bn, TB}, min(ld, (M + 15) & ~15),
            M - bm, M - bn, smem);
  w.put_to(static_cast<float *>(J.C) + (size_t)bm * ld + bn, ld, alpha,
           J.cscale ? J.cscale + bm : nullptr, ld - bm, ld - bn);
}

// Broadcast lane src (wave-uniform) of a double to the whole wavefront.
__device__ __forceinline__ double bcast_lane(double x, int src) {
  const long long u = __double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)u, src);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(u >> 32), src);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Broadcast lane k (a compile-time constant after unrolling) of each
// 16-lane row to the whole row: DPP row_newbcast (gfx90a and later).
__device__ __forceinline__ int dpp_row_bcast(int x, int k) {
  switch (k) {
#define DDST_BC(K) \
  case K: return __builtin_amdgcn_mov_dpp(x, 0x150 + K, 0xF, 0xF, false);
    DDST_BC(0) DDST_BC(1) DDST_BC(2) DDST_BC(3) DDST_BC(4) DDST_BC(5) DDST_BC(6) DDST_BC(7)
    DDST_BC(8) DDST_BC(9) DDST_BC(10) DDST_BC(11) DDST_BC(12) DDST_BC(13) DDST_BC(14)
    DDST_BC(15)
#undef DDST_BC
  }
  return 0;
}
__device__ __forceinline__ double row_bcast(double x, int k) {
  const long long u = __double_as_longlong(x);
  const unsigned lo = (unsigned)dpp_row_bcast((int)u, k);
  const unsigned hi = (unsigned)dpp_row_bcast((int)(u >> 32), k);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// In-place Gauss-Jordan inversion, without pivoting, of a 16 x 16 FP64 block
// held by one wavefront: lane l holds row l % 16, columns l / 16 + 4c in
// v[c].  That is the A-operand layout of four chained 16x16x4 FP64 MFMAs
// (v[c] feeds k = 4c + l / 16), so the inverse multiplies without a
// reshuffle.  Returns false if a pivot is not finite, or not positive
// unless ANY_SIGN (indefinite, nonsingular blocks).
template <bool ANY_SIGN>
__device__ __forceinline__ bool leaf_invert16(double (&v)[4]) {
  const int l = threadIdx.x & 63;
  const int i = l & 15, g = l >> 4;
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int kg = k & 3, kc = k >> 2;  // column k: lanes with g == kg, v[kc]
    const double piv = bcast_lane(v[kc], kg * 16 + k);
    const double colk = __shfl(v[kc], kg * 16 + i);  // P[i][k]
    ok = ok && isfinite(piv) && (ANY_SIGN ? piv != 0.0 : piv > 0.0);
    // 1 / piv to about an ulp (the bits of an IEEE division cost the chain
    // of 128 eliminations a third of its length)
    double inv = __builtin_amdgcn_rcp(piv);
    inv = fma(fma(-piv, inv, 1.0), inv, inv);
    inv = fma(fma(-piv, inv, 1.0), inv, inv);
    // column k becomes the unit vector: the pivot row then gives 1 / piv and
    // the other rows -P[i][k] / piv there
    if (g == kg) v[kc] = i == k ? 1.0 : 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double rk = row_bcast(v[c], k) * inv;  // new pivot row
      v[c] = i == k ? rk : fma(-colk, rk, v[c]);
    }
  }
  return ok;
}

// One Gauss-Jordan step, pivot part: one work-group (5 wavefronts) per
// matrix inverts the kNB x kNB (128 x 128) pivot block P = D[p, p] in FP64,
// without pivoting, and writes P^{-1} (row-major, rounded to T) to Pinv[b],
// the operand of the panel product.  FP64 throughout: the transfer blocks
// inherit the error of these inverses amplified by the conditioning of the
// interface Schur block.
//
// The block stays in the registers of wavefronts 0..3 for the whole
// inversion, as 16 x 16 tiles in the FP64 MFMA output layout: wave w owns
// column tiles 2w and 2w + 1 of all eight row tiles.  It is inverted by
// blocked Gauss-Jordan with 16-wide leaves.  Sub-step q: the row block q and
// the column block q are in LDS (double-buffered), the inverted leaf
// P_qq^{-1} too; the four wavefronts form R_J = P_qq^{-1} P_qJ for their
// column tiles and apply the rank-16 update on the matrix cores, with the
// tiles as accumulators:
//   row tile q:        T_qJ = R_J                   (R_q = P_qq^{-1})
//   column tile q:     T_Iq = -P_Iq P_qq^{-1}       (formed from zero)
//   others:            T_IJ = T_IJ - P_Iq R_J
// The MFMA output layout of R_J (row 4r + l / 16 in register r) is the
// B-operand layout of the update's k-step r, and the leaf layout is the
// A-operand layout, so no data moves between the two.  The sub-step loop is
// unrolled so that every tile index is static, and no vector ALU operation
// touches a tile.
//
// What bounds it: a serial chain of 128 eliminations, and 64 FP64 MFMAs of 64
// cycles per sub-step and wavefront (33 k cycles in all).  The next leaf is
// therefore updated first and inverted by wavefront 4 beside the other
// tiles' MFMAs, so that a sub-step takes the longer of the two instead of
// their sum (63 matrices: 38 us; with each of four wavefronts inverting the
// leaf itself, between two rounds of MFMAs, 51, of which the leaves were 32;
// with three wavefronts of tiles and the leaf on a SIMD of its own, 38).
// With Rprev and Cprev (the previous step's panels), that step's update of
// the block is applied first.
// WPE: wavefronts per SIMD to fit.  Its 181 registers (FP32) leave room for one
// work-group on a CU; with WPE 3 (168, one of them spilled) and exactly half of
// the LDS two fit, for launches of more matrices than CUs: a build of 319
// matrices of 639 rows without transfer blocks takes 10.2 ms with one on a CU
// (246 us a pivot launch, in two rounds), 9.7 with two.
constexpr int kLeaf = 16;
constexpr int kCqS = 20;        // LDS row stride of the column block (doubles)
constexpr int kRqS = kNB + 16;  // LDS row stride of the row block (doubles)
static_assert(kNB == 128, "the register layout below assumes 128-wide pivots");

template <typename T, bool ANY_SIGN, int WPE>
__global__ __launch_bounds__(320, WPE) void k_gj_pivot(void *const *__restrict__ mats,
                                                     T *__restrict__ Pinv,
                                                     const T *__restrict__ Rprev,
                                                     const T *__restrict__ Cprev, int ld, int o,
                                                     int lw, int p, int M,
                                                     int *__restrict__ flag) {
  constexpr int kCqN = 2 * kNB * kCqS, kRqN = 2 * kLeaf * kRqS;
  constexpr int KS = sizeof(T) == 4 ? 32 : 16;  // operand slices of the previous update
  __shared__ __align__(16) double lds[kCqN + kRqN];
  double (*Cq)[kNB][kCqS] = reinterpret_cast<double (*)[kNB][kCqS]>(lds);
  double (*Rq)[kLeaf][kRqS] = reinterpret_cast<double (*)[kLeaf][kRqS]>(lds + kCqN);
  __shared__ double Lt[kLeaf][kLeaf];  // the next leaf, entry (i, j) at [i][i ^ j]
  __shared__ double Lv[4][64];             // the inverted leaf, in leaf_invert16's layout
  const int b = blockIdx.x, l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lr = l >> 4, lc = l & 15;
  constexpr int NQ = kNB / kLeaf;
  if (w == 4) {
    if (Rprev)
      for (int i = 0; i < 2 * (kNB / KS) + 1; ++i) __syncthreads();  // those of the product
    bool ok = true;
    for (int q = 0; q < NQ; ++q) {
      __syncthreads();  // the leaf q is in Lt
      double v[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = Lt[lc][lc ^ (lr + 4 * c)];
      ok = leaf_invert16<ANY_SIGN>(v) && ok;
#pragma unroll
      for (int c = 0; c < 4; ++c) Lv[c][l] = v[c];
      __syncthreads();  // row block q, column block q and the inverted leaf are in LDS
    }
    if (!ok && l == 0) atomicOr(flag, 1);
    return;
  }
  const int g0 = o + p * kNB;  // the block's row and column in the matrix
  const auto *D = gp(static_cast<const T *>(mats[b]) + (size_t)g0 * ld + g0);
  f64x4 t[8][2];  // t[I][jj][r] = P[16 I + 4 r + lr][16 (2 w + jj) + lc]
  auto load_block = [&]() {
#pragma unroll
    for (int I = 0; I < 8; ++I)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          t[I][jj][r] = (double)D[(size_t)(16 * I + 4 * r + lr) * ld + 16 * (2 * w + jj) + lc];
  };
  if (Rprev) {
    // The previous step's update of this block, P = D - Cprev[p] Rprev[:, p].
    // FP32: the arithmetic of the update kernel (products accumulated over k
    // in order from zero, subtracted once in FP32), so the block equals what
    // that kernel would have written; the A rows are fed permuted (row
    // 4 (i % 4) + i / 4 at position i) so that the accumulators come out in
    // the FP64 layout of t.  FP64: accumulated into the block itself (a
    // second set of FP64 accumulators would not fit next to it).  Operands
    // are staged through LDS in KS-deep slices.
    static_assert(2 * KS * LW * sizeof(T) <= sizeof(lds), "operand slices fit the LDS");
    static_assert(sizeof(lds) + sizeof(Lt) + sizeof(Lv) <= 80 * 1024, "two work-groups a CU");
    T (*As)[LW] = reinterpret_cast<T (*)[LW]>(lds);
    T (*Bs)[LW] = reinterpret_cast<T (*)[LW]>(reinterpret_cast<T *>(lds) + KS * LW);
    const T *A = Cprev + ((size_t)b * lw + p * kNB) * kNB;  // rows p, kNB wide
    const T *B = Rprev + (size_t)b * kNB * lw + p * kNB;  // kNB rows, cols p
    const int tid = threadIdx.x;
    constexpr int AE = kNB * KS / 256;  // A elements per thread (128 rows x KS)
    constexpr int BE = KS * kNB / 256;  // B elements per thread (KS rows x 128)
    const int ar = tid / (KS / AE), ak = (tid % (KS / AE)) * AE;
    const int bk = tid / (kNB / BE), bc = (tid % (kNB / BE)) * BE;
    const int arow = sizeof(T) == 4 ? 4 * (lc & 3) + (lc >> 2) : lc;
    auto product = [&](auto &C, T sign) {
      for (int k0 = 0; k0 < kNB; k0 += KS) {
        T ra[AE], rb[BE];
        ld16n<AE>(A + (size_t)ar * kNB + k0 + ak, ra);
        ld16n<BE>(B + (size_t)(k0 + bk) * lw + bc, rb);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < AE; ++e) As[ak + e][ar] = sign * ra[e];
#pragma unroll
        for (int e = 0; e < BE; ++e) Bs[bk][bc + e] = rb[e];
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < KS; kk += 4) {
          T bv[2];
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) bv[jj] = Bs[kk + lr][16 * (2 * w + jj) + lc];
#pragma unroll
          for (int I = 0; I < 8; ++I) {
            const T av = As[kk + lr][16 * I + arow];
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) C[I][jj] = mfma16(av, bv[jj], C[I][jj]);
          }
        }
      }
      __syncthreads();  // the slices alias the blocks used below
    };
    if constexpr (sizeof(T) == 4) {
      f32x4 acc[8][2];
#pragma unroll
      for (int I = 0; I < 8; ++I)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[I][jj][r] = 0.f;
      product(acc, 1.f);
#pragma unroll
      for (int I = 0; I < 8; ++I)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float d = D[(size_t)(16 * I + 4 * r + lr) * ld + 16 * (2 * w + jj) + lc];
            t[I][jj][r] = (double)(d - acc[I][jj][r]);
          }
    } else {
      load_block();
      product(t, -1.0);
    }
  } else {
    load_block();
  }
  auto put_leaf = [&](const f64x4 &x) {
#pragma unroll
    for (int r = 0; r < 4; ++r) Lt[4 * r + lr][(4 * r + lr) ^ lc] = x[r];
  };
  // row block q and column block q (its owner holds it as jj = q & 1) to LDS
  auto put_blocks = [&](int q) {
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int r = 0; r < 4; ++r) Rq[q & 1][4 * r + lr][16 * (2 * w + jj) + lc] = t[q][jj][r];
    if (w == (q >> 1)) {
#pragma unroll
      for (int I = 0; I < 8; ++I)
#pragma unroll
        for (int r = 0; r < 4; ++r) Cq[q & 1][16 * I + 4 * r + lr][lc] = t[I][q & 1][r];
    }
  };
  if (w == 0) put_leaf(t[0][0]);
  __syncthreads();
  put_blocks(0);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int buf = q & 1, qj = q & 1;
    const bool owner = w == (q >> 1);  // this wave holds column tile q (as jj = qj)
    double v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = Lv[c][l];
    f64x4 R[2];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      const bool pc = owner && jj == qj;
#pragma unroll
      for (int r = 0; r < 4; ++r) R[jj][r] = 0.0;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const double id = 4 * s + lr == lc ? 1.0 : 0.0;
        const double bs = pc ? id : Rq[buf][4 * s + lr][16 * (2 * w + jj) + lc];
        R[jj] = mfma16(v[s], bs, R[jj]);
      }
    }
    auto update = [&](int I) {
      double a[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) a[s] = -Cq[buf][16 * I + lc][4 * s + lr];
#pragma unroll
      for (int s = 0; s < 4; ++s) t[I][1 - qj] = mfma16(a[s], R[1 - qj][s], t[I][1 - qj]);
      if (owner) {  // pivot-column tile, formed from zero
        f64x4 z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) z = mfma16(a[s], R[qj][s], z);
        t[I][qj] = z;
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) t[I][qj] = mfma16(a[s], R[qj][s], t[I][qj]);
      }
    };
    if (q + 1 < NQ) {  // the next leaf first
      update(q + 1);
      if (w == ((q + 1) >> 1)) put_leaf(t[q + 1][(q + 1) & 1]);
      __syncthreads();
    }
#pragma unroll
    for (int I = 0; I < 8; ++I)
      if (I != q && I != q + 1) update(I);
    t[q][0] = R[0];
    t[q][1] = R[1];
    if (q + 1 < NQ) {
      put_blocks(q + 1);
      __syncthreads();
    }
  }
  T *out = Pinv + (size_t)b * kNB * kNB;
  // largest |entry| of the inverse outside the identity padding (rows and
  // columns >= M), for the pivot growth
  double amax = 0.0;
  const int lim = M - g0;  // local rows / columns below M
#pragma unroll
  for (int I = 0; I < 8; ++I)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        put<T>(out + (16 * I + 4 * r) * kNB + 16 * jj,
               (unsigned)sizeof(T) * (lr * kNB + 32 * w + lc), (T)t[I][jj][r]);
#pragma unroll
  for (int I = 0; I < 8; ++I)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
      if (16 * (2 * w + jj) + lc < lim)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (lim >= kNB || 16 * I + 4 * r + lr < lim) amax = fmax(amax, fabs(t[I][jj][r]));
  for (int off = 32; off > 0; off >>= 1) amax = fmax(amax, __shfl_xor(amax, off));
  if (l == 0)
    atomicMax(reinterpret_cast<unsigned long long *>(flag) + 1,
              (unsigned long long)__double_as_longlong(amax));
}

// One Gauss-Jordan step, panel part (o: row and column where the block being
// inverted begins, lw its width, M its rows that are not padding; here and
// below products over the padding are left out).  Work-group (jt, b), 4
// wavefronts, for the 128 columns j0 = 128 jt:
//  * R[:, j0..j0+127] = P^{-1} D[p, j0..j0+127], a 128 x 128 x 128 product
//    on the matrix cores through the LDS-staged tile routine (R = P^{-1}
//    itself on the pivot block);
//  * Cbuf[j0..j0+127, :] = D[j0..j0+127, p] (copy of the old pivot columns)
//    when copy_c is set; after the first step the update that produced
//    column block p writes this copy itself.
template <typename T>
__global__ __launch_bounds__(256, 2) void k_gj_panel(void *const *__restrict__ mats,
                                                  const T *__restrict__ Pinv,
                                                  T *__restrict__ Rbuf, T *__restrict__ Cbuf,
                                                  int ld, int o, int lw, int M, int p,
                                                  int copy_c) {
  __shared__ __align__(16) unsigned char smem[MmaLds<T>::bytes];
  T (*As)[LW] = reinterpret_cast<T (*)[LW]>(smem);
  const int b = blockIdx.y, jt = blockIdx.x, tid = threadIdx.x;
  const T *D = static_cast<const T *>(mats[b]) + (size_t)o * ld + o;
  T *R = Rbuf + (size_t)b * kNB * lw;
  T *Cb = Cbuf + (size_t)b * lw * kNB;
  const T *Pi = Pinv + (size_t)b * kNB * kNB;
  const int p0 = p * kNB, j0 = jt * kTile;
  constexpr int V = 16 / sizeof(T);  // elements per 16-byte access
  for (int e = tid * V; copy_c && e < kTile * kNB; e += 256 * V) {
    const int r = e / kNB, c = e % kNB;
    st16(Cb + (size_t)(j0 + r) * kNB + c, ld16(D + (size_t)(j0 + r) * ld + p0 + c));
  }
  if (jt == p) {
    for (int e = tid * V; e < kNB * kTile; e += 256 * V) {
      const int r = e / kTile, c = e % kTile;
      st16(R + (size_t)r * lw + j0 + c, ld16(Pi + r * kNB + c));
    }
    return;
  }
  Tile<T> acc;
  acc.zero();
  const int rows = part_of_tile(M, p0);
  mma_tile<T>(Pi, kNB, D + (size_t)p0 * ld + j0, ld, nullptr, depth_of(rows), As, acc, rows,
              part_of_tile(M, j0));
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        R[(size_t)acc_row<T>(i, r) * lw + j0 + acc_col(j)] = acc.v[i][j][r];
}

// (i, j) of the t-th tile of a lower triangle of tiles, in row order
__device__ __forceinline__ void tri_index(int t, int &i, int &j) {
  int r = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while (r > 0 && r * (r + 1) / 2 > t) --r;
  while ((r + 1) * (r + 2) / 2 <= t) ++r;
  i = r;
  j = t - r * (r + 1) / 2;
}

// Transposed copy of a 128 x 128 tile through LDS, 32 source rows at a
// time: dst[r][c] = sg * src[c][r] (src row-major with leading dim lds_,
// dst with leading dim ldd).  X: 32 x (kTile + 1) elements of LDS.
template <typename T>
__device__ __forceinline__ void tile_transpose(const T *__restrict__ src, int lds_,
                                               T *__restrict__ dst, int ldd, T sg,
                                               T (*X)[kTile + 1]) {
  const int tid = threadIdx.x;
  for (int c0 = 0; c0 < kTile; c0 += 32) {
    __syncthreads();
    for (int e = tid; e < 32 * kTile; e += 256) {
      const int rr = e / kTile, cc = e % kTile;
      X[rr][cc] = gp(src)[(size_t)(c0 + rr) * lds_ + cc];
    }
    __syncthreads();
    for (int e = tid; e < kTile * 32; e += 256) {
      const int r = e / 32, cc = e % 32;
      gp(dst)[(size_t)r * ldd + c0 + cc] = sg * X[cc][r];
    }
  }
  __syncthreads();
}

// One step of the symmetric elimination, panel part (the general update's
// layout; see k_gj_update).  Work-group (it, b) takes row block i = it:
//  * i == p: Rbuf[:, p] = P^{-1};
//  * otherwise C_i = D[i, p] (i > p) or -D[p, i]^T (i < p), read from the
//    lower triangle, is copied to Cbuf rows i (the operand of the update,
//    which overwrites column and row block p), and W_i = C_i P^{-1} is
//    formed on the matrix cores and written transposed to Rbuf[:, i].
template <typename T>
__global__ __launch_bounds__(256, 2) void k_gj_panel_sym(void *const *__restrict__ mats,
                                                      const T *__restrict__ Pinv,
                                                      T *__restrict__ Rbuf, T *__restrict__ Cbuf,
                                                      int ld, int o, int lw, int M, int p) {
  __shared__ __align__(16) unsigned char smem[MmaLds<T>::bytes];
  static_assert(32 * (kTile + 1) * sizeof(T) <= MmaLds<T>::bytes, "transpose chunk fits");
  T (*As)[LW] = reinterpret_cast<T (*)[LW]>(smem);
  const int b = blockIdx.y, it = blockIdx.x, tid = threadIdx.x;
  const T *D = static_cast<const T *>(mats[b]) + (size_t)o * ld + o;
  T *R = Rbuf + (size_t)b * kNB * lw;
  T *Cb = Cbuf + (size_t)b * lw * kNB;
  const T *Pi = Pinv + (size_t)b * kNB * kNB;
  const int p0 = p * kNB, i0 = it * kTile;
  constexpr int V = 16 / sizeof(T);
  if (it == p) {
    for (int e = tid * V; e < kNB * kTile; e += 256 * V) {
      const int r = e / kTile, c = e % kTile;
      st16(R + (size_t)r * lw + p0 + c, ld16(Pi + r * kNB + c));
    }
    return;
  }
  Tile<T> acc;
  acc.zero();
  const int cols = part_of_tile(M, p0), rows = part_of_tile(M, i0), K = depth_of(cols);
  if (it > p)
    mma_tile<T>(D + (size_t)i0 * ld + p0, ld, Pi, kNB, nullptr, K, As, acc, rows, cols);
  else
    mma_tile<T, true, true>(D + (size_t)p0 * ld + i0, ld, Pi, kNB, nullptr, K, As, acc, rows,
                            cols);
  // Rbuf[c][i0 + r] = W_i[r][c]
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        R[(size_t)acc_col(j) * lw + i0 + acc_row<T>(i, r)] = acc.v[i][j][r];
  if (it > p) {
    for (int e = tid * V; e < kTile * kNB; e += 256 * V) {
      const int r = e / kNB, c = e % kNB;
      st16(Cb + (size_t)(i0 + r) * kNB + c, ld16(D + (size_t)(i0 + r) * ld + p0 + c));
    }
  } else {
    __syncthreads();  // the product's LDS is reused
    tile_transpose<T>(D + (size_t)p0 * ld + i0, ld, Cb + (size_t)i0 * kNB, kNB, T(-1),
                      reinterpret_cast<T (*)[kTile + 1]>(smem));
  }
}

// Diagonal tiles made exactly symmetric from their lower triangle, before a
// symmetric elimination: work-group (q, t, b) mirrors the q-th 32 x 32 piece of
// the lower triangle of tile (t, t) of matrix b (one work-group for the whole
// tile, 32 columns after another: 22.7 us for 16 matrices of one tile).
// The elimination reads only lower tiles and assumes symmetry; an input whose
// diagonal tiles carry rounding asymmetry (the previous plane's inverse
// after the Schur update) is then inverted inconsistently, and along a sweep
// of an indefinite problem that error grows geometrically with the planes.
template <typename T>
__global__ __launch_bounds__(256) void k_sym_diag(void *const *__restrict__ mats, int ld) {
  constexpr int P = 32;
  __shared__ T X[P][P + 1];
  T *D = static_cast<T *>(mats[blockIdx.z]) + (size_t)blockIdx.y * kTile * (ld + 1);
  int pi, pj;
  tri_index(blockIdx.x, pi, pj);
  const int c = threadIdx.x % P, r0 = threadIdx.x / P;
#pragma unroll
  for (int r = r0; r < P; r += 256 / P) X[r][c] = gp(D)[(size_t)(pi * P + r) * ld + pj * P + c];
  __syncthreads();
#pragma unroll
  for (int r = r0; r < P; r += 256 / P)
    if (pi > pj || c > r) gp(D)[(size_t)(pj * P + r) * ld + pi * P + c] = X[c][r];
}

// Upper triangle of every matrix from its lower triangle (the inverse left
// by the symmetric elimination is symmetric): work-group (t, b) copies the
// transpose of the t-th tile strictly below the diagonal to its mirror, in
// the block that begins at row and column o.
template <typename T>
__global__ __launch_bounds__(256) void k_mirror_lower(void *const *__restrict__ mats, int ld,
                                                      int o) {
  __shared__ T X[32][kTile + 1];
  T *D = static_cast<T *>(mats[blockIdx.y]) + (size_t)o * ld + o;
  int ti, tj;
  tri_index(blockIdx.x, ti, tj);
  ti += 1;  // strictly lower: the t-th tile of the triangle of nt - 1 rows, shifted
  tile_transpose<T>(D + (size_t)ti * kTile * ld + tj * kTile, ld,
                    D + (size_t)tj * kTile * ld + ti * kTile, ld, T(1), X);
}

// One Gauss-Jordan step, update part (Cbuf = old column p, R = P^{-1} D[p,:]):
//   pivot rows               D[p, :] = R             (P^{-1} on the block p)
//   other rows, column p     D[i, p] = -D[i, p] P^{-1}
//   other rows, other cols   D[i, j] -= D[i, p] P^{-1} D[p, j]
// The 128 x 128 tile of D is read after the product.  FP32: it is read and
// written with 16-byte accesses, each wavefront covering whole rows (VEC
// elements per lane), half a tile at a time, and the MFMA accumulators are
// exchanged into its row layout through LDS (64 rows, the two wavefronts
// holding them write, all four read; the operand stages live in the same
// buffer).  FP64: in the accumulators' own layout, whose 16 lanes cover a
// 128-byte line of a row.  With Cnext, tiles of column block p + 1 are
// also written to the next step's column panel.  The product is formed from
// zero and subtracted once, keeping the rounding at the scale of the update
// rather than of D; the pivot column is written as -acc rather than
// D - (D + D P^{-1}), which would add O(1) to O(|P^{-1}|) entries.
template <typename T> struct UpdGeom;
template <> struct UpdGeom<float> {
  static constexpr int VEC = 4;     // floats per 16-byte access
  static constexpr int RPI = 8;     // rows covered by one pass of 256 threads
  static constexpr int NQ = 16;     // passes per tile (128 / RPI)
};
template <> struct UpdGeom<double> {
  static constexpr int VEC = 2;
  static constexpr int RPI = 4;
  static constexpr int NQ = 32;
};

// Tile subsets of one update (q = p + 1, the next pivot block): all tiles
// (last step); the row and column blocks of q, with the block (q, q) or without
// it; everything outside them.
enum { kSelAll = 0, kSelCross, kSelArms, kSelRest };
__host__ __device__ inline int sel_tiles(int sel, int nt) {
  return sel == kSelAll    ? nt * nt
         : sel == kSelRest ? (nt - 1) * (nt - 1)
                           : 2 * nt - 1 - (sel == kSelArms);
}
__device__ __forceinline__ void sel_tile(int sel, int nt, int q, int t, int &tr, int &tc) {
  if (sel == kSelAll) {
    tr = t / nt;
    tc = t % nt;
  } else if (sel != kSelRest) {  // row block q, column block q, (q, q)
    tr = tc = q;
    if (t < nt - 1)
      tc = t + (t >= q);
    else if (t < 2 * nt - 2)
      tr = t - (nt - 1) + (t - (nt - 1) >= q);
  } else {  // everything outside row and column block q
    tr = t / (nt - 1);
    tc = t % (nt - 1);
    tr += tr >= q;
    tc += tc >= q;
  }
}

// Tile subsets of the symmetric elimination, which updates only the lower
// triangle of tiles (tr >= tc): all of them (last step); row block q up to
// (q, q) and column block q below it; everything outside row and column
// block q.
__host__ __device__ inline int sel_tiles_sym(int sel, int nt) {
  return sel == kSelAll    ? nt * (nt + 1) / 2
         : sel == kSelRest ? (nt - 1) * nt / 2
                           : nt - (sel == kSelArms);
}
__device__ __forceinline__ void sel_tile_sym(int sel, int nt, int q, int t, int &tr, int &tc) {
  if (sel == kSelAll) {
    tri_index(t, tr, tc);
  } else if (sel != kSelRest) {  // (q, 0..q-1), (q+1..nt-1, q), (q, q)
    tr = tc = q;
    if (t < q)
      tc = t;
    else if (t < nt - 1)
      tr = t + 1;
  } else {  // the lower triangle of the nt - 1 blocks other than q
    tri_index(t, tr, tc);
    tr += tr >= q;
    tc += tc >= q;
  }
}

// SYM: the symmetric elimination (a symmetric matrix, Gauss-Jordan without
// pivoting in block order).  After the steps 0..p-1 the matrix is
//   [ A_SS^{-1}              A_SS^{-1} A_SN          ]
//   [ -A_NS A_SS^{-1}        A_NN - A_NS A_SS^{-1} A_SN ]
// (S the eliminated blocks, N the others): its SS and NN parts are
// symmetric and NS = -(SN)^T, so the lower triangle of tiles determines it.
// With C_i the current column block p (C_i = D[i, p] for i > p, -D[p, i]^T
// for i < p) and W_i = C_i P^{-1}, a step is, on lower tiles only:
//   D[i, j] -= s_j C_i W_j^T  (s_j = +1 for j > p, -1 for j < p)
//   D[i, p] = -W_i (i > p),  D[p, j] = -W_j^T (j < p),  D[p, p] = P^{-1}
// Rbuf holds W^T (kNB x ld, W_p^T taken as P^{-1}), so every product is the
// one of the general update, only its sign and the pivot-row copy differ.
template <typename T, bool SYM>
__global__ __launch_bounds__(256, 2) void k_gj_update(void *const *__restrict__ mats,
                                                   const T *__restrict__ Rbuf,
                                                   const T *__restrict__ Cbuf,
                                                   T *__restrict__ Cnext, int ld, int o, int nt,
                                                   int M, int p, int sel) {
  using G = UpdGeom<T>;
  constexpr int XW = kTile + 4;  // exchange row width
  constexpr int HR = kTile / 2;  // rows per exchange half
  // the staging buffers of the product live inside the exchange buffer
  static_assert(HR * XW * (int)sizeof(float) <= MmaLds<float>::bytes);
  __shared__ __align__(16) unsigned char smem[MmaLds<T>::bytes];
  T *lds = reinterpret_cast<T *>(smem);
  T (*As)[LW] = reinterpret_cast<T (*)[LW]>(lds);
  T (*Xs)[XW] = reinterpret_cast<T (*)[XW]>(lds);
  const int lw = nt * kTile;  // width of the block being inverted
  const int tiles_per_mat = SYM ? sel_tiles_sym(sel, nt) : sel_tiles(sel, nt);
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int b = lin / tiles_per_mat;
  int tr, tc;
  if (SYM)
    sel_tile_sym(sel, nt, p + 1, lin % tiles_per_mat, tr, tc);
  else
    sel_tile(sel, nt, p + 1, lin % tiles_per_mat, tr, tc);
  const int bm = tr * kTile, bn = tc * kTile;
  T *D = static_cast<T *>(mats[b]) + (size_t)o * ld + o;
  const T *R = Rbuf + (size_t)b * kNB * lw;
  const T *Cb = Cbuf + (size_t)b * lw * kNB;
  const int p0 = p * kNB;
  const int tid = threadIdx.x;
  constexpr int LPR = kTile / G::VEC;           // lanes per row
  const int trow = tid / LPR, tcol = (tid % LPR) * G::VEC;
  using VT = typename V16<T>::type;
  // tiles of column block p + 1 also go to the next step's column panel
  T *Cn = (!SYM && Cnext && bn == p0 + kNB) ? Cnext + (size_t)b * lw * kNB : nullptr;
  if (bm == p0) {  // pivot rows: D[p, :] = R (SYM: -W^T left of the pivot), no product
    const T sg = (SYM && bn < p0) ? T(-1) : T(1);
#pragma unroll
    for (int q = 0; q < G::NQ; ++q) {
      const int row = bm + q * G::RPI + trow;
      VT v = ld16(R + (size_t)(row - p0) * lw + bn + tcol);
#pragma unroll
      for (int e = 0; e < G::VEC; ++e) v[e] *= sg;
      st16(D + (size_t)row * ld + bn + tcol, v);
      if (Cn) st16(Cn + (size_t)row * kNB + tcol, v);
    }
    return;
  }
  Tile<T> acc;
  acc.zero();
  mma_tile<T>(Cb + (size_t)bm * kNB, kNB, R + bn, lw, nullptr, depth_of(part_of_tile(M, p0)), As,
              acc, part_of_tile(M, bm), part_of_tile(M, bn));
  const bool plus = SYM && bn < p0;  // s_j = -1: the product is added
  if constexpr (sizeof(T) == 8) {
    const double f = plus ? 1.0 : -1.0;
    const unsigned off = 8u * (unsigned)(acc_row<T>(0, 0) * ld + acc_col(0));
    const unsigned cof = 8u * (unsigned)(acc_row<T>(0, 0) * kNB + acc_col(0));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double dv[4][4];
      if (bn == p0) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < 4; ++j) dv[r][j] = 0.0;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            dv[r][j] = at<double>(D + (size_t)(bm + 16 * i + 4 * r) * ld + bn + 16 * j, off);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double v = dv[r][j] + f * acc.v[i][j][r];
          put<double>(D + (size_t)(bm + 16 * i + 4 * r) * ld + bn + 16 * j, off, v);
          if (Cn) put<double>(Cn + (size_t)(bm + 16 * i + 4 * r) * kNB + 16 * j, cof, v);
        }
    }
    return;
  }
  const bool pivcols = (bn + tcol >= p0) && (bn + tcol < p0 + kNB);
  const int wave = tid >> 6;
  constexpr int NH = G::NQ / 2;  // row passes per half
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    VT dv[NH];
#pragma unroll
    for (int q = 0; q < NH; ++q)
      dv[q] = ld16(D + (size_t)(bm + h * HR + q * G::RPI + trow) * ld + bn + tcol);
    __syncthreads();
    if ((wave >> 1) == h) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            Xs[acc_row<T>(i, r) - h * HR][acc_col(j)] = acc.v[i][j][r];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NH; ++q) {
      const int lrow = q * G::RPI + trow;
      VT v;
#pragma unroll
      for (int e = 0; e < G::VEC; ++e)
        v[e] = (pivcols ? T(0) : dv[q][e]) + (plus ? Xs[lrow][tcol + e] : -Xs[lrow][tcol + e]);
      st16(D + (size_t)(bm + h * HR + lrow) * ld + bn + tcol, v);
      if (Cn) st16(Cn + (size_t)(bm + h * HR + lrow) * kNB + tcol, v);
    }
  }
}

// ---- outer elimination: blocks of kOuter = 512 ------------------------------
// Where outer_blocks (rules.h) says so, matrices are eliminated in outer blocks
// P: D[P, P] is inverted by the 128-wide steps above, and the rest of the
// matrix takes one step of rank w <= 512 per outer block:
//   left     D[P, j] = P^{-1} D[P, j]                       (over its operand)
//   update   D[i, j] -= D[i, P] D[P, j]
//   right    D[i, P] = -D[i, P] P^{-1}                      (over its operand)
// Why: an update of rank 128 moves D once for 128 multiply-adds an entry,
// which is 81 us of HBM time a step for 63 matrices of 1023 rows and left the
// matrix cores 21% busy; rank 512 moves it a quarter as often, and the serial
// chain of pivots runs on 512 x 512 blocks alone, beside which the
// remaining products of the previous outer block run on another stream.
// Work-groups of left and right own all the rows, or columns, that they read
// of their operand, so both write over it, with no panel copies.
constexpr int kOuter = 512;
using OuterLeft = WgTile<4>;   // 512 x 128
using OuterRight = WgTile<1>;  // 128 x 512
using OuterUpd = WgTile<2>;    // 256 x 256

// An outer step: n rows eliminated in all (a multiple of 128), M of them not
// padding, P = [p0, p1), the next block Q = [p1, q1).
struct OuterStep {
  int ld, n, M, p0, p1, q1;
  __host__ __device__ int w() const { return p1 - p0; }
  __host__ __device__ int k() const { return ((M < p1 ? M : p1) - p0 + 15) & ~15; }
};
// First row or column of tile t (width tw) outside P; p0 is a multiple of tw.
__host__ __device__ inline int outside_tiles(const OuterStep &s, int tw) {
  return s.p0 / tw + (s.n - s.p1 + tw - 1) / tw;
}
__device__ __forceinline__ int outside_tile(const OuterStep &s, int tw, int t) {
  const int nl = s.p0 / tw;
  return t < nl ? t * tw : s.p1 + (t - nl) * tw;
}

__global__ __launch_bounds__(512, 2) void k_gj_left(void *const *__restrict__ mats, OuterStep s) {
  using W = OuterLeft;
  __shared__ __align__(16) unsigned char smem[W::lds];
  const int tpm = outside_tiles(s, W::TN);
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  float *D = static_cast<float *>(mats[lin / tpm]);
  const int j0 = outside_tile(s, W::TN, lin % tpm);
  float *X = D + (size_t)s.p0 * s.ld + j0;
  const int rows = min(s.w(), s.M - s.p0), cols = s.M - j0;
  W w;
  w.product(Opnd{D + (size_t)s.p0 * s.ld + s.p0, s.ld, s.w(), true},
            Opnd{X, s.ld, s.n - j0, false}, s.k(), rows, cols, smem);
  w.put_to(X, s.ld, 1.f, nullptr, rows, cols);
}

__global__ __launch_bounds__(512, 2) void k_gj_right(void *const *__restrict__ mats, OuterStep s) {
  using W = OuterRight;
  __shared__ __align__(16) unsigned char smem[W::lds];
  const int tpm = outside_tiles(s, W::TM);
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  float *D = static_cast<float *>(mats[lin / tpm]);
  const int i0 = outside_tile(s, W::TM, lin % tpm);
  float *X = D + (size_t)i0 * s.ld + s.p0;
  const int rows = s.M - i0, cols = min(s.w(), s.M - s.p0);
  W w;
  w.product(Opnd{X, s.ld, s.n - i0, true},
            Opnd{D + (size_t)s.p0 * s.ld + s.p0, s.ld, s.w(), false}, s.k(), rows, cols, smem);
  w.put_to(X, s.ld, -1.f, nullptr, rows, cols);
}

// Symmetric elimination (lower tiles only, see k_gj_update): the products with
// P^{-1} are formed once, R_j = P^{-1} C_j^T with C_j the lower-triangle
// column block (D[P, j] left of P, D[j, P]^T below it), into a buffer, since
// the update still reads the old blocks.
__global__ __launch_bounds__(512, 2) void k_gj_left_sym(void *const *__restrict__ mats,
                                                        float *__restrict__ Rbuf, OuterStep s) {
  using W = OuterLeft;
  __shared__ __align__(16) unsigned char smem[W::lds];
  const int tpm = outside_tiles(s, W::TN);
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int b = lin / tpm;
  const float *D = static_cast<const float *>(mats[b]);
  const int j0 = outside_tile(s, W::TN, lin % tpm);
  const int rows = min(s.w(), s.M - s.p0), cols = s.M - j0;
  const Opnd A{D + (size_t)s.p0 * s.ld + s.p0, s.ld, s.w(), true};
  W w;
  if (j0 < s.p0)
    w.product(A, Opnd{D + (size_t)s.p0 * s.ld + j0, s.ld, s.n - j0, false}, s.k(), rows, cols,
              smem);
  else
    w.product(A, Opnd{D + (size_t)j0 * s.ld + s.p0, s.ld, s.n - j0, true}, s.k(), rows, cols,
              smem);
  // whole tiles (the padding's zeros are read by the update)
  w.put_to(Rbuf + (size_t)b * kOuter * s.ld + j0, s.ld, 1.f, nullptr, s.w(), s.n - j0);
}
// ... and go to their places after the update: D[P, j] = R_j left of P,
// D[i, P] = -R_i^T below it.  Work-group (t, b): a 128 x 128 tile.
__global__ __launch_bounds__(256) void k_gj_out_sym(void *const *__restrict__ mats,
                                                    const float *__restrict__ Rbuf, OuterStep s) {
  __shared__ float X[32][kTile + 1];
  const int pr = s.w() / kTile, nl = s.p0 / kTile;
  const int r0 = (blockIdx.x % pr) * kTile, t = blockIdx.x / pr;
  float *D = static_cast<float *>(mats[blockIdx.y]);
  const float *R = Rbuf + (size_t)blockIdx.y * kOuter * s.ld + (size_t)r0 * s.ld;
  if (t < nl) {
    constexpr int V = 4;
    for (int e = threadIdx.x * V; e < kTile * kTile; e += 256 * V) {
      const int r = e / kTile, c = t * kTile + e % kTile;
      st16(D + (size_t)(s.p0 + r0 + r) * s.ld + c, ld16(R + (size_t)r * s.ld + c));
    }
    return;
  }
  const int i0 = s.p1 + (t - nl) * kTile;
  tile_transpose<float>(R + i0, s.ld, D + (size_t)i0 * s.ld + s.p0 + r0, s.ld, -1.f, X);
}

// Tiles of the outer update: those of the next block's diagonal (kOutNext),
// all others (kOutRest), or all (kOutAll, last block), outside row and
// column block P; in the symmetric elimination only tiles with an entry on
// or below the diagonal.  Counts the tiles up to the wanted one, column by
// column; returns their number (`want` < 0: none wanted).
enum { kOutAll = 0, kOutNext = 1, kOutRest = 2 };
__host__ __device__ inline int outer_tiles(const OuterStep &s, int sel, bool sym, int want,
                                           int &i0, int &j0) {
  constexpr int W = OuterUpd::TM;
  static_assert(OuterUpd::TN == W && kOuter % W == 0, "square tiles that fit the blocks");
  const int nt = (s.n + W - 1) / W;
  const int p0 = s.p0 / W, p1 = (s.p1 + W - 1) / W, q1 = (s.q1 + W - 1) / W;
  int count = 0;
  for (int c = sel == kOutNext ? p1 : 0; c < (sel == kOutNext ? q1 : nt); ++c) {
    if (c >= p0 && c < p1) continue;
    // rows [a, e) without [h0, h1)
    int a = sym ? c : 0, e = nt, h0 = p0, h1 = p1;
    if (sel == kOutNext) {
      a = a > p1 ? a : p1;
      e = q1;
    } else if (sel == kOutRest && c >= p1 && c < q1) {
      h1 = q1;  // P and Q are neighbours
    }
    // clip the hole to [a, e)
    h0 = h0 < a ? a : h0 > e ? e : h0;
    h1 = h1 < h0 ? h0 : h1 > e ? e : h1;
    const int m = (e - a) - (h1 - h0);
    if (want >= count && want < count + m) {
      int r = a + (want - count);
      if (r >= h0) r += h1 - h0;
      i0 = r * W;
      j0 = c * W;
    }
    count += m;
  }
  return count;
}

template <bool SYM>
__global__ __launch_bounds__(512, 2) void k_gj_update_outer(void *const *__restrict__ mats,
                                                            const float *__restrict__ Rbuf,
                                                            OuterStep s, int sel, int tpm) {
  using W = OuterUpd;
  __shared__ __align__(16) unsigned char smem[W::lds];
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int b = lin / tpm;
  float *D = static_cast<float *>(mats[b]);
  int i0 = 0, j0 = 0;
  outer_tiles(s, sel, SYM, lin % tpm, i0, j0);
  const Opnd B{SYM ? Rbuf + (size_t)b * kOuter * s.ld + j0 : D + (size_t)s.p0 * s.ld + j0, s.ld,
               s.n - j0, false};
  const int rows = s.M - i0, cols = s.M - j0;
  W w;
  if (SYM && i0 < s.p0)  // left of P: C_i = -D[P, i]^T
    w.product(Opnd{D + (size_t)s.p0 * s.ld + i0, s.ld, s.n - i0, false}, B, s.k(), rows, cols,
              smem);
  else
    w.product(Opnd{D + (size_t)i0 * s.ld + s.p0, s.ld, s.n - i0, true}, B, s.k(), rows, cols,
              smem);
  w.add_to(D + (size_t)i0 * s.ld + j0, s.ld, SYM && i0 < s.p0 ? 1.f : -1.f, rows, cols);
}

// D = A_plane - diag(r1) G1 diag(c1) - diag(r2) G2 diag(c2).  Streams G
// and D once (HBM-bound): work-group (x, b) covers kAsmRows rows of job b,
// each thread V consecutive columns with 16-byte loads and stores; the
// column scales are read once per thread and reused over the rows.
constexpr int kAsmRows = 4;

template <typename T>
__global__ __launch_bounds__(256) void k_assemble(const AsmJob *__restrict__ jobs,
                                                  const double *__restrict__ coef, int n,
                                                  int dim, int M, int ld) {
  constexpr int V = 16 / sizeof(T);
  using VT = typename V16<T>::type;
  const AsmJob J = jobs[blockIdx.y];
  const size_t N = (size_t)M * n;
  const T *G1 = static_cast<const T *>(J.G1);
  const T *G2 = static_cast<const T *>(J.G2);
  for (int c0 = threadIdx.x * V; c0 < ld; c0 += 256 * V) {
    double sc1[V], sc2[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const bool in = c0 + e < M;
      sc1[e] = (G1 && in) ? gp(J.c1)[c0 + e] : 0.0;
      sc2[e] = (G2 && in) ? gp(J.c2)[c0 + e] : 0.0;
    }
#pragma unroll
    for (int rr = 0; rr < kAsmRows; ++rr) {
      const int r = blockIdx.x * kAsmRows + rr;
      T out[V];
      if (r >= M) {
#pragma unroll
        for (int e = 0; e < V; ++e) out[e] = (c0 + e == r) ? T(1) : T(0);
      } else {
        VT g1 = {}, g2 = {};
        if (G1) g1 = ld16(G1 + (size_t)r * ld + c0);
        if (G2) g2 = ld16(G2 + (size_t)r * ld + c0);
        const double s1 = G1 ? gp(J.r1)[r] : 0.0;
        const double s2 = G2 ? gp(J.r2)[r] : 0.0;
        double v[V];
#pragma unroll
        for (int e = 0; e < V; ++e)
          v[e] = c0 + e < M ? -s1 * (double)g1[e] * sc1[e] - s2 * (double)g2[e] * sc2[e] : 0.0;
        // in-plane stencil entries of row r (boundary neighbours are not in A_plane)
        const size_t node = (size_t)(J.plane - 1) * M + r;
        auto add = [&](int col, double val) {
          if (col >= c0 && col < c0 + V) {
#pragma unroll
            for (int e = 0; e < V; ++e)
              if (c0 + e == col) v[e] += val;
          }
        };
        add(r, coef[node]);
        if (dim == 2) {
          if (r >= 1) add(r - 1, coef[3 * N + node]);
          if (r <= n - 2) add(r + 1, coef[4 * N + node]);
        } else {
          const int y = r / n, z = r % n;
          if (y >= 1) add(r - n, coef[3 * N + node]);
          if (y <= n - 2) add(r + n, coef[4 * N + node]);
          if (z >= 1) add(r - 1, coef[5 * N + node]);
          if (z <= n - 2) add(r + 1, coef[6 * N + node]);
        }
#pragma unroll
        for (int e = 0; e < V; ++e) out[e] = (T)v[e];
      }
      VT o;
#pragma unroll
      for (int e = 0; e < V; ++e) o[e] = out[e];
      st16(static_cast<T *>(J.D) + (size_t)r * ld + c0, o);
    }
  }
}

// Products of the sampling chains: C (ld x ldc) = alpha op(A) diag(bscale) B
// with A ld x ld (op(A) = A, or A^T when TRANS), B and C ld x ldc (ldc a
// multiple of 128), all row-major; 128 x 128 output tiles and padding left out
// as in k_gemm.
template <typename T, bool TRANS>
__global__ __launch_bounds__(256, 2) void k_gemm_rect(const GemmJob *__restrict__ jobs, int ld,
                                                      int ldc, int M, int tiles_per_job,
                                                      T alpha) {
  __shared__ __align__(16) unsigned char smem[MmaLds<T>::bytes];
  T (*As)[LW] = reinterpret_cast<T (*)[LW]>(smem);
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int b = lin / tiles_per_job;
  const int t = lin % tiles_per_job;
  const int ntc = ldc / kTile;
  const int bm = (t / ntc) * kTile, bn = (t % ntc) * kTile;
  const GemmJob J = jobs[b];
  const T *A = static_cast<const T *>(J.A);
  const T *B = static_cast<const T *>(J.B);
  auto *C = gp(static_cast<T *>(J.C));
  Tile<T> acc;
  acc.zero();
  mma_tile<T, false, TRANS>(TRANS ? A + bm : A + (size_t)bm * ld, ld, B + bn, ldc, J.bscale,
                            depth_of(min(ld, M)), As, acc, M - bm);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        C[(size_t)(bm + acc_row<T>(i, r)) * ldc + bn + acc_col(j)] = alpha * acc.v[i][j][r];
}

template <typename T>
__global__ __launch_bounds__(256) void k_scale_cols(const GemmJob *__restrict__ jobs, int ld,
                                                    T alpha) {
  const GemmJob J = jobs[blockIdx.y];
  const int r = blockIdx.x;
  const auto *A = gp(static_cast<const T *>(J.A) + (size_t)r * ld);
  auto *C = gp(static_cast<T *>(J.C) + (size_t)r * ld);
  if (J.cscale) alpha *= (T)gp(J.cscale)[r];
  for (int c = threadIdx.x; c < ld; c += blockDim.x)
    C[c] = alpha * A[c] * (T)gp(J.bscale)[c];
}

}  // namespace

template <typename T>
void launch_assemble(const AsmJob *jobs, int njobs, const double *coef, int n, int dim,
                     int M, int ld, hipStream_t s) {
  if (njobs <= 0) return;
  const ProfSpan ps = prof_open(KK_ASSEMBLE);
  hipExtLaunchKernelGGL(k_assemble<T>, dim3(ld / kAsmRows, njobs), dim3(256), 0, s, ps.a, ps.b,
                        0, jobs, coef, n, dim, M, ld);
  // reads G (and up to one more) and writes D: 2 M^2 elements per job
  prof_close(ps, KK_ASSEMBLE, 2.0 * njobs * (double)M * M * sizeof(T));
}

template <typename T>
void launch_scale_cols(const GemmJob *jobs, int njobs, int ld, double alpha, hipStream_t s) {
  if (njobs <= 0) return;
  hipLaunchKernelGGL(k_scale_cols<T>, dim3(ld, njobs), dim3(256), 0, s, jobs, ld, (T)alpha);
}

template <typename T>
void launch_gemm(const GemmJob *jobs, int njobs, int ld, int M, double alpha, bool trans_b,
                 hipStream_t s) {
  if (njobs <= 0) return;
  const int nt = ld / kTile, nbig = (ld + WgTile<2>::TM - 1) / WgTile<2>::TM;
  const ProfSpan ps = prof_open(KK_GEMM);
  const bool big = std::is_same<T, float>::value && gemm_big_tiles(njobs, ld);
  if (big)
    hipExtLaunchKernelGGL((trans_b ? k_gemm_big<true> : k_gemm_big<false>),
                          dim3(nbig * nbig * njobs), dim3(512), 0, s, ps.a, ps.b, 0, jobs, ld, M,
                          (float)alpha);
  else
    hipExtLaunchKernelGGL((trans_b ? k_gemm<T, true> : k_gemm<T, false>), dim3(nt * nt * njobs),
                          dim3(256), 0, s, ps.a, ps.b, 0, jobs, ld, M, (T)alpha, T(0));
  prof_close(ps, KK_GEMM, 2.0 * njobs * (double)M * M * M);
}

template <typename T>
void launch_gemm_full(const GemmJob *jobs, int njobs, int ld, bool bscale, double alpha,
                      double beta, hipStream_t s) {
  if (njobs <= 0) return;
  if (!bscale && beta == 0.0) return launch_gemm<T>(jobs, njobs, ld, ld, alpha, false, s);
  const int nt = ld / kTile;
  const ProfSpan ps = prof_open(KK_GEMM);
  hipExtLaunchKernelGGL((k_gemm<T, false>), dim3(nt * nt * njobs), dim3(256), 0, s, ps.a, ps.b, 0,
                        jobs, ld, ld, (T)alpha, (T)beta);
  prof_close(ps, KK_GEMM, 2.0 * njobs * (double)ld * ld * ld);
}

template <typename T>
void launch_gemm_rect(const GemmJob *jobs, int njobs, int ld, int ldc, int M, int ncols,
                      int trans, double alpha, hipStream_t s) {
  if (njobs <= 0) return;
  const int tpj = (ld / kTile) * (ldc / kTile);
  const ProfSpan ps = prof_open(KK_GEMM);
  hipExtLaunchKernelGGL(trans ? k_gemm_rect<T, true> : k_gemm_rect<T, false>, dim3(tpj * njobs),
                        dim3(256), 0, s, ps.a, ps.b, 0, jobs, ld, ldc, M, tpj, (T)alpha);
  prof_close(ps, KK_GEMM, 2.0 * njobs * (double)M * M * ncols);
}

GjStreams::~GjStreams() {
  for (hipStream_t st : {h, x, o})
    if (st) (void)hipStreamSynchronize(st);
  for (hipEvent_t ev : {panel, arms, upd, left, next, rest})
    if (ev) (void)hipEventDestroy(ev);
  for (hipStream_t st : {h, x, o})
    if (st) (void)hipStreamDestroy(st);
}

// Steps from which the look-ahead schedule pays (below, its events and streams
// cost more than the overlap gives: 361 rows, 3.2 ms against 2.25 in all).
constexpr int kLookAhead = 4;
// Rows that the 128-wide steps invert at a time.
static int block_width(int nmat, int ld, size_t esz, int sym) {
  return outer_blocks(nmat, ld, esz, sym != 0) ? kOuter : ld;
}

// A stream costs more to make (and end) than the elimination of a small block
// takes: only those that the schedule uses.
hipError_t GjStreams::create(int nmat, int ld, int M, size_t esz, int sym) {
  const int n = (M + kTile - 1) / kTile * kTile;
  hipError_t e = hipSuccess;
  auto stream = [&](hipStream_t &st) {
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
  };
  auto events = [&](std::initializer_list<hipEvent_t *> evs) {
    for (hipEvent_t *ev : evs)
      if (e == hipSuccess)
        e = hipEventCreateWithFlags(ev, hipEventDisableTiming | hipEventDisableSystemFence);
  };
  if (n / kTile >= kLookAhead) {
    stream(h);
    stream(x);
    events({&panel, &arms, &upd});
  }
  if (n > block_width(nmat, ld, esz, sym)) {
    stream(o);
    events({&left, &next, &rest});
  }
  return e;
}

size_t gj_workspace_bytes(int nmat, int ld, size_t esz, int sym) {
  const size_t lw = block_width(nmat, ld, esz, sym);
  return (size_t)nmat * esz *
         (4 * (size_t)kNB * lw + (size_t)kNB * kNB +
          (sym && lw != (size_t)ld ? (size_t)kOuter * ld : 0));
}

// Inversion of the nt x nt tiles from row and column o, in steps of 128 (buffers
// of step p: R, Cbuf index p & 1; q = p + 1; Ux(p) = the tiles of row and
// column block q except (q, q), Ur(p) = all tiles outside them):
//   s    : pivot(0) panel(0) | pivot(1) . panel(1) | pivot(2) . panel(2) ...
//   gs.x :                     Ux(0)                 Ux(1)
//   gs.h :                     Ur(0)                 Ur(1) ...
// pivot(q) first applies step p's update to the block (q, q) itself, so the
// next pivot is inverted while the other tiles are updated; Ux(p), which
// the panel of step q needs, runs beside the larger Ur(p) rather than before
// it (behind it on one stream: 188 ms against 180, 1023^2 FP64 on 16 slabs).
// Ux(p) also writes column block q to the column panel of step q.
// Dependencies: Ux(p) and Ur(p) wait for panel(p); Ux(p) and pivot(q) wait
// for Ur(p - 1) (which last wrote their tiles and read the buffers that
// Ux(p) and panel(q) overwrite); panel(q) waits for Ux(p), and with it
// Ur(q).  The last step updates all tiles on s.  Few steps run in order on s.
//
// sym: the matrices are symmetric; the updates touch only the lower
// triangle of tiles (about half the work, see k_gj_update), the panel
// kernel forms C and W^T from it, and one last launch mirrors the lower
// triangle of the (symmetric) inverse into the upper one.  The pivot
// kernel is the same: W_q^T is the block q of its R operand.
template <typename T>
static hipError_t invert_block(void *const *mats, int nmat, int ld, int o, int nt, int M, T *work,
                               int *flag, int any_sign, int sym, GjStreams &gs, hipStream_t s) {
  const int lw = nt * kTile;
  const size_t pan = (size_t)nmat * kNB * lw;
  T *Rb[2] = {work, work + 2 * pan}, *Cb[2] = {work + pan, work + 3 * pan};
  T *PinvT = work + 4 * pan;  // nmat kNB x kNB inverses, rounded to T
  const double m = std::min(lw, M - o);  // rows that are not padding
  const double step_flops = 2.0 * nmat * kNB * m * std::max(m - kNB, 0.0);
  const double mfma_tiles = (double)nt * (nt - 1);  // tiles off the pivot rows
  auto update = [&](int p, int sel, hipStream_t st) {
    const int ntiles = sym ? sel_tiles_sym(sel, nt) : sel_tiles(sel, nt);
    // tiles that take a product (the pivot-row tiles are copies)
    const bool cross = sel != kSelAll && sel != kSelRest;
    const double tiles = sym ? (cross ? ntiles : ntiles - (p + 1.0))
                         : sel == kSelAll ? mfma_tiles
                         : cross          ? ntiles - 1.0
                                          : (nt - 1.0) * (nt - 2);
    T *Cn = (!sym && cross) ? Cb[(p + 1) & 1] : nullptr;
    const ProfSpan ps = prof_open(KK_GJ_UPDATE);
    hipExtLaunchKernelGGL(sym ? k_gj_update<T, true> : k_gj_update<T, false>,
                          dim3(ntiles * nmat), dim3(256), 0, st, ps.a, ps.b, 0, mats,
                          (const T *)Rb[p & 1], (const T *)Cb[p & 1], Cn, ld, o, nt, M - o, p, sel);
    prof_close(ps, KK_GJ_UPDATE, mfma_tiles > 0 ? step_flops * tiles / mfma_tiles : 0.0);
  };
  hipError_t e = hipSuccess;
#define GJCHK(call)                           \
  do {                                        \
    if ((e = (call)) != hipSuccess) return e; \
  } while (0)
  const bool look = nt >= kLookAhead;
  constexpr int DENSE = sizeof(T) == 4 ? 3 : 2;  // FP64 takes 248 registers
  auto *pivot = pivots_share_cus(nmat) ? (any_sign ? k_gj_pivot<T, true, DENSE>
                                                   : k_gj_pivot<T, false, DENSE>)
                                       : (any_sign ? k_gj_pivot<T, true, 2>
                                                   : k_gj_pivot<T, false, 2>);
  for (int p = 0; p < nt; ++p) {
    const bool fused = p > 0 && look;  // the pivot kernel applies step p - 1 to its block
    if (p > 0 && !look) {
      update(p - 1, kSelCross, s);
      update(p - 1, kSelRest, s);
    } else if (p > 0) {
      if (p > 1) GJCHK(hipStreamWaitEvent(s, gs.upd, 0));
      GJCHK(hipEventRecord(gs.panel, s));
      GJCHK(hipStreamWaitEvent(gs.h, gs.panel, 0));
      GJCHK(hipStreamWaitEvent(gs.x, gs.panel, 0));
      if (p > 1) GJCHK(hipStreamWaitEvent(gs.x, gs.upd, 0));
      update(p - 1, kSelArms, gs.x);
      GJCHK(hipEventRecord(gs.arms, gs.x));
      update(p - 1, kSelRest, gs.h);
      GJCHK(hipEventRecord(gs.upd, gs.h));
    }
    ProfSpan ps = prof_open(KK_GJ_PANEL);
    hipExtLaunchKernelGGL(pivot, dim3(nmat), dim3(320), 0, s, ps.a, ps.b, 0, mats, PinvT,
                          fused ? (const T *)Rb[(p - 1) & 1] : nullptr,
                          (const T *)Cb[(p - 1) & 1], ld, o, lw, p, M, flag);
    prof_close(ps, KK_GJ_PANEL, (fused ? 4.0 : 2.0) * nmat * (double)kNB * kNB * kNB);
    if (fused) GJCHK(hipStreamWaitEvent(s, gs.arms, 0));
    ps = prof_open(KK_GJ_PANEL);
    if (sym)
      hipExtLaunchKernelGGL(k_gj_panel_sym<T>, dim3(nt, nmat), dim3(256), 0, s, ps.a, ps.b, 0,
                            mats, (const T *)PinvT, Rb[p & 1], Cb[p & 1], ld, o, lw, M - o, p);
    else
      hipExtLaunchKernelGGL(k_gj_panel<T>, dim3(nt, nmat), dim3(256), 0, s, ps.a, ps.b, 0, mats,
                            (const T *)PinvT, Rb[p & 1], Cb[p & 1], ld, o, lw, M - o, p,
                            p == 0 ? 1 : 0);
    prof_close(ps, KK_GJ_PANEL, 2.0 * nmat * (double)kNB * kNB * std::max(m - kNB, 0.0));
  }
  if (nt > 1 && look) GJCHK(hipStreamWaitEvent(s, gs.upd, 0));
  update(nt - 1, kSelAll, s);
  if (sym && nt > 1)
    hipLaunchKernelGGL(k_mirror_lower<T>, dim3(nt * (nt - 1) / 2, nmat), dim3(256), 0, s, mats, ld,
                       o);
#undef GJCHK
  return hipSuccess;
}

// The outer elimination.  Schedule (Q the block after P):
//   s    : invert(P) left(P) | next(P), invert(Q)    | left(Q) ...
//   gs.o :                   | rest(P), right(P)     |
// next(P) updates D[Q, Q], so that Q is inverted while the other products of P
// run (right(P) waits for next(P), which reads column block P); left(Q) waits
// for them.
static hipError_t invert_outer(void *const *mats, int nmat, int ld, int n, int M, float *w,
                               int *flag, int any_sign, int sym, GjStreams &gs, hipStream_t s) {
  float *R = w + (size_t)nmat * (4 * (size_t)kNB * kOuter + (size_t)kNB * kNB);  // sym only
  hipError_t e = hipSuccess;
#define GJCHK(call)                           \
  do {                                        \
    if ((e = (call)) != hipSuccess) return e; \
  } while (0)
  auto rows = [&](int a, int b) { return (double)std::max(std::min(b, M) - a, 0); };
  for (int p0 = 0; p0 < n; p0 += kOuter) {
    const OuterStep st{ld, n, M, p0, std::min(p0 + kOuter, n), std::min(p0 + 2 * kOuter, n)};
    const bool last = st.p1 == n;
    GJCHK(invert_block<float>(mats, nmat, ld, p0, st.w() / kTile, M, w, flag, any_sign, sym, gs,
                              s));
    if (p0 > 0) GJCHK(hipStreamWaitEvent(s, gs.rest, 0));
    const double kf = 2.0 * nmat * rows(p0, st.p1);
    const double out = (double)M - rows(p0, st.p1);
    const int nleft = outside_tiles(st, OuterLeft::TN);
    ProfSpan ps = prof_open(KK_GJ_UPDATE);
    if (sym)
      hipExtLaunchKernelGGL(k_gj_left_sym, dim3(nleft * nmat), dim3(512), 0, s, ps.a, ps.b, 0,
                            mats, R, st);
    else
      hipExtLaunchKernelGGL(k_gj_left, dim3(nleft * nmat), dim3(512), 0, s, ps.a, ps.b, 0, mats,
                            st);
    prof_close(ps, KK_GJ_UPDATE, kf * rows(p0, st.p1) * out);
    auto update = [&](int sel, hipStream_t q) {
      int i0, j0;
      const int tpm = outer_tiles(st, sel, sym != 0, -1, i0, j0);
      if (tpm <= 0) return;
      const ProfSpan pu = prof_open(KK_GJ_UPDATE);
      hipExtLaunchKernelGGL(sym ? k_gj_update_outer<true> : k_gj_update_outer<false>,
                            dim3(tpm * nmat), dim3(512), 0, q, pu.a, pu.b, 0, mats,
                            (const float *)R, st, sel, tpm);
      const double qn = rows(st.p1, st.q1), nx = sym ? qn * (qn + 1) / 2 : qn * qn;
      const double all = sym ? out * (out + 1) / 2 : out * out;
      prof_close(pu, KK_GJ_UPDATE, kf * (sel == kOutNext ? nx : sel == kOutRest ? all - nx : all));
    };
    auto finish = [&](hipStream_t q) {  // column block P (and row block P if sym)
      if (sym) {
        hipLaunchKernelGGL(k_gj_out_sym, dim3((n - st.w()) / kTile * (st.w() / kTile), nmat),
                           dim3(256), 0, q, mats, (const float *)R, st);
        return;
      }
      const ProfSpan pu = prof_open(KK_GJ_UPDATE);
      hipExtLaunchKernelGGL(k_gj_right, dim3(outside_tiles(st, OuterRight::TM) * nmat), dim3(512),
                            0, q, pu.a, pu.b, 0, mats, st);
      prof_close(pu, KK_GJ_UPDATE, kf * rows(p0, st.p1) * out);
    };
    if (last) {
      update(kOutAll, s);
      finish(s);
    } else {
      GJCHK(hipEventRecord(gs.left, s));
      GJCHK(hipStreamWaitEvent(gs.o, gs.left, 0));
      update(kOutNext, s);
      GJCHK(hipEventRecord(gs.next, s));
      update(kOutRest, gs.o);
      // column block P is overwritten: the update of the next diagonal reads it
      GJCHK(hipStreamWaitEvent(gs.o, gs.next, 0));
      finish(gs.o);
      GJCHK(hipEventRecord(gs.rest, gs.o));
    }
  }
  if (sym) {
    const int nt = n / kTile;
    hipLaunchKernelGGL(k_mirror_lower<float>, dim3(nt * (nt - 1) / 2, nmat), dim3(256), 0, s, mats,
                       ld, 0);
  }
#undef GJCHK
  return hipSuccess;
}

template <typename T>
hipError_t gj_invert(void *const *mats, int nmat, int ld, int M, void *work, int *flag,
                     int any_sign, int sym, GjStreams &gs, hipStream_t s) {
  if (nmat <= 0) return hipSuccess;
  static_assert(kNB == kTile && kOuter % kTile == 0, "one pivot block per tile row");
  T *w = static_cast<T *>(work);
  const int n = (M + kTile - 1) / kTile * kTile;  // blocks of padding alone need no step
  if (sym && n > 0)
    hipLaunchKernelGGL(k_sym_diag<T>, dim3(10, n / kTile, nmat), dim3(256), 0, s, mats, ld);
  hipError_t e;
  if (n <= block_width(nmat, ld, sizeof(T), sym))
    e = invert_block<T>(mats, nmat, ld, 0, n / kTile, M, w, flag, any_sign, sym, gs, s);
  else if constexpr (std::is_same<T, float>::value)
    e = invert_outer(mats, nmat, ld, n, M, w, flag, any_sign, sym, gs, s);
  else
    e = hipErrorInvalidValue;  // not reached: FP64 blocks are as wide as the matrix
  return e == hipSuccess ? hipGetLastError() : e;
}

#define DDST_INST(T)                                                                      \
  template void launch_assemble<T>(const AsmJob *, int, const double *, int, int, int, int, \
                                   hipStream_t);                                           \
  template void launch_scale_cols<T>(const GemmJob *, int, int, double, hipStream_t);       \
  template void launch_gemm<T>(const GemmJob *, int, int, int, double, bool, hipStream_t);    \
  template void launch_gemm_full<T>(const GemmJob *, int, int, bool, double, double,          \
                                    hipStream_t);                                            \
  template void launch_gemm_rect<T>(const GemmJob *, int, int, int, int, int, int, double,     \
                                    hipStream_t);                                              \
  template hipError_t gj_invert<T>(void *const *, int, int, int, void *, int *, int, int,   \
                                   GjStreams &, hipStream_t);
DDST_INST(float)
DDST_INST(double)
#undef DDST_INST

}  // namespace ddst

namespace ddst {
namespace {
template <typename T>
__global__ void k_extract(const T *__restrict__ src, int M, int ld, double *__restrict__ dst) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)M * M) return;
  const size_t r = e / M, c = e % M;
  dst[e] = (double)src[r * ld + c];
}
}  // namespace

void launch_extract_block(const void *src, int prec, int M, int ld, double *dst,
                          hipStream_t s) {
  const size_t len = (size_t)M * M;
  const unsigned nb = (unsigned)((len + 255) / 256);
  if (prec == DDST_FP32)
    hipLaunchKernelGGL(k_extract<float>, dim3(nb), dim3(256), 0, s,
                       static_cast<const float *>(src), M, ld, dst);
  else
    hipLaunchKernelGGL(k_extract<double>, dim3(nb), dim3(256), 0, s,
                       static_cast<const double *>(src), M, ld, dst);
}
}  // namespace ddst

// Memory-bound kernels of libddst: stencil set-up and FP64 residual, batched
// dense matrix-vector products (slab sweeps, interface blocks), interface
// right-hand sides, Krylov helpers and the cellwise gradient.
//
// The stencil follows the FD model problem: on every grid edge the
// coefficient is the mean of the 2^(dim-1) cells sharing the edge,
// convection uses centred differences, and boundary neighbours carry g.
#include <stdexcept>
#include <type_traits>

#include "internal.h"

namespace ddst {
namespace {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// Block-wide sum of 256 threads; result valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double *sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += sh[w];
  __syncthreads();
  return s;
}

__device__ __forceinline__ double kappa_at(const double *kappa, int dim, int n, int c0, int c1,
                                           int c2) {
  if (!kappa) return 1.0;
  const size_t nc = (size_t)n + 1;
  if (dim == 2) return kappa[(size_t)c0 * nc + c1];
  return kappa[((size_t)c0 * nc + c1) * nc + c2];
}

// Mean coefficient of the edge from node p to p + e_axis (p 1-based).
__device__ double edge_coef(const double *kappa, int dim, int n, const int *p, int axis) {
  if (!kappa) return 1.0;
  int base[3] = {p[0] - 1, p[1] - 1, dim == 3 ? p[2] - 1 : 0};
  base[axis] = p[axis];  // cell index along the edge axis = node index of the lower end
  double s = 0.0;
  if (dim == 2) {
    const int o = 1 - axis;  // the other axis
    for (int t = 0; t < 2; ++t) {
      int c[2] = {base[0], base[1]};
      c[o] += t;
      s += kappa_at(kappa, 2, n, c[0], c[1], 0);
    }
    return 0.5 * s;
  }
  int oa = (axis == 0) ? 1 : 0, ob = (axis == 2) ? 1 : 2;
  for (int t = 0; t < 4; ++t) {
    int c[3] = {base[0], base[1], base[2]};
    c[oa] += t & 1;
    c[ob] += t >> 1;
    s += kappa_at(kappa, 3, n, c[0], c[1], c[2]);
  }
  return 0.25 * s;
}

__global__ void k_setup_coef(const double *__restrict__ kappa, const double *__restrict__ cz,
                             double b0, double b1, double b2, int dim, int n, double h,
                             double *__restrict__ coef) {
  const size_t N = (dim == 2) ? (size_t)n * n : (size_t)n * n * n;
  const size_t node = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= N) return;
  int p[3];
  if (dim == 2) {
    p[0] = (int)(node / n) + 1;
    p[1] = (int)(node % n) + 1;
    p[2] = 0;
  } else {
    p[0] = (int)(node / ((size_t)n * n)) + 1;
    p[1] = (int)((node / n) % n) + 1;
    p[2] = (int)(node % n) + 1;
  }
  const double ih2 = 1.0 / (h * h), i2h = 0.5 / h;
  const double b[3] = {b0, b1, b2};
  double diag = cz ? cz[node] : 0.0;
  for (int a = 0; a < dim; ++a) {
    const double kp = edge_coef(kappa, dim, n, p, a) * ih2;
    int q[3] = {p[0], p[1], p[2]};
    q[a] -= 1;
    const double km = edge_coef(kappa, dim, n, q, a) * ih2;
    diag += kp + km;
    coef[(size_t)(1 + 2 * a) * N + node] = -km - b[a] * i2h;
    coef[(size_t)(2 + 2 * a) * N + node] = -kp + b[a] * i2h;
  }
  coef[node] = diag;
}

// Em[i][r] = coupling of plane i to plane i-1, Ep[i][r] = to plane i+1
// (rows 0 and n+1 and the padding stay zero).
__global__ void k_fill_couplings(const double *__restrict__ coef, int n, int M, int ld,
                                 size_t N, double *__restrict__ Em, double *__restrict__ Ep) {
  const int i = blockIdx.y;  // plane 0..n+1
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < ld; r += gridDim.x * blockDim.x) {
    double em = 0.0, ep = 0.0;
    if (i >= 1 && i <= n && r < M) {
      const size_t node = (size_t)(i - 1) * M + r;
      em = coef[1 * N + node];
      ep = coef[2 * N + node];
    }
    Em[(size_t)i * ld + r] = em;
    Ep[(size_t)i * ld + r] = ep;
  }
}

// Residual r = f - A_full(x; g) (or f - A^T x), padded volume layout.
__global__ void k_residual(const double *__restrict__ coef, int dim, int n, int M, int ld,
                           const double *__restrict__ f, const double *__restrict__ g,
                           const double *__restrict__ x, double *__restrict__ r,
                           int transpose) {
  const size_t N = (size_t)M * n;
  const size_t node = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= N) return;
  const int i = (int)(node / M);  // 0-based plane
  const int ip = (int)(node % M);
  int p[3];
  p[0] = i + 1;
  if (dim == 2) {
    p[1] = ip + 1;
    p[2] = 0;
  } else {
    p[1] = ip / n + 1;
    p[2] = ip % n + 1;
  }
  const size_t nb = (size_t)n + 2;
  double acc = coef[node] * x[(size_t)i * ld + ip];
  for (int a = 0; a < dim; ++a) {
    for (int sgn = -1; sgn <= 1; sgn += 2) {
      int q[3] = {p[0], p[1], p[2]};
      q[a] += sgn;
      const bool inside = q[a] >= 1 && q[a] <= n;
      const int slot = (sgn < 0) ? 1 + 2 * a : 2 + 2 * a;
      if (inside) {
        const size_t qi = (size_t)(q[0] - 1);
        const size_t qip = (dim == 2) ? (size_t)(q[1] - 1)
                                      : (size_t)(q[1] - 1) * n + (size_t)(q[2] - 1);
        const size_t qnode = qi * M + qip;
        const double xv = x[qi * ld + qip];
        // A^T_{p,q} = A_{q,p}: the opposite slot of node q
        const int oslot = (sgn < 0) ? 2 + 2 * a : 1 + 2 * a;
        acc += (transpose ? coef[(size_t)oslot * N + qnode] : coef[(size_t)slot * N + node]) * xv;
      } else if (!transpose && g) {
        const size_t bidx = (dim == 2) ? (size_t)q[0] * nb + q[1]
                                       : ((size_t)q[0] * nb + q[1]) * nb + q[2];
        acc += coef[(size_t)slot * N + node] * g[bidx];
      }
    }
  }
  const double fv = f ? f[node] : 0.0;
  r[(size_t)i * ld + ip] = fv - acc;
}

__global__ void k_pad(const double *__restrict__ src, double *__restrict__ dst, int rows, int M,
                      int ld) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)rows * ld) return;
  const size_t row = e / ld, c = e % ld;
  dst[e] = (c < (size_t)M) ? src[row * M + c] : 0.0;
}

__global__ void k_unpad(const double *__restrict__ src, double *__restrict__ dst, int rows,
                        int M, int ld) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)rows * M) return;
  const size_t row = e / M, c = e % M;
  dst[e] = src[row * ld + c];
}

// four consecutive matrix entries as doubles (global-memory vector loads)
template <typename T>
__device__ __forceinline__ void ld4(const T *p, double *o) {
  constexpr int V = 16 / sizeof(T);
#pragma unroll
  for (int h = 0; h < 4 / V; ++h) {
    const typename V16<T>::type v = ld16(p + V * h);
#pragma unroll
    for (int e = 0; e < V; ++e) o[V * h + e] = (double)v[e];
  }
}

// out[r] = w[r] + alpha * (G[r,:] (x1 - e.*x2) + G2[r,:] x3); kGemvRows rows per
// work-group.  HBM-bound: each wavefront owns kGemvR rows and takes CH columns
// of a matrix at a time, all its 16-byte loads before using any (no branches
// between them: columns past the chunk re-read an in-bounds address and meet
// x = 0); the first loads are issued before x, staged in LDS kGemvX columns at a
// time, which they do not depend on.  Rows and columns that are padding are not
// read.  Two rows and 512 columns: little per wavefront, but six and more
// wavefronts per SIMD, whose number evens out the last round of work-groups; in
// large FP32 launches 1024 (gemv_wide, rules.h).  Planes of a sweep over 1023^2
// on 32 slabs, 134 MB: 33 us with four rows and 1024 columns, 28 with these (with
// one row 32, with eight 34); FP64 79 and 63.
constexpr int kGemvR = 2, kGemvRows = 4 * kGemvR, kGemvX = 1024;
template <int CH, typename T>
__device__ __forceinline__ void gemv_rows_load(const T *M, int ld, int cn, int lane,
                                               T (&g)[kGemvR][CH / 256][4]) {
#pragma unroll
  for (int q = 0; q < kGemvR; ++q)
#pragma unroll
    for (int i = 0; i < CH / 256; ++i) {
      const int c = lane * 4 + 256 * i;
      const T *src = M + (size_t)q * ld + (c < cn ? c : 0);
      constexpr int V = 16 / sizeof(T);
#pragma unroll
      for (int h = 0; h < 4 / V; ++h) {
        const typename V16<T>::type v = ld16(src + V * h);
#pragma unroll
        for (int e = 0; e < V; ++e) g[q][i][V * h + e] = v[e];
      }
    }
}
// x: CH doubles in LDS, zero past the chunk
template <int CH, typename T>
__device__ __forceinline__ void gemv_rows_fma(const T (&g)[kGemvR][CH / 256][4],
                                              const double *x, int lane, double (&acc)[kGemvR]) {
#pragma unroll
  for (int i = 0; i < CH / 256; ++i) {
    const int c = lane * 4 + 256 * i;
    const double x0 = x[c], x1 = x[c + 1], x2 = x[c + 2], x3 = x[c + 3];
#pragma unroll
    for (int q = 0; q < kGemvR; ++q)
      acc[q] += (double)g[q][i][0] * x0 + (double)g[q][i][1] * x1 +
                (double)g[q][i][2] * x2 + (double)g[q][i][3] * x3;
  }
}

template <int CH, typename T>
__device__ __forceinline__ void gemv_n_body(const GemvJob *__restrict__ jobs, int ld, int M,
                                            double alpha) {
  __shared__ double xs[2][kGemvX];
  const GemvJob J = jobs[blockIdx.y];
  const T *G = static_cast<const T *>(J.G);
  const T *G2 = static_cast<const T *>(J.G2);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row0 = blockIdx.x * kGemvRows + wave * kGemvR;
  const size_t ro = (size_t)row0 * ld;
  if ((!G && !G2) || (int)blockIdx.x * kGemvRows >= M) {
    // no matrix term (an end of a sweep, or padding): out = w
    if (lane < kGemvR) {
      const int r = row0 + lane;
      gp(J.out)[r] = J.w ? gp(J.w)[r] : 0.0;
    }
    return;
  }
  double acc[kGemvR];
#pragma unroll
  for (int q = 0; q < kGemvR; ++q) acc[q] = 0.0;
  // step t: chunk t of the first matrix, or, with two, chunk t / 2 of either
  const int two = G && G2 ? 1 : 0;
  const T *first = G ? G : G2;
  const int mc = min(ld, (M + 3) & ~3);  // whole 16-byte loads
  const int x0 = G ? 0 : 1;              // the first matrix's entries
  T g[kGemvR][CH / 256][4];
  for (int c0 = 0; c0 < mc; c0 += kGemvX) {
    const int xn = min(kGemvX, mc - c0);
    const int steps = (xn + CH - 1) / CH << two;
    auto load = [&](int t) {
      const int c = (t >> two) * CH;
      gemv_rows_load<CH, T>((t & two ? G2 : first) + ro + c0 + c, ld, xn - c, lane, g);
    };
    auto use = [&](int t) {
      gemv_rows_fma<CH, T>(g, xs[t & two ? 1 : x0] + (t >> two) * CH, lane, acc);
    };
    load(0);
    if (c0 > 0) __syncthreads();  // the previous columns' x is no longer read
    for (int c = threadIdx.x; c < kGemvX; c += 256) {
      double v = 0.0, v3 = 0.0;
      if (c < xn) {
        v = J.x1 ? gp(J.x1)[c0 + c] : 0.0;
        if (J.e) v -= gp(J.e)[c0 + c] * gp(J.x2)[c0 + c];
        v3 = (G2 && J.x3) ? gp(J.x3)[c0 + c] : 0.0;
      }
      xs[0][c] = v;
      xs[1][c] = v3;
    }
    __syncthreads();
    use(0);
    for (int t = 1; t < steps; ++t) {
      // not earlier: more registers, fewer wavefronts
      asm volatile("" ::: "memory");
      load(t);
      use(t);
    }
  }
#pragma unroll
  for (int q = 0; q < kGemvR; ++q) {
    const double s = wave_sum(acc[q]);
    if (lane == 0) {
      const int r = row0 + q;
      gp(J.out)[r] = (J.w ? gp(J.w)[r] : 0.0) + alpha * s;
    }
  }
}

template <int CH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k_gemv_n_f32(
    const GemvJob *__restrict__ jobs, int ld, int M, double alpha) {
  gemv_n_body<CH, float>(jobs, ld, M, alpha);
}
__global__ __launch_bounds__(256) void k_gemv_n_f64(const GemvJob *__restrict__ jobs, int ld,
                                                    int M, double alpha) {
  gemv_n_body<512, double>(jobs, ld, M, alpha);
}

// Several right-hand sides per launch, on the matrix cores: vector v of a job
// is the job's vector shifted by v * vs (x1, x2, x3, w and out; the matrices
// and e are shared), up to 16 per launch.  Y = Mat X is a product of the
// matrix rows with a 16-column block of vectors, done by the FP64
// 16 x 16 x 4 MFMA (matrix entries converted exactly to FP64, FP64
// accumulation, as in the one-vector kernel): each wavefront owns a strip
// of 16 rows; per 16-column step lane l loads four
// consecutive entries of row l % 16 (columns 4 (l / 16) + 0..3), which feed
// the A operand of four MFMAs, the i-th taking columns {4 q + i}; the B
// operand is the matching entries of the 16 vectors, staged column-major in
// LDS per chunk of columns (zero for vectors past nv); the next chunk's
// matrix entries and vectors are loaded while a chunk is used.  The FP64 output holds
// vector l % 16 of rows 4 r + l / 16 in register r.
typedef double f64x4v __attribute__((ext_vector_type(4)));
constexpr int kMvLd = 17;  // LDS row stride (doubles) of the staged block
// columns staged per chunk: a divisor of every leading dimension (a multiple
// of 128)
constexpr int kMvCh = 64;

template <typename T, int NS>
__device__ __forceinline__ void mv_load(const T *Mt, size_t row_off, int c0, int kq,
                                        T (&a)[NS][4]) {
  constexpr int V = 16 / sizeof(T);
#pragma unroll
  for (int st = 0; st < NS; ++st) {
    const T *src = Mt + row_off + c0 + 16 * st + 4 * kq;
#pragma unroll
    for (int h = 0; h < 4 / V; ++h) {
      const typename V16<T>::type v = ld16(src + V * h);
#pragma unroll
      for (int e = 0; e < V; ++e) a[st][V * h + e] = v[e];
    }
  }
}

// W strips of 16 rows per work-group: 8 share each staged block of x over 128
// rows (fewer staging loads per row, better from 8 vectors on), 4 give twice
// the work-groups (better for 2 to 4 vectors).  The chunks are dealt to H = 2
// sets of W wavefronts, whose sums are added at the end: a sweep over 32 FP32
// planes of 1024 rows would be 8 wavefronts per CU with one set, too few
// loads in flight.  That sweep and the interface products, on average: 44 us
// with 8 vectors, 40 with 3 (one set, chunks of 128 with x loaded between two
// barriers: 54 and 48).
template <typename T, int W, int H>
__global__ __launch_bounds__(64 * W * H) void k_gemv_mfma(const GemvJob *__restrict__ jobs, int ld,
                                                          double alpha, int nv, size_t vs) {
  constexpr int CH = kMvCh, NS = CH / 16, RB = 16 * W, NX = 16 * CH / (64 * W);
  __shared__ double xt[2][H][CH * kMvLd];
  static_assert((H - 1) * W * 64 * 4 <= 2 * H * CH * kMvLd, "the sums of the other sets fit");
  const GemvJob J = jobs[blockIdx.y];
  const T *G = static_cast<const T *>(J.G);
  const T *G2 = static_cast<const T *>(J.G2);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int strip = wave % W, set = wave / W, tid = threadIdx.x - set * 64 * W;
  const int m = lane & 15, kq = lane >> 4;
  const int rowb = blockIdx.x * RB;  // first row of the work-group
  const int roww = rowb + strip * 16;  // first row of this wavefront's strip
  if (!G && !G2) {  // no matrix term: out = w
    for (int e = threadIdx.x; e < RB * nv; e += 64 * W * H) {
      const size_t o = (size_t)(e / RB) * vs + rowb + e % RB;
      gp(J.out)[o] = J.w ? gp(J.w)[o] : 0.0;
    }
    return;
  }
  f64x4v acc = {0.0, 0.0, 0.0, 0.0};
  const size_t row_off = (size_t)(roww + m) * ld;
  // chunks of the first matrix, then of the second; set h takes every H-th
  const int nc = ld / CH, total = nc << (G && G2 ? 1 : 0), steps = (total + H - 1) / H;
  T a[NS][4], an[NS][4];
  double xr[NX];
  auto load = [&](int t, T (&q)[NS][4]) {
    const int ch = t * H + set;
    if (ch >= total) return;
    const bool one = G && ch < nc;
    const int c0 = (ch < nc ? ch : ch - nc) * CH;
    mv_load<T, NS>(one ? G : G2, row_off, c0, kq, q);
    const double *xa = one ? J.x1 : J.x3, *xe = one ? J.e : nullptr;
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int idx = tid + 64 * W * i, v = idx / CH, k = c0 + idx % CH;
      double x = 0.0;
      if (v < nv) {
        const size_t o = (size_t)v * vs + k;
        x = xa ? gp(xa)[o] : 0.0;
        if (xe) x -= gp(xe)[k] * gp(J.x2)[o];
      }
      xr[i] = x;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int idx = tid + 64 * W * i;
      xt[buf][set][idx % CH * kMvLd + idx / CH] = xr[i];
    }
  };
  load(0, a);
  store(0);
  __syncthreads();
#pragma unroll 1
  for (int t = 0; t < steps; ++t) {
    if (t + 1 < steps) load(t + 1, an);
    const double *xb = xt[t & 1][set];
    if (t * H + set < total)
#pragma unroll
      for (int st = 0; st < NS; ++st)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(
              (double)a[st][i], xb[(16 * st + 4 * kq + i) * kMvLd + m], acc, 0, 0, 0);
    if (t + 1 < steps) {
      store((t + 1) & 1);
#pragma unroll
      for (int st = 0; st < NS; ++st)
#pragma unroll
        for (int i = 0; i < 4; ++i) a[st][i] = an[st][i];
    }
    __syncthreads();
  }
  if constexpr (H > 1) {
    double *red = &xt[0][0][0];
    if (set > 0)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[(((set - 1) * W + strip) * 4 + r) * 64 + lane] = acc[r];
    __syncthreads();
    if (set > 0) return;
#pragma unroll
    for (int h = 0; h < H - 1; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] += red[((h * W + strip) * 4 + r) * 64 + lane];
  }
  if (m < nv) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const size_t o = (size_t)m * vs + roww + 4 * r + kq;
      gp(J.out)[o] = (J.w ? gp(J.w)[o] : 0.0) + alpha * acc[r];
    }
  }
}

// Transposed product, partial sums over row chunks:
// part[(job*nchunk + chunk)*ld + c] = sum_{r in chunk} G[r,c] xe[r] + G2[r,c] x3[r]
// A work-group takes 256 columns (a strip) of a chunk's rows, a quarter of them
// per wavefront, eight rows' loads in flight; rows and columns of padding are not
// read.  Its place in the grid: (strip, chunk, job) with ROWS, so that whole rows
// are read at a time, else (chunk, job, strip); gemv_t_rows (rules.h) says when.
// 24 planes of 767 rows in FP32: 15 us and 5 for the reduction (one row at a
// time over all columns in chunks of 32 rows 23 and 8).
template <typename T, bool ROWS>
__global__ __launch_bounds__(256) void k_gemv_t_part(const GemvJob *__restrict__ jobs, int ld,
                                                     int M, int rows_per_chunk,
                                                     double *__restrict__ part) {
  constexpr int U = 8;
  __shared__ double red[4][256];
  extern __shared__ double sh[];
  const int strip = ROWS ? blockIdx.x : blockIdx.z, chunk = ROWS ? blockIdx.y : blockIdx.x;
  const int job = ROWS ? blockIdx.z : blockIdx.y, nchunk = ROWS ? gridDim.y : gridDim.x;
  const GemvJob J = jobs[job];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = chunk * rows_per_chunk, rn = max(0, min(rows_per_chunk, M - r0));
  const int c = strip * 256 + lane * 4;
  double *xs[2] = {sh, sh + rows_per_chunk};
  for (int r = threadIdx.x; r < rn; r += 256) {
    double v = J.x1 ? gp(J.x1)[r0 + r] : 0.0;
    if (J.e) v -= gp(J.e)[r0 + r] * gp(J.x2)[r0 + r];
    xs[0][r] = v;
    xs[1][r] = (J.G2 && J.x3) ? gp(J.x3)[r0 + r] : 0.0;
  }
  __syncthreads();
  double s[4] = {0, 0, 0, 0};
  if (c < M)
    for (int k = 0; k < 2; ++k) {
      const T *G = static_cast<const T *>(k == 0 ? J.G : J.G2);
      if (!G) continue;
      G += (size_t)r0 * ld + c;
      const double *x = xs[k];
      int r = wave * U;
      for (; r + U <= rn; r += 4 * U) {
        double g[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) ld4<T>(G + (size_t)(r + u) * ld, g[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) s[e] += g[u][e] * x[r + u];
      }
      for (; r < rn; ++r) {  // the ragged last rows (of one wavefront)
        double g[4];
        ld4<T>(G + (size_t)r * ld, g);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += g[e] * x[r];
      }
    }
#pragma unroll
  for (int e = 0; e < 4; ++e) red[wave][lane * 4 + e] = s[e];
  __syncthreads();
  const int cc = strip * 256 + threadIdx.x;
  if (cc < ld)
    part[((size_t)job * nchunk + chunk) * ld + cc] =
        (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

__global__ void k_gemv_t_reduce(const GemvJob *__restrict__ jobs, int ld, int nchunk,
                                const double *__restrict__ part, double alpha) {
  const int job = blockIdx.y;
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ld) return;
  const GemvJob J = jobs[job];
  double s = 0.0;
  for (int k = 0; k < nchunk; ++k) s += part[((size_t)job * nchunk + k) * ld + c];
  gp(J.out)[c] = (J.w ? gp(J.w)[c] : 0.0) + alpha * s;
}

__global__ void k_interface_rhs(const double *__restrict__ vol, const double *__restrict__ Zl,
                                const double *__restrict__ Zr, const double *__restrict__ Ea,
                                const double *__restrict__ Eb, int n_ds, int m, int ld,
                                int a_off, int b_off, double *__restrict__ out) {
  const int j = blockIdx.y + 1;  // interface 1..n_ds
  const int pl = j * m;          // node plane (1-based)
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < ld; r += gridDim.x * blockDim.x) {
    const double v = (vol ? vol[(size_t)(pl - 1) * ld + r] : 0.0) -
                     Ea[(size_t)(pl + a_off) * ld + r] * Zl[(size_t)(pl - 2) * ld + r] -
                     Eb[(size_t)(pl + b_off) * ld + r] * Zr[(size_t)pl * ld + r];
    out[(size_t)(j - 1) * ld + r] = v;
  }
}

__global__ void k_copy_planes(const double *__restrict__ src, int src_stride, int src_off,
                              double *__restrict__ dst, int dst_stride, int dst_off, int ld,
                              int M) {
  const int k = blockIdx.y;
  const double *s = src + (size_t)(src_off + (size_t)k * src_stride) * ld;
  double *d = dst + (size_t)(dst_off + (size_t)k * dst_stride) * ld;
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < ld; r += gridDim.x * blockDim.x)
    d[r] = (r < M) ? s[r] : 0.0;
}

__global__ void k_axpy(double *__restrict__ y, const double *__restrict__ x, double a,
                       size_t len) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < len) y[e] += a * x[e];
}

__global__ void k_fill(double *__restrict__ y, double v, size_t len) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < len) y[e] = v;
}

// ---- passes over a Krylov basis ---------------------------------------------
// V: vectors of len entries, `stride` apart, 10 to 1000 of them, len 10^3 to
// 10^6.  What bounds them is the loads in flight: a work-group takes a chunk of
// 64 T entries (T per lane) and its 16 wavefronts share the vectors, eight at
// a time with their loads issued together, so that short vectors still fill
// the chip.  A classical step's passes over FP32 bases of 15872 entries and
// about 240 vectors take 4.6 us each; with 256 entries per work-group and
// every vector in turn, by one thread an entry (updates) or by four
// wavefronts (products), they took 15 and 19.  T = 1, 2, 4, the largest that
// leaves a chunk per CU (kDotChunks).
// Sums are FP64, in a fixed order.
constexpr int kDotWaves = 16;  // wavefronts per work-group
constexpr int kDotVecs = 8;    // basis vectors per wavefront and round
constexpr int kDotRound = kDotWaves * kDotVecs;

// Entries of the work-group's chunk of 64 T.  Lengths are multiples of 128
// (with_dot_width checks), so that only chunks of 256 can be partial.  In 32
// bits: the compiler takes a uniform 64-bit minimum's select from a condition
// that its comparison does not set, and the last chunk then came out whole.
template <int T> __device__ __forceinline__ int chunk_len(size_t len) {
  if constexpr (128 % (64 * T) == 0) return 64 * T;
  return blockIdx.x + 1 < gridDim.x ? 64 * T : (int)(len - (size_t)blockIdx.x * 64 * T);
}

// T entries of v from e0 (FULL: all inside the chunk; else those past its cn
// entries repeat the last one, and the caller drops or zeroes what they give).
template <int T, bool FULL, typename B>
__device__ __forceinline__ void ld_entries(const B *v, int e0, int cn, double (&x)[T]) {
  if constexpr (FULL && T > 1) {
    // stride is any number: only the alignment of an entry
    typedef B vec __attribute__((ext_vector_type(T), aligned(sizeof(B))));
    const vec q = *reinterpret_cast<const vec *>(v + e0);
#pragma unroll
    for (int t = 0; t < T; ++t) x[t] = (double)q[t];
  } else {
#pragma unroll
    for (int t = 0; t < T; ++t) x[t] = (double)v[FULL ? e0 + t : min(e0 + t, cn - 1)];
  }
}

// Sums over the wavefront of N values per lane (N a power of two), halved at
// each exchange: lane l returns the sum of value l / (64 / N).
template <int N, int OFF = 32> __device__ __forceinline__ double wave_sums(const double (&v)[N]) {
  if constexpr (N > 1) {
    const bool up = threadIdx.x & OFF;
    double r[N / 2];
#pragma unroll
    for (int u = 0; u < N / 2; ++u)
      r[u] = (up ? v[u + N / 2] : v[u]) + __shfl_xor(up ? v[u] : v[u + N / 2], OFF);
    return wave_sums<N / 2, OFF / 2>(r);
  } else {
    double r = v[0];
#pragma unroll
    for (int off = OFF; off > 0; off >>= 1) r += __shfl_xor(r, off);
    return r;
  }
}

// sum[c][t] += coef_c[i] V_i (NC sets of coefficients) over the wavefront's
// share of the nvec vectors, at its lanes' entries of the chunk.
template <int NC, int T, bool FULL, typename B>
__device__ __forceinline__ void chunk_combine(const B *V, size_t stride, int nvec,
                                              const double *const (&coef)[NC], int cn,
                                              double (&sum)[NC][T]) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int t = 0; t < T; ++t) sum[c][t] = 0.0;
  for (int i0 = wave * kDotVecs; i0 < nvec; i0 += kDotRound) {
    double x[kDotVecs][T];
#pragma unroll
    for (int u = 0; u < kDotVecs; ++u)
      ld_entries<T, FULL>(V + (size_t)min(i0 + u, nvec - 1) * stride, lane * T, cn, x[u]);
#pragma unroll
    for (int u = 0; u < kDotVecs; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const double h = i0 + u < nvec ? coef[c][min(i0 + u, nvec - 1)] : 0.0;
#pragma unroll
        for (int t = 0; t < T; ++t) sum[c][t] += x[u][t] * h;
      }
  }
}

// The wavefronts' sums added up: the first 64 T threads get entry threadIdx.x
// of every set.  red: NC kDotWaves 64 T doubles.
template <int NC, int T>
__device__ __forceinline__ void chunk_gather(const double (&sum)[NC][T], double *red,
                                             double (&out)[NC]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int t = 0; t < T; ++t)
      red[(c * kDotWaves + wave) * 64 * T + lane * T + t] = sum[c][t];
  __syncthreads();
  if (threadIdx.x < 64 * T)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < kDotWaves; ++w) s += red[(c * kDotWaves + w) * 64 * T + threadIdx.x];
      out[c] = s;
    }
}

// Sum of x over the first 64 T threads of the work-group, in thread 0.
template <int T> __device__ __forceinline__ double chunk_sum(double x, double *sh) {
  if (threadIdx.x < 64 * T) {
    x = wave_sum(x);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = x;
  }
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < T; ++w) s += sh[w];
  return s;
}

// Per chunk: w += sign V h (nvec vectors; 0: none), then, of the updated
// chunk, the partial dot products with the same basis (ndot vectors),
// part[chunk * ndot + i], or its partial squared norm part[chunk] (ndot 0), or
// nothing (ndot < 0).
template <typename B, int T>
__global__ __launch_bounds__(64 * kDotWaves) void k_mgs_update_dots(
    double *__restrict__ w, const B *__restrict__ V, size_t stride, int nvec,
    const double *__restrict__ h, double sign, size_t len, int ndot, double *__restrict__ part) {
  __shared__ double red[kDotWaves * 64 * T], ws[64 * T], sh[T];
  const size_t base = (size_t)blockIdx.x * 64 * T;
  const int cn = chunk_len<T>(len);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const B *v = V + base;
  double we = tid < cn ? w[base + tid] : 0.0;
  if (nvec > 0) {
    double sum[1][T], r[1] = {0.0};
    const double *const coef[1] = {h};
    if (cn == 64 * T)
      chunk_combine<1, T, true>(v, stride, nvec, coef, cn, sum);
    else
      chunk_combine<1, T, false>(v, stride, nvec, coef, cn, sum);
    chunk_gather<1, T>(sum, red, r);
    if (tid < cn) {
      we += sign * r[0];
      w[base + tid] = we;
    }
  }
  if (ndot < 0) return;
  if (ndot == 0) {
    const double s = chunk_sum<T>(tid < cn ? we * we : 0.0, sh);
    if (tid == 0) part[blockIdx.x] = s;
    return;
  }
  if (tid < 64 * T) ws[tid] = we;
  __syncthreads();
  double wv[T];
#pragma unroll
  for (int t = 0; t < T; ++t) wv[t] = ws[lane * T + t];
  auto dots = [&](auto full) {
    for (int i0 = wave * kDotVecs; i0 < ndot; i0 += kDotRound) {
      double x[kDotVecs][T], s[kDotVecs];
#pragma unroll
      for (int u = 0; u < kDotVecs; ++u)
        ld_entries<T, decltype(full)::value>(v + (size_t)min(i0 + u, ndot - 1) * stride, lane * T,
                                             cn, x[u]);
#pragma unroll
      for (int u = 0; u < kDotVecs; ++u) {
        s[u] = 0.0;
#pragma unroll
        for (int t = 0; t < T; ++t) s[u] += x[u][t] * wv[t];
      }
      const double r = wave_sums<kDotVecs>(s);
      const int i = i0 + lane / (64 / kDotVecs);
      if (lane % (64 / kDotVecs) == 0 && i < ndot) part[(size_t)blockIdx.x * ndot + i] = r;
    }
  };
  if (cn == 64 * T)
    dots(std::true_type{});
  else
    dots(std::false_type{});
}

// Partial squared norms per chunk of 256 entries.
__global__ __launch_bounds__(256) void k_norm_part(const double *__restrict__ w, size_t len,
                                                   double *__restrict__ part) {
  __shared__ double sh[4];
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  const double x = e < len ? w[e] : 0.0;
  const double s = block_sum(x * x, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// Column j of H, staged in LDS cl[0..j+1] (cl[j+1] = hn, the subdiagonal
// entry), is rotated by the j previous Givens rotations (cs, sn staged in
// LDS), a new rotation zeroes its subdiagonal entry and is applied to g;
// writes column j of d.H, the rotation, g and res[2j], res[2j+1].  All 256
// threads of the work-group.  The rotations form the recurrence
//   a_0 = c_0,  a_{i+1} = -sn_i a_i + cs_i c_{i+1},  c_i <- cs_i a_i + sn_i c_{i+1}
// (c_j <- a_j before the new rotation): a first-order linear recurrence,
// evaluated as a parallel prefix of affine maps x -> m x + b (each thread
// composes the maps of a contiguous segment, the work-group scans the 256
// segment maps, then each thread replays its segment from its prefix), so
// the column costs O(j / 256 + log 256) steps instead of a serial chain of
// j rotations.
constexpr int kGivensLds = 2048;
__device__ __forceinline__ void givens_column_lds(double *cl, const double *cs,
                                                  const double *sn, int j, GmresDev d,
                                                  double beta, double hn) {
  __shared__ double sm[256], sb[256], co[kGivensLds + 1];
  __shared__ double aj;
  const int t = threadIdx.x;
  const int seg = (j + 255) / 256;
  const int i0 = min(t * seg, j), i1 = min(i0 + seg, j);
  double m = 1.0, b = 0.0;
  for (int i = i0; i < i1; ++i) {  // compose T_i after the segment so far
    const double mi = -sn[i], bi = cs[i] * cl[i + 1];
    b = mi * b + bi;
    m = mi * m;
  }
  sm[t] = m;
  sb[t] = b;
  __syncthreads();
  // inclusive scan over threads: P_t = S_t o ... o S_0
  for (int off = 1; off < 256; off <<= 1) {
    double pm = 1.0, pb = 0.0;
    const bool has = t >= off;
    if (has) {
      pm = sm[t - off];
      pb = sb[t - off];
    }
    __syncthreads();
    if (has) {  // (S_t o P_{t-off}): m = m_t pm, b = m_t pb + b_t
      const double mt = sm[t], bt = sb[t];
      sm[t] = mt * pm;
      sb[t] = mt * pb + bt;
    }
    __syncthreads();
  }
  // a at the start of this thread's segment: exclusive prefix applied to c_0
  double a = cl[0];
  if (t > 0) a = sm[t - 1] * cl[0] + sb[t - 1];
  for (int i = i0; i < i1; ++i) {
    const double bnext = cl[i + 1];
    co[i] = cs[i] * a + sn[i] * bnext;
    a = -sn[i] * a + cs[i] * bnext;
  }
  if (i1 == j && i0 < i1) aj = a;  // the thread that took the last step
  if (j == 0 && t == 0) aj = cl[0];
  __syncthreads();
  double *col = d.H + gmres_hoff(j);
  for (int i = t; i < j; i += 256) col[i] = co[i];
  if (t == 0) {
    const double av = aj;
    const double r = hypot(av, hn);
    const double ck = r > 0.0 ? av / r : 1.0;
    const double sk = r > 0.0 ? hn / r : 0.0;
    d.cs[j] = ck;
    d.sn[j] = sk;
    col[j] = r;
    col[j + 1] = 0.0;
    const double gk = j == 0 ? beta : d.g[j];
    d.g[j + 1] = -sk * gk;
    d.g[j] = ck * gk;
    d.res[2 * j] = fabs(d.g[j + 1]) / beta;
    d.res[2 * j + 1] = (hn > 0.0 && isfinite(hn)) ? 0.0 : 1.0;
  }
}

// The same for a column too long for LDS (j + 2 > kGivensLds): thread 0 runs
// the rotations serially on the column in global memory.
__device__ __forceinline__ void givens_column_global(double *col, int j, GmresDev d,
                                                     double beta, double hn) {
  if (threadIdx.x == 0) {
    col[j + 1] = hn;
    double a = col[0];
    for (int i = 0; i < j; ++i) {
      const double bnext = col[i + 1];
      col[i] = d.cs[i] * a + d.sn[i] * bnext;
      a = -d.sn[i] * a + d.cs[i] * bnext;
    }
    const double r = hypot(a, hn);
    const double ck = r > 0.0 ? a / r : 1.0;
    const double sk = r > 0.0 ? hn / r : 0.0;
    d.cs[j] = ck;
    d.sn[j] = sk;
    col[j] = r;
    col[j + 1] = 0.0;
    const double gk = j == 0 ? beta : d.g[j];
    d.g[j + 1] = -sk * gk;
    d.g[j] = ck * gk;
    d.res[2 * j] = fabs(d.g[j + 1]) / beta;
    d.res[2 * j + 1] = (hn > 0.0 && isfinite(hn)) ? 0.0 : 1.0;
  }
}

// Column k of H from the two classical Gram-Schmidt passes (hd[0..k] +
// hd[k+1..2k+1], new norm hn): kept unrotated in d.Hraw (for a later lagged
// step, which multiplies by H), then rotated.  All threads of one work-group.
__device__ __forceinline__ void gmres_givens_block(const double *__restrict__ hd, GmresDev d,
                                                   int k, double beta, double hn) {
  __shared__ double cl[kGivensLds + 2], cs[kGivensLds], sn[kGivensLds];
  for (int i = threadIdx.x; i <= k + 1; i += blockDim.x) {
    const double v = i <= k ? hd[i] + hd[k + 1 + i] : hn;
    d.Hraw[gmres_rix(i, k, d.maxit)] = v;
    if (k + 2 <= kGivensLds) {
      cl[i] = v;
      if (i < k) {
        cs[i] = d.cs[i];
        sn[i] = d.sn[i];
      }
    } else {
      d.H[gmres_hoff(k) + i] = v;
    }
  }
  __syncthreads();
  if (k + 2 <= kGivensLds)
    givens_column_lds(cl, cs, sn, k, d, beta, hn);
  else
    givens_column_global(d.H + gmres_hoff(k), k, d, beta, hn);
}

// Column j of H from d.Hraw (rows 0..j+1), rotated (the lagged steps).
__device__ __forceinline__ void gmres_givens_raw(GmresDev d, int j, double beta) {
  __shared__ double cl[kGivensLds + 2], cs[kGivensLds], sn[kGivensLds];
  const double hn = d.Hraw[gmres_rix(j + 1, j, d.maxit)];
  for (int i = threadIdx.x; i <= j + 1; i += blockDim.x) {
    const double v = d.Hraw[gmres_rix(i, j, d.maxit)];
    if (j + 2 <= kGivensLds) {
      cl[i] = v;
      if (i < j) {
        cs[i] = d.cs[i];
        sn[i] = d.sn[i];
      }
    } else {
      d.H[gmres_hoff(j) + i] = v;
    }
  }
  __syncthreads();
  if (j + 2 <= kGivensLds)
    givens_column_lds(cl, cs, sn, j, d, beta, hn);
  else
    givens_column_global(d.H + gmres_hoff(j), j, d, beta, hn);
}

// Last kernel of Arnoldi step k: dst = src / sqrt(sum of the nchunk partial
// squared norms) (and its FP32 rounding in slot, if given), every
// work-group summing the partials in the same order; the first one stores
// the norm in hd and then applies the Givens rotations (column k of H from
// hd), concurrently with the others' scaling.
__global__ __launch_bounds__(256) void k_norm_scale_givens(const double *__restrict__ part,
                                                           int nchunk, double *__restrict__ hd,
                                                           const double *__restrict__ src,
                                                           double *__restrict__ dst,
                                                           float *__restrict__ slot, size_t len,
                                                           GmresDev gd, int k, double beta) {
  __shared__ double sh[4], snorm;
  double s = 0.0;
  for (int c = threadIdx.x; c < nchunk; c += 256) s += part[c];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) {
    snorm = sqrt(s);
    if (blockIdx.x == 0) hd[2 * (k + 1)] = snorm;
  }
  __syncthreads();
  const double d = snorm;
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < len) {
    const double v = (d > 0.0) ? src[e] / d : 0.0;
    dst[e] = v;
    if (slot) slot[e] = (float)v;
  }
  if (blockIdx.x == 0) gmres_givens_block(hd, gd, k, beta, d);
}

// ---- Arnoldi with lagged reorthogonalization (see launch_arnoldi_lagged) --

// Pass A: partial dot products of the m - 1 basis vectors Q (V, stride) and
// of the candidate u with u and with w (null: only those with u), per
// kLagChunk-entry chunk: part[chunk][i] = V_i . u, part[chunk][m + i] =
// V_i . w (i < m - 1), part[chunk][m - 1] = u . u, part[chunk][2 m - 1] =
// u . w.  Work-group (chunk, g): vectors g kDotRound .., eight per wavefront;
// group 0 also forms the products of u.  FP64 bases of 64512 entries, 500
// vectors on average: 47 us, 5.4 TB/s (54 with chunks of 2048 and 32 vectors
// per work-group).
constexpr int kLagChunk = 256;
template <typename B>
__global__ __launch_bounds__(64 * kDotWaves) void k_lag_dots(const B *__restrict__ V, size_t stride,
                                                             int m, const double *__restrict__ u,
                                                             const double *__restrict__ w,
                                                             size_t len,
                                                             double *__restrict__ part) {
  constexpr int T = kLagChunk / 64;
  const size_t base = (size_t)blockIdx.x * kLagChunk;
  const int cn = chunk_len<T>(len);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nq = m - 1;
  const int i0 = blockIdx.y * kDotRound + wave * kDotVecs;
  const bool own = blockIdx.y == 0 && wave == kDotWaves - 1;
  if (i0 >= nq && !own) return;
  double *pc = part + (size_t)blockIdx.x * 2 * m;
  double a[T], c[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int e = lane * T + t;
    a[t] = e < cn ? u[base + e] : 0.0;
    c[t] = (w && e < cn) ? w[base + e] : 0.0;
  }
  if (own) {
    double s[2] = {0.0, 0.0};
#pragma unroll
    for (int t = 0; t < T; ++t) {
      s[0] += a[t] * a[t];
      s[1] += a[t] * c[t];
    }
    const double r = wave_sums<2>(s);
    if (lane % 32 == 0) pc[lane == 0 ? m - 1 : 2 * m - 1] = r;
  }
  if (i0 >= nq) return;
  double s[2 * kDotVecs];
  auto dots = [&](auto full) {
    double x[kDotVecs][T];
#pragma unroll
    for (int q = 0; q < kDotVecs; ++q)
      ld_entries<T, decltype(full)::value>(V + (size_t)min(i0 + q, nq - 1) * stride + base,
                                           lane * T, cn, x[q]);
#pragma unroll
    for (int q = 0; q < kDotVecs; ++q) {
      s[q] = s[kDotVecs + q] = 0.0;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        s[q] += x[q][t] * a[t];
        s[kDotVecs + q] += x[q][t] * c[t];
      }
    }
  };
  if (cn == kLagChunk)
    dots(std::true_type{});
  else
    dots(std::false_type{});
  const double r = wave_sums<2 * kDotVecs>(s);
  const int q = lane / (32 / kDotVecs), i = i0 + q % kDotVecs;
  if (lane % (32 / kDotVecs) == 0 && i < nq) pc[(q < kDotVecs ? 0 : m) + i] = r;
}

// nu = |u - Q a| = sqrt(|u|^2 - |a|^2) from the pass-A products (every
// thread of the work-group gets it).
__device__ __forceinline__ double lag_nu(const GmresDev &d, int k) {
  __shared__ double sh[4], snu;
  double t = 0.0;
  for (int i = threadIdx.x; i < k; i += 256) t += d.dA[i] * d.dA[i];
  t = block_sum(t, sh);
  if (threadIdx.x == 0) {
    const double nu2 = d.dA[k] - t;
    snu = nu2 > 0.0 ? sqrt(nu2) : 0.0;
  }
  __syncthreads();
  return snu;
}

// d = H a over rows 0..k (one wavefront per row, four rows per work-group),
// with column k - 1 taken as finalized now (unless col_final: it is in
// Hraw already): prov + rho a above the diagonal, rho nu below it; work-group
// 0 stores that column in Hraw.
__global__ __launch_bounds__(256) void k_lag_hmul(GmresDev d, int k, int col_final) {
  const double *a = d.dA;
  const bool fin = k >= 1 && !col_final;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = blockIdx.x * 4 + wave;
  const int jend = fin ? k - 1 : k;  // stored columns [j0, jend)
  double acc = 0.0;
  if (r <= k) {  // needs no norm: its loads are under way beside it
    const int j0 = r > 0 ? r - 1 : 0;
    const double *row = d.Hraw + gmres_roff(r, d.maxit) - j0;
#pragma unroll 4
    for (int j = j0 + lane; j < jend; j += 64) acc += row[j] * a[j];
  }
  const double nu = lag_nu(d, k);
  const double rho = d.sc[2];
  auto lastcol = [&](int i) { return i < k ? d.prov[i] + rho * a[i] : rho * nu; };
  if (blockIdx.x == 0 && fin)
    for (int i = threadIdx.x; i <= k; i += 256) d.Hraw[gmres_rix(i, k - 1, d.maxit)] = lastcol(i);
  if (r > k) return;
  acc = wave_sum(acc);
  if (lane == 0) d.dv[r] = acc + (fin ? lastcol(r) * a[k - 1] : 0.0);
}

// Coefficients of pass B (one work-group): with d = dv, b = Q^T w, gamma =
// u.w, the provisional column h_i = (b_i - d_i) / nu (i < k), h_k =
// ((gamma - a.b) / nu - d_k) / nu; e = d / nu + h; pass B forms
// z = w / nu - Q f - g u with f = e[0:k] - e_k a / nu, g = e_k / nu.
__global__ __launch_bounds__(256) void k_lag_coef(GmresDev d, int k) {
  __shared__ double sh[2][4], sek, sinv;
  const int m = k + 1;
  const double *a = d.dA, *b = d.dA + m;
  double aa = 0.0, t = 0.0;
  for (int i = threadIdx.x; i < k; i += 256) {
    const double x = a[i];
    aa += x * x;
    t += x * b[i];
  }
  aa = wave_sum(aa);
  t = wave_sum(t);
  if ((threadIdx.x & 63) == 0) {
    sh[0][threadIdx.x >> 6] = aa;
    sh[1][threadIdx.x >> 6] = t;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    aa = t = 0.0;
    for (int w = 0; w < 4; ++w) {
      aa += sh[0][w];
      t += sh[1][w];
    }
    const double nu2 = d.dA[k] - aa;  // as lag_nu
    const double inv = nu2 > 0.0 ? 1.0 / sqrt(nu2) : 0.0;
    sinv = inv;
    const double hk = ((b[k] - t) * inv - d.dv[k]) * inv;
    d.prov[k] = hk;
    sek = d.dv[k] * inv + hk;
    d.sc[0] = inv;
    d.sc[1] = sek * inv;
  }
  __syncthreads();
  const double ek = sek, inv = sinv;
  for (int i = threadIdx.x; i < k; i += 256) {
    const double h = (b[i] - d.dv[i]) * inv;
    d.prov[i] = h;
    d.cf[i] = d.dv[i] * inv + h - ek * a[i] * inv;
  }
}

// Pass B, per chunk of 64 T entries: q_k = (u - Q a) / nu into slot k of V, w =
// w / nu - Q f - g u, and the chunk's partial squared norm of the new w.
// u may be slot k itself (an FP64 basis): each entry is read before it is
// overwritten, by the same thread.  As above: 44 us, 5.8 TB/s (50 with one
// thread an entry for all vectors).
template <typename B, int T>
__global__ __launch_bounds__(64 * kDotWaves) void k_lag_update(B *V, size_t stride, int k,
                                                               const double *u,
                                                               double *__restrict__ w, size_t len,
                                                               GmresDev d,
                                                               double *__restrict__ part) {
  __shared__ double red[2 * kDotWaves * 64 * T], sh[T];
  const size_t base = (size_t)blockIdx.x * 64 * T;
  const int cn = chunk_len<T>(len);
  const int tid = threadIdx.x;
  double sum[2][T], r[2] = {0.0, 0.0};
  const double *const coef[2] = {d.dA, d.cf};
  if (cn == 64 * T)
    chunk_combine<2, T, true>(V + base, stride, k, coef, cn, sum);
  else
    chunk_combine<2, T, false>(V + base, stride, k, coef, cn, sum);
  chunk_gather<2, T>(sum, red, r);
  double zn = 0.0;
  if (tid < cn) {
    const size_t e = base + tid;
    const double inv = d.sc[0], g = d.sc[1];
    const double ue = u[e];
    V[(size_t)k * stride + e] = (B)((ue - r[0]) * inv);
    zn = w[e] * inv - r[1] - g * ue;
    w[e] = zn;
  }
  const double s = chunk_sum<T>(zn * zn, sh);
  if (tid == 0) part[blockIdx.x] = s;
}

// rho = |w| (every work-group sums the partials in the same order; the
// first stores it), vnext = w / rho; beside them the last work-group rotates
// column givens_col of H (< 0: none) from Hraw.
__global__ __launch_bounds__(256) void k_lag_norm_scale(const double *__restrict__ part, int nchunk,
                                                        const double *__restrict__ w,
                                                        double *__restrict__ vnext, size_t len,
                                                        GmresDev d, int givens_col, double beta) {
  if (blockIdx.x == gridDim.x - 1) {
    if (givens_col >= 0) gmres_givens_raw(d, givens_col, beta);
    return;
  }
  __shared__ double sh[4], snorm;
  double s = 0.0;
  for (int c = threadIdx.x; c < nchunk; c += 256) s += part[c];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) {
    snorm = sqrt(s);
    if (blockIdx.x == 0 && len > 0) d.sc[2] = snorm;
  }
  __syncthreads();
  const double r = snorm;
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < len) vnext[e] = (r > 0.0) ? w[e] / r : 0.0;
}

// One work-group per vector sums its partials (strided, then a tree).
__global__ __launch_bounds__(256) void k_multidot_reduce(const double *__restrict__ part,
                                                         int nchunk, int nvec,
                                                         double *__restrict__ out,
                                                         int take_sqrt) {
  __shared__ double sh[4];
  const int i = blockIdx.x;
  double s = 0.0;
  for (int c = threadIdx.x; c < nchunk; c += 256) s += part[(size_t)c * nvec + i];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) out[i] = take_sqrt ? sqrt(s) : s;
}

__global__ void k_to_float(float *__restrict__ dst, const double *__restrict__ src, size_t len) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < len) dst[e] = (float)src[e];
}

__global__ void k_scale_by_inv(double *__restrict__ dst, const double *__restrict__ src,
                               const double *__restrict__ nrm, size_t len) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < len) {
    const double d = nrm[0];
    dst[e] = (d > 0.0) ? src[e] / d : 0.0;
  }
}

// dL/dkappa on cells: -1/(2^(d-1) h^2) sum_edges (lam_p - lam_q)(u_p - u_q).
__global__ void k_cell_gradient(const double *__restrict__ u, const double *__restrict__ lam,
                                const double *__restrict__ g, int dim, int n, int M, int ld,
                                double h, double *__restrict__ grad) {
  const size_t nc = (size_t)n + 1;
  const size_t ncell = (dim == 2) ? nc * nc : nc * nc * nc;
  const size_t cell = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= ncell) return;
  int c[3];
  if (dim == 2) {
    c[0] = (int)(cell / nc); c[1] = (int)(cell % nc); c[2] = 0;
  } else {
    c[0] = (int)(cell / (nc * nc)); c[1] = (int)((cell / nc) % nc); c[2] = (int)(cell % nc);
  }
  const size_t nb = (size_t)n + 2;
  // corner values of the cell: node c + o, o in {0,1}^dim
  double U[8], L[8];
  const int ncorner = 1 << dim;
  for (int o = 0; o < ncorner; ++o) {
    int q[3] = {c[0] + (o & 1), c[1] + ((o >> 1) & 1), dim == 3 ? c[2] + ((o >> 2) & 1) : 0};
    bool inside = true;
    for (int a = 0; a < dim; ++a) inside = inside && q[a] >= 1 && q[a] <= n;
    if (inside) {
      const size_t ip = (dim == 2) ? (size_t)(q[1] - 1) : (size_t)(q[1] - 1) * n + (q[2] - 1);
      U[o] = u[(size_t)(q[0] - 1) * M + ip];
      L[o] = lam[(size_t)(q[0] - 1) * ld + ip];
    } else {
      const size_t bidx = (dim == 2) ? (size_t)q[0] * nb + q[1]
                                     : ((size_t)q[0] * nb + q[1]) * nb + q[2];
      U[o] = g ? g[bidx] : 0.0;
      L[o] = 0.0;
    }
  }
  double s = 0.0;
  for (int o = 0; o < ncorner; ++o)
    for (int a = 0; a < dim; ++a)
      if (!((o >> a) & 1)) {
        const int o2 = o | (1 << a);
        s += (L[o] - L[o2]) * (U[o] - U[o2]);
      }
  grad[cell] = -s / ((double)(1 << (dim - 1)) * h * h);
}

__global__ void k_check_finite(const double *__restrict__ x, size_t len, double lo, int *bad) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < len) {
    const double v = x[e];
    if (!isfinite(v) || !(v > lo)) atomicOr(bad, 1);
  }
}

// Largest |x_e| into *out (bit pattern of a non-negative double, which
// orders like an unsigned integer; NaN entries are skipped).
__global__ void k_maxabs(const double *__restrict__ x, size_t len,
                         unsigned long long *__restrict__ out) {
  double v = 0.0;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < len;
       e += (size_t)gridDim.x * blockDim.x)
    v = fmax(v, fabs(x[e]));
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  if ((threadIdx.x & 63) == 0) atomicMax(out, (unsigned long long)__double_as_longlong(v));
}

inline unsigned nblk(size_t len, unsigned b = 256) { return (unsigned)((len + b - 1) / b); }

}  // namespace

void launch_setup_coef(const double *kappa, const double *c, const double *b, int dim, int n,
                       double h, double *coef, int *, hipStream_t s) {
  const size_t N = (dim == 2) ? (size_t)n * n : (size_t)n * n * n;
  hipLaunchKernelGGL(k_setup_coef, dim3(nblk(N)), dim3(256), 0, s, kappa, c, b[0], b[1], b[2],
                     dim, n, h, coef);
}

void launch_fill_couplings(const double *coef, int dim, int n, int M, int ld, double *Em,
                           double *Ep, hipStream_t s) {
  const size_t N = (size_t)M * n;
  hipLaunchKernelGGL(k_fill_couplings, dim3(nblk(ld), n + 2), dim3(256), 0, s, coef, n, M, ld,
                     N, Em, Ep);
  (void)dim;
}

void launch_residual(const double *coef, int dim, int n, int M, int ld, const double *f,
                     const double *g, const double *x, double *r, int transpose,
                     hipStream_t s) {
  const size_t N = (size_t)M * n;
  hipLaunchKernelGGL(k_residual, dim3(nblk(N)), dim3(256), 0, s, coef, dim, n, M, ld, f, g, x,
                     r, transpose);
}

void launch_pad(const double *src, double *dst, int rows, int M, int ld, hipStream_t s) {
  hipLaunchKernelGGL(k_pad, dim3(nblk((size_t)rows * ld)), dim3(256), 0, s, src, dst, rows, M,
                     ld);
}

void launch_unpad(const double *src, double *dst, int rows, int M, int ld, hipStream_t s) {
  hipLaunchKernelGGL(k_unpad, dim3(nblk((size_t)rows * M)), dim3(256), 0, s, src, dst, rows, M,
                     ld);
}

template <typename T>
void launch_gemv(const GemvJob *jobs, int njobs, int ld, int M, int transpose, double alpha,
                 double *partial, hipStream_t s) {
  if (njobs <= 0) return;
  const ProfSpan ps = prof_open(KK_GEMV);
  if (!transpose) {
    auto kern = sizeof(T) == 8           ? k_gemv_n_f64
                : gemv_wide(njobs, ld) ? k_gemv_n_f32<1024>
                                       : k_gemv_n_f32<512>;
    hipExtLaunchKernelGGL(kern, dim3(ld / kGemvRows, njobs), dim3(256), 0, s, ps.a, ps.b, 0, jobs,
                          ld, M, alpha);
  } else {
    const int nchunk = std::min(ld / 64, 64);  // 64 rows and more
    const int rpc = ld / nchunk;
    static_assert(kGemvChunk <= 64, "the partial sums fit the workspace");
    const bool rows = gemv_t_rows(njobs, ld, sizeof(T));
    const unsigned strips = nblk(ld);
    hipExtLaunchKernelGGL((rows ? k_gemv_t_part<T, true> : k_gemv_t_part<T, false>),
                          rows ? dim3(strips, nchunk, njobs) : dim3(nchunk, njobs, strips),
                          dim3(256), 2 * rpc * sizeof(double), s, ps.a, nullptr, 0, jobs, ld, M,
                          rpc, partial);
    hipExtLaunchKernelGGL(k_gemv_t_reduce, dim3(nblk(ld), njobs), dim3(256), 0, s, nullptr, ps.b,
                          0, jobs, ld, nchunk, partial, alpha);
  }
  // matrix bytes dominate: one or two M x M matrices per job (upper bound 1)
  prof_close(ps, KK_GEMV, (double)njobs * M * M * sizeof(T));
}
template <typename T>
void launch_gemv_many(const GemvJob *jobs, int njobs, int ld, int M, double alpha, int nv,
                      size_t vs, double *partial, hipStream_t s) {
  if (nv <= 1) {
    launch_gemv<T>(jobs, njobs, ld, M, 0, alpha, partial, s);
    return;
  }
  if (njobs <= 0) return;
  // one launch takes up to 16 vectors (the most ddst_solve_many allows)
  if (nv > 16) throw std::invalid_argument("launch_gemv_many: more than 16 vectors");
  const ProfSpan ps = prof_open(KK_GEMV_MANY);
  // 64 or 128 rows per work-group (ld % 128 == 0: whole work-groups and chunks)
  constexpr int H = 2;
  if (nv <= 4)
    hipExtLaunchKernelGGL((k_gemv_mfma<T, 4, H>), dim3(ld / 64, njobs), dim3(256 * H), 0, s, ps.a,
                          ps.b, 0, jobs, ld, alpha, nv, vs);
  else
    hipExtLaunchKernelGGL((k_gemv_mfma<T, 8, H>), dim3(ld / 128, njobs), dim3(512 * H), 0, s, ps.a,
                          ps.b, 0, jobs, ld, alpha, nv, vs);
  // one M x M matrix per job (interface jobs read two: a lower bound)
  prof_close(ps, KK_GEMV_MANY, (double)njobs * M * M * sizeof(T));
}
template void launch_gemv_many<float>(const GemvJob *, int, int, int, double, int, size_t,
                                      double *, hipStream_t);
template void launch_gemv_many<double>(const GemvJob *, int, int, int, double, int, size_t,
                                       double *, hipStream_t);
template void launch_gemv<float>(const GemvJob *, int, int, int, int, double, double *,
                                 hipStream_t);
template void launch_gemv<double>(const GemvJob *, int, int, int, int, double, double *,
                                  hipStream_t);

void launch_interface_rhs(const double *vol, const double *Zl, const double *Zr,
                          const double *Ea, const double *Eb, int n_ds, int m, int ld,
                          int a_off, int b_off, double *out, hipStream_t s) {
  hipLaunchKernelGGL(k_interface_rhs, dim3(nblk(ld), n_ds), dim3(256), 0, s, vol, Zl, Zr, Ea,
                     Eb, n_ds, m, ld, a_off, b_off, out);
}

void launch_copy_planes(const double *src, int src_stride, int src_off, double *dst,
                        int dst_stride, int dst_off, int count, int ld, int M, hipStream_t s) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_copy_planes, dim3(nblk(ld), count), dim3(256), 0, s, src, src_stride,
                     src_off, dst, dst_stride, dst_off, ld, M);
}

void launch_axpy(double *y, const double *x, double a, size_t len, hipStream_t s) {
  hipLaunchKernelGGL(k_axpy, dim3(nblk(len)), dim3(256), 0, s, y, x, a, len);
}

void launch_fill(double *y, double v, size_t len, hipStream_t s) {
  if (len == 0) return;
  hipLaunchKernelGGL(k_fill, dim3(nblk(len)), dim3(256), 0, s, y, v, len);
}

namespace {
// f(std::integral_constant<int, T>) for vectors of len entries
template <typename F> void with_dot_width(size_t len, F f) {
  if (len % kTile) throw std::invalid_argument("Krylov passes: length not a multiple of 128");
  switch (dot_width(len)) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    default: return f(std::integral_constant<int, 4>{});
  }
}
template <typename B>
void update_dots(double *w, const B *V, size_t stride, int nvec, const double *h, double sign,
                 size_t len, int ndot, double *part, hipStream_t s) {
  with_dot_width(len, [&](auto t) {
    constexpr int T = decltype(t)::value;
    hipLaunchKernelGGL((k_mgs_update_dots<B, T>), dim3(nblk(len, 64 * T)), dim3(64 * kDotWaves), 0,
                       s, w, V, stride, nvec, h, sign, len, ndot, part);
  });
}
}  // namespace

template <typename B>
void launch_mgs_update(double *w, const B *V, size_t stride, int nvec, const double *h,
                       double sign, size_t len, hipStream_t s) {
  if (len == 0 || nvec <= 0) return;
  update_dots<B>(w, V, stride, nvec, h, sign, len, -1, nullptr, s);
}
template void launch_mgs_update<double>(double *, const double *, size_t, int, const double *,
                                        double, size_t, hipStream_t);
template void launch_mgs_update<float>(double *, const float *, size_t, int, const double *,
                                       double, size_t, hipStream_t);

void launch_to_float(float *dst, const double *src, size_t len, hipStream_t s) {
  hipLaunchKernelGGL(k_to_float, dim3(nblk(len)), dim3(256), 0, s, dst, src, len);
}

template <typename B>
void launch_arnoldi_step(const B *V, size_t stride, int k, double *w, size_t len, double *hd,
                         double *vnext, float *vslot, double *part, GmresDev gd, double beta,
                         hipStream_t s) {
  const int nvec = k + 1;
  const int nchunk = (int)dot_chunks(len);
  auto reduce = [&](double *out) {
    hipLaunchKernelGGL(k_multidot_reduce, dim3(nvec), dim3(256), 0, s, (const double *)part,
                       nchunk, nvec, out, 0);
  };
  // pass 1: h1 = V^T w
  update_dots<B>(w, V, stride, 0, nullptr, 0.0, len, nvec, part, s);
  reduce(hd);
  // w -= V h1, then pass 2 partials
  update_dots<B>(w, V, stride, nvec, hd, -1.0, len, nvec, part, s);
  reduce(hd + nvec);
  // w -= V h2, then partial squared norms; v_next = w / |w| and the rotations
  update_dots<B>(w, V, stride, nvec, hd + nvec, -1.0, len, 0, part, s);
  hipLaunchKernelGGL(k_norm_scale_givens, dim3(nblk(len)), dim3(256), 0, s,
                     (const double *)part, nchunk, hd, (const double *)w, vnext, vslot, len, gd,
                     k, beta);
}
template void launch_arnoldi_step<double>(const double *, size_t, int, double *, size_t,
                                          double *, double *, float *, double *, GmresDev,
                                          double, hipStream_t);
template void launch_arnoldi_step<float>(const float *, size_t, int, double *, size_t, double *,
                                         double *, float *, double *, GmresDev, double,
                                         hipStream_t);

template <typename B>
void launch_arnoldi_lagged(B *V, size_t stride, int k, const double *u, double *w,
                           double *unext, size_t len, double *part, GmresDev gd, double beta,
                           int col_final, int finalize_only, hipStream_t s) {
  const int m = k + 1;
  const int nlchunk = (int)nblk(len, kLagChunk);
  const int ngroup = std::max((m - 1 + kDotRound - 1) / kDotRound, 1);
  hipLaunchKernelGGL(k_lag_dots<B>, dim3(nlchunk, ngroup), dim3(64 * kDotWaves), 0, s,
                     (const B *)V, stride, m, u,
                     finalize_only ? (const double *)nullptr : (const double *)w, len, part);
  hipLaunchKernelGGL(k_multidot_reduce, dim3(2 * m), dim3(256), 0, s, (const double *)part,
                     nlchunk, 2 * m, gd.dA, 0);
  hipLaunchKernelGGL(k_lag_hmul, dim3((m + 3) / 4), dim3(256), 0, s, gd, k, col_final);
  const int gcol = (k >= 1 && !col_final) ? k - 1 : -1;
  if (finalize_only) {
    hipLaunchKernelGGL(k_lag_norm_scale, dim3(1), dim3(256), 0, s, (const double *)part, 0,
                       (const double *)nullptr, (double *)nullptr, (size_t)0, gd, gcol, beta);
    return;
  }
  hipLaunchKernelGGL(k_lag_coef, dim3(1), dim3(256), 0, s, gd, k);
  with_dot_width(len, [&](auto t) {
    constexpr int T = decltype(t)::value;
    hipLaunchKernelGGL((k_lag_update<B, T>), dim3(nblk(len, 64 * T)), dim3(64 * kDotWaves), 0, s, V,
                       stride, k, u, w, len, gd, part);
  });
  hipLaunchKernelGGL(k_lag_norm_scale, dim3(nblk(len) + 1), dim3(256), 0, s, (const double *)part,
                     (int)dot_chunks(len), (const double *)w, unext, len, gd, gcol, beta);
}
template void launch_arnoldi_lagged<double>(double *, size_t, int, const double *, double *,
                                            double *, size_t, double *, GmresDev, double, int,
                                            int, hipStream_t);
template void launch_arnoldi_lagged<float>(float *, size_t, int, const double *, double *,
                                           double *, size_t, double *, GmresDev, double, int,
                                           int, hipStream_t);

void launch_norm(const double *w, size_t len, double *out, double *part, hipStream_t s) {
  const int nchunk = (int)nblk(len);
  hipLaunchKernelGGL(k_norm_part, dim3(nchunk), dim3(256), 0, s, w, len, part);
  hipLaunchKernelGGL(k_multidot_reduce, dim3(1), dim3(256), 0, s, part, nchunk, 1, out, 1);
}

namespace {
// Back substitution R y = g, 64 columns at a time from the last: the first
// wavefront solves their triangle, row j in lane j, with no barrier between the
// unknowns, then every thread removes the 64 from its rows above (one column
// and two barriers at a time: 1.56 ms at 1017 columns).
__global__ __launch_bounds__(256) void k_gmres_backsub(GmresDev d, int k) {
  constexpr int NB = 64;
  __shared__ double ys[NB];
  for (int i = threadIdx.x; i < k; i += blockDim.x) d.y[i] = d.g[i];
  __syncthreads();
  for (int j0 = (k - 1) / NB * NB; j0 >= 0; j0 -= NB) {
    const int nb = min(NB, k - j0);
    if (threadIdx.x < NB) {
      const int l = threadIdx.x, i = j0 + l;
      double y = l < nb ? d.y[i] : 0.0, R[NB];  // R[c]: entry (i, j0 + c)
#pragma unroll
      for (int c = 0; c < NB; ++c)
        R[c] = c < nb && l <= c ? d.H[gmres_hoff(j0 + c) + i] : 0.0;
#pragma unroll
      for (int c = NB - 1; c >= 0; --c)
        if (c < nb) {
          const double piv = __shfl(R[c], c), yc = __shfl(y, c);
          const double v = piv != 0.0 ? yc / piv : 0.0;
          y = l == c ? v : y - R[c] * v;
        }
      ys[l] = y;
      if (l < nb) d.y[i] = y;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < j0; i += blockDim.x) {
      double s = 0.0;
#pragma unroll 8
      for (int c = 0; c < nb; ++c) s += d.H[gmres_hoff(j0 + c) + i] * ys[c];
      d.y[i] -= s;
    }
    __syncthreads();
  }
}
}  // namespace


template <typename B>
void launch_gmres_solution(GmresDev d, int k, double *x, const B *V, size_t len, hipStream_t s) {
  if (k <= 0) return;
  hipLaunchKernelGGL(k_gmres_backsub, dim3(1), dim3(256), 0, s, d, k);
  launch_mgs_update<B>(x, V, len, k, d.y, 1.0, len, s);
}
template void launch_gmres_solution<double>(GmresDev, int, double *, const double *, size_t,
                                            hipStream_t);
template void launch_gmres_solution<float>(GmresDev, int, double *, const float *, size_t,
                                           hipStream_t);

void launch_scale_by_inv(double *dst, const double *src, const double *nrm, size_t len,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_scale_by_inv, dim3(nblk(len)), dim3(256), 0, s, dst, src, nrm, len);
}

void launch_cell_gradient(const double *u, const double *lam, const double *g, int dim, int n,
                          int M, int ld, double h, double *grad, hipStream_t s) {
  const size_t nc = (size_t)n + 1;
  const size_t ncell = (dim == 2) ? nc * nc : nc * nc * nc;
  hipLaunchKernelGGL(k_cell_gradient, dim3(nblk(ncell)), dim3(256), 0, s, u, lam, g, dim, n, M,
                     ld, h, grad);
}

void launch_maxabs(const double *x, size_t len, unsigned long long *out, hipStream_t s) {
  if (len == 0) return;
  hipLaunchKernelGGL(k_maxabs, dim3(std::min<unsigned>(nblk(len), 1024)), dim3(256), 0, s, x, len,
                     out);
}

void launch_check_finite(const double *x, size_t len, double lo, int *bad, hipStream_t s) {
  if (len == 0) return;
  hipLaunchKernelGGL(k_check_finite, dim3(nblk(len)), dim3(256), 0, s, x, len, lo, bad);
}

}  // namespace ddst

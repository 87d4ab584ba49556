// FP32 tile products of 512-thread work-groups on the BF16 matrix cores.
//
// Eight wavefronts in WR rows form one output tile; each owns a 128 x 64 piece
// of it (4 x 2 tiles of v_mfma_f32_32x32x16_bf16), so that WR chooses between
// tiles of 256 x 256, tiles of 512 x 128, as tall as an outer elimination block
// (they may be written over their right operand), and of 128 x 512, as wide
// as one (over their left operand).  Operands are split into three BF16 parts
// and multiplied by six BF16 products (Split3 in dense.hip says why).
//
// Why this shape.  Per 16-deep stage a 256 x 256 tile splits 8192 entries for
// 2^20 multiply-adds, half of what four 128 x 128 tiles split, and its fragment
// reads take half the LDS bandwidth.  Stages are double buffered in LDS with
// one barrier each, their loads issued two stages before they are stored; a
// stage is split between the MFMAs of the stage before it.  Batched product
// of 12 x 4096^3: 177 TFLOP/s with 128 x 128 tiles, 218 with these (235 and
// 291 on matrices of zeros: what bounds both is power, the clock falls to 1.6
// GHz; the library's 8192^3 BF16 product reaches 1.14 PFLOP/s on the same
// card, these 1.31 PFLOP/s of BF16 products).  Where the tiles are few or half
// empty the 128 x 128 ones are the better (gemm_big_tiles, rules.h).
#pragma once

#include "internal.h"

namespace ddst {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// One operand of a tile product: entry (r, k) of its R x K block is
// p[r * ld + k] when the k index is contiguous, else p[k * ld + r] (r: rows of
// the left operand, columns of the right one).  rows: how many r may be
// read (beyond them the last is read again; those results are not used).
struct Opnd {
  const float *p;
  int ld;
  int rows;
  bool kcontig;
};

// Accesses at a byte offset below 4 GiB from a pointer that the whole
// work-group shares: the pointer stays in scalar registers, and stepping it
// costs no vector instruction.
template <typename V> __device__ __forceinline__ V at(const void *base, unsigned off) {
  typedef __attribute__((address_space(1))) const char gchar;
  typedef __attribute__((address_space(1))) const V gv;
  return *(gv *)((gchar *)base + off);
}
template <typename V> __device__ __forceinline__ void put(void *base, unsigned off, V v) {
  typedef __attribute__((address_space(1))) char gchar;
  typedef __attribute__((address_space(1))) V gv;
  *(gv *)((gchar *)base + off) = v;
}

// Stage of one operand (R rows, 16 k).  load: this thread's entries into
// registers; split: the p-th pair of them, to LDS with the last pair of an
// item; frag: an MFMA's operand fragments.  LDS: three parts, each two halves
// of eight k with 16 bytes per row, so that a fragment read (32 consecutive
// rows of one half) is 512 contiguous bytes; the second half is shifted by 64
// bytes, so that the stores of k-contiguous operands (lanes alternate between
// halves) meet different banks.
template <int R> struct Stage {
  static constexpr int half = R * 16 + 64;
  static constexpr int part = 2 * half;
  static constexpr int bytes = 3 * part;
  static constexpr int NE = R / 32;           // entries per thread
  static constexpr int IE = NE < 8 ? NE : 8;  // entries per item (consecutive k)
  static constexpr int NI = NE / IE;
  static constexpr int NP = NE / 2;  // pairs per thread
  float x[NI][IE];
  unsigned s[3][IE / 2];  // parts of the item being split

  __device__ __forceinline__ static void item(int i, bool kcontig, int &r, int &k) {
    const int q = threadIdx.x + 512 * i;
    r = kcontig ? q / (16 / IE) : q % R;
    k = IE * (kcontig ? q % (16 / IE) : q / R);
  }
  // byte offsets of this thread's items
  __device__ __forceinline__ static void offsets(const Opnd &o, unsigned (&off)[NI]) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      int r, k;
      item(i, o.kcontig, r, k);
      r = min(r, o.rows - 1);
      off[i] = 4u * (o.kcontig ? (unsigned)r * o.ld + k : (unsigned)k * o.ld + r);
    }
  }
  __device__ __forceinline__ void load(const Opnd &o, const unsigned (&off)[NI], int k0) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (o.kcontig) {
#pragma unroll
        for (int h = 0; h < IE / 4; ++h) {
          const f32x4_t a = at<f32x4_t>(o.p + k0 + 4 * h, off[i]);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[i][4 * h + e] = a[e];
        }
      } else {
#pragma unroll
        for (int e = 0; e < IE; ++e) x[i][e] = at<float>(o.p + (size_t)(k0 + e) * o.ld, off[i]);
      }
    }
  }
  // pair p of this thread's entries: x = h + m + l, two of each in one register
  __device__ __forceinline__ void split(unsigned char *st, bool kcontig, int p) {
    auto pk = [](float a, float b) {
      const f32x2_t v = {a, b};
      return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2_t));
    };
    const int i = p / (IE / 2), j = p % (IE / 2);
    const float x0 = x[i][2 * j], x1 = x[i][2 * j + 1];
    const unsigned hp = pk(x0, x1);
    const float r0 = x0 - __uint_as_float(hp << 16);
    const float r1 = x1 - __uint_as_float(hp & 0xffff0000u);
    const unsigned mp = pk(r0, r1);
    s[0][j] = hp;
    s[1][j] = mp;
    s[2][j] = pk(r0 - __uint_as_float(mp << 16), r1 - __uint_as_float(mp & 0xffff0000u));
    if (j < IE / 2 - 1) return;
    int r, k;
    item(i, kcontig, r, k);
    unsigned char *d = st + (k >> 3) * half + r * 16 + 2 * (k & 7);
    typedef unsigned vec __attribute__((ext_vector_type(IE / 2)));
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      vec v;
#pragma unroll
      for (int e = 0; e < IE / 2; ++e) v[e] = s[q][e];
      *reinterpret_cast<vec *>(d + q * part) = v;
    }
  }
  // fragment of the 32 rows from r0: lane l holds row l % 32, k = 8 (l / 32) + 0..7
  __device__ __forceinline__ static void frag(const unsigned char *st, int r0, bf16x8_t (&f)[3]) {
    const int l = threadIdx.x & 63;
    const unsigned char *d = st + (l >> 5) * half + (r0 + (l & 31)) * 16;
#pragma unroll
    for (int p = 0; p < 3; ++p) f[p] = *reinterpret_cast<const bf16x8_t *>(d + p * part);
  }
};

template <int WR> struct WgTile {
  static constexpr int WC = 8 / WR;
  static constexpr int NI = 4, NJ = 2, NR = 16, E = 32;  // a piece: NI x NJ tiles, E x E each
  static constexpr int TM = NI * E * WR, TN = NJ * E * WC;
  using SA = Stage<TM>;
  using SB = Stage<TN>;
  static constexpr int stage = SA::bytes + SB::bytes;
  static constexpr int lds = 2 * stage;
  static_assert(lds <= 160 * 1024, "two stages fit the LDS");
  f32x16 v[NI][NJ];

  // first row / column of this wavefront's piece; for four columns their order
  // is rotated for the second half of the wavefronts, so that a tile with few
  // valid columns still loads all four SIMDs (wavefronts w and w + 4 share one)
  __device__ __forceinline__ static int row0() { return (int)(threadIdx.x >> 6) / WC * NI * E; }
  __device__ __forceinline__ static int col0() {
    const int w = threadIdx.x >> 6;
    return ((w % WC) ^ (WC == 4 && w >= 4 ? 2 : 0)) * NJ * E;
  }
  // row of entry (i, j, r) in the tile, column of entry (i, 0, r)
  __device__ __forceinline__ static int row(int i, int r) {
    return row0() + E * i + 8 * (r >> 2) + 4 * ((threadIdx.x & 63) >> 5) + (r & 3);
  }
  __device__ __forceinline__ static int col() { return col0() + (threadIdx.x & 31); }
  // byte offset of entry (i, 0, r); entry (i, j, r) follows E j entries later
  __device__ __forceinline__ static unsigned offset(int ld, int i, int r) {
    return 4u * (unsigned)(row(i, r) * ld + col());
  }

  // X[row, col] += sg * v on the first `rows` x `cols` entries.  Whole tiles
  // read a row of MFMA tiles while the previous one is written: entry by entry
  // (load, add, store) this took 60 us of a 155 us launch.
  __device__ __forceinline__ void add_to(float *X, int ld, float sg, int rows, int cols) const {
    if (rows >= TM && cols >= TN) {
      float d[2][NR][NJ];
      auto load = [&](int i, float (&o)[NR][NJ]) {
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int j = 0; j < NJ; ++j) o[r][j] = at<float>(X + E * j, offset(ld, i, r));
      };
      load(0, d[0]);
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        if (i + 1 < NI) load(i + 1, d[(i + 1) & 1]);
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            put<float>(X + E * j, offset(ld, i, r), d[i & 1][r][j] + sg * v[i][j][r]);
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          if (row(i, r) < rows && col() + E * j < cols) {
            const unsigned o = offset(ld, i, r);
            put<float>(X + E * j, o, at<float>(X + E * j, o) + sg * v[i][j][r]);
          }
  }
  // X[row, col] = sg * rs[row] * v on the first `rows` x `cols` entries (rs
  // null: 1)
  __device__ __forceinline__ void put_to(float *X, int ld, float sg, const double *rs, int rows,
                                         int cols) const {
    const bool whole = rows >= TM && cols >= TN;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int rr = row(i, r);
        if (!whole && rr >= rows) continue;
        const unsigned o = offset(ld, i, r);
        const float f = rs ? sg * (float)at<double>(rs, 8u * rr) : sg;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          if (whole || col() + E * j < cols) put<float>(X + E * j, o, f * v[i][j][r]);
      }
  }

  // the six products of one 32 x 32 tile and 16 k, smallest first
  __device__ __forceinline__ static f32x16 six(const bf16x8_t (&a)[3], const bf16x8_t (&b)[3],
                                               f32x16 c) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[2], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], c, 0, 0, 0);
  }

  // FULL false: only the first ni x nj MFMA tiles of this wavefront's piece
  template <bool FULL>
  __device__ __forceinline__ void run(const Opnd &A, const Opnd &B, int K, unsigned char *smem,
                                      int ni, int nj) {
    const int nk = K / 16;
    const int r0 = row0(), c0 = col0();
    unsigned oa[SA::NI], ob[SB::NI];
    SA::offsets(A, oa);
    SB::offsets(B, ob);
    SA xa[2];
    SB xb[2];
    // stages past the end load the last one again, and are never used
    auto load = [&](int t, int q) {
      const int k0 = 16 * min(t, nk - 1);
      xa[q].load(A, oa, k0);
      xb[q].load(B, ob, k0);
    };
    // part c of 8 of taking the registers q to stage t's buffer
    auto produce = [&](int t, int q, int c) {
      unsigned char *st = smem + (t & 1) * stage;
      constexpr int NP = SA::NP + SB::NP, PER = (NP + 7) / 8;
#pragma unroll
      for (int p = PER * c; p < PER * c + PER; ++p) {
        if (p < SA::NP)
          xa[q].split(st, A.kcontig, p);
        else if (p < NP)
          xb[q].split(st + SA::bytes, B.kcontig, p - SA::NP);
      }
    };
    // Stage t's products; between those of two MFMA tiles (6 x 32 cycles) an
    // eighth of the next stage is split (from registers q), and stays there:
    // left to itself the compiler splits after all of them, when no wavefront
    // has MFMAs to run.
    auto step = [&](int t, int q) {
      const unsigned char *sa = smem + (t & 1) * stage, *sb = sa + SA::bytes;
      bf16x8_t fb[NJ][3], fa[2][3];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (FULL || j < nj) SB::frag(sb, c0 + E * j, fb[j]);
      SA::frag(sa, r0, fa[0]);
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        if (i + 1 < NI && (FULL || i + 1 < ni)) SA::frag(sa, r0 + E * (i + 1), fa[(i + 1) & 1]);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          if (FULL || (i < ni && j < nj)) v[i][j] = six(fa[i & 1], fb[j], v[i][j]);
          produce(t + 1, q, NJ * i + j);  // the other buffer was read in the previous stage
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      load(t + 3, q);
      __syncthreads();
    };
    load(0, 0);
    load(1, 1);
#pragma unroll
    for (int c = 0; c < 8; ++c) produce(0, 0, c);
    load(2, 0);
    __syncthreads();
#pragma unroll 1
    for (int t = 0; t < nk; t += 2) {
      step(t, 1);
      if (t + 1 < nk) step(t + 1, 0);
    }
  }

  // v = A[0:TM, 0:K] B[0:K, 0:TN]; K a positive multiple of 16.  MFMA tiles that
  // begin past valid_rows or valid_cols are skipped and stay zero.  Ends with
  // a barrier: every read of A and B that counts is done, the LDS is free.
  __device__ __forceinline__ void product(const Opnd &A, const Opnd &B, int K, int valid_rows,
                                          int valid_cols, unsigned char *smem) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < NR; ++r) v[i][j][r] = 0.f;
    // the branch is the same for the whole work-group: the loops hold barriers
    if (valid_rows >= TM && valid_cols >= TN) {
      run<true>(A, B, K, smem, NI, NJ);
    } else {
      const int ni = __builtin_amdgcn_readfirstlane(
          min(NI, max(0, (valid_rows - row0() + E - 1) / E)));
      const int nj = __builtin_amdgcn_readfirstlane(
          min(NJ, max(0, (valid_cols - col0() + E - 1) / E)));
      run<false>(A, B, K, smem, ni, nj);
    }
  }
};

}  // namespace
}  // namespace ddst

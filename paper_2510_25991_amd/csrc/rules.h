// Sizes and variants that the host chooses by the shape of a call.  Plain C++
// (no HIP), so that the rules are checked without a GPU
// (tests/test_dispatch_rules.py).
#pragma once

#include <algorithm>
#include <cstddef>

namespace ddst {

// ---- passes over a Krylov basis ---------------------------------------------
// They take chunks of 64 dot_width entries: 64, 128 or 256, the most that leave
// one per CU.
constexpr size_t kDotChunks = 256;
inline int dot_width(size_t len) {
  return len >= 64 * 4 * kDotChunks ? 4 : len >= 64 * 2 * kDotChunks ? 2 : 1;
}
inline size_t dot_chunks(size_t len) {
  const size_t c = 64 * (size_t)dot_width(len);
  return (len + c - 1) / c;
}
// Doubles of workspace for the partial sums of nvec products over vectors of
// up to len entries.  The number of chunks is not monotone (32767 entries: 512,
// 65536: 256), so the most of all shorter lengths counts: chunks of 64 and 128
// entries number 2 kDotChunks at most, those of 256 grow with the length.
inline size_t dots_part_len(size_t len, int nvec) {
  const size_t most = std::min((len + 63) / 64, 2 * kDotChunks);
  return std::max(dot_chunks(len), most) * (size_t)nvec;
}

// ---- FP32 batched products -----------------------------------------------------
// Whether njobs products of ld x ld matrices take 256 x 256 tiles (one
// work-group a CU) or 128 x 128 ones.  Both take the same rows and columns;
// what decides is how many CUs have a tile, and the halves of the last tiles
// that an odd multiple of 128 leaves empty.  us, 256 x 256 against 128 x 128:
//   16 x 1024   (256 tiles)   162  178        33 x 1024  (528)    445  389
//   60 x 1024   (960)         628  668        65 x 1024 (1040)    755  754
//   188 x 1024 (3008)        1993 2143        14 x 896   (224)    139  152
//   900 x 128   (900)          87   41        225 x 384  (900)    253  166
//   100 x 640   (900)         350  320        94 x 896  (1504)    774  715
//   36 x 1152   (900)         618  591        25 x 1408  (900)    789  742
//   21 x 1664  (1029)        1024 1014        16 x 1920 (1024)   1130 1227
//   1 x 1024     (16)         129   63        4 x 256      (4)     43   21
// Between 256 and 900 tiles the last round of work-groups decides; in a build
// other launches run beside it: symmetric 1023^2 on 32 slabs (30 chains, 480
// tiles) 57.8 ms with either, on 64 (992) 65.5 against 69.0 with 128 x 128.
constexpr int kGemmMany = 900;     // 256 x 256 tiles from which
constexpr int kGemmOddRows = 1664; // rows from which an odd multiple of 128
inline bool gemm_big_tiles(int njobs, int ld) {
  const int nt = (ld + 255) / 256;
  return (ld % 256 == 0 || ld >= kGemmOddRows) && (long long)njobs * nt * nt >= kGemmMany;
}

// ---- Gauss-Jordan inversion ---------------------------------------------------
// Whether nmat matrices of ld rows (element size esz) are eliminated in outer
// blocks of 512 rows.  An outer block's products take 256 x 256 tiles at the
// matrix cores' rate, where a rank-128 update is bound by its traffic, but they
// put a second elimination in series: they pay where the tiles fill the chip
// several times over, so the rule counts the tiles of all matrices (half of
// them where the symmetric elimination touches the lower triangle only).
// Builds, ms:                           tiles   one level   outer blocks
//   2D 1151, 4 slabs (7 matrices)         142       205          315
//   2D 1535, 4 slabs                      252       383          601
//   2D 1023, 16 slabs                     496        75.1         89.8
//   2D 1023, 32 slabs, symmetric          503        53.4         57.7
//   2D 1791, 8 slabs                      734       563          562
//   3D 47, 12 slabs, symmetric            856        21.3         21.5
//   2D 1407, 16 slabs                     936       237          222
//   2D 2047, 8 slabs                      959       949          828
//   2D 1023, 32 slabs                    1006        69.5         64.4
//   2D 1023, 64 slabs, symmetric         1014        51.0         48.5
//   2D 1535, 16 slabs                    1115       317          294
//   2D 1151, 32 slabs                    1274       107          110
//   3D 63, 8 slabs, symmetric            1803       117           95.0
//   2D 1023, 64 slabs                    2028        64.7         58.5
// Below 896 rows the second block is half a block or less: 767 on 64 slabs
// (1140 tiles) 25.6 and 25.8 ms, 639 on 128 (1589) 14.6 and 14.5.
// FP64: one level, whose update of rank 128 takes as long on the matrix cores
// as in memory.
constexpr int kOuterRows = 896;    // rows (with padding) from which
constexpr int kOuterTiles = 900;   // 256 x 256 tiles from which
inline bool outer_blocks(int nmat, int ld, size_t esz, bool sym) {
  const double side = ld / 256.0;
  return esz == 4 && ld >= kOuterRows && nmat * side * side >= (sym ? 2 : 1) * kOuterTiles;
}

// Whether the pivots' work-groups (one per matrix) share CUs two by two: where
// there are more of them than CUs, a second round takes as long as the first.
// With fewer, the registers that this costs buy nothing (builds of 15 to 255
// matrices within 2% either way).
constexpr int kCus = 256;
inline bool pivots_share_cus(int nmat) { return nmat > kCus; }

// ---- sampled (HBS) product ------------------------------------------------------
// Most rows that a group of lanes of the product's kernels takes at a time, for
// nodes of up to `rows` rows.  Four rows' loads pay for their registers (more
// than the 64 that leave eight wavefronts on a SIMD) where a group has that many
// rows.  us, up to four against up to two: leaves of 128 (3D 31, rank 64) BF16
// 45.0 and 50.3, FP32 46.6 and 55.6, FP64 62.4 and 62.8, transposed 56.8 and
// 61.7; leaves of 64 (2D 511 on 32 slabs, rank 32) 32.6 and 33.0, 34.3 and 35.0,
// 39.6 and 38.4; of 32 (2D 1023 on 64, rank 16) 66.4 and 63.5, 67.1 and 64.2,
// 73.2 and 69.7.  (Four rows always, also where a group has one: 75.9, 74.8 and
// 89.4; one row at a time: 63.4, 64.0 and 70.5, leaves of 128 80.5 to 99.4.)
inline int hbs_rows_in_flight(int rows) { return rows > 64 ? 4 : 2; }

// ---- matrix-vector products ----------------------------------------------------
// Whether an FP32 launch over njobs matrices takes 1024 columns of its two rows
// at a time instead of 512.  Where a launch is long, its last round of
// work-groups counts for less than the loads in flight of each wavefront.  us
// with 512 and 1024 columns, by bytes of the matrices (planes of a sweep):
//   2D 511 on 64 slabs    67 MB   19.7 20.2    3D 47 on 6    127 MB   25.2 26.4
//   2D 1023 on 32 slabs  134 MB   29.2 28.8    3D 63 on 4    252 MB   48.6 48.1
//   2D 1023 on 64 slabs  268 MB   75.8 69.3    2D 2047 on 16 268 MB   50.3 47.0
//   2D 1023 on 128 slabs 537 MB    164  160
// FP64, twice the loads per column: 152 and 149 at 537 MB, 95.5 and 96.5 at 2047
// on 16 slabs, so 512.
// Four rows and 1024 columns, three wavefronts per SIMD, against this rule's two
// rows: sweeps of 2D 1023 on 64 slabs 72 and 69 us, 2047 on 16 51 and 47, 3D 63 on 4
// 59 and 47; large interface products are faster so (2D 1023 on 128 slabs 171 and
// 179, on 512 slabs 669 and 697).
constexpr double kGemvLargeBytes = 192e6;
inline bool gemv_wide(int njobs, int ld) {
  return 4.0 * njobs * ld * ld >= kGemvLargeBytes;
}
// Whether a transposed launch (partial sums over strips of 256 columns and chunks
// of rows) runs strip by strip over whole rows, or through all chunks of all
// matrices for the first strip, then for the next.  The second way reads a
// quarter of every row at a time, which matters where the matrices come from
// memory rather than from the last-level cache (256 MB).  us, both passes,
// sweeps, strips of all chunks first against whole rows:
//   FP32 2D 1023 on 16 slabs   67 MB   20.6 21.6   FP64 511 on 64   134 MB   45.1 46.5
//   FP32 2D 1023 on 32 slabs  134 MB   37.1 37.5   FP64 1023 on 32  268 MB   81.5 75.4
//   FP32 3D 63 on 4 slabs     252 MB   71.6 68.3   FP64 767 on 64   302 MB    111  108
//   FP32 2D 2047 on 16 slabs  268 MB   70.9 64.5   FP64 1023 on 64  537 MB    208  173
//   FP32 2D 1023 on 128 slabs 537 MB    210  191   FP64 1023 on 128 1.1 GB    405  358
inline bool gemv_t_rows(int njobs, int ld, size_t esz) {
  return (double)esz * njobs * ld * ld >= kGemvLargeBytes;
}

}  // namespace ddst

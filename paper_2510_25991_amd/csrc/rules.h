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

}  // namespace ddst

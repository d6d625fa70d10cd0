// Dynamic LDS sizes that follow a call's data, rounded up to a few steps each
// (host code only).  A kernel's residency is looked up once per (kernel, size)
// and kept in a table that never shrinks, so a size of every query length and
// vocabulary would fill it; and the size a kernel is allowed is set to its
// largest, not to the launch's, because contexts on other threads set it too.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace lcemd {

// query words that the bf16 tables' layout is made for: the batch's longest
// query, in steps of 64 (a pass's words).  max_words: a multiple of 64.
inline int bf16_layout_words(int hmax, int max_words) {
  const int h = (hmax + 63) / 64 * 64;
  return h < max_words ? h : max_words;
}

// bytes of a workgroup that owns its CU's LDS, in steps of 16 KB
inline size_t lds_launch_bytes(size_t bytes, size_t max_bytes) {
  constexpr size_t kStep = 16 * 1024;
  const size_t b = (bytes + kStep - 1) / kStep * kStep;
  return b < max_bytes ? b : max_bytes;
}

}  // namespace lcemd

// Slices of a launch: a launch counts its threads in 32 bits, so a grid of
// more than 2^32 - 1 of them is issued in several.
#pragma once

#include <cstdint>

namespace stp {

// Most workgroups of `threads` threads that one launch takes.
constexpr int64_t max_blocks(int threads) { return INT64_C(0xffffffff) / threads; }

// Calls f(first, count) for consecutive slices of `blocks` workgroups of
// `threads` threads until it returns something other than `ok`; returns the last result.
template <class Result, class F>
Result for_slices(int64_t blocks, int threads, Result ok, F&& f) {
  const int64_t most = max_blocks(threads);
  for (int64_t first = 0; first < blocks; first += most) {
    const Result r = f(first, static_cast<unsigned>(blocks - first < most ? blocks - first : most));
    if (r != ok) return r;
  }
  return ok;
}

}  // namespace stp

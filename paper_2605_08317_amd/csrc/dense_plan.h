// What decides the form of the uncompressed step's launches, as host code that needs no HIP header.
#pragma once

#include <cstddef>
#include <cstdint>
#include <initializer_list>

namespace rdkv {

// bytes at an address
struct Span {
  const void* at;
  size_t bytes;
};
inline bool overlap(const Span& a, const Span& b) {
  const uintptr_t a0 = reinterpret_cast<uintptr_t>(a.at), b0 = reinterpret_cast<uintptr_t>(b.at);
  return a.bytes > 0 && b.bytes > 0 && a0 < b0 + b.bytes && b0 < a0 + a.bytes;
}

// Whether the launch may write its outputs before all of it has read its inputs, as it does where it merges its own partials: an item's
// rows and log-sum-exps are written (and its rows hold the chunks' tags before that) while workgroups of other items have not started.
// A second launch writes them when everything has been read (of up to kDenseMaxSeqs sequences): there a caller may have any of them in
// an input's memory.
inline bool dense_outputs_apart(const Span& k, const Span& v, const Span& q, const Span& out, const Span& lse) {
  for (const Span& o : {out, lse})
    for (const Span& in : {k, v, q})
      if (overlap(o, in)) return false;
  return true;
}

}  // namespace rdkv

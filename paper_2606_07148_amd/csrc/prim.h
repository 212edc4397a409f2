// Device-wide primitives of the build and the export, called on rocPRIM
// directly: radix sort of 64-bit keys, exclusive prefix sum of 64-bit
// counts.  Each follows rocPRIM's two-call protocol
// (temp == nullptr: *bytes receives the temporary storage needed); counts
// are size_t, so no input size is narrowed to int.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/types/double_buffer.hpp>

namespace abc {
namespace prim {

// Stable LSD radix sort of n keys on bits [begin, end).
inline hipError_t sort_keys(void *temp, size_t &bytes, const uint64_t *in, uint64_t *out,
                            size_t n, int begin, int end, hipStream_t s) {
  return rocprim::radix_sort_keys(temp, bytes, in, out, n, (unsigned)begin, (unsigned)end, s);
}

// The same between two buffers: `cur` holds the keys before and after, `alt`
// is the other buffer (they may change places).  Needs no third buffer of n
// keys, as the form above does.
inline hipError_t sort_keys_two(void *temp, size_t &bytes, uint64_t *&cur, uint64_t *&alt,
                                size_t n, int begin, int end, hipStream_t s) {
  rocprim::double_buffer<uint64_t> keys(cur, alt);
  const hipError_t e =
      rocprim::radix_sort_keys(temp, bytes, keys, n, (unsigned)begin, (unsigned)end, s);
  cur = keys.current();
  alt = keys.alternate();
  return e;
}

// out[i] = in[0] + ... + in[i - 1] (out[0] = 0).
inline hipError_t exclusive_sum(void *temp, size_t &bytes, const int64_t *in, int64_t *out,
                                size_t n, hipStream_t s) {
  return rocprim::exclusive_scan(temp, bytes, in, out, (int64_t)0, n, rocprim::plus<int64_t>(),
                                 s);
}

}  // namespace prim
}  // namespace abc

// Conditions under which a launcher takes a kernel that cannot take every call, as plain host functions (no HIP types), so that
// they can be checked without a GPU and without tensors of the sizes they speak of.
#pragma once

#include <stdint.h>

namespace mamba {

// do the byte ranges [p, p + pn) and [q, q + qn) share a byte (null or empty: no)
inline bool overlap(const void *p, int64_t pn, const void *q, int64_t qn)
{
    if (!p || !q || pn <= 0 || qn <= 0) return false;
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
    return a < b + (uintptr_t)qn && b < a + (uintptr_t)pn;
}

// Scalar-decay scan, second pass stitching the segments itself (the figures are at launch_ssd): every workgroup of a head then
// reads h0, of its batch row, while the last one writes h_final, so the two must not share a byte: not in place, and not
// shifted against each other by a row or a part of one either.  before: pass 1 segments ahead of the last pass 2 segment.
inline bool ssd_folds(int n_seg1, int before, const void *h0, const void *h_final, int64_t state_bytes)
{
    return n_seg1 > 1 && before <= 10 && !overlap(h0, state_bytes, h_final, state_bytes);
}

// The few-row product counts k and columns in 32 bits and a workgroup of 512 threads takes 16 columns: k rounded up to a step
// of 64 has to fit an int, and the grid's threads along x have to stay below 2^32.  What does not fit takes the kernels
// that count in 64 bits (at a draft position: the chain of separate launches).
inline bool linear_few_fits(int64_t N, int64_t K)
{
    return K <= (int64_t)INT32_MAX - 63 && N <= ((int64_t)1 << 27) - 16;
}

}  // namespace mamba

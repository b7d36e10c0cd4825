// Calls between the library's source files; not part of its C ABI.
#ifndef SSS_INTERNAL_H
#define SSS_INTERNAL_H

#include <cstdint>

#include "sss.h"

// The bytes that range-checked loads may read of `count` values of `size`
// bytes each: whole 32-bit words that end with the last value or, where an odd
// number of 16-bit values ends inside a word, one value before it.
constexpr uint32_t value_range(uint32_t count, uint32_t size) { return count * size & ~3u; }

// sss_csr_spmv_execute in double precision for a square matrix, with partial
// sums of x . y beside it: *dots (device) holds *n_dots of them, in a fixed
// order, until the plan's next call.  *n_dots = 0: this plan's product does
// not form them (y is complete all the same).
extern "C" __attribute__((visibility("hidden"))) int sss_execute_dot(sss_plan p, const int32_t *row_ptr, const int32_t *col,
                                                          const double *val, const double *x, double *y,
                                                          void *stream, const double **dots, int *n_dots);

#endif  // SSS_INTERNAL_H

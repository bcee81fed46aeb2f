/*
 * pf_testing.h -- measurement and testing aids exported by libpf.so beside
 * the C ABI of pf.h.  Neither is part of the power-flow method; benchmarks
 * and tests use them.  Same conventions as pf.h (status codes, device
 * pointers, pf_last_error()).
 */
#ifndef PF_TESTING_H
#define PF_TESTING_H

#include <stdint.h>

#include "pf.h"

#ifdef __cplusplus
extern "C" {
#endif

/* A streaming device copy of n doubles from src to dst (DEVICE buffers,
 * 16-byte aligned, not overlapping): 16-byte loads, then 16-byte streaming
 * stores, two pairs of doubles per thread up to 8M pairs and one above (the
 * faster pattern at each size), one workgroup per chunk of the buffers.  A
 * copy moves its bytes with no dependent loads, so at
 * a given byte count it is the practical bandwidth ceiling for a kernel that
 * reads half and writes half of those bytes; the benchmark times it beside
 * the evaluation kernels.  One launch on `stream`.  Errors: PF_EINVAL
 * (n < 0, NULL, misaligned or overlapping buffers), PF_EHIP. */
int pf_stream_copy(const double *src, double *dst, int64_t n, void *stream);

/* The next n device allocations made by the library (pf_build_pattern,
 * pf_set_schedule) fail as if the device were out of memory, so that tests
 * can check the failure paths: the call returns PF_ENOMEM and leaves any
 * existing handle as it was.  n = 0 clears the count.  Process-wide.
 * Errors: PF_EINVAL for n < 0. */
int pf_debug_fail_allocs(int32_t n);

/* The launch that the evaluation call for (op, method) (as in pf_op) makes for
 * nstate states under the handle's present schedule; nothing is launched.
 * plan (5 values): states per workgroup, work order (PF_ORDER_TILE_MAJOR,
 * PF_ORDER_STATE_MAJOR or PF_ORDER_GROUPED), 1 if later states are read ahead
 * (else 0), workgroups, threads per workgroup.  On a PF_BUILD_HOST_ONLY handle
 * a device of 256 compute units is assumed.  Errors: PF_EINVAL. */
int pf_debug_launch(const pf_grid *g, int32_t op, int32_t method, int32_t nstate, int64_t *plan);

#ifdef __cplusplus
}
#endif

#endif /* PF_TESTING_H */

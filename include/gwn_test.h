/*
 * gwn_test.h -- test hooks of the MI355X GWN library (not needed in normal use).
 *
 * gwn_test_fail_alloc_after(n): the library's device allocations (hipMalloc /
 * hipMallocAsync, made by any call of include/gwn.h or include/gwn_prims.h)
 * succeed n more times, then every further one fails with out-of-memory --
 * without touching the device -- until the hook is reset; n < 0 resets it (the
 * default: no failures).  The failing call returns GWN_E_OOM with a message in
 * gwn_last_error() and releases whatever it had allocated.  Process-wide, for
 * all devices and threads.  Returns the number of allocations made since the
 * previous call (host-side count), so a test can find out how many a call makes.
 *
 * gwn_test_far_plan(...): the far part that a grid call would lay out (host code
 * only, no device needed) for a mesh of the bounding box bbox (minimum x, y, z,
 * maximum x, y, z), nchunk boundary chunks and a mean chunk extent of chunk_w
 * fixed-point cells, along the z ray; values: 1 for w, 3 for the gradient.  Writes
 * the number of levels (0: no far part), then per level, finest first, the far
 * distance in cells and for x and y the number of blocks and each block's first
 * and last sample.  Returns the count of numbers, -1 if cap is too small.
 *
 * gwn_test_plan_launches(nitems, kernel, work_items): how many launches a plan of
 * nitems work items makes of its kernels for the keys of its orders (0), the
 * crossings of ordered queries (1), of others by a wave each (2) or by a lane each in
 * items of 512 (3), and in *work_items the largest one's (host code only).
 *
 * gwn_test_boxes(...): the number of boxes of samples in which an FP32 grid call
 * would be summed (0: in columns) for such a mesh of nb boundary edges in nloops
 * loops and nclusters lowest clusters, and the work-items of its largest launch
 * (host code only).
 */
#ifndef GWN_TEST_H
#define GWN_TEST_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

int64_t gwn_test_fail_alloc_after(int64_t n);

int64_t gwn_test_far_plan(const double* bbox, int64_t nchunk, double chunk_w, const double* origin,
                          const double* spacing, const int64_t* dims, int32_t prec, int32_t values, int64_t* out,
                          int64_t cap);

int64_t gwn_test_boxes(const double* bbox, int64_t nchunk, double chunk_w, int64_t nb, int64_t nloops,
                       int64_t nclusters, const double* origin, const double* spacing, const int64_t* dims,
                       int64_t* work_items);
int64_t gwn_test_plan_launches(int64_t nitems, int32_t kernel, int64_t* work_items);

#ifdef __cplusplus
}
#endif

#endif /* GWN_TEST_H */

/*
 * nimbus_route.h: which kernels a call of nimbus_cop.h launches, exported by the same shared
 * library.  The answer comes out of the dispatch code itself (it runs with the launches written
 * down instead of made), so that a test of a kernel variant can check that its sizes still
 * reach the variant it is there for, and a benchmark can name the kernel it times.
 *
 * Host only: nothing is enqueued, no device is needed (without one the rules that ask for
 * the number of compute units assume 256).
 *
 * text   receives one line per launch, in order:
 *            <kernel with its template arguments> grid=<x>,<y> block=<threads>
 *        zero-terminated, cut off at `size` bytes
 * Return value: NIMBUS_COP_OK or the status that the entry point gives for these sizes.
 */
#ifndef NIMBUS_ROUTE_H
#define NIMBUS_ROUTE_H

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* nimbus_cop_prepare */
int nimbus_route_prepare(int k, int n, int N, int L, const uint64_t *moduli, char *text, size_t size);

/*
 * staged = 0: nimbus_cop_matmul_prepared (and its _static variant); count is 1.
 * staged = 1: nimbus_cop_matmul_staged with count = 1, nimbus_cop_matmul_staged_batch of `count`
 *             problems otherwise.
 * masked: with (1) or without (0) a mask.
 * units:  the number of compute units the rules are to assume, 0 for the current device's.
 */
int nimbus_route_matmul(int staged, int count, int m, int k, int x_bits, int n, int N, int L,
                        const uint64_t *moduli, int masked, int units, char *text, size_t size);

#ifdef __cplusplus
}
#endif
#endif /* NIMBUS_ROUTE_H */

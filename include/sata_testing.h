/*
 * sata_testing.h - entry points for the tests and measurements of this library:
 * which kernels a call takes, and the same call by one way of the caller's
 * choice.  Programs have no use for them: sata_prefill and sata_backward take
 * the way that is estimated to be the faster one.
 */
#ifndef SATA_TESTING_H
#define SATA_TESTING_H

#include "sata.h"

#ifdef __cplusplus
extern "C" {
#endif

typedef enum {
  SATA_ROUTE_PAIRS = 0,    /* pair by pair                                         */
  SATA_ROUTE_MFMA32 = 1,   /* chunked scans: the kernel for bfloat16, P = 4, d = 32 */
  SATA_ROUTE_BLOCKS = 2,   /* bfloat16, P = 4, d = 16 (and other chunks of d = 32)  */
  SATA_ROUTE_FEATURES = 3, /* generated features on the matrix cores               */
  SATA_ROUTE_FLOAT32 = 4   /* float32 arithmetic                                   */
} sata_route;

/* The kernels that sata_prefill (G = 1) or sata_prefill_grouped takes for these
 * arguments and 16-byte aligned tensors, with or without a state (host only;
 * the calls' own validation). */
sata_status sata_testing_prefill_route(sata_dtype dt, int B, int H_kv, int G, int n, int d_k, int d_v, int P,
                                       int chunk, int want_state, sata_route* route);
/* The scan's kernels for these arguments, whether or not the call goes by them. */
sata_status sata_testing_scan_route(sata_dtype dt, int B, int H_kv, int n, int d_k, int d_v, int P, int chunk,
                                    sata_route* route);
/* The kernels of sata_backward: SATA_ROUTE_PAIRS, or SATA_ROUTE_FLOAT32 for the scans. */
sata_status sata_testing_backward_route(sata_dtype dt, int B, int H, int n, int d_k, int d_v, int P, int chunk,
                                        sata_route* route);

/* sata_prefill_grouped and sata_backward pair by pair (pairs != 0;
 * SATA_ERR_UNSUPPORTED where those kernels do not cover the shape) or by the
 * scans (pairs = 0), whatever the estimates say. */
sata_status sata_testing_prefill(int pairs, const void* q, const void* k, const void* v, sata_dtype dt, int B,
                                 int H_kv, int G, int n, int d_k, int d_v, int P, int chunk, void* y, float* S_out,
                                 void* stream);
sata_status sata_testing_backward(int pairs, const void* q, const void* k, const void* v, const void* dy,
                                  sata_dtype dt, int B, int H, int n, int d_k, int d_v, int P, int chunk, void* dq,
                                  void* dk, void* dv, void* stream);

#ifdef __cplusplus
}
#endif

#endif /* SATA_TESTING_H */

/*
 * blr_measure.h - flag bits of the forward calls of blr.h and a query that exist for tests and measurements only.
 * An application never needs them; bench.py uses the stage flags to time the kernels of a multi-kernel
 * call one by one, the tests use BLR_FORCE_GENERIC to cross-check the two GPU code paths.
 */
#ifndef BLR_MEASURE_H
#define BLR_MEASURE_H

#include "blr.h"

/* every forward: run the portable scalar-ALU kernels even where an MFMA kernel exists */
#define BLR_FORCE_GENERIC           0x100u
/* Monarch, low-rank and BLAST forwards: enqueue only the kernels up to and including the one that
 * writes the workspace intermediate (FIRST), or only the kernel that consumes it (LAST; the workspace
 * must hold the intermediate of an earlier call with identical arguments). Mutually exclusive;
 * BLR_ERR_UNSUPPORTED, with nothing enqueued, where the call is a single kernel. Where BLAST walks the
 * tokens in several chunks the workspace holds one chunk only, so LAST is then good for timing, not
 * for values. */
#define BLR_ONLY_FIRST_STAGE        0x200u
#define BLR_ONLY_LAST_STAGE         0x400u

/* The kernels, by name, that a bf16 matrix product of a forward call runs on, as the rules on sizes choose them: what a test
 * of one tile checks its sizes with. No device is needed. C(g, m, n) = sum_k A(g, m, k) B(g, n, k), g < G, m < M, n < N,
 * k < K, C in G blocks of N columns or, by `form`, interleaved (column n G + g) or as 8-bit floats; A in 64-column windows of
 * its rows where such tiles exist. run > 0: a first product of a Monarch layer, its rows gathered and its columns scattered
 * in runs of `run`. members 2, 3: the last product of a chain's group, combined. `names` receives e.g. "128x192 w8 k64x3
 * i16 partial" (tile, wavefronts, contraction indices of a step x stages, rows of the matrix instruction, kind of last step),
 * several joined by " + ", "" where members are not combined. BLR_ERR_WORKSPACE where `size` bytes do not hold it, BLR_ERR_UNSUPPORTED where
 * the call would be refused. */
#define BLR_PRODUCT_INTERLEAVED     1u
#define BLR_PRODUCT_WINDOWS         2u
#define BLR_PRODUCT_8_BIT           4u
#ifdef __cplusplus
extern "C"
#endif
blr_status blr_product_tiles(int64_t M, int N, int K, int G, int run, unsigned form, int members, char* names, size_t size);

#endif /* BLR_MEASURE_H */

/*
 * igdebug.h - test hooks of libigfilter: injected allocation failures and a
 * count of the library's live allocations, for checking that every entry
 * point that allocates reports IG_ERR_OUT_OF_MEMORY when an allocation fails
 * and leaks nothing.  Not for production use.
 *
 * Every device allocation of the library (and the pinned host table of a
 * batch plan) goes through one counting wrapper.  The environment variable
 * IG_FAULT_INJECT=alloc[:N] makes the N-th such allocation after the library
 * loads fail (N = 1 when omitted), as ig_debug_fail_alloc(N) does at run time.
 */
#ifndef IGDEBUG_H
#define IGDEBUG_H

#include <stdint.h>

#include "igfilter.h"

#ifdef __cplusplus
extern "C" {
#endif

/* The nth allocation from now (1 = the next one) fails with out-of-memory,
 * once; nth <= 0 cancels a pending failure.  Host only; process-wide. */
void ig_debug_fail_alloc(int64_t nth);

/* Allocations of the library alive now (made and not yet freed).  Host only. */
int64_t ig_debug_live_allocations(void);

/* Free the library's process-lifetime caches (the reduction scratch of
 * ig_compare / ig_reduce of the calling thread, the per-device scratch of
 * ig_quality, every cached batch plan) after the work using them has
 * finished; later calls allocate them again. */
void ig_debug_release_caches(void);

/* Largest piece ig_surrogate_infer runs in one pass, in voxels (larger cubes
 * are cut into slabs or tiles with a halo of the network's depth, which gives
 * the same result bit for bit); voxels <= 0 restores the default, 2^28.
 * Returns the previous limit.  Host only; process-wide: lets tests exercise
 * the tiled path on small cubes. */
int64_t ig_debug_set_infer_piece_limit(int64_t voxels);

/* The schedules ig_filter_autotune times for p on ncu compute units, the
 * automatic one first; writes at most cap of them to out and returns how many
 * there are (-1: bad arguments).  Host only. */
int32_t ig_debug_tune_candidates(const ig_params* p, int32_t ncu, ig_schedule* out, int32_t cap);

/* Voxels per lane, rows per wavefront and wavefronts (layout[3]) that the
 * handle's passes of this depth run with; zeros before the first.  Host only. */
ig_status ig_debug_filter_layout(const ig_filter* f, int32_t depth, int32_t* layout);

/* The form of ig_smooth's rotated kernel: 0 the general one, 1 and 2 columns with
 * one and two output rows per thread, 3 columns in the least LDS.  The first
 * fixes the form of later calls where its tile fits (-1: the library's choice;
 * process-wide), the second returns the form chosen for half-widths radius[3] on
 * a cube and ncu compute units (-1: refused).  Host only. */
ig_status ig_debug_set_dense_form(int32_t form);
int32_t ig_debug_dense_form(const int32_t* radius, int64_t nx, int64_t ny, int64_t nz, int32_t ncu);

#ifdef __cplusplus
}
#endif
#endif /* IGDEBUG_H */

/*
 * atomo_debug.h - switches for tests of libatomo (not part of the method): they make a context take paths that the placement
 * and the timing of a call choose otherwise.
 */
#ifndef ATOMO_DEBUG_H
#define ATOMO_DEBUG_H

#include "atomo.h"

#ifdef __cplusplus
extern "C" {
#endif

/* The direct SVD encode reduces matrices of more than 128 vectors by groups of workgroups that exchange data.
 * spread != 0: the workgroups of a group are dealt over all dies instead of one.  start_ticks: how long a workgroup waits for the
 * others of its group to start, in ticks of the 100 MHz clock; 0 gives up at once, and the matrix is reduced by one
 * workgroup; negative: the library's own bound.  Results agree with the usual path to rounding. */
int atomo_debug_direct_groups(atomo_ctx* ctx, int spread, int64_t start_ticks);

/* Where the entry-wise encoder has no list of open draws (water levels below the normal range), its workgroups count what they keep
 * and read the counts of those before them.  loads: how often a workgroup looks for a count before it makes it itself; 0: never;
 * negative: the library's own bound.  Results are the same. */
int atomo_debug_entrywise_counts(atomo_ctx* ctx, int loads);

#ifdef __cplusplus
}
#endif
#endif /* ATOMO_DEBUG_H */

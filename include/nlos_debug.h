/*
 * nlos_debug.h -- test hooks of libnlos (not needed by applications).
 */
#ifndef NLOS_DEBUG_H
#define NLOS_DEBUG_H

#include "nlos.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Makes the next n allocations of the library fail as if memory were exhausted: device
 * allocations (plan tables, the context's workspace pool and tables) and host allocation
 * points (plan and kernel construction).  The call that meets one returns
 * NLOS_ERR_OUT_OF_MEMORY with nothing enqueued and nothing leaked, and the context stays
 * usable; memory that only saves time (f-k work lists) is done without.  n = 0 clears the injection.  Process wide; for fault-path tests. */
void nlos_debug_fail_allocations(int n);

/* The same after letting the next k allocations through. */
void nlos_debug_fail_allocations_after(int k, int n);

/* Host only: entries of the work lists (tiles and columns that can be non-zero after the
 * Stolt remap) an f-k plan of this descriptor is created with; 0 where its passes run over
 * every tile and column. */
nlos_status nlos_debug_fk_lists(const nlos_fk_desc *desc, size_t *n_items);

#ifdef __cplusplus
}
#endif

#endif /* NLOS_DEBUG_H */

// Residuals on their way to the host (readback.hip): a kernel writes them to
// pinned host memory, which the host reads after the synchronisation it makes
// anyway.
#pragma once

#include "ofl_internal.hpp"

namespace ofl {

// Weak: the host code also links without the device code (it then copies each
// residual).

// A double of pinned host memory that every device can write, from a page that
// the process keeps, or null: the page is full or cannot be had.
__attribute__((weak)) double *host_slot_take();
__attribute__((weak)) void host_slot_return(double *slot);
// n of them of the caller's own, or null. Returning or freeing needs every
// launch that writes them to have ended.
__attribute__((weak)) double *host_slots_alloc(int n);
__attribute__((weak)) void host_slots_free(double *slots);
// *slot = *gosa.
__attribute__((weak)) void launch_publish(const double *gosa, double *slot, hipStream_t s);
// slots[b] = views[b]'s gosa, b < ngrids.
__attribute__((weak)) void launch_publish_batch(const GridView *views, int ngrids, double *slots, hipStream_t s);
// *gosa = sum(parts[0..n)) / omega^2 in a fixed order, and *slot unless null.
__attribute__((weak)) void launch_fold_publish(const double *parts, long long n, float omega, double *gosa,
                                               double *slot, hipStream_t s);

}  // namespace ofl

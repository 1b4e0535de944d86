/*
 * Entry points of librok for its own tests; not part of the library's
 * interface (include/rok.h).
 */
#ifndef ROK_TESTING_H
#define ROK_TESTING_H

#include "rok.h"

#ifdef __cplusplus
extern "C" {
#endif

/* The resident kernels of 256 blocks behave as if only the first `blocks` of
 * them had found room on the device in time (0, the default: off).  The
 * results do not change.  ROK_EINVAL outside 0 .. 256. */
rok_status rok_set_gang_hold(rok_ctx* ctx, int blocks);

#ifdef __cplusplus
}
#endif

#endif

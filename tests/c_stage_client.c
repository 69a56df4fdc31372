/* A C client in which memory runs out after the context exists: its own
 * hipHostMalloc and hipMalloc (taken for the runtime's, which they call until
 * then) fail and leave the runtime's error recorded, as the runtime's do.
 * Without pinned memory state transfers go by the plain copies; without device
 * memory an admission fails, and the boxes admitted before run on.  Prints "ok"
 * or the first failed check; exit status 0 ok, 1 a failed check, 77 no usable
 * device. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "mpcd.h"

int hipSetDevice(int device);

static int exhausted = 0, refused = 0;

int hipHostMalloc(void** p, size_t bytes, unsigned flags)
{
    int (*real)(void**, size_t, unsigned);
    *(void**)&real = dlsym(RTLD_NEXT, "hipHostMalloc");
    if (exhausted) {
        ++refused;
        (void)hipSetDevice(-1);   /* an error for the runtime to remember */
        *p = NULL;
        return 2;                 /* hipErrorOutOfMemory */
    }
    return real(p, bytes, flags);
}

int hipMalloc(void** p, size_t bytes)
{
    int (*real)(void**, size_t);
    *(void**)&real = dlsym(RTLD_NEXT, "hipMalloc");
    if (exhausted) {
        ++refused;
        (void)hipSetDevice(-1);
        *p = NULL;
        return 2;
    }
    return real(p, bytes);
}

static int failed(const char* what, int rc)
{
    printf("FAILED %s: %d (%s)\n", what, rc, mpcd_strerror(rc));
    return 1;
}

int main(void)
{
    mpcd_ctx* ctx = NULL;
    int rc = mpcd_create(NULL, &ctx);
    if (rc == MPCD_EDEVICE) {
        printf("no device\n");
        return 77;
    }
    if (rc != MPCD_OK) return failed("create", rc);
    const int64_t n = 5000;
    mpcd_box_desc d;
    memset(&d, 0, sizeof d);
    d.L[0] = d.L[1] = d.L[2] = 8;
    d.a = 1.0;
    d.n_particles = n;
    d.dt = 0.1;
    d.alpha = 2.0;
    d.kT = 1.0;
    d.mass = 1.0;
    d.seed = 5u;
    d.flags = MPCD_INIT_MAXWELL;
    int32_t slot = -1;
    if ((rc = mpcd_admit(ctx, &d, &slot)) != MPCD_OK) return failed("admit", rc);
    if ((rc = mpcd_step(ctx, 20)) != MPCD_OK) return failed("step", rc);
    float* s = (float*)malloc(sizeof(float) * 6 * (size_t)n);
    float* t = (float*)malloc(sizeof(float) * 6 * (size_t)n);
    int64_t step = -1;
    if (!s || !t) return failed("malloc", 0);
    mpcd_observables o;
    if ((rc = mpcd_observe(ctx, slot, &o)) != MPCD_OK) return failed("observe", rc);
    exhausted = 1;
    if ((rc = mpcd_get_state(ctx, slot, s, &step)) != MPCD_OK || step != 20) return failed("get_state", rc);
    if ((rc = mpcd_set_state(ctx, slot, s, 4)) != MPCD_OK) return failed("set_state", rc);
    if ((rc = mpcd_get_state(ctx, slot, t, &step)) != MPCD_OK || step != 4) return failed("get_state 2", rc);
    if (memcmp(s, t, sizeof(float) * 6 * (size_t)n) != 0) return failed("state round trip", 0);
    if (refused < 3) return failed("refusals", refused);
    exhausted = 0;
    if ((rc = mpcd_get_state(ctx, slot, t, &step)) != MPCD_OK) return failed("get_state 3", rc);
    if (memcmp(s, t, sizeof(float) * 6 * (size_t)n) != 0) return failed("state", 0);
    exhausted = 1;
    int32_t other = -1;
    if ((rc = mpcd_admit(ctx, &d, &other)) != MPCD_ENOMEM) return failed("admit without memory", rc);
    if (refused < 4) return failed("refusals 2", refused);
    if ((rc = mpcd_step(ctx, 20)) != MPCD_OK) return failed("step after it", rc);
    if ((rc = mpcd_observe(ctx, slot, &o)) != MPCD_OK || o.step != 24) return failed("observe after it", rc);
    mpcd_destroy(ctx);
    free(s);
    free(t);
    printf("ok\n");
    return 0;
}

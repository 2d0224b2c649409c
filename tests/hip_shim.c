/* Stands before the HIP runtime in a test's process: counts cooperative
 * launches and allocations, refuses them on demand, and remembers the device
 * memory cleared by the last hipMemsetAsync of a size. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>

typedef struct { unsigned x, y, z; } dim3_t;

int shim_cooperative = 0;        /* cooperative launches asked for */
int shim_no_launch = 0;          /* count them only */
int shim_strict = 0;             /* a refusal of the runtime's own stands */
int shim_refuse_launch = 0;      /* refuse the one that would be this many (0: none) */
int shim_mallocs = 0;            /* allocations asked for */
int shim_refuse_malloc = 0;      /* refuse the one that would be this many (0: none) */
int shim_pinned = 0;             /* pinned allocations held */
size_t shim_watch_bytes = 0;     /* hipMemsetAsync of this size: */
void *shim_cleared = NULL;       /* the memory it last cleared */

static void *next_of(const char *name) {
    void *f = dlsym(RTLD_NEXT, name);
    if (!f) {
        void *h = dlopen("libamdhip64.so.7", RTLD_NOLOAD | RTLD_LAZY);
        if (!h) h = dlopen("libamdhip64.so", RTLD_NOLOAD | RTLD_LAZY);
        if (h) f = dlsym(h, name);
    }
    return f;
}

int hipLaunchCooperativeKernel(const void *f, dim3_t grid, dim3_t block, void **args, unsigned lds, void *stream) {
    static int (*real)(const void *, dim3_t, dim3_t, void **, unsigned, void *) = NULL;
    if (!real) real = (int (*)(const void *, dim3_t, dim3_t, void **, unsigned, void *))next_of("hipLaunchCooperativeKernel");
    if (++shim_cooperative == shim_refuse_launch) return 720; /* hipErrorCooperativeLaunchTooLarge */
    if (shim_no_launch) return 0;
    int e = real(f, grid, block, args, lds, stream);
    if (e && !shim_strict) { /* one process at a time may launch cooperatively: the few workgroups of a small model fit all the same */
        int (*clear)(void) = (int (*)(void))next_of("hipGetLastError");
        int (*plain)(const void *, dim3_t, dim3_t, void **, size_t, void *) =
            (int (*)(const void *, dim3_t, dim3_t, void **, size_t, void *))next_of("hipLaunchKernel");
        clear();
        if (grid.x <= 64) e = plain(f, grid, block, args, lds, stream);
    }
    return e;
}

int hipMalloc(void **p, size_t bytes) {
    static int (*real)(void **, size_t) = NULL;
    if (!real) real = (int (*)(void **, size_t))next_of("hipMalloc");
    if (++shim_mallocs == shim_refuse_malloc) return 2; /* hipErrorOutOfMemory */
    return real(p, bytes);
}

int hipHostMalloc(void **p, size_t bytes, unsigned flags) {
    static int (*real)(void **, size_t, unsigned) = NULL;
    if (!real) real = (int (*)(void **, size_t, unsigned))next_of("hipHostMalloc");
    ++shim_pinned;
    return real(p, bytes, flags);
}

int hipHostFree(void *p) {
    static int (*real)(void *) = NULL;
    if (!real) real = (int (*)(void *))next_of("hipHostFree");
    --shim_pinned;
    return real(p);
}

int hipMemsetAsync(void *p, int value, size_t bytes, void *stream) {
    static int (*real)(void *, int, size_t, void *) = NULL;
    if (!real) real = (int (*)(void *, int, size_t, void *))next_of("hipMemsetAsync");
    if (bytes == shim_watch_bytes) shim_cleared = p;
    return real(p, value, bytes, stream);
}

int shim_poke(void *p, unsigned value) { /* writes a 32-bit word of device memory */
    int (*copy)(void *, const void *, size_t, int) = (int (*)(void *, const void *, size_t, int))next_of("hipMemcpy");
    return p ? copy(p, &value, sizeof value, 1 /* host to device */) : 1;
}

void *shim_masked_stream(unsigned words, const unsigned *mask) { /* a stream on some compute units */
    int (*create)(void **, unsigned, const unsigned *) =
        (int (*)(void **, unsigned, const unsigned *))next_of("hipExtStreamCreateWithCUMask");
    void *s = NULL;
    return create(&s, words, mask) == 0 ? s : NULL;
}

/* hipMalloc with a limit, for tests of plans at the edge of memory: loaded
 * ahead of the HIP runtime (LD_PRELOAD), it counts the bytes that are
 * allocated and refuses what would pass the limit, as a full device does. */
#include <dlfcn.h>
#include <stddef.h>

enum { SLOTS = 4096 };
static struct { void *p; size_t n; } live[SLOTS];
static size_t used, peak, limit = (size_t)-1;

void alloc_limit_set(size_t bytes) { limit = bytes; }
void alloc_limit_reset_peak(void) { peak = used; }
size_t alloc_limit_used(void) { return used; }
size_t alloc_limit_peak(void) { return peak; }

/* The runtime's function: the library is loaded by then, not into the global scope. */
static void *runtime(const char *name) {
    void *lib = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
    return lib ? dlsym(lib, name) : NULL;
}

int hipMalloc(void **p, size_t n) {
    static int (*real)(void **, size_t);
    if (!real) real = (int (*)(void **, size_t))runtime("hipMalloc");
    if (!real) return 999; /* hipErrorUnknown */
    if (n > limit || used > limit - n) return 2; /* hipErrorOutOfMemory */
    const int e = real(p, n);
    if (e != 0) return e;
    for (int i = 0; i < SLOTS; ++i)
        if (!live[i].p) {
            live[i].p = *p;
            live[i].n = n;
            used += n;
            if (used > peak) peak = used;
            break;
        }
    return 0;
}

int hipFree(void *p) {
    static int (*real)(void *);
    if (!real) real = (int (*)(void *))runtime("hipFree");
    if (!real) return 999;
    if (p)
        for (int i = 0; i < SLOTS; ++i)
            if (live[i].p == p) {
                used -= live[i].n;
                live[i].p = 0;
                break;
            }
    return real(p);
}

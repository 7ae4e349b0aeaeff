/* Loaded before the library: hipMallocAsync that refuses the next few large requests, as a device without that much memory does. */
#include <dlfcn.h>
#include <stddef.h>

static int refusals, refused;
void refuse_next(int count) { refusals = count; refused = 0; }
int refused_so_far(void) { return refused; }
int hipMallocAsync(void **p, size_t n, void *stream)
{
    static int (*real)(void **, size_t, void *);
    if (!real) {
        void *hip = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
        if (!hip) hip = dlopen("libamdhip64.so", RTLD_LAZY | RTLD_NOLOAD);
        if (hip) real = (int (*)(void **, size_t, void *))dlsym(hip, "hipMallocAsync");
    }
    if (n > (1u << 20) && refused < refusals) { ++refused; return 2; }
    return real ? real(p, n, stream) : 2;
}

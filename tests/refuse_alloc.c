/* Loaded before the library: hipMallocAsync that refuses what is larger than a limit, as a device without that much memory does. */
#include <dlfcn.h>
#include <stddef.h>

static size_t most = (size_t)-1;
static int refused;
void refuse_above(size_t bytes) { most = bytes; refused = 0; }
int refused_so_far(void) { return refused; }
int hipMallocAsync(void **p, size_t n, void *stream)
{
    static int (*real)(void **, size_t, void *);
    if (!real) {
        void *hip = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
        if (!hip) hip = dlopen("libamdhip64.so", RTLD_LAZY | RTLD_NOLOAD);
        if (hip) real = (int (*)(void **, size_t, void *))dlsym(hip, "hipMallocAsync");
    }
    if (n > most || !real) { refused += n > most; return 2; }
    return real(p, n, stream);
}

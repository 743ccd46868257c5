/* Counts the calls to the HIP runtime that make or free memory, streams and events, and passes them
 * on.  Loaded with RTLD_GLOBAL before the runtime, so that later libraries bind to these. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <link.h>
#include <stddef.h>
#include <string.h>

static long calls;
long counted_calls(void) { return calls; }

static int find(struct dl_phdr_info* info, size_t size, void* out) {
    (void)size;
    if (!info->dlpi_name || !strstr(info->dlpi_name, "libamdhip64")) return 0;
    *(void**)out = dlopen(info->dlpi_name, RTLD_NOLOAD | RTLD_LAZY);
    return 1;
}

static void* real(const char* name) {
    static void* lib;
    if (!lib) dl_iterate_phdr(find, &lib);
    return dlsym(lib, name);
}

#define COUNTED(name, params, args)                      \
    int name params {                                    \
        static int(*f) params;                           \
        if (!f) f = (int(*) params)real(#name);          \
        ++calls;                                         \
        return f args;                                   \
    }

COUNTED(hipMalloc, (void** p, size_t n), (p, n))
COUNTED(hipMallocAsync, (void** p, size_t n, void* s), (p, n, s))
COUNTED(hipFree, (void* p), (p))
COUNTED(hipFreeAsync, (void* p, void* s), (p, s))
COUNTED(hipHostMalloc, (void** p, size_t n, unsigned f_), (p, n, f_))
COUNTED(hipHostFree, (void* p), (p))
COUNTED(hipHostRegister, (void* p, size_t n, unsigned f_), (p, n, f_))
COUNTED(hipStreamCreate, (void** s), (s))
COUNTED(hipStreamCreateWithFlags, (void** s, unsigned f_), (s, f_))
COUNTED(hipStreamDestroy, (void* s), (s))
COUNTED(hipEventCreate, (void** e), (e))
COUNTED(hipEventCreateWithFlags, (void** e, unsigned f_), (e, f_))
COUNTED(hipEventDestroy, (void* e), (e))

/* The HIP calls through which the library takes memory and sends it pointers, with limits
 * that a test sets: loaded before everything else, these come first in the lookup of
 * their names and pass on to the runtime what the limits allow.  A refused call changes
 * nothing and returns the runtime's own error code.  Kernel launches are passed on and
 * those of a name counted. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <string.h>

typedef int (*malloc_t)(void **, size_t);
typedef int (*host_malloc_t)(void **, size_t, unsigned);
typedef struct { unsigned x, y, z; } dim3_t;
typedef int (*launch_t)(const void *, dim3_t, dim3_t, void **, size_t, void *);
typedef int (*copy_t)(void *, const void *, size_t, int, void *);

/* hipErrorOutOfMemory, hipErrorUnknown, hipMemcpyHostToDevice */
enum { kOutOfMemory = 2, kUnknown = 999, kHostToDevice = 1 };

static size_t host_from = (size_t)-1, dev_from = (size_t)-1, copy_to = 0;
static long host_left = 0, dev_left = 0, copy_left = 0, refused = 0;

/* pinned (device) allocations of at least `from` bytes: `left` more succeed */
void limit_host(size_t from, long left) { host_from = from; host_left = left; }
void limit_device(size_t from, long left) { dev_from = from; dev_left = left; }
/* copies to the device of at most `to` bytes: the next `n` fail */
void fail_copies(size_t to, long n) { copy_to = to; copy_left = n; }
/* calls refused since last asked */
long refusals(void)
{
    long n = refused;
    refused = 0;
    return n;
}

static void *runtime(const char *name)
{
    void *lib = dlopen("libamdhip64.so.7", RTLD_NOW | RTLD_NOLOAD);
    return lib ? dlsym(lib, name) : NULL;
}

int hipHostMalloc(void **p, size_t n, unsigned flags)
{
    if (n >= host_from && host_left-- <= 0) return refused++, kOutOfMemory;
    return ((host_malloc_t)runtime("hipHostMalloc"))(p, n, flags);
}

int hipMalloc(void **p, size_t n)
{
    if (n >= dev_from && dev_left-- <= 0) return refused++, kOutOfMemory;
    return ((malloc_t)runtime("hipMalloc"))(p, n);
}

int hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *stream)
{
    if (kind == kHostToDevice && n <= copy_to && copy_left > 0) return copy_left--, refused++, kUnknown;
    return ((copy_t)runtime("hipMemcpyAsync"))(dst, src, n, kind, stream);
}

static char counted[128];
static long launches;

/* launches since last asked of kernels whose (mangled) name holds the one given then;
 * from here on those of `name` */
long launches_of(const char *name)
{
    long n = launches;
    launches = 0;
    strncpy(counted, name, sizeof counted - 1);
    return n;
}

int hipLaunchKernel(const void *f, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream)
{
    Dl_info at;
    if (counted[0] && dladdr(f, &at) && at.dli_sname && strstr(at.dli_sname, counted)) launches++;
    return ((launch_t)runtime("hipLaunchKernel"))(f, grid, block, args, lds, stream);
}

/* Stands between the library and the HIP runtime's allocation calls in a test's
 * process: counts them, and refuses device allocations above a limit.  Loaded
 * with global symbols before the library, so the library's calls bind here. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>

static unsigned long calls;         /* allocations and frees seen */
static unsigned long refused;       /* device allocations refused */
static size_t limit = (size_t)-1;   /* largest device allocation let through */

unsigned long shim_calls(void) { return calls; }
unsigned long shim_refused(void) { return refused; }
void shim_limit(size_t bytes) { limit = bytes; }

static void* next(const char* name) {
  return dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD), name);
}

int hipMalloc(void** p, size_t n) {
  ++calls;
  if (n > limit) {
    ++refused;
    return 2; /* hipErrorOutOfMemory */
  }
  return ((int (*)(void**, size_t))next("hipMalloc"))(p, n);
}
int hipFree(void* p) {
  ++calls;
  return ((int (*)(void*))next("hipFree"))(p);
}
int hipHostMalloc(void** p, size_t n, unsigned flags) {
  ++calls;
  return ((int (*)(void**, size_t, unsigned))next("hipHostMalloc"))(p, n, flags);
}
int hipHostFree(void* p) {
  ++calls;
  return ((int (*)(void*))next("hipHostFree"))(p);
}

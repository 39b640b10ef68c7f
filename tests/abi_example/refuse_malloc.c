/* Device allocations from a size on are refused: loaded in front of libsailor.so, its hipMalloc is the one
 * that the library finds. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <stdint.h>

static size_t refused_from = SIZE_MAX;
static int refused;

void refuse_from(size_t bytes) { refused_from = bytes; }
int times_refused(void) { return refused; }

int hipMalloc(void **out, size_t bytes) {
  static int (*real)(void **, size_t);
  if (bytes >= refused_from) {
    ++refused;
    return 2; /* hipErrorOutOfMemory */
  }
  if (!real) *(void **)&real = dlsym(RTLD_NEXT, "hipMalloc");
  return real(out, bytes);
}

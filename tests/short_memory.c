/* Stands in front of hipMalloc so that a test can have allocations fail as
 * the runtime lets them fail when memory is short.  Loaded with global scope
 * before the HIP runtime's users. */
#include <stddef.h>

typedef int (*malloc_fn)(void **, size_t);
static malloc_fn real;
static size_t fail_lo = 1, fail_hi = 0;
static int fail_left = 0;

void short_memory_real(malloc_fn f) { real = f; }

/* The next `count` requests of lo to hi bytes fail. */
void short_memory(size_t lo, size_t hi, int count)
{
    fail_lo = lo;
    fail_hi = hi;
    fail_left = count;
}

int short_memory_left(void) { return fail_left; }

int hipMalloc(void **p, size_t bytes)
{
    if (fail_left > 0 && bytes >= fail_lo && bytes <= fail_hi) {
        --fail_left;
        return real(p, (size_t)1 << 60); /* more than any device has: the runtime's own error */
    }
    return real(p, bytes);
}

/* Stands in front of hipMalloc so that a test can have allocations fail as
 * the runtime lets them fail when memory is short.  Loaded with global scope
 * before the HIP runtime's users. */
#include <stddef.h>

typedef int (*malloc_fn)(void **, size_t);
static malloc_fn real;
static size_t fail_lo = 1, fail_hi = 0;
static unsigned fail_mask = 0;

void short_memory_real(malloc_fn f) { real = f; }

/* Of the next requests of lo to hi bytes, the i-th (from 0) fails where bit i of `mask` is set. */
void short_memory(size_t lo, size_t hi, unsigned mask)
{
    fail_lo = lo;
    fail_hi = hi;
    fail_mask = mask;
}

/* The requests of the mask that have not come yet. */
unsigned short_memory_left(void) { return fail_mask; }

int hipMalloc(void **p, size_t bytes)
{
    if (bytes >= fail_lo && bytes <= fail_hi) {
        const int fail = fail_mask & 1;
        fail_mask >>= 1;
        if (fail) return real(p, (size_t)1 << 60); /* more than any device has: the runtime's own error */
    }
    return real(p, bytes);
}

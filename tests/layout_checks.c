/* The layout that cl_create takes at a given free device memory, on the host: the HIP
 * runtime calls that creation makes are defined here, so that device memory is host
 * memory of a stated free size and the bytes that a context allocates are counted.
 * Built and run by tests/test_layout_choice.py; exits non-zero on a failed expectation. */
#include "claire_hip.h"

#include <stdio.h>
#include <stdlib.h>
#include <string.h>

static size_t free_bytes, allocated;

int hipMemGetInfo(size_t *fr, size_t *tot)
{
    *fr = free_bytes;
    *tot = (size_t)1 << 40;
    return 0;
}
int hipMalloc(void **p, size_t n)
{
    allocated += n;
    *p = malloc(n);
    return *p ? 0 : 2;
}
int hipFree(void *p) { free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned flags) { (void)flags; *p = malloc(n); return *p ? 0 : 2; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) { (void)st; return hipMemcpy(d, s, n, kind); }
int hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)st; memset(d, v, n); return 0; }
int hipStreamSynchronize(void *st) { (void)st; return 0; }

static int fails = 0;

/* layout of a context (0 full, 1 lean) or the error code of its creation */
static int layout(int n1, int n2, int n3, const cl_options *o, size_t fr)
{
    cl_ctx *c = NULL;
    free_bytes = fr;
    allocated = 0;
    int st = cl_create(&c, n1, n2, n3, o);
    if (st != CL_OK) return st;
    st = cl_layout(c);
    cl_destroy(c);
    return st;
}

static void expect(const char *what, int n3, const cl_options *o, int got, int want)
{
    if (got == want) return;
    fprintf(stderr, "FAILED n3 %d nt %d precond %d, %s: %d, not %d\n", n3, o->nt, o->precond, what, got, want);
    ++fails;
}

int main(void)
{
    static const int nts[] = {2, 4, 5, 8, 16}, n3s[] = {64, 32, 128};
    for (unsigned a = 0; a < sizeof(nts) / sizeof(nts[0]); ++a)
        for (unsigned b = 0; b < sizeof(n3s) / sizeof(n3s[0]); ++b)
            for (int pc = CL_PRECOND_SPECTRAL; pc <= CL_PRECOND_H0_2LEVEL; ++pc) {
                const int n1 = 32, n2 = 64, n3 = n3s[b], refused = pc == CL_PRECOND_SPECTRAL ? 1 : CL_ERR_UNSUPPORTED;
                cl_options o;
                cl_default_options(&o);
                o.nt = nts[a];
                o.precond = pc;
                unsigned long long size = 0;
                expect("query", n3, &o, cl_query_workspace(n1, n2, n3, &o, &size), CL_OK);
                /* what the full layout allocates; the size is an upper bound of it */
                expect("room for all", n3, &o, layout(n1, n2, n3, &o, (size_t)1 << 40), 0);
                const size_t need = allocated;
                expect("size below the allocation", n3, &o, need > size, 0);
                /* no cap: by free memory, of which a sixteenth stays free (the size counts up to
                 * 1 MB more for tables and partial sums) */
                expect("free memory for it", n3, &o, layout(n1, n2, n3, &o, need / 15 * 16 + (1 << 20)), 0);
                expect("less free memory", n3, &o, layout(n1, n2, n3, &o, need / 16 * 16 - (4 << 20)), refused);
                /* a cap is compared with the size */
                o.workspace_cap_bytes = size;
                expect("cap of the size", n3, &o, layout(n1, n2, n3, &o, (size_t)1 << 40), 0);
                o.workspace_cap_bytes = size - 1;
                expect("cap below the size", n3, &o, layout(n1, n2, n3, &o, (size_t)1 << 40), refused);
            }
    printf("layout checks: %d failure(s)\n", fails);
    return fails ? 1 : 0;
}

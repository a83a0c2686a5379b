/* A stand-in for the HIP runtime, for tests of libtid's host code without a
   GPU: device memory is addresses that nothing is stored at, kernels are not
   run (their names are noted), and what the host reads back is a value that
   the test sets.  A host buffer that a copy to the device starts from is
   compared, at the next wait for the stream, with what it held when the copy
   was queued: a runtime may read it at any time until then. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#define DEVICE_BASE 0x600000000000ull
#define MOST 65536

/* what a test sets and reads */
uint64_t host_word = 0;        /* every 64-bit word of new pinned memory */
uint32_t read_word = 1;        /* every 32-bit word of a copy to the host */
uint64_t live_bytes = 0, peak_bytes = 0, most_bytes = ~0ull; /* device memory */
uint64_t pinned = 0;           /* allocations of pinned host memory */
uint64_t copies = 0, changed = 0;   /* copies from the host; those whose source changed */
char launched[1 << 20];        /* names of the launched kernels and the copies, a line each */

static uint64_t next_addr = DEVICE_BASE;
static struct { uint64_t at, bytes; } blocks[MOST];
static int nblocks;
static struct { const void *src; void *was; size_t n; } pending[MOST];
static int npending;
static struct { const void *fn; char name[160]; } kernels[4096];
static int nkernels;

static void note(const char *what) {
    static size_t at;
    if (at + 200 < sizeof launched) at += (size_t)sprintf(launched + at, "%s\n", what);
}

int hipMalloc(void **p, size_t n) {
    if (live_bytes + n > most_bytes || nblocks == MOST) return 2; /* out of memory */
    *p = (void *)next_addr;
    blocks[nblocks].at = next_addr;
    blocks[nblocks++].bytes = n;
    next_addr += (n + 4095) / 4096 * 4096 + 4096;
    live_bytes += n;
    if (live_bytes > peak_bytes) peak_bytes = live_bytes;
    return 0;
}
int hipFree(void *p) {
    for (int i = 0; i < nblocks; ++i)
        if (blocks[i].at == (uint64_t)p) {
            live_bytes -= blocks[i].bytes;
            blocks[i] = blocks[--nblocks];
            return 0;
        }
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned flags) {
    (void)flags;
    uint64_t *w = malloc((n + 7) / 8 * 8);
    if (!w) return 2;
    ++pinned;
    for (size_t i = 0; i < (n + 7) / 8; ++i) w[i] = host_word;
    *p = w;
    return 0;
}
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *stream) {
    (void)stream;
    note(kind == 1 ? "copy up" : kind == 2 ? "copy down" : "copy across");
    if (kind == 1) {
        ++copies;
        if (npending < MOST && n) {
            pending[npending].src = src;
            pending[npending].n = n;
            pending[npending].was = malloc(n);
            memcpy(pending[npending++].was, src, n);
        }
    } else if (kind == 2) {
        for (size_t i = 0; i + 4 <= n; i += 4) memcpy((char *)dst + i, &read_word, 4);
    }
    return 0;
}
int hipMemsetAsync(void *p, int v, size_t n, void *s) { (void)p; (void)v; (void)n; (void)s; return 0; }
int hipStreamSynchronize(void *stream) {
    (void)stream;
    for (int i = 0; i < npending; ++i) {
        changed += memcmp(pending[i].src, pending[i].was, pending[i].n) != 0;
        free(pending[i].was);
    }
    npending = 0;
    return 0;
}
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = (void *)1; return 0; }
int hipStreamDestroy(void *s) { return hipStreamSynchronize(s); }
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { (void)e; return "stand-in"; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t lds) {
    (void)f; (void)b; (void)lds;
    *n = 2;
    return 0;
}
int hipGetSymbolAddress(void **p, const void *s) { *p = (void *)s; return 0; }
struct attributes { int type, device; void *dev, *host; int managed; unsigned flags; };
int hipPointerGetAttributes(struct attributes *a, const void *p) {
    memset(a, 0, sizeof *a);
    if ((uint64_t)p < DEVICE_BASE || (uint64_t)p >= next_addr) return 1;
    a->type = 2; /* device memory */
    return 0;
}

/* what the compiler's launch stubs and module constructors call */
void **__hipRegisterFatBinary(const void *d) { static void *m; (void)d; return &m; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *a, char *b, int e, size_t n, int c, int g) {
    (void)m; (void)v; (void)a; (void)b; (void)e; (void)n; (void)c; (void)g;
}
void __hipRegisterFunction(void **m, const void *fn, char *name, const char *dev, unsigned limit,
                           void *t, void *b, void *bd, void *gd, int *w) {
    (void)m; (void)dev; (void)limit; (void)t; (void)b; (void)bd; (void)gd; (void)w;
    if (nkernels < 4096) {
        kernels[nkernels].fn = fn;
        snprintf(kernels[nkernels++].name, sizeof kernels[0].name, "%s", name);
    }
}
typedef struct { unsigned x, y, z; } dim3_t;
static struct { dim3_t g, b; size_t lds; void *s; } call;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void *s) {
    call.g = g; call.b = b; call.lds = lds; call.s = s;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *lds, void **s) {
    *g = call.g; *b = call.b; *lds = call.lds; *s = call.s;
    return 0;
}
int hipLaunchKernel(const void *fn, dim3_t g, dim3_t b, void **args, size_t lds, void *s) {
    (void)g; (void)b; (void)args; (void)lds; (void)s;
    for (int i = 0; i < nkernels; ++i)
        if (kernels[i].fn == fn) note(kernels[i].name);
    return 0;
}

/* The HIP calls of libmhdchem.so on the CPU, for tests of its host code: "device"
 * memory is host memory, copies are memcpy, kernels do nothing.  Loaded globally
 * before the library, so that its symbols come first.  The switches make a call
 * fail as a test asks for. */
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;

int stub_fail_new;        /* let the n-th array allocation of stub_new_bytes from now on fail (0: none) */
size_t stub_new_bytes;
int stub_capturing;       /* the stream is being captured: work is recorded, not done, and nothing can be waited for */
int stub_other_device;    /* the events are of another device than the stream */

/* operator new[](size_t, nothrow) */
void *_ZnamRKSt9nothrow_t(size_t n, const void *tag)
{
    (void)tag;
    if (stub_fail_new && n == stub_new_bytes && --stub_fail_new == 0) return 0;
    return malloc(n);
}

void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
/* kernels by host address, and the blocks launched of each */
static struct { const void *f; const char *name; long blocks; } kernel[4096];
static int kernels;
static unsigned pushed;
void __hipRegisterFunction(void **m, const void *f, char *dev, const char *name)
{
    (void)m;
    (void)dev;
    if (kernels < 4096) {
        kernel[kernels].f = f;
        kernel[kernels++].name = strdup(name);
    }
}
long stub_blocks(const char *part)   /* blocks launched of the kernels with this in their (mangled) names */
{
    long n = 0;
    for (int k = 0; k < kernels; k++)
        if (strstr(kernel[k].name, part)) n += kernel[k].blocks;
    return n;
}
void __hipRegisterVar(void) {}
void __hipUnregisterFatBinary(void) {}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t shm, void *s) { (void)b; (void)shm; (void)s; pushed = g.x; return 0; }
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *shm, void **s)
{
    memset(g, 0, sizeof(*g));
    memset(b, 0, sizeof(*b));
    *shm = 0;
    *s = 0;
    return 0;
}
int hipLaunchKernel(const void *f)
{
    for (int k = 0; k < kernels; k++)
        if (kernel[k].f == f) kernel[k].blocks += pushed;
    return 0;
}
int hipFuncSetAttribute(void) { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *v) { *v = 1; return 0; }
int hipGetLastError(void) { return 0; }
int hipStreamSynchronize(void *s) { (void)s; return stub_capturing ? 900 : 0; }
int hipStreamIsCapturing(void *s, int *st) { (void)s; *st = stub_capturing; return 0; }
int hipEventCreate(void **e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = malloc(1); return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return stub_other_device ? 400 : 0; }
int hipEventSynchronize(void *e) { (void)e; return stub_capturing ? 907 : 0; }
int hipEventElapsedTime(float *ms) { *ms = 0; return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = malloc(n); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)k; (void)st; if (!stub_capturing) memcpy(d, s, n); return 0; }
int hipGetSymbolAddress(void **p) { *p = 0; return 1; }
int hipPointerGetAttributes(void *a, const void *p) { (void)p; memset(a, 0, 32); return 0; }

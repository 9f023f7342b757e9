/* HIP's calls on host memory, for tests of what the library's host side does
 * when one of them fails (no GPU).  Loaded before libgsp.so with its symbols
 * global, it stands in for the runtime.  Of the kernels only k_post, which
 * hands results to the host, does anything, and k_bin_post, which finds no
 * vertex in any work list.  Pinned allocations beyond fake_pinned_limit bytes
 * fail, and device allocations once fake_mallocs_left have been made. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
size_t fake_pinned_limit = (size_t)1 << 40;
int fake_pinned_alive = 0, fake_device_alive = 0, fake_mallocs_left = 1 << 30;

static const void *post_kernel, *bin_post_kernel;
static struct { dim3 grid, block; size_t shared; void *stream; } config;

void **__hipRegisterFatBinary(const void *data) { (void)data; static void *module; return &module; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) {
    (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned lim, void *tid,
                           void *bid, dim3 *bd, dim3 *gd, int *ws) {
    (void)m; (void)dev; (void)lim; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
    if (strstr(name, "6k_post")) post_kernel = host;   /* mangled names */
    if (strstr(name, "10k_bin_post")) bin_post_kernel = host;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void *stream) {
    config.grid = grid; config.block = block; config.shared = shared; config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, void **stream) {
    *grid = config.grid; *block = config.block; *shared = config.shared; *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t shared, void *stream) {
    (void)grid; (void)block; (void)shared; (void)stream;
    if (f == post_kernel) {
        struct { const uint64_t *src[4]; int64_t n[4]; } a;
        uint64_t *box = *(uint64_t **)args[1], *o = box + 16;
        memcpy(&a, args[0], sizeof(a));
        for (int r = 0; r < 4; r++)
            for (int64_t k = 0; k < a.n[r]; k++) *o++ = a.src[r][k];
        box[0] = 1;
    }
    if (f == bin_post_kernel) {
        const int buckets = *(int *)args[2];
        uint64_t *box = *(uint64_t **)args[3];
        memset(box + 16, 0, 2 * sizeof(uint64_t) * (size_t)buckets);
        box[0] = 1;
    }
    return 0;
}
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
static int last_error;   /* kept until it is asked for */
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { (void)e; return "a fake error"; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = malloc(1); return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = malloc(1); return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipMalloc(void **p, size_t n) {
    *p = fake_mallocs_left-- > 0 ? calloc(n ? n : 1, 1) : NULL;
    fake_device_alive += *p != NULL;
    return *p ? 0 : (last_error = 2);
}
int hipFree(void *p) { fake_device_alive -= p != NULL; free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) {
    (void)f;
    if (n > fake_pinned_limit) return last_error = 2;   /* out of memory; *p stays as it is */
    *p = calloc(n, 1);
    fake_pinned_alive++;
    return 0;
}
int hipHostFree(void *p) { fake_pinned_alive -= p != 0; free(p); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)k; (void)st; memmove(d, s, n); return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)st; memset(d, v, n); return 0; }

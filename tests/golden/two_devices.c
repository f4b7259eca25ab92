/* A host that has two devices, for checks of which of them a call uses: the
 * runtime calls that the library makes outside its kernels, on host memory.
 * Streams 0x100 + d belong to device d, the null stream to the current device.
 * An event recorded on another device's stream, or a kernel launched on the null
 * stream of a device other than `home`, is an invalid handle (400). */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

static int current, home, last;
void two_devices(int cur, int run) { current = cur; home = run; }
int two_devices_current(void) { return current; }

static int device_of(void *stream) { return stream ? (int)((uintptr_t)stream - 0x100) : current; }

typedef struct { uint32_t x, y, z; } dim;
static struct { dim g, b; size_t lds; void *stream; } config;
int __hipPushCallConfiguration(dim g, dim b, size_t lds, void *stream)
{
    config.g = g; config.b = b; config.lds = lds; config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim *g, dim *b, size_t *lds, void **stream)
{
    *g = config.g; *b = config.b; *lds = config.lds; *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void *f, dim g, dim b, void **args, size_t lds, void *stream)
{
    return last = device_of(stream) == home ? 0 : 400;
}
int hipGetDevice(int *d) { *d = current; return 0; }
int hipSetDevice(int d) { current = d; return 0; }
int hipStreamGetDevice(void *stream, int *d) { *d = device_of(stream); return 0; }
int hipGetLastError(void)
{
    const int e = last;
    last = 0;
    return e;
}
int hipEventCreateWithFlags(int **e, unsigned flags)
{
    *e = malloc(sizeof(int));
    **e = current;
    return 0;
}
int hipEventCreate(int **e) { return hipEventCreateWithFlags(e, 0); }
int hipEventRecord(int *e, void *stream) { return *e == device_of(stream) ? 0 : 400; }
int hipEventSynchronize(int *e) { return 0; }
int hipEventDestroy(int *e) { free(e); return 0; }
int hipStreamIsCapturing(void *stream, int *status) { *status = 0; return 0; }
int hipStreamSynchronize(void *stream) { return 0; }
int hipHostMalloc(void **p, size_t n, unsigned flags) { *p = calloc(n, 1); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpy(void *to, const void *from, size_t n, int kind) { memcpy(to, from, n); return 0; }
int hipMemcpyAsync(void *to, const void *from, size_t n, int kind, void *stream)
{
    memcpy(to, from, n);
    return 0;
}
int hipMemsetAsync(void *p, int v, size_t n, void *stream) { memset(p, v, n); return 0; }

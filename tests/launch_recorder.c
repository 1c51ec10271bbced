// Stands in for the HIP runtime where no device is there: calls of the library run up to their launches, which are recorded instead.
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct { const void *kernel; uint32_t groups, threads; uint64_t lds; } launch_t;

launch_t recorded[1 << 16];
int n_recorded = 0;
struct { const void *kernel; int bytes; } allowed[256];
int n_allowed = 0;

static struct { dim3_t grid, block; size_t lds; void *stream; } pushed;

int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream) {
    pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream) {
    *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void *kernel, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream) {
    (void)args; (void)stream;
    if (n_recorded < (int)(sizeof recorded / sizeof recorded[0])) recorded[n_recorded++] = (launch_t){kernel, grid.x, block.x, lds};
    return 0;
}
int hipFuncSetAttribute(const void *kernel, int attribute, int value) {
    (void)attribute;
    if (n_allowed < 256) { allowed[n_allowed].kernel = kernel; allowed[n_allowed++].bytes = value; }
    return 0;
}
int hipGetDevice(int *device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int *value, int attribute, int device) { (void)attribute; (void)device; *value = 256; return 0; }
int hipGetLastError(void) { return 0; }
int hipMalloc(void **p, size_t n) { *p = malloc(n); return *p ? 0 : 2; }
int hipFree(void *p) { free(p); return 0; }
int hipMemcpyAsync(void *to, const void *from, size_t n, int kind, void *stream) {
    (void)to; (void)from; (void)n; (void)kind; (void)stream;
    return 0;
}
int hipStreamSynchronize(void *stream) { (void)stream; return 0; }

// Launches beyond what HIP takes: LDS past 64 KB that the kernel was not allowed, work-items past 32 bits, workgroups past 1024 or empty.
int launches_refused(void) {
    int refused = 0;
    for (int i = 0; i < n_recorded; ++i) {
        const launch_t *l = &recorded[i];
        uint64_t most = 65536;
        for (int j = 0; j < n_allowed; ++j)
            if (allowed[j].kernel == l->kernel && (uint64_t)allowed[j].bytes > most) most = (uint64_t)allowed[j].bytes;
        refused += l->lds > most || l->lds > 163840 || l->threads < 64 || l->threads > 1024 || l->groups < 1 ||
                   (uint64_t)l->groups * l->threads > 0xFFFFFFFFull;
    }
    return refused;
}

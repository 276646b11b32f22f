/* Stands in for the HIP runtime's launch path (loaded ahead of it): nothing is launched; each launch is held against what was asked for its
 * kernel with hipFuncSetAttribute.  Dynamic LDS beyond 64 KB has to have been asked for. */
#include <stddef.h>
#include <stdio.h>

typedef struct { unsigned x, y, z; } dim3;

enum { KERNELS = 4096, DYNAMIC_LDS = 8 };                  /* hipFuncAttributeMaxDynamicSharedMemorySize */
static const void* kernel[KERNELS];
static size_t asked[KERNELS];
static int kernels;
static struct { dim3 grid, block; size_t lds; void* stream; } call;
int recorded_launches, recorded_wide, recorded_unasked;
int recorded_last_grid, recorded_last_block, recorded_last_lds;

static size_t* of(const void* f) {
    int i = 0;
    while (i < kernels && kernel[i] != f) ++i;
    if (i == kernels && kernels < KERNELS) kernel[kernels++] = f;
    return &asked[i];
}
int hipFuncSetAttribute(const void* f, int attribute, int value) {
    if (attribute == DYNAMIC_LDS) *of(f) = (size_t)value;
    return 0;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) {
    call.grid = grid; call.block = block; call.lds = lds; call.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
    *grid = call.grid; *block = call.block; *lds = call.lds; *stream = call.stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, void* stream) {
    (void)args; (void)stream;
    ++recorded_launches;
    recorded_last_grid = (int)grid.x; recorded_last_block = (int)block.x; recorded_last_lds = (int)lds;
    if (lds > 64 * 1024) {
        ++recorded_wide;
        if (*of(f) < lds) {
            ++recorded_unasked;
            printf("kernel %p: %zu bytes of LDS, %zu asked for\n", f, lds, *of(f));
        }
    }
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipMalloc(void** p, size_t n) { (void)n; *p = (void*)(size_t)0x10000; return 0; }
int hipFree(void* p) { (void)p; return 0; }
int hipStreamIsCapturing(void* stream, int* status) { (void)stream; *status = 0; return 0; }
int hipStreamSynchronize(void* stream) { (void)stream; return 0; }

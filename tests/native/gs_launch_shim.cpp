// Stands in for the HIP runtime in front of the gradient search's host code
// (preloaded, no GPU): device copies are host copies, launches run nothing,
// and every limit that a kernel asks for and every launch's dynamic LDS is
// printed, with the kernel told apart by its address.
#include <cstdint>
#include <cstdio>
#include <cstring>

struct dim3 {
    uint32_t x, y, z;
};
static thread_local struct {
    dim3 grid, block;
    size_t lds;
    void *stream;
} cfg;

extern "C" {
int hipMemcpyAsync(void *dst, const void *src, size_t n, int, void *) {
    memcpy(dst, src, n);
    return 0;
}
int hipStreamSynchronize(void *) { return 0; }
int hipGetLastError() { return 0; }
int hipGetDevice(int *dev) {
    *dev = 0;
    return 0;
}
int hipDeviceGetAttribute(int *value, int, int) {
    *value = 256;  // the one that is asked for: compute units
    return 0;
}
int hipFuncSetAttribute(const void *f, int attr, int value) {
    printf("limit %p %d %d\n", f, attr, value);
    return 0;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) {
    cfg = {grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
    *grid = cfg.grid;
    *block = cfg.block;
    *lds = cfg.lds;
    *stream = cfg.stream;
    return 0;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t lds, void *) {
    printf("launch %p %u %u %zu\n", f, grid.x, block.x, lds);
    return 0;
}
}

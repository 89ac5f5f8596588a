// Records what the entry points of libsvdq.so ask of the HIP runtime, without a GPU: this program defines the few runtime
// functions that a forward calls, so the library, loaded below, binds to them instead of to the runtime's.  Nothing is
// launched and no pointer is followed.
//   argv[1]: the library.  stdin, one call a line:  device group M K N rank options
//            (group 64 INT4, 65 INT4 on the library's own workspace, 32 MXFP4, 0 INT8, 16 W4A16)
//   stdout:  "attr device kernel bytes" | "launch device kernel grid_x grid_y threads lds" | "status s", in order
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>

#include "../include/svdq.h"

struct dim3 { uint32_t x, y, z; };
static int g_device = 0;
static struct { dim3 grid, block; size_t lds; void *stream; } g_call;

extern "C" {
int hipGetDevice(int *d) { *d = g_device; return 0; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = (void *)0x20000000; return 0; }
int hipFuncSetAttribute(const void *f, int, int value) { printf("attr %d %p %d\n", g_device, f, value); return 0; }
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) { g_call = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
    *grid = g_call.grid; *block = g_call.block; *lds = g_call.lds; *stream = g_call.stream;
    return 0;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t lds, void *) {
    printf("launch %d %p %u %u %u %zu\n", g_device, f, grid.x, grid.y, block.x, lds);
    return 0;
}
}

typedef int (*forward_t)(const svdq_layer_dev *, const void *, int, void *, void *, size_t, void *);

int main(int argc, char **argv) {
    void *lib = argc > 1 ? dlopen(argv[1], RTLD_NOW) : nullptr;
    if (!lib) { fprintf(stderr, "%s\n", argc > 1 ? dlerror() : "no library"); return 2; }
    auto options = (int (*)(int))dlsym(lib, "svdq_forward_options");
    const forward_t int4 = (forward_t)dlsym(lib, "svdq_linear_forward"), fp4 = (forward_t)dlsym(lib, "svdq_fp4_linear_forward"),
                    w8a8 = (forward_t)dlsym(lib, "svdq_w8a8_linear_forward"), w4a16 = (forward_t)dlsym(lib, "svdq_w4a16_forward");
    auto own = (int (*)(const svdq_layer_dev *, const void *, int, void *, void *))dlsym(lib, "svdq_linear_forward_static");
    if (!options || !int4 || !fp4 || !w8a8 || !w4a16 || !own) return 3;
    int group, M, K, N, rank, opts;
    while (scanf("%d %d %d %d %d %d %d", &g_device, &group, &M, &K, &N, &rank, &opts) == 7) {
        char *at = (char *)0x10000000;      // aligned, never followed
        svdq_layer_dev layer;
        layer.rinv = at; layer.l1s = at; layer.l2 = at; layer.wcodes = at; layer.wscales = at; layer.bias = at;
        layer.shape = svdq_shape{K, N, rank, group == 16 || group == 65 ? 64 : group, 0.5f};
        options(opts);
        const forward_t f = group == 64 ? int4 : group == 32 ? fp4 : group == 0 ? w8a8 : w4a16;
        printf("status %d\n", group == 65 ? own(&layer, at, M, at, nullptr) : f(&layer, at, M, at, at, (size_t)1 << 40, nullptr));
        fflush(stdout);
    }
    return 0;
}

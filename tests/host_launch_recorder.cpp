// Records what the entry points of libsvdq.so ask of the HIP runtime, without a GPU: this program defines the few runtime
// functions that a forward calls, so the library, loaded below, binds to them instead of to the runtime's.  Nothing is
// launched and no pointer is followed.
//   argv[1]: the library.  stdin, one call a line:  device group M K N rank options output
//            (group 64 INT4, 65 INT4 on the library's own workspace, 32 MXFP4, 0 INT8, 16 W4A16;
//            output 0: memory of its own, 1: the same at an odd address, 2: the input's)
//   stdout:  "attr device kernel bytes" | "launch device kernel grid_x grid_y threads lds" | "status s", in order;
//            a kernel is its name with template arguments, e.g. act_wide_kernel<0>
#include <cxxabi.h>
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <map>
#include <string>

#include "../include/svdq.h"

struct dim3 { uint32_t x, y, z; };
static int g_device = 0;
static struct { dim3 grid, block; size_t lds; void *stream; } g_call;

static std::map<const void *, std::string> &names() {      // (filled while the library's constructors run)
    static std::map<const void *, std::string> m;
    return m;
}
static const char *name(const void *f) { return names().count(f) ? names()[f].c_str() : "?"; }

extern "C" {
void __hipRegisterFunction(void **, const void *f, char *, const char *mangled, unsigned, void *, void *, void *, void *, int *) {
    int status = 0;
    char *text = abi::__cxa_demangle(mangled, nullptr, nullptr, &status);
    std::string s = text ? text : mangled;      // "void svdq::(anonymous namespace)::act_wide_kernel<0>(svdq::ActParams)"
    free(text);
    for (const char *drop : {"void ", "svdq::", "(anonymous namespace)::"})
        for (size_t at; (at = s.find(drop)) != std::string::npos;) s.erase(at, std::string(drop).size());
    s.erase(s.find('('));
    for (size_t at; (at = s.find(' ')) != std::string::npos;) s.erase(at, 1);
    names()[f] = s;
}
int hipGetDevice(int *d) { *d = g_device; return 0; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = (void *)0x20000000; return 0; }
int hipFuncSetAttribute(const void *f, int, int value) { printf("attr %d %s %d\n", g_device, name(f), value); return 0; }
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) { g_call = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
    *grid = g_call.grid; *block = g_call.block; *lds = g_call.lds; *stream = g_call.stream;
    return 0;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t lds, void *) {
    printf("launch %d %s %u %u %u %zu\n", g_device, name(f), grid.x, grid.y, block.x, lds);
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
    int group, M, K, N, rank, opts, output;
    while (scanf("%d %d %d %d %d %d %d %d", &g_device, &group, &M, &K, &N, &rank, &opts, &output) == 8) {
        char *at = (char *)0x10000000, *ws = at + ((size_t)1 << 45);      // aligned, never followed
        char *y = output == 2 ? at : at + ((size_t)1 << 44) + 2 * output;
        svdq_layer_dev layer;
        layer.rinv = at; layer.l1s = at; layer.l2 = at; layer.wcodes = at; layer.wscales = at; layer.bias = at;
        layer.shape = svdq_shape{K, N, rank, group == 16 || group == 65 ? 64 : group, 0.5f};
        options(opts);
        const forward_t f = group == 64 ? int4 : group == 32 ? fp4 : group == 0 ? w8a8 : w4a16;
        printf("status %d\n", group == 65 ? own(&layer, at, M, y, nullptr) : f(&layer, at, M, y, ws, (size_t)1 << 40, nullptr));
        fflush(stdout);
    }
    return 0;
}

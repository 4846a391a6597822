// Loads the built library without a GPU and prints the launches its calls
// make: the HIP entry points below stand in for the runtime's (a program's own
// definitions come first in a shared library's symbol search), and a launch is
// recorded instead of run.  No pointer given to the library is dereferenced on
// the host.
// Usage: launch_drive LIB, then lines "OP WANT B C H W k corner" on stdin, OP
// backward (WANT: 1 dx, 2 dK, 3 both), forward, unit (the unit's forward) or step
// (the Step's forward, WANT the network's width); per line one output line
// "rc;kernel,blocks,threads,lds;..." (the kernel's mangled name).
// Test infrastructure: built and run by tests/test_launches_cpu.py.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdio.h>

#include <map>
#include <string>

#include "finc.h"

static std::map<const void *, std::string> &names() {
    static std::map<const void *, std::string> m;
    return m;
}
static std::string launches;
static struct {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
} pushed;

static void record(const void *f, dim3 g, dim3 b, size_t lds) {
    char s[512];
    snprintf(s, sizeof s, ";%s,%llu,%u,%zu", names()[f].c_str(),
             (unsigned long long)g.x * g.y * g.z, b.x * b.y * b.z, lds);
    launches += s;
}

extern "C" {
void **__hipRegisterFatBinary(const void *) {
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *,
                           void *, dim3 *, dim3 *, int *) {
    names()[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) {
    pushed = {g, b, lds, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *st) {
    *g = pushed.grid;
    *b = pushed.block;
    *lds = pushed.lds;
    *st = pushed.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t) {
    record(f, g, b, lds);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {   // LDS of a workgroup
    *v = 160 * 1024;
    return hipSuccess;
}
}

int main(int argc, char **argv) {
    void *lib = argc > 1 ? dlopen(argv[1], RTLD_NOW) : nullptr;
    if (!lib) {
        fprintf(stderr, "%s\n", argc > 1 ? dlerror() : "no library named");
        return 2;
    }
    auto backward = reinterpret_cast<decltype(&finc_backward)>(dlsym(lib, "finc_backward"));
    auto forward = reinterpret_cast<decltype(&finc_forward)>(dlsym(lib, "finc_forward"));
    auto unit = reinterpret_cast<decltype(&finc_unit_forward)>(dlsym(lib, "finc_unit_forward"));
    auto step = reinterpret_cast<decltype(&finc_step_forward)>(dlsym(lib, "finc_step_forward"));
    if (!backward || !forward || !unit || !step || names().empty())
        return 3;
    // buffers far apart, none of them there
    auto at = [](int i) { return reinterpret_cast<float *>((uintptr_t)(i + 1) << 40); };
    char op[32];
    int want, B, C, H, W, k, corner;
    while (scanf("%31s %d %d %d %d %d %d %d", op, &want, &B, &C, &H, &W, &k, &corner) == 8) {
        launches.clear();
        const std::string o = op;
        const int rc = o == "forward"
                           ? forward(at(0), at(1), at(2), nullptr, nullptr, B, C, H, W, k, corner,
                                     nullptr)
                       : o == "step"
                           ? step(at(0), at(1), nullptr, at(2), at(3), B, C, H, W, k, want, at(5),
                                  nullptr)
                       : o == "unit"
                           ? unit(at(0), at(1), at(2), nullptr, nullptr, B, C, H, W, k, nullptr)
                           : backward(at(0), at(1), at(2), want & 1 ? at(3) : nullptr,
                                      want & 2 ? at(4) : nullptr, -1.0, B, C, H, W, k, corner, at(5),
                                      nullptr);
        printf("%d%s\n", rc, launches.c_str());
    }
    return 0;
}

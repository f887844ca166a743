// Prints the launches that calls of the library make, without a GPU: this
// program's own definitions of the few runtime functions behind a launch take
// precedence over the runtime library's, and record instead of launching.
// Commands on standard input, one per line:
//   set OP DIM PHYSICS RULE DTYPE STRATEGY VEC WAVES BLOCKS_PER_CU
//   residual DIM PHYSICS RULE SPACE DTYPE N OFFSET      (P1)
//   backward DIM PHYSICS RULE SPACE DTYPE N OFFSET      (P1)
//   jacobian DIM PHYSICS RULE SPACE DTYPE N OFFSET ORDER
// OFFSET: words by which the arrays start off a page. A call prints "kernel
// grid.x grid.y block order", order being the kernel's second argument.
#include <cxxabi.h>
#include <stddef.h>
#include <stdint.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include "fem.h"

struct Dim3 { uint32_t x, y, z; };

static std::map<const void*, std::string>& kernels() {   // filled before main's own statics are
    static std::map<const void*, std::string>* m = new std::map<const void*, std::string>;
    return *m;
}

static struct { Dim3 grid, block; size_t lds; void* stream; } g_call;

extern "C" {
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, Dim3*, Dim3*, int*) {
    kernels()[host] = name;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
    g_call = {grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = g_call.grid;
    *block = g_call.block;
    *lds = g_call.lds;
    *stream = g_call.stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void** args, size_t, void*) {
    int status = 0;
    char* s = abi::__cxa_demangle(kernels()[f].c_str(), nullptr, nullptr, &status);
    std::string name = status == 0 ? s : kernels()[f];
    std::free(s);
    for (size_t p; (p = name.find(' ')) != std::string::npos;) name.erase(p, 1);
    name = name.substr(0, name.find('('));
    std::printf("%s %u %u %u %d\n", name.c_str(), grid.x, grid.y, block.x, *(const int*)args[1]);
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int* value, int, int) { *value = 256; return 0; }
}

int main() {
    char line[256], what[32];
    while (std::fgets(line, sizeof line, stdin)) {
        long long v[9] = {0};
        const int k = std::sscanf(line, "%31s %lld %lld %lld %lld %lld %lld %lld %lld %lld", what, v, v + 1, v + 2, v + 3, v + 4,
                                  v + 5, v + 6, v + 7, v + 8) - 1;
        fem_status st = FEM_ERR_INVALID_ARG;
        if (!std::strcmp(what, "set") && k == 9) {
            const fem_tuning t{(int)v[5], (int)v[6], (int)v[7], (int)v[8]};
            st = fem_set_tuning((int)v[0], (int)v[1], (int)v[2], (int)v[3], (int)v[4], &t);
        } else if (k >= 7) {
            // rows of an array are never touched here: any address will do
            void* p = (void*)(uintptr_t)(0x10000000 + v[6] * (v[4] == FEM_F32 ? 4 : 8));
            const int dim = (int)v[0], phys = (int)v[1], rule = (int)v[2], space = (int)v[3], dtype = (int)v[4];
            if (!std::strcmp(what, "residual"))
                st = fem_integrate_residual(dim, phys, rule, space, dtype, v[5], p, p, p, p, p, nullptr);
            else if (!std::strcmp(what, "backward"))
                st = fem_integrate_residual_backward(dim, phys, rule, space, dtype, v[5], p, p, p, p, p, p, p, nullptr);
            else if (!std::strcmp(what, "jacobian"))
                st = fem_integrate_jacobian(dim, phys, rule, space, (int)v[7], dtype, v[5], p, p, p, p, nullptr);
        }
        if (st != FEM_OK) {
            std::printf("error: %s", line);
            return 1;
        }
    }
    return 0;
}

// Runs calls of libdwt2.so on the host and prints the kernel launches they
// would make: this program's own hipLaunchKernel and what leads to it, which the
// library's launches resolve to, record a launch instead of enqueueing it.  Buffers are addresses
// that nothing reads.
//
// launch_trace LIB, then one call a line on stdin:
//   planes fwd|inv|adj WAVELET DTYPE PLANES H W LEVELS FLAGS
//   batch DTYPE LEVELS FLAGS COUNT H W [H W ...]      (COUNT times these sizes)
// prints for each call its status and per launch "offset:work-groups:threads",
// offset being the kernel's symbol within the library.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "dwt2.h"

namespace {
struct Launch {
    const void* f;
    uint64_t groups, threads;
};
std::vector<Launch> launches;
dim3 next_grid, next_block;
}  // namespace

extern "C" {
// the two halves of a launch statement
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
    next_grid = grid;
    next_block = block;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
    *grid = next_grid;
    *block = next_block;
    *lds = 0;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
    launches.push_back({f, (uint64_t)grid.x * grid.y * grid.z, (uint64_t)block.x * block.y * block.z});
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
// what a persistent launch asks for
hipError_t hipGetDevice(int* dev) {
    *dev = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 100000;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 2;
    return hipSuccess;
}
}

int main(int argc, char** argv) {
    void* lib = argc > 1 ? dlopen(argv[1], RTLD_NOW) : nullptr;
    if (!lib) {
        std::fprintf(stderr, "%s\n", argc > 1 ? dlerror() : "usage: launch_trace LIB");
        return 2;
    }
    char* const src = (char*)((uintptr_t)1 << 50);
    char* const dst = (char*)((uintptr_t)1 << 51);
    char* const ws = (char*)((uintptr_t)1 << 52);
    const size_t ws_bytes = (size_t)1 << 51;
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        std::string kind, dir;
        in >> kind;
        launches.clear();
        int st = -1000;
        if (kind == "planes") {
            int wav, dt, levels;
            int64_t planes, h, w;
            unsigned flags;
            in >> dir >> wav >> dt >> planes >> h >> w >> levels >> flags;
            auto fn = (decltype(&dwt2_fwd_planes))dlsym(lib, ("dwt2_" + dir + "_planes").c_str());
            if (in && fn)
                st = fn(src, dst, (int32_t)planes, h * w, h * w, (int32_t)h, (int32_t)w, w, w, (dwt2_dtype)dt,
                        (dwt2_wavelet)wav, levels, DWT2_SYMMETRIC_WHOLE, flags, ws, ws_bytes, nullptr);
        } else if (kind == "batch") {
            int dt, levels;
            unsigned flags;
            int64_t count, h, w, at = 0;
            in >> dt >> levels >> flags >> count;
            std::vector<dwt2_image> imgs;
            std::vector<std::pair<int64_t, int64_t>> sizes;
            while (in >> h >> w) sizes.push_back({h, w});
            for (int64_t k = 0; k < count; ++k)
                for (const auto& s : sizes) {
                    imgs.push_back({src + at, dst + at, (int32_t)s.first, (int32_t)s.second, s.second, s.second});
                    at += s.first * s.second * 4;
                }
            auto fn = (decltype(&dwt2_fwd_batched))dlsym(lib, "dwt2_fwd_batched");
            if (fn)
                st = fn(imgs.data(), (const dwt2_image*)ws, (int)imgs.size(), (dwt2_dtype)dt, DWT2_CDF97, levels,
                        DWT2_SYMMETRIC_WHOLE, flags, ws, ws_bytes, nullptr);
        }
        std::printf("%d", st);
        for (const Launch& l : launches) {
            Dl_info info{};
            dladdr(l.f, &info);
            std::printf(" %llx:%llu:%llu", (unsigned long long)((const char*)l.f - (const char*)info.dli_fbase),
                        (unsigned long long)l.groups, (unsigned long long)l.threads);
        }
        std::printf("\n");
    }
    return 0;
}

// for_each_launch: every launch is of fewer than 2^32 work-items, has a
// work-group for each of its tiles, and the launches cover every plane once; one
// plane with more tiles than a launch may have is refused.
#include <cstdio>

#include "dwt2_internal.h"

int main() {
    int bad = 0;
    for (int waves : {1, 4, 8, 12, 16})
        for (int64_t near : {2, 16, 74, 600})
            for (int64_t nt : {(int64_t)1, (int64_t)2, (int64_t)3, (int64_t)1000, (int64_t)999983,
                               dwt2::max_tiles(waves) / 2, dwt2::max_tiles(waves) / 2 + 1, dwt2::max_tiles(waves)})
                for (int64_t planes : {(int64_t)1, (int64_t)2, (int64_t)7, ((int64_t)1 << 23) - 1, (int64_t)1 << 23,
                                       (int64_t)9000000, (int64_t)0x7fffffff}) {
                    if (nt * planes >> 40) continue;
                    int64_t next = 0;
                    const hipError_t e = dwt2::for_each_launch(nt, near, waves, planes, [&](int64_t p0, int32_t n, dwt2::Deal d) {
                        bad += p0 != next || n < 1 || d.chunk < 1 || d.grid % (8 * d.chunk) != 0 || d.grid < nt * n ||
                               d.grid * waves * 64 >= (int64_t)1 << 32;
                        next = p0 + n;
                        return hipSuccess;
                    });
                    bad += e != hipSuccess || next != planes;
                }
    for (int waves : {4, 8, 16})
        bad += dwt2::for_each_launch(dwt2::max_tiles(waves) + 1, 2, waves, 1, [&](int64_t, int32_t, dwt2::Deal) {
                   return hipSuccess;
               }) == hipSuccess;
    std::printf("bad %d\n", bad);
    return bad != 0;
}

// Checks the launch grids of csrc/hga_device.hpp on the host: every workgroup
// number of a launch occurs, no dimension passes what the runtime takes, and a
// one-dimensional grid stays one.  Exit code 0: right.
#include "hga_device.hpp"

#include <cstdio>

int main() {
    const int64_t x_threads = int64_t(1) << 32;
    for (int threads : {64, 128, 256, 512, 640, 1024}) {
        const int64_t most = (x_threads - 1) / threads;
        for (int64_t n : {int64_t(1), int64_t(8), int64_t(77), most / 8 * 8 - 8, most / 8 * 8,
                          most / 8 * 8 + 1, most, most + 1, 2 * most, int64_t(1) << 30}) {
            const dim3 g = hga::grid_of(n, threads);
            const int64_t x = g.x, y = g.y;
            const bool ok = x * threads < x_threads && y <= 65535 && g.z == 1 && x * y >= n &&
                            x * y < int64_t(1) << 31 && x * (y - 1) < n &&
                            (y == 1 ? x == n : x % 8 == 0 && x == hga::grid_row(threads));
            if (ok) continue;
            std::printf("%lld workgroups of %d: %u x %u x %u\n", static_cast<long long>(n), threads, g.x,
                        g.y, g.z);
            return 1;
        }
    }
    return 0;
}

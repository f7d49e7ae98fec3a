"""Index arithmetic of device loops, compiled for the host and run over the
sizes where 32 bits are too few."""
import os
import subprocess


def test_sample_walk_of_the_tile_kernel_stays_in_bounds(tmp_path):
    """The device walk over samples, compiled for the host: every workgroup
    leaves its loop, never at a negative sample, all samples are taken once,
    and a forward launch has fewer than 2^32 threads, also for 2^30 and more
    samples (where 32-bit sample numbers wrap)."""
    src = tmp_path / "walk.cpp"
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_14340_amd", "csrc")
    src.write_text(r'''
#include "mlp_walk.h"
#include <cstdio>
using namespace jk;
int main() {
    const int ns[] = {1, 15, 16, 17, 1024, 1025, 1 << 24, (1 << 24) + 1, 1 << 28, (1 << 30) - 1, (1 << 30) + 1,
                      1073741872, INT32_MAX - 15, INT32_MAX};
    const int64_t limits[] = {64, kMlpMaxForward};
    for (int64_t most : limits)
        for (int n : ns) {
            const unsigned groups = mlp_groups(n, most);
            if ((int64_t)groups * kMlpThreads >= (int64_t)1 << 32) return std::printf("threads n=%d\n", n), 1;
            int64_t taken = 0;
            for (unsigned g = 0; g < groups; ++g) {
                int64_t steps = 0;
                for (int64_t b = mlp_first(g); b < n; b = mlp_next(b, groups)) {
                    if (b < 0 || ++steps > mlp_tiles(n)) return std::printf("walk n=%d\n", n), 1;
                    taken += n - b < kMlpTile ? n - b : kMlpTile;
                }
            }
            if (taken != n) return std::printf("taken n=%d\n", n), 1;
        }
    return 0;
}
''')
    exe = str(tmp_path / "walk")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", csrc, str(src), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout

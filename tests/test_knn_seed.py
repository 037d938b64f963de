"""The particles that the nearest-neighbour kernels start their lists from, on the CPU: the
index functions of the kernels' own header, for every lane of the first and last wavefronts
and every k, stay inside the particle array and name the neighbours of the sorted order."""
import os
import subprocess

from paper_1312_1128_amd import build_ext

MAIN = r"""
#include <stdio.h>

#include "knn_list.hpp"

int main()
{
    const int64_t sizes[] = {2, 3, 33, 63, 64, 65, 66, 127, 128, 129, 1000, 4097, 2147483647ll - 64, 2147483647ll};
    for (const int64_t n : sizes)
        for (int64_t g0 = 0; g0 < n; g0 += 64) {
            if (g0 > 4 * 64 && g0 < n - 4 * 64) g0 = (n - 4 * 64) / 64 * 64;
            for (int lane = 0; lane < 64; ++lane) {
                const int64_t j = g0 + lane < n ? g0 + lane : g0;
                if (glm::knn_particle((int)g0, lane, (int)n) != j) return printf("particle %lld %lld %d\n", (long long)n, (long long)g0, lane), 1;
                for (int o = 1; o <= 64; ++o) {
                    const glm::KnnSeed s = glm::knn_seed((int)j, o, (int)n);
                    const bool before = j - o >= 0, after = j + o < n;
                    if (s.has_before != before || s.has_after != after || s.before != (before ? j - o : j) ||
                        s.after != (after ? j + o : j))
                        return printf("seed %lld %lld %d\n", (long long)n, (long long)j, o), 1;
                }
            }
        }
    return 0;
}
"""


def test_seeds_stay_inside_the_particles(tmp_path):
    src, exe = tmp_path / "seed.hip", tmp_path / "seed"
    src.write_text(MAIN)
    cmd = [build_ext.hipcc(), "--offload-host-only", "-O1", "-std=c++17", f"-I{build_ext.CSRC}",
           f"-I{os.path.join(build_ext.ROOT, 'include')}", str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout

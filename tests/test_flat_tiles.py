"""Host check of the chunks a flat chunked tile loads (step_kernel.hpp's own
flat_first and flat_load): every index lies in the arrays, also where a tile's
rows, the last ones of the last network among them, have no connections."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "step_kernel.hpp"
int main() {
    using namespace infoli;
    long loads = 0, empty = 0;
    for (int n : {1, 7, 64, 65, 300})
        for (int rows : {1, 8, 100, 256})
            for (int isolated = 0; isolated <= n; isolated += 1 + n / 9)     // the last rows
                for (int deg : {1, 8, 9, 200}) {
                    std::vector<int> ca(n + 1, 0);
                    for (int i = 0; i < n; ++i) ca[i + 1] = ca[i] + (i < n - isolated ? (deg + kChunkCols - 1) / kChunkCols : 0);
                    const long network = 3, total = network + ca[n];    // three chunks of another network ahead
                    for (int r0 = 0; ca[n] > 0 && r0 < n; r0 += rows) {
                        const int r1 = r0 + rows < n ? r0 + rows : n;
                        const int m = ca[r1] - ca[r0];
                        const long first = flat_first(network, ca[r0], m);
                        for (int base = 0; base == 0 || base < m; base += kFlatChunks * 256)
                            for (int k = base; k < base + kFlatChunks * 256; ++k) {
                                const int i = flat_load(k, m);
                                if (i < 0 || first < 0 || first + i >= total || (k < m && first + i != network + ca[r0] + k)) {
                                    std::printf("n %d rows %d tile %d chunks %d slot %d: %d\n", n, rows, r0, m, k, i);
                                    return 1;
                                }
                                ++loads;
                                empty += m == 0;
                            }
                    }
                }
    std::printf("%ld %ld\n", loads, empty);
    return 0;
}
"""


def test_every_load_lies_in_the_chunks(tmp_path):
    src, exe = tmp_path / "flat.hip", tmp_path / "flat"
    src.write_text(PROGRAM)
    subprocess.run(["hipcc", "--offload-host-only", "-std=c++17", "-O1", "-I",
                    os.path.join(ROOT, "paper_1612_01501_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    loads, empty = (int(x) for x in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert loads > empty > 0

"""CPU-only check of the rules that pick the register-ring kernels: their 32-bit
byte offsets reach fields of less than 4 GiB, so on larger ones (the library
takes grids of up to 2^31 cells) the other kernels have to run.

The rules are C++ functions of the built library; a small host program asks
them about grids of 2^29 and 2^30 cells and a little less and more, with the
tiles that the launches use.
"""
import os
import subprocess

import pytest

from paper_2204_02107_amd import build

LIB = build.LIB

PROGRAM = r"""
#include <cstdio>
#include "stencil.h"
using namespace dnslab;
int main() {
    const int grids[][3] = {{972, 972, 486}, {1024, 1024, 512}, {972, 972, 576}, {864, 864, 864},
                            {1296, 972, 768}, {1024, 1024, 1024}, {972, 1296, 864}};
    for (const auto& n : grids) {
        Grid g = {};
        g.nx = n[0]; g.ny = n[1]; g.nz = n[2];
        g.nxy = (long long)g.nx * g.ny;
        g.n = g.nxy * g.nz;
        const StencilLaunch pair = stencil_launch(g, DNSLAB_PROWS, 64, 1), ring = stencil_launch(g, DNSLAB_FROWS, 64, 1);
        for (size_t esz : {sizeof(double), sizeof(float)})
            std::printf("%d %d %d %zu %d %d %d\n", g.nx, g.ny, g.nz, esz, (int)mom_pair_supported(g, pair, esz),
                        (int)filter_ring_supported(g, ring, esz), (int)correct_ring_supported(g, ring, esz));
    }
}
"""


@pytest.mark.skipif(not os.path.exists(LIB), reason="libdnslab.so not built")
def test_ring_kernels_stop_at_four_gib(tmp_path):
    src, exe = tmp_path / "rules.hip", tmp_path / "rules"
    src.write_text(PROGRAM)
    where = os.path.dirname(LIB)
    subprocess.run([build.hipcc(), "-std=c++17", "--offload-host-only", "-I", build.CSRC, "-I", build.INCLUDE, str(src),
                    "-o", str(exe), f"-L{where}", "-ldnslab", f"-Wl,-rpath,{where}"], check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    rows = [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    assert len(rows) == 14
    for nx, ny, nz, esz, *picked in rows:
        fits = nx * ny * nz * esz < 1 << 32
        assert picked == [fits] * 3, (nx, ny, nz, esz, picked)

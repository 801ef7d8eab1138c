"""Grid sizes of a batch's copy launches (no GPU needed): below 2^32 threads for
every problem count a batch may have, however large its largest grid, and a
thread for every cell or row of few and small grids."""
import os
import subprocess

from paper_2306_13002_amd import build as B, stencil as S

PROGRAM = r"""
#include <array>
#include <cstdio>
#include "internal.hpp"
int main() {
    for (long long n : {1LL, 64LL, 1LL << 16, 1LL << 17, (1LL << 20) - 1, 1LL << 20})
        for (long long largest : {1LL, 2048LL, 64LL * 64 * 64, 160LL * 160 * 160, 1LL << 40})
            std::printf("%lld %lld %d\n", n, largest, stn::batch_copy_chunks(n, largest));
    for (auto e : {std::array<int, 3>{13, 10, 63}, {7, 276, 20}, {5000, 3, 2}, {1, 1, 1}, {2, 200, 200}}) {
        stn::Geom g{};
        g.nx = e[0], g.ny = e[1], g.nz = e[2], g.r = 1;
        for (bool tail : {false, true})
            std::printf("%d %d %d %d %lld %d\n", e[0], e[1], e[2], tail, stn::batch_copy_work(tail, g),
                        stn::batch_copy_chunks(1, stn::batch_copy_work(tail, g)));
    }
}
"""


def test_copy_grids_fit_a_launch(tmp_path):
    S.lib()
    src, exe = tmp_path / "chunks.cpp", tmp_path / "chunks"
    src.write_text(PROGRAM)
    flags = [f for f in B.CXXFLAGS if not f.startswith("--offload-arch")]
    subprocess.run([B.hipcc(), "-x", "hip", "--offload-host-only", *flags, "-I", B.CSRC, str(src), "-x", "none", "-o",
                    str(exe), B.LIB, "-Wl,-rpath," + os.path.dirname(B.LIB)], check=True, capture_output=True, timeout=300)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=120).stdout
    rows = [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    sizes, copies = [r for r in rows if len(r) == 3], [r for r in rows if len(r) == 6]
    assert len(sizes) == 30 and len(copies) == 10
    for n, largest, c in sizes:
        assert 1 <= c <= 65536 and n * c * 256 < 2 ** 32
    assert (64, 160 ** 3, 4000) in sizes  # four elements per thread where the problems are few
    for nx, ny, nz, tail, work, c in copies:
        # one wave per row (per 256 cells of a row longer than 1024), one thread per cell
        pieces = 1 if nx + 2 <= 1024 else -(-(nx + 2) // 256)
        need = nx * ny * nz if tail else max(64 * pieces * (2 * (ny + 2) + 2 * nz), 2 * ny * nz)
        assert work == need and c * 256 >= need

"""Grid sizes of a batch's copy launches (no GPU needed): below 2^32 threads for
every problem count a batch may have, however large its largest grid."""
import os
import subprocess

from paper_2306_13002_amd import build as B, stencil as S

PROGRAM = r"""
#include <cstdio>
#include "internal.hpp"
int main() {
    for (long long n : {1LL, 64LL, 1LL << 16, 1LL << 17, (1LL << 20) - 1, 1LL << 20})
        for (long long largest : {1LL, 2048LL, 64LL * 64 * 64, 160LL * 160 * 160, 1LL << 40})
            std::printf("%lld %lld %d %d\n", n, largest, stn::batch_copy_chunks(true, n, largest),
                        stn::batch_copy_chunks(false, n, largest));
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
    assert len(rows) == 30
    for n, largest, tail, halo in rows:
        for c in (tail, halo):
            assert 1 <= c <= 1024 and n * c * 256 < 2 ** 32
    assert (64, 160 ** 3, 1024, 250) in rows  # about eight elements per thread where the problems are few

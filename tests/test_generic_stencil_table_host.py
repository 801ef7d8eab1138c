"""The process's table of GENERIC stencils (no GPU needed): one entry per
stencil, whatever the pitch and extents of the grids planned with it."""
import os
import subprocess

from paper_2306_13002_amd import build as B, stencil as S

PROGRAM = r"""
#include <cstdio>
#include "internal.hpp"
#include "rtc.hpp"
using namespace stn;
int main() {
    for (int coef = 1; coef <= 2; ++coef)
        for (long long pitch : {66, 130, 131, 1 << 20, 1 << 28}) {
            RtcSpec sp;
            sp.R = 1;
            sp.row_bytes = pitch * 8;
            sp.slots.resize(3);
            for (auto &s : sp.slots) s.push_back({0.25 * coef, {{-1, 0}, {1, 0}}});
            Geom g{};
            g.nx = 64; g.ny = 40; g.nz = 30; g.r = 1; g.py = pitch; g.pz = pitch * 42;
            const Tile t = rtc_default_tile(sp, g);
            const bool wide = rtc_generic_source(sp, t.tx, t.ty, gen_rows(t.tx, t.ty)).find("unsigned long long>") != std::string::npos;
            std::printf("%d %d\n", (int)rtc_stencils(), (int)wide);
        }
}
"""


def test_one_entry_per_stencil(tmp_path):
    S.lib()
    src, exe = tmp_path / "table.cpp", tmp_path / "table"
    src.write_text(PROGRAM)
    flags = [f for f in B.CXXFLAGS if not f.startswith("--offload-arch")]
    subprocess.run([B.hipcc(), "-x", "hip", "--offload-host-only", *flags, "-I", B.CSRC, str(src), "-x", "none", "-o",
                    str(exe), B.LIB, "-Wl,-rpath," + os.path.dirname(B.LIB)], check=True, capture_output=True, timeout=300)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=120).stdout.splitlines()
    assert out == ["1 0", "1 0", "1 0", "1 0", "1 1"] + ["2 0", "2 0", "2 0", "2 0", "2 1"]

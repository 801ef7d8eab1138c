"""What a tuned plan launches beside its pick (settle_run; no GPU needed): only
a launch that leaves the reported form's grids, bit for bit.  The cases run in
a small host program linked with the library."""
import os
import subprocess

from paper_2306_13002_amd import build as B, stencil as S

PROGRAM = r"""
#include <cstdio>
#include "tune.hpp"
using namespace stn;
struct Case { int kind; std::vector<Cand> cands; std::vector<double> us; std::vector<Cand> runs; std::vector<double> run_us; };
int main() {
    const Tile p{64, 4, 1}, s{32, 8, 8}, t{28, 28, 8}, r{62, 14, 4}, m{5, 16, 0};
    const int h2 = STENCIL_HEAT2D5, h3 = STENCIL_HEAT3D7;
    const std::vector<Case> cases = {
        {h3, {{V_PLAIN, p, 0}, {V_SATURATED, s, 1}, {V_SAT3, t, 0}}, {1.0, 3.0, 2.0}, {{V_SATURATED, r, 1}}, {0.5}},
        {h3, {{V_PLAIN, p, 0}, {V_SATURATED, s, 1}}, {1.0, 3.0}, {{V_SATURATED, r, 1}}, {1.5}},
        {h3, {{V_PLAIN, p, 0}}, {1.0}, {{V_SATURATED, r, 1}}, {0.5}},
        {h3, {{V_PLAIN, p, 0}, {V_SAT2, s, 1}}, {4.0, 1.0}, {{V_SATURATED, r, 1}, {V_SAT3, r, 1}}, {0.9, 0.5}},
        {h3, {{V_PLAIN, p, 0}}, {1.0}, {}, {}},
        {h2, {{V_PLAIN, p, 0}}, {1.0}, {{V_MARCH, m, 0}}, {0.5}},
    };
    for (const Case &c : cases) {
        std::vector<std::pair<double, size_t>> timed;
        for (size_t i = 0; i < c.us.size(); ++i) timed.push_back({c.us[i], i});
        std::sort(timed.begin(), timed.end());
        const Cand &b = c.cands[timed[0].second];
        TuneEntry e{b.variant, b.tile, b.remap, timed[0].first};
        settle_run(c.kind, c.cands, timed, c.runs, c.run_us, &e);
        std::printf("%d %d %d %d %g %d %d\n", e.variant, e.tile.tx, e.tile.tz, e.remap, e.us, e.run_variant, e.run_tile.tx);
    }
}
"""

# reported form, its tile x and z, map, us; launched form (-1: the reported one) and tile x
WANT = ["7 28 8 0 2 1 62",   # a faster saturated launch: the fastest saturated candidate is reported
        "0 64 1 0 1 -1 0",   # slower than the PLAIN pick: not taken
        "0 64 1 0 1 -1 0",   # no saturated candidate to report: not taken
        "6 32 8 1 1 7 62",   # the saturated forms stand for each other
        "0 64 1 0 1 -1 0",
        "0 64 1 0 1 8 5"]    # HEAT2D5 PLAIN marches


def test_launches_keep_the_reported_result(tmp_path):
    S.lib()
    src, exe = tmp_path / "pick.cpp", tmp_path / "pick"
    src.write_text("#include <algorithm>\n" + PROGRAM)
    flags = [f for f in B.CXXFLAGS if not f.startswith("--offload-arch")]
    subprocess.run([B.hipcc(), "-x", "hip", "--offload-host-only", *flags, "-I", B.CSRC, str(src), "-x", "none", "-o", str(exe),
                    B.LIB, "-Wl,-rpath," + os.path.dirname(B.LIB)], check=True, capture_output=True, timeout=300)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=120).stdout
    assert out.strip().splitlines() == WANT

"""What the kernels' launches reserve of the LDS, front by front, against the
budget that the symbolic analysis gave the fronts (no GPU).

For every front of at most 128 columns that fits a budget as the analysis counts
it: the factor launches (column-major or blocked panel) reserve at most 5,288
bytes past the budget and the sweeps 376, as the header of kkt_options says, and
none more than a workgroup may have; the blocked panel of every front that the
panel waves cover is reserved in full.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2403_15913_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "lds_layout.hpp"
using namespace kkt;
int main() {
    const int full = 158 * 1024, budgets[] = {4096, 5 * 1024, 8192, 16 * 1024, 36000, 79 * 1024, full};
    const long over_factor = 5288, over_sweep = 376;
    long fronts = 0, blocked = 0, bad = 0, most_factor = 0, most_sweep = 0;
    for (const int budget : budgets)
        for (int c = 1; c <= 128; c++)
            for (int r = c; front_lds_bytes(r, c) <= budget; r++) {
                fronts++;
                const long got = factor_launch_lds_bytes(r, c);
                const long sweep = fwd_lds_bytes(r, c) > bwd_lds_bytes(r, c) ? fwd_lds_bytes(r, c) : bwd_lds_bytes(r, c);
                // panel waves: one per 64 rows below the first diagonal block
                const int rt = 16 * ((c + 15) / 16 + (r - c + 15) / 16), waves = (rt - 16 + 63) / 64;
                for (int maxp = 3; maxp <= 4; maxp++) {
                    const bool is = front_blocked(r, c, maxp);
                    blocked += is;
                    if (is != (waves <= maxp) || (is && got < blocked_lds_bytes(r, c))) bad++;
                }
                if (got - budget > most_factor) most_factor = got - budget;
                if (sweep - budget > most_sweep) most_sweep = sweep - budget;
                if (got < factor_lds_bytes(r, c) || got > budget + over_factor || sweep > budget + over_sweep ||
                    got > full || sweep > full + 1024) {
                    if (bad++ < 5) std::printf("budget %d: front %d x %d reserves %ld, sweep %ld\n", budget, r, c, got, sweep);
                }
            }
    std::printf("%ld fronts, %ld blocked, %ld bad, most past the budget %ld and %ld\n", fronts, blocked, bad, most_factor, most_sweep);
    return bad != 0 || fronts == 0 || blocked == 0;
}
"""


def test_launches_keep_the_budget(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "budget.cpp", tmp_path / "budget"
    src.write_text(PROGRAM)
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout

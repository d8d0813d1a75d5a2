"""The cell of the Maxwell table that the step kernels look a temperature up in, compiled for the host with traps on
conversions that are not defined: every temperature a node can reach, NaN and infinities among them, gives a cell
inside the table."""
import os
import subprocess

import pytest

from paper_1705_10045_amd import build

PROGRAM = r"""
#include "physics.hpp"
#include <cstdio>
#include <cmath>
#include <limits>
int main()
{
    using namespace lbm;
    const double s0 = std::sqrt(1.0 - kLatentTmax), ds = (std::sqrt(1.0 - kLatentTmin) - s0) / (kMaxwellPoints - 1);
    const double inf = std::numeric_limits<double>::infinity();
    const double Tr[] = {0.4, 0.5, 0.8, 0.95, 0.9985, 0.998999, 0.999, 1.0, 1.0000001, 1.3, 50.0, 1e30, 1e300, inf, -inf,
                         std::nan(""), 0.39999, 0.1, 0.0, -0.0, -1.0, -1e12, -1e30, -1e300, 5e-324};
    for (double T : Tr) {
        int j = -7;
        double t;
        const bool band = band_cell(T, s0, 1.0 / ds, j, t);
        const double pos = (std::sqrt(1.0 - T) - s0) / ds;
        if (j < 1 || j > kMaxwellPoints - 3) { printf("cell %d of T %g\n", j, T); return 1; }
        if (band != (T >= kLatentTmin && T < kLatentTmax)) { printf("band of T %g\n", T); return 1; }
        if (band && !(std::fabs(j + t - pos) < 1e-9 * kMaxwellPoints && t > -1.0 - 1e-9 && t < 2.0 + 1e-9)) {
            printf("T %.17g: cell %d offset %g position %.17g\n", T, j, t, pos);
            return 1;
        }
    }
    return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
def test_every_temperature_has_a_cell(tmp_path):
    src, exe = tmp_path / "cell.hip", tmp_path / "cell"
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, "--offload-arch=" + build.ARCH, "-std=c++17", "-O1", "-I", build.CSRC,
                    "-Xarch_host", "-fsanitize=float-cast-overflow", "-Xarch_host", "-fsanitize-trap=float-cast-overflow",
                    "-o", str(exe), str(src)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout)

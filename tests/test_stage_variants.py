"""The compiled variants of the stage kernel differ from one another at every
degree and in both precisions: two with the same workgroup size, register
budget, partner unroll and staging rows are one kernel, which the autotuner
would time twice.  The configurations are read from the kernel header by a
host-only program."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "esdg_kernels.hpp"
using namespace esdg;
template <int N, int V>
void show()
{
    using C = StageCfg<N, V>;
    printf("%d 64 %d %d %d %d %d %d\n", N, V, C::T, StageWaves<N, double, 1, V>::value, C::VU, C::PAD, (int)C::SWZ);
    printf("%d 32 %d %d %d %d %d %d\n", N, V, C::T, StageWaves<N, float, 1, V>::value, C::VU32, C::PAD, (int)C::SWZ);
    if constexpr (V + 1 < kStageVariants) show<N, V + 1>();
    else if constexpr (N < kMaxN) show<N + 1, 0>();
}
int main() { show<2, 0>(); }
"""


@pytest.fixture(scope="module")
def table(tmp_path_factory):
    from paper_1804_02221_amd import build
    d = tmp_path_factory.mktemp("variants")
    (d / "show.hip").write_text(PROGRAM)
    exe = str(d / "show")
    flags = [f for f in build.FLAGS if f not in ("-O3", "-fPIC")]
    r = subprocess.run([build.HIPCC, *flags, "-O0", "--cuda-host-only", str(d / "show.hip"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    rows = [tuple(map(int, l.split())) for l in subprocess.check_output([exe], text=True).splitlines()]
    return {(r[0], r[1], r[2]): r[3:] for r in rows}


@pytest.mark.parametrize("precision", [64, 32])
def test_no_two_variants_are_one_kernel(table, precision):
    from paper_1804_02221_amd import esdg
    for N in range(2, 9):
        cfg = [table[N, precision, v] for v in range(esdg.STAGE_VARIANTS)]
        assert len(set(cfg)) == len(cfg), (N, cfg)

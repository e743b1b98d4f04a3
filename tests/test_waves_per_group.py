"""The number of waves that share one group's list (csrc/waves.h), compiled for
the host: lists of few tiles and trees that fill the chip take one wave, whose
kernels were up to 2.7 times as fast there as those of four and eight; small
trees with work for them take more.  The benchmark names the same instances."""
import os
import subprocess

import pytest

import bench

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1211_4406_amd", "csrc")
# groups, mean entries, mean targets: waves of force, adjoint, quadrupole pass
SETS = [
    ((20000, 39, 1), (1, 1, 1)),          # single-particle groups
    ((6591, 87, 3), (1, 1, 1)),
    ((3444, 144, 5.8), (1, 1, 1)),
    ((1628, 216, 12.3), (1, 1, 1)),
    ((35405, 227, 11.3), (1, 1, 1)),
    ((16463, 385, 24.3), (1, 1, 1)),
    ((43303, 425, 46.2), (1, 1, 1)),
    ((21139, 515, 47.3), (1, 1, 1)),
    ((11262, 573, 45.5), (1, 1, 1)),
    ((42, 453, 47.6), (8, 8, 8)),         # small trees of full groups
    ((250, 1517, 40.0), (8, 8, 8)),
    ((2061, 383, 24.3), (4, 4, 4)),
    ((3063, 1642, 42.8), (4, 4, 4)),
    ((12715, 1504, 41.2), (4, 4, 1)),     # long lists
    ((24459, 1626, 42.9), (4, 4, 1)),
    ((33441, 1433, 62.7), (4, 1, 1)),
    ((265000, 1424, 63.3), (1, 1, 1)),
]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("waves")
    src = d / "waves.cpp"
    src.write_text(f"""#include "{CSRC}/waves.h"
#include <cstdio>
int main() {{
    long long g, e, i;
    while (std::scanf("%lld %lld %lld", &g, &e, &i) == 3)
        std::printf("%d %d %d\\n", srf::waves_per_group(g, e, i, srf::kForceReach),
                    srf::waves_per_group(g, e, i, srf::kAdjointReach), srf::waves_per_group(g, e, i, srf::kQuadrupoleReach));
}}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-o", str(d / "waves"), str(src)], check=True)
    return str(d / "waves")


def test_waves_of_measured_sets(rule):
    rows = [(g, round(g * e), round(g * e * t)) for (g, e, t), _ in SETS]
    out = subprocess.run([rule], input="\n".join("%d %d %d" % r for r in rows), capture_output=True, text=True, check=True)
    got = [tuple(int(v) for v in line.split()) for line in out.stdout.split("\n") if line]
    assert got == [w for _, w in SETS]
    for (g, e, i), w in zip(rows, got):
        info = dict(n_groups=g, n_particle_entries=e, n_node_entries=0, interactions=i)
        assert (bench.waves_per_group(info, 26.0), bench.waves_per_group(info, 18.0)) == w[:2]

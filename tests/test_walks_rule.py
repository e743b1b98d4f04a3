"""Which walk builds the lists (csrc/walks.h), compiled for the host, on trees
that both walks were timed on: short lists in large trees go to the threads,
whose walk took as little as 0.43 of the waves' time there; small trees and
long lists to the waves (down to 0.36 of the threads')."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1211_4406_amd", "csrc")
UNIFORM = [1, 8, 64, 512, 4096, 32768]
# n, groups, n_leaf, cutoff (spacings), cells of each level, by waves
TREES = [
    (20000, 500, 16, 1.6, [1, 8, 64, 512, 4000], True),
    (190000, 62071, 4, 1.6, UNIFORM + [50000, 9000], True),
    (8000000, 133334, 16, 3.0, [1, 8, 64, 512, 4096, 32176, 104405, 129298, 132820, 133273, 133328, 1066245, 6356], False),
    (8000000, 160866, 16, 3.0, [1, 8, 64, 512, 4096, 23109, 37110, 39641, 39952, 39994, 40000, 320000, 2367516, 7], False),
    (8000000, 170688, 16, 3.0, [1, 8, 64, 512, 3527, 7110, 7871, 7991, 8000, 8000, 8000, 64000, 511999, 1501546], False),
    (190000, 190000, 1, 1.6, [1, 8, 64, 512, 4096, 32676, 134319, 89967, 15361, 2052, 244, 27, 1, 2], False),
    (1000000, 168001, 8, 1.6, UNIFORM + [256343, 24697], False),
    (8000000, 169344, 16, 1.6, UNIFORM + [262144, 2045068, 7], True),
    (4000000, 178839, 8, 2.75, UNIFORM + [262036, 679914, 122018, 190105, 208298, 160638, 85874, 7398], True),
    (8000000, 185791, 16, 5.0, UNIFORM + [262143, 866703, 145991, 222552, 241588, 182302, 96597, 6991], True),
    (12000000, 262898, 16, 4.0, UNIFORM + [262144, 2090214, 1782], False),
    (16777216, 265973, 16, 6.0, UNIFORM + [262144, 2097152], False),
    (13000000, 299593, 16, 2.75, UNIFORM + [262144, 1960338, 217497, 328293, 409989, 325341, 197271, 33468], True),
    (16000000, 321748, 16, 3.0, [1, 8, 64, 512, 4096, 29851, 68991, 78556, 79820, 79980, 79999, 639992, 4734331, 14], False),
    (1000000, 330377, 4, 2.75, UNIFORM + [226859, 93667, 58383, 83518, 75937, 55818, 22062, 933], False),
    (400000, 400000, 1, 2.75, UNIFORM[:5] + [32699, 146745, 128541, 67123, 69084, 64336, 47608, 24259, 5960, 851, 85, 14], False),
]


def by_waves(trees, where):
    """Whether waves walk the trees (n, groups, n_leaf, cutoff, theta, cells of each level)."""
    src = where / "walks.cpp"
    src.write_text(f"""#include "{CSRC}/walks.h"
#include <cstdio>
int main() {{
    long long n, ng;
    int leaf, max_level;
    double rc, th;
    while (std::scanf("%lld %lld %d %lf %lf %d", &n, &ng, &leaf, &rc, &th, &max_level) == 6) {{
        int32_t cells[22] = {{0}};
        for (int L = 0; L <= max_level; ++L) if (std::scanf("%d", &cells[L]) != 1) return 1;
        std::printf("%d ", srf::may_wave_walk(n, ng, leaf, max_level) && srf::wave_walk(n, ng, cells, max_level, rc, th));
    }}
}}
""")
    exe = str(where / "walks")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-o", exe, str(src)], check=True)
    rows = "\n".join(" ".join(str(v) for v in (n, ng, leaf, rc, th, len(c) - 1, *c)) for n, ng, leaf, rc, th, c in trees)
    out = subprocess.run([exe], input=rows, capture_output=True, text=True, check=True).stdout.split()
    return [v == "1" for v in out]


def test_walks_of_timed_trees(tmp_path):
    got = by_waves([(n, ng, leaf, rc * n ** (-1 / 3), 0.5, c) for n, ng, leaf, rc, c, _ in TREES], tmp_path)
    assert got == [t[-1] for t in TREES]

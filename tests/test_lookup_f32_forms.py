"""The rule that chooses an unquantised lookup's form (csrc/lookup_f32_forms.h), compiled alone (no GPU needed)."""
import os
import subprocess

import pytest

from paper_2302_03213_amd import build

PROGRAM = r"""
#include <cstdio>
#include "lookup_f32_forms.h"
int main() {
    int C, K, M, rows_ok;
    long long N;
    const char* names[] = {"gather", "rows", "matrix"};
    while (std::scanf("%lld %d %d %d %d", &N, &C, &K, &M, &rows_ok) == 5) {
        const lutnn::LookupF32Us us = lutnn::lookup_f32_us(C, K, M, N, rows_ok != 0, 256);
        std::printf("%s %.17g %.17g %.17g\n", names[(int)us.least(N, M)], us.gather, us.rows, us.matrix);
    }
}
"""


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    folder = tmp_path_factory.mktemp("forms")
    (folder / "forms.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", build.CSRC, "-o", str(folder / "forms"), str(folder / "forms.cpp")], check=True)

    def run(shapes):
        text = "".join("%d %d %d %d %d\n" % s for s in shapes)
        out = subprocess.run([str(folder / "forms")], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        return [(l.split()[0], dict(zip(("gather", "rows", "matrix"), map(float, l.split()[1:])))) for l in out if l]
    return run


def rows_ok(N, K, M):
    """rows_kernel_preferred for fp32."""
    return N >= 1024 and -(-N // 256) * -(-M // 64) >= 256 and K * (64 * 4 + 16) <= 40 * 1024


# N, C, K, M and the form that was at least 1.3 times as fast as the others there (us: gather, rows, matrix)
MEASURED = [(16384, 4, 16, 1024, "gather"),    # 23, 48, -
            (16384, 1, 16, 4096, "gather"),    # 67, 163, -
            (100352, 16, 16, 32, "gather"),    # 12, 23, 17
            (7237, 11, 16, 755, "gather"),     # 16, 46, -
            (33175, 452, 64, 107, "gather"),   # 355, 1207, -
            (4910, 6, 24, 1566, "gather"),     # 18, 50, -
            (256, 128, 16, 512, "gather"),
            (10238, 163, 24, 2368, "rows"),    # 1849, 519, -
            (34102, 33, 64, 3328, "rows"),     # 1788, 815, -
            (12408, 136, 64, 1280, "rows"),    # 1009, 387, -
            (3260, 96, 16, 1647, "matrix"),    # 164, 121, 61
            (18236, 567, 8, 384, "matrix"),    # 697, 481, 283
            (5204, 133, 16, 3200, "matrix"),   # 985, 309, 195
            (300000, 256, 16, 3, "gather"),    # 139, 379, 329
            (2000000, 1, 16, 1, "gather")]     # 6, 47, -


def test_measured_shapes(choose):
    got = choose([(N, C, K, M, rows_ok(N, K, M)) for N, C, K, M, _ in MEASURED])
    assert [g[0] for g in got] == [m[4] for m in MEASURED]


def test_the_least_of_the_forms_that_run(choose):
    shapes = [(N, C, K, M, ok) for N in (1, 64, 1000, 4096, 70000) for C in (1, 3, 15, 16, 100, 700) for K in (1, 8, 16, 17, 150, 256)
              for M in (1, 3, 4, 63, 256, 1000, 2048, 4096) for ok in (0, 1)]
    for (N, C, K, M, ok), (form, us) in zip(shapes, choose(shapes)):
        assert us[form] == min(us.values()) < 1e30
        assert ok or us["rows"] == 1e30
        assert (us["matrix"] < 1e30) == (K <= 16 and C >= 16)


def test_outputs_past_the_gathers_grid(choose):
    (form, us), = choose([(70000000, 1, 24, 132, 1)])
    assert form == "rows" and us["gather"] < us["rows"]

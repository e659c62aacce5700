"""The encoder's workgroup target: a value asked for is taken as it is, in small
and mid-size passes too; the default stands for the library's own choice."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include "encode_rule.hpp"
int main()
{
    unsigned asked, f64, B, m, nunits, small;
    unsigned long long tiles;
    while (std::scanf("%u %u %u %u %u %u %llu", &asked, &f64, &B, &m, &nunits, &small, &tiles) == 7)
        std::printf("%u\n", mdr::encode_target_wg(asked, f64 != 0, B, m, nunits, small != 0, tiles));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("rule")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run([gxx, "-std=c++17", "-I", os.path.join(ROOT, "paper_2505_00227_amd", "csrc"), str(d / "main.cpp"),
                    "-o", str(d / "main")], check=True)

    def call(rows):
        text = "\n".join(" ".join(str(int(v)) for v in r) for r in rows)
        got = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True)
        return [int(v) for v in got.stdout.split()]

    return call


# f64, planes, group, units, small, tiles: small passes of few and many units, mid-size passes
# at and past the last tile count of one round, a general one, and a large one
PASSES = [(0, 32, 4, 9, 1, 2048), (0, 32, 1, 33, 1, 2048), (1, 64, 4, 17, 1, 1024), (0, 32, 4, 9, 0, 4096),
          (0, 32, 4, 9, 0, 4097), (1, 64, 4, 17, 0, 12288), (1, 64, 4, 17, 0, 12289), (1, 40, 4, 11, 0, 300),
          (0, 32, 4, 9, 0, 1 << 20)]


def test_asked_for_is_taken(rule):
    asked = [64, 300, 768, 1024, 1152, 2303, 2305, 4608, 9216, 65536]
    rows = [(a, *p) for a in asked for p in PASSES]
    assert rule(rows) == [r[0] for r in rows]


def test_default(rule):
    assert rule([(2304, *p) for p in PASSES]) == [1024, 512, 512, 1024, 2304, 1024, 2304, 2304, 2304]

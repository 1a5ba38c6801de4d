"""The host layer's rules for shaping the edge path's launches (schedule.h),
compiled for the host and held against what their comments say."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++") or shutil.which("c++")
PLAIN, STAGED = 0, 2
CUS = 256

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "paper_2603_08661_amd/csrc/schedule.h"
using namespace igsp;
int main() {
  char what;
  int n, a, b, w, h;
  while (std::scanf(" %c %d %d %d", &what, &n, &a, &b) == 4) {
    std::vector<igsp_view> v;
    for (int i = 0; i < n && std::scanf("%d %d", &w, &h) == 2; ++i) v.push_back(igsp_view{w, h, 0, 0});
    if (what == 'm') std::printf("%d\n", marched_rows(v.data(), n, a, b, 256));
  }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if not CXX:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(DRIVER)
    subprocess.run([CXX, "-std=c++17", "-Wall", "-Werror", "-I", ROOT, str(d / "rules.cpp"), "-o", str(d / "rules")], check=True)

    def run(questions):
        text = "\n".join(f"{q} {len(v)} {a} {b} " + " ".join(f"{w} {h}" for w, h in v) for q, a, b, v in questions)
        return [int(x) for x in subprocess.run([str(d / "rules")], input=text, capture_output=True, text=True, check=True).stdout.split()]

    return run


def waves(views, seg):
    return sum(-(-w // 248) * -(-h // seg) for w, h in views)


def test_heights_are_marched_in_whole_rounds(ask):
    views = [(2000, 1500)]
    got = ask([("m", seg, STAGED, views) for seg in (8, 9, 10, 11, 12, 13, 64, 100, 4096)])
    assert got == [12, 12, 12, 12, 12, 18, 66, 102, 4098]


def test_single_rounds_where_a_launch_leaves_simds_idle(ask):
    """Ten rows become one round of six where a launch has at most 1.5 wavefronts
    per SIMD (6 per CU) at six rows, or 1 in a plain call of several views: a
    batched call's launch covers every view, a plain call's one of them."""
    one, line4, line6 = (1297, 840), (992, 1536), (1984, 1152)
    assert waves([one], 6) == 840 and waves([line4], 6) == 4 * CUS and waves([line6], 6) == 6 * CUS
    for views in ([one], [one] * 2, [one] * 12, [line4] * 3, [(992, 1537)] * 3, [line6], [line6] * 3, [(1984, 1153)],
                  [one, (1984, 1000)], [(64, 48)] * 300):
        total, n = waves(views, 6), len(views)
        assert ask([("m", 10, form, views) for form in (PLAIN, STAGED)]) == [
            6 if total // n <= (4 if n > 1 else 6) * CUS else 12, 6 if total <= 6 * CUS else 12], views
    assert ask([("m", 10, PLAIN, [one] * 2), ("m", 10, STAGED, [one] * 2)]) == [6, 12]

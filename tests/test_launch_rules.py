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
    if (what == 'c') std::printf("%d\n", median_chain(a, v.data(), n));
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


FP32, FP16, BF16 = 0, 1, 2
LONG, SHORT, GUARDED = 0, 1, 2


def view(chunks):
    return (248, 16 * chunks)          # one strip: 16 rows a chunk


def test_median_chain_counts_the_views_chunks(ask):
    """A 1297x840 view is 6 strips of 840 slots, 315 chunks of 16. The lines: the
    largest view's chunks, and all views' together."""
    got = ask([("c", FP32, 0, v) for v in (
        [(1297, 840)], [(1297, 840)] * 2, [(1297, 840)] * 3, [(1297, 840)] * 4, [(1297, 840)] * 8, [(1297, 840)] * 9,
        [view(360)], [view(361)], [view(700)], [view(701)], [view(700)] * 3, [view(700)] * 4, [(64, 48)] * 64, [(64, 48)] * 65)])
    assert got == [SHORT, SHORT, GUARDED, GUARDED, GUARDED, LONG, SHORT, GUARDED, GUARDED, LONG, GUARDED, LONG, SHORT, LONG]
    got = ask([("c", FP16, 0, v) for v in (
        [(1297, 840)] * 4, [(1297, 840)] * 5, [(1984, 1376)], [view(510)], [view(511)], [(300, 187)] * 100, [(300, 187)] * 103)])
    assert got == [SHORT, LONG, LONG, SHORT, LONG, SHORT, LONG]
    assert ask([("c", BF16, 0, [(64, 48)])]) == [LONG]


def test_median_chain_follows_its_figures(ask):
    """Each measured launch of the rule's comment lies on the side that its line
    was drawn for: FP32's short chain where stripes with noise are no slower than
    with the five launches, its guarded chain where they are not and photographs
    are faster than with the long one; FP16's short chain where it is faster."""
    fp32 = {(1, 315): SHORT, (1, 413): GUARDED, (1, 688): GUARDED, (1, 816): LONG, (3, 250): SHORT, (3, 315): GUARDED,
            (8, 315): GUARDED, (10, 315): LONG, (12, 90): SHORT, (24, 90): GUARDED, (40, 65): LONG,
            (64, 24): GUARDED}
    fp16 = {(1, 438): SHORT, (1, 504): SHORT, (1, 550): LONG, (1, 688): LONG, (4, 315): SHORT, (5, 315): LONG,
            (3, 404): SHORT, (4, 404): LONG, (20, 90): SHORT, (70, 24): SHORT, (95, 24): SHORT, (120, 24): LONG}
    for prec, want in ((FP32, fp32), (FP16, fp16)):
        assert ask([("c", prec, 0, [view(c)] * n) for n, c in want]) == list(want.values())

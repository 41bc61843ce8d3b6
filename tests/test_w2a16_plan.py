"""The weight-only kernel's rule from a shape to a workgroup form (csrc/w2a16_plan.hpp), walked on the host over the shapes
that the call accepts."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_15779_amd", "csrc")
CUS = 256
F16, F32 = 0, 1   # bf16 activations take the rule of f32: both are staged in binary32

SOURCE = r"""
#include "w2a16_plan.hpp"
#include <cstdio>
int main()
{
    int f32, N, K, lanes;
    while (scanf("%d %d %d %d", &f32, &N, &K, &lanes) == 4) {
        const rcp::WoPlan p = rcp::wo_plan(f32 != 0, N, K, 256, lanes);
        printf("%d %d %d %d %zu\n", p.ws, p.slots, p.unr, p.chains, rcp::wo_lds_bytes(f32 != 0, K, p.ws, p.slots, p.unr));
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    exe = str(d / "plan")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "plan.cpp"), "-o", exe], check=True)

    def walk(shapes):
        """[(f32, N, K, forced lanes)] -> [(wavefronts per row group, row groups per workgroup, loads a stage, running sums, LDS bytes)]"""
        text = "\n".join("%d %d %d %d" % s for s in shapes)
        lines = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        out = [tuple(int(v) for v in line.split()) for line in lines if line]
        assert len(out) == len(shapes)
        return out
    return walk


def busiest(n, slots):
    """Row groups of the compute unit that gets the most."""
    blocks = -(-(n // 4) // slots)
    return -(-blocks // CUS) * slots


def padded(k, ws):
    return -(-(k // 16) // (64 * ws)) * 64 * ws


ROWS = sorted({4 * g for base in range(256, 2049, 256) for g in (base - 1, base, base + 1, base + 3, base + 4, base + 100)} | {4, 32, 1000})


def test_a_long_token_leaves_the_busiest_unit_no_more_than_either_form_of_eight_wavefronts(plan):
    """Units that the busiest compute unit computes on, padding included: four row groups a workgroup on 1028 rows would leave
    most units without work and the others with four row groups."""
    shapes = [(f, n, k, 0) for f, lo in ((F32, 8224), (F16, 16416)) for n in ROWS if n <= 8192
              for k in list(range(lo, 32768, 352)) + [11008, 14336, 16384, 28672] if k >= lo]
    for (f, n, k, _), (ws, slots, _, _, _) in zip(shapes, plan(shapes)):
        eight = min(busiest(n, 2) * padded(k, 4), busiest(n, 4) * padded(k, 2))
        assert busiest(n, slots) * padded(k, ws) <= eight, (f, n, k, ws, slots)


def test_forms_of_four_wavefronts_are_resident_at_once_on_a_long_token(plan):
    shapes = [(f, n, k, 0) for f, lo in ((F32, 8224), (F16, 16416)) for n in ROWS if 1024 < n <= 8192 for k in range(lo, 32768, 352)]
    for (f, n, k, _), (ws, slots, _, _, lds) in zip(shapes, plan(shapes)):
        if ws * slots == 4:
            assert busiest(n, slots) // slots * lds <= 160 * 1024, (f, n, k, ws, slots)


@pytest.mark.parametrize("k", [4096, 4608, 6144, 8192])
def test_a_handful_of_second_row_groups_does_not_halve_the_workgroups(plan, k):
    for n, slots in ((1024, 1), (1028, 1), (1036, 1), (1040, 2), (1280, 2), (2048, 2), (2304, 1), (3072, 1), (4096, 2)):
        for f in (F16, F32):
            assert plan([(f, n, k, 0)])[0][:2] == (4, slots), (f, n, k)


def test_every_form_that_is_chosen_is_built_and_fits(plan):
    """Every accepted size has a kernel whose tables, token and exchange slots fit the LDS."""
    built = {(1, 4), (2, 2), (2, 4), (4, 1), (4, 2)}
    shapes = [(f, n, k, lanes) for f in (F16, F32) for n in ROWS + [5632, 6144, 6148, 8196, 12288, 65536, 131072]
              for k in list(range(32, 1056, 32)) + list(range(1056, 32769, 992)) + [32768] for lanes in (0, 16, 64, 128, 256)]
    for s, (ws, slots, unr, chains, lds) in zip(shapes, plan(shapes)):
        assert (ws, slots) in built and unr in (1, 2, 4) and lds <= 160 * 1024, s
        assert unr == 1 or (ws, slots) != (4, 2), s   # the one form that is built with one load a stage only
        assert chains == 1 or (chains, ws, slots, unr) == (2, 2, 4, 1), s
        if s[3] >= 64 and s[2] // 16 >= s[3]:
            assert ws * 64 == s[3] and ws * slots == 4, s


def test_a_row_of_few_is_summed_in_as_many_parts_as_by_four_wavefronts(plan):
    """256 partial sums a row up to four row groups a unit: half as many are twice as long, and their rounding errors larger."""
    shapes = [(f, n, k, 0) for f in (F16, F32) for n in ROWS if n <= 4096 for k in range(4096, 32769, 352)]
    for s, (ws, _, _, chains, _) in zip(shapes, plan(shapes)):
        assert ws * chains >= 4, s


@pytest.mark.parametrize("k", [2080, 2976, 4064])
def test_two_units_a_lane_are_one_stage_while_few_rows_fall_on_a_unit(plan, k):
    for f in (F16, F32):
        for n, unr in ((1028, 2), (2048, 2), (4096, 2), (8192, 1)):
            assert plan([(f, n, k, 0)])[0][:3] == (2, 2, unr), (f, n, k)

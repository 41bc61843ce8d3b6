"""The matrix-core attention's rule from the lengths of a call to the split length (csrc/kv4_plan.hpp), walked on the host."""
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_15779_amd", "csrc")
CUS = 256

SOURCE = r"""
#include "kv4_plan.hpp"
#include <cstdio>
int main()
{
    int n, heads, lengths[16];
    while (scanf("%d %d", &heads, &n) == 2) {
        for (int b = 0; b < n; ++b)
            if (scanf("%d", lengths + b) != 1) return 1;
        const int tokens = rcp::kv_split_tokens(lengths, n, heads, 256);
        printf("%d %lld\n", tokens, rcp::kv_workgroups(lengths, n, heads, tokens));
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    exe = str(d / "plan")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "plan.cpp"), "-o", exe], check=True)

    def walk(calls):
        """[(heads, lengths)] -> [(tokens of a split, workgroups)]"""
        text = "\n".join(" ".join(map(str, (heads, len(lengths)) + tuple(lengths))) for heads, lengths in calls)
        lines = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        out = [tuple(int(v) for v in line.split()) for line in lines if line]
        assert len(out) == len(calls)
        return out
    return walk


def splits(lengths, tokens):
    return sum(-(-v // tokens) for v in lengths)


def test_every_call_gets_whole_blocks_within_the_scratch(plan):
    """Splits of 256 to 1024 tokens, so that no head has more of them than its scratch has slots (one for every 64 tokens)."""
    rng = random.Random(1)
    calls = [(h, [s]) for h in (1, 4, 8, 32, 65535) for s in (1, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 4096, 70000, 262144)]
    calls += [(rng.choice([1, 4, 8, 10, 32]), [int(2 ** rng.uniform(0, 16)) for _ in range(rng.randint(2, 16))]) for _ in range(400)]
    for (heads, lengths), (tokens, groups) in zip(calls, plan(calls)):
        assert tokens % 256 == 0 and 256 <= tokens <= 1024
        assert groups == heads * splits(lengths, tokens)
        assert all(-(-v // tokens) <= -(-v // 64) for v in lengths)


def test_no_other_split_leaves_the_fullest_unit_less(plan):
    """Where two lengths put the same number of workgroups on the fullest compute unit the shorter one is taken."""
    rng = random.Random(2)
    calls = [(rng.choice([4, 8, 16, 32]), [rng.randint(300, 6000) for _ in range(rng.randint(1, 16))]) for _ in range(300)]
    fullest = lambda heads, lengths, tokens: -(-heads * splits(lengths, tokens) // CUS)
    for (heads, lengths), (tokens, _) in zip(calls, plan(calls)):
        for shorter in range(256, tokens, 256):
            if fullest(heads, lengths, shorter) > 1:
                assert fullest(heads, lengths, shorter) > fullest(heads, lengths, tokens) or heads * splits(lengths, tokens) <= CUS + CUS // 32

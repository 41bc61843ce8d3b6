"""The attention's rules from the lengths and heads of a call to the kernel's form and split length (csrc/kv4_plan.hpp), walked on the
host."""
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


FORMS = r"""
#include "kv4_plan.hpp"
#include <cstdio>
int main()
{
    int batched, H_q, H_kv, forced, n, lengths[16];
    const char* names[] = {"at_once", "stream", "matrix"};
    while (scanf("%d %d %d %d %d", &batched, &H_q, &H_kv, &forced, &n) == 5) {
        for (int b = 0; b < n; ++b)
            if (scanf("%d", lengths + b) != 1) return 1;
        const rcp::KvPlan plan = rcp::kv_plan(lengths, n, batched != 0, H_q, H_kv, 256, forced);
        printf("%s %d\n", names[static_cast<int>(plan.form)], plan.tokens);
    }
}
"""


def _compiled(d, source):
    (d / "plan.cpp").write_text(source)
    exe = str(d / "plan")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "plan.cpp"), "-o", exe], check=True)
    return lambda text: subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    run = _compiled(tmp_path_factory.mktemp("plan"), SOURCE)

    def walk(calls):
        """[(heads, lengths)] -> [(tokens of a split, workgroups)]"""
        lines = run("\n".join(" ".join(map(str, (heads, len(lengths)) + tuple(lengths))) for heads, lengths in calls))
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


def _microseconds(heads, lengths, blocks):
    """The model in hundredths: a workgroup's share of the fullest unit; whether the units over one workgroup each count."""
    tokens = 256 * blocks
    groups, end = heads * splits(lengths, tokens), (lengths[-1] - 1) % tokens + 1
    spare = 8 if blocks == 2 or (blocks == 3 and len(lengths) > 1 and end <= 256 and groups <= CUS + heads) else 0
    if groups <= CUS + spare:
        return 860 + 173 * blocks
    return 640 + -(-groups // CUS) * (205 + 122 * blocks)


def test_the_split_is_the_one_of_least_cost(plan):
    """The shortest of those of least cost, none longer than the longest sequence needs, at most four blocks."""
    rng = random.Random(5)
    calls = [(rng.choice([1, 2, 4, 8, 10, 16, 24, 32, 65]), [int(2 ** rng.uniform(4, 15)) for _ in range(rng.choice([1, 1, 2, 5, 16]))]) for _ in range(1500)]
    taken = set()
    for (heads, lengths), (tokens, _) in zip(calls, plan(calls)):
        blocks = range(1, min(4, -(-max(lengths) // 256)) + 1)
        assert tokens == 256 * min(blocks, key=lambda c: (_microseconds(heads, lengths, c), c)), (heads, lengths)
        taken.add(tokens)
    assert taken == {256, 512, 768, 1024}


@pytest.mark.parametrize("heads,lengths,want", [
    (8, [40000], 768), (8, [65536], 1024), (16, [12483], 512), (8, [131072], 1024), (8, [4096], 256),
    (32, [4096], 512), (1, [300], 256), (1, [256 * 256], 256), (1, [256 * 256 + 1], 512), (1, [264 * 512], 512), (1, [264 * 512 + 1], 768)])
def test_split_lengths_of_some_calls(plan, heads, lengths, want):
    assert plan([(heads, lengths)])[0][0] == want


@pytest.mark.parametrize("heads,lengths,want", [
    (66, [2951], 512), (65, [2447], 512), (10, [19286], 512), (4, [8837, 7645], 512),
    (33, [1188, 951, 814, 803], 768), (43, [1424, 940, 1333], 512), (4, [9997, 9939, 9300, 9583, 9873], 512),
    (2, [24780] * 4, 512), (10, [12847], 512)])
def test_a_few_units_with_a_second_workgroup(plan, heads, lengths, want):
    """Just over one workgroup a unit: whole second ones are not free."""
    assert any(CUS < heads * splits(lengths, t) <= CUS + CUS // 32 for t in (256, 512, 768, 1024))
    assert plan([(heads, lengths)])[0][0] == want


@pytest.fixture(scope="module")
def form(tmp_path_factory):
    run = _compiled(tmp_path_factory.mktemp("form"), FORMS)

    def walk(H_q, H_kv, lengths, batched=None, forced=0):
        """(form, tokens of a workgroup)"""
        batched = len(lengths) > 1 if batched is None else batched
        name, tokens = run(" ".join(map(str, [int(batched), H_q, H_kv, forced, len(lengths)] + list(lengths))))[0].split()
        return name, int(tokens)
    return walk


# (query heads, cache heads, lengths, form): the faster one on the card, both timed
@pytest.mark.parametrize("H_q,H_kv,lengths,want", [
    (64, 4, [468] * 2, "at_once"), (64, 4, [117] * 8, "matrix"), (64, 4, [703] * 2, "at_once"), (128, 8, [423] * 2, "at_once"),
    (96, 8, [353] * 3, "matrix"), (64, 2, [162] * 4, "matrix"), (16, 1, [1281, 1280, 1200, 1205], "at_once"),          # more than eight query heads
    (32, 4, [468] * 4, "at_once"), (64, 8, [324] * 2, "at_once"), (32, 4, [703] * 4, "matrix"), (32, 4, [168] * 5 + [70] * 11, "matrix"),
    (48, 8, [312] * 4, "matrix"),                                                                                     # five to eight
    (32, 8, [468] * 4, "at_once"), (32, 8, [104] * 16, "matrix"), (32, 8, [440] * 9, "matrix"),                       # three or four
    (32, 16, [648] * 2, "matrix"), (64, 32, [428] * 3, "matrix"),                                                     # two
    (32, 32, [117] * 16, "at_once"), (32, 32, [234] * 8, "matrix"), (32, 32, [168] * 4 + [68] * 12, "matrix"),
    (32, 32, [378, 300, 300, 300, 294], "at_once"), (64, 64, [68] * 13, "matrix"),                                    # one
    (32, 32, [160] * 8, "matrix"), (32, 8, [319] * 4, "at_once"), (32, 32, [159] * 8, "at_once"),                     # 40960 pairs
    (32, 4, [511] * 4, "at_once"), (32, 4, [512] * 4, "matrix")])                                                     # 65536 pairs
def test_a_batch_takes_the_form_that_is_faster_for_it(form, H_q, H_kv, lengths, want):
    assert form(H_q, H_kv, lengths)[0] == want


@pytest.mark.parametrize("H_q,H_kv,S,want", [
    (32, 32, 4095, "at_once"), (32, 4, 4095, "at_once"), (32, 4, 4096, "matrix"), (64, 4, 2047, "at_once"), (64, 4, 2048, "matrix"),
    (32, 8, 2047, "at_once"), (32, 8, 2048, "matrix"), (32, 16, 2047, "at_once"), (32, 16, 2048, "matrix"), (32, 32, 9000, "matrix"),
    (32, 32, 4096, "stream"), (32, 32, 4097, "matrix"), (32, 32, 6144, "matrix"), (32, 32, 7500, "stream"),
    (32, 32, 8192, "stream"), (32, 32, 8193, "matrix"), (8, 8, 30625, "stream"), (64, 64, 4096, "stream"), (32, 16, 7500, "matrix")])
def test_the_form_for_one_sequence(form, H_q, H_kv, S, want):
    name, tokens = form(H_q, H_kv, [S])
    assert name == want and (want == "matrix" or tokens == (512 if want == "stream" else 128 if S * H_q < 65536 else 256))


@pytest.mark.parametrize("H,lengths,want", [
    (16, [2048] * 4, "stream"), (8, [1024] * 16, "stream"), (16, [2048] * 3 + [2000], "matrix"),                  # one workgroup a unit
    (32, [293] * 16, "stream"), (32, [430] * 8 + [300] * 8, "stream"), (64, [196] * 16, "stream"), (64, [180] * 16, "matrix"),   # one split a sequence
    (32, [512] * 16, "stream"), (32, [513] + [505] * 15, "matrix"), (32, [600] + [300] * 15, "matrix"),
    (16, [782] * 16, "stream"), (32, [1024] * 8, "stream"), (32, [1024] * 7 + [512], "matrix"),                   # two
    (32, [1098] * 7, "stream"), (16, [1101] * 13, "stream"), (64, [1489, 1300, 1224], "matrix"), (32, [1098] * 8, "matrix"),   # three
    (32, [2048] * 4, "stream"), (8, [1797] * 16, "stream"), (32, [1563] * 4, "matrix"),                           # four
    (48, [887] * 10, "stream"), (32, [809] * 10 + [456] * 5, "stream"), (40, [827] * 10, "stream"), (48, [978] * 8, "matrix"),   # 1024 tokens
    (48, [1025] + [887] * 9, "matrix"), (40, [940] * 13, "stream"), (64, [640] * 16, "matrix"), (96, [400] * 11, "matrix"),
    (8, [4096] * 8, "matrix"), (16, [3438] * 4, "matrix"), (8, [18750], "matrix"), (32, [4000, 2120], "matrix")])
def test_one_query_head_streams_where_that_is_faster(form, H, lengths, want):
    tokens = 512 if H * sum(lengths) <= 262144 else 1024
    assert form(H, H, lengths) == (want, tokens if want == "stream" else form(H, H, lengths)[1])


def test_streaming_splits_leave_no_workgroup_without_tokens(form):
    rng = random.Random(3)
    seen = 0
    for _ in range(4000):
        H, n = rng.choice([4, 8, 16, 32, 40, 64]), rng.randint(1, 16)
        S = int(2 ** rng.uniform(17, 19.4) / H / n) + 1
        lengths = [S] + [max(1, int(S * (1 - rng.choice([0, 0.02, 0.3]) * rng.random()))) for _ in range(n - 1)]
        if rng.random() < 0.9 and len({-(-v // 512) for v in lengths}) > 1:
            continue
        name, tokens = form(H, H, lengths)
        if name == "stream":
            seen += 1
            pairs = H * sum(lengths)
            assert tokens == (512 if pairs <= 262144 else 1024) and 131072 <= pairs < 655360
            assert len({-(-v // tokens) for v in lengths}) == 1
        if seen == 60:
            return
    assert seen == 60

def test_the_option_asks_for_a_form(form):
    for tokens in (64, 128, 256, 512, 1024, 2048):
        for lengths in ([7], [9000], [100] * 16):
            assert form(32, 8, lengths, forced=tokens) == ("at_once" if tokens <= 256 else "matrix", tokens)

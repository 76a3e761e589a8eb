"""The key-split planner of attn_block and attn_f32 launches (CPU): split_plan.h compiled on
its own, against a heap simulation of the dispatch and against the floor of any plan."""
import heapq
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAX_SPLITS = 128
MAIN = r"""
#include "split_plan.h"
#include <cstdio>
#include <cstdlib>
// a plan a line: slots force ws_limit fixed merge merge_floats min_tiles n {tiles wgs floats}
int main() {
    a2t::SplitPlanner p;
    p.reserve(64, 256);
    int slots, force, n;
    long long limit, mf;
    a2t::SplitCosts c;
    while (std::scanf("%d %d %lld %d %d %lld %d %d", &slots, &force, &limit, &c.fixed, &c.merge, &mf, &c.min_tiles,
                      &n) == 8) {
        c.merge_floats = mf;
        a2t::SplitStream s[64];
        int out[64];
        for (int i = 0; i < n; ++i) {
            long long f;
            if (std::scanf("%d %d %lld", &s[i].tiles, &s[i].wgs, &f) != 3) return 1;
            s[i].floats = f;
        }
        for (int again = 0; again < 2; ++again) p.plan(n, s, c, slots, force, limit, out);   // the second from memory
        std::printf("%lld", (long long)p.makespan(n, s, out, c.fixed, slots));
        for (int i = 0; i < n; ++i) std::printf(" %d", out[i]);
        std::printf("\n");
    }
}
"""
BLOCK = dict(fixed=16, merge=6, merge_floats=1 << 20, min_tiles=4)
F32 = dict(fixed=5, merge=3, merge_floats=1 << 20, min_tiles=2)


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    tmp = tmp_path_factory.mktemp("split_plan")
    (tmp / "main.cpp").write_text(MAIN)
    exe = str(tmp / "main")
    subprocess.run([cxx, "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=address,undefined",
                    f"-I{os.path.join(ROOT, 'paper_2609_31224_amd', 'csrc')}", str(tmp / "main.cpp"), "-o", exe], check=True)

    def run(asked):
        """[(streams [(tiles, wgs, floats)], costs, slots, force, limit)] -> [(makespan, splits)]"""
        text = "\n".join(
            f"{slots} {force} {limit} {c['fixed']} {c['merge']} {c['merge_floats']} {c['min_tiles']} {len(s)} "
            + " ".join("%d %d %d" % x for x in s) for s, c, slots, force, limit in asked)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        return [(int(a.split()[0]), [int(x) for x in a.split()[1:]]) for a in out if a]
    return run


def _partials(splits, floats):
    return (splits * floats + 63) // 64 * 64 if splits > 1 else 0


def _dispatch(streams, splits, fixed, slots):
    """When the last workgroup ends: each goes to the CU that is free first."""
    cost = [-(-t // k) + fixed for (t, _, _), k in zip(streams, splits)]
    free = [0] * slots
    for i in sorted(range(len(streams)), key=lambda i: -cost[i]):
        for _ in range(splits[i] * streams[i][1]):
            heapq.heapreplace(free, free[0] + cost[i])
    return max(free)


def _launches():
    rng = random.Random(7)
    for _ in range(300):
        n = rng.choice([1, 2, 5, 21, 64])
        streams = [(rng.choice([1, 2, rng.randint(1, 40), rng.randint(1, 300)]), rng.choice([1, 4, 8, 24, 64]),
                    rng.randint(1, 200000)) for _ in range(n)]
        yield streams, rng.choice([BLOCK, F32]), rng.choice([1, 64, 256]), rng.choice([0, 0, 0, 1, 3, 500]), \
            rng.choice([0, 100000, 67108864])


def test_plans_hold(plan):
    """Every plan respects the workspace, the tiles and the most splits; what it says about its
    length is what the dispatch gives; and no single budget of tiles does better."""
    asked = list(_launches())
    for (streams, c, slots, force, limit), (span, splits) in zip(asked, plan(asked)):
        assert all(1 <= k <= min(t, MAX_SPLITS) for k, (t, _, _) in zip(splits, streams))
        partials = sum(_partials(k, f) for k, (_, _, f) in zip(splits, streams))
        assert partials <= limit or max(splits) == 1
        assert span == _dispatch(streams, splits, c["fixed"], slots) or sum(k * w for k, (_, w, _) in zip(splits, streams)) <= slots
        if force:
            want = [min(force, t, MAX_SPLITS) for t, _, _ in streams]
            assert splits == (want if sum(_partials(k, f) for k, (_, _, f) in zip(want, streams)) <= limit else [1] * len(streams))
            continue
        longest = max(t for t, _, _ in streams)
        mine = span + (c["merge"] + partials // c["merge_floats"] if max(splits) > 1 else 0)
        for budget in sorted({min(longest, b) for b in (c["min_tiles"], 5, 8, 13, 16, longest)}):
            other = [min(-(-t // budget), MAX_SPLITS) for t, _, _ in streams]
            ws = sum(_partials(k, f) for k, (_, _, f) in zip(other, streams))
            if ws <= limit and budget >= min(c["min_tiles"], longest):
                theirs = _dispatch(streams, other, c["fixed"], slots)
                theirs += c["merge"] + ws // c["merge_floats"] if max(other) > 1 else 0
                assert mine <= theirs, (streams, splits, other)


@pytest.mark.parametrize("costs,streams", [
    (F32, [(256, 8, 1040)] + [(2, 8, 1040)] * 40),                       # one long session among many short ones
    (F32, [(16 + i, 8, 1040) for i in range(63)] + [(129, 8, 1040)]),
    (BLOCK, [(130, 24, 137280)] + [(5, 24, 137280)] * 10),
    (BLOCK, [(131, 64, 540672)] + [(7, 24, 158400)] * 8),
])
def test_a_long_session_is_split_among_many(plan, costs, streams):
    """Launches that fill the CUs without splits still split the one session that would outlast
    all others: to within a half of the least that any plan of their tiles takes."""
    span, splits = plan([(streams, costs, 256, 0, 67108864)])[0]
    assert splits[max(range(len(streams)), key=lambda i: streams[i][0])] > 1
    work = sum(t * w for t, w, _ in streams) + costs["fixed"] * sum(w for _, w, _ in streams)
    assert span <= 1.5 * (work / 256 + costs["fixed"]), (span, work / 256)


def test_launches_just_past_one_round(plan):
    """264 workgroups of 64 tiles on 256 CUs: no second round of whole workgroups."""
    span, _ = plan([([(64, 8, 1040)] * 33, F32, 256, 0, 67108864)])[0]
    # unsplit, two rounds of 64 + 5 tiles: 138; in four splits, five rounds of 16 + 5
    assert span <= 5 * (16 + 5)

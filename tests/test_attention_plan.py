"""Host only: the attention launch's planner (csrc/attention_plan.h), compiled on its own and swept over block lengths,
compute-unit counts and request mixes, up to 16 parts a block and an exhausted split buffer.

Checked for every plan: each (request, KV head, block of rows) is covered exactly once, by one whole item or by consecutive
parts; a part has at least 6 tiles (every row of a block must see keys of each part) and a block at most 16; slots are numbered
without gaps, stay inside the buffer and belong to one block; items come heaviest first, or the heaviest alone and the others in
pairs; and what was built costs what was estimated, never more than leaving every block whole.
"""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <cstdio>
#include "attention_plan.h"
int main() {
    int n_cu, split, plain, group, heads, n;
    while (scanf("%d %d %d %d %d %d", &n_cu, &split, &plain, &group, &heads, &n) == 6) {
        std::vector<AttnRequest> reqs(n);
        for (auto& r : reqs) if (scanf("%d %d", &r.T, &r.P) != 2) return 1;
        AttnPlanSettings s{};
        s.n_cu = n_cu;
        s.split = split;
        s.plain_order = plain != 0;
        const AttnPlan p = plan_attention(s, reqs, group, heads);
        printf("plan %d %zu %zu %d %d\n", p.waves, p.items.size(), p.merges.size(), p.cost, attn_cost(attn_groups(attn_blocks(reqs, group, heads, p.waves == ATT_WAVES_SMALL && ((int)p.items.size() <= n_cu || !p.merges.empty()) ? ATT_WAVES_SMALL : ATT_WAVES)), AttnCut{}, n_cu));
        for (auto& i : p.items) printf("%d %d %d %d %d %d\n", i.req, i.kvh, i.qblock, i.kb0, i.nkb, i.slot);
        for (auto& m : p.merges) printf("%d %d %d %d %d\n", m.req, m.kvh, m.qblock, m.n_parts, m.slot0);
    }
}
"""


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "harness.cpp", d / "harness"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wall",
                    "-I", os.path.join(ROOT, "paper_2509_24381_amd", "csrc"), str(src), "-o", str(exe)], check=True)

    def run(cases, plain=0):
        text = "\n".join(" ".join(map(str, [n_cu, split, plain, g, h, len(reqs), *[v for r in reqs for v in r]]))
                         for n_cu, split, g, h, reqs in cases)
        env = dict(os.environ, LD_PRELOAD="", ASAN_OPTIONS="detect_leaks=0")
        out = iter(subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True, env=env).stdout.splitlines())
        plans = []
        for _ in cases:
            _, waves, n_items, n_merges, cost, whole = next(out).split()
            rows = lambda k: [tuple(map(int, next(out).split())) for _ in range(int(k))]
            plans.append((int(waves), rows(n_items), rows(n_merges), int(cost), int(whole)))
        return plans
    return run


def _list_schedule(costs, units):
    loads = [0] * units
    for c in sorted(costs, reverse=True):
        loads[loads.index(min(loads))] += c
    return max(loads)


def _check(case, plan):
    n_cu, split, g, heads, reqs = case
    waves, items, merges, estimate, whole_cost = plan
    rows = 32 * waves
    tiles = {}
    for r, (t, p) in enumerate(reqs):
        for qb in range(-(-t * g // rows)):
            last = min(t - 1, (qb * rows + rows - 1) // g)
            for c in range(heads):
                tiles[r, c, qb] = -(-(p + last + 1) // 64)
    parts = {}
    for r, c, qb, kb0, nkb, slot in items:
        parts.setdefault((r, c, qb), []).append((kb0, nkb, slot))
    assert set(parts) == set(tiles)
    n_slots, cut_blocks = 0, {m[:3]: m[3:] for m in merges}
    assert len(cut_blocks) == len(merges)
    for key, n in tiles.items():
        ps = sorted(parts[key])
        assert ps[0][0] == 0 and ps[-1][1] == n and all(a[1] == b[0] for a, b in zip(ps, ps[1:]))
        if len(ps) == 1:
            assert ps[0][2] == -1 and key not in cut_blocks
            continue
        n_parts, slot0 = cut_blocks[key]
        assert len(ps) == n_parts <= 16 and all(b - a >= 6 for a, b, _ in ps)
        assert [s for _, _, s in ps] == list(range(slot0, slot0 + n_parts))
        n_slots += n_parts
    assert n_slots <= 384 and sorted(s for *_, s in items if s >= 0) == list(range(n_slots))
    lens = [nkb - kb0 for *_, kb0, nkb, _ in items]
    if waves == 4 and len(items) > n_cu and not merges:   # item k and item k + n_cu share a compute unit: ranks lone + k and n - 1 - k
        n, paired = len(items), len(items) - n_cu
        ranks = sorted(lens, reverse=True)
        assert split <= 1
        if n > 2 * n_cu:                   # heaviest first, on two places per compute unit
            assert lens == ranks and lens[0] <= 64 and estimate == _list_schedule([n + 2 for n in lens], 2 * n_cu)
            return
        assert lens == ranks[n_cu - paired: n_cu] + ranks[:n_cu - paired] + ranks[n_cu:][::-1]
        ends = [16 * b + 11 * (a - b) for a, b in zip(lens, lens[n_cu:])] + [11 * a for a in lens[paired:n_cu]]
        assert -(-max(ends) // 16) + 2 == estimate <= whole_cost
        return
    assert lens == sorted(lens, reverse=True)
    if split == 1 or max(tiles.values()) < 16:
        assert split > 1 or not merges
    if split <= 1 and estimate == 0:   # (too short to cut and no more than a block per compute unit: nothing was weighed)
        assert not merges and len(items) <= n_cu and (split == 1 or (waves == 4 and lens[0] < 16))
    elif split <= 1:   # (tiles + 2 per whole item, + 4 per part, 4 and 1 per 36 parts for the merge)
        cost = _list_schedule([nkb - kb0 + (4 if s >= 0 else 2) for *_, kb0, nkb, s in items], n_cu)
        assert cost + (4 + n_slots // 36 if merges else 0) == estimate <= whole_cost


CASES = [
    # (compute units, RS_ATTN_SPLIT, query heads per KV head, KV heads, [(rows, cached)])
    (256, 0, 7, 4, [(2048, 6144)]), (256, 0, 7, 4, [(2048, 0)]), (256, 0, 4, 8, [(2048, 2000)]), (256, 0, 8, 8, [(4096, 28672)]),
    (256, 0, 7, 4, [(1, 32767)]), (256, 0, 1, 1, [(1, 0)]), (256, 0, 1, 8, [(1024, 512)]), (1, 0, 7, 1, [(300, 4000)]),
    (256, 0, 7, 4, [(64, 2048)]), (256, 1, 7, 4, [(64, 2048)]), (256, 3, 7, 4, [(64, 2048)]), (256, 16, 8, 8, [(4096, 28672)]),
    # more than 16 parts asked for: 15 to 17 shares a block, alone and beside short ones that hold the share down
    *[(256, 0, 8, 1, [(32, 64 * 16 * k - 33)] + [(31, 64 * 15)] * m) for k in (6, 7, 8, 12) for m in (0, 15, 60, 200)],
    *[(n, 0, 8, 2, [(32, t * 64)] * 2 + [(32, 0)] * 20) for n in (30, 36, 40, 64) for t in (95, 96, 97, 200)],
    (128, 0, 8, 2, [(32, 7488)] * 4 + [(1, 768)] * 20), (100, 0, 8, 2, [(32, 6464)] * 2 + [(1, 448)] * 20),
    (256, 0, 8, 1, [(32, 8064)] * 2 + [(1, 576)] * 20), (128, 0, 8, 1, [(32, 2944)] * 6 + [(32, 512)] * 20),
    # an exhausted split buffer: 200 blocks that want two or three parts each
    *[(256, 0, 8, 1, [(32, 64 * t)] * 200) for t in (15, 16, 30, 61)], (256, 16, 8, 1, [(32, 64 * 100)] * 60),
]


def test_listed_plans(planner):
    for case, plan in zip(CASES, planner(CASES)):
        _check(case, plan)


def test_swept_plans(planner):
    rng = random.Random(5)
    cases = []
    for _ in range(400):
        reqs = [(rng.choice([1, 7, 32, 100, 256, 700]), rng.randint(0, 6000) if rng.random() < 0.8 else 0)
                for _ in range(rng.choice([1, 1, 2, 5, 16, 48]))]
        cases.append((rng.choice([1, 3, 7, 40, 256, 300]), rng.choice([0, 0, 0, 0, 1, 2, 3, 16]), rng.choice([1, 4, 7, 8]),
                      rng.choice([1, 2, 4, 8]), reqs))
    for case, plan in zip(cases, planner(cases)):
        _check(case, plan)


def test_the_forms_are_reached(planner):
    """Whole blocks, equal parts, an even share with a rest, blocks of four wavefronts, and pairs of them occur where the rules
    put them; RS_ATTN_ORDER=plain gives the same blocks in another order."""
    whole, equal, share, small = planner([(256, 0, 8, 8, [(4096, 28672)]), (256, 0, 7, 4, [(250, 8192)]), (256, 0, 7, 4, [(1000, 12000)]),
                                          (256, 0, 2, 2, [(128, 384)])])
    cut_small, = planner([(256, 0, 7, 4, [(250, 2000)])])
    assert not whole[2] and whole[0] == 8
    assert equal[2] and len(equal[1]) <= 256
    lens = {m[:3]: sorted(i[4] - i[3] for i in share[1] if i[:3] == m[:3]) for m in share[2]}
    assert any(v[-1] - v[0] > 1 for v in lens.values()) and len(share[1]) > 256
    assert small[0] == 4 and len(small[1]) <= 256 and equal[0] == 8
    assert cut_small[0] == 4 and cut_small[2] and max(i[4] - i[3] for i in cut_small[1]) == 9
    for reqs, waves in (([(1200, 0)], 4), ([(4096, 0)], 4), ([(4096, 1)], 8), ([(2048, 8000)], 8), ([(200, 200)] * 16, 4)):
        plan, = planner([(256, 0, 8, 8, reqs)])
        assert plan[0] == waves and len(plan[1]) > 256
    for case in ((256, 0, 7, 4, [(2048, 0)]), (256, 0, 4, 8, [(2048, 2000)]), (7, 0, 2, 2, [(384, 0)]), (7, 0, 2, 2, [(384, 384)])):
        paired, plain = planner([case])[0], planner([case], plain=1)[0]
        assert paired[0] == plain[0] == 4 and case[0] < len(paired[1]) <= 2 * case[0]
        assert paired[1] != plain[1] and sorted(paired[1]) == sorted(plain[1])
        assert [i[4] for i in plain[1]] == sorted((i[4] for i in plain[1]), reverse=True)

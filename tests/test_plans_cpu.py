"""The host's launch plans, read on the CPU (tests/plan_probe.py): what they
launch, that every work item is launched once, and the sizes they ask for."""
import random
import subprocess

import pytest

import paper_2606_25041_amd as ws
from tests import plan_probe

MAX_GRID = ((1 << 32) - 1) // 512   # work-groups of 512 threads in one launch


def _dealt_items(p):
    """(group, item) of every work-group of a prefill in dealt order, as the
    kernel decodes its block id; None where it finds no item."""
    for j in range(p.launched // 8):
        pos = j // p.units
        for xcd in range(8):
            unit = xcd * p.units + j - pos * p.units
            idx = (pos << p.deal_log2) + (unit & ((1 << p.deal_log2) - 1))
            yield (unit >> p.deal_log2, idx) if idx < p.per_group else None


def test_prefill_order_launches_every_item_once():
    rng = random.Random(3)
    dealt = 0
    for _ in range(300):
        hkv, g = rng.choice((1, 1, 2, 3, 4, 5, 8)), rng.choice((1, 1, 2, 3, 5))
        batch, seq = rng.choice((1, 2, 3, 7, 33, 120)), rng.choice((1, 64, 200, 300, 700, 1300, 2500))
        p = plan_probe.prefill(batch, hkv * g, hkv, 64, seq)
        assert p.status == 0
        if p.units:
            dealt += 1
            got = [x for x in _dealt_items(p) if x is not None]
            assert len(got) == len(set(got)) == p.items == batch * hkv * p.per_group
        else:
            assert p.items <= p.launched < p.items + 8
    assert dealt > 50


@pytest.mark.parametrize("batch,hq,hkv,seq", [(501, 1, 1, 160), (1001, 1, 1, 17), (67, 3, 1, 240), (333, 1, 1, 400),
                                              (1 << 20 | 1, 1, 1, 1)])
def test_prefill_of_small_groups_launches_its_items_only(batch, hq, hkv, seq):
    """Many groups of few items, no multiple of 8 of them: dealt to classes,
    most of the launch (up to 7 of 8 work-groups) held no item, and the largest
    no longer fitted a grid."""
    p = plan_probe.prefill(batch, hq, hkv, 64, seq)
    assert p.status == 0 and p.launched <= MAX_GRID
    assert p.launched <= max(256, 1.05 * p.items + 8), p


@pytest.mark.parametrize("batch,hq,hkv,seq,block,groups", [
    (3, 12, 4, 1000, 1000, 1),    # 144 items of 16 tiles each: one round of 256-row items, two of 128-row ones
    (1, 24, 24, 2000, 2000, 1),
    (1, 32, 8, 2000, 1000, 1),
    (1, 8, 8, 1000, 1000, 2),     # both fit one round: the shorter items win
    (3, 12, 4, 1000, 40, 2),      # nearly causal: the longest items are few
    (1, 32, 8, 1100, 100, 2),
    (3, 8, 8, 3075, 190, 2),      # 75 items on 32 units a XCD
    (5, 16, 4, 956, 956, 1),
    (1, 40, 8, 3300, 200, 1),
    (1, 8, 8, 192, 192, 1),
    (1, 64, 8, 2686, 1343, 1),    # 2.75 rounds
])
def test_prefill_tile_follows_the_blocks(batch, hq, hkv, seq, block, groups):
    """The 128-row tile is chosen by the keys the rows really see: taken as
    causal, long blocks looked shorter than they are."""
    assert plan_probe.prefill(batch, hq, hkv, 128, seq, block).key_groups == groups


@pytest.mark.parametrize("batch,hq,hkv,new", [(24, 64, 8, 3), (32, 64, 8, 3), (32, 8, 8, 16)])
def test_one_round_of_unsplit_streams_keeps_the_common_plan(batch, hq, hkv, new):
    """Unsplit items that all fit one round gain nothing from another order,
    and the per-stream kernel is slower."""
    lens = [10 + 60 * (7 * i % batch) for i in range(batch)]
    p = plan_probe.step(batch, hq, hkv, 128, new, lens)
    assert p.status == 0 and not p.ragged and p.splits == [1] * batch
    # more than a round of them is still taken longest first
    assert plan_probe.step(batch, hq, hkv, 128, 300, lens).ragged


def test_plans_of_extreme_sizes_stay_in_range(tmp_path):
    """The host side under UBSan, over accepted sizes whose products pass 32
    bits (2^25 key tiles, 2^22 query tiles): no signed overflow."""
    main = tmp_path / "main.cpp"
    main.write_text(r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
extern "C" {
int probe_step(int, int, int, int, int, const int32_t *, const int32_t *, int, int *, int32_t *, int64_t *);
int probe_prefill(int, int, int, int, int, int, int *, int64_t *);
}
int main() {
    std::mt19937 rng(5);
    auto upto = [&](int64_t n) { return (int32_t)(1 + rng() % n); };
    int32_t ns[32];
    int64_t work[2];
    int ragged, out[4], done = 0;
    const int32_t two[2] = {2097152, 1000000};
    if (probe_step(2, 64, 8, 128, 524288, two, nullptr, 0, &ragged, ns, work)) return 1;
    for (int i = 0; i < 400; ++i) {
        const int hkv = 1 << rng() % 4, g = 1 << rng() % 7, b = 1 + rng() % (i % 4 ? 8 : 32);
        const int n = upto(1 << (1 + rng() % 23));
        int32_t lens[32], nl[32];
        for (int k = 0; k < b; ++k) lens[k] = upto(1 << (1 + rng() % 24)), nl[k] = upto(n);
        done += !probe_step(b, g * hkv, hkv, 128, n, lens, i & 1 ? nl : nullptr, i & 2, &ragged, ns, work);
        done += !probe_prefill(b, g * hkv, hkv, 128, n, 1 + n / upto(64), out, work);
    }
    printf("done %d\n", done);
    return done < 400;
}
""")
    exe = tmp_path / "plans"
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                    *plan_probe.SOURCES, str(main), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr


def test_gradient_workspace_is_host_arithmetic():
    """The size query asks no device: the same bytes with none, on a partition
    and on the whole chip, and room for the split sums of a short sequence."""
    for batch, hq, hkv, seq in ((1, 32, 8, 2400), (1, 8, 1, 520), (2, 32, 8, 16384), (1, 6, 2, 100)):
        got = {plan_probe.workspace_bytes(ws.WS_OP_PREFILL_BWD, batch, hq, hkv, seq, seq, cus) for cus in (0, 32, 256)}
        assert len(got) == 1, (batch, hq, hkv, seq, got)
        rows = -(-8 * batch * hq * seq // 256) * 256 + 4 * batch * seq
        assert got.pop() > rows if seq in (2400, 520) else True


@pytest.mark.parametrize("hq,hkv,d,new,lens,f32,ragged", [
    (16, 4, 64, 174, [916, 226], False, False),
    (32, 8, 128, 246, [2, 394], False, False),
    (12, 4, 128, 100, [50, 900], False, False),
    (12, 4, 128, 3, [1567, 2299, 1953, 2354], False, False),
    (8, 8, 64, 40, [139, 144, 4, 33, 10, 103, 69, 199], True, False),
    (64, 8, 128, 40, [134, 76, 560, 22], True, True),    # one tile, and 12 MB less of partials
    (64, 8, 128, 3, [32768, 9001, 2750, 517], False, True),
    (16, 4, 64, 37, [5003, 1200, 64, 2777, 333, 0], True, True),
    (24, 24, 128, 256, [63, 1332, 2019], False, True),
])
def test_per_stream_splits_have_to_win_their_cost(hq, hkv, d, new, lens, f32, ragged):
    """The per-stream kernel costs about a key tile more than the common one,
    which a modelled gain of one tile alone does not pay for."""
    assert plan_probe.step(len(lens), hq, hkv, d, new, lens, f32=f32).ragged == ragged

"""Whole-sequence calls over block layouts at the edges of the block search
(64 blocks per load, more levels past 64 and 4096 blocks, empty blocks, many
blocks inside one query tile): forward and gradients against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_25041_amd as ws
from paper_2606_25041_amd import inputs
from tests import gpu_support as gs

pytestmark = pytest.mark.gpu


def _layout(kind):
    g = np.random.default_rng(61)
    if kind == "units_300":            # one token per block: 256 blocks per tile
        return np.ones(300, int)
    if kind == "empties":              # 2000 blocks, most of them empty
        return (g.random(2000) < 0.15).astype(int) * g.integers(1, 4, size=2000)
    if kind == "blocks_64":
        return g.integers(1, 9, size=64)
    if kind == "blocks_65":
        return g.integers(1, 9, size=65)
    if kind == "past_4096":            # three levels
        return (np.arange(4200) % 7 == 3).astype(int)
    if kind == "leading_empty":
        return np.array([0] * 70 + [5] + [0] * 70 + [200] + [0] * 5)
    raise ValueError(kind)


@pytest.mark.parametrize("text", [False, True])
@pytest.mark.parametrize("kind", ["units_300", "empties", "blocks_64", "blocks_65", "past_4096", "leading_empty"])
def test_block_search(kind, text):
    lens = _layout(kind)
    L = int(lens.sum())
    gs.say(f"[gpu] block search {kind} text={text}: {len(lens)} blocks, {L} tokens")
    wl = inputs.prefill_workload(kind, 1, 2, 1, 64, [lens], seed=71)
    starts = None
    if text:
        starts = (wl.offsets[:, 1:] - np.random.default_rng(5).integers(0, lens + 1)).astype(np.int32)
    q, k, v = (gs.to_dev_bf16(t) for t in (wl.q, wl.k, wl.v))
    dout = inputs.bf16_normal(inputs.rng(71, 9), tuple(wl.q.shape))
    out, lse = ws.block_causal_prefill(q, k, v, wl.offsets, want_lse=True, text_starts=starts)
    grads = ws.block_causal_prefill_bwd(q, k, v, out, gs.to_dev_bf16(dout), lse, wl.offsets, text_starts=starts)
    bits = [inputs.bf16_bits(t) for t in (wl.q, wl.k, wl.v)]
    ref, rl = oracle.prefill(*bits, wl.offsets, wl.scale, text_starts=starts)
    assert np.abs(lse.double().cpu().numpy() - rl).max() <= 1e-3
    refs = (ref,) + tuple(oracle.prefill_bwd(*bits, inputs.bf16_bits(dout), wl.offsets, wl.scale, text_starts=starts))
    for name, x, r in zip(("out", "dq", "dk", "dv"), (out,) + tuple(grads), refs):
        err = np.abs(x.double().cpu().numpy() - r)
        assert err.max() <= gs.MAX_ABS and err.mean() <= gs.MEAN_ABS, (name, err.max(), err.mean())

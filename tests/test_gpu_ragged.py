"""Steps over streams of very different lengths, whose plan gives every stream
its own KV split count (checked of every case): every output against the
oracle, at the edges of the plan (one stream far longer than the rest, streams
with one split beside streams with many, no splits at all in more than one
round of items, empty caches, several query tiles, KV head counts that do and
do not divide the 8 XCDs, 2 and 32 streams), with segments, padded blocks,
both output types, lse and the fused append (pool bit for bit)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_25041_amd as ws
from paper_2606_25041_amd import inputs
from tests import gpu_support as gs
from tests import plan_probe

pytestmark = pytest.mark.gpu

CASES = [
    # Hq, Hkv, D, Lq, caches, new_lens, starts, f32
    (8, 8, 128, 3, [9000, 0, 70, 1], None, [0, 0, 0, 0], False),
    (16, 2, 128, 40, [9000, 17, 40, 0, 5], None, None, False),
    (6, 3, 64, 20, [12000, 64, 1000, 40, 200], [20, 1, 7, 20, 2], None, True),
    (12, 4, 128, 90, [4000, 300, 300, 8], [90, 33, 64, 1], [80, 33, 0, 0], False),
    (24, 24, 128, 30, [2500, 3], None, None, True),
    (4, 1, 64, 300, [7000, 129, 0], None, [290, 300, 0], False),
    (2, 2, 64, 1, [6000] + [5] * 31, None, None, False),
    (16, 8, 128, 2, [40000, 1], None, [0, 1], True),
    (24, 24, 64, 3, [900, 3, 500] + [40] * 13, None, None, False),   # unsplit
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_ragged_step(case):
    Hq, Hkv, D, Lq, caches, nls, starts, f32 = CASES[case]
    B = len(caches)
    wl = inputs.step_workload(f"ragged_{case}", B, Hq, Hkv, D, Lq, caches, seed=4000 + case, fuse_append=True)
    gs.say(f"[gpu] ragged step {case}: {Hq}/{Hkv}x{D} Lq={Lq} caches={caches}")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    plan = plan_probe.step(B, Hq, Hkv, D, Lq, caches, nls, f32, cus=cus)
    assert plan.ragged and (max(plan.splits) > 1 or plan.items > cus), plan
    cache = ws.PagedCache.allocate(wl.num_pages, Hkv, D, torch.from_numpy(wl.page_table), fill_bits=0x7FC1)
    for b in range(B):
        n = int(wl.cache_lens[b])
        if n:
            one = ws.PagedCache(cache.k_pool, cache.v_pool, torch.from_numpy(wl.page_table[b:b + 1]))
            ws.kv_append(one, [0], gs.to_dev_bf16(wl.k[b:b + 1, :n]), gs.to_dev_bf16(wl.v[b:b + 1, :n]))
    kn, vn = wl.k_new.clone(), wl.v_new.clone()
    real = nls or [Lq] * B
    for b in range(B):   # padding keys would poison the rows
        kn[b, real[b]:] = float("nan")
        vn[b, real[b]:] = float("nan")
    kw = dict(out_dtype=torch.float32 if f32 else torch.bfloat16, want_lse=True,
              text_starts=None if starts is None else np.asarray(starts, np.int32),
              new_lens=None if nls is None else np.asarray(nls, np.int32))
    args = (gs.to_dev_bf16(wl.q), gs.to_dev_bf16(kn), gs.to_dev_bf16(vn), cache, wl.cache_lens)
    out, lse = ws.block_causal_attn_fwd(*args, **kw)
    again, lse2 = ws.block_causal_attn_fwd(*args, fuse_append=True, **kw)
    torch.cuda.synchronize()
    for b in range(B):
        n, c = real[b], int(wl.cache_lens[b])
        sl = slice(b, b + 1)
        k = torch.cat([wl.k[sl, :c], wl.k_new[sl, :n]], 1)
        v = torch.cat([wl.v[sl, :c], wl.v_new[sl, :n]], 1)
        ref, rl = oracle.step(inputs.bf16_bits(wl.q[sl, :n]), inputs.bf16_bits(k[:, :c]), inputs.bf16_bits(v[:, :c]),
                              np.asarray([c], np.int32), inputs.bf16_bits(k[:, c:]), inputs.bf16_bits(v[:, c:]),
                              wl.scale, text_starts=None if starts is None else np.asarray([min(starts[b], n)]))
        err = np.abs(out[sl, :n].double().cpu().numpy() - ref)
        assert err.max() <= gs.MAX_ABS and err.mean() <= gs.MEAN_ABS, (b, err.max(), err.mean())
        assert np.abs(lse[sl, :, :n].double().cpu().numpy() - rl).max() <= 1e-3, b
        # a committed step gives the same bits, and commits the real tokens
        assert torch.equal(out[b, :n], again[b, :n]) and torch.equal(lse[b, :, :n], lse2[b, :, :n]), b
        pos = np.arange(c, c + n)
        page = torch.from_numpy(wl.page_table[b][pos // 64].astype(np.int64)).cuda()
        slot = torch.from_numpy(pos % 64).cuda()
        assert torch.equal(cache.k_pool[page, :, slot].view(torch.int16), args[1][b, :n].view(torch.int16)), b
        assert torch.equal(cache.v_pool[page, :, slot].view(torch.int16), args[2][b, :n].view(torch.int16)), b
    # nothing but the caches and the committed tokens was written
    used = int(wl.cache_lens.sum()) + sum(real)
    assert int((cache.k_pool.view(torch.int16)[:, 0, :, 0] != 0x7FC1).sum()) <= used

"""The merge of KV-split partials at the edges of its unrolled loops (split
counts around 4, 8, 12, 16 and 32), with a last 32-row block of one row, a GQA
ratio that is no power of two and an output view with gaps between its heads
and tokens: every output and lse against the oracle, the gaps untouched."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_25041_amd as ws
from paper_2606_25041_amd import inputs
from tests import gpu_support as gs

pytestmark = pytest.mark.gpu

B, HQ, HKV, LQ = 2, 6, 2, 11   # 33 packed rows per KV head


@pytest.mark.parametrize("splits", [2, 4, 5, 8, 9, 12, 13, 16, 17, 32])
@pytest.mark.parametrize("D,f32", [(128, False), (64, False), (128, True), (64, True)])
def test_merge(splits, D, f32):
    n = 128 * splits - LQ   # two 64-key tiles per split
    wl = inputs.step_workload("merge", B, HQ, HKV, D, LQ, [n] * B, seed=5000 + splits)
    gs.say(f"[gpu] merge of {splits} splits, D={D}, f32={f32}")
    assert ws.step_plan(B, HQ, HKV, LQ, wl.cache_lens, num_cus=256)[0] == splits
    cache = gs.device_cache(wl, wl.cache_lens, fill_on_gpu=True)
    dt = torch.float32 if f32 else torch.bfloat16
    whole = torch.full((B, LQ + 1, HQ + 2, D), 7.0, dtype=dt, device=gs.dev())
    out = whole[:, :LQ, 1:HQ + 1]
    q, kn, vn = (gs.to_dev_bf16(t) for t in (wl.q, wl.k_new, wl.v_new))
    _, lse = ws.block_causal_attn_fwd(q, kn, vn, cache, wl.cache_lens, out=out, want_lse=True)
    torch.cuda.synchronize()
    ref, rl = oracle.step(inputs.bf16_bits(wl.q), inputs.bf16_bits(wl.k[:, :n]), inputs.bf16_bits(wl.v[:, :n]),
                          wl.cache_lens, inputs.bf16_bits(wl.k_new), inputs.bf16_bits(wl.v_new), wl.scale)
    err = np.abs(out.double().cpu().numpy() - ref)
    assert err.max() <= gs.MAX_ABS and err.mean() <= gs.MEAN_ABS, (err.max(), err.mean())
    assert np.abs(lse.double().cpu().numpy() - rl).max() <= gs.LSE_ABS
    out.fill_(7.0)
    assert bool((whole == 7.0).all())


@pytest.mark.parametrize("padded", [False, True])
@pytest.mark.parametrize("D,hkv", [(128, 4), (64, 8)])
def test_merge_of_many_blocks(D, hkv, padded):
    """More 32-row blocks than the merge's small work-groups are launched for
    (one per compute unit: D / 32 of them per block), the last block ragged."""
    B, G, Lq = (2, 3, 91) if padded else (1, 3, 175)
    n = 3000
    wl = inputs.step_workload("merge_many", B, G * hkv, hkv, D, Lq, [n] * B, seed=5100 + D)
    blocks = B * hkv * -(-G * Lq // 32)
    assert blocks * (D // 32) > torch.cuda.get_device_properties(0).multi_processor_count
    nl = [Lq, 40] if padded else None
    splits = ws.step_plan(B, G * hkv, hkv, Lq, wl.cache_lens, new_lens=nl)[0]
    gs.say(f"[gpu] merge of {splits} splits, {blocks} blocks, D={D}, padded={padded}")
    assert splits > 4
    cache = gs.device_cache(wl, wl.cache_lens, fill_on_gpu=True)
    q, kn, vn = (gs.to_dev_bf16(t) for t in (wl.q, wl.k_new, wl.v_new))
    out, lse = ws.block_causal_attn_fwd(q, kn, vn, cache, wl.cache_lens, want_lse=True, new_lens=nl)
    torch.cuda.synchronize()
    for b in range(B):
        sl, m = slice(b, b + 1), nl[b] if nl else Lq
        ref, rl = oracle.step(*(inputs.bf16_bits(t[sl, :k]) for t, k in ((wl.q, m), (wl.k, n), (wl.v, n))),
                              wl.cache_lens[sl], inputs.bf16_bits(wl.k_new[sl, :m]), inputs.bf16_bits(wl.v_new[sl, :m]),
                              wl.scale)
        err = np.abs(out[sl, :m].double().cpu().numpy() - ref)
        assert err.max() <= gs.MAX_ABS and err.mean() <= gs.MEAN_ABS, (b, err.max(), err.mean())
        assert np.abs(lse[sl, :, :m].double().cpu().numpy() - rl).max() <= gs.LSE_ABS

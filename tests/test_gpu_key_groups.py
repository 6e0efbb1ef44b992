"""Whole-sequence attention on sequences short enough for the plan that gives
a work-group 128 rows and its two halves the even and the odd key tiles: an
odd and an even number of tiles, more tiles than the ring holds, a half that
sees no key of some rows (token-causal segments), ragged last rows; and, up to
192 tokens, where the plan keeps 256 rows, the short ends of that tile.  Which
one a case runs is checked.  Contiguous and paged, both outputs, lse; every
value against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_25041_amd as ws
from paper_2606_25041_amd import inputs
from tests import gpu_support as gs
from tests import plan_probe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("L", [1, 64, 65, 128, 129, 192, 193, 256, 257, 320, 449, 1000])
def test_key_groups(L, D, paged):
    g = np.random.default_rng([L, D])
    cuts = np.sort(g.integers(0, L + 1, size=4))
    lens = np.diff(np.concatenate([[0], cuts, [L]]))
    f32 = bool((L + D // 64 + paged) % 2)
    gs.say(f"[gpu] key groups L={L} D={D} paged={paged} f32={f32} blocks={lens.tolist()}")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for block in (1, L):   # every layout's key ends lie between these two's
        assert plan_probe.prefill(1, 3, 1, D, L, block, cus=cus).key_groups == (2 if L > 192 else 1)
    wl = inputs.prefill_workload("key_groups", 1, 3, 1, D, [lens], seed=5000 + L, paged=paged)
    text = (wl.offsets[:, 1:] - g.integers(0, lens + 1)).astype(np.int32) if L % 2 else None
    q, k, v = (gs.to_dev_bf16(t) for t in (wl.q, wl.k, wl.v))
    cache = None
    if paged:
        cache = ws.PagedCache.allocate(wl.num_pages, 1, D, torch.from_numpy(wl.page_table), fill_bits=0x7FC1)
        ws.kv_append(cache, [0], k, v)
        k = v = None
    out, lse = ws.block_causal_prefill(q, k, v, wl.offsets, cache=cache, want_lse=True, text_starts=text,
                                       out_dtype=torch.float32 if f32 else torch.bfloat16)
    again = ws.block_causal_prefill(q, k, v, wl.offsets, cache=cache, text_starts=text,
                                    out_dtype=torch.float32 if f32 else torch.bfloat16)
    assert torch.equal(out, again)
    ref, rl = oracle.prefill(*(inputs.bf16_bits(t) for t in (wl.q, wl.k, wl.v)), wl.offsets, wl.scale, text_starts=text)
    err = np.abs(out.double().cpu().numpy() - ref)
    assert err.max() <= gs.MAX_ABS and err.mean() <= gs.MEAN_ABS, (err.max(), err.mean())
    assert np.abs(lse.double().cpu().numpy() - rl).max() <= 1e-3

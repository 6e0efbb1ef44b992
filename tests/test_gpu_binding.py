"""The native marshalling against the Python (ctypes) marshalling: the same
calls give bitwise the same results through either, whatever form the
arguments take, and what one refuses the other refuses with the same error."""
import ctypes
import subprocess
import threading
import time

import numpy as np
import pytest
import torch

import paper_2606_25041_amd as ws

pytestmark = pytest.mark.gpu


class _Declines:
    """Takes no call, so every call goes through the Python code."""

    @staticmethod
    def _none(*_):
        return None

    append = step = prefill = prefill_bwd = _none


class _Watched:
    """The native marshalling, and whether it took the calls made through it."""

    def __init__(self, native):
        self.taken = []
        for name in ("append", "step", "prefill", "prefill_bwd"):
            setattr(self, name, self._watch(getattr(native, name)))

    def _watch(self, f):
        def call(*args):
            got = f(*args)
            self.taken.append(got is not None)
            return got
        return call


@pytest.fixture
def both(monkeypatch):
    """Calls f through the native and through the Python marshalling, and
    compares.  taken: whether the native one is to take the call (or decline it
    before anything is enqueued); None: it is not asked."""
    ws.library()

    def call(f, taken):
        def once():
            try:
                r = f()
            except Exception as e:   # compared below
                return type(e), str(e)
            torch.cuda.synchronize()
            return r
        watched = _Watched(ws._NATIVE)
        monkeypatch.setattr(ws, "_NATIVE", watched)
        native = once()
        assert watched.taken == ([] if taken is None else [taken]), (watched.taken, taken)
        monkeypatch.setattr(ws, "_NATIVE", _Declines())
        python = once()
        monkeypatch.undo()
        flat = lambda r: [r] if isinstance(r, torch.Tensor) else list(r) if isinstance(r, (tuple, list)) else [r]
        a, b = flat(native), flat(python)
        assert len(a) == len(b)
        for x, y in zip(a, b):
            assert torch.equal(x, y) and x.dtype == y.dtype if isinstance(x, torch.Tensor) else x == y, (native, python)
        return native
    return call


def _randn(*shape, seed=0):
    g = torch.Generator("cuda").manual_seed(seed + sum(shape))
    return torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)


def _cache(B, pages, Hkv, D):
    return ws.PagedCache(_randn(B * pages, Hkv, 64, D, seed=1), _randn(B * pages, Hkv, 64, D, seed=2),
                         torch.arange(B * pages, dtype=torch.int32).reshape(B, pages))


def _pair(x):
    h = torch.as_tensor(x, dtype=torch.int32)
    return h, h.cuda()


B, L, HQ, HKV, D = 2, 20, 4, 2, 64

STEP_FORMS = {
    "plain": dict(), "lens_list": dict(cache_lens=[70, 5]), "lens_numpy": dict(cache_lens=np.array([70, 5])),
    "f32_lse": dict(out_dtype=torch.float32, want_lse=True), "scale": dict(scale=0.2), "scale_int": dict(scale=1),
    "scale_numpy": dict(scale=np.float64(0.3)), "fuse": dict(fuse_append=True), "fuse_int": dict(fuse_append=1),
    "text": dict(text_starts=_pair), "text_list": dict(text_starts=[3, 20]), "new_lens": dict(new_lens=_pair),
    "new_lens_column": dict(new_lens="column"), "out": dict(out="out"), "strided": dict(q="view"),
    "parameter": dict(q="parameter"), "workspace": dict(workspace="big"), "lse_given": dict(lse="lse"),
    # refused
    "q_f16": dict(q="f16"), "k_shape": dict(k="short"), "lens_shape": dict(cache_lens="long"),
    "lens_int64": dict(cache_lens="int64"), "capacity": dict(cache_lens=[70, 125], fuse_append=True),
    "scale_zero": dict(scale=0.0), "text_range": dict(text_starts=[0, 21]), "workspace_small": dict(workspace="small"),
    "table_rows": dict(cache="one"), "out_shape": dict(out="short"), "q_cpu": dict(out="cpu"),
}
STEP_TAKEN = {"plain", "f32_lse", "scale", "fuse", "text", "new_lens", "new_lens_column", "out", "strided", "workspace",
              "lse_given", "scale_zero", "workspace_small"}


@pytest.mark.parametrize("form", sorted(STEP_FORMS))
def test_step_forms(both, form):
    q, k, v = _randn(B, L, HQ, D), _randn(B, L, HKV, D, seed=3), _randn(B, L, HKV, D, seed=4)
    cache = _cache(B, 2, HKV, D)
    kw = dict(STEP_FORMS[form])
    lens = kw.pop("cache_lens", _pair([70, 5]))
    lens = {"long": _pair([70, 5, 1]), "int64": tuple(t.long() for t in _pair([70, 5]))}.get(lens, lens) \
        if isinstance(lens, str) else lens
    how = kw.pop("q", None)
    if how == "view":
        q = torch.cat([q, k, v], 2)[:, :, :HQ]
    elif how == "parameter":
        q = torch.nn.Parameter(q, requires_grad=False)
    elif how == "f16":
        q = q.half()
    if kw.pop("k", None):
        k = k[:, :L - 1]
    if kw.pop("cache", None):
        cache = ws.PagedCache(cache.k_pool, cache.v_pool, cache.page_table_host[:1])
    if kw.get("text_starts") is _pair:
        kw["text_starts"] = _pair([3, 20])
    if kw.get("new_lens") is _pair:
        kw["new_lens"] = _pair([20, 7])
    if kw.get("new_lens") == "column":
        kw["new_lens"] = tuple(t[:, None] for t in _pair([20, 20]))
    sizes = dict(big=1 << 20, small=16)
    if "workspace" in kw:
        kw["workspace"] = torch.empty(sizes[kw["workspace"]], dtype=torch.uint8, device="cuda")
    if "lse" in kw:
        kw.update(lse=torch.empty(B, HQ, L, device="cuda"), want_lse=True)
    if "out" in kw:
        kw["out"] = {"out": torch.empty(B, L, HQ, 2 * D, dtype=torch.bfloat16, device="cuda")[..., :D],
                     "short": torch.empty(B, L - 1, HQ, D, dtype=torch.bfloat16, device="cuda"),
                     "cpu": torch.empty(B, L, HQ, D, dtype=torch.bfloat16)}[kw["out"]]
    real = [7 if form == "new_lens" and b else L for b in range(B)]

    def f():
        r = ws.block_causal_attn_fwd(q, k, v, cache, lens, **kw)
        rows = r if isinstance(r, tuple) else (r,)
        return [rows[0][b, :real[b]].clone() for b in range(B)] + [x.clone() for x in rows[1:]] + \
            [cache.k_pool.clone(), cache.v_pool.clone()]
    both(f, form in STEP_TAKEN)


@pytest.mark.parametrize("form", ["plain", "lse", "lens_list", "out_none", "out_shape"])
def test_noalloc_forms(both, form):
    q, k, v = _randn(B, L, HQ, D), _randn(B, L, HKV, D, seed=3), _randn(B, L, HKV, D, seed=4)
    cache, lens = _cache(B, 2, HKV, D), _pair([70, 5])
    out = None if form == "out_none" else torch.empty(B, L - (form == "out_shape"), HQ, D, dtype=torch.bfloat16, device="cuda")
    lse = torch.empty(B, HQ, L, device="cuda") if form == "lse" else None

    def f():
        r = ws.block_causal_attn_fwd_noalloc(q, k, v, cache, [70, 5] if form == "lens_list" else lens, out, lse=lse)
        return [r.clone()] + ([lse.clone()] if lse is not None else [])
    both(f, None if form == "out_none" else form in ("plain", "lse"))


@pytest.mark.parametrize("form", ["plain", "list", "new_lens", "new_lens_list", "strided", "shape", "capacity", "table"])
def test_append_forms(both, form):
    k, v = _randn(B, L, HKV, D, seed=3), _randn(B, L, HKV, D, seed=4)
    if form == "strided":
        k, v = torch.cat([k, v], 2).split(HKV, 2)
    lens = {"list": [70, 5], "capacity": _pair([70, 125])}.get(form, _pair([70, 5]))
    nl = {"new_lens": _pair([0, 9]), "new_lens_list": [20, 9]}.get(form)

    def f():
        cache = _cache(B, 2, HKV, D)
        if form == "table":
            cache.page_table_host = cache.page_table_host[:1]
        ws.kv_append(cache, lens, k[:, :, :1] if form == "shape" else k, v, new_lens=nl)
        return [cache.k_pool, cache.v_pool]
    both(f, form in ("plain", "new_lens", "strided", "capacity"))


@pytest.mark.parametrize("form", ["plain", "list", "paged", "paged_heads", "text", "f32_lse", "cache_too", "empty",
                                  "offsets", "v_none", "heads_wrong"])
def test_prefill_and_gradient_forms(both, form):
    n = 0 if form == "empty" else 50
    q, k, v = _randn(B, n, HQ, D), _randn(B, n, HKV, D, seed=3), _randn(B, n, HKV, D, seed=4)
    off = [[0, n // 3, n], [0, n, n]]
    offsets = off if form == "list" else _pair([[0, 3, 5]] * 2) if form == "offsets" else _pair(off)
    text = _pair([[n // 4, n], [5, n]]) if form == "text" else None
    cache = _cache(B, 1, HKV, D) if form in ("paged", "paged_heads", "cache_too", "heads_wrong") else None
    kk, vv = (None, None) if form in ("paged", "paged_heads", "heads_wrong") else (k, None if form == "v_none" else v)
    heads = {"paged_heads": HKV, "heads_wrong": 1}.get(form)
    kw = dict(cache=cache, num_kv_heads=heads, text_starts=text,
              out_dtype=torch.float32 if form == "f32_lse" else torch.bfloat16)
    both(lambda: ws.block_causal_prefill(q, kk, vv, offsets, want_lse=form == "f32_lse", **kw), form not in ("list", "v_none"))
    if form in ("plain", "list", "text", "offsets", "empty"):
        out, lse = ws.block_causal_prefill(q, k, v, _pair(off), want_lse=True, text_starts=text)
        taken = form not in ("list", "empty")
        both(lambda: ws.block_causal_prefill_bwd(q, k, v, out, q, lse, offsets, text_starts=text), taken)
        both(lambda: ws.block_causal_prefill_bwd(q, k, v[:, :, :1], out, q, lse, offsets), False)
        small = torch.empty(16, dtype=torch.uint8, device="cuda")
        both(lambda: ws.block_causal_prefill_bwd(q, k, v, out, q, lse, offsets, workspace=small), taken)


def test_empty_arrays_are_not_taken_for_absent_ones(both):
    """No block (or no stream) and an array of none of their starts (or
    lengths): refused, as a NULL pointer, by the text and varlen entry points."""
    q, k, v = _randn(B, 0, HQ, D), _randn(B, 0, HKV, D), _randn(B, 0, HKV, D)
    off, none = _pair(np.zeros((B, 1))), _pair(np.zeros((B, 0)))
    for got in (both(lambda: ws.block_causal_prefill(q, k, v, off, text_starts=none), False),
                both(lambda: ws.kv_append(_cache(B, 2, HKV, D), _pair([]), k[:0], v[:0], new_lens=_pair([])), False)):
        assert isinstance(got, tuple) and got[0] is ws.WsError and "NULL" in got[1], got


def test_a_cache_with_its_own_descriptor(both):
    """A subclass that overrides desc() (here: keys and values read from other
    pools than its attributes') is asked for it."""
    class Other(ws.PagedCache):
        def desc(self):
            d = super().desc()
            d.k_pool, d.v_pool = self.v_pool.data_ptr(), self.k_pool.data_ptr()
            return d
    q, k, v = _randn(B, L, HQ, D), _randn(B, L, HKV, D, seed=3), _randn(B, L, HKV, D, seed=4)
    plain, lens = _cache(B, 2, HKV, D), _pair([70, 5])
    other = Other(plain.k_pool, plain.v_pool, plain.page_table_host)
    got = both(lambda: ws.block_causal_attn_fwd(q, k, v, other, lens), False)
    swapped = ws.PagedCache(plain.v_pool, plain.k_pool, plain.page_table_host)
    assert torch.equal(got, ws.block_causal_attn_fwd(q, k, v, swapped, lens))


def test_calls_run_without_the_gil(tmp_path):
    """While a call is inside the library, other Python threads run (a launch
    may block on a full hardware queue).  The library's functions are replaced
    by one that sleeps 0.3 s, through the native marshalling of every entry
    point; a thread beside it that sleeps 1 ms at a time has to get on."""
    src, so = tmp_path / "slow.c", tmp_path / "slow.so"
    src.write_text("#include <unistd.h>\nint slow(void) { usleep(300000); return 0; }\n"
                   "unsigned long size(void) { return 256; }\n")
    subprocess.run(["gcc", "-O1", "-fPIC", "-shared", str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    slow, size = (ctypes.cast(f, ctypes.c_void_p).value for f in (lib.slow, lib.size))
    native = ws._native()
    q, k, v = _randn(B, L, HQ, D), _randn(B, L, HKV, D, seed=3), _randn(B, L, HKV, D, seed=4)
    cache, lens, off = _cache(B, 2, HKV, D), _pair([70, 5]), _pair([[0, L]] * B)
    out, lse = torch.empty_like(q), torch.empty(B, HQ, L, device="cuda")
    calls = {
        "append": lambda: ws.kv_append(cache, lens, k, v),
        "step": lambda: ws.block_causal_attn_fwd(q, k, v, cache, lens),
        "noalloc": lambda: ws.block_causal_attn_fwd_noalloc(q, k, v, cache, lens, out),
        "prefill": lambda: ws.block_causal_prefill(q, k, v, off),
        "prefill_bwd": lambda: ws.block_causal_prefill_bwd(q, k, v, out, q, lse, off),
    }
    turns, stop = [0], threading.Event()

    def beside():
        while not stop.is_set():
            time.sleep(0.001)
            turns[0] += 1
    thread = threading.Thread(target=beside)
    thread.start()
    try:
        native.bind(ws.PagedCache, *[slow] * 9, size, size)
        for name, call in calls.items():
            before, start = turns[0], time.perf_counter()
            call()
            assert time.perf_counter() - start > 0.25, (name, "did not reach the library natively")
            assert turns[0] - before > 30, (name, turns[0] - before)
    finally:
        stop.set()
        thread.join()
        ws._bind_native(ws.library())
    got = ws.block_causal_attn_fwd(q, k, v, cache, lens)   # the library is back
    assert torch.isfinite(got.float()).all()

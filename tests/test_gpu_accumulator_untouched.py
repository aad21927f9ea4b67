"""Calls that only read the |q| accumulator leave it alone, whatever it holds, and nothing but the token counts and the five
buffers' defined contents decides what a call does: a handle that was never reset, and a snapshot whose qacc buffer was
copied while a call was running, give the same results."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
KW = dict(B=3, Hq=14, Hkv=2, D=128, T_max=2048, Gk=128, Gv=128, R=128, k4=16, k16=0)


@pytest.fixture(scope="module")
def H():
    assert torch.cuda.is_available(), "these tests need the GPU"
    import gpu_common
    return gpu_common


def _tensors(rng, n):
    draw = lambda *s: rng.standard_normal(s).astype(np.float16)
    return draw(3, 2, n, 128), draw(3, 2, n, 128), draw(3, 14, 128)


@pytest.mark.parametrize("ragged", [0, 1])
def test_read_only_calls_ignore_and_keep_the_accumulator(H, ragged):
    """Several workgroups per pair (the merge), every bit of the sums and counts set to something else meanwhile."""
    rng = np.random.default_rng(7800 + ragged)
    oc, gc = H.make_pair(**KW)
    n = 128 * 9 + 50
    K, V, q = _tensors(rng, n)
    gc.quantize_append(H.dev(K), H.dev(V))
    oc.append(K, V)
    if ragged:
        gc.quantize_append_seq(1, H.dev(K[1, :, :5]), H.dev(V[1, :, :5]))
    acc, cnt = gc.query_accumulator()
    sel_before = gc.select_channels(None, H.dev(K)).clone()
    acc.fill_(3)      # (every channel alike: the ranges alone decide)
    sel_before = gc.select_channels(None, H.dev(K)).clone()
    cnt.fill_((0x7B5A << 48) + 12345)
    want = (acc.clone(), cnt.clone())
    for i in range(2):
        out, lse = torch.full((3, 14, 128), 9.0, dtype=torch.float16, device="cuda"), torch.full((3, 14), 9.0, device="cuda")
        gc.decode_attention(H.dev(q), out=out, lse=lse)
        sel = torch.full((3, 2, 16), 77, dtype=torch.uint8, device="cuda")
        gc.select_channels(None, H.dev(K), sel=sel)
        torch.cuda.synchronize()
        assert torch.equal(acc, want[0]) and torch.equal(cnt, want[1])
        assert torch.equal(sel, sel_before)
        ro, rl = oc.decode_attention(q)
        for b in (0, 2):
            assert np.all(np.abs(out[b].float().cpu().numpy() - ro[b]) <= H.ATOL + H.RTOL * np.abs(ro[b]))
            assert np.all(np.abs(lse[b].cpu().numpy() - rl[b]) <= H.LSE_ATOL + 1e-4 * np.abs(rl[b]))


def test_a_handle_that_was_never_reset(H):
    """Only the accumulator needs the reset: attention over a cache that never uses it merges without one."""
    import paper_2512_19206_amd as M
    rng = np.random.default_rng(7810)
    oc, gc = H.make_pair(**KW)
    lib = gc.lib
    lib.mixkvq_cache_destroy(gc.handle)
    gc.qacc.fill_(0xFF)
    bufs = M.binding.Buffers(*(t.data_ptr() for t in (gc.blocks, gc.res_k, gc.res_v, gc.qacc, gc.workspace)))
    h = C.c_void_p()
    assert lib.mixkvq_cache_create(C.byref(gc.cfg), C.byref(bufs), C.byref(h)) == 0
    gc.handle = h
    n = 128 * 9 + 50
    K, V, q = _tensors(rng, n)
    sel = np.tile(np.arange(16, dtype=np.uint8) * 7, (3, 2, 1))
    gc.quantize_append(H.dev(K), H.dev(V), sel=H.dev(sel))
    oc.append(K, V, sel)
    for _ in range(2):
        H.check_attention(oc, gc, q)


@pytest.mark.parametrize("older", [0, 1])
def test_snapshot_taken_while_a_call_runs(H, older):
    """Such a copy of the qacc buffer holds a number of workgroups behind the counts.  older: a snapshot that ends ahead of
    those words."""
    rng = np.random.default_rng(7820)
    oc, gc = H.make_pair(**KW)
    K, V, q = _tensors(rng, 128 * 9 + 50)
    gc.quantize_append(H.dev(K), H.dev(V))
    oc.append(K, V)
    H.check_attention(oc, gc, q)
    bufs, states = gc.snapshot()
    used = 3 * 2 * 129 * 8
    bufs[3][used:].fill_(1)
    gc.qacc.fill_(0x55)
    gc.restore((bufs[:3] + [bufs[3][:-(-used // 256) * 256]] + bufs[4:] if older else bufs, states))
    for _ in range(2):
        H.check_attention(oc, gc, q)
    H.check_state(oc, gc)

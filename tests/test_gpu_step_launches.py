"""How many launches a decode step of sequences of different lengths enqueues (counted in a captured graph), and that the
step leaves what the oracle has."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    assert torch.cuda.is_available(), "these tests need the GPU"
    import gpu_common
    return gpu_common


def _filled(H, rng, lens, kw):
    """Library cache and one oracle per sequence, filled to `lens` tokens."""
    import paper_2512_19206_amd as M
    from oracle import mixkvq_oracle as O
    gc = M.Cache(M.make_config(B=len(lens), **kw))
    ocs = []
    for b, n in enumerate(lens):
        K, V = (rng.standard_normal((1, kw["Hkv"], n, 128)).astype(np.float16) for _ in range(2))
        gc.quantize_append_seq(b, H.dev(K[0]), H.dev(V[0]))
        ocs.append(O.OracleCache(O.OracleConfig(B=1, **kw)))
        ocs[-1].append(K, V)
    return gc, ocs


def _launches(gc, body):
    """Nodes of one captured call (nothing runs during the capture)."""
    states = [gc.state_seq(b) for b in range(gc.cfg.B)]
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        body()
    for b, st in enumerate(states):
        gc.lib.mixkvq_cache_set_state_seq(gc.handle, b, *st)
    n = C.c_size_t(0)
    gc.lib.hipGraphGetNodes.argtypes = [C.c_void_p, C.c_void_p, C.POINTER(C.c_size_t)]
    assert gc.lib.hipGraphGetNodes(graph.raw_cuda_graph(), None, C.byref(n)) == 0
    return n.value


def _step(H, gc, ocs, rng, accumulate_q):
    B, Hq, Hkv = gc.cfg.B, gc.cfg.Hq, gc.cfg.Hkv
    kn, vn = (rng.standard_normal((B, Hkv, 1, 128)).astype(np.float16) for _ in range(2))
    q = rng.standard_normal((B, Hq, 128)).astype(np.float16)
    t = [H.dev(x) for x in (kn, vn, q)]
    out, lse = torch.empty_like(t[2]), torch.empty((B, Hq), device="cuda")
    call = lambda: gc.decode_step(*t, out=out, lse=lse, accumulate_q=accumulate_q)
    n = _launches(gc, call)
    call()
    torch.cuda.synchronize()
    got, got_lse = out.float().cpu().numpy(), lse.cpu().numpy()
    rk, rv = (x.cpu().numpy().view(np.uint16) for x in gc.residual())
    acc, cnt = (x.cpu().numpy().astype(np.uint64) for x in gc.query_accumulator())
    rec = gc.block_records().cpu().numpy()
    for b, oc in enumerate(ocs):
        oc.append(kn[b:b + 1], vn[b:b + 1])
        ro, rl = oc.decode_attention(q[b:b + 1], accumulate_q=accumulate_q)
        assert np.all(np.abs(got[b] - ro[0]) <= H.ATOL + H.RTOL * np.abs(ro[0])), b
        assert np.all(np.abs(got_lse[b] - rl[0]) <= H.LSE_ATOL + 1e-4 * np.abs(rl[0])), b
        p = slice(b * Hkv, (b + 1) * Hkv)
        assert gc.state_seq(b)[:2] == (oc.n_quant, oc.n_res)
        assert np.array_equal(rk[p, :oc.n_res], oc.res_k[:, :oc.n_res].view(np.uint16)), b
        assert np.array_equal(rv[p, :oc.n_res], oc.res_v[:, :oc.n_res].view(np.uint16)), b
        assert np.array_equal(acc[p], oc.qacc) and np.array_equal(cnt[p], oc.qcnt), b
        nb = oc.n_quant // gc.rec_tokens
        assert np.array_equal(rec[p, :nb], oc.packed_blocks()), b
    return n


@pytest.mark.parametrize("lens", [(100, 101, 100, 101, 70, 100, 101, 3, 100, 99, 98, 101)])
def test_vector_path_keeps_the_books_of_all_sequences_in_one_launch(H, lens):
    """Records of 48 tokens run on the vector-ALU path: rows and |q|, attention, merge."""
    import paper_2512_19206_amd as M
    rng = np.random.default_rng(7600)
    gc, ocs = _filled(H, rng, lens, dict(Hq=6, Hkv=2, D=128, T_max=192, Gk=16, Gv=128, R=48, k4=8, k16=0))
    assert _step(H, gc, ocs, rng, True) <= 3
    assert gc.decode_path() == M.PATH_VECTOR


@pytest.mark.parametrize("R,Gk", [(128, 128), (256, 128)])
def test_accumulators_of_all_packed_sequences_are_cleared_in_one_launch(H, R, Gk):
    """Six of eight full windows leave in one step (records of one block each: one pack launch; of two records: scored and
    packed per run of neighbours in equal state), their accumulators are cleared with one launch, then attention."""
    rng = np.random.default_rng(7700 + R)
    lens = (R, R, 70, 2 * R, R, R, 100, R)
    gc, ocs = _filled(H, rng, lens, dict(Hq=6, Hkv=2, D=128, T_max=4 * R, Gk=Gk, Gv=128, R=R, k4=8, k16=0,
                                         qacc_reset_on_flush=1))
    _step_q = rng.standard_normal((len(lens), 6, 128)).astype(np.float16)
    gc.decode_attention(H.dev(_step_q), accumulate_q=True)      # something to clear
    for b, oc in enumerate(ocs):
        oc.decode_attention(_step_q[b:b + 1], accumulate_q=True)
    runs = 4                                                     # (R, R) (2 R) (R, R) (R)
    assert _step(H, gc, ocs, rng, True) <= (1 if R == 128 else 2 * runs) + 2
    assert _step(H, gc, ocs, rng, True) == 1

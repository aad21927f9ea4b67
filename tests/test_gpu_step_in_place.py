"""The decode step that moves its own tokens: sequences of different lengths (several full windows packed by one
launch, blocks of several records, eager flush, vector-ALU kernel, sink rows).  Every sequence against its own
single-sequence oracle, state bit for bit."""
import numpy as np
import pytest
import torch

from oracle import mixkvq_oracle as O
from test_gpu_ragged import _check_seq as check_seq_record_r

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    assert torch.cuda.is_available(), "these tests need the GPU"
    import gpu_common
    return gpu_common


def _check_seq(H, gc, b, oc, Hkv):
    """check_seq_record_r for caches whose blocks may be several records."""
    torch.cuda.synchronize()
    assert gc.state_seq(b) == (oc.n_quant, oc.n_res, oc.n_sink)
    nb = oc.n_quant // O.rec_tokens(oc.cfg)
    if nb:
        got = gc.block_records()[b * Hkv:(b + 1) * Hkv, :nb].cpu().numpy()
        assert np.array_equal(got, oc.packed_blocks()), f"records of sequence {b} differ"
    if O.rec_tokens(oc.cfg) == oc.cfg.R:
        check_seq_record_r(H, gc, b, oc, Hkv)


@pytest.mark.parametrize("over,path", [
    (dict(R=128, Gk=128, Gv=128, k4=16, k16=0), 1),
    (dict(R=128, Gk=32, Gv=32, k4=16, k16=8, policy=1, tau16=5.0, tau4=2.0), 1),
    (dict(R=32, Gk=32, Gv=32, k4=8, k16=0, qacc_reset_on_flush=1), 1),
    (dict(R=256, Gk=128, Gv=128, k4=16, k16=0, qacc_reset_on_flush=1), 1),      # two records per block
    (dict(R=64, Gk=64, Gv=64, k4=16, k16=0, sink=32), 1),
    (dict(R=64, Gk=64, Gv=128, k4=16, k16=0, flush_mode=1), 1),                 # eager: the new token is packed at once
    (dict(R=48, Gk=16, Gv=16, k4=8, k16=4), 2),                                 # vector-ALU kernel
])
def test_ragged_steps_with_flushes(H, over, path):
    import paper_2512_19206_amd as M
    rng = np.random.default_rng(7100 + over["R"])
    B, Hkv, g, R = 5, 2, 3, over["R"]
    sink = over.get("sink", 0)
    kw = dict(Hq=Hkv * g, Hkv=Hkv, D=128, T_max=6 * R, **over)
    gc = M.Cache(M.make_config(B=B, **kw))
    ocs = [O.OracleCache(O.OracleConfig(B=1, **kw)) for _ in range(B)]
    # sequences 0, 2 and 3 fill their windows on the same step (at different lengths), 1 a step later, 4 starts empty
    full = 3
    for b, n in enumerate((2 * R - full + sink, R - full - 1 + sink, 3 * R - full + sink, 2 * R - full + sink, 0)):
        if n:
            K = (rng.standard_normal((1, Hkv, n, 128)) * rng.uniform(0.3, 8, 128)).astype(np.float16)
            V = rng.standard_normal((1, Hkv, n, 128)).astype(np.float16)
            Qp = rng.standard_normal((1, Hkv * g, 8, 128)).astype(np.float16)
            sel = ocs[b].select_channels(Qp, K)
            got = gc.select_channels_seq(b, H.dev(Qp)[0], H.dev(K)[0])
            ocs[b].append(K, V, sel)
            gc.quantize_append_seq(b, H.dev(K)[0], H.dev(V)[0], sel=got)
    for step in range(full + 4):
        k1 = (rng.standard_normal((B, Hkv, 1, 128)) * rng.uniform(0.3, 8, 128)).astype(np.float16)
        v1 = rng.standard_normal((B, Hkv, 1, 128)).astype(np.float16)
        q1 = rng.standard_normal((B, Hkv * g, 128)).astype(np.float16)
        out, lse = gc.decode_step(H.dev(k1), H.dev(v1), H.dev(q1), accumulate_q=True)
        torch.cuda.synchronize()
        assert gc.decode_path() == path
        go, gl = out.float().cpu().numpy(), lse.cpu().numpy()
        for b in range(B):
            ocs[b].append(k1[b:b + 1], v1[b:b + 1])
            ro, rl = ocs[b].decode_attention(q1[b:b + 1], accumulate_q=True)
            assert np.all(np.abs(go[b] - ro[0]) <= H.ATOL + H.RTOL * np.abs(ro[0])), (step, b)
            assert np.all(np.abs(gl[b] - rl[0]) <= H.LSE_ATOL + 1e-4 * np.abs(rl[0])), (step, b)
        for b in range(B):
            _check_seq(H, gc, b, ocs[b], Hkv)

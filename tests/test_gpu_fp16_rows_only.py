"""Caches that hold nothing but fp16 rows (sink, window), attended by the matrix-core kernel."""
import numpy as np
import pytest
import torch

from oracle import mixkvq_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    assert torch.cuda.is_available(), "these tests need the GPU"
    import gpu_common
    return gpu_common


@pytest.mark.parametrize("R,sink,n,g,bf16", [(128, 0, 1, 7, 0), (128, 0, 90, 5, 1), (32, 0, 31, 8, 0), (64, 32, 20, 1, 0),
                                             (256, 128, 383, 2, 0), (256, 128, 129, 3, 1)])
def test_fp16_rows_only(H, R, sink, n, g, bf16):
    """Nothing packed yet: one step over the sink and window rows, on the matrix-core kernel."""
    import paper_2512_19206_amd as M
    rng = np.random.default_rng(7200 + R + n)
    B, Hkv = 3, 2
    kw = dict(B=B, Hq=Hkv * g, Hkv=Hkv, D=128, T_max=4 * R, Gk=32, Gv=32, R=R, k4=16, k16=0, sink=sink)
    oc = O.OracleCache(O.OracleConfig(**kw))
    gc = M.Cache(M.make_config(**dict(kw, in_dtype=bf16)))
    t = torch.bfloat16 if bf16 else torch.float16
    draw = lambda *s: torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda().to(t)
    as_np = lambda x: x.to(torch.float16).cpu().numpy()
    K, V, q = draw(B, Hkv, n + 1, 128), draw(B, Hkv, n + 1, 128), draw(B, Hkv * g, 128)
    gc.quantize_append(K[:, :, :n], V[:, :, :n])
    oc.append(as_np(K), as_np(V))
    out, lse = gc.decode_step(K[:, :, n:], V[:, :, n:], q, accumulate_q=True)
    torch.cuda.synchronize()
    assert gc.decode_path() == M.PATH_MATRIX
    ro, rl = oc.decode_attention(as_np(q), accumulate_q=True)
    rtol = H.RTOL + (2.0 ** -9 if bf16 else 0.0)      # bfloat16 output: 8 significant bits
    assert np.all(np.abs(out.float().cpu().numpy() - ro) <= H.ATOL + rtol * np.abs(ro))
    assert np.all(np.abs(lse.cpu().numpy() - rl) <= H.LSE_ATOL + 1e-4 * np.abs(rl))
    H.check_state(oc, gc)

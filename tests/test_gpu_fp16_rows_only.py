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


@pytest.mark.parametrize("n,g,R,sink,far", [(2, 7, 128, 0, 0), (5, 1, 64, 32, 1), (33, 8, 128, 0, 1), (90, 7, 128, 0, 0), (290, 4, 256, 64, 1)])
def test_fp16_rows_in_binary32(H, n, g, R, sink, far):
    """The softmax weights and the queries of fp16 rows keep what binary32 gives them.  Bars: a logit is four matrix steps
    of 32 products each, whose binary32 sums round at most a few times per step (16 in all, 2^-20 of the sum of
    magnitudes); exp2, log2, the sum of the weights and their two binary16 parts (22 bits) add 2^-20 of the result; the
    output is then rounded to binary16 once (2^-11).  Weights rounded to binary16 miss the log-sum-exp bar by up to 2^-13.
    far: an element 2^15 above the others in the queries meets zeros in the keys, so the small ones decide."""
    import paper_2512_19206_amd as M
    rng = np.random.default_rng(7300 + n)
    B, Hkv = 2, 2
    kw = dict(B=B, Hq=Hkv * g, Hkv=Hkv, D=128, T_max=4 * R, Gk=64, Gv=64, R=R, k4=16, k16=0, sink=sink)
    gc = M.Cache(M.make_config(**kw))
    K = rng.standard_normal((B, Hkv, n, 128)).astype(np.float16)
    V = rng.standard_normal((B, Hkv, n, 128)).astype(np.float16)
    q = (0.5 * rng.standard_normal((B, Hkv * g, 128))).astype(np.float16)
    if far:
        q[..., 5] = np.float16(32768.0)
        K[..., 5] = 0
    d = lambda a: torch.from_numpy(a).cuda()
    gc.quantize_append(d(K), d(V))
    out, lse = gc.decode_attention(d(q))
    torch.cuda.synchronize()
    assert gc.decode_path() == M.PATH_MATRIX
    k64, v64 = (np.repeat(x.astype(np.float64), g, axis=1) for x in (K, V))
    prod = q.astype(np.float64)[:, :, None] * k64
    s = prod.sum(-1) / np.sqrt(128.0)
    ds = (np.abs(prod).sum(-1) / np.sqrt(128.0)).max(-1) * 2.0 ** -20      # error of a logit
    m = s.max(-1, keepdims=True)
    p = np.exp(s - m)
    ref_lse = (m + np.log(p.sum(-1, keepdims=True)))[..., 0]
    p /= p.sum(-1, keepdims=True)
    ref = np.einsum("bht,bhtd->bhd", p, v64)
    err_lse = np.abs(lse.cpu().numpy() - ref_lse)
    assert np.all(err_lse <= ds + 2.0 ** -20 * (1.0 + np.abs(ref_lse))), f"lse off by {err_lse.max():.2e}"
    err = np.abs(out.float().cpu().numpy() - ref)
    mass = np.einsum("bht,bhtd->bhd", p, np.abs(v64))
    bar = 2.0 ** -11 * np.abs(ref) * (1 + 2.0 ** -11) + (2.0 * ds[..., None] + 2.0 ** -19) * mass + 2.0 ** -25
    assert np.all(err <= bar), f"out: excess {(err - bar).max():.2e} of {err.max():.2e}"

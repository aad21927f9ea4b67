"""`out` may start at any element: outputs into a tensor 2, 4, 6 or 8 bytes off are those of an aligned one, and nothing
around them is written.  The same for the queries of a cache that holds fp16 rows only."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [1, 2, 3, 4])
@pytest.mark.parametrize("T,noalloc", [(90, 0), (128 * 12 + 7, 0), (128 * 12 + 7, 1)])      # one workgroup per pair; a merge inside; a merge launch
def test_outputs_at_any_element(T, noalloc, off):
    assert torch.cuda.is_available(), "these tests need the GPU"
    import gpu_common as H
    rng = np.random.default_rng(7900 + T)
    B, Hq, Hkv = 2, 10, 2
    _, gc = H.make_pair(B=B, Hq=Hq, Hkv=Hkv, D=128, T_max=2048, Gk=128, Gv=128, R=128, k4=16, k16=0)
    K = H.dev(rng.standard_normal((B, Hkv, T, 128)).astype(np.float16))
    gc.quantize_append(K, K)
    q = H.dev(rng.standard_normal((B, Hq, 128)).astype(np.float16))
    want, lse = gc.decode_attention(q)
    n = B * Hq * 128
    room = torch.full((n + 16,), 7.0, dtype=torch.float16, device="cuda")
    out = room[off:off + n].view(B, Hq, 128)
    (gc.decode_attention_noalloc if noalloc else gc.decode_attention)(q, out=out, lse=torch.empty_like(lse))
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    assert bool((room[:off] == 7.0).all()) and bool((room[off + n:] == 7.0).all())


@pytest.mark.parametrize("off", [1, 2, 3, 4])
def test_queries_at_any_element_over_fp16_rows(off):
    import gpu_common as H
    import paper_2512_19206_amd as M
    rng = np.random.default_rng(7950)
    oc, gc = H.make_pair(B=2, Hq=10, Hkv=2, D=128, T_max=2048, Gk=128, Gv=128, R=128, k4=16, k16=0)
    K, V = (rng.standard_normal((2, 2, 91, 128)).astype(np.float16) for _ in range(2))
    q = rng.standard_normal((2, 10, 128)).astype(np.float16)
    gc.quantize_append(H.dev(K[:, :, :90]), H.dev(V[:, :, :90]))
    oc.append(K, V)
    room = torch.full((q.size + 16,), 7.0, dtype=torch.float16, device="cuda")
    at = room[off:off + q.size].view(2, 10, 128)
    at.copy_(H.dev(q))
    out, lse = gc.decode_step(H.dev(K[:, :, 90:]), H.dev(V[:, :, 90:]), at, accumulate_q=True)
    torch.cuda.synchronize()
    ro, rl = oc.decode_attention(q, accumulate_q=True)
    assert gc.decode_path() == (M.PATH_MATRIX if off == 4 else M.PATH_VECTOR)
    assert np.all(np.abs(out.float().cpu().numpy() - ro) <= H.ATOL + H.RTOL * np.abs(ro))
    assert np.all(np.abs(lse.cpu().numpy() - rl) <= H.LSE_ATOL + 1e-4 * np.abs(rl))
    H.check_state(oc, gc)

"""32 fp16 channels with value groups of 32: the widest fp16 tier, whose variants of the decode kernel have no register to spare."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Gk,paged", [(64, 0), (128, 1)])
def test_attention_over_the_widest_fp16_tier(Gk, paged):
    assert torch.cuda.is_available(), "these tests need the GPU"
    import gpu_common as H
    import paper_2512_19206_amd as M
    rng = np.random.default_rng(7500 + Gk)
    B, Hkv, g, T = 2, 2, 5, 128 * 9 + 40
    kw = dict(B=B, Hq=Hkv * g, Hkv=Hkv, D=128, T_max=128 * 12, Gk=Gk, Gv=32, R=128, k4=0, k16=32)
    oc, gc = H.make_pair(**kw)
    if paged:
        gc.set_block_table(torch.from_numpy(rng.permutation(B * 12).astype(np.int32)).cuda().view(B, 12).contiguous())
    K = (rng.standard_normal((B, Hkv, T, 128)) * np.where(rng.random((B, Hkv, 1, 128)) < 0.2, 8.0, 1.0)).astype(np.float16)
    V = rng.standard_normal((B, Hkv, T, 128)).astype(np.float16)
    gc.quantize_append(H.dev(K), H.dev(V))
    oc.append(K, V)
    for i in range(2):
        H.check_attention(oc, gc, rng.standard_normal((B, Hkv * g, 128)).astype(np.float16))
        assert gc.decode_path() == M.PATH_MATRIX

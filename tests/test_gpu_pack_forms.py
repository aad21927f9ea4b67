"""The forms of the pack kernel (512 or 1 024 threads; keys and values apart; both together; room for one group's parameters or
for eight) give the same records: a batch large enough for one form against its sequences one by one, which take another,
and the first of those against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scored", [False, True])
@pytest.mark.parametrize("B,blocks,G,over", [
    (16, 33, 128, dict(k4=16, k16=0)),                 # 2 112 blocks together / 132 apart per sequence
    (16, 33, 32, dict(k4=16, k16=8)),
    (8, 14, 128, dict(k4=16, k16=0)),                  # 448 blocks apart, up to four workgroups per compute unit / 56 with 512 threads
    (4, 12, 128, dict(k4=0, k16=12)),                  # 192 blocks apart, three per compute unit / 48 with 512 threads
    (4, 12, 64, dict(k4=8, k16=4)),
    (4, 12, 16, dict(k4=16, k16=0)),                   # eight key groups, eight value groups
    (4, 12, 32, dict(k4=32, k16=12, policy=1, tau16=4.0, tau4=1.0)),
])
def test_same_records(B, blocks, G, over, scored):
    import gpu_common as H
    import paper_2512_19206_amd as M
    Hkv, R, T = 4, 128, 128 * blocks + 37
    kw = dict(Hq=Hkv, Hkv=Hkv, D=128, T_max=R * (blocks + 1), Gk=G, Gv=G, R=R, **over)
    gen = torch.Generator(device="cuda").manual_seed(B + G)
    k = (torch.randn((B, Hkv, T, 128), generator=gen, device="cuda") * torch.linspace(0.3, 5, 128, device="cuda")).half()
    v, q = torch.randn((B, Hkv, T, 128), generator=gen, device="cuda").half(), torch.randn((B, Hkv, 8, 128), generator=gen, device="cuda").half()
    batch = M.Cache(M.make_config(B=B, **kw))
    sel = batch.select_channels(q, k)
    batch.quantize_append(k, v, sel=None if scored else sel)
    n = blocks * (R // batch.rec_tokens)
    for b in range(0, B, max(1, B // 4)):
        oc, one = H.make_pair(B=1, **kw)
        s1 = one.select_channels(q[b:b + 1], k[b:b + 1])
        assert torch.equal(s1[0], sel[b])
        one.quantize_append(k[b:b + 1], v[b:b + 1], sel=None if scored else s1)
        torch.cuda.synchronize()
        assert torch.equal(one.block_records()[:, :n], batch.block_records()[b * Hkv:(b + 1) * Hkv, :n]), b
        for x, y in zip(one.fp16_rows(), batch.fp16_rows()):
            assert torch.equal(x[:, :37], y[b * Hkv:(b + 1) * Hkv, :37])
        if b == 0 and blocks < 20:
            K, V, Q = (t[:1].cpu().numpy() for t in (k, v, q))
            rs = oc.select_channels(Q, K)
            oc.append(K, V, None if scored else rs)
            H.check_state(oc, one)

"""Small launches pack the keys and the values of a block in two workgroups and move the tokens that stay in the window in
the same launch: in workgroups of their own when no block reads the window, by the first block when that one does.
Records, window rows and counts are compared byte for byte with the oracle, on either side of both rules (blocks per
launch, tokens waiting in the window, blocks of two records)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import gpu_common
    return gpu_common


@pytest.mark.parametrize("kw", [
    dict(Gk=128, Gv=128, R=128, k4=16, k16=0),
    dict(Gk=32, Gv=32, R=128, k4=8, k16=4, policy=1, tau16=1.5, tau4=0.3),
    dict(Gk=128, Gv=64, R=256, k4=8, k16=0),          # two records per block
    dict(Gk=32, Gv=32, R=32, k4=8, k16=0, in_dtype=0, sink=32),
])
@pytest.mark.parametrize("first", [0, 1, 100, 128, 200])      # tokens in the cache before
@pytest.mark.parametrize("n", [29, 129, 385])                 # tokens of the call
def test_append_onto_a_window(H, kw, first, n):
    kw = dict(B=2, Hq=4, Hkv=2, D=128, T_max=1024, **kw)
    oc, gc = H.make_pair(**kw)
    rng = np.random.default_rng(first * 1000 + n)
    K = (rng.standard_normal((2, 2, first + n, 128)) * rng.uniform(0.3, 9, 128)).astype(np.float16)
    V = rng.standard_normal((2, 2, first + n, 128)).astype(np.float16)
    Q = rng.standard_normal((2, 4, 3, 128)).astype(np.float16)
    gc.select_channels(H.dev(Q), H.dev(K))
    oc.select_channels(Q, K)
    for a, b in ((0, first), (first, first + n)):
        if b > a:
            gc.quantize_append(H.dev(K[:, :, a:b]), H.dev(V[:, :, a:b]))
            oc.append(K[:, :, a:b], V[:, :, a:b])
    H.check_state(oc, gc)


@pytest.mark.parametrize("blocks", [2047, 2048, 2049])
def test_both_forms_give_the_same_records(H, blocks):
    """One pair, more blocks than any oracle run is worth: records of a launch just above the line against records of
    the same tokens appended in pieces far below it."""
    import torch
    import paper_2512_19206_amd as M
    kw = dict(B=1, Hq=2, Hkv=1, D=128, T_max=(blocks + 1) * 32, Gk=32, Gv=128, R=32, k4=8, k16=0)
    gen = torch.Generator(device="cuda").manual_seed(blocks)
    n = blocks * 32 + 5
    k = (torch.randn((1, 1, n, 128), generator=gen, device="cuda") * 3).half()
    v = torch.randn((1, 1, n, 128), generator=gen, device="cuda").half()
    caches = [M.Cache(M.make_config(**kw)) for _ in range(2)]
    q = torch.cat((k[:, :, :300], v[:, :, :300]), dim=1)
    sel = [c.select_channels(q, k) for c in caches]
    assert torch.equal(sel[0], sel[1])
    caches[0].quantize_append(k, v, sel=sel[0])
    for t in range(0, n, 1000):
        caches[1].quantize_append(k[:, :, t:t + 1000], v[:, :, t:t + 1000], sel=sel[1])
    assert caches[0].state() == caches[1].state() == (blocks * 32, 5)
    assert torch.equal(caches[0].block_records()[:, :blocks], caches[1].block_records()[:, :blocks])
    for a, b in zip(caches[0].residual(), caches[1].residual()):
        assert torch.equal(a[:, :5], b[:, :5])


def _behind_a_window(R, blocks, first, Gk, Gv, dtype="float16"):
    import torch
    import paper_2512_19206_amd as M
    first = R if first < 0 else first
    kw = dict(B=1, Hq=2, Hkv=2, D=128, T_max=(blocks // 2 + 2) * R, Gk=Gk, Gv=Gv, R=R, k4=8, k16=0, in_dtype=int(dtype == "bfloat16"))
    gen = torch.Generator(device="cuda").manual_seed(blocks + first)
    n = first + (blocks // 2) * R + R // 2
    k = (torch.randn((1, 2, n, 128), generator=gen, device="cuda") * 3).to(getattr(torch, dtype))
    v = torch.randn((1, 2, n, 128), generator=gen, device="cuda").to(getattr(torch, dtype))
    caches = [M.Cache(M.make_config(**kw)) for _ in range(2)]
    sel = caches[0].select_channels(k[:, :, :300], k)
    for c, piece in zip(caches, (n, 5 * R + 3)):
        cuts = ([0, first] if first else [0]) + list(range(first + piece, n, piece)) + [n]
        for a, b in zip(cuts, cuts[1:]):
            c.quantize_append(k[:, :, a:b], v[:, :, a:b], sel=sel)
    assert caches[0].state() == caches[1].state()
    nq, r = caches[0].state()
    assert nq // R >= blocks // 2 and r > 0
    assert torch.equal(caches[0].block_records()[:, :nq // R], caches[1].block_records()[:, :nq // R])
    for x, y in zip(caches[0].residual(), caches[1].residual()):
        assert torch.equal(x[:, :r], y[:, :r])


@pytest.mark.parametrize("R,blocks", [(64, 1406), (64, 1408), (64, 1410), (16, 1410), (32, 1600), (128, 2050)])
@pytest.mark.parametrize("first", [0, 7, -1])      # tokens that wait in the window before the call (-1: a full window)
def test_large_launches_behind_a_window(R, blocks, first):
    """On either side of the line, and above it with the window read (and then overwritten) by the first block: records,
    window rows and the selection against the same tokens in pieces far below the line."""
    _behind_a_window(R, blocks, first, min(R, 32), 64)


@pytest.mark.parametrize("R,blocks,dtype", [(128, 2050, "float16"), (128, 2050, "bfloat16"), (64, 1410, "bfloat16"), (128, 380, "float16"), (128, 800, "bfloat16")])
@pytest.mark.parametrize("first", [0, 7, -1])
def test_one_group_launches_behind_a_window(R, blocks, dtype, first):
    """The same with one key and one value group, where the values are asked for behind the 2-bit keys: above the line (the
    first block's values come from the window it overwrites), three and four workgroups to a compute unit below it."""
    _behind_a_window(R, blocks, first, R, 128, dtype)


@pytest.mark.parametrize("per_pair", [15, 16, 17])      # 120, 128 and 136 records in a launch of 8 pairs
@pytest.mark.parametrize("kw", [
    dict(Gk=128, Gv=128, R=128, k4=16, k16=0),
    dict(Gk=64, Gv=64, R=128, k4=0, k16=12),
    dict(Gk=16, Gv=16, R=128, k4=24, k16=4),
    dict(Gk=32, Gv=32, R=128, k4=16, k16=8, policy=1, tau16=1.5, tau4=0.3),
])
def test_both_widths_give_the_same_records(H, kw, per_pair):
    """Records of one launch around the line between workgroups of 512 or 1 024 and of 256 threads against the oracle's."""
    kw = dict(B=2, Hq=8, Hkv=4, D=128, T_max=(per_pair + 1) * 128, **kw)
    oc, gc = H.make_pair(**kw)
    rng = np.random.default_rng(per_pair)
    n = per_pair * 128 + 3
    K = (rng.standard_normal((2, 4, n, 128)) * rng.uniform(0.3, 9, 128)).astype(np.float16)
    V = rng.standard_normal((2, 4, n, 128)).astype(np.float16)
    Q = rng.standard_normal((2, 8, 3, 128)).astype(np.float16)
    sel, ref = gc.select_channels(H.dev(Q), H.dev(K)), oc.select_channels(Q, K)
    scored = kw.get("policy", 0) == 1
    gc.quantize_append(H.dev(K), H.dev(V), sel=None if scored else sel)
    oc.append(K, V, None if scored else ref)
    H.check_state(oc, gc)

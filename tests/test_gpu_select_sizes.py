"""Scoring and selection run as one launch whose workgroups take pieces of the queries and of the keys: lengths around
its passes of 16 rows, batches of eight loads and pieces of 256 rows, rows of any alignment, one sequence of a batch, and
the |q| counts (exact after every call).  Everything is compared with the oracle as whole numbers."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import gpu_common
    return gpu_common


def _draw(seed, B, H, L):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((B, H, L, 128)) * rng.uniform(0.2, 9, (1, H, 1, 128)) * rng.uniform(0.3, 3, (B, H, L, 1))
    return x.astype(np.float16)


def _padded(a):
    """The same values in rows of 133 elements that start at an odd element: no row is 16-byte aligned."""
    t = torch.zeros(a.shape[:-1] + (133,), dtype=torch.float16, device="cuda")
    t[..., 1:129] = torch.from_numpy(a).cuda()
    return t[..., 1:129]


@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("policy", [dict(k4=16, k16=4), dict(k4=8, k16=8, policy=1, tau16=2.0, tau4=0.5)])
@pytest.mark.parametrize("L,Lq", [(1, 1), (15, 17), (112, 113), (128, 0), (255, 256), (257, 129), (8449, 300)])
def test_selection_and_sums(H, L, Lq, policy, aligned):
    kw = dict(B=2, Hq=6, Hkv=2, D=128, T_max=256, Gk=128, Gv=128, R=128, **policy)
    oc, gc = H.make_pair(**kw)
    put = H.dev if aligned else _padded
    for call in range(2):      # (Lq = 0: the second call scores with the sums of the first)
        K, Q = _draw(10 * L + call, 2, 2, L), _draw(10 * L + call + 5, 2, 6, Lq or 1)
        sel = gc.select_channels(None if Lq == 0 and call else put(Q), put(K)).cpu().numpy()
        ref = oc.select_channels(None if Lq == 0 and call else Q, K)
        assert np.array_equal(sel, ref)
        acc, cnt = gc.query_accumulator()
        assert np.array_equal(acc.cpu().numpy().astype(np.uint64), oc.qacc)
        assert np.array_equal(cnt.cpu().numpy().astype(np.uint64), oc.qcnt)


def test_one_sequence_of_a_batch(H):
    kw = dict(B=3, Hq=4, Hkv=2, D=128, T_max=256, Gk=128, Gv=128, R=128, k4=16, k16=0)
    _, gc = H.make_pair(**kw)
    o1, _ = H.make_pair(**dict(kw, B=1))
    K, Q = _draw(1, 1, 2, 600), _draw(2, 1, 4, 300)
    sel = gc.select_channels_seq(1, H.dev(Q[0]), H.dev(K[0])).cpu().numpy()
    assert np.array_equal(sel, o1.select_channels(Q, K)[0])
    acc, cnt = gc.query_accumulator()
    acc, cnt = acc.cpu().numpy().astype(np.uint64), cnt.cpu().numpy().astype(np.uint64)
    assert np.array_equal(acc[2:4], o1.qacc) and np.array_equal(cnt[2:4], o1.qcnt)
    assert not acc[:2].any() and not acc[4:].any() and not cnt[:2].any() and not cnt[4:].any()

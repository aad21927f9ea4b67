"""Ranking of channels whose scores tie: equal scores (lower index first) and scores that differ only in the lower half of
their binary64 bit pattern, in the selection and in blocks that the pack kernel scores itself, against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _tensors(kind, T, seed):
    """Keys of range 2 in every channel; queries whose |q| sums are 1024 + n_d 2^-14 with n_d a permutation ('lower': runs of
    16 share the upper half), all equal ('equal'), or equal in every second channel ('mixed').  'ranges': keys of a few
    ranges, n_d as in 'lower'."""
    rng = np.random.default_rng(seed)
    K = rng.uniform(-1, 1, (1, 2, T, 128)).astype(np.float16)
    K[:, :, 0::128], K[:, :, 1::128] = 1.0, -1.0      # (in every block of 128 or 32 tokens that starts there)
    K[:, :, 32::128], K[:, :, 33::128] = 1.0, -1.0
    K[:, :, 64::128], K[:, :, 65::128] = 1.0, -1.0
    K[:, :, 96::128], K[:, :, 97::128] = 1.0, -1.0
    Q = np.zeros((1, 2, 2, 128), np.float16)
    n = rng.permutation(128)
    if kind == "equal":
        n[:] = 5
    elif kind == "mixed":
        n[::2] = 5
    elif kind == "ranges":
        K *= rng.choice([0.25, 0.5, 1.0, 2.0], 128).astype(np.float16)
    Q[:, :, 0] = 1024.0
    Q[:, :, 1] = (n * 2.0 ** -14).astype(np.float16)
    return K, rng.standard_normal((1, 2, T, 128)).astype(np.float16), Q


@pytest.mark.parametrize("policy", [dict(k4=16, k16=0), dict(k4=16, k16=8, policy=1, tau16=1000.0, tau4=10.0),
                                    dict(k4=24, k16=12, score_mode=1)])
@pytest.mark.parametrize("R,G,blocks", [(128, 128, 1), (128, 32, 2), (128, 128, 70), (128, 64, 70), (32, 32, 3)])
@pytest.mark.parametrize("kind", ["equal", "lower", "mixed", "ranges"])
def test_ties(kind, R, G, blocks, policy):
    import gpu_common as H
    T = R * blocks + 1
    K, V, Q = _tensors(kind, T, R + blocks)
    kw = dict(B=1, Hq=2, Hkv=2, D=128, T_max=R * (blocks + 1), Gk=G, Gv=G, R=R, **policy)
    oc, gc = H.make_pair(**kw)
    ref = oc.select_channels(Q, K)
    assert np.array_equal(gc.select_channels(H.dev(Q), H.dev(K)).cpu().numpy(), ref)
    gc.quantize_append(H.dev(K), H.dev(V))      # every block scored on its own tokens
    oc.append(K, V)
    H.check_state(oc, gc)


def test_no_query_has_been_seen():
    """All scores 0: the first channels by index."""
    import gpu_common as H
    oc, gc = H.make_pair(B=1, Hq=2, Hkv=1, D=128, T_max=512, Gk=128, Gv=128, R=128, k4=8, k16=4)
    K = np.random.default_rng(1).standard_normal((1, 1, 300, 128)).astype(np.float16)
    sel = gc.select_channels(None, H.dev(K)).cpu().numpy()
    assert np.array_equal(sel, oc.select_channels(None, K)) and np.array_equal(sel[0, 0], np.arange(12))
    gc.quantize_append(H.dev(K), H.dev(K))
    oc.append(K, K)
    H.check_state(oc, gc)

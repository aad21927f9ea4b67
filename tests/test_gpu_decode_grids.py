"""Both sides of the lines at which the matrix-core kernel changes its grid or its variant: four or eight wavefronts in a
workgroup, one workgroup per pair or several, merges of one and of several rounds, caches with fp16 rows only, launches that
read more than the last-level cache holds."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,g,blocks,over", [
    (1, 1, 1, 40, {}),               # eleven workgroups of four
    (2, 4, 1, 52, {}),               # fourteen of four: sixteen partials in flight
    (1, 2, 3, 110, {}),              # twenty-nine
    (1, 3, 1, 240, {}),              # sixty-one of four: thirty-one of eight
    (16, 2, 5, 62, {}),              # sixteen of four, more than 256 of them: eight of eight
    (20, 2, 7, 62, {}),              # twelve of four
    (24, 8, 1, 7, {}),               # two of four: one of eight, nothing to merge
    (33, 8, 8, 3, {}),               # one of four
    (38, 8, 1, 2, dict(R=256)),      # two of four, no room for all of eight at once
    (3, 8, 2, 20, dict(R=32, Gk=32, Gv=32)),
    (2, 2, 3, 30, dict(R=256, sink=128)),      # twelve sub-units of fp16 rows
    (5, 4, 6, 0, dict(sink=64)),     # fp16 rows only
    (70, 4, 3, 0, dict(R=256)),
    # up to three pairs of more than 512 records: the ceiling of 64 workgroups a pair, eight wavefronts each
    (1, 1, 5, 1100, dict(R=32, Gk=32, Gv=32)),
    (2, 1, 7, 520, dict(R=32, Gk=32, Gv=32)),
    (1, 3, 1, 640, dict(R=64, Gk=64)),
])
def test_against_the_oracle(B, Hkv, g, blocks, over):
    import gpu_common as H
    kw = dict(B=1, Hq=Hkv * g, Hkv=Hkv, D=128, Gk=128, Gv=128, R=128, k4=16, k16=0)
    kw.update(over)
    R = kw["R"]
    kw["T_max"] = R * (blocks + 2)
    T = kw.get("sink", 0) + R * blocks + R - 3
    rng = np.random.default_rng(B + blocks)
    K = (rng.standard_normal((1, Hkv, T, 128)) * rng.uniform(0.3, 4, 128)).astype(np.float16)
    V = rng.standard_normal((1, Hkv, T, 128)).astype(np.float16)
    import paper_2512_19206_amd as M
    from oracle import mixkvq_oracle as O
    oc, gc = O.OracleCache(O.OracleConfig(**kw)), M.Cache(M.make_config(**dict(kw, B=B)))
    one = M.Cache(M.make_config(**kw))
    oc.append(K, V)
    one.quantize_append(H.dev(K), H.dev(V))
    # every sequence of the batch is a copy of the one
    for dst, src in ((gc.block_records(), one.block_records()), (gc.fp16_rows()[0], one.fp16_rows()[0]), (gc.fp16_rows()[1], one.fp16_rows()[1])):
        dst.view(B, Hkv, *dst.shape[1:]).copy_(src[None].expand(B, *src.shape))
    M.load_library().mixkvq_cache_set_state(gc.handle, *one.state_seq(0))
    for step in range(2):      # (twice: the tickets are back at 0)
        q = rng.standard_normal((1, Hkv * g, 128)).astype(np.float16)
        kn, vn = (rng.standard_normal((1, Hkv, 1, 128)).astype(np.float16) for _ in range(2))
        rep = lambda a: H.dev(np.repeat(a, B, axis=0))
        out, lse = gc.decode_step(rep(kn), rep(vn), rep(q), accumulate_q=True)
        torch.cuda.synchronize()
        oc.append(kn, vn)
        ref, ref_lse = oc.decode_attention(q, accumulate_q=True)
        assert gc.decode_path() == M.PATH_MATRIX
        err = np.abs(out.float().cpu().numpy() - ref)
        assert np.all(err <= H.ATOL + H.RTOL * np.abs(ref)), err.max()
        assert np.all(np.abs(lse.cpu().numpy() - ref_lse) <= H.LSE_ATOL + 1e-4 * np.abs(ref_lse))
        assert torch.equal(out, out[:1].expand_as(out)) and torch.equal(lse, lse[:1].expand_as(lse))
        acc, cnt = gc.query_accumulator()
        assert np.array_equal(acc[-Hkv:].cpu().numpy().astype(np.uint64), oc.qacc) and int(cnt[-1]) == int(oc.qcnt.ravel()[-1])
    # through the entry point with partials of its own: the same grid, the merge a launch of its own
    again, lse2 = gc.decode_attention_noalloc(rep(q), torch.empty_like(out), torch.empty_like(lse))
    torch.cuda.synchronize()
    assert gc.decode_path() == M.PATH_MATRIX and torch.equal(again, out) and torch.equal(lse2, lse)


@pytest.mark.parametrize("k4,k16", [(16, 0), (0, 12), (8, 0)])
def test_more_than_the_last_level_cache(k4, k16):
    """300 MB of records, copies of one sequence's: the same outputs for all of them, and as the sequence's own cache."""
    import paper_2512_19206_amd as M
    B, Hkv, g, blocks = 64, 8, 5, 63
    kw = dict(Hq=Hkv * g, Hkv=Hkv, D=128, T_max=128 * (blocks + 1), Gk=128, Gv=128, R=128, k4=k4, k16=k16)
    gen = torch.Generator(device="cuda").manual_seed(k4)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda").half()
    one, gc = M.Cache(M.make_config(B=1, **kw)), M.Cache(M.make_config(B=B, **kw))
    assert B * Hkv * blocks * gc.layout.rec_bytes > 256 << 20
    k, v, q = rnd(1, Hkv, 128 * blocks + 5, 128), rnd(1, Hkv, 128 * blocks + 5, 128), rnd(1, Hkv * g, 128)
    one.prefill(rnd(1, Hkv * g, 16, 128), k, v)
    for dst, src in ((gc.block_records(), one.block_records()), (gc.fp16_rows()[0], one.fp16_rows()[0]), (gc.fp16_rows()[1], one.fp16_rows()[1])):
        dst.view(B, Hkv, *dst.shape[1:]).copy_(src[None].expand(B, *src.shape))
    M.load_library().mixkvq_cache_set_state(gc.handle, *one.state_seq(0))
    out, lse = gc.decode_attention(q.expand(B, -1, -1).contiguous())
    ref, ref_lse = one.decode_attention(q)
    torch.cuda.synchronize()
    assert torch.equal(out, out[:1].expand_as(out)) and torch.equal(lse, lse[:1].expand_as(lse))
    # (the one sequence's sums run in another order: twice the distance of either from binary64)
    assert torch.all((out[:1].float() - ref.float()).abs() <= 2e-3 + 1e-2 * ref.float().abs())
    assert torch.all((lse[:1] - ref_lse).abs() <= 2e-3 + 1e-4 * ref_lse.abs())
    # one sequence a block shorter: the launch over different lengths reads as much, the others' outputs stay what they were
    n_quant, n_res, n_sink = one.state_seq(0)
    M.load_library().mixkvq_cache_set_state_seq(gc.handle, 5, n_quant - 128, n_res, n_sink)
    assert (B * blocks - 1) * Hkv * gc.layout.rec_bytes > 256 << 20
    ragged, ragged_lse = gc.decode_attention(q.expand(B, -1, -1).contiguous())
    M.load_library().mixkvq_cache_set_state(one.handle, n_quant - 128, n_res, n_sink)
    short, short_lse = one.decode_attention(q)
    torch.cuda.synchronize()
    assert gc.decode_path() == M.PATH_MATRIX
    want = torch.cat([ref.expand(5, -1, -1), short, ref.expand(B - 6, -1, -1)]).float()
    want_lse = torch.cat([ref_lse.expand(5, -1), short_lse, ref_lse.expand(B - 6, -1)])
    assert torch.all((ragged.float() - want).abs() <= 2e-3 + 1e-2 * want.abs())
    assert torch.all((ragged_lse - want_lse).abs() <= 2e-3 + 1e-4 * want_lse.abs())

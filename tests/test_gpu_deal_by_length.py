"""Batches whose sequences get workgroups by their lengths: the step's outputs against the same sequences in caches of
their own (which take the equal deal), over chains of one and several records, a sequence with fp16 rows only, an empty
one, sink rows, paged blocks, and several steps in a row (the merge leaves its tickets at 0)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hkv,g,lens,paged,over", [
    (1, 1, (1, 0, 33, 2049), False, dict(R=32, Gk=32, Gv=32, k4=8, k16=0)),              # far below one round of workgroups
    (8, 2, (9000, 40, 700, 2500, 0, 129), False, dict(R=32, Gk=32, Gv=32, k4=16, k16=0)),  # two records and more per wavefront
    (4, 7, (3000, 130, 64, 1500, 257), True, dict(R=128, Gk=128, Gv=128, k4=16, k16=0)),
    (4, 5, (2000, 5, 400), False, dict(R=128, Gk=32, Gv=32, k4=16, k16=8, sink=128)),
    (2, 3, (5000, 255, 513), False, dict(R=256, Gk=128, Gv=128, k4=0, k16=12, sink=96)),   # windows of up to 12 sub-units
    (1, 4, (20000, 31), False, dict(R=64, Gk=64, Gv=64, k4=16, k16=0)),                   # the ceiling of 64 workgroups
    (8, 1, (1100,) * 20 + (2200,) * 20, False, dict(R=128, Gk=128, Gv=128, k4=16, k16=0)),  # 320 pairs
])
def test_a_batch_equals_its_sequences(Hkv, g, lens, paged, over):
    import paper_2512_19206_amd as M
    assert torch.cuda.is_available(), "these tests need the GPU"
    gen = torch.Generator(device="cuda").manual_seed(len(lens) * 100 + Hkv)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda").half()
    B, R, steps = len(lens), over["R"], 3
    kw = dict(Hq=Hkv * g, Hkv=Hkv, D=128, T_max=-(-(max(lens) + steps) // R) * R, **over)
    batch = M.Cache(M.make_config(B=B, **kw))
    if paged:
        slots = B * (batch.cfg.T_max // batch.rec_tokens)
        batch.set_block_table(torch.randperm(slots, generator=gen, device="cuda").to(torch.int32).view(B, -1).contiguous())
    alone = [M.Cache(M.make_config(B=1, **kw)) for _ in range(B)]
    scale = 0.3 + 4 * torch.rand(128, generator=gen, device="cuda")
    for b, n in enumerate(lens):
        if n:
            k, v, q = (rnd(Hkv, n, 128) * scale).half(), rnd(Hkv, n, 128), rnd(Hkv * g, 16, 128)
            sel = batch.select_channels_seq(b, q, k)
            batch.quantize_append_seq(b, k, v, sel=sel)
            alone[b].select_channels_seq(0, q, k)
            alone[b].quantize_append_seq(0, k, v, sel=sel)
    for step in range(steps):
        if step == 1:      # without a token: an empty sequence stays empty only if no step has fed it
            q = rnd(B, Hkv * g, 128)
            out, lse = batch.decode_attention(q, accumulate_q=True)
            parts = [c.decode_attention(q[b:b + 1], accumulate_q=True) for b, c in enumerate(alone)]
        else:
            k, v, q = (rnd(B, Hkv, 1, 128) * scale).half(), rnd(B, Hkv, 1, 128), rnd(B, Hkv * g, 128)
            out, lse = batch.decode_step(k, v, q, accumulate_q=True)
            parts = [c.decode_step(k[b:b + 1], v[b:b + 1], q[b:b + 1], accumulate_q=True) for b, c in enumerate(alone)]
        torch.cuda.synchronize()
        assert batch.decode_path() == 1
        # both sides are within 1e-3 + 5e-3 |x| of binary64 attention over the same records: twice that between them
        ref, ref_lse = torch.cat([p[0] for p in parts]).float(), torch.cat([p[1] for p in parts])
        assert torch.all((out.float() - ref).abs() <= 2e-3 + 1e-2 * ref.abs()), step
        assert torch.all((lse - ref_lse).abs() <= 2e-3 + 1e-4 * ref_lse.abs()), step
        acc, cnt = batch.query_accumulator()
        for b, c in enumerate(alone):
            a1, c1 = c.query_accumulator()
            assert torch.equal(acc[b * Hkv:(b + 1) * Hkv], a1) and torch.equal(cnt[b * Hkv:(b + 1) * Hkv], c1), (step, b)
            assert batch.state_seq(b) == c.state_seq(0)
            n = sum(c.state_seq(0)[1:])
            for x, y in zip(batch.fp16_rows(), c.fp16_rows()):
                assert torch.equal(x[b * Hkv:(b + 1) * Hkv, :n], y[:, :n]), (step, b)


@pytest.mark.parametrize("Hkv,g,lens,paged,over", [
    (2, 2, (4500, 40, 700, 1250, 129), False, dict(R=32, Gk=32, Gv=32, k4=16, k16=0)),
    (4, 7, (2900, 130, 64, 1500, 257), True, dict(R=128, Gk=128, Gv=128, k4=16, k16=0)),
    (2, 5, (2000, 5, 400), False, dict(R=128, Gk=32, Gv=32, k4=16, k16=8, sink=128)),
    (1, 3, (5000, 255, 513), False, dict(R=256, Gk=128, Gv=128, k4=0, k16=12, sink=96)),
])
def test_a_batch_against_the_oracle(Hkv, g, lens, paged, over):
    """The same kind of batch at the plain bar: every sequence against an oracle cache of its own."""
    import gpu_common as H
    import paper_2512_19206_amd as M
    from oracle import mixkvq_oracle as O
    rng = np.random.default_rng(8000 + Hkv * 10 + g)
    B, R = len(lens), over["R"]
    kw = dict(Hq=Hkv * g, Hkv=Hkv, D=128, T_max=-(-(max(lens) + 3) // R) * R, **over)
    gc = M.Cache(M.make_config(B=B, **kw))
    if paged:
        slots = B * (gc.cfg.T_max // gc.rec_tokens)
        gc.set_block_table(H.dev(rng.permutation(slots).astype(np.int32)).view(B, -1).contiguous())
    scale, ocs = rng.uniform(0.3, 4.0, 128), []
    draw = lambda *s: rng.standard_normal(s).astype(np.float16)
    for b, n in enumerate(lens):
        K, V, Q = (draw(1, Hkv, n, 128) * scale).astype(np.float16), draw(1, Hkv, n, 128), draw(1, Hkv * g, 16, 128)
        ocs.append(O.OracleCache(O.OracleConfig(B=1, **kw)))
        ref = ocs[-1].select_channels(Q, K)
        sel = gc.select_channels_seq(b, H.dev(Q[0]), H.dev(K[0]))
        assert np.array_equal(sel.cpu().numpy(), ref[0])
        gc.quantize_append_seq(b, H.dev(K[0]), H.dev(V[0]), sel=sel)
        ocs[-1].append(K, V, ref)
    for _ in range(2):
        k, v, q = (draw(B, Hkv, 1, 128) * scale).astype(np.float16), draw(B, Hkv, 1, 128), draw(B, Hkv * g, 128)
        out, lse = gc.decode_step(H.dev(k), H.dev(v), H.dev(q), accumulate_q=True)
        torch.cuda.synchronize()
        assert gc.decode_path() == M.PATH_MATRIX
        out, lse = out.float().cpu().numpy(), lse.cpu().numpy()
        for b, oc in enumerate(ocs):
            oc.append(k[b:b + 1], v[b:b + 1])
            ro, rl = oc.decode_attention(q[b:b + 1], accumulate_q=True)
            assert np.all(np.abs(out[b] - ro[0]) <= H.ATOL + H.RTOL * np.abs(ro[0])), b
            assert np.all(np.abs(lse[b] - rl[0]) <= H.LSE_ATOL + 1e-4 * np.abs(rl[0])), b


def test_an_empty_sequence_among_long_ones():
    import paper_2512_19206_amd as M
    gen = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda").half()
    gc = M.Cache(M.make_config(B=3, Hq=8, Hkv=4, D=128, T_max=2048, Gk=128, Gv=128, R=128, k4=16, k16=0))
    for b, n in ((0, 1500), (2, 200)):
        k, v, q = rnd(4, n, 128), rnd(4, n, 128), rnd(8, 16, 128)
        gc.quantize_append_seq(b, k, v, sel=gc.select_channels_seq(b, q, k))
    for _ in range(2):
        out, lse = gc.decode_attention(rnd(3, 8, 128))
        torch.cuda.synchronize()
        assert torch.isfinite(out).all() and torch.all(out[1] == 0) and torch.all(lse[1] == -np.inf)
        assert torch.isfinite(lse[0]).all() and torch.isfinite(lse[2]).all()

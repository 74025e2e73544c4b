"""Attention of batched passes at the edges of the threshold kernel's blocks (16 or 32 query rows), parts (512, 1024 or 2048
keys) and row-length classes (256, 1024, 2048, 4096 keys), against the definition in 64 bits on the same bf16 q, K, V.

Tolerance: probabilities are split into two bf16 halves (2^-17) and sums are fp32, far below 1e-4 of a row's largest value,
unless two scores within the 32-bit rounding of a dot product of 64 or 128 terms (2^-22 of the row's scale) lie across the
threshold; then the row moves by at most that key's weight, the smallest of at least 15 kept ones. Asserted: median row within
1e-4, at most 1 % of rows over 1e-3, none over 1/15."""
import pytest
import torch

from paper_2605_10875_amd import sol, synth

pytestmark = pytest.mark.gpu

TABLE = synth.action_table((0.0625, 0.125, 0.5, 0.9, 1.0), (0.0,), (16,))


@pytest.mark.parametrize("last", [256, 257, 272, 511, 513, 1023, 1024, 1025, 1041, 1281, 2047, 2048, 2049, 3073, 4095, 4096])
@pytest.mark.parametrize("dh,Hq,Hkv,T", [(64, 8, 2, 16), (64, 4, 4, 33), (128, 4, 1, 31), (128, 4, 2, 47)])
def test_attention_at_the_edges_of_blocks_and_parts(dh, Hq, Hkv, T, last):
    g = torch.Generator(device="cuda").manual_seed(last * 5 + T)
    shape = synth.ModelShape(d_model=Hq * dh, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=dh, d_ff=256, n_layers=1, vocab=100)
    n_seq, L = 2, last                                             # the second sequence ends 9 keys earlier
    ends = (last, last - 9)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()  # noqa: E731
    q, kc, vc = rnd(n_seq, T, Hq * dh), rnd(n_seq, Hkv, L, dh), rnd(n_seq, Hkv, L, dh)
    ids = torch.randint(0, len(TABLE), (n_seq, T), generator=g, device="cuda", dtype=torch.int32)
    pos0 = torch.tensor([e - T for e in ends], dtype=torch.int32, device="cuda")
    ctx = sol.Sol(shape, TABLE, dtype=sol.BF16, max_positions=L)
    o = ctx.test_attention_stage(q, ids, kc, vc, pos0=pos0)
    assert ctx.device_status() == sol.OK
    ctx.close()
    keep = torch.tensor([[a[0], a[1]] for a in TABLE], device="cuda")[ids.long()]
    err = []
    for s in range(n_seq):
        pos = int(pos0[s]) + torch.arange(T, device="cuda")
        n = pos + 1
        budget = torch.minimum(-(-keep[s, :, 0] * n // keep[s, :, 1]), n)
        causal = torch.arange(L, device="cuda")[None] <= pos[:, None]
        for h in range(Hq):
            k, v = kc[s, h // (Hq // Hkv)].double(), vc[s, h // (Hq // Hkv)].double()
            x = (q[s, :, h * dh:(h + 1) * dh].double() @ k.t().contiguous() / dh ** 0.5).masked_fill(~causal, -torch.inf)
            kth = x.sort(-1, descending=True).values.gather(1, (budget - 1)[:, None])
            want = torch.softmax(x.masked_fill(x < kth, -torch.inf), -1) @ v
            got = o[s, :, h * dh:(h + 1) * dh].double()
            err.append((got - want).abs().amax(1) / want.abs().amax(1))
    err = torch.cat(err)
    print(f"row error median {err.median():.1e} max {err.max():.1e}, over 1e-3: {(err > 1e-3).double().mean():.4f}")
    assert err.median() < 1e-4 and (err > 1e-3).double().mean() <= 0.01 and err.max() < 1 / 15


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("rule", [{}, sol.PAPER_PRESET], ids=["topk", "pages"])
def test_a_sequence_has_the_bits_it_has_among_others(dh, rule):
    """1, 25 and 300 sequences of 200 rows: one block of 16 rows per workgroup, pairs of them, pairs of blocks of 32 rows"""
    g = torch.Generator(device="cuda").manual_seed(dh)
    T, Hq, Hkv = 200, 16, 4
    shape = synth.ModelShape(d_model=256, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=dh, d_ff=256, n_layers=1, vocab=100)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()  # noqa: E731
    q, kc, vc = rnd(1, T, Hq * dh), rnd(1, Hkv, T, dh), rnd(1, Hkv, T, dh)
    ids = torch.randint(0, len(TABLE), (1, T), generator=g, device="cuda", dtype=torch.int32)
    ctx = sol.Sol(shape, TABLE, dtype=sol.BF16, max_positions=T, **rule)
    want = ctx.test_attention_stage(q, ids, kc, vc)
    for n in (25, 300):
        many = lambda t: t.expand(n, *t.shape[1:]).contiguous()  # noqa: E731
        got = ctx.test_attention_stage(many(q), many(ids), many(kc), many(vc))
        assert torch.equal(got, many(want)), n
    assert ctx.device_status() == sol.OK
    ctx.close()


@pytest.mark.parametrize("T", [17, 33, 64])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("rule", [{}, sol.PAPER_PRESET], ids=["topk", "pages"])
def test_rows_behind_a_past_have_the_bits_they_have_among_others(dh, rule, T):
    """1, 40, 80 and 150 sequences of two to four 16-row blocks behind 300 keys: every way the blocks are dealt to workgroups"""
    g = torch.Generator(device="cuda").manual_seed(dh + T)
    past, Hq, Hkv = 300, 16, 4
    shape = synth.ModelShape(d_model=256, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=dh, d_ff=256, n_layers=1, vocab=100)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()  # noqa: E731
    q, kc, vc = rnd(1, T, Hq * dh), rnd(1, Hkv, past + T, dh), rnd(1, Hkv, past + T, dh)
    ids = torch.randint(0, len(TABLE), (1, T), generator=g, device="cuda", dtype=torch.int32)
    pos0 = torch.full((1,), past, dtype=torch.int32, device="cuda")
    ctx = sol.Sol(shape, TABLE, dtype=sol.BF16, max_positions=past + T, **rule)
    want = ctx.test_attention_stage(q, ids, kc, vc, pos0=pos0)
    for n in (40, 80, 150):
        many = lambda t: t.expand(n, *t.shape[1:]).contiguous()  # noqa: E731
        got = ctx.test_attention_stage(many(q), many(ids), many(kc), many(vc), pos0=many(pos0))
        assert torch.equal(got, many(want)), n
    assert ctx.device_status() == sol.OK
    ctx.close()


def _attend64(q, k, v, pos, budget):
    """q [T][dh] at positions pos, k and v [L][dh]: softmax over the `budget` largest causal scores, in 64 bits"""
    x = q.double() @ k.double().t().contiguous() / q.shape[-1] ** 0.5
    x = x.masked_fill(torch.arange(k.shape[0], device="cuda")[None] > pos[:, None], -torch.inf)
    kth = x.sort(-1, descending=True).values.gather(1, (budget - 1)[:, None])
    return torch.softmax(x.masked_fill(x < kth, -torch.inf), -1) @ v.double()


@pytest.mark.parametrize("last", [16, 17, 31, 64, 255, 256, 257, 509, 513, 1000, 1023, 1024])
@pytest.mark.parametrize("dh,Hq,Hkv,T", [(64, 4, 2, 16), (128, 4, 4, 33)])
def test_fp32_attention_of_blocks_of_rows(dh, Hq, Hkv, T, last):
    """fp32 q, K, V: scores in four chains of dh / 4 products, outputs in chains of n / 16, trees above: 2^-24 times a few,
    times the score's size in the exponent (up to about 16): under 1e-5 of a row's largest value; a swapped near-tie
    (2^-21 of the scores' scale apart) moves a row by a kept key's weight: at most 1 % of rows."""
    T = min(T, last)
    g = torch.Generator(device="cuda").manual_seed(last * 3 + dh)
    shape = synth.ModelShape(d_model=Hq * dh, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=dh, d_ff=256, n_layers=1, vocab=100)
    ends = (last, max(T, last - 9))
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    q, kc, vc = rnd(2, T, Hq * dh), rnd(2, Hkv, last, dh), rnd(2, Hkv, last, dh)
    ids = torch.randint(0, len(TABLE), (2, T), generator=g, device="cuda", dtype=torch.int32)
    pos0 = torch.tensor([e - T for e in ends], dtype=torch.int32, device="cuda")
    ctx = sol.Sol(shape, TABLE, dtype=sol.F32, max_positions=last)
    o = ctx.test_attention_stage(q, ids, kc, vc, pos0=pos0)
    keep = torch.tensor([[a[0], a[1]] for a in TABLE], device="cuda")[ids.long()]
    err = []
    for s in range(2):
        pos = int(pos0[s]) + torch.arange(T, device="cuda")
        budget = torch.minimum(-(-keep[s, :, 0] * (pos + 1) // keep[s, :, 1]), pos + 1)
        for h in range(Hq):
            c = slice(h * dh, (h + 1) * dh)
            want = _attend64(q[s, :, c], kc[s, h // (Hq // Hkv)], vc[s, h // (Hq // Hkv)], pos, budget)
            err.append((o[s, :, c].double() - want).abs().amax(1) / want.abs().amax(1))
    err = torch.cat(err)
    assert (err > 1e-5).double().mean() <= 0.01 and err.median() < 2e-6, (err.max(), err.median())
    # the kernel that takes a workgroup per row (caches of more than 1024 positions) makes every sum in the same order
    pad = lambda t: torch.cat([t, t.new_zeros((2, Hkv, 1100 - last, dh))], 2).contiguous()  # noqa: E731
    wide = sol.Sol(shape, TABLE, dtype=sol.F32, max_positions=1100)
    assert torch.equal(o, wide.test_attention_stage(q, ids, pad(kc), pad(vc), pos0=pos0))
    wide.close()
    # what a row does not see does not reach it: the V row of the last position, under the causal mask of all rows but the last
    vc[0, :, -1] = torch.inf
    clean = vc.clone()
    clean[0, :, -1] = 0.0
    a, b = (ctx.test_attention_stage(q, ids, kc, t, pos0=pos0) for t in (vc, clean))
    assert torch.isfinite(a[0, :-1]).all() and (a[0, :-1] - b[0, :-1]).abs().max() < 1e-5 * b.abs().max()
    assert torch.equal(a[1], b[1])
    assert ctx.device_status() == sol.OK
    ctx.close()


@pytest.mark.parametrize("last", [16, 17, 31, 64, 255])
@pytest.mark.parametrize("dh,Hq,Hkv,T", [(64, 4, 1, 16), (128, 8, 2, 33)])
def test_fp32_attention_of_blocks_of_short_rows(dh, Hq, Hkv, T, last):
    """as above for short rows, at the heads per group (four) where no pass of 16 rows or more goes to the kernel per row"""
    test_fp32_attention_of_blocks_of_rows(dh, Hq, Hkv, T, last)

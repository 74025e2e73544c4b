"""The bf16 GEMM's smaller tiles: every tile the row rule can take, at the edges of its range, against the fp64 product;
and the same rows in products of other heights, which take other tiles, the same sequences in layer calls of other sizes, of whole
tiles and not, and beside a sequence that does not fit: equal bit for bit."""
import pytest
import torch

from paper_2605_10875_amd import sol, synth

pytestmark = pytest.mark.gpu


def _mats(M, N, K, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16),
            torch.randn((N, K), generator=g, device="cuda").to(torch.bfloat16))


# 256 CUs: 64 x 64 tiles up to 64 tiles of 128 x 128, then 128 x 64, 128 x 128, 128 x 256, 256 x 256 and mixtures
@pytest.mark.parametrize("M", [1, 63, 64, 65, 127, 129, 449, 512, 513, 1023, 1025, 1281, 2049, 4097, 4361])
@pytest.mark.parametrize("N,K", [(2048, 128), (4096, 384)])
def test_rows_against_the_product(M, N, K):
    a, w = _mats(M, N, K, M + N)
    c = sol.gemm(a, w).double()
    # products of bf16 values are exact in fp32; a sum of K of them in any order: K 2^-24 of the sum of magnitudes at most
    bound = K * 2.0 ** -24 * (a.double().abs() @ w.double().abs().t())
    assert bool(((c - a.double() @ w.double().t()).abs() <= bound).all())


@pytest.mark.parametrize("M", [1, 65, 200, 512, 700, 1536, 2304])
def test_the_tile_does_not_show(M):
    a, w = _mats(8192, 2048, 512, 7)
    assert torch.equal(sol.gemm(a[:M].contiguous(), w), sol.gemm(a, w)[:M])


@pytest.mark.parametrize("shape", [synth.LLAMA_1B, synth.LLAMA_8B], ids=["head64", "head128"])
@pytest.mark.parametrize("rule", [{}, sol.PAPER_PRESET], ids=["topk", "pages"])
def test_a_layer_row_does_not_depend_on_the_batch(shape, rule):
    """One sequence of 160 tokens alone, with 2, 6, 7, 12, 15 and 29 others: small tiles, mixtures and whole rounds of large ones
    in all four fused epilogues, with the sequences at different cache positions."""
    T, n = 160, 30
    g = torch.Generator(device="cuda").manual_seed(3)

    def rnd(*sz):
        return torch.randn(sz, generator=g, device="cuda")

    d, nq, nkv, ff = shape.d_model, shape.n_q_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim, shape.d_ff
    w = {k: (0.02 * rnd(*sz)).to(torch.bfloat16) for k, sz in dict(
        wq=(nq, d), wk=(nkv, d), wv=(nkv, d), wo=(d, nq), w_gate=(ff, d), w_up=(ff, d), w_down=(d, ff)).items()}
    w["w_in_norm"], w["w_post_norm"] = ((1 + 0.1 * rnd(d)).to(torch.bfloat16) for _ in range(2))
    x = rnd(n, T, d).to(torch.bfloat16)
    ids = torch.randint(0, len(synth.TABLE_C2), (n, T), generator=g, device="cuda", dtype=torch.int32)
    pos0 = torch.arange(n, device="cuda", dtype=torch.int32) * 3 + 5
    L = 300
    kc, vc = (rnd(n, shape.n_kv_heads, L, shape.head_dim).to(torch.bfloat16) for _ in range(2))
    ctx = sol.Sol(shape, synth.TABLE_C2, max_positions=L, **rule)
    outs = []
    for m in (1, 3, 7, 8, 13, 16, n):
        k, v = kc[:m].clone(), vc[:m].clone()
        y = ctx.layer_forward(w, x[:m].contiguous(), ids[:m].contiguous(), k, v, pos0=pos0[:m].contiguous())
        outs.append((y[0], k[0], v[0]))
    assert ctx.device_status() == sol.OK
    for o in outs[1:]:
        assert all(torch.equal(p, q) for p, q in zip(o, outs[0]))


def test_rotated_rows_do_not_depend_on_the_rows_in_the_call():
    """32 sequences of 136 tokens in one call (17 whole tiles of 256 rows), each alone (one ragged tile), and among one that
    does not fit its cache, also in the next call before the status is read. 4.5 million keys in each half of the heads: a
    last bit of the fp32 rotation that differs changes some sixty of their bf16 values."""
    shape, T, n = synth.ModelShape(512, 32, 32, 64, 256), 136, 32
    g = torch.Generator(device="cuda").manual_seed(4)

    def rnd(*sz):
        return torch.randn(sz, generator=g, device="cuda").to(torch.bfloat16)

    w = dict(wq=rnd(2048, 512), wk=rnd(2048, 512), wv=rnd(2048, 512), wo=rnd(512, 2048), w_gate=rnd(256, 512), w_up=rnd(256, 512),
             w_down=rnd(512, 256), w_in_norm=rnd(512), w_post_norm=rnd(512))
    x, ids = rnd(n, T, 512), torch.zeros((n, T), dtype=torch.int32, device="cuda")
    ctx = sol.Sol(shape, [synth.DENSE_ACTION], max_positions=T)

    def layer(rows, pos0=None):
        k, v = (torch.zeros((x[rows].shape[0], 32, T, 64), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        return ctx.layer_forward(w, x[rows].contiguous(), ids[rows].contiguous(), k, v, pos0=pos0), k, v

    whole = layer(slice(0, n))
    assert ctx.device_status() == sol.OK
    for i in range(n):
        assert all(torch.equal(a[0], b[i]) for a, b in zip(layer(slice(i, i + 1)), whole)), i
    pos0 = torch.zeros(n, dtype=torch.int32, device="cuda")
    pos0[5] = 1
    rest = [i for i in range(n) if i != 5]
    flagged, after = layer(slice(0, n), pos0), layer(slice(0, n), torch.zeros_like(pos0))
    assert ctx.device_status() == sol.ERR_CACHE_OVERFLOW
    for a, b, c in zip(flagged, after, whole):
        assert torch.equal(a[rest], c[rest]) and torch.equal(b, c)


def test_rows_of_a_wide_layer_do_not_depend_on_the_call():
    """One sequence of 100 tokens alone and with 1, 2, 3 and 15 others: the 128 x 64 and 128 x 128 tiles of the fused epilogues (gate / up
    at 100 and 200 rows, q/k/v at 400 and 1600)."""
    shape, T, n = synth.ModelShape(512, 32, 8, 64, 8192), 100, 16
    g = torch.Generator(device="cuda").manual_seed(6)

    def rnd(*sz):
        return torch.randn(sz, generator=g, device="cuda").to(torch.bfloat16)

    w = dict(wq=rnd(2048, 512), wk=rnd(512, 512), wv=rnd(512, 512), wo=rnd(512, 2048), w_gate=rnd(8192, 512), w_up=rnd(8192, 512),
             w_down=rnd(512, 8192), w_in_norm=rnd(512), w_post_norm=rnd(512))
    x, ids = rnd(n, T, 512), torch.zeros((n, T), dtype=torch.int32, device="cuda")
    ctx = sol.Sol(shape, [synth.DENSE_ACTION], max_positions=T)
    outs = []
    for m in (1, 2, 3, 4, n):
        k, v = (torch.zeros((m, 8, T, 64), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        outs.append((ctx.layer_forward(w, x[:m].contiguous(), ids[:m].contiguous(), k, v)[0], k[0], v[0]))
    assert ctx.device_status() == sol.OK
    for o in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(o, outs[0]))

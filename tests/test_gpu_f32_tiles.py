"""fp32 linear maps: a sequence's rows in calls of other sizes, which take other tiles (32 x 32; 64 x 64 with two slices of K per
barrier and with one; 128 x 128), with K of an even and an odd number of slices: equal bit for bit, since every tile adds k in order."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import host
from paper_2605_10875_amd import sol, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [synth.ModelShape(1056, 4, 2, 64, 2112), synth.ModelShape(2048, 8, 2, 64, 8192), synth.ModelShape(64, 16, 16, 64, 4128)],
                         ids=["odd_slices", "wide", "one_slice_pair"])
def test_rows_do_not_depend_on_the_call(shape):
    T, n = 70, 30
    g = torch.Generator(device="cuda").manual_seed(5)

    def rnd(*sz):
        return torch.randn(sz, generator=g, device="cuda")

    d, nq, nkv, ff = shape.d_model, shape.n_q_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim, shape.d_ff
    w = {k: 0.02 * rnd(*sz) for k, sz in dict(wq=(nq, d), wk=(nkv, d), wv=(nkv, d), wo=(d, nq), w_gate=(ff, d), w_up=(ff, d),
                                              w_down=(d, ff)).items()}
    w["w_in_norm"], w["w_post_norm"] = 1 + 0.1 * rnd(d), 1 + 0.1 * rnd(d)
    x, ids = rnd(n, T, d), torch.zeros((n, T), dtype=torch.int32, device="cuda")
    ctx = sol.Sol(shape, [synth.DENSE_ACTION], dtype=sol.F32, max_positions=T)
    outs = []
    for m in (1, 2, 4, 9, n):
        k, v = (torch.zeros((m, shape.n_kv_heads, T, shape.head_dim), device="cuda") for _ in range(2))
        outs.append((ctx.layer_forward(w, x[:m].contiguous(), ids[:m].contiguous(), k, v)[0], k[0], v[0]))
    assert ctx.device_status() == sol.OK
    for o in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(o, outs[0]))
    # v of the first rows against 64 bits: chains of d fp32 sums
    h = x[0].double() * torch.rsqrt(x[0].double().square().mean(-1, keepdim=True) + shape.rms_eps) * w["w_in_norm"].double()
    ref = (h @ w["wv"].double().t()).view(T, shape.n_kv_heads, shape.head_dim).transpose(0, 1)
    bound = (d + 16) * 2.0 ** -23 * (h.abs() @ w["wv"].double().abs().t()).view(T, shape.n_kv_heads, shape.head_dim).transpose(0, 1)
    assert bool(((outs[0][2].double() - ref).abs() <= bound).all())


def _tile(rows, cols, k, cus, pairs=False):
    """The library's rule: the tile that a product takes, "64/2" and "64/1" being the 64 x 64 one with two slices of K per barrier
    and one; pairs: rotary or SiLU * up at its end."""
    r32, r64, r128 = (-(-(-(-rows // b) * -(-cols // b)) // cus) for b in (32, 64, 128))
    c32, c64, c128 = 10 + 11.6 * r32, 47 if r64 == 1 else 2 + 35 * r64, 147 if r128 == 1 else 126 * (r128 + r128 % 2)
    c64 += 10 if r64 <= 2 and (pairs or k < 1024) else 0
    if c128 <= c64 and c128 <= c32:
        return "128"
    if c64 > c32:
        return "32"
    return "64/2" if r64 in (2, 4) and k % 64 == 0 else "64/1"


# (rows of 2 sequences) q/k/v, gate / up, o and down; each beside its first 30 tokens alone, in 32 x 32 tiles
@pytest.mark.parametrize("shape,T,tiles", [
    (synth.ModelShape(2048, 32, 8, 64, 8192), 509, ("64/1", "128", "64/2", "64/2")),       # many steps of the two-slice pipeline
    (synth.ModelShape(2048, 64, 32, 32, 4096), 500, ("64/2", "128", "64/2", "64/2")),      # four rounds; two
    (synth.ModelShape(2048, 33, 33, 32, 1056), 500, ("64/2", "64/1", "64/1", "64/1")),     # two rounds, K an odd number of slices (o, down)
    (synth.ModelShape(1056, 32, 8, 64, 16384), 1000, ("64/1", "128", "64/1", "64/1")),      # 128 x 128 with K an odd number of slices
])
def test_every_tile_gives_the_small_calls_bits(shape, T, tiles):
    n, few, cus = 2, 30, torch.cuda.get_device_properties(0).multi_processor_count
    d, nq, nkv, ff = shape.d_model, shape.n_q_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim, shape.d_ff
    maps = ((nq + 2 * nkv, d, cus, True), (2 * ff, d, cus, True), (d, nq, cus), (d, ff, cus))
    if cus == 256:                                    # (other dies have other rounds)
        assert tuple(_tile(n * T, *m) for m in maps) == tiles
        assert all(_tile(few, *m) == "32" for m in maps)
    weights = synth.layer_weights(shape, 31, std=0.05)
    w = {k: torch.from_numpy(np.ascontiguousarray(a)).cuda() for k, a in weights.items()}
    g = torch.Generator(device="cuda").manual_seed(8)
    x, ids = torch.randn((n, T, d), generator=g, device="cuda"), torch.zeros((n, T), dtype=torch.int32, device="cuda")
    ctx = sol.Sol(shape, [synth.DENSE_ACTION], dtype=sol.F32, max_positions=T)

    def layer(seqs, t):
        k, v = (torch.zeros((seqs, shape.n_kv_heads, t, shape.head_dim), device="cuda") for _ in range(2))
        y = ctx.layer_forward(w, x[:seqs, :t].contiguous(), ids[:seqs, :t].contiguous(), k, v)
        return y[0, :few], k[0, :, :few], v[0, :, :few]

    large, small = layer(n, T), layer(1, few)
    assert ctx.device_status() == sol.OK
    for a, b in zip(large, small):
        assert torch.equal(a, b)
    ko, vo = (np.zeros((1, shape.n_kv_heads, few, shape.head_dim), np.float32) for _ in range(2))
    ref, _ = oracle.layer_forward(oracle.make_cfg(shape), oracle.make_table([synth.DENSE_ACTION]), weights, host(x[:1, :few]),
                                  np.zeros((1, few), np.int32), ko, vo)
    # sums of at most 16384 fp32 products in chains: 16384 * 2^-24 = 1e-3 of the largest, were all errors of one sign
    for got, want in zip(small, (ref[0], ko[0], vo[0])):
        assert np.abs(host(got) - want).max() <= 1e-4 * max(1.0, np.abs(want).max())

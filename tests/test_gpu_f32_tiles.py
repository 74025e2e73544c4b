"""fp32 linear maps: a sequence's rows in calls of other sizes, which take other tiles (32 x 32; 64 x 64 with two slices of K per
barrier and with one; 128 x 128), with K of an even and an odd number of slices: equal bit for bit, since every tile adds k in order."""
import pytest
import torch

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

"""Layers of one row (the linear maps whose waves finish their sums) and of a few more (the K-split kernel), against the
oracle under non-quantising actions: sequences and tokens per sequence, widths of one and of several chunks of K with a
short last one, the page preset's MLP path (pruning at the MLP input, quantiser on the output off), both head sizes; and a
row alone against the same row among others, bit for bit."""
import numpy as np
import pytest
import torch

from gpu_util import check_rows, dev, dev_weights, host
import oracle
from paper_2605_10875_amd import sol, synth

pytestmark = pytest.mark.gpu

TABLE = synth.action_table((0.25, 0.5, 1.0), (0.0, 0.5), (16,))


@pytest.mark.parametrize("opts", [{}, dict(prune_site=1, quant_sites=sol.QS_MLP_OUT)], ids=["default", "mlp_in"])
@pytest.mark.parametrize("shape", [synth.ModelShape(512, 8, 2, 64, 2560), synth.ModelShape(2560, 4, 1, 128, 1024)],
                         ids=["head64", "head128"])
@pytest.mark.parametrize("n_seq,T", [(1, 1), (2, 1), (1, 3)])
def test_layer_of_few_rows(n_seq, T, shape, opts):
    L = 40
    w = synth.layer_weights(shape, 11, bf16=True)
    x = synth.hidden_states(n_seq, T, shape.d_model, 12, bf16=True)
    ids = synth.iid_actions(len(TABLE), (n_seq, T), 13)
    pos0 = (7 * np.arange(n_seq) % (L - T)).astype(np.int32)
    kc, vc = synth.kv_cache(n_seq, shape.n_kv_heads, L, shape.head_dim, 14, bf16=True)
    ko, vo = kc.copy(), vc.copy()
    ref, _ = oracle.layer_forward(oracle.make_cfg(shape, act_bf16=True, **opts), oracle.make_table(TABLE), w, x, ids, ko, vo, pos0=pos0)
    ctx = sol.Sol(shape, TABLE, max_positions=L, **opts)
    kd, vd = dev(kc, sol.BF16), dev(vc, sol.BF16)
    out = ctx.layer_forward(dev_weights(w, sol.BF16), dev(x, sol.BF16), dev(ids), kd, vd, pos0=dev(pos0))
    assert ctx.device_status() == sol.OK
    # the contract for rows of non-quantising actions
    check_rows(host(out), ref, 2e-2, 2e-2, 0.0, "layer output", median=1e-2)
    check_rows(host(kd), ko, 2e-2, 2e-2, 0.0, "K cache")
    check_rows(host(vd), vo, 2e-2, 2e-2, 0.0, "V cache")


def test_a_row_that_does_not_fit_is_skipped_and_flagged():
    shape, L = synth.ModelShape(512, 8, 2, 64, 1024), 16
    w = dev_weights(synth.layer_weights(shape, 1, bf16=True), sol.BF16)
    x = dev(synth.hidden_states(1, 1, 512, 2, bf16=True), sol.BF16)
    ids = torch.zeros((1, 1), dtype=torch.int32, device="cuda")
    kc, vc = (dev(t, sol.BF16) for t in synth.kv_cache(1, 2, L, 64, 3, bf16=True))
    before = kc.clone(), vc.clone()
    ctx = sol.Sol(shape, TABLE, max_positions=L)
    ctx.layer_forward(w, x, ids, kc, vc, pos0=torch.tensor([L], dtype=torch.int32, device="cuda"))
    assert ctx.device_status() == sol.ERR_CACHE_OVERFLOW
    assert torch.equal(kc, before[0]) and torch.equal(vc, before[1])
    ctx.layer_forward(w, x, ids, kc, vc, pos0=torch.tensor([3], dtype=torch.int32, device="cuda"))
    assert ctx.device_status() == sol.OK
    for t, b in ((kc, before[0]), (vc, before[1])):
        assert not torch.equal(t[0, :, 3], b[0, :, 3])
        assert torch.equal(t[0, :, :3], b[0, :, :3]) and torch.equal(t[0, :, 4:], b[0, :, 4:])


# widths whose maps split K in 4, 16 and 32; in 10 and 20 (no powers of two); in 2 and in more than a wave takes (K-split kernel)
@pytest.mark.parametrize("opts", [{}, dict(prune_site=1, quant_sites=sol.QS_MLP_OUT)], ids=["default", "mlp_in"])
@pytest.mark.parametrize("shape", [synth.LLAMA_1B, synth.ModelShape(2560, 20, 4, 128, 1280), synth.ModelShape(1024, 4, 1, 64, 14336)],
                         ids=["1b", "odd_splits", "wide"])
def test_a_row_alone_has_the_bits_it_has_among_others(shape, opts):
    L, n = 40, 5
    g = torch.Generator(device="cuda").manual_seed(shape.d_ff)

    def rnd(*size, scale=1.0):
        return torch.randn(size, generator=g, device="cuda").mul_(scale).to(torch.bfloat16)

    d, nq, nkv, ff = shape.d_model, shape.n_q_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim, shape.d_ff
    w = {k: rnd(*size, scale=0.02) for k, size in dict(wq=(nq, d), wk=(nkv, d), wv=(nkv, d), wo=(d, nq), w_gate=(ff, d),
                                                       w_up=(ff, d), w_down=(d, ff)).items()}
    w["w_in_norm"], w["w_post_norm"] = rnd(d), rnd(d)
    x, kc, vc = rnd(n, 1, d), rnd(n, shape.n_kv_heads, L, shape.head_dim), rnd(n, shape.n_kv_heads, L, shape.head_dim)
    ids = torch.arange(n, dtype=torch.int32, device="cuda").view(n, 1) % len(TABLE)
    pos0 = 7 * torch.arange(n, dtype=torch.int32, device="cuda")
    ctx = sol.Sol(shape, TABLE, max_positions=L, **opts)

    def layer(rows):
        k, v = kc[rows].clone(), vc[rows].clone()
        return ctx.layer_forward(w, x[rows].clone(), ids[rows].clone(), k, v, pos0=pos0[rows].clone()), k, v

    among = {m: layer(slice(0, m)) for m in (2, n)}
    for i in range(n):
        for alone, m in ((layer(slice(i, i + 1)), m) for m in among if i < m):
            for a, b in zip(alone, among[m]):
                assert torch.equal(a[0], b[i]), (i, m)
    assert ctx.device_status() == sol.OK


# widths whose norm is done inside the maps (2048, 4096) with quantising actions: gate / up over 4, 2 and 16 splits with a last
# workgroup that is not full, q / k / v over 16, 8 and 32 splits (these take the norm's own kernel); and without quantisers there
@pytest.mark.parametrize("opts", [{}, dict(quant_sites=sol.QS_MLP_OUT)], ids=["default", "no_input_sites"])
@pytest.mark.parametrize("shape", [synth.LLAMA_1B, synth.LLAMA_8B, synth.ModelShape(2048, 8, 2, 64, 1600)], ids=["1b", "8b", "narrow"])
def test_a_row_alone_is_normalised_and_quantised_as_among_others(shape, opts, monkeypatch):
    monkeypatch.setitem(globals(), "TABLE", synth.action_table((0.5, 1.0), (0.0, 0.5), (4, 8, 16)))
    test_a_row_alone_has_the_bits_it_has_among_others(shape, opts)


# a width without the norm in the maps, one where q / k / v has 32 splits and takes the norm's own kernel, both norms inside
@pytest.mark.parametrize("shape", [synth.ModelShape(1024, 4, 1, 64, 512), synth.ModelShape(2048, 8, 2, 64, 1600), synth.LLAMA_1B],
                         ids=["1024", "narrow", "1b"])
def test_each_stage_of_a_row_alone_is_recorded_once(shape):
    d, nq, nkv, ff = shape.d_model, shape.n_q_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim, shape.d_ff
    w = {k: torch.zeros(size, dtype=torch.bfloat16, device="cuda") for k, size in dict(
        w_in_norm=(d,), wq=(nq, d), wk=(nkv, d), wv=(nkv, d), wo=(d, nq), w_post_norm=(d,), w_gate=(ff, d), w_up=(ff, d), w_down=(d, ff)).items()}
    x, cache = torch.ones((1, 1, d), dtype=torch.bfloat16, device="cuda"), torch.zeros((1, shape.n_kv_heads, 8, shape.head_dim), dtype=torch.bfloat16, device="cuda")
    one = torch.ones(1, dtype=torch.int32, device="cuda")
    ctx = sol.Sol(shape, TABLE, max_positions=8)
    ctx.profile_enable(64)
    ctx.layer_forward(w, x, one.view(1, 1), cache, cache.clone(), pos0=one)
    calls = {k: v[1] for k, v in ctx.profile_read().items()}
    assert ctx.device_status() == sol.OK
    ctx.close()
    assert calls["qkv_gemm"] == calls["gate_up_gemm"] == 1 and max(calls.values()) == 1, calls

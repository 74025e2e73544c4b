"""GPU parity of the episode pass (dense prefill once per input, K schedules of T controlled steps on top of it)
against the oracle's definition; tolerances of test_gpu_parity.py."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2605_10875_amd import sol, synth

from gpu_util import dev, dev_weights, host

pytestmark = pytest.mark.gpu

SMALL_GQA = synth.ModelShape(d_model=256, n_q_heads=8, n_kv_heads=2, head_dim=64, d_ff=768, n_layers=2, vocab=1024)


def _run(shape, table, dt, B, K, P, T, seed, **opts):
    bf = dt == sol.BF16
    layers = [synth.layer_weights(shape, seed + l, bf16=bf) for l in range(shape.n_layers)]
    head = synth.head_weights(shape, seed + 10, bf16=bf)
    rng = np.random.default_rng(seed + 11)
    prefix = rng.integers(0, shape.vocab, (B, P)).astype(np.int32)
    tokens, targets = synth.tokens_and_targets(B, T, shape.vocab, seed + 12)
    ids = synth.iid_actions(len(table), (B, K, T), seed + 13)
    o_opts = dict(opts)
    qs = o_opts.pop("quant_sites", oracle.QS_NORTHSTAR)
    ref = oracle.episode_loglik(oracle.make_cfg(shape, quant_sites=qs, act_bf16=bf, **o_opts), oracle.make_table(table),
                                table.index(synth.DENSE_ACTION), head["embed"], layers, head["w_final_norm"],
                                head["lm_head"], prefix, tokens, targets, ids)
    ctx = sol.Sol(shape, table, dtype=dt, max_positions=P + T, quant_sites=qs, **o_opts)
    nll = ctx.episode_loglik([dev_weights(w, dt) for w in layers], dev_weights(head, dt), dev(prefix), dev(tokens),
                             dev(targets), dev(ids))
    assert ctx.device_status() == sol.OK
    ctx.close()
    return host(nll), ref, ids


def test_fp32_episode_pass():
    shape = dataclasses.replace(synth.TINY, n_layers=2)
    nll, ref, _ = _run(shape, synth.TABLE_C1, sol.F32, 2, 3, 20, 6, 8000)
    err = np.abs(nll - ref)
    assert np.quantile(err, 0.95) < 1e-3 and err.max() < 2e-2, (np.quantile(err, 0.95), err.max())


WIDE_HEADS = synth.ModelShape(d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=512, n_layers=2, vocab=1024)


@pytest.mark.parametrize("shape,P,T,K", [(SMALL_GQA, 64, 16, 4), (SMALL_GQA, 128, 40, 3), (WIDE_HEADS, 64, 16, 2),
                                         (SMALL_GQA, 50, 4, 3), (SMALL_GQA, 72, 16, 2),
                                         (SMALL_GQA, 1024, 16, 3), (WIDE_HEADS, 1088, 32, 2)])   # the paper's prefix length: rows over 1024 keys
def test_bf16_episode_pass(shape, P, T, K):
    """Prefix a multiple of 64 and at least 16 steps: the schedules read the prefix caches in place (tiled kernels with
    two-segment addressing); (50, 4) and (72, 16): every schedule gets a copy (row-per-workgroup kernel for fewer than 16
    steps, tiled kernels at pos0 = P otherwise). Prefixes of 1024 and more: the threshold kernel reads the prefix keys
    from their copy in MFMA operand order and the schedule's own keys from its cache."""
    table = synth.action_table((0.125, 0.5, 1.0), (0.0, 0.75), (6, 16))
    nll, ref, ids = _run(shape, table, sol.BF16, 2, K, P, T, 8100 + T + P)
    bits = np.array([a[4] for a in table])[ids]
    err = np.abs(nll - ref)
    # a step is held to 2e-2 nats if no step of its schedule so far quantised (a flipped code in an earlier step's K/V
    # entries moves every later step of that schedule)
    # (one swapped key among the 8-10 kept keys of a short row moves its NLL by a few 1e-2: one such step in ten allowed)
    clean = np.logical_and.accumulate(bits >= 16, axis=2)
    over = int((err[clean] >= 2e-2).sum())                 # (a handful of clean steps: one such step is still one in ten)
    assert (err[clean] < 5e-2).all() and over <= max(1, 0.1 * clean.sum()) and np.median(err) < 1e-2 and err.max() < 0.5, \
        (np.median(err), err.max(), over, int(clean.sum()))


@pytest.mark.parametrize("P,T,K", [(48, 8, 3), (256, 16, 3), (256, 40, 2)])
def test_bf16_episode_pass_paper_configuration(P, T, K):
    """Pages of 16 keys, sink and window keys, pruning at the MLP input, quantiser on the MLP output. A prefix of a multiple
    of 16 pages and at least 16 steps: prefix caches and prefix page metadata read in place; (48, 8): copies."""
    table = synth.action_table((0.125, 0.5, 1.0), (0.0, 0.75), (6, 16))
    nll, ref, ids = _run(SMALL_GQA, table, sol.BF16, 1, K, P, T, 8200 + P + T, **sol.PAPER_PRESET)
    err = np.abs(nll - ref)
    assert np.median(err) < 1e-2 and err.max() < 0.5, (np.median(err), err.max())


def test_identical_schedules_give_identical_likelihoods():
    table = synth.action_table((0.25, 1.0), (0.0, 0.5), (8, 16))
    shape = SMALL_GQA
    layers = [dev_weights(synth.layer_weights(shape, 8300 + l, bf16=True), sol.BF16) for l in range(2)]
    head = dev_weights(synth.head_weights(shape, 8310, bf16=True), sol.BF16)
    rng = np.random.default_rng(8311)
    prefix = rng.integers(0, shape.vocab, (1, 32)).astype(np.int32)
    tokens, targets = synth.tokens_and_targets(1, 16, shape.vocab, 8312)
    one = synth.iid_actions(len(table), (1, 1, 16), 8313)
    ids = np.repeat(one, 5, axis=1)
    ctx = sol.Sol(shape, table, dtype=sol.BF16, max_positions=48)
    nll = host(ctx.episode_loglik(layers, head, dev(prefix), dev(tokens), dev(targets), dev(ids)))
    ctx.close()
    assert all(np.array_equal(nll[0, 0], nll[0, k]) for k in range(1, 5))


@pytest.mark.parametrize("preset,P", [("{}", 192), ("{}", 1024), ("sol.PAPER_PRESET", 256), ("dict(sol.PAPER_PRESET, page_size=4)", 64),
                                      ("dict(sol.PAPER_PRESET, page_size=64, n_sink=0)", 1024)])
def test_reading_the_prefix_in_place_equals_working_on_copies(preset, P):
    """The two layouts of the episode pass run the same arithmetic on the same values: bit-identical likelihoods, under
    the plain top-k rule and under the page rule with sink / window keys. The copying layout is forced through the
    library's test hook."""
    preset = eval(preset, {"sol": sol, "dict": dict})
    shape = synth.ModelShape(d_model=256, n_q_heads=8, n_kv_heads=2, head_dim=64, d_ff=768, n_layers=2, vocab=1024)
    table = synth.action_table((0.125, 0.5, 1.0), (0.0, 0.75), (6, 16))
    layers = [dev_weights(synth.layer_weights(shape, 8400 + l, bf16=True), sol.BF16) for l in range(2)]
    head = dev_weights(synth.head_weights(shape, 8410, bf16=True), sol.BF16)
    rng = np.random.default_rng(8411)
    prefix = rng.integers(0, shape.vocab, (3, P)).astype(np.int32)
    tokens, targets = synth.tokens_and_targets(3, 24, shape.vocab, 8412)
    ids = synth.iid_actions(len(table), (3, 5, 24), 8413)
    ctx = sol.Sol(shape, table, dtype=sol.BF16, max_positions=P + 24, **preset)
    outs, sizes = [], []
    for copies in (False, True):
        outs.append(host(ctx.episode_loglik(layers, head, dev(prefix), dev(tokens), dev(targets), dev(ids), force_copies=copies)))
        assert ctx.device_status() == sol.OK
        fn = ctx.L.sol_test_episode_copies_workspace_bytes if copies else ctx.L.sol_episode_workspace_bytes
        sizes.append(int(fn(ctx.cfg, 3, 5, P, 24)))
    ctx.close()
    assert np.isfinite(outs[0]).all() and np.array_equal(outs[0], outs[1])
    assert sizes[0] < sizes[1], sizes          # the in-place layout was the one that ran: no per-schedule prefix copies


HEADS128 = synth.ModelShape(d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=512, n_layers=1, vocab=512)
HEADS64 = synth.ModelShape(d_model=256, n_q_heads=8, n_kv_heads=2, head_dim=64, d_ff=512, n_layers=1, vocab=512)


def _in_place_equals_copies(shape, B, K, P, T, seed):
    table = synth.action_table((0.125, 0.5, 0.9, 1.0), (0.0, 0.75), (6, 16))
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").mul_(0.05).bfloat16()  # noqa: E731
    ints = lambda hi, *s: torch.randint(0, hi, s, generator=g, device="cuda", dtype=torch.int32)  # noqa: E731
    d, nq, nkv, ff = shape.d_model, shape.n_q_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim, shape.d_ff
    w = dict(w_in_norm=rnd(d) + 1, wq=rnd(nq, d), wk=rnd(nkv, d), wv=rnd(nkv, d), wo=rnd(d, nq), w_post_norm=rnd(d) + 1,
             w_gate=rnd(ff, d), w_up=rnd(ff, d), w_down=rnd(d, ff))
    head = dict(embed=rnd(shape.vocab, d), w_final_norm=rnd(d) + 1, lm_head=rnd(shape.vocab, d))
    args = ([w], head, ints(shape.vocab, B, P), ints(shape.vocab, B, T), ints(shape.vocab, B, T), ints(len(table), B, K, T))
    ctx = sol.Sol(shape, table, dtype=sol.BF16, max_positions=P + T)
    here, copies = (ctx.episode_loglik(*args, force_copies=f) for f in (False, True))
    assert ctx.device_status() == sol.OK
    small, large = (int(f(ctx.cfg, B, K, P, T)) for f in (ctx.L.sol_episode_workspace_bytes, ctx.L.sol_test_episode_copies_workspace_bytes))
    ctx.close()
    assert torch.isfinite(here).all() and torch.equal(here, copies)
    return small, large


@pytest.mark.parametrize("P,T", [(192, 24), (960, 40), (1216, 24), (1280, 17), (1984, 64), (2048, 24), (2112, 40), (4032, 33)])
@pytest.mark.parametrize("shape", [HEADS64, HEADS128], ids=["64", "128"])
def test_every_row_length_of_the_prefix_read_in_place(shape, P, T):
    """each class of the threshold kernel on a shared prefix (256, 1024, 1280, 2048 and 4096 keys), blocks of 16 rows with a
    rest: the bits of the kernels of one cache per sequence"""
    small, large = _in_place_equals_copies(shape, 2, 3, P, T, P + T)
    assert small < large                           # the in-place layout was the one that ran: no prefix copies per schedule


@pytest.mark.parametrize("P", [1216, 1984, 2112])
@pytest.mark.parametrize("shape", [HEADS64, HEADS128], ids=["64", "128"])
def test_a_prefix_whose_copy_in_operand_order_is_out_of_reach(shape, P):
    """sizes at which the schedules' own caches lie less than 2^32 bytes behind the prefix caches, but more than that behind
    the copy of the prefix keys in the matrix instruction's order (the prefix's hidden states lie between the two): the
    threshold kernel reads the prefix cache itself"""
    shape, T = dataclasses.replace(shape, d_model=4096), 17
    cfg = sol.make_cfg(shape, sol.BF16, P + T)
    B = -(-10 ** 9 // (4 * P * shape.d_model))
    hidden = 2 * 2 * B * P * shape.d_model                            # two buffers of the prefix's hidden states

    def reach(K):                                                     # both prefix caches, the steps' workspace and hidden states
        return (2 * 2 * B * shape.n_kv_heads * P * shape.head_dim + sol.workspace_bytes(cfg, sol.OP_LAYER_FORWARD, B * K, T, T)
                + 3 * 2 * B * K * T * shape.d_model)

    K = max(k for k in range(1, 200) if reach(k) < 4 * 10 ** 9)
    assert reach(K) < 0.95 * 2 ** 32 and reach(K) + hidden > 1.05 * 2 ** 32, (K, reach(K), hidden)
    small, large = _in_place_equals_copies(shape, B, K, P, T, P)
    assert small < large

"""The search for a decode row's threshold where it ends in a ranking of the few keys left in its bracket: rows that have few keys
from the start, and ties inside the bracket, beyond and within the budget, against the definition and across both kernels."""
import numpy as np
import pytest
import torch

import oracle
import test_gpu_decode_split as split
from gpu_util import dev, host
from paper_2605_10875_amd import sol, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh,L,lens,dup", [
    (64, 1536, (1, 15, 62, 63, 64, 65), 0),    # at most 64 keys, one more, two more
    (64, 1600, (63, 64, 65, 127, 128, 129), 50),
    (64, 4096, (1000, 1001, 3000, 4095), 1500),
    (128, 9216, (64, 500, 5000, 9215), 4000),
    (64, 2048, (1100, 1500, 2047), 20),        # more ties than the ranking takes: the bracket closes on one key
])
def test_rows_that_end_in_a_ranking(dh, L, lens, dup):
    split.test_attention_of_few_sequences(dh, L, lens, dup)


def _against_the_definition(dh, k, v, q, lens, table):
    """Attention of sequences of lens[s] keys beside the new one under table[s], by both kernels: the same bits; and in 64 bits."""
    B, hkv, L, _ = k.shape
    ctx = sol.Sol(synth.ModelShape(256, 4 * hkv, hkv, dh, 256), table, max_positions=L)
    ids = np.arange(B, dtype=np.int32)
    args = [dev(q, sol.BF16).view(B, 1, -1), dev(ids).view(B, 1), dev(k, sol.BF16), dev(v, sol.BF16), dev(np.array(lens, np.int32))]
    out = ctx.test_attention_stage(*args[:4], pos0=args[4])
    reps = -(-100 // (B * hkv))
    assert B * hkv <= 32 < reps * B * hkv and L >= 64 * B * hkv           # spread over workgroups; one workgroup per item
    many = [t.repeat((reps,) + (1,) * (t.dim() - 1)) for t in args]
    assert torch.equal(ctx.test_attention_stage(*many[:4], pos0=many[4])[:B].nan_to_num(7.0), out.nan_to_num(7.0))
    assert ctx.device_status() == sol.OK
    o, qh = host(out).reshape(B, 4 * hkv, dh), q.reshape(B, 4 * hkv, dh).astype(np.float64)
    for s, p in enumerate(lens):
        n, b = p + 1, oracle.budget(table[s][0], table[s][1], p + 1)
        for h in range(4 * hkv):
            with np.errstate(invalid="ignore"):
                sc = (k[s, h // 4, :n].astype(np.float64) @ qh[s, h] / np.sqrt(dh)).astype(np.float32)
            if np.isnan(sc).any():
                continue                                                   # (their place among the keys is not defined)
            if np.isinf(sc.max()):
                assert np.isnan(o[s, h]).all(), (s, h)                     # infinity minus infinity
                continue
            ref, _ = oracle.softmax_v(sc, oracle.select_keys(sc, b), v[s, h // 4, :n])
            # weights within e^3 of each other: one other key kept moves an output by some 1 / b > 2e-4 of its V row; fp32 sums are far below
            assert np.abs(o[s, h] - ref).max() <= 2e-4 * max(1.0, np.abs(ref).max()), (s, h)


@pytest.mark.parametrize("n", [2, 17, 62, 63, 64, 65, 66, 127, 128, 129])
@pytest.mark.parametrize("dup", [0, 9])
def test_every_budget_of_short_rows(n, dup):
    """Rows around the 64 keys that are ranked without a search: budgets of one key, a quarter, half and all but one."""
    rng, hkv, L = np.random.default_rng(n), 2, 1536
    table = [(1, n, 1, 1, 16), (1, 4, 1, 1, 16), (1, 2, 1, 1, 16), (n - 1, n, 1, 1, 16)]
    k = rng.standard_normal((4, hkv, L, 64)).astype(np.float32)
    if dup:
        k = k[:, :, rng.integers(0, dup, L)]
    k, v = synth.round_to_bf16(k), synth.round_to_bf16(rng.standard_normal((4, hkv, L, 64)).astype(np.float32))
    q = synth.round_to_bf16(rng.standard_normal((4, 8 * 64)).astype(np.float32))
    _against_the_definition(64, k, v, q, [n - 1] * 4, table)


def _rows(kind, n, rng):
    sign = rng.choice([-1.0, 1.0], n)
    return {
        "constant": np.full(n, 0.75), "two_values": np.where(rng.random(n) < 0.3, 0.5, -1.0),
        "one_above": np.where(np.arange(n) == n // 3, 1.0, 0.25),
        # magnitudes over 100 powers of two, and clusters far narrower than their distance: straight lines between pivots creep, so that
        # the search bisects after its twelfth round (16 to 27 rounds at 1536 to 9216 keys) before 64 keys are left
        "magnitudes": 2.0 ** -rng.uniform(0, 100, n), "both_signs": sign * 2.0 ** -rng.uniform(0, 100, n),
        "clusters": sign * (1.0 + 1e-5 * rng.standard_normal(n)),
        "outliers": np.where(rng.random(n) < 0.002, 3.0, 0.01 * rng.standard_normal(n)),
        "far_below": np.where(rng.random(n) < 0.01, -1e4, 0.1 * rng.standard_normal(n)),
        "minus_infinity": np.where(rng.random(n) < 0.6, -np.inf, 0.1 * rng.standard_normal(n)),
        "plus_infinity": np.where(rng.random(n) < 0.1, np.inf, 0.1 * rng.standard_normal(n)),
        "no_number": np.where(rng.random(n) < 0.1, np.nan, 0.1 * rng.standard_normal(n)),
    }[kind].astype(np.float32)


@pytest.mark.parametrize("n", [1536, 4096, 9216])
@pytest.mark.parametrize("kind", ["constant", "two_values", "one_above", "magnitudes", "both_signs", "clusters", "outliers", "far_below",
                                  "minus_infinity", "plus_infinity", "no_number"])
def test_rows_of_any_distribution(kind, n):
    """Scores that are far from normal, beside a sequence of normal ones, under three budgets. A key is its score in three bf16 pieces, of
    which the query makes that score again exactly."""
    rng, hkv, dh = np.random.default_rng(n), 2, 64
    table = [(1, 16, 1, 1, 16), (1, 4, 1, 1, 16), (1, 2, 1, 1, 16), (1, 4, 1, 1, 16)]
    k, v = (np.zeros((4, hkv, n, dh), np.float32) for _ in range(2))
    q = np.zeros((4, 4 * hkv, dh), np.float32)
    for s in range(4):
        for g in range(hkv):
            rest = _rows(kind, n, rng) if s < 3 else rng.standard_normal(n).astype(np.float32)
            for i in range(3):
                k[s, g, :, i] = synth.round_to_bf16(np.ldexp(rest, 8 * i).astype(np.float32))
                with np.errstate(invalid="ignore"):
                    rest = np.where(np.isfinite(rest), rest - np.ldexp(k[s, g, :, i], -8 * i), 0.0).astype(np.float32)
        for h in range(4 * hkv):
            q[s, h, :3] = (1.0, -1.0, 0.5, -0.25)[h % 4] * 8.0 * 2.0 ** np.array([0, -8, -16])
    v[...] = synth.round_to_bf16(rng.standard_normal(v.shape).astype(np.float32))
    _against_the_definition(dh, k, v, q.reshape(4, -1), [n - 1] * 4, table)

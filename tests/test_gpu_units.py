"""GPU unit parity: the selection / quantisation device code on fp32 inputs must reproduce the
oracle's integer decisions bit for bit (index sets, channel masks, quantisation codes)."""
import os

import numpy as np
import pytest
import torch

import oracle
from paper_2605_10875_amd import sol

from gpu_util import dev, host

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(__file__), "golden")


def _rows(rng, rows, n, kind):
    if kind == "normal":
        return rng.standard_normal((rows, n)).astype(np.float32)
    if kind == "ties":                      # few distinct values: ties everywhere, incl. +-0
        return (rng.integers(-3, 4, (rows, n)) * 0.5).astype(np.float32)
    if kind == "const":
        return np.full((rows, n), 1.25, np.float32)
    if kind == "wide":                      # many binades, both signs
        return (rng.standard_normal((rows, n)) * np.exp(rng.uniform(-20, 20, (rows, n)))).astype(np.float32)
    if kind == "signed0":                   # both zeros, subnormals of both signs and a few ordinary values: compared as floats
        vals = np.array([0.0, -0.0, 1e-42, -1e-42, 3e-39, -3e-39, 1.0, -1.0, 1.1754944e-38], np.float32)
        return vals[rng.integers(0, len(vals), (rows, n))]
    if kind == "heavy":                     # heavy tails plus a few outliers at the start of the row (sink keys)
        x = rng.standard_normal((rows, n)) * np.abs(rng.standard_normal((rows, n))) * 1.3
        x[:, :min(4, n)] += 6.0
        return x.astype(np.float32)
    raise ValueError(kind)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 257, 1024, 1025, 2048, 4096, 4097, 8192, 20000])
@pytest.mark.parametrize("kind", ["normal", "ties", "const", "wide", "signed0"])
def test_topk_select_bit_exact(n, kind):
    rng = np.random.default_rng(n * 7 + len(kind))
    rows = 12
    s = _rows(rng, rows, n, kind)
    n_valid = rng.integers(1, n + 1, rows).astype(np.int32)
    n_valid[0] = n
    k = np.array([rng.integers(1, nv + 1) for nv in n_valid], np.int32)
    k[0] = n
    k[1] = 1
    if rows > 2:
        k[2] = max(1, n_valid[2] - 1)
    keep = host(sol.topk_select(dev(s), dev(n_valid), dev(k))).astype(np.uint8)
    for r in range(rows):
        want = np.zeros(n, np.uint8)
        want[:n_valid[r]] = oracle.select_keys(s[r, :n_valid[r]], int(k[r]))
        assert np.array_equal(keep[r], want), (r, n_valid[r], k[r])
        assert keep[r].sum() == k[r]


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 700, 1024, 1025, 1280, 1281, 2048, 2049, 4096])
@pytest.mark.parametrize("kind", ["normal", "ties", "const", "wide", "heavy", "signed0"])
def test_attn_threshold_stage_bit_exact(n, kind):
    """the threshold search of the batched attention path (every row-length variant) against the definition"""
    rng = np.random.default_rng(n * 11 + len(kind))
    rows = 24
    s = _rows(rng, rows, n, kind)
    n_valid = rng.integers(1, n + 1, rows).astype(np.int32)
    n_valid[0] = n
    k = np.array([rng.integers(1, nv + 1) for nv in n_valid], np.int32)
    k[0] = n
    k[1] = 1
    k[2] = max(1, n_valid[2] - 1)
    for r, frac in zip(range(3, 9), (0.125, 0.25, 0.5, 0.75, 0.9, 0.02)):      # the action table's keep-rates
        n_valid[r] = n
        k[r] = max(1, int(np.ceil(frac * n)))
    keep = host(sol.attn_threshold(dev(s), dev(n_valid), dev(k))).astype(np.uint8)
    for r in range(rows):
        want = np.zeros(n, np.uint8)
        want[:n_valid[r]] = oracle.select_keys(s[r, :n_valid[r]], int(k[r]))
        assert np.array_equal(keep[r], want), (r, n_valid[r], k[r])


@pytest.mark.parametrize("n", [1, 64, 255, 256, 257, 700, 1023, 1024])
@pytest.mark.parametrize("kind", ["normal", "ties", "const", "wide", "heavy", "signed0"])
def test_attn_threshold_of_two_and_of_four_rows_per_wave(n, kind):
    """rows of up to 1024 keys are searched four to a wave or two, by head size and cache layout; the hook takes four for the
    first half of the rows and two for the second: the same rows in both halves"""
    rng = np.random.default_rng(n * 13 + len(kind))
    rows = 18                                                         # the last waves of both halves are not full
    s = _rows(rng, rows, n, kind)
    n_valid = rng.integers(1, n + 1, rows).astype(np.int32)
    n_valid[::3] = n
    k = np.array([rng.integers(1, nv + 1) for nv in n_valid], np.int32)
    twice = lambda a: np.concatenate([a, a])  # noqa: E731
    keep = host(sol.attn_threshold(dev(twice(s)), dev(twice(n_valid)), dev(twice(k)))).astype(np.uint8)
    for r in range(rows):
        want = np.zeros(n, np.uint8)
        want[:n_valid[r]] = oracle.select_keys(s[r, :n_valid[r]], int(k[r]))
        assert np.array_equal(keep[r], want) and np.array_equal(keep[rows + r], want), (r, n_valid[r], k[r])


def test_attn_threshold_stage_rejects_long_rows():
    s = torch.zeros((1, 4097), dtype=torch.float32, device="cuda")
    one = torch.ones(1, dtype=torch.int32, device="cuda")
    with pytest.raises(sol.SolError):
        sol.attn_threshold(s, one, one)


@pytest.mark.parametrize("n", [1, 96, 1024, 8192, 14336])
@pytest.mark.parametrize("kind", ["normal", "ties", "const"])
def test_prune_mask_bit_exact(n, kind):
    rng = np.random.default_rng(n + len(kind))
    rows = 8
    a = _rows(rng, rows, n, kind)
    m = rng.integers(1, n + 1, rows).astype(np.int32)
    m[0] = n
    m[1] = 1
    for r, frac in zip(range(2, 6), (0.25, 0.5, 0.75, 0.125)):
        m[r] = max(1, int(np.ceil(frac * n)))
    keep = host(sol.prune_mask(dev(a), dev(m))).astype(np.uint8)
    for r in range(rows):
        assert np.array_equal(keep[r], oracle.topm_mask(a[r], int(m[r]))), (r, m[r])


@pytest.mark.parametrize("n", [1, 5, 256, 2048, 8192])
def test_quant_codes_bit_exact(n):
    rng = np.random.default_rng(n)
    bits = np.array([4, 5, 6, 7, 8, 10, 12, 15, 16, 17, 4, 8], np.int32)
    rows = len(bits)
    z = (rng.standard_normal((rows, n)) * np.exp(rng.uniform(-3, 3, (rows, 1)))).astype(np.float32)
    z[10] = 0.0                                                  # all-zero row
    z[11] = np.round(z[11] * 4) / 4                              # many exact halves after scaling
    codes, scale, zhat = sol.quant_codes(dev(z), dev(bits))
    codes, scale, zhat = host(codes).astype(np.int32), host(scale), host(zhat)
    for r in range(rows):
        o, c, s = oracle.fake_quant(z[r], int(bits[r]))
        assert np.array_equal(codes[r], c), r
        assert np.float32(scale[r]) == np.float32(s)
        assert np.array_equal(zhat[r], o), r


@pytest.mark.parametrize("n,dtype,rows", [(1024, "bf16", 24), (8192, "bf16", 24), (8192, "bf16", 600), (14336, "bf16", 24), (14336, "bf16", 600),
                                          (11264, "bf16", 24), (11264, "bf16", 600), (768, "bf16", 24), (1024, "f32", 24),
                                          (8192, "f32", 24)])
def test_prune_quant_kernel_bit_exact(n, dtype, rows):
    """The production prune + quantise kernel (wave-per-row for bf16 rows of 512*k channels, workgroup
    radix select otherwise) against oracle top-m mask -> fake-quant -> storage rounding."""
    from paper_2605_10875_amd import synth
    rng = np.random.default_rng(n)     # up to 512 rows: four waves per row; more: one, or four / two for rows over 8192 channels
    a = (rng.standard_normal((rows, n)) * rng.standard_normal((rows, n))).astype(np.float32) * 0.4
    a[3] = np.round(a[3] * 2) / 2                                   # few distinct values, many exact zeros
    a[4] = 0.0
    if dtype == "bf16":
        a = synth.round_to_bf16(a)
    m = np.array([max(1, int(np.ceil(f * n))) for f in (1, .75, .5, .25, .5, .125)] * (rows // 6), np.int32)
    bits = np.repeat(np.array([16, 8, 6, 4], np.int32), rows // 4)
    m[6] = n                                                        # quantise only
    t = dev(a).to(torch.bfloat16) if dtype == "bf16" else dev(a)
    out = host(sol.prune_quant(t, dev(m), dev(bits)))
    for r in range(rows):
        keep = oracle.topm_mask(a[r], int(m[r]))
        want, _, _ = oracle.fake_quant(a[r] * keep, int(bits[r]))
        if dtype == "bf16":
            want = synth.round_to_bf16(want)
        assert np.array_equal(out[r], want), (r, m[r], bits[r], np.flatnonzero(out[r] != want)[:8])


@pytest.mark.parametrize("n,rows", [(1024, 24), (2048, 600), (8192, 24), (8192, 600), (11264, 600), (14336, 24)])
def test_prune_search_at_extreme_ranks_and_rows(n, rows):
    """the search for the m-th magnitude where its first pivots are far off: ranks 1, 2, n - 2 and n - 1, rows of many
    binades, of one value, of two values, half zeros, one element 2^60 times the others (no quantiser: the kept values)"""
    from paper_2605_10875_amd import synth
    rng = np.random.default_rng(n + rows)
    a = rng.standard_normal((rows, n)).astype(np.float32)
    a[1::7] *= np.exp(rng.uniform(-60, 60, a[1::7].shape)).astype(np.float32)
    a[2::7] = 1.25
    a[3::7] = np.where(a[3::7] > 0, 3.0, -1e-30)
    a[4::7, ::2] = 0.0
    a[5::7, n // 3] = 2.0 ** 60
    a[6::7] *= 1e-38                                                # subnormals among them
    a = synth.round_to_bf16(a)
    m = np.array([(1, 2, n - 1, n - 2, n // 2, n // 16, 7)[(r // 7) % 7] for r in range(rows)], np.int32)
    out = host(sol.prune_quant(dev(a).to(torch.bfloat16), dev(m), dev(np.full(rows, 16, np.int32))))
    for r in range(rows):
        want = a[r] * oracle.topm_mask(a[r], int(m[r]))
        assert np.array_equal(out[r], want), (r, m[r], np.flatnonzero(out[r] != want)[:8])


@pytest.mark.parametrize("n,rows", [(2048, 24), (8192, 600), (11264, 600), (14336, 24)])
def test_prune_search_with_infinities_and_nans(n, rows):
    """rows whose mean, and with it the first pivots, is infinite or a NaN: magnitudes rank by their bit patterns, a NaN above
    an infinity, equal ones by channel"""
    rng = np.random.default_rng(n)
    t = torch.from_numpy(rng.standard_normal((rows, n)).astype(np.float32)).to(torch.bfloat16)
    t[0::6, 5] = torch.inf
    t[1::6, 8::3] = -torch.inf
    t[2::6, n - 1] = torch.nan
    t[3::6, :] = torch.nan
    t[4::6, ::2] = torch.inf
    t[4::6, 1::4] = torch.nan
    t[5::6, :] *= 2.0 ** 120                                          # the mean overflows, no value does
    t[5::6, :] = torch.nan_to_num(t[5::6, :] * 64.0)
    m = np.array([(1, 2, n - 1, n // 2, n // 3, n // 16, 7)[(r // 6) % 7] for r in range(rows)], np.int32)
    words = t.view(torch.int16).numpy()
    got = sol.prune_quant(t.cuda(), dev(m), dev(np.full(rows, 16, np.int32))).view(torch.int16).cpu().numpy()
    for r in range(rows):
        order = np.argsort(-(words[r].astype(np.int32) & 0x7FFF), kind="stable")
        want = np.zeros(n, np.int16)
        want[order[:m[r]]] = words[r][order[:m[r]]]
        assert np.array_equal(got[r], want), (r, m[r], np.flatnonzero(got[r] != want)[:8])


def test_quant_codes_worked_examples():
    with open(os.path.join(GOLDEN, "fake_quant_worked.txt")) as f:
        for line in f:
            if line.startswith("#") or not line.strip():
                continue
            b, z, c, zh = [p.strip() for p in line.split("|")]
            z = np.array(z.split(), np.float32)[None]
            codes, _, zhat = sol.quant_codes(dev(z), dev(np.array([int(b)], np.int32)))
            assert host(codes)[0].astype(np.int32).tolist() == [int(v) for v in c.split()]
            assert np.array_equal(host(zhat)[0], np.array(zh.split(), np.float32))


def test_empty_inputs_are_no_ops():
    z = torch.zeros((0, 8), dtype=torch.float32, device="cuda")
    e = torch.zeros(0, dtype=torch.int32, device="cuda")
    assert sol.topk_select(z, e, e).shape == (0, 8)
    assert sol.prune_mask(z, e).shape == (0, 8)


def test_rates_of_the_matrix_instructions():
    """Four rates below the published dense peak; operands that are no constants cost power and never gain."""
    ones32, normal32, ones16, normal16 = sol.measure_mfma(reps=10)
    assert all(0.0 < r <= 2600.0 for r in (ones32, normal32, ones16, normal16))
    assert normal32 <= 1.05 * ones32 and normal16 <= 1.05 * ones16
    L = sol.lib()
    assert L.sol_measure_mfma(None, 1 << 20, 1, None, None) == sol.ERR_INVALID_ARG

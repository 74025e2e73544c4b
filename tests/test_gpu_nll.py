"""The fold of the LM head's partial maxima and sums of exponentials, against 64 bits, at logits known exactly: each the product
of one channel of the hidden state and one weight. The logits are chosen where an exponential by way of a rounded product with
log2(e) is at its worst and the tiles' own exponentials are exact."""
import numpy as np
import pytest
import torch

from gpu_util import host
from paper_2605_10875_amd import sol, synth

pytestmark = pytest.mark.gpu

D, GROUPS = 256, 16                                   # 16 tokens, each with 16 channels of its own (value 4: mean square 1)
LOG2E = np.float64(np.float32(1.4426950408889634))


def _residue(x):
    """x * log2(e) in fp32 minus the product, in units of the natural exponent."""
    exact = np.float64(np.float32(x)) * LOG2E
    return float((np.float64(np.float32(exact)) - exact) * np.log(2.0))


def _bf16(x):
    return float(torch.tensor(x, dtype=torch.float64).to(torch.bfloat16))


def _logits(rng, vocab):
    """A channel's gain, the target's weight and that of the other tiles' entries, in bf16: half of the mass each, logits 4 * gain * weight."""
    while True:
        gain = _bf16(rng.uniform(0.25, 0.5))
        top = _bf16(rng.uniform(-0.2, 0.2))
        low = _bf16((4 * gain * top - np.log(vocab - 128.0) + rng.uniform(-0.3, 0.3)) / (4 * gain))
        t, o = 4 * gain * top, 4 * gain * low
        if float(np.float32(o - t)) == o - t and abs(_residue(t)) < 3e-8 and abs(_residue(o)) < 3e-8 and _residue(o - t) > 5e-7:
            return gain, top, low


@pytest.mark.parametrize("vocab", [128256, 152064])   # 1002 tiles, all in registers; 1188, the last of them read twice
def test_fold_of_the_tiles_is_accurate_to_fp32(vocab):
    shape = synth.ModelShape(D, 4, 2, 64, 512, 1, vocab)
    rng = np.random.default_rng(vocab)
    chosen = [_logits(rng, vocab) for _ in range(GROUPS)]
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    layer = dict(wq=z(256, D), wk=z(128, D), wv=z(128, D), wo=z(D, 256), w_gate=z(512, D), w_up=z(512, D), w_down=z(D, 512),
                 w_in_norm=z(D) + 1, w_post_norm=z(D) + 1)          # hands the embedding on
    embed, lm, norm = z(vocab, D), z(vocab, D), z(D)
    for g, (gain, top, low) in enumerate(chosen):                   # the 16 channels of token g: one of them counts
        embed[g, 16 * g:16 * g + 16] = 4.0
        norm[16 * g] = gain
        lm[:, 16 * g] = low
        lm[:128, 16 * g] = -100.0
        lm[7 * g, 16 * g] = top                                     # its target, the only entry of its tile that counts
    tokens = torch.arange(GROUPS, dtype=torch.int32, device="cuda").view(1, GROUPS)
    ctx = sol.Sol(shape, [synth.DENSE_ACTION], max_positions=GROUPS)
    nll = host(ctx.schedule_loglik([layer], dict(embed=embed, w_final_norm=norm, lm_head=lm), tokens, 7 * tokens,
                                   torch.zeros((1, 1, GROUPS), dtype=torch.int32, device="cuda"))).reshape(-1).astype(np.float64)
    assert ctx.device_status() == sol.OK
    ref = np.array([np.log1p((vocab - 128) * np.exp(low - top)) for top, low in ((4 * a * t, 4 * a * o) for a, t, o in chosen)])
    err = np.abs(nll - ref)
    # The other tiles are alike, so that a token's roundings add up. Relative error of their mass: a tile's exponentials 1 ulp
    # (2^-23), its factor 1 ulp and a rounding, a rounding (2^-24) on each of ten levels of sums, two more where tiles are read
    # twice: 1.05e-6 at most, times a share of the mass of at most 0.6; then 1 ulp and two roundings of values below 1: 8.5e-7. Over
    # the tokens these are of either sign (8e-8 on average in a model of the fold on the CPU), but a rounded product with log2(e)
    # alone is 3.8e-7 off on average.
    assert err.max() < 8.5e-7, err
    assert err.mean() < 2e-7, err


# tiles of 32, 64 and 256 columns: a token's partial results are the same chains and sums in all of them
@pytest.mark.parametrize("d,vocab", [(256, 256), (640, 1280), (2048, 128256)])
def test_the_head_of_few_tokens_has_the_bits_of_the_large_tiles(d, vocab):
    shape = synth.ModelShape(d, 4, 2, 64, 512, 1, vocab)
    g = torch.Generator(device="cuda").manual_seed(vocab)
    r = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    layer = dict(wq=z(256, d), wk=z(128, d), wv=z(128, d), wo=z(d, 256), w_gate=z(512, d), w_up=z(512, d), w_down=z(d, 512),
                 w_in_norm=z(d) + 1, w_post_norm=z(d) + 1)          # hands the embedding on
    head = dict(embed=r(vocab, d), w_final_norm=r(d), lm_head=r(vocab, d) * d ** -0.5)
    tokens, targets = (torch.randint(0, vocab, (1, 70), generator=g, device="cuda", dtype=torch.int32) for _ in range(2))
    ctx = sol.Sol(shape, [synth.DENSE_ACTION], max_positions=70)

    def nll(n):
        return ctx.schedule_loglik([layer], head, tokens[:, :n].contiguous(), targets[:, :n].contiguous(),
                                   torch.zeros((1, 1, n), dtype=torch.int32, device="cuda")).reshape(-1)

    ref = nll(70)
    for n in (1, 31, 32, 33, 63, 64, 65):
        assert torch.equal(nll(n), ref[:n]), n
    assert ctx.device_status() == sol.OK
    x = head["embed"][tokens[0].long()].double()                    # all 70 rows, in 64 bits; the normalised row rounds to bf16
    h = (x * (x.square().mean(1, keepdim=True) + 1e-5).rsqrt() * head["w_final_norm"].double()).to(torch.bfloat16).double()
    logits = h @ head["lm_head"].double().T
    want = torch.logsumexp(logits, 1) - logits.gather(1, targets[0].long()[:, None])[:, 0]
    # logits are sums of d products, of about one in all: 2^-24 sqrt(d) of them by rounding, and 2^-9 of the row where a rounding of h flips
    assert (ref.double() - want).abs().max() < 1e-3

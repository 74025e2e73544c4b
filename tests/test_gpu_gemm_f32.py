"""fp32 linear maps on the fp32 matrix instructions: stacked q/k/v and gate/up matrices whose widths are no multiples of
the tile, ragged row counts, a ragged vocabulary, the shortest K, every tile of the cost rule, and a width (K no multiple
of 32) that stays on the fmaf kernel; under the dense action, where no decision amplifies a rounding, against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, dev_weights, host
from paper_2605_10875_amd import sol, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hq,hkv,dh,ff,vocab,n_seq,T", [
    (32, 1, 1, 32, 32, 33, 1, 1),             # one row, one slice of K, one tile
    (96, 3, 1, 32, 160, 77, 1, 37),           # q | k | v of 96 + 32 + 32 columns in one product
    (96, 3, 1, 32, 160, 1001, 2, 65),         # rows and vocabulary one past a tile
    (128, 2, 2, 64, 2080, 130, 3, 129),       # gate | up boundary inside a tile
    (256, 4, 4, 64, 16400, 100, 16, 128),     # 128 x 128 tiles in rounds
    (72, 9, 3, 8, 200, 50, 2, 40),            # K = 72 and 200: the fmaf kernel
])
def test_dense_fp32_pass_matches_the_oracle(d, hq, hkv, dh, ff, vocab, n_seq, T):
    shape = synth.ModelShape(d, hq, hkv, dh, ff, 1, vocab)
    layers, head = [synth.layer_weights(shape, 5, std=0.1)], synth.head_weights(shape, 6, std=0.5)
    tokens, targets = synth.tokens_and_targets(n_seq, T, vocab, 7)
    ids = np.zeros((n_seq, 1, T), np.int32)
    table = [synth.DENSE_ACTION]
    ref = oracle.schedule_loglik(oracle.make_cfg(shape), oracle.make_table(table), head["embed"], layers,
                                 head["w_final_norm"], head["lm_head"], tokens, targets, ids)
    ctx = sol.Sol(shape, table, dtype=sol.F32, max_positions=T)
    nll = host(ctx.schedule_loglik([dev_weights(layers[0], sol.F32)], dev_weights(head, sol.F32), dev(tokens), dev(targets), dev(ids)))
    assert ctx.device_status() == sol.OK
    # chains of at most 16400 fp32 sums of unit-scale terms through five products: well under 1e-4 of the logits' scale
    assert np.abs(nll - ref).max() <= 1e-4 * max(1.0, np.abs(ref).max())


# the 32 x 32 tile of few rows, 64 x 64 and 128 x 128 tiles of many; heads of 8 to 64, column pairs that cross a tile's edge
@pytest.mark.parametrize("d,hq,hkv,dh,ff,n_seq,T", [(96, 3, 1, 32, 161, 2, 3), (64, 8, 2, 8, 32, 3, 33), (128, 6, 3, 64, 8192, 4, 127)])
def test_fp32_layer_behind_a_past_and_a_sequence_that_does_not_fit(d, hq, hkv, dh, ff, n_seq, T):
    shape, L, last = synth.ModelShape(d, hq, hkv, dh, ff), T + 9, n_seq - 1
    w = synth.layer_weights(shape, 21, std=0.1)
    x = synth.hidden_states(n_seq, T, d, 22)
    ids = np.zeros((n_seq, T), np.int32)
    pos0 = (4 * np.arange(n_seq) % 10).astype(np.int32)
    kc, vc = synth.kv_cache(n_seq, hkv, L, dh, 23)
    ko, vo = kc.copy(), vc.copy()
    ref, _ = oracle.layer_forward(oracle.make_cfg(shape), oracle.make_table([synth.DENSE_ACTION]), w, x, ids, ko, vo, pos0=pos0)
    ctx = sol.Sol(shape, [synth.DENSE_ACTION], dtype=sol.F32, max_positions=L)
    kd, vd = dev(kc), dev(vc)
    out = host(ctx.layer_forward(dev_weights(w, sol.F32), dev(x), dev(ids), kd, vd, pos0=dev(pos0)))
    assert ctx.device_status() == sol.OK
    # sums of at most 8192 fp32 products in chains of that length: 8192 * 2^-24 = 5e-4 of the largest, were all errors of one sign
    for got, want in ((out, ref), (host(kd), ko), (host(vd), vo)):
        assert np.abs(got - want).max() <= 1e-4 * max(1.0, np.abs(want).max())
    pos0[last] = L - T + 1
    kd, vd = dev(kc), dev(vc)
    again = host(ctx.layer_forward(dev_weights(w, sol.F32), dev(x), dev(ids), kd, vd, pos0=dev(pos0)))
    assert ctx.device_status() == sol.ERR_CACHE_OVERFLOW
    assert np.array_equal(again[:last], out[:last])
    assert np.array_equal(host(kd)[last], kc[last]) and np.array_equal(host(vd)[last], vc[last])   # untouched

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

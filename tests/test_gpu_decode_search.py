"""The search for a decode row's threshold where it ends in a ranking of the few keys left in its bracket: rows that have few keys
from the start, and ties inside the bracket, beyond and within the budget, against the definition and across both kernels."""
import pytest

import test_gpu_decode_split as split

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

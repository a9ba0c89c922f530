"""How a prompt that the workspace does not hold at once is cut into slices (csrc/api.hip, sled_prefill), counted by the projections
it launches.  A prompt of n tokens runs in blocks of nine rows here (too few for blocks of sixteen), `blocks` of them at most at a time."""
import numpy as np
import pytest
import torch

from paper_2506_09397_amd import sled, synth
from paper_2506_09397_amd.runtime import Verifier

pytestmark = pytest.mark.gpu


def _slices(shape, n, blocks):
    v = Verifier(shape, synth.SynthWeights(shape, seed=1, device="cuda"), n // 16 + 8, 1, blocks, n + 64)
    tokens = torch.from_numpy(synth.context_tokens(n, shape.vocab, seed=1).astype(np.int32)).cuda()
    r = v.open()
    sled.sled_profile_enable(v.model, True)
    v.prefill(r, tokens, want_logits=False)
    _, launches = sled.sled_profile_read(v.model)
    sled.sled_profile_enable(v.model, False)
    v.destroy()
    assert launches[sled.PROF_PROJ] % (4 * shape.n_layers) == 0
    return launches[sled.PROF_PROJ] // (4 * shape.n_layers)


SMALL = dict(d_model=1024, d_ffn=4096)


@pytest.mark.parametrize("dims,n,blocks,want", [
    # 15 blocks are 135 rows: past 128 a layer costs 237 us instead of 165.  Five slices of 135 lose to five of 126 and one of 45.
    ({}, 675, 15, 6),
    # small layers, where a launch weighs more than the weights: 85 us a layer at 126 rows, 112 at 225.  Nine of 225 or less; sixteen of 126 took 22.4
    # instead of 17.8 ms for sixteen layers, and four of 126 or less 5.2 instead of three in 4.5
    (SMALL, 2000, 25, 9),
    (SMALL, 483, 25, 3),
    # gate/up in two K slices whatever the rows (64 column blocks), where other projections thin theirs out: four of 225 or less, not seven of 126
    (SMALL, 853, 25, 4),
])
def test_number_of_slices(dims, n, blocks, want):
    shape = synth.scaled_shape(synth.SHAPES["llama8b"], n_layers=1, vocab=1024, **dims)
    assert _slices(shape, n, blocks) == want

"""Prompts long enough for blocks of sixteen rows (sled_prefill, csrc/api.hip: four query tiles, three page groups in the attention), in one
slice and in several whose length is chosen, against the oracle's causal forward over the whole sequence."""
import numpy as np
import pytest
import torch

from oracle import sled_oracle as O
from paper_2506_09397_amd import sled, synth
from gpu_common import build_verifier
from helpers import oracle_model

pytestmark = pytest.mark.gpu

# The oracle attends to the stored K/V (audited), so what is left is activations rounded to 2^-17 and float32 sums: as test_gpu_tile_rows.py has it
# about 1e-5 of a logit's standard deviation (0.64 here) a layer, five times that for the worst of two thousand; two layers.
TOL = 2 * 5e-5


def _block_bytes(shape, blocks, rows, n):
    """workspace of `blocks` blocks of `rows` rows that see n tokens: that of a verification whose requests have as many"""
    m = sled.sled_model_create(synth.scaled_shape(shape, k_max=rows - 1))
    need = sled.sled_verify_workspace_bytes(m, blocks, blocks * rows, blocks * n) - 256
    sled.sled_model_destroy(m)
    return need


# 112 blocks of nine rows hold 1008 rows, 60 hold 540: 34 blocks of sixteen, of the prompt's 44 to 63
@pytest.mark.parametrize("n", [700, 1001])
@pytest.mark.parametrize("b_max", [112, 60])
def test_blocks_of_sixteen_rows(n, b_max):
    shape = synth.scaled_shape(synth.SHAPES["llama8b"], n_layers=2, d_model=1024, d_ffn=2048, vocab=2048)
    v, w = build_verifier(shape, 7, n_pages=n // 16 + 8, max_requests=1, B_max=b_max, ctx_tokens_max=n + 64)
    room = v.ws.numel()
    assert _block_bytes(shape, 32, 16, n) <= room          # a work item for every CU with blocks of sixteen: they are taken
    whole = _block_bytes(shape, -(-n // 16), 16, n) <= room
    assert whole == (b_max == 112)
    p = synth.context_tokens(n, shape.vocab, seed=n)
    r = v.open()
    sled.sled_profile_enable(v.model, True)
    got = v.prefill(r, torch.from_numpy(p.astype(np.int32)).cuda()).cpu().numpy().astype(np.float64)
    launches = sled.sled_profile_read(v.model)[1]
    slices = launches[sled.PROF_ATTN] // shape.n_layers
    assert slices == 1 if whole else slices >= 2
    K, V = (synth.as_f64(x) for x in v.read_kv(r, 0, n))
    v.destroy()
    K0, V0 = O.empty_kv(oracle_model(shape, w))
    res = O.verify_batch(oracle_model(shape, w), [{"tokens": p, "K": K0, "V": V0, "K_stored": K, "V_stored": V}])[0]
    err, au = np.abs(got - res["logits"][-1]).max(), res["audit"]
    print(f"{n} tokens, {slices} slices: max |logit error| = {err:.3e}; stored K/V: {au['flips']} of {au['elements']} differ, worst excess {au['max_excess']:.2e}")
    assert err < TOL
    # roundings of values within 1e-4 of their head vector a layer, as there
    assert au["max_excess"] < 2e-4 and au["flips"] < 0.02 * au["elements"]

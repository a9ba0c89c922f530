"""Projections of few rows (csrc/gemm.hip, gemm_kwave_kernel) give the very bits of the kernels that larger batches run.

A row's sums are those of the k-steps 0, 4, ..; 1, 5, ..; and so on of its K slice, added in ascending order, in every kernel for up to 128 rows,
and up to 128 rows the K slices are the same.  So requests verified in a batch of up to 32 rows (4-bit weights: 64) have the logits that
they have in a batch of more rows, bit for bit.  Contexts are short enough not to be cut by the attention, and the larger batch stays
below 97 rows, where the LM head takes a shape of its own."""
import pytest
import torch

from paper_2506_09397_amd import synth
from paper_2506_09397_amd.runtime import Verifier

pytestmark = pytest.mark.gpu

WEIGHTS = {16: synth.SynthWeights, 8: synth.SynthWeightsW8, 4: synth.SynthWeightsW4}
# a vocabulary whose last column block holds two of its four column tiles
SHAPES = {"tiny": synth.SHAPES["tiny_bf16"], "8b_layer": synth.scaled_shape(synth.SHAPES["llama8b"], n_layers=1, vocab=1024 + 64),
          # 272 k-steps, whole: 68 to a wavefront, so the eight-set loop of 4-bit weights ends with twelve steps left instead of eight
          "272_steps": synth.scaled_shape(synth.SHAPES["llama8b"], n_layers=1, d_model=4352, d_ffn=1024, vocab=1024 + 64)}


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bits", [16, 8, 4])
def test_rows_of_a_small_batch_have_the_bits_of_a_larger_one(shape, bits):
    s = SHAPES[shape]
    B, k = 96, 0
    v = Verifier(s, WEIGHTS[bits](s, seed=3, device="cuda"), n_pages=4 * B, max_requests=B, B_max=B, ctx_tokens_max=64 * B)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    reqs = [v.open() for _ in range(B)]
    for i, r in enumerate(reqs):
        n = 1 + 7 * i % 40
        v.append_context([r], *[[torch.randn(s.n_layers, n, s.n_kv_heads, s.head_dim, generator=g, device="cuda").to(s.torch_dtype)] for _ in range(2)])
    tokens = torch.randint(0, s.vocab, (B,), generator=g, device="cuda", dtype=torch.int32)
    rows = [1, 31, 32, 33, 63, 64]
    got = {T: v.verify(reqs[:T], [k] * T, tokens[:T]).clone() for T in rows}
    want = v.verify(reqs, [k] * B, tokens).clone()
    assert torch.isfinite(want).all()
    for T in rows:
        assert torch.equal(got[T], want[:T]), f"{T} rows"
    v.destroy()

"""Models small enough for a cache load their weights in the caches' ordinary order, larger ones past it (csrc/gemm.hip): the same kernels
otherwise, so the same bits.  A model and one that differs only in more vocabulary, which puts it past the line of 224 MB, must agree
in the logits that they share, in every kernel of up to 128 rows."""
import pytest
import torch

from paper_2506_09397_amd import synth
from paper_2506_09397_amd.runtime import Verifier

pytestmark = pytest.mark.gpu

WEIGHTS = {16: synth.SynthWeights, 8: synth.SynthWeightsW8, 4: synth.SynthWeightsW4}


class FirstTokens:
    """another weights object without the tokens from `vocab` on"""

    def __init__(self, w, shape):
        self.w, self.shape, self.bits = w, shape, getattr(w, "bits", 16)
        self.MATRICES = getattr(w, "MATRICES", ())

    def _cut(self, name, x):
        return x[: self.shape.vocab].contiguous() if name == "lm_head" else x

    def embed(self):
        return self.w.embed()[: self.shape.vocab].contiguous()

    def tensor(self, name, layer=-1):
        return self._cut(name, self.w.tensor(name, layer))

    def q(self, name, layer=-1):
        return self._cut(name, self.w.q(name, layer))

    def scale(self, name, layer=-1):
        return self._cut(name, self.w.scale(name, layer))


@pytest.mark.parametrize("invariant", [False, True])
@pytest.mark.parametrize("bits", [16, 8, 4])
def test_a_cached_model_has_the_bits_of_a_larger_one(bits, invariant):
    big = synth.scaled_shape(synth.SHAPES["llama8b"], n_layers=1, d_ffn=2048, vocab=97280)   # (fewer columns than the shape for 97 to 128 rows of a large head needs)
    small = synth.scaled_shape(big, vocab=1024 + 64)
    assert small.streamed_params() * bits / 8 < 224e6 < big.streamed_params() * bits / 8
    w = WEIGHTS[bits](big, seed=3, device="cuda")
    got = {}
    rows = [1, 32, 33, 64, 65, 96, 97, 128, 129]
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    tokens = torch.randint(0, small.vocab, (max(rows),), generator=g, device="cuda", dtype=torch.int32)
    K, V = (torch.randn(1, 20, big.n_kv_heads, big.head_dim, generator=g, device="cuda").to(big.torch_dtype) for _ in range(2))
    for shape, weights in ((big, w), (small, FirstTokens(w, small))):
        B = (max(rows) + 8) // 9
        v = Verifier(shape, weights, n_pages=4 * B, max_requests=B, B_max=B, ctx_tokens_max=64 * B, batch_invariant=invariant)
        reqs = [v.open() for _ in range(B)]
        v.append_context(reqs, [K] * B, [V] * B)
        for T in rows:
            n = (T + 8) // 9
            out = v.verify(reqs[:n], [8] * (n - 1) + [T - 9 * (n - 1) - 1], tokens[:T])[:, : small.vocab].clone()
            assert torch.isfinite(out).all()
            if shape is big:
                got[T] = out
            else:
                assert torch.equal(out, got[T]), f"{T} rows"
        v.destroy()

"""How the projections add up their products: k-steps (of 16 products) go to several sums that are added at the end -- four in
steps of up to 128 rows, two beyond -- so that no sum's rounding grows with the whole length of a row.

The LM head is given rows in which a large product enters the first of these sums with the first k-step and leaves it with its
last one, and products too small to be seen beside it go to another sum.  One running sum would lose all of them."""
import pytest
import torch

from paper_2506_09397_amd import synth
from paper_2506_09397_amd.runtime import Verifier

pytestmark = pytest.mark.gpu

BIG, SMALL = 65536.0, 2.0 ** -14


class _Weights(synth.SynthWeights):
    """Embedding rows of ones and no layer output, so that the LM head sees 1 / sqrt(1 + eps) everywhere."""

    def tensor(self, name, layer=-1):
        t = super().tensor(name, layer)
        if name == "embed":
            return torch.ones_like(t)
        if name in ("wo", "wd"):
            return torch.zeros_like(t)
        if name == "lm_head":
            t = torch.zeros_like(t)
            for s in range(1, t.shape[1] // 16, 4):          # k-steps 1, 5, 9, ..: the second of four sums, the odd one of two
                t[:, 16 * s:16 * s + 16] = SMALL
            t[:, 0] = BIG                                    # k-step 0 and the last multiple of four: the first sum either way
            t[:, t.shape[1] - 64] = -BIG
        return t

    def embed(self):
        return self.tensor("embed")


# one to four row tiles; beyond 128 rows both heights of a workgroup: 28672 columns are 112 blocks, so 372 rows are
# 336 workgroups at four row tiles and 224 at six
@pytest.mark.parametrize("T,vocab", [(9, 1024), (45, 1024), (81, 1024), (126, 1024), (135, 1024), (207, 1024), (372, 28672)])
def test_small_products_beside_a_large_one(T, vocab):
    shape = synth.scaled_shape(synth.SHAPES["tiny_bf16"], n_layers=1, d_model=4096, vocab=vocab)
    k = [8] * (T // 9) + ([T % 9 - 1] if T % 9 else [])
    v = Verifier(shape, _Weights(shape, seed=0, device="cuda"), 4 * len(k) + 8, len(k), len(k), 32 * len(k))
    reqs = [v.open() for _ in k]
    KV = [synth.context_kv(shape, 3, seed=1, req=i, device="cuda") for i in range(len(k))]
    v.append_context(reqs, [a for a, _ in KV], [b for _, b in KV])
    got = v.verify(reqs, k, torch.zeros(T, dtype=torch.int32, device="cuda"))
    want = shape.d_model // 4 * SMALL                        # the activations are 1 - 5e-6
    # the large products leave what their sum's roundings at 2^16 (half of 2^-7, a few of them) do not cancel
    err = (got - want).abs().max().item()
    print(f"T={T}: {err:.2e} of {want}")
    assert err < 4 * 2.0 ** -8
    v.destroy()

"""Attention whose requests are cut into several work items, for every number of query tiles and item counts around the merge's chunks.

The page groups of a workgroup add up their states by dims, and the last of a request's items to arrive merges the stored ones, four
(up to three query tiles) or two (four and five tiles) at a time.  A request of n * 512 tokens on a single kv head is cut into
n items of 32 pages (at most eight), a batch-invariant model's into fixed runs of 48 pages."""
import numpy as np
import pytest
import torch

from oracle import sled_oracle as O
from paper_2506_09397_amd import sled, synth
from paper_2506_09397_amd.runtime import Verifier
from helpers import oracle_model, oracle_requests

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("invariant", [False, True])
@pytest.mark.parametrize("k", [0, 2, 4, 6, 8])    # G = 8: 8, 24, 40, 56, 72 query rows, one to five tiles
def test_requests_in_several_items(k, invariant):
    shape = synth.scaled_shape(synth.SHAPES["tiny_bf16"], n_layers=1, n_q_heads=8, n_kv_heads=1, k_max=k)
    w = synth.SynthWeights(shape, seed=11, device="cuda", std=0.03, gain_jitter=0.1)
    items = [1, 2, 3, 4, 5, 8]
    ctx_len = [n * 512 - k - 1 - 5 * (n % 2) for n in items]      # whole and ragged last pages
    B, ks = len(items), [k] * len(items)
    if not invariant:
        pages = [-(-(L + k + 1) // 16) for L in ctx_len]
        tgt, _ = sled.sled_attention_partition(1, pages)
        assert {-(-n // tgt) for n in pages} >= {1, 2, 3, 4, 5, 8}, tgt
    budget = sum(ctx_len) + (k + 1) * B
    v = Verifier(shape, w, budget // 16 + 3 * B + 8, B, B, budget, batch_invariant=invariant)
    batch = synth.make_batch(ctx_len, ks, shape.vocab, seed=3)
    reqs = [v.open() for _ in range(B)]
    KV = [synth.context_kv(shape, L, seed=3, req=i, device="cuda") for i, L in enumerate(ctx_len)]
    v.append_context(reqs, [K for K, _ in KV], [V for _, V in KV])
    tokens = torch.from_numpy(batch.tokens).cuda()
    first = v.verify(reqs, ks, tokens).clone()
    for _ in range(3):     # whichever item arrives last, the result is the same
        assert torch.equal(v.verify(reqs, ks, tokens), first)
    want = np.concatenate([r["logits"] for r in O.verify_batch(oracle_model(shape, w), oracle_requests(batch, [K for K, _ in KV], [V for _, V in KV]))], axis=0)
    err = np.abs(first.cpu().numpy().astype(np.float64) - want).max()
    assert err < 5e-3, err      # the bound of the other tests of this model (bf16 pairs between the kernels)
    v.destroy()

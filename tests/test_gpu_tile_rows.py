"""Verification steps against the oracle at the row counts where the projections' workgroups change height (1 to 4 tiles of
32 rows in one block; 4, 6 or 8 beyond 128 rows), at whole and ragged last tiles, and with a vocabulary whose last column block is
partial.  One layer of small width but wide FFN and vocabulary, so that all heights occur."""
import numpy as np
import pytest
import torch

from oracle import sled_oracle as O
from paper_2506_09397_amd import synth
from gpu_common import build_verifier, oracle_requests
from helpers import oracle_model

pytestmark = pytest.mark.gpu

# sums over at most 14336 products in float32 and activations kept to 16 bits are good to 1e-5 here; a K/V value next to a
# bf16 rounding boundary may round the other way, which moves a logit by up to a few 1e-3 (the bound of the small bf16 models)
TOL = 5e-3


@pytest.mark.parametrize("T", [1, 31, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 227, 256, 257, 367, 385, 500])
def test_rows_at_the_edges_of_tiles_and_blocks(T):
    shape = synth.scaled_shape(synth.SHAPES["tiny_bf16"], n_layers=1, d_model=256, n_q_heads=2, n_kv_heads=1, d_ffn=14336, vocab=57376)
    k = [8] * (T // 9) + ([T % 9 - 1] if T % 9 else [])
    ctx = [1 + 7 * i % 40 for i in range(len(k))]
    batch = synth.make_batch(ctx, k, shape.vocab, seed=T)
    assert batch.T == T
    v, w = build_verifier(shape, 5, n_pages=4 * len(k) + 8, max_requests=len(k), B_max=len(k), ctx_tokens_max=64 * len(k))
    reqs = [v.open() for _ in k]
    KV = [synth.context_kv(shape, n, seed=5, req=i, device="cuda") for i, n in enumerate(ctx)]
    v.append_context(reqs, [a for a, _ in KV], [b for _, b in KV])
    got = v.verify(reqs, k, torch.from_numpy(batch.tokens).cuda()).cpu().numpy()
    res = O.verify_batch(oracle_model(shape, w), oracle_requests(batch, [a for a, _ in KV], [b for _, b in KV]))
    want = np.concatenate([r["logits"] for r in res], axis=0)
    err = np.abs(got - want).max()
    print(f"T={T}: max |logit error| = {err:.3e}")
    assert err < TOL
    v.destroy()

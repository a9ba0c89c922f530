"""Verification steps against the oracle at the row counts where the projections' workgroups change height (1 to 4 tiles of
32 rows in one block; 4 or 6 beyond 128 rows), at whole and ragged last tiles, and with a vocabulary whose last column block is
partial.  One layer of small width but wide FFN and vocabulary: gate/up and the LM head get both heights beyond 128 rows (16
k-steps each, in one slice), the other projections 4 (O and QKV in one slice, down in up to 16 equal ones).  Then one layer of the
large shapes, whose K is long enough for unequal slices and whose projections in slices get both heights: which case has
which is asserted, without a GPU, in test_host_planning.py."""
import numpy as np
import pytest
import torch

from oracle import sled_oracle as O
from paper_2506_09397_amd import synth
from gpu_common import build_verifier, oracle_requests
from helpers import oracle_model
from test_host_planning import LARGE_LAYER_CASES

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


# The oracle attends to the K/V that the library stored (audited), so no rounding to the cache is left in the comparison: each of the
# five projections adds activations rounded to 2^-17 and float32 sums, about 1e-5 of a logit's standard deviation (1.3 to 1.8) in all,
# and a million logits reach five times that; four times as much for what the norms and the attention do to it.
TOL_STORED = 4e-4


@pytest.mark.parametrize("model,T", [(m, T) for m, T, _ in LARGE_LAYER_CASES])
def test_slices_of_a_large_layer(model, T):
    shape = synth.scaled_shape(synth.SHAPES[model], n_layers=1, vocab=1024)
    k = [8] * (T // 9) + ([T % 9 - 1] if T % 9 else [])
    batch = synth.make_batch([3] * len(k), k, shape.vocab, seed=T)
    v, w = build_verifier(shape, 5, n_pages=len(k) + 8, max_requests=len(k), B_max=len(k), ctx_tokens_max=16 * len(k))
    reqs = [v.open() for _ in k]
    KV = [synth.context_kv(shape, 3, seed=5, req=i, device="cuda") for i in range(len(k))]
    v.append_context(reqs, [a for a, _ in KV], [b for _, b in KV])
    got = v.verify(reqs, k, torch.from_numpy(batch.tokens).cuda()).cpu().numpy()
    v.commit(reqs, torch.tensor(k, dtype=torch.int32, device="cuda"))
    stored = [v.read_kv(r, 3, n + 1) for r, n in zip(reqs, k)]
    oreqs = [dict(r, K_stored=synth.as_f64(a), V_stored=synth.as_f64(b))
             for r, (a, b) in zip(oracle_requests(batch, [a for a, _ in KV], [b for _, b in KV]), stored)]
    v.destroy()
    res = O.verify_batch(oracle_model(shape, w), oreqs)
    excess, flips = max(r["audit"]["max_excess"] for r in res), sum(r["audit"]["flips"] for r in res)
    elements = sum(r["audit"]["elements"] for r in res)
    err = np.abs(got - np.concatenate([r["logits"] for r in res], axis=0)).max()
    print(f"{model} T={T}: max |logit error| = {err:.3e}; stored K/V: {flips} of {elements} differ, worst excess {excess:.2e}")
    assert err < TOL_STORED
    # a stored number may be the rounding of a value 1e-4 of its head vector away (2^-17 on the way in, five times that at worst);
    # that close to a midpoint of two bf16 numbers lie about 2 x 1e-5 / 2^-8 of them at the typical distance
    assert excess < 1e-4 and flips < elements * 0.02

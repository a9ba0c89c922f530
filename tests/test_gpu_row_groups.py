"""Row kernels that put the rows of a line or page on one XCD, around the row counts where the mapping begins and its groups end, and the
prompt's QKV kernel for head counts that leave its last workgroup of a row part empty: against the oracle."""
import numpy as np
import pytest
import torch

from oracle import sled_oracle as O
from paper_2506_09397_amd import synth
from paper_2506_09397_amd.runtime import Verifier
from helpers import oracle_model, oracle_requests

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [64, 65, 71, 72, 73, 127, 129, 136])
def test_batches_around_whole_groups_of_rows(rows):
    shape = synth.SHAPES["tiny_bf16"]
    w = synth.SynthWeights(shape, seed=21, device="cuda", std=0.03, gain_jitter=0.1)
    ks = [8] * (rows // 9) + ([rows % 9 - 1] if rows % 9 else [])
    B = len(ks)
    ctx_len = [7 * i % 40 for i in range(B)]
    v = Verifier(shape, w, 5 * B + 8, B, B, sum(ctx_len) + 9 * B)
    batch = synth.make_batch(ctx_len, ks, shape.vocab, seed=rows)
    reqs = [v.open() for _ in range(B)]
    KV = [synth.context_kv(shape, L, seed=3, req=i, device="cuda") for i, L in enumerate(ctx_len)]
    v.append_context(reqs, [K for K, _ in KV], [V for _, V in KV])
    got = v.verify(reqs, ks, torch.from_numpy(batch.tokens).cuda()).cpu().numpy().astype(np.float64)
    want = np.concatenate([r["logits"] for r in O.verify_batch(oracle_model(shape, w), oracle_requests(batch, [K for K, _ in KV], [V for _, V in KV]))], axis=0)
    assert got.shape[0] == rows and np.abs(got - want).max() < 5e-3     # the bound of the other tests of this model
    v.destroy()


@pytest.mark.parametrize("n_q,n_kv", [(8, 2), (8, 1), (8, 8), (16, 4)])
@pytest.mark.parametrize("rows", [1, 15, 16, 17, 127, 130])
def test_prompt_rows_and_heads(n_q, n_kv, rows):
    """A prompt's cache and last logits equal those of a verification that is handed the same tokens behind the same context."""
    shape = synth.scaled_shape(synth.SHAPES["tiny_bf16"], n_q_heads=n_q, n_kv_heads=n_kv)
    w = synth.SynthWeights(shape, seed=5, device="cuda", std=0.03, gain_jitter=0.1)
    v = Verifier(shape, w, 64, 2, 16, 2048)
    tokens = synth.context_tokens(rows, shape.vocab, seed=rows)
    r = v.open()
    logits = v.prefill(r, torch.from_numpy(np.asarray(tokens, dtype=np.int32)).cuda()).cpu().numpy().astype(np.float64)
    K, V = v.read_kv(r, 0, rows)
    s = v.open()                                   # the same tokens, nine at a time, through the verification step's own kernels
    for a in range(0, rows, 9):
        part = np.asarray(tokens[a:a + 9], dtype=np.int32)
        last = v.verify([s], [len(part) - 1], torch.from_numpy(part).cuda())[-1].cpu().numpy().astype(np.float64)
        v.commit([s], torch.full((1,), len(part) - 1, dtype=torch.int32, device="cuda"))
    K2, V2 = v.read_kv(s, 0, rows)
    # Stored in 16 bits: two values on either side of a rounding boundary lie a step apart (2^-7 of the value at most), and what is
    # rounded differs by round-off and by such steps in the layer before, for which the oracle's audit of stored K/V allows
    # 1e-3 of the head vector's rms.
    for x, y in ((K, K2), (V, V2)):
        x, y = x.float(), y.float()
        rms = y.pow(2).mean(dim=-1, keepdim=True).sqrt()
        assert bool(((x - y).abs() <= 2.0**-7 * y.abs() + 1e-3 * rms).all()) and float((x != y).float().mean()) < 0.05
    assert np.abs(logits - last).max() < 5e-3
    v.destroy()


@pytest.mark.parametrize("heads", [12, 16])
def test_pages_of_many_heads_move_unchanged(heads):
    shape = synth.scaled_shape(synth.SHAPES["tiny_bf16"], n_q_heads=heads, n_kv_heads=heads)
    w = synth.SynthWeights(shape, seed=5, device="cuda")
    v = Verifier(shape, w, 16, 1, 1, 128)
    r = v.open()
    K, V = synth.context_kv(shape, 70, seed=2, req=0, device="cuda")
    for a, b in ((0, 3), (3, 16), (16, 48), (48, 70)):      # part of a page, its rest, whole pages, whole and part
        v.append_context([r], [K[:, a:b].contiguous()], [V[:, a:b].contiguous()])
    K2, V2 = v.read_kv(r, 0, 70)
    assert torch.equal(K, K2) and torch.equal(V, V2)
    v.destroy()

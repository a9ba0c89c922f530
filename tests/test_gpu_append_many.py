"""One append call for many requests (sixteen to a launch): just opened ones beside ones that hold tokens, pieces of no token, slots that
an earlier request has left with a length, buffers aligned to an element only."""
import numpy as np
import pytest
import torch

from paper_2506_09397_amd import synth
from gpu_common import build_verifier

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["tiny_bf16", "tiny"])
@pytest.mark.parametrize("B", [1, 16, 17, 33])
def test_mixed_pieces(kind, B):
    shape = synth.SHAPES[kind]
    v, _ = build_verifier(shape, 1, n_pages=12 * B, max_requests=B, B_max=B, ctx_tokens_max=160 * B)
    rng = np.random.default_rng(B)
    reqs = [v.open() for _ in range(B)]
    v.append_context(reqs, *zip(*[synth.context_kv(shape, 5, seed=9, req=i, device="cuda") for i in range(B)]))
    for r in reqs[::2]:                       # half of the slots are left and taken again: their old length must not count
        v.close_request(r)
    for i in range(0, B, 2):
        reqs[i] = v.open()
    held = [0 if i % 2 == 0 else 5 for i in range(B)]
    want = [tuple(x[:, :h] for x in synth.context_kv(shape, 5, seed=9, req=i, device="cuda")) for i, h in enumerate(held)]
    for turn in range(2):
        n = rng.integers(0, 70, size=B)
        n[::5] = 0
        new = [synth.context_kv(shape, max(int(x), 1), seed=20 + turn, req=i, device="cuda") for i, x in enumerate(n)]
        new = [tuple(x[:, :int(c)].contiguous() for x in kv) for kv, c in zip(new, n)]
        if turn:                              # a buffer that starts one element past an aligned address
            k = new[0][0]
            flat = torch.empty(k.numel() + 1, dtype=k.dtype, device="cuda")[1:]
            new[0] = (flat.copy_(k.reshape(-1)).view(k.shape), new[0][1])
        v.append_context(reqs, [k for k, _ in new], [x for _, x in new])
        want = [tuple(torch.cat(p, dim=1) for p in zip(a, b)) for a, b in zip(want, new)]
    assert v.lengths(reqs) == [int(k.shape[1]) for k, _ in want]
    for r, (K, V) in zip(reqs, want):
        if K.shape[1]:
            K2, V2 = v.read_kv(r, 0, K.shape[1])
            assert torch.equal(K, K2) and torch.equal(V, V2)
    v.destroy()

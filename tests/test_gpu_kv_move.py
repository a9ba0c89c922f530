"""K/V handed in and read back must be the same bits: pieces that start and end anywhere inside a page, one token to several
pages, buffers that are aligned to an element only, one to eight kv heads, both model types."""
import pytest
import torch

from paper_2506_09397_amd import sled, synth
from gpu_common import build_verifier

pytestmark = pytest.mark.gpu


def _shifted(x):
    """the same values in a buffer that starts one element past an aligned address"""
    flat = torch.empty(x.numel() + 1, dtype=x.dtype, device=x.device)
    flat[1:] = x.reshape(-1)
    return flat[1:].view(x.shape)


@pytest.mark.parametrize("kind,hkv", [("tiny_bf16", 1), ("tiny_bf16", 2), ("tiny_bf16", 8), ("tiny", 4)])
@pytest.mark.parametrize("shift", [False, True])
def test_pieces_in_and_out(kind, hkv, shift):
    shape = synth.scaled_shape(synth.SHAPES[kind], n_kv_heads=hkv)
    v, _ = build_verifier(shape, 1, n_pages=64, max_requests=2, B_max=2, ctx_tokens_max=600)
    pieces = [1, 14, 1, 16, 17, 3, 2, 64, 31, 100]
    K, V = synth.context_kv(shape, sum(pieces), seed=3, req=0, device="cuda")
    other = synth.context_kv(shape, 21, seed=3, req=1, device="cuda")
    r, r2 = v.open(), v.open()
    v.append_context([r2], [other[0]], [other[1]])
    at = 0
    for n in pieces:
        a, b = K[:, at:at + n].contiguous(), V[:, at:at + n].contiguous()
        v.append_context([r], [_shifted(a) if shift else a], [_shifted(b) if shift else b])
        at += n
    for first, n in [(0, at), (0, 1), (5, 9), (15, 2), (16, 16), (17, 64), (at - 1, 1), (30, at - 30)]:
        Ko, Vo = (torch.empty(shape.n_layers, n, hkv, shape.head_dim, dtype=shape.torch_dtype, device="cuda") for _ in range(2))
        if shift:
            Ko, Vo = _shifted(Ko), _shifted(Vo)
        sled.sled_kv_read(v.pool, r, first, n, Ko, Vo)
        assert torch.equal(Ko, K[:, first:first + n]) and torch.equal(Vo, V[:, first:first + n]), (first, n)
    Ko, Vo = v.read_kv(r2, 0, 21)
    assert torch.equal(Ko, other[0]) and torch.equal(Vo, other[1])
    v.destroy()

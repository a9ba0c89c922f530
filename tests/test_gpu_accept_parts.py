"""Acceptance of a large batch, whose rows are scanned in several launches that leave out what lies behind a rejection:
the same requests handed over a few at a time (one launch, every row scanned) must give the same lengths and tokens."""
import numpy as np
import pytest
import torch

from paper_2506_09397_amd import sled, synth

pytestmark = pytest.mark.gpu


def _run(mode, k, vocab, logits, tokens, q, u_acc, u_smp, pairs, ws=None):
    a = torch.zeros(len(k), dtype=torch.int32, device="cuda")
    t = torch.zeros_like(a)
    if ws is None:
        ws = sled.workspace(sled.sled_accept_workspace_bytes(len(k), sum(k) + len(k), vocab))
    ws.fill_(0xFF)   # statistics that nobody wrote read as NaN
    if pairs:
        ids, probs, rest = q
        sled.sled_accept_sparse(k, vocab, 1.0, logits, tokens, ids, probs, u_acc, u_smp, a, t, ws, q_rest=rest)
    elif mode == sled.SAMPLE:
        sled.sled_accept(mode, k, vocab, 1.0, logits, tokens, q, u_acc, u_smp, a, t, ws)
    else:
        sled.sled_accept(mode, k, vocab, 1.0, logits, tokens, None, None, None, a, t, ws)
    return a.cpu().numpy(), t.cpu().numpy()


# 128256 x 4 bytes: a cut at row 2 from 250 rows behind it, at 4 from 499; an odd vocabulary takes the scalar
# path; pairs: shorter and longer lists than a wavefront
@pytest.mark.parametrize("mode,vocab,B,k_max,pairs", [("sample", 128256, 220, 4, 0), ("sample", 128256, 150, 12, 0), ("greedy", 128256, 120, 9, 0),
                                                      ("sample", 50001, 320, 8, 0), ("sample", 128256, 130, 8, 3), ("sample", 128256, 120, 8, 70)])
def test_parts_match_small_batches(mode, vocab, B, k_max, pairs):
    rng = np.random.default_rng(B + vocab)
    k = rng.integers(0, k_max + 1, size=B).tolist()
    c = synth.accept_case(k, vocab, 0.5, seed=B, device="cuda")
    m = sled.GREEDY if mode == "greedy" else sled.SAMPLE
    tokens = c.tokens.clone()
    if mode == "greedy":   # four drafts out of five follow the argmax
        hit = torch.from_numpy(rng.random(tokens.numel() - 1) < 0.8).cuda()
        tokens[1:] = torch.where(hit, c.logits[:-1].argmax(dim=1).to(torch.int32), tokens[1:])
    tokens[rng.integers(0, tokens.numel(), size=4)] = vocab   # a few ids outside the vocabulary
    q = c.q
    if pairs:
        top = torch.topk(c.q, pairs, dim=1)
        q = (top.indices.int().contiguous(), top.values.contiguous(), (1.0 - top.values.double().sum(dim=1)).clamp_min(0.0).float())
    a, t = _run(m, k, vocab, c.logits, tokens, q, c.u_acc, c.u_smp, pairs)
    cu, cd = np.concatenate([[0], np.cumsum(np.add(k, 1))]), np.concatenate([[0], np.cumsum(k)])
    for i in range(0, B, 8):
        e = min(B, i + 8)
        r, d = slice(cu[i], cu[e]), slice(cd[i], cd[e])
        if not pairs:
            qq = c.q[d].contiguous()
        else:
            qq = tuple(x[d].contiguous() for x in q)
        a2, t2 = _run(m, k[i:e], vocab, c.logits[r].contiguous(), tokens[r].contiguous(), qq, c.u_acc[d].contiguous(), c.u_smp[i:e].contiguous(), pairs)
        assert a[i:e].tolist() == a2.tolist() and t[i:e].tolist() == t2.tolist(), f"requests {i}..{e - 1}"
    assert 0 < a.sum() < sum(k)


def _stat_bytes(T, vocab, segments=None):
    """the row statistics' share of a workspace: 16 bytes for each of a row's segments, whole 256 bytes"""
    n = min(16, -(-8192 // T))
    while n > 1 and vocab // n < 2048:
        n -= 1
    return (T * (segments or n) * 16 + 255) // 256 * 256


def _unwritten(ws):
    """16-byte records that nobody wrote, before the last one that somebody did"""
    r = (ws[:ws.numel() // 16 * 16].view(-1, 16) != 0xFF).any(dim=1).cpu().numpy()
    return int((~r[:np.flatnonzero(r)[-1]]).sum())


# the least workspace that is accepted has room for the statistics alone; one of 16 segments a row, the size for every call before the
# sweeps had launches of their own, has room for the word on every request that the scan in parts needs, but not for the sweeps; the
# least one and that word have room for the scan in parts with the five segments that 1800 rows get, not for the eight behind a cut
@pytest.mark.parametrize("mode,B", [("greedy", 200), ("sample", 200), ("sample", 120)])
def test_smaller_workspaces_and_the_static_one(mode, B):
    vocab, k = 128256, [8] * B
    T, m = 9 * B, sled.GREEDY if mode == "greedy" else sled.SAMPLE
    c = synth.accept_case(k, vocab, 0.5, seed=B + 1, device="cuda")
    args = (m, k, vocab, c.logits, c.tokens, c.q, c.u_acc, c.u_smp, 0)
    want = [x.tolist() for x in _run(*args)]
    sizes = {"least": _stat_bytes(T, vocab), "earlier": _stat_bytes(T, vocab, 16) + 256}
    if B == 200:
        sizes["coarse"] = _stat_bytes(T, vocab) + 1024
        assert sizes["coarse"] < _stat_bytes(T, vocab, 8)
    for size, n_bytes in sizes.items():
        ws = sled.workspace(n_bytes)
        assert [x.tolist() for x in _run(*args, ws=ws)] == want, size
        if size != "least":
            assert _unwritten(ws) > T // 4          # rows behind a rejection were left out
    with pytest.raises(sled.SledError):
        _run(*args, ws=sled.workspace(_stat_bytes(T, vocab))[:-256])
    a = torch.zeros(B, dtype=torch.int32, device="cuda")
    t = torch.zeros_like(a)
    q, ua, us = (c.q, c.u_acc, c.u_smp) if m == sled.SAMPLE else (None, None, None)
    sled.sled_accept_static(m, k, vocab, 1.0, c.logits, c.tokens, q, ua, us, a, t)
    assert [a.tolist(), t.tolist()] == want


def test_all_three_cuts():
    """Cuts at rows 2, 4 and 8 (about 1400 rows behind the last one): the later tests read rows that earlier cuts left out."""
    vocab, B = 128256, 110
    rng = np.random.default_rng(7)
    k = rng.integers(16, 25, size=B).tolist()
    T = sum(k) + B
    g = torch.Generator(device="cuda").manual_seed(7)
    logits = torch.randn(T, vocab, generator=g, device="cuda")
    tokens = torch.randint(0, vocab, (T,), generator=g, device="cuda", dtype=torch.int32)
    hit = torch.from_numpy(rng.random(T - 1) < 0.85).cuda()       # a third of the requests get past row 8
    best = logits.argmax(dim=1)
    tokens[1:] = torch.where(hit, best[:-1].to(torch.int32), tokens[1:])
    ws = sled.workspace(sled.sled_accept_workspace_bytes(B, T, vocab))
    a, t = _run(sled.GREEDY, k, vocab, logits, tokens, None, None, None, 0, ws=ws)
    assert _unwritten(ws) > T // 4
    tk, bt, row, want = tokens.cpu().numpy(), best.cpu().numpy(), 0, []
    for n in k:
        j = 0
        while j < n and tk[row + j + 1] == bt[row + j]:
            j += 1
        want.append((j, int(bt[row + j])))
        row += n + 1
    assert list(zip(a.tolist(), t.tolist())) == want
    assert sum(x > 8 for x, _ in want) > 10 and sum(x < 2 for x, _ in want) > 10


def test_a_few_long_requests_among_short_ones_are_scanned_in_parts():
    """20 requests of 16 drafts and 180 of one: 300 rows, 154 MB, lie behind row 2, and those of requests that end before are left out."""
    vocab, k = 128256, [1] * 200
    for i in range(0, 200, 10):
        k[i] = 16
    T = sum(k) + len(k)
    c = synth.accept_case(k, vocab, 1.0, seed=4, device="cuda")
    args = (sled.SAMPLE, k, vocab, c.logits, c.tokens, c.q, c.u_acc, c.u_smp, 0)
    ws = sled.workspace(sled.sled_accept_workspace_bytes(len(k), T, vocab))
    got = [x.tolist() for x in _run(*args, ws=ws)]
    assert _unwritten(ws) > 300          # of 8 statistics a row
    assert [x.tolist() for x in _run(*args, ws=sled.workspace(_stat_bytes(T, vocab)))] == got       # every row, in one launch
    assert 0 < sum(got[0]) < sum(k)

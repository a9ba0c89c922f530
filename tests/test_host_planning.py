"""Host-side planning of a verification step, through the C ABI, without a GPU.

Two choices are made on the host for every step: how the attention over requests of different lengths (Sec. 3.4: one
batch of heterogeneous requests) is cut into work items, and how many K slices each projection runs with.  Both are
exported as planning aids (sled_attention_partition, sled_projection_slices); here their contracts are checked:
the limits the header states, and that the partition never loses to the two simple rules it replaced."""
import heapq

import numpy as np
import pytest

from paper_2506_09397_amd import sled, synth

CUS = 256

# Steps of one layer of the large shapes that test_gpu_tile_rows.py runs, and what they are there for: per projection the K slices
# (unequal ones marked) and the rows of a workgroup.  Between them the projections in slices have both heights, equal and unequal.
LARGE_LAYER_CASES = [
    ("llama8b", 545, {"qkv": (2, False, 128), "o": (3, True, 128), "gu": (1, False, 192), "dn": (3, True, 128)}),
    ("llama8b", 700, {"qkv": (3, True, 128), "o": (2, False, 128), "gu": (1, False, 192), "dn": (5, True, 128)}),
    ("llama8b", 1300, {"qkv": (2, False, 192), "o": (1, False, 128), "gu": (1, False, 128), "dn": (4, False, 192)}),
    ("llama70b", 1030, {"qkv": (2, False, 192), "o": (2, False, 192), "gu": (1, False, 128), "dn": (5, True, 192)}),
]


def _projections(shape):
    s = synth.SHAPES[shape]
    heads = s.n_q_heads * s.head_dim
    return {"qkv": (heads + 2 * s.n_kv_heads * s.head_dim, s.d_model), "o": (s.d_model, heads), "gu": (2 * s.d_ffn, s.d_model), "dn": (s.d_model, s.d_ffn)}


def _items(n_pages, tgt, H):
    """sizes of the work items of one launch, in launch order (longest requests first, even split per request, the heads of a piece together)"""
    out = []
    for n in sorted(n_pages, reverse=True):
        pieces = -(-n // tgt)
        chunk = -(-n // pieces)
        sizes = [min(chunk, n - p0) for p0 in range(0, n, chunk)]
        assert len(sizes) == pieces
        out += [x for x in sizes for _ in range(H)]
    return out


def _makespan(n_pages, tgt, H):
    """when the last item ends, in pages: items go to the XCDs round robin in launch order and start as their CUs become free; 48 pages for an
    item's fixed part, 16 more where a request is split"""
    free = [[0] * (CUS // 8) for _ in range(8)]
    split = [-(-n // tgt) > 1 for n in sorted(n_pages, reverse=True) for _ in range(-(-n // tgt) * H)]
    for i, (pages, cut) in enumerate(zip(_items(n_pages, tgt, H), split)):
        t = heapq.heappop(free[i % 8])
        heapq.heappush(free[i % 8], t + pages + 48 + (16 if cut else 0))
    return max(max(x) for x in free)


def _pages(kind, shape):
    b = synth.draw_batch(kind, synth.SHAPES[shape].vocab, seed=0)
    return [-(-(int(L) + int(k) + 1) // 16) for L, k in zip(b.ctx_len, b.k)], synth.SHAPES[shape].n_kv_heads


@pytest.mark.parametrize("kind,shape", [("b16", "llama8b"), ("hetero64", "llama8b"), ("b32", "llama70b"), ("tiny4", "tiny_bf16")])
def test_partition_keeps_its_limits_on_the_benchmark_batches(kind, shape):
    n_pages, H = _pages(kind, shape)
    tgt, n_items = sled.sled_attention_partition(H, n_pages)
    sizes = _items(n_pages, tgt, H)
    assert n_items == len(sizes) and sum(sizes) == H * sum(n_pages)          # every page of every head exactly once
    longest = max(n_pages)
    assert 1 <= tgt <= longest
    for n in n_pages:
        pieces = -(-n // tgt)
        assert pieces <= 8
        if pieces > 1:
            assert n // pieces >= 16          # halves of at least 32 pages, split evenly
            assert tgt >= 32
    base = CUS * -(-len(n_pages) * H // CUS)
    assert n_items <= 4 * base


def test_partition_splits_the_long_requests_of_a_mixed_batch_and_leaves_an_even_batch_alone():
    n_pages, H = _pages("hetero64", "llama8b")
    tgt, n_items = sled.sled_attention_partition(H, n_pages)
    assert tgt < max(n_pages) and n_items > H * len(n_pages)      # the 8192-token request does not stay one item per head
    # the busiest CU's share: no worse than leaving every request whole
    assert max(_items(n_pages, tgt, H)) < max(n_pages)
    # 32 requests of one length on 8 heads: 256 equal items, nothing to gain from cutting them
    tgt, n_items = sled.sled_attention_partition(8, [100] * 32)
    assert (tgt, n_items) == (100, 256)
    # one long request alone: cut into the most items the limits allow (eight per head)
    tgt, n_items = sled.sled_attention_partition(8, [4096])
    assert n_items == 64 and tgt == 512
    # a request shorter than 32 pages is never cut
    tgt, n_items = sled.sled_attention_partition(8, [20, 31, 7])
    assert n_items == 24


def test_partition_on_random_batches():
    rng = np.random.default_rng(0)
    for _ in range(60):
        B = int(rng.integers(1, 97))
        H = int(rng.choice([1, 2, 8]))
        n_pages = [int(x) for x in np.exp(rng.uniform(np.log(1), np.log(600), size=B)).astype(int) + 1]
        tgt, n_items = sled.sled_attention_partition(H, n_pages)
        sizes = _items(n_pages, tgt, H)
        assert n_items == len(sizes) and sum(sizes) == H * sum(n_pages)
        assert all(-(-n // tgt) <= 8 for n in n_pages)
        assert all(n <= tgt or tgt >= 32 for n in n_pages)
        assert n_items <= 4 * CUS * -(-B * H // CUS)


@pytest.mark.parametrize("H,B,seed,others", [(16, 23, 87, (109, 145)), (24, 34, 17, (306, 544))])
def test_partition_plays_the_launch_through_in_its_own_order(H, B, seed, others):
    """Head counts and batches where pieces of a head side by side, an order the launch does not have, make another bound look best."""
    rng = np.random.default_rng(seed)
    rng.choice([3, 6, 12, 16, 24, 32]), rng.integers(2, 40)       # (how the batch was found)
    n_pages = [int(x) + 1 for x in np.exp(rng.uniform(0, np.log(600), size=B))]
    tgt, _ = sled.sled_attention_partition(H, n_pages)
    ends = {t: _makespan(n_pages, t, H) for t in others}
    assert len(set(ends.values())) == 2
    assert _makespan(n_pages, tgt, H) <= min(ends.values()), (tgt, ends)


def test_partition_rejects_bad_arguments():
    with pytest.raises(Exception):
        sled.sled_attention_partition(8, [0, 5])
    with pytest.raises(Exception):
        sled.sled_attention_partition(0, [5])


def test_projection_slices_of_the_benchmark_model():
    d, F, nqkv = 4096, 14336, (32 + 2 * 8) * 128
    # one block of rows (up to 128): the model's plan
    assert sled.sled_projection_slices(nqkv, d, 101) == (4, 8)
    assert sled.sled_projection_slices(d, d, 101) == (8, 16)
    assert sled.sled_projection_slices(d, F, 101) == (8, 16)
    assert sled.sled_projection_slices(2 * F, d, 101) == (1, 1)      # gate/up: enough column blocks, SwiGLU in the epilogue
    # three blocks of rows: whole rounds of 256 workgroups (24 x 3 x 3 = 216, 16 x 3 x 5 = 240)
    assert sled.sled_projection_slices(nqkv, d, 372)[0] == 3
    assert sled.sled_projection_slices(d, d, 372)[0] == 5
    assert sled.sled_projection_slices(d, F, 372)[0] == 5
    # one plan for weights of every width, whatever the height of a workgroup: partial sums count against rounds of blocks of 128 rows
    assert [sled.sled_projection_slices(d, K, 700)[0] for K in (d, F)] == [2, 5]
    assert [sled.sled_projection_slices(N, K, 129)[0] for N, K in ((nqkv, d), (d, d), (d, F))] == [5, 8, 8]
    for N, K in ((nqkv, d), (d, d), (d, F), (10240, 8192), (8192, 28672)):
        for T in (1, 33, 128, 129, 225, 372, 512, 1008, 2016, 4096):
            s, cap = sled.sled_projection_slices(N, K, T)
            assert 1 <= s <= cap and s <= K // 256        # every slice holds at least one trip of the stage loop
            if T <= 128:
                assert s == sled.sled_projection_slices(N, K, 1)[0]
                assert K % (256 * s) == 0                     # equal slices of whole trips of 16 k-steps: what the kernels of one block of rows assume
    with pytest.raises(Exception):
        sled.sled_projection_slices(100, 4096, 10)


@pytest.mark.parametrize("shape,T,want", LARGE_LAYER_CASES)
def test_the_large_layer_cases_have_the_slices_and_heights_they_are_there_for(shape, T, want):
    got = {}
    for name, (N, K) in _projections(shape).items():
        s = sled.sled_projection_slices(N, K, T)[0]
        got[name] = (s, (K // 128) % s != 0, sled.sled_projection_rows(N, K, T))      # K is dealt out in units of 128
    assert got == want


def test_rows_of_a_workgroup():
    d, F = 4096, 14336
    assert [sled.sled_projection_rows(d, d, T) for T in (1, 32, 33, 96, 97, 128)] == [32, 32, 64, 96, 128, 128]
    # 112 column blocks: 336 workgroups in two rounds at 128 rows, 224 in one at 192; four blocks of 128 fill two rounds as well
    assert [sled.sled_projection_rows(2 * F, d, T) for T in (129, 256, 257, 372, 384, 500)] == [128, 128, 192, 192, 192, 128]
    with pytest.raises(Exception):
        sled.sled_projection_rows(100, 4096, 10)

"""GPU parity of dsv_verify_attn where its work forms meet: row-tile counts
around the limits of the wave roles (one and two tiles split their dims over
the waves, three and more have waves of their own, twice over beyond four, at
G = 16 beyond eight or, at d = 64, four times over), with key counts around the 32-key stages of the ring
and the 16-token pages.  The bar is the attention bar of gpu_util."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

try:
    from gpu_util import assert_attn_close, run_attn, say
except Exception:  # pragma: no cover
    pass


def check(name, seed, ctx, qlens, hq, hkv, d):
    inp = W.make_attn_inputs(np.random.default_rng(seed), ctx_lens=ctx, qlens=qlens,
                             capacity=int(sum(qlens)) + 3, num_q_heads=hq, num_kv_heads=hkv,
                             head_dim=d, spare_pages=2)
    say("attn-tiles", name)
    ref = oracle.verify_attn(inp.q, inp.cu_qlens, inp.kv_pages, inp.page_table, inp.ctx_lens,
                             **inp.oracle_kwargs())
    assert_attn_close(run_attn(inp), ref, inp)


# contexts that end a stage, a page, or one key to either side of them
EDGES = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 97, 127, 129, 255, 300]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group,k", [
    (1, 16), (2, 8), (2, 9), (4, 4), (4, 5), (4, 8), (4, 9), (4, 12), (4, 16),
    (8, 8), (8, 9), (8, 10), (8, 11), (8, 15), (8, 16),
    (16, 1), (16, 2), (16, 3), (16, 8), (16, 9), (16, 15), (16, 16)])
def test_row_tiles(group, k, d):
    # 17 requests with k rows each: ceil(group * k / 16) row tiles
    check("G=%d k=%d d=%d" % (group, k, d), 100 * group + k, EDGES, [k] * len(EDGES),
          2 * group, 2, d)


@pytest.mark.parametrize("k", [4, 5, 12, 13])
@pytest.mark.parametrize("d", [64, 128])
def test_row_tiles_of_sixteen_heads(k, d):
    # four waves at d = 64: tiles of one, two and up to four to a wave
    check("G=16 k=%d d=%d" % (k, d), 1700 + k, EDGES, [k] * len(EDGES), 32, 2, d)


@pytest.mark.parametrize("group", [4, 8, 16])
def test_mixed_tiles_in_one_share_of_head_dim_64(group):
    rng = np.random.default_rng(64 + group)
    qlens = [int(k) for k in rng.integers(1, 17, size=48)]
    ctx = [int(c) for c in rng.integers(200, 2600, size=48)]
    check("G=%d d=64 mixed" % group, 107 + group, ctx, qlens, 4 * group, 4, 64)


@pytest.mark.parametrize("group", [8, 16])
def test_mixed_tiles_in_one_share(group):
    # stream-K shares that walk requests of every tile count
    rng = np.random.default_rng(group)
    qlens = [int(k) for k in rng.integers(1, 17, size=48)]
    ctx = [int(c) for c in rng.integers(200, 2600, size=48)]
    check("G=%d mixed" % group, 7 + group, ctx, qlens, 4 * group, 4, 128)


@pytest.mark.parametrize("hi", [60, 240])
@pytest.mark.parametrize("d,reqs,hkv", [(128, 65, 4), (128, 64, 4), (64, 33, 2), (64, 32, 2)])
def test_many_short_segments_of_sixteen_heads(d, reqs, hkv, hi):
    # to either side of the segment counts (256 and 64) at which a batch of sixteen heads
    # to a KV head changes its kernel, every tile count among the requests
    rng = np.random.default_rng(reqs + hi)
    qlens = [1 + i % 16 for i in range(reqs)]
    ctx = [int(c) for c in rng.integers(0, hi - 16, size=reqs)]
    check("G=16 d=%d %d x %d to %d" % (d, reqs, hkv, hi), 900 + reqs, ctx, qlens, 16 * hkv, hkv, d)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group,k", [(1, 16), (2, 16), (4, 8), (4, 16), (8, 16), (16, 4), (16, 16)])
@pytest.mark.parametrize("reqs,hkv", [(1, 2), (6, 8)])
def test_small_batch_pieces(reqs, hkv, group, k, d):
    # segments of two to nine blocks, about where the smallest batches begin to cut
    for blocks in (2, 3, 4, 5, 6, 9):
        ctx = [32 * blocks - k - i % 3 for i in range(reqs)]
        check("pieces G=%d k=%d d=%d %d x %d, %d blocks" % (group, k, d, reqs, hkv, blocks),
              31 * blocks + group, ctx, [k] * reqs, group * hkv, hkv, d)

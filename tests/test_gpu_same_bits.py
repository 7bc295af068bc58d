"""A head's attention output depends on its own blocking, lists and rows alone: what else
the call holds (heads of other blockings, more heads) must not change a bit of it.
"""
import numpy as np
import pytest
import torch

from paper_2608_03335_amd import spade as S

from . import _parity as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _lists(H, NB, seed):
    """Rows of 1 .. NB // 2 random blocks, ascending (device tensors, B = 1)."""
    rng = np.random.default_rng(seed)
    counts = rng.integers(1, max(2, NB // 2), size=(1, H, NB)).astype(np.int32)
    idx = np.zeros((1, H, NB, NB), np.int32)
    for r in np.ndindex(1, H, NB):
        idx[r][:counts[r]] = np.sort(rng.choice(NB, counts[r], replace=False))
    return torch.from_numpy(counts).to(DEV), torch.from_numpy(idx).to(DEV)


def _buffers(g, Q):
    ws = torch.empty(max(S.spade_attn_workspace_bytes(g), 1), dtype=torch.uint8, device=DEV)
    lse = torch.full(Q.shape[:3], float("nan"), dtype=torch.float32, device=DEV)
    return torch.full_like(Q, float("nan")), lse, ws


def _raster(g, Q, K, V, c, i):
    o, lse, ws = _buffers(g, Q)
    S.spade_sparse_attn_raster(g, Q, K, V, c, i, P.scale_of(g.d), o, lse, workspace=ws)
    return o, lse


def _same(a, b):
    return torch.equal(a.view(torch.int16 if a.dtype == torch.bfloat16 else torch.int32),
                       b.view(torch.int16 if b.dtype == torch.bfloat16 else torch.int32))


# The keys of the second blocking's rows are walked as one stream, the first's are not
# (its edge blocks along y waste 2% of the chunks); both have the same number of row tiles.
@pytest.mark.parametrize("d,grid,blocks", [
    (128, (4, 45, 32), ((2, 8, 8), (3, 5, 8))), (64, (4, 45, 32), ((2, 8, 8), (3, 5, 8))),
    (128, (6, 47, 72), ((3, 4, 8), (2, 5, 9))), (64, (35, 24, 24), ((16, 4, 4), (5, 6, 8)))],
    ids=str)
@pytest.mark.parametrize("swap", [False, True])
def test_multi_equals_own_blocking(d, grid, blocks, swap):
    print("multi against own blocking", d, grid, blocks, swap, flush=True)
    blocks = blocks[::-1] if swap else blocks
    H = 2
    geoms = [S.geom(1, H, d, *grid, *b) for b in blocks]
    Q, K, V = P.bf16_inputs(P.small_cfg(*grid, *blocks[0], d=d, H=H), seed=d)
    own = [_lists(H, g.NB, seed=g.NB) for g in geoms]
    o, lse, ws = _buffers(geoms[0], Q)
    S.spade_sparse_attn_raster_multi(
        geoms, [(h, own[h][0][:, h], own[h][1][:, h], 0, 0) for h in range(H)], Q, K, V,
        P.scale_of(d), o, lse, workspace=ws)
    for h, g in enumerate(geoms):
        ro, rl = _raster(g, Q, K, V, *own[h])
        assert _same(o[:, h], ro[:, h]) and _same(lse[:, h], rl[:, h]), (h, blocks[h])


def _blocked(g, Q, K, V, c, i):
    """Blocked attention and the inverse reorder; O only."""
    blk = [torch.empty((1, g.H, g.NB * g.BS, g.d), dtype=torch.bfloat16, device=DEV)
           for _ in range(3)]
    for x, xb in zip((Q, K, V), blk):
        S.spade_block_reorder(g, x, xb)
    ws = torch.empty(max(S.spade_attn_workspace_bytes(g), 1), dtype=torch.uint8, device=DEV)
    ob, o = torch.full_like(blk[0], float("nan")), torch.empty_like(Q)
    S.spade_block_sparse_attn(g, *blk, c, i, P.scale_of(g.d), ob, None, workspace=ws)
    S.spade_block_reorder(g, ob, o, inverse=True)
    return o


def _short_lists(H, NB, longest, seed):
    """Rows of 1 .. longest distinct blocks, ascending: steps of 1 .. NB // longest."""
    rng = np.random.default_rng(seed)
    steps = rng.integers(1, NB // longest + 1, size=(1, H, NB, longest))
    idx = np.zeros((1, H, NB, NB), np.int32)
    idx[..., :longest] = np.cumsum(steps, axis=3) - 1
    counts = rng.integers(1, longest + 1, size=(1, H, NB)).astype(np.int32)
    return torch.from_numpy(counts).to(DEV), torch.from_numpy(idx).to(DEV)


# Launches whose size decides the kernel: H heads of one call against one head alone. A
# ragged axis (the edge blocks' keys do not fill their chunks) and, last, none.
@pytest.mark.parametrize("d,grid,block,H", [
    (128, (16, 37, 64), (1, 8, 8), 13), (128, (16, 37, 64), (1, 8, 8), 6),
    (128, (16, 32, 80), (1, 8, 8), 13), (128, (9, 32, 56), (3, 4, 8), 25),
    (128, (4, 25, 62), (3, 5, 6), 38), (64, (9, 32, 56), (3, 4, 8), 25),
    (64, (8, 26, 40), (4, 6, 8), 13), (64, (6, 33, 40), (3, 7, 8), 13)], ids=str)
def test_many_heads_equal_one(d, grid, block, H):
    print("many heads against one", d, grid, block, H, flush=True)
    g, g1 = S.geom(1, H, d, *grid, *block), S.geom(1, 1, d, *grid, *block)
    Q, K, V = P.bf16_inputs(P.small_cfg(*grid, *block, d=d, H=H), seed=H)
    c, i = _short_lists(H, g.NB, 9, seed=H)
    o, lse = _raster(g, Q, K, V, c, i)
    mo, ml, ws = _buffers(g, Q)
    S.spade_sparse_attn_raster_multi([g], [(0, c[:, h], i[:, h], 0, 0) for h in range(H)], Q, K,
                                     V, P.scale_of(d), mo, ml, workspace=ws)
    assert _same(mo, o) and _same(ml, lse)
    assert _same(_blocked(g, Q, K, V, c, i), o)
    for h in (0, H // 2, H - 1):
        one = [x[:, h:h + 1].contiguous() for x in (Q, K, V, c, i)]
        ro, rl = _raster(g1, *one)
        assert _same(o[:, h:h + 1], ro) and _same(lse[:, h:h + 1], rl), h
        assert _same(_blocked(g1, *one), ro), h

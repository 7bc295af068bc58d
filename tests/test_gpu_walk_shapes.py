"""The attention walk on every block size, against the oracle on the same lists.

A row's kept keys are walked in chunks of 32, either chunk by chunk of each block or, where
that saves enough chunks, as one stream in which a chunk can span blocks; lists are staged
in segments (256 entries for blocks of up to 64 slots, 512 for 129..160, 1024 for the
others); launches of more than 256 work items are ranked, by one workgroup up to 1024
(batch, head) pairs and 24576 counts; the kernel with a loading wave takes 64-slot blocks
at d = 128 from 4096 work items and 608 blocks on, 65..96-slot ones that are not streamed
from 4096 items on (at d = 64 in the blocked form only) and 161..192-slot ones at d = 64
past 640 items. Each case sits on one of these edges. The tolerances are those of every
attention parity test (bf16 inputs and weights, fp32 accumulation).
"""
import numpy as np
import pytest
import torch

from oracle import spade_oracle as O
from paper_2608_03335_amd import spade as S

from . import _parity as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _lists(H, NB, lengths, seed):
    """Rows keep lengths[(i + 3 h) mod len] random blocks (clipped to NB), ascending."""
    rng = np.random.default_rng(seed)
    counts = np.zeros((1, H, NB), np.int32)
    idx = np.zeros((1, H, NB, NB), np.int32)
    for h in range(H):
        for i in range(NB):
            k = min(lengths[(i + 3 * h) % len(lengths)], NB)
            counts[0, h, i] = k
            idx[0, h, i, :k] = np.sort(rng.choice(NB, k, replace=False))
    return counts, idx


def _check(grid, block, d, H, lengths, raster, rows=None, heads=None):
    """Runs one layer and compares the query blocks `rows` (default all) of `heads`."""
    cfg = P.small_cfg(*grid, *block, d=d, H=H)
    og = P.geometry(cfg)
    g = S.geom(1, H, d, *grid, *block)
    NB, BS = g.NB, g.BS
    Q, K, V = P.bf16_inputs(cfg, seed=NB + d)
    counts, idx = _lists(H, NB, lengths, seed=NB)
    c, i = torch.from_numpy(counts).to(DEV), torch.from_numpy(idx).to(DEV)
    scale = P.scale_of(d)
    ws = torch.empty(max(S.spade_attn_workspace_bytes(g), 1), dtype=torch.uint8, device=DEV)
    lse = torch.full((1, H, g.N if raster else NB * BS), float("nan"), dtype=torch.float32,
                     device=DEV)
    o = torch.full_like(Q, float("nan"))
    if raster:
        S.spade_sparse_attn_raster(g, Q, K, V, c, i, scale, o, lse, workspace=ws)
    else:
        blk = [torch.empty((1, H, NB * BS, d), dtype=torch.bfloat16, device=DEV)
               for _ in range(3)]
        for x, xb in zip((Q, K, V), blk):
            S.spade_block_reorder(g, x, xb)
        ob = torch.full_like(blk[0], float("nan"))
        S.spade_block_sparse_attn(g, *blk, c, i, scale, ob, lse, workspace=ws)
        S.spade_block_reorder(g, ob, o, inverse=True)
    torch.cuda.synchronize()
    heads = list(range(H)) if heads is None else heads
    got = P.to_np64(o[:, heads])
    got_lse = lse[:, heads].cpu().numpy().astype(np.float64)
    if not raster:
        got_lse = got_lse[:, :, O.token_position(og)]
    cs, xs = counts[:, heads], idx[:, heads]
    wanted = [(0, h, r) for h in range(len(heads)) for r in (range(NB) if rows is None else rows)]
    full = [w for w in wanted if cs[w] > 0]
    ref_o, ref_l = P.oracle_attention_on_lists(*(P.to_np64(x[:, heads]) for x in (Q, K, V)), og,
                                               cs, xs, scale, rows=full)
    for w in wanted:
        if cs[w] == 0:
            toks = P.row_tokens(og, w[2])
            assert np.all(got[0, w[1], toks] == 0) and np.all(np.isneginf(got_lse[0, w[1], toks]))
    worst = P.compare_rows_raster(got, got_lse, ref_o, ref_l, og, full)
    print(f"max-abs {worst:.3e} over {len(full)} query blocks", flush=True)
    assert worst <= P.ATTN_MAX_ABS


LENGTHS = (0, 1, 2, 3, 4, 5, 7, 9, 12)


# (grid, block): one to eight row tiles; blocks that are multiples of 32 keys and blocks
# that are not, edge blocks of at least 32 keys and of fewer
@pytest.mark.parametrize("raster", [True, False], ids=["raster", "blocked"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grid,block", [
    ((5, 9, 10), (2, 4, 4)), ((7, 5, 9), (3, 2, 4)),
    ((3, 16, 21), (1, 8, 8)), ((7, 9, 13), (3, 4, 5)),
    ((7, 9, 17), (3, 4, 8)), ((5, 11, 19), (2, 5, 9)),
    ((9, 10, 16), (4, 4, 8)), ((8, 11, 20), (3, 5, 8)), ((6, 15, 20), (3, 5, 8)),
    ((8, 13, 20), (3, 6, 8)), ((6, 12, 20), (3, 6, 8)),
    ((9, 13, 17), (4, 6, 8)), ((9, 11, 19), (4, 5, 9)),
    ((9, 15, 17), (4, 7, 8)), ((7, 17, 19), (3, 8, 9)),
    ((9, 17, 17), (4, 8, 8)), ((11, 15, 15), (5, 7, 7))],
    ids=lambda x: "x".join(map(str, x)))
def test_walk_block_sizes(grid, block, d, raster):
    print("walk", grid, block, d, raster, flush=True)
    _check(grid, block, d, 2, LENGTHS, raster)


@pytest.mark.parametrize("d,block,n,lengths", [
    (64, (1, 4, 8), 520, (255, 256, 257, 511, 512, 513, 520)),
    (128, (1, 6, 10), 514, (256, 257, 512, 513, 514)),
    (128, (3, 6, 8), 514, (511, 512, 513, 514)), (64, (4, 5, 8), 514, (511, 512, 513)),
    (64, (2, 5, 7), 1026, (1023, 1024, 1025)), (64, (3, 4, 8), 1026, (1024, 1025))])
def test_list_segments(d, block, n, lengths):
    print("segments", d, block, n, flush=True)
    bt, bh, bw = block
    _check((bt * n - 1 if bt > 1 else n, bh, bw), block, d, 1, lengths, True,
           rows=range(len(lengths)))


@pytest.mark.parametrize("d,H,n", [(64, 4, 64), (128, 3, 86), (64, 192, 128), (64, 193, 128),
                                   (64, 1025, 2)])
def test_ranking_launches(d, H, n):
    print("ranking", d, H, n, flush=True)
    _check((n, 4, 8), (1, 4, 8), d, H, LENGTHS, True, heads=[0, 1, H - 1])


# 608, 608, 600 and 640 blocks per head (64 slots; the last grid is ragged along y); 168 of
# 96 slots; 110 of 90 slots, half of them of fewer than 32 keys; 50 of 192 and of 168 slots
@pytest.mark.parametrize("raster", [True, False], ids=["raster", "blocked"])
@pytest.mark.parametrize("d,H,grid,block", [
    (128, 6, (19, 32, 64), (1, 8, 8)), (128, 7, (19, 32, 64), (1, 8, 8)),
    (128, 7, (15, 40, 64), (1, 8, 8)), (128, 7, (16, 37, 64), (1, 8, 8)),
    (128, 24, (9, 32, 56), (3, 4, 8)), (128, 25, (9, 32, 56), (3, 4, 8)),
    (64, 24, (9, 32, 56), (3, 4, 8)), (64, 25, (9, 32, 56), (3, 4, 8)),
    (128, 37, (4, 25, 62), (3, 5, 6)), (128, 38, (4, 25, 62), (3, 5, 6)),
    (64, 12, (8, 26, 40), (4, 6, 8)), (64, 13, (8, 26, 40), (4, 6, 8)),
    (64, 13, (6, 33, 40), (3, 7, 8))], ids=str)
def test_loading_wave_threshold(d, H, grid, block, raster):
    print("loading wave", d, H, grid, block, raster, flush=True)
    NB = S.geom(1, H, d, *grid, *block).NB
    _check(grid, block, d, H, (3, 9, 30, 12, 0), raster, rows=range(0, NB, max(7, NB // 16)),
           heads=[0, H - 1])

"""The selection kernel's row groups (4 rows for 4 waves, 12 for 4, 16 for 8) give the
oracle's lists exactly, for every estimator, at both sides of each change of group.

The summaries are small whole numbers, even where an estimator halves them, so every
score is exact in fp64 whatever the order of its sum and ties are plentiful: kept sets
and counts must equal the oracle's, with no exemption. Sizes are (heads, blocks): the
4-row group takes launches of up to 256 items (1024 for the exact interval estimator,
`dsa2`), the 16-row group starts where two 12-row workgroups no longer fit in 160 KB:
above 729 blocks at d = 64 and 680 at d = 128 (723 there for `dsa`, 725 and 597 for `dsa2`).
"""
import numpy as np
import pytest
import torch

from oracle import spade_oracle as O
from paper_2608_03335_amd.pipeline import Scheme

from . import _parity as P
from .test_gpu_parity import _path

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("est,d,H,NB", [
    ("mean", 128, 2, 9), ("mean", 64, 4, 256), ("mean", 128, 4, 257), ("mean", 128, 1, 1024),
    ("mean", 64, 2, 641), ("mean", 128, 3, 680), ("mean", 128, 3, 681), ("mean", 128, 2, 1024),
    ("mean", 64, 2, 729), ("mean", 64, 2, 730), ("mean", 64, 2, 1024),
    ("dsa", 64, 3, 65), ("dsa", 128, 4, 253), ("dsa", 128, 5, 253), ("dsa", 128, 2, 680),
    ("dsa", 128, 2, 681), ("dsa", 128, 2, 723),
    ("dsa", 128, 2, 724), ("dsa", 128, 2, 1021), ("dsa", 64, 2, 530), ("dsa", 64, 2, 729),
    ("dsa", 64, 2, 730),
    ("dsa2", 64, 1, 1), ("dsa2", 128, 4, 65), ("dsa2", 128, 5, 1024), ("dsa2", 64, 4, 1021),
    ("dsa2", 64, 5, 1021), ("dsa2", 128, 17, 251), ("dsa2", 128, 9, 513), ("dsa2", 128, 7, 597),
    ("dsa2", 128, 7, 598), ("dsa2", 64, 6, 725), ("dsa2", 64, 6, 726)])
def test_row_groups_exact(est, d, H, NB):
    cfg = P.small_cfg(1, 1, NB, 1, 1, 1, d=d, H=H)
    print("row groups", est, d, H, NB, flush=True)
    rng = np.random.default_rng(NB + H)
    topk = max(1, NB // 7)
    p = _path(cfg, virtual=True, scheme=Scheme(est, "topk", topk=topk))
    shape = (1, H, NB, d)
    scale = P.scale_of(d)
    if est == "mean":
        q, k = (rng.integers(-2, 3, shape).astype(np.float64) for _ in range(2))
        dst, src, s = (p.qbar, p.kbar), (q, k), O.block_scores(q, k, scale)
    else:
        lo = [2 * rng.integers(-3, 4, shape) for _ in range(2)]
        hi = [x + 4 * rng.integers(0, 2, shape) for x in lo]
        src = [x.astype(np.float64) for x in (hi[0], lo[0], hi[1], lo[1])]
        f = O.dsa_scores if est == "dsa" else O.dsa2_scores
        dst, s = p.ext, f(*src, scale)
    for t, x in zip(dst, src):
        t.copy_(torch.from_numpy(x))
    p.counts.fill_(-7)
    p.select()
    torch.cuda.synchronize()
    c_o, i_o = O.select(s, "topk", topk=topk)
    c_g, i_g = p.counts.cpu().numpy(), p.indices.cpu().numpy()
    assert np.array_equal(c_g, c_o)
    assert np.array_equal(i_g[..., :topk], i_o[..., :topk])

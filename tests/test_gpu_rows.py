"""The ascending order of the GPU planner's task rows, for every row length
class of its sorter (up to 64, 128, 256, 512 and 1024 values in a wave's
registers, longer ones by a workgroup), against the host planner."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2107_14008_amd import binding as B

pytestmark = pytest.mark.gpu

SIZES = (30, 63, 64, 65, 100, 128, 129, 250, 257, 500, 513, 1000, 1030, 1100)


def clumps(seed):
    """Clumps of SIZES particles, each within r_cut of itself only: with one
    particle per leaf a row holds about as many tasks as its clump has
    particles."""
    rng = np.random.default_rng(seed)
    at = [(x, y, 5.0) for x in np.arange(3.0, 40.0, 8.0) for y in np.arange(3.0, 40.0, 8.0)]
    pos = np.concatenate([np.array(c) + rng.normal(0, 0.05, (n, 3)) for c, n in zip(at, SIZES)])
    return pos[rng.permutation(len(pos))]


@pytest.mark.parametrize("row_lds", [None, "64"])
def test_rows_of_every_length(row_lds, monkeypatch):
    if row_lds is not None:
        monkeypatch.setenv("PMFMM_ROW_LDS", row_lds)
    pos = clumps(11)
    m = np.ones(len(pos))
    par = dict(box=40.0, r_s=0.6, r_cut=2.7, max_leaf=1, order=-1, theta=0.0)
    host = B.Context(**par)
    host.plan(pos, m)
    H = host.lists()
    bins = np.histogram(np.diff(H["p2p_row"]), [2, 65, 129, 257, 513, 1025, 1 << 20])[0]
    assert (bins > 0).all(), bins
    print(f"case: gpu plan rows of {bins} (row lds {row_lds})", flush=True)
    ctx = B.Context(planner=0, **par)
    ctx.build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"))
    L = ctx.lists()
    for k in ("perm", "p2p_row", "p2p_j", "p2p_shift"):
        assert np.array_equal(L[k], H[k]), k

"""The work-item cut and the persistent launch's queue: every schedule gives
the same forces, and the automatic cut follows its rule."""

import math

import numpy as np
import pytest

from paper_2107_14008_amd import binding as B
from paper_2107_14008_amd import inputs


def _auto_chunk(n_tasks, n_leaves):
    """The rule of plan.h: about sqrt(tasks) / 56 tasks per item, 2 to 32, and
    never more than 32,768 items below 32."""
    if n_leaves >= 32768:
        return 32
    least = -(-n_tasks // (32768 - n_leaves))
    return min(32, max(2, least, int(math.sqrt(n_tasks) / 56.0 + 0.5)))


@pytest.mark.parametrize("n_side,max_leaf", [(4, 64), (9, 8), (16, 64), (24, 32), (24, 2)])
def test_automatic_cut_of_the_host_plan(n_side, max_leaf):
    w = inputs.clustered_small(12 if n_side < 12 else n_side, 3, max_leaf=max_leaf, order=-1)
    ctx = B.Context(box=w.box, r_s=w.r_s, r_cut=w.r_cut, max_leaf=max_leaf, order=-1)
    n = n_side ** 3
    ctx.plan(w.pos[:n], w.mass[:n])
    L = ctx.lists()
    rows = np.diff(L["p2p_row"])
    chunk = _auto_chunk(int(L["n_p2p"]), int(L["n_leaves"]))
    assert L["n_items"] == int(np.sum(-(-rows // chunk)))
    assert chunk == 32 or L["n_items"] <= 32768


@pytest.mark.gpu
@pytest.mark.parametrize("form", [dict(precision=B.PMFMM_FP32, trunc=B.TRUNC_R2, table_size=64,
                                       table_level=2),
                                  dict(precision=B.PMFMM_FP32, trunc=B.TRUNC_TABLE,
                                       table_size=512, table_level=2),
                                  dict(precision=B.PMFMM_FP64)])
@pytest.mark.parametrize("n", [700, 13 ** 3, 20 ** 3])
def test_every_launch_shape_gives_the_same_bits(form, n):
    """Grids below, at and above the eight queue segments, fewer and more
    waves than items, rows longer than the 64 tasks read ahead: bit for bit
    the forces of the default launch at one work-item size."""
    import torch
    w = inputs.clustered_small(20, 11, max_leaf=64, order=-1)
    pos = torch.tensor(w.pos[:n], device="cuda")
    mass = torch.tensor(w.mass[:n], device="cuda")
    wv = torch.tensor(inputs.cotangent(n, 5), device="cuda")
    for chunk in (1, 5, 1000):
        want = None
        for wg, grid in ((0, 0), (1, 1), (4, 7), (2, 8), (4, 9), (1, 40), (4, 3000)):
            print(f"case: {n} particles, chunk {chunk}, wg {wg}, grid {grid}", flush=True)
            ctx = B.Context(box=w.box, r_s=w.r_s, r_cut=w.r_cut, max_leaf=64, order=-1,
                            chunk=chunk, wg_waves=wg, grid_wgs=grid, **form)
            ctx.build(pos, mass)
            out = torch.empty((n, 3), dtype=torch.float64, device="cuda")
            gp, gm = torch.empty_like(out), torch.empty(n, dtype=torch.float64, device="cuda")
            ctx.forward(out)
            ctx.adjoint(wv, gp, gm)
            got = [t.cpu().numpy() for t in (out, gp, gm)]
            ctx.close()
            want = want or got
            assert all(np.array_equal(a, b) for a, b in zip(got, want))


@pytest.mark.gpu
@pytest.mark.parametrize("form", [dict(precision=B.PMFMM_FP32, trunc=B.TRUNC_R2, table_size=64,
                                       table_level=2),
                                  dict(precision=B.PMFMM_FP32, trunc=B.TRUNC_TABLE,
                                       table_size=512, table_level=2),
                                  dict(precision=B.PMFMM_FP32, trunc=B.TRUNC_TABLE,
                                       table_size=4096, table_level=4),
                                  dict(precision=B.PMFMM_FP32), dict(precision=B.PMFMM_FP64)])
@pytest.mark.parametrize("max_leaf", [16, 32])
def test_workgroup_size_leaves_small_leaves_bits_alone(form, max_leaf):
    """Leaves of at most 32, whose lanes may be split over the sources: the
    choice of that form, which adds in another order, must not hang on the
    workgroup's size, whatever the table's size leaves of a CU's LDS."""
    import torch
    n = 16 ** 3
    w = inputs.clustered_small(16, 7, max_leaf=max_leaf, order=-1)
    pos, mass = torch.tensor(w.pos, device="cuda"), torch.tensor(w.mass, device="cuda")
    want = None
    for wg in (0, 1, 2, 4, 8, 16):
        print(f"case: leaves of {max_leaf}, {form}, wg {wg}", flush=True)
        ctx = B.Context(box=w.box, r_s=w.r_s, r_cut=w.r_cut, max_leaf=max_leaf, order=-1, wg_waves=wg,
                        **form)
        ctx.build(pos, mass)
        out = torch.empty((n, 3), dtype=torch.float64, device="cuda")
        ctx.forward(out)
        got = out.cpu().numpy()
        ctx.close()
        want = got if want is None else want
        assert np.array_equal(got, want)

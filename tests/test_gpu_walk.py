"""The dual walk sized by the build before it, where that build's frontiers
were another size: a spread-out set, then a clump whose frontiers outgrow the
walk's first workgroup, and back, each against the host planner."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2107_14008_amd import binding as B

pytestmark = pytest.mark.gpu

PAR = dict(box=20.0, r_s=0.4, r_cut=1.8, max_leaf=32)


def spread(rng, n):
    return rng.uniform(0, 20.0, (n, 3))


def clump(rng, n):
    return 10.0 + rng.uniform(-0.5, 0.5, (n, 3))


# 2,000 particles: 64 leaves and at most 2,080 pairs of them in the clump,
# more than one workgroup's threads; 60,000: frontiers on both sides of the
# switch to the larger workgroups.
@pytest.mark.parametrize("n, order, theta", [(500, -1, 0.0), (2000, -1, 0.0), (2000, 2, 0.5), (60000, -1, 0.0)])
def test_frontiers_of_another_size(n, order, theta):
    rng = np.random.default_rng(n)
    ctx = B.Context(planner=0, order=order, theta=theta, **PAR)
    m = np.ones(n)
    for k, make in enumerate((spread, spread, clump, clump, spread) if n < 10000 else (clump, spread, spread)):
        if n >= 10000 and make is clump:
            pos = np.concatenate([clump(rng, n // 20), spread(rng, n - n // 20)])
        else:
            pos = make(rng, n)
        print(f"case: gpu walk n {n} order {order} build {k}", flush=True)
        ctx.build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"))
        L = ctx.lists()
        host = B.Context(order=order, theta=theta, **PAR)
        host.plan(pos, m)
        H = host.lists()
        for key in ("perm", "p2p_row", "p2p_j", "p2p_shift", "m2l_row", "m2l_src", "m2l_shift"):
            assert np.array_equal(L[key], H[key]), (k, key)


def test_more_roots_than_threads():
    """80 boxes: the 14 root pairs of each are more than the first workgroup
    takes.  Against each box alone: the same pairs in another order, so sums of
    at most n = 200 terms, each rounded up to n times at the size of the
    largest, about the largest force: n^2 2^-52 of that."""
    rng = np.random.default_rng(80)
    n, nbox = 200, 80
    par = dict(box=4.0, r_s=0.3, r_cut=1.2, max_leaf=16, order=-1, theta=0.0, G=1.0)
    pos = rng.uniform(0, 4.0, (nbox * n, 3))
    m = rng.uniform(0.5, 1.0, nbox * n)
    dpos, dm = torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda")
    ctx = B.Context(planner=0, **par)
    got = torch.empty_like(dpos)
    for k in range(2):                       # the second build is sized by the first
        print(f"case: gpu walk {nbox} boxes build {k}", flush=True)
        ctx.build_batch([B.make_params(**par)] * nbox, [n] * nbox, dpos, dm)
        ctx.forward(got)
        for b in (0, 37, nbox - 1):
            one = B.Context(planner=0, **par)
            s = slice(b * n, (b + 1) * n)
            one.build(dpos[s].contiguous(), dm[s].contiguous())
            want = torch.empty_like(dpos[s])
            one.forward(want)
            err = (got[s] - want).abs().max().item()
            assert err <= n * n * 2.0 ** -52 * want.abs().max().item(), (b, err)

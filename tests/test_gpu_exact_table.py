"""Float64 exact pair force from its segment table: single pairs over every
octave of the table, its ends and the cutoffs on both sides of its range."""

import numpy as np
import pytest

from paper_2107_14008_amd import binding as B

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
mpmath = pytest.importorskip("mpmath")


def _pairs(xc, seed, mass_ratio):
    """512 isolated pairs on an 8^3 grid of nodes 12.5 apart, r_cut = 5, with
    separations over 24 octaves of r^2 down from just inside the cutoff and
    at the table's octave edges y = 2^e."""
    rng = np.random.default_rng(seed)
    r_cut = 5.0
    r_s = r_cut / (2.0 * xc)
    y = np.concatenate([xc * xc * 2.0 ** -rng.uniform(0, 24, 440),
                        2.0 ** np.arange(-20, 3), np.nextafter(2.0 ** np.arange(-20, 3), 0),
                        xc * xc * (1 - 1e-9 * np.arange(1, 27))])
    r = 2.0 * r_s * np.sqrt(y[:512])
    r = np.where(r < r_cut, r, 0.5 * r_cut)
    g = (np.arange(8) + 0.5) * 12.5
    c = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    v = rng.standard_normal((512, 3))
    v /= np.linalg.norm(v, axis=1)[:, None]
    pos = np.concatenate([c, c + r[:, None] * v])
    mass = np.concatenate([np.full(512, 1.0), np.full(512, mass_ratio)])
    return pos, mass, r_s, r_cut


@pytest.mark.parametrize("xc", [0.4, 2.25, 3.0, 3.2])
@pytest.mark.parametrize("mass_ratio", [1.0, 0.37])
def test_single_pairs_against_forty_digits(xc, mass_ratio):
    # tolerance: r^2 and y carry about three roundings (3.3e-16), which the
    # slope |d ln F / d ln y| <= 1.5 + x_c^2 multiplies; T, the products and
    # the sums add at most 2e-15
    tol = (1.5 + xc * xc) * 3.4e-16 + 2e-15
    pos, mass, r_s, r_cut = _pairs(xc, 3, mass_ratio)
    print(f"case: single pairs, x_c {xc}, mass ratio {mass_ratio}", flush=True)
    ctx = B.Context(box=100.0, r_s=r_s, r_cut=r_cut, max_leaf=7, order=-1)
    ctx.build(torch.tensor(pos, device="cuda"), torch.tensor(mass, device="cuda"))
    out = torch.empty((1024, 3), dtype=torch.float64, device="cuda")
    ctx.forward(out)
    got = out.cpu().numpy()
    mpmath.mp.dps = 40
    worst = 0.0
    for k in range(512):
        d = [mpmath.mpf(float(pos[k + 512, a])) - mpmath.mpf(float(pos[k, a])) for a in range(3)]
        # the definition's displacement is the rounded float64 difference
        d = [mpmath.mpf(float(x)) for x in d]
        r2 = d[0] ** 2 + d[1] ** 2 + d[2] ** 2
        r = mpmath.sqrt(r2)
        if abs(r / r_cut - 1) < 1e-14:
            continue
        x = r / (2 * mpmath.mpf(r_s))
        t = mpmath.erfc(x) + 2 * x / mpmath.sqrt(mpmath.pi) * mpmath.exp(-x * x)
        a = float(t / r2) if r < r_cut else 0.0
        for i, m in ((k, mass_ratio), (k + 512, 1.0)):
            e = abs(np.linalg.norm(got[i]) - m * a)
            worst = max(worst, e / (m * a) if a else e)
    assert worst <= tol, (worst, tol)


@pytest.mark.parametrize("max_leaf", [32, 64])
@pytest.mark.parametrize("mass_ratio", [1.0, 0.37])
@pytest.mark.parametrize("xc,y0", [(2.25, 4.0), (3.0, 8.0)])
def test_outer_shell_in_small_and_full_leaves(xc, y0, mass_ratio, max_leaf):
    """The pairs of the table's last rows, y from y0 to the cutoff, in leaves
    of 32 (the form that splits a leaf's lanes) and of 64 (one mass or several
    to a leaf), some of them across the box's faces."""
    tol = (1.5 + xc * xc) * 3.4e-16 + 2e-15     # as above
    rng = np.random.default_rng(29)
    r_cut = 5.0
    r_s = r_cut / (2.0 * xc)
    y = rng.uniform(y0, xc * xc * (1 - 1e-9), 512)
    y[:16] = 8.375 if y0 == 8.0 else 4.3126      # the float32 t^4 term's worst
    y[:16] += rng.uniform(-1e-3, 1e-3, 16)
    r = 2.0 * r_s * np.sqrt(y)
    g = np.arange(8) * 12.5 + 10.0
    c = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    # into the positive octant: the particles of different pairs stay 7.5 apart
    v = np.abs(rng.standard_normal((512, 3)))
    v /= np.linalg.norm(v, axis=1)[:, None]
    pos = np.concatenate([c, c + r[:, None] * v]) % 100.0
    mass = np.concatenate([np.full(512, 1.0), np.full(512, mass_ratio)])
    print(f"case: outer shell, x_c {xc}, mass ratio {mass_ratio}, leaves of {max_leaf}", flush=True)
    ctx = B.Context(box=100.0, r_s=r_s, r_cut=r_cut, max_leaf=max_leaf, order=-1)
    ctx.build(torch.tensor(pos, device="cuda"), torch.tensor(mass, device="cuda"))
    assert (np.diff(np.append(ctx.lists()["leaf_first"], 1024)) == max_leaf).all()
    out = torch.empty((1024, 3), dtype=torch.float64, device="cuda")
    ctx.forward(out)
    got = out.cpu().numpy()
    d = pos[512:] - pos[:512]
    assert (np.abs(d) > 50).any()
    d = np.where(d > 50, d - 100.0, np.where(d < -50, d + 100.0, d))
    mpmath.mp.dps = 40
    worst = 0.0
    for k in range(512):
        r2 = sum(mpmath.mpf(float(a)) ** 2 for a in d[k])
        x = mpmath.sqrt(r2) / (2 * mpmath.mpf(r_s))
        t = mpmath.erfc(x) + 2 * x / mpmath.sqrt(mpmath.pi) * mpmath.exp(-x * x)
        a = float(t / r2)
        for i, m in ((k, mass_ratio), (k + 512, 1.0)):
            worst = max(worst, abs(np.linalg.norm(got[i]) - m * a) / (m * a))
    assert worst <= tol, (worst, tol)


@pytest.mark.parametrize("xc", [0.4, 2.25, 3.0])
@pytest.mark.parametrize("mass_ratio", [1.0, 0.37])
def test_full_leaves_agree_with_small_ones_in_every_octave(xc, mass_ratio):
    """The pairs of the first test in leaves of 64 (one mass to a leaf, or
    several) against leaves of 7, whose kernel splits a leaf's lanes: one
    lookup, then at most four roundings of the products each (9e-16)."""
    pos, mass, r_s, r_cut = _pairs(xc, 3, mass_ratio)
    got = []
    for max_leaf, largest in ((7, 4), (64, 64)):
        print(f"case: single pairs, x_c {xc}, mass ratio {mass_ratio}, leaves of {max_leaf}", flush=True)
        ctx = B.Context(box=100.0, r_s=r_s, r_cut=r_cut, max_leaf=max_leaf, order=-1)
        ctx.build(torch.tensor(pos, device="cuda"), torch.tensor(mass, device="cuda"))
        assert np.diff(np.append(ctx.lists()["leaf_first"], 1024)).max() == largest
        out = torch.empty((1024, 3), dtype=torch.float64, device="cuda")
        ctx.forward(out)
        got.append(out.cpu().numpy())
    d = np.linalg.norm(got[0] - got[1], axis=1)
    assert (d <= 1e-15 * np.linalg.norm(got[0], axis=1)).all()

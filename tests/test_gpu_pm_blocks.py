"""Block deposit of the long-range mesh: meshes with full, ragged and single
blocks, chunks of one block, particles on faces and outside the box, against
the plain numpy mesh force."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pm
from paper_2107_14008_amd import binding as B
from paper_2107_14008_amd import inputs

pytestmark = pytest.mark.gpu

BOX = 100.0
N = 600_000        # enough particles for the block form up to 130^3


def _positions(kind):
    rng = np.random.default_rng(8)
    x = rng.uniform(0, BOX, (N, 3))
    if kind == "clump":            # one block with many chunks
        x[:40000] = 37.0 + rng.normal(0, 0.4, (40000, 3))
    if kind == "faces":            # on nodes, at the box edge and beyond it
        x[:4000] = np.round(x[:4000] / 12.5) * 12.5
        x[4000:8000] += BOX * rng.integers(-2, 3, (4000, 3))
        x[8000:8010] = np.nextafter(BOX, 0.0)
    return x


@pytest.mark.parametrize("kind,n_pm", [("uniform", 64), ("clump", 64), ("faces", 32), ("faces", 66),
                                       ("clump", 100), ("uniform", 130), ("uniform", 6)])
def test_block_deposit_matches_the_oracle_mesh(kind, n_pm):
    x = _positions(kind)
    m = np.random.default_rng(9).uniform(0.5, 1.5, N) / N
    r_s = 1.2 * BOX / n_pm
    print(f"case: block deposit, {kind}, {n_pm}^3", flush=True)
    ref = pm.long_range_accel(inputs.wrap(x, BOX), m, BOX, r_s, n_pm)
    ctx = B.Context(box=BOX, r_s=r_s, r_cut=min(4.5 * r_s, 49.0))
    pos, mass = torch.tensor(x, device="cuda"), torch.tensor(m, device="cuda")
    out = torch.empty_like(pos)
    # the second and third call find the counts cleared by the one before; a
    # smaller set in between takes the direct form
    for k in range(3):
        ctx.long_range(n_pm, pos, mass, out)
        got = out.cpu().numpy()
        # the mesh test's own bound: atomics and FFT rounding, 1e-11 of the
        # largest acceleration
        assert np.abs(got - ref).max() <= 1e-11 * np.abs(ref).max()
        if k == 0:
            small = pos[:500].contiguous()
            ctx.long_range(n_pm, small, mass[:500].contiguous(), torch.empty_like(small))

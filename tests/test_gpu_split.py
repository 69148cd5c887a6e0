"""Leaves of few targets in launches with an item per wave: the pair forms that
give a leaf's idle lanes every second or fourth source, around the leaf sizes
where that changes, against brute force."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import direct, metrics
from paper_2107_14008_amd import binding as B

pytestmark = pytest.mark.gpu

FORMS = {
    "fp64": dict(precision=B.PMFMM_FP64, trunc=B.TRUNC_EXACT),
    "fp32": dict(precision=B.PMFMM_FP32, trunc=B.TRUNC_EXACT),
    "fp32_table": dict(precision=B.PMFMM_FP32, trunc=B.TRUNC_TABLE, table_size=512, table_level=2),
    "fp32_r2": dict(precision=B.PMFMM_FP32, trunc=B.TRUNC_R2, table_size=64, table_level=2),
}


# 64 leaves of `count` particles each (an even split at every cell).  Bounds:
# float64, the sums of test_gpu_batch.py; float32, its bounds too.
@pytest.mark.parametrize("count", [1, 2, 15, 16, 17, 31, 32, 33])
@pytest.mark.parametrize("form", list(FORMS))
def test_small_leaves(form, count):
    rng = np.random.default_rng(count)
    n, L, r_s = 64 * count, 8.0, 0.45
    pos = rng.uniform(0, L, (n, 3))
    pos[: n // 4] = (pos[: n // 4] - 4.0) * 0.2        # a clump over the box's corner
    pos %= L
    mass = rng.uniform(0.5, 1.0, n) if count % 2 else np.full(n, 0.7)
    print(f"case: split leaves of {count} {form}", flush=True)
    ctx = B.Context(box=L, r_s=r_s, r_cut=4.5 * r_s, max_leaf=count, order=-1, theta=0.0, **FORMS[form])
    ctx.build(torch.tensor(pos, device="cuda"), torch.tensor(mass, device="cuda"))
    assert (np.diff(np.append(ctx.lists()["leaf_first"], n)) == count).all()
    out = torch.empty((n, 3), dtype=torch.float64, device="cuda")
    ctx.forward(out)
    ref, _ = direct.brute_force(pos, mass, L, r_s, 4.5 * r_s)
    s = metrics.error_summary(out.cpu().numpy(), ref)
    if form == "fp64":
        assert s["max"] <= 1e-12, s
    else:
        assert s["median"] <= 1e-5 and s["p999"] <= 1e-4, s

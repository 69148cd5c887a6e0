"""The schedule autotuner picks one of its candidates, applies it, and the
forces stay within tolerance of the oracle for every schedule."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import direct, metrics
from paper_2107_14008_amd import binding as B
from paper_2107_14008_amd import inputs, tune

pytestmark = pytest.mark.gpu


def test_autotune_batch(tmp_path):
    boxes = inputs.batch_64(n_box=4, lo=16, hi=24)
    per_box = [B.make_params(box=w.box, r_s=w.r_s, r_cut=w.r_cut,
                             max_leaf=w.max_leaf, order=-1, theta=0.0)
               for w in boxes]
    counts = [len(w.mass) for w in boxes]
    pos = torch.tensor(np.concatenate([w.pos for w in boxes]), device="cuda")
    mass = torch.tensor(np.concatenate([w.mass for w in boxes]), device="cuda")
    ctx = B.Context(precision=B.PMFMM_FP32, trunc=B.TRUNC_TABLE, table_size=512,
                    table_level=2)
    ctx.build_batch(per_box, counts, pos, mass)
    out = torch.empty((sum(counts), 3), dtype=torch.float64, device="cuda")
    cands = [(0, 4, 0), (8, 2, 0), (1 << 20, 8, 0), (16, 16, 64)]
    cache = str(tmp_path / "tune.json")
    best, res = tune.autotune(ctx, out, cands=cands, repeats=2, cache_path=cache)
    assert (best["chunk"], best["wg_waves"], best["grid_wgs"]) in cands
    assert len(res) == len(cands)
    again, res2 = tune.autotune(ctx, out, cache_path=cache)   # from the cache
    assert res2 == {} and again["chunk"] == best["chunk"]
    ctx.forward(out)
    torch.cuda.synchronize()
    acc = out.cpu().numpy()
    p0 = 0
    for w, n in zip(boxes, counts):
        ref, _ = direct.brute_force(w.pos, w.mass, w.box, w.r_s, w.r_cut)
        s = metrics.error_summary(acc[p0:p0 + n], ref)
        assert s["median"] <= 1e-5 and s["p999"] <= 1e-4
        p0 += n


def test_autotune_default_candidates_through_the_abi(tmp_path):
    """pmfmm_autotune with the library's 24 default schedules on a float64
    exact context: the schedules with more than 4 waves per workgroup are
    skipped (that form runs at most 4), the winner is among the timed ones,
    it is applied, and a second call takes it from the cache file."""
    w = inputs.clustered_small(16, 9)
    ctx = B.Context(box=w.box, r_s=w.r_s, r_cut=w.r_cut, max_leaf=64, order=-1,
                    precision=B.PMFMM_FP64)
    ctx.build(torch.tensor(w.pos, device="cuda"), torch.tensor(w.mass, device="cuda"))
    out = torch.empty((len(w.mass), 3), dtype=torch.float64, device="cuda")
    ref = torch.empty_like(out)
    ctx.forward(ref)
    cache = str(tmp_path / "tune.txt")
    best, timed = ctx.autotune(out, repeats=1, cache_path=cache)
    assert len(timed) == 24
    ran = [r for r in timed if r["p2p_ms"] >= 0]
    assert len(ran) == 12 and all(r["wg_waves"] <= 4 for r in ran)
    assert (best["chunk"], best["wg_waves"]) in [(r["chunk"], r["wg_waves"]) for r in ran]
    assert best["p2p_ms"] == min(r["p2p_ms"] for r in ran)
    assert (ctx.params.chunk, ctx.params.wg_waves) == (best["chunk"], best["wg_waves"])
    assert open(cache).read().count("\n") == 1
    again, timed2 = ctx.autotune(out, cache_path=cache)
    assert timed2 == []
    assert [again[k] for k in ("chunk", "wg_waves", "grid_wgs")] == \
        [best[k] for k in ("chunk", "wg_waves", "grid_wgs")]
    assert abs(again["p2p_ms"] - best["p2p_ms"]) <= 1e-6      # kept to 6 decimals
    ctx.forward(out)
    torch.cuda.synchronize()
    # workgroup size and grid leave the result bitwise alone; the work-item
    # size regroups the float64 sums (rounding only)
    a, b = out.cpu().numpy(), ref.cpu().numpy()
    if best["chunk"] == 0:
        assert np.array_equal(a, b)
    assert np.max(np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)) <= 1e-12


@pytest.mark.parametrize("form,ran_per_chunk", [(dict(precision=B.PMFMM_FP64), 2),
                                                (dict(precision=B.PMFMM_FP64, trunc=B.TRUNC_R2,
                                                      table_size=64, table_level=6), 4)])
def test_schedules_of_one_launch_are_timed_once(form, ran_per_chunk):
    """The forms of the built-in float64 table run 16 waves whatever is asked:
    schedules that differ in wg_waves alone are one launch and have one time."""
    w = inputs.clustered_small(16, 9)
    ctx = B.Context(box=w.box, r_s=w.r_s, r_cut=w.r_cut, max_leaf=64, order=-1, **form)
    ctx.build(torch.tensor(w.pos, device="cuda"), torch.tensor(w.mass, device="cuda"))
    out = torch.empty((len(w.mass), 3), dtype=torch.float64, device="cuda")
    _, timed = ctx.autotune(out, repeats=1)
    times = {}
    for r in timed:
        if r["p2p_ms"] >= 0:
            times.setdefault(r["chunk"], []).append(r["p2p_ms"])
    assert len(times) == 6
    assert all(len(t) == ran_per_chunk and len(set(t)) == 1 for t in times.values()), times


def test_cached_schedule_is_of_the_kernel_that_runs(tmp_path):
    """A schedule tuned for the built-in float64 table is not taken for the
    polynomial form of a wider cutoff, nor one of full leaves for small ones,
    in plans of one coarse size."""
    rng = np.random.default_rng(4)
    n, box, r_s = 512, 100.0, 3.0
    pos = torch.tensor(rng.uniform(0, box, (n, 3)), device="cuda")
    mass = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    out = torch.empty((n, 3), dtype=torch.float64, device="cuda")
    cache = str(tmp_path / "tune.txt")
    for k, (reach, leaf) in enumerate([(4.5, 64), (7.0, 64), (4.5, 32), (7.0, 32)]):
        ctx = B.Context(box=box, r_s=r_s, r_cut=reach * r_s, max_leaf=leaf, order=-1,
                        precision=B.PMFMM_FP64)
        ctx.build(pos, mass)
        for timed_now in (True, False):       # the second time from the cache
            _, timed = ctx.autotune(out, cands=[(0, 2, 0), (0, 4, 0)], repeats=1, cache_path=cache)
            assert (len(timed) > 0) == timed_now
        assert open(cache).read().count("\n") == k + 1

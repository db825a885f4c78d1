"""The z-marching passes at the edges of their tiles, against the oracle.

Shapes take every launch form: 256 and 512 threads, tile rows that are whole
wavefronts or not, a remainder of tile rows and of planes, one column, the
smallest grid, XCD runs of tiles and one range per XCD, up to 32 planes a
block.  Outputs are filled with NaN first, so a tile nobody owns shows.
k_rhs is held to the rounding of Eq. (29) at every cell, k_correct to 1e-12 in
l2 and 1e-11 pointwise of the velocity change, two sweeps of the
variable-coefficient iteration (k_rhs without the split term) to 1e-12.
"""
import numpy as np
import pytest

import oracle as O
import parity_util as PU
from paper_2103_01874_amd import binding, synth
from test_gpu_configs import assembly_bound, run_single
from test_gpu_varcoef import gpu_varcoef, oracle_fp

pytestmark = pytest.mark.gpu

SHAPES = [(1, 2, 1), (2, 3, 4), (64, 9, 3), (72, 29, 18), (162, 6, 4), (128, 130, 6), (256, 258, 3), (96, 685, 6),
          (512, 257, 36)]


def _run(pr, f):
    import torch
    plan = binding.Plan(pr.nx, pr.ny, pr.nz, pr.lx, pr.ly, pr.lz, ybc=pr.ybc)
    b = torch.full_like(f["rho"], float("nan"))
    u, v, w = (torch.full_like(f[k], float("nan")) for k in ("us", "vs", "ws"))
    ins = [[f[k]] for k in ("us", "vs", "ws", "rho", "pn", "pnm1")]
    plan.rhs([pr.rho0], [pr.dt], *ins, [f["S"]], [b])
    info = plan.correct([pr.dt], *ins, [f["pn"]], [f["S"]], [u], [v], [w], rho0=[pr.rho0])
    torch.cuda.synchronize()
    plan.close()
    return [a.cpu().numpy() for a in (b, u, v, w)], binding.decode_info(info)[0]


@pytest.mark.parametrize("ybc", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_march_tile_edges(shape, ybc, monkeypatch):
    pr = synth.random_problem(*shape, seed=9500 + sum(shape), ybc=ybc)
    g = O.Grid(pr.nx, pr.ny, pr.nz, pr.lx, pr.ly, pr.lz, ybc=ybc)
    f = binding.to_device(pr)
    got, rec = _run(pr, f)
    b = O.assemble_rhs(g, pr.rho0, pr.dt, pr.us, pr.vs, pr.ws, pr.rho, pr.pn, pr.pnm1, pr.S)
    assert np.all(np.abs(got[0] - b) <= assembly_bound(pr, pr.rho0))
    want = O.correct(g, pr.rho0, pr.dt, pr.us, pr.vs, pr.ws, pr.rho, pr.pn, pr.pnm1, pr.pn)
    for a, o, st in zip(got[1:], want, (pr.us, pr.vs, pr.ws)):
        assert np.all(np.isfinite(a))
        assert PU.rel(a - st, o - st) <= 1e-12 and PU.rel_inf(a - st, o - st) <= 1e-11
    chk = O.divergence_check(g, pr.us, pr.vs, pr.ws, pr.S, *want)
    assert abs(rec["res_rel"] - chk["rel"]) <= 1e-10 * chk["rel"]
    # the tile order and the block size change no cell's arithmetic
    for bands, nt in (("1", "256"), ("16", "512"), ("5", "512")):
        monkeypatch.setenv("PPE_TUNE_BANDS", bands)
        monkeypatch.setenv("PPE_TUNE_NT_RHS", nt)
        monkeypatch.setenv("PPE_TUNE_NT_COR", nt)
        alt, _ = _run(pr, f)
        for x, y in zip(got, alt):
            assert np.array_equal(x, y), (bands, nt)


@pytest.mark.parametrize("ybc", [0, 1])
@pytest.mark.parametrize("shape", [(64, 9, 3), (128, 130, 6)])
def test_march_without_the_split_term(shape, ybc):
    pr = synth.random_problem(*shape, seed=9600 + sum(shape), ybc=ybc)
    (p,), _, _, _ = gpu_varcoef([pr], 2, 0.0)
    _, ref = oracle_fp(pr, 2)
    assert PU.rel(p, ref["p"]) <= 1e-12


@pytest.mark.parametrize("precision", [binding.PPE_PREC_FP64, binding.PPE_PREC_MIXED])
def test_statistics_of_a_batch_equal_single_runs(precision):
    """The sums reduced inside other launches (block 0 of the row transform,
    the last block of the projection): instances that converge after different
    sweeps, twice in a row, give the fields they give alone, bit for bit, and
    the statistics to the rounding of their sums (the blocks of a pass depend
    on the batch; a residual of 1e-7 leaves 1e-9 of it)."""
    prs = [synth.sheet_problem(32, 16, 24, seed=9700 + r, rho_l=100.0 * r) for r in (1, 3, 10)]
    alone = [gpu_varcoef([pr], 40, 1e-7, precision=precision, correct=True) for pr in prs]
    close = lambda a, b: abs(a - b) <= 1e-9 * abs(b)
    for _ in range(2):
        p, recs, hist, outs = gpu_varcoef(prs, 40, 1e-7, precision=precision, correct=True)
        for i, (p1, r1, h1, o1) in enumerate(alone):
            assert np.array_equal(p[i], p1[0])
            assert all(np.array_equal(outs[i][k], o1[0][k]) for k in ("u", "v", "w"))
            assert recs[i]["iters"] == r1[0]["iters"] and recs[i]["status"] == r1[0]["status"]
            assert np.allclose(hist[i], h1[0], rtol=1e-9, atol=0.0)
            assert all(close(outs[i]["info"][k], o1[0]["info"][k]) for k in ("res_rel", "div_l2", "div_max", "div0_l2"))
    assert len({r["iters"] for r in recs}) > 1


@pytest.mark.parametrize("ybc", [0, 1])
@pytest.mark.parametrize("shape", [(2, 3, 4), (72, 29, 18), (128, 130, 6), (96, 131, 6)])
def test_residual_marches_at_tile_edges(shape, ybc):
    """k_resid and k_resid_var where a tile has no second row of tiles, a
    remainder of rows or planes, few columns: two fixed-point sweeps and a
    refined mixed step against the oracle."""
    pr = synth.random_problem(*shape, seed=9900 + sum(shape), ybc=ybc)
    (p,), (rec,), H, _ = gpu_varcoef([pr], 2, 0.0)
    _, ref = oracle_fp(pr, 2)
    assert PU.rel(p, ref["p"]) <= 1e-12
    r = np.array(ref["res"])
    big = r > 1e-9
    assert np.all(np.abs(H[0][big] - r[big]) <= 1e-8 * r[big])
    got, rec = run_single(pr, binding.PPE_PREC_MIXED, 3, tol=1e-13)
    PU.check(pr, got, rec, PU.oracle_step(pr), label=f"{shape} ybc={ybc} ")


@pytest.mark.parametrize("precision,batch", [(binding.PPE_PREC_FP64, 8), (binding.PPE_PREC_MIXED, 13)])
def test_padded_spectrum_tiles_equal_unpadded(precision, batch):
    """A batch whose spectrum passes 64 MiB (its tiles lie further apart)
    gives the fields of each instance alone (tiles end to end), bit for bit."""
    import torch
    prs = [synth.random_problem(128, 64, 128, seed=9950 + i, ybc=1) for i in range(3)]
    kw = dict(precision=precision, tol=1e-12, max_refine=1, ybc=1)
    pr = prs[0]
    plan = binding.Plan(pr.nx, pr.ny, pr.nz, pr.lx, pr.ly, pr.lz, batch=batch, **kw)
    f = [binding.to_device(p) for p in prs]
    outs, _ = binding.step(plan, [f[i % 3] for i in range(batch)], [prs[i % 3].rho0 for i in range(batch)],
                           [pr.dt] * batch)
    torch.cuda.synchronize()
    plan.close()
    for i in range(3):
        one = binding.Plan(pr.nx, pr.ny, pr.nz, pr.lx, pr.ly, pr.lz, **kw)
        (alone,), _ = binding.step(one, [f[i]], [prs[i].rho0], [pr.dt])
        torch.cuda.synchronize()
        one.close()
        for n in range(i, batch, 3):
            for k in ("p", "u", "v", "w"):
                assert torch.equal(outs[n][k], alone[k]), (n, k)

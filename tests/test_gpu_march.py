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
from test_gpu_configs import assembly_bound
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

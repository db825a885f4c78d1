"""Grouping is invisible: an instance's fields and info record do not depend on
what else shares its launch, bit for bit.

The shapes are those at which the launch shape of the marching passes (planes
per block) is chosen by the number of instances, so that the sums behind the
gauge, the compatibility defect, the residual norms and the continuity check
are split differently between blocks alone and in a group.
"""
import numpy as np
import pytest

from paper_2103_01874_amd import binding, synth
from test_gpu_varcoef import gpu_varcoef

pytestmark = pytest.mark.gpu

STEPS = [((64, 64, 64), 8, binding.PPE_PREC_MIXED, 0), ((64, 64, 64), 4, binding.PPE_PREC_MIXED, 1),
         ((96, 64, 96), 5, binding.PPE_PREC_FP64, 0), ((72, 29, 54), 18, binding.PPE_PREC_MIXED, 0),
         ((32, 16, 24), 16, binding.PPE_PREC_FP64, 0)]


def _step(prs, precision):
    import torch
    pr = prs[0]
    plan = binding.Plan(pr.nx, pr.ny, pr.nz, pr.lx, pr.ly, pr.lz, batch=len(prs), precision=precision, tol=1e-13,
                        max_refine=2, ybc=pr.ybc)
    f = [binding.to_device(p) for p in prs]
    outs, info = binding.step(plan, f, [p.rho0 for p in prs], [p.dt for p in prs])
    d = plan.residual([o["u"] for o in outs], [o["v"] for o in outs], [o["w"] for o in outs], [x["S"] for x in f])
    torch.cuda.synchronize()
    plan.close()
    return outs, binding.decode_info(info), d.cpu().numpy().reshape(len(prs), 3)


@pytest.mark.parametrize("shape,batch,precision,ybc", STEPS)
def test_step_of_a_group_equals_alone(shape, batch, precision, ybc):
    import torch
    prs = [synth.random_problem(*shape, seed=4100 + i, ybc=ybc) for i in range(3)]
    outs, recs, div = _step([prs[i % 3] for i in range(batch)], precision)
    for i, pr in enumerate(prs):
        (alone,), (rec,), d1 = _step([pr], precision)
        for n in range(i, batch, 3):
            for k in ("p", "u", "v", "w"):
                assert torch.equal(outs[n][k], alone[k]), (n, k)
            assert recs[n] == rec, (n, recs[n], rec)
            assert np.array_equal(div[n], d1[0])


@pytest.mark.parametrize("precision", [binding.PPE_PREC_FP64, binding.PPE_PREC_MIXED])
@pytest.mark.parametrize("shape,batch", [((64, 64, 64), 8), ((96, 64, 96), 3)])
def test_fixed_point_of_a_group_equals_alone(shape, batch, precision):
    prs = [synth.random_problem(*shape, seed=4200 + i) for i in range(2)]
    p, recs, hist, _ = gpu_varcoef([prs[i % 2] for i in range(batch)], 5, 1e-3, precision=precision)
    for i, pr in enumerate(prs):
        (p1,), (r1,), (h1,), _ = gpu_varcoef([pr], 5, 1e-3, precision=precision)
        for n in range(i, batch, 2):
            assert np.array_equal(p[n], p1) and np.array_equal(hist[n], h1), n
            assert recs[n] == r1, (n, recs[n], r1)

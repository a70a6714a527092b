"""The segmented M2L (one column per target box and source parent, reflected
offsets sharing an operator), where its tiles can go wrong: rank remainders
from the smallest to the largest order, narrow and wide column tasks, several
density columns.

Single precision is held against the pairwise M2L, which one plan evaluated
alone takes: the same truncated operators, so the two differ by rounding (sums
of about 200 terms of relative rounding 6e-8: 1e-6; bf16x3 products rounded to
2^-16 of the far field: 1e-5).  FP64 is held against the FP64 direct sum at the
error of the expansion order (potential and gradient on this cloud: 5e-2, 5e-3,
1e-4, 1e-6, 1e-8 for p = 2, 3, 5, 8, 10, several times the measured ones of the
paper's orders)."""
import numpy as np
import pytest

import synth
from oracle import direct as D
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu
KAPPA = 0.125
FP64_TOL = {2: 5e-2, 3: 5e-3, 5: 1e-4, 8: 1e-6, 10: 1e-8}


def _rel(a, b):
    return D.rel_l2(a.double().cpu().numpy(), b.double().cpu().numpy())


def _cloud(n_tri, seed=141):
    su = synth.sphere_union_spheres(30, seed=seed, box=14.0)
    v, t = synth.sphere_union_mesh(su, n_tri, seed=seed)
    return synth.three_point_cloud(v, t)


@pytest.mark.parametrize("precision,tol", [("fp64", None), ("fp32", 1e-6), ("bf16x3", 1e-5)])
@pytest.mark.parametrize("p,n_tri,ncrit", [(2, 700, 20), (3, 333, 16), (5, 2000, 24), (8, 1001, 16), (8, 9000, 32),
                                           (10, 1500, 40)])
def test_segmented_m2l(precision, tol, p, n_tri, ncrit):
    torch = require_gpu()
    from paper_2103_01048_amd import FMMPlan, eval_pair
    x = _cloud(n_tri)
    xt = torch.tensor(x, device="cuda")
    dt = torch.float64 if precision == "fp64" else torch.float32
    q = torch.tensor(np.random.default_rng(142).standard_normal((4, len(x))), device="cuda", dtype=dt)
    plans = [FMMPlan(xt, kernel=k, kappa=KAPPA, p=p, ncrit=ncrit, precision=precision) for k in ("laplace", "yukawa")]
    print(f"[m2l] {precision} p={p} n={len(x)}", flush=True)
    one = eval_pair(plans[0], plans[1], q[0])
    rows = np.arange(0, len(x), 5)
    for plan, kernel, (pot, grad) in zip(plans, ("laplace", "yukawa"), one):
        if precision == "fp64":
            p0, g0 = D.direct(x[rows], x, q[0].cpu().numpy(), kernel, KAPPA)
            ep, eg = D.rel_l2(pot.cpu().numpy()[rows], p0), D.rel_l2(grad.cpu().numpy()[rows], g0)
            assert max(ep, eg) < FP64_TOL[p], (ep, eg)
        else:
            pot0, grad0 = plan.eval(q[0])
            assert _rel(pot, pot0) < tol and _rel(grad, grad0) < tol
    four = eval_pair(plans[0], plans[1], q)
    for (pot, grad), (pot4, grad4) in zip(one, four):
        assert _rel(pot4[0], pot) < (tol or 1e-12) and _rel(grad4[0], grad) < (tol or 1e-12)


def test_one_column_after_four_keeps_its_bits():
    """Rows that a four-column evaluation wrote must not show in a one-column one."""
    torch = require_gpu()
    from paper_2103_01048_amd import FMMPlan, eval_pair
    x = torch.tensor(_cloud(1500, seed=143), device="cuda")
    q = torch.tensor(np.random.default_rng(144).standard_normal((4, len(x))), device="cuda", dtype=torch.float32)
    for precision in ("fp32", "bf16x3"):
        pl = [FMMPlan(x, kernel=k, kappa=KAPPA, p=6, ncrit=32, precision=precision) for k in ("laplace", "yukawa")]
        first = [t.clone() for o in eval_pair(pl[0], pl[1], q[0]) for t in o]
        alone = [t.clone() for t in pl[1].eval(q[0])]
        eval_pair(pl[0], pl[1], q)
        pl[1].eval(q)
        for u, w in zip(first, [t for o in eval_pair(pl[0], pl[1], q[0]) for t in o]):
            assert torch.equal(u, w)
        for u, w in zip(alone, pl[1].eval(q[0])):
            assert torch.equal(u, w)

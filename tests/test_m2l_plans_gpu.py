"""The segmented M2L of two plans that differ in what they have met or in how
they were set up: the evaluations that each did alone before, the tunables
each was set up under, and the plans whose operators they took."""
import numpy as np
import pytest

import synth
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu
KAPPA = 0.125


def _cloud(n_tri=1500, seed=161):
    su = synth.sphere_union_spheres(30, seed=seed, box=14.0)
    v, t = synth.sphere_union_mesh(su, n_tri, seed=seed)
    return synth.three_point_cloud(v, t)


def _plans(xt, precision, **kw):
    from paper_2103_01048_amd import FMMPlan
    kw = {"p": 6, "ncrit": 32, **kw}
    return [FMMPlan(xt, kernel=k, kappa=KAPPA, precision=precision, **kw) for k in ("laplace", "yukawa")]


def _m2l_columns(plan):
    """M2L columns of a plan: source parents of each target box."""
    t = plan.tree()
    return sum(len({int(t["parent"][a]) for a in v}) for v in t["V"])


def _pair(plans, q):
    from paper_2103_01048_amd import eval_pair
    return [t.clone() for o in eval_pair(plans[0], plans[1], q) for t in o]


@pytest.mark.parametrize("precision", ["bf16x3", "fp32", "fp64"])
@pytest.mark.parametrize("first,cols", [(0, 4), (1, 4), (0, 2), (1, 3)])
def test_pair_after_one_plan_met_more_columns(precision, first, cols):
    """Each plan's buffers are sized for the columns that it has met; the pair
    evaluation is the same to the bit as on plans that met nothing before."""
    torch = require_gpu()
    xt = torch.tensor(_cloud(), device="cuda")
    dt = torch.float64 if precision == "fp64" else torch.float32
    q = torch.tensor(np.random.default_rng(162).standard_normal((4, len(xt))), device="cuda", dtype=dt)
    print(f"[m2l plans] {precision} plan {first} first, {cols} columns", flush=True)
    plans = _plans(xt, precision)
    assert _m2l_columns(plans[0]) >= 1024  # enough for the segmented form
    want = _pair(plans, q[0])
    del plans
    plans = _plans(xt, precision)
    plans[first].eval(q[:cols])
    for _ in range(2):
        for got, ref in zip(_pair(plans, q[0]), want):
            assert torch.equal(got, ref)
    # and two columns after it, where only one plan's buffers grow or none do
    want = _pair(_plans(xt, precision), q[1:3])
    for got, ref in zip(_pair(plans, q[1:3]), want):
        assert torch.equal(got, ref)


def _operator(precision, level=4):
    from paper_2103_01048_amd import BEMOperator
    v, t = synth.octa_sphere(level, 4.0)
    return BEMOperator(v, t, quad_pts=3, kappa=KAPPA, p=6, ncrit=32, precision=precision)


def _operator_points(torch, level=4):
    """The quadrature points of _operator, to the bit."""
    v, t = synth.octa_sphere(level, 4.0)
    l1, l2 = np.array([1 / 6, 2 / 3, 1 / 6])[None, :, None], np.array([1 / 6, 1 / 6, 2 / 3])[None, :, None]
    tri = v[t][:, None]
    x = ((1 - l1 - l2) * tri[:, :, 0] + l1 * tri[:, :, 1] + l2 * tri[:, :, 2]).reshape(-1, 3)
    return torch.tensor(x, device="cuda")


class _OperatorPlans:
    """The operator's two plans (bem_fmm_plan) as FMMPlans that do not own
    their handles."""

    def __init__(self, torch, op):
        import ctypes
        from paper_2103_01048_amd import FMMPlan, _lib
        self.op, self.plans = op, []
        for name, kernel in (("laplace", _lib.FMM_LAPLACE), ("yukawa", _lib.FMM_YUKAWA)):
            pl = FMMPlan.__new__(FMMPlan)
            pl._h = ctypes.c_void_p(_lib.lib().bem_fmm_plan(op._h, kernel))
            pl.kernel, pl.device = name, op.device
            pl.dtype = torch.float64 if op.precision == "fp64" else torch.float32
            pl.n = pl.info()["n_points"]
            self.plans.append(pl)

    def __enter__(self):
        return self.plans

    def __exit__(self, *a):
        for pl in self.plans:
            pl._h = None
        self.op = None


@pytest.mark.parametrize("precision", ["bf16x3", "fp32", "fp64"])
def test_operator_plans_evaluated_after_the_operator_they_took_from_is_gone(precision):
    """A second operator on the same mesh takes the first one's translation
    operators, also after the first one's plans were evaluated as a pair and
    with several columns; freeing the first changes nothing."""
    torch = require_gpu()
    dt = torch.float64 if precision == "fp64" else torch.float32

    def both(plans):
        return _pair(plans, q[0]) + _pair(plans, q[1:3]) + [t.clone() for pl in plans for t in pl.eval(q)]

    print(f"[m2l plans] operator {precision}", flush=True)
    op = _operator(precision)
    with _OperatorPlans(torch, op) as plans:
        assert _m2l_columns(plans[0]) >= 1024
        q = torch.tensor(np.random.default_rng(163).standard_normal((4, plans[0].n)), device="cuda", dtype=dt)
        want = both(plans)
    op2 = _operator(precision)
    with _OperatorPlans(torch, op2) as plans:
        first = both(plans)
    del op
    torch.cuda.synchronize()
    junk = torch.full((1 << 26,), float("nan"), device="cuda")  # takes freed device memory
    with _OperatorPlans(torch, op2) as plans:
        again = both(plans)
    del junk
    for a, b, c in zip(want, first, again):
        assert torch.equal(a, b) and torch.equal(a, c)


@pytest.mark.parametrize("widths", [(128, 64), (64, 128), (128, 128)])
def test_pair_of_plans_set_up_under_different_m2l_cols(widths):
    """Columns per task differ between the two plans; a column's products and
    their order do not depend on it, so neither does a bit of the results."""
    torch = require_gpu()
    from paper_2103_01048_amd import FMMPlan, autotune
    xt = torch.tensor(_cloud(9000), device="cuda")
    q = torch.tensor(np.random.default_rng(164).standard_normal((2, len(xt))), device="cuda", dtype=torch.float32)

    def plans(cols):
        out = []
        for kernel, c in zip(("laplace", "yukawa"), cols):
            with autotune.tuning(**{**autotune.DEFAULTS, "m2l_cols": c}):
                out.append(FMMPlan(xt, kernel=kernel, kappa=KAPPA, p=6, ncrit=32, precision="bf16x3"))
        return out

    print(f"[m2l plans] m2l_cols {widths}", flush=True)
    ref = plans((64, 64))
    # at least 160 tasks of 64 columns, so that the plans' widths are their m2l_cols
    assert _m2l_columns(ref[0]) >= 160 * 64
    want = [_pair(ref, q[0]), _pair(ref, q)]
    pl = plans(widths)
    for qq, w in zip((q[0], q), want):
        for got, r in zip(_pair(pl, qq), w):
            assert torch.equal(got, r)


def _replay_equals_eager(torch, warm, fn):
    """fn captured after `warm` ran eagerly and before fn itself ever did;
    three replays with eager work between them against the eager result."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        warm()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = fn()
    want = [t.clone() for t in fn()]
    for _ in range(3):
        for t in out:
            t.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))
        warm()
        torch.cuda.synchronize()


@pytest.mark.parametrize("precision", ["bf16x3", "fp32", "fp64"])
@pytest.mark.parametrize("form", ["single after pair", "pair after products", "single after five columns",
                                  "chained pair after products"])
def test_one_column_captured_after_another_form_of_evaluation(precision, form):
    """A plan that has evaluated one column in one way evaluates one in
    another inside a graph capture, where nothing can be allocated."""
    torch = require_gpu()
    from paper_2103_01048_amd import autotune, eval_pair
    from paper_2103_01048_amd.fmm import eval_pair_md
    xt = torch.tensor(_cloud(), device="cuda")
    dt = torch.float64 if precision == "fp64" else torch.float32
    rng = np.random.default_rng(165)
    q = torch.tensor(rng.standard_normal((5, len(xt))), device="cuda", dtype=dt)
    dip = torch.tensor(rng.standard_normal((len(xt), 3)), device="cuda", dtype=dt)
    with autotune.tuning(**{**autotune.DEFAULTS, "gemm_chain": int(form.startswith("chained"))}):
        a, b = _plans(xt, precision)
    assert _m2l_columns(a) >= 1024
    print(f"[m2l plans] capture {precision} {form}", flush=True)
    if form == "single after pair":
        _replay_equals_eager(torch, lambda: eval_pair(a, b, q[0]), lambda: list(b.eval(q[1])))
    elif form.endswith("pair after products"):
        _replay_equals_eager(torch, lambda: eval_pair_md(a, b, q[0], dip),
                             lambda: [t for o in eval_pair(a, b, q[1]) for t in o])
    else:
        _replay_equals_eager(torch, lambda: eval_pair(a, b, q), lambda: list(a.eval(q[1])))


@pytest.mark.parametrize("precision", ["bf16x3", "fp32"])
def test_factored_m2l_buffers_after_fewer_columns(precision):
    """Four columns, then one, then four again: the buffers of the four stay."""
    torch = require_gpu()
    from paper_2103_01048_amd import autotune
    xt = torch.tensor(_cloud(700), device="cuda")
    q = torch.tensor(np.random.default_rng(166).standard_normal((4, len(xt))), device="cuda", dtype=torch.float32)
    with autotune.tuning(**{**autotune.DEFAULTS, "m2l_factored": 1}):
        plans = _plans(xt, precision)
    print(f"[m2l plans] factored {precision}", flush=True)
    four, one = _pair(plans, q), _pair(plans, q[0])
    for got, want in ((_pair(plans, q), four), (_pair(plans, q[0]), one)):
        assert all(torch.equal(u, w) for u, w in zip(got, want))


@pytest.mark.parametrize("precision", ["bf16x3", "fp32", "fp64"])
def test_plan_takes_the_operators_that_a_live_operator_has(precision):
    """A plan on a live operator's quadrature points builds only the operators
    that the operator does not hold, keeps what it took when the operator is
    freed, and gives the same results to the bit as one that built them all."""
    torch = require_gpu()
    x = _operator_points(torch)
    dt = torch.float64 if precision == "fp64" else torch.float32
    q = torch.tensor(np.random.default_rng(167).standard_normal((2, len(x))), device="cuda", dtype=dt)

    def results(plans):
        return _pair(plans, q[0]) + [u.clone() for pl in plans for u in pl.eval(q[0]) + pl.eval(q)]

    print(f"[m2l plans] operators of an operator {precision}", flush=True)
    alone = _plans(x, precision)
    inf = alone[0].info()
    bytes_alone, ns, want = inf["device_bytes"], inf["n_surf"], results(alone)
    del alone
    op = _operator(precision)
    plans = _plans(x, precision)
    inf = plans[0].info()
    assert inf["tree_shared"] == 1
    # what it took holds n_surf x n_surf M2L operators: the segmented form's 56 at most per level in
    # FP64, the pairwise form's 316 at most in single precision (this surface uses most of them)
    taken = 50 * 8 * ns * ns if precision == "fp64" else 200 * 4 * ns * ns
    assert bytes_alone - inf["device_bytes"] > taken
    del op
    torch.cuda.synchronize()
    junk = torch.full((1 << 26,), float("nan"), device="cuda")
    for a, b in zip(results(plans), want):
        assert torch.equal(a, b)
    del junk


@pytest.mark.parametrize("cols", [1, 3])
@pytest.mark.parametrize("precision,tol", [("bf16x3", 1e-5), ("fp32", 1e-6)])
def test_pair_of_an_operators_plan_and_a_plan_of_the_callers(precision, tol, cols):
    """One plan in the pairwise and one in the segmented form: two M2L launches
    and two sums, the other passes of both in one launch.  The two forms differ
    by rounding (sums of about 200 terms in FP32; bf16x3 products rounded to
    2^-16 of the far field)."""
    torch = require_gpu()
    x = _operator_points(torch)
    q = torch.tensor(np.random.default_rng(168).standard_normal((cols, len(x))), device="cuda", dtype=torch.float32)
    print(f"[m2l plans] mixed forms {precision} {cols}", flush=True)
    plans = _plans(x, precision)
    want = _pair(plans, q)
    with _OperatorPlans(torch, _operator(precision)) as of_op:
        for mixed in ([of_op[0], plans[1]], [plans[0], of_op[1]], of_op):
            for got, ref in zip(_pair(mixed, q), want):
                assert float((got.double() - ref.double()).norm() / ref.double().norm()) < tol


def test_threads_set_up_evaluate_and_free_plans_on_the_same_points():
    """Plans take trees and operators from plans that other threads free."""
    import threading
    torch = require_gpu()
    xt = torch.tensor(_cloud(700), device="cuda")
    q = torch.tensor(np.random.default_rng(169).standard_normal(len(xt)), device="cuda", dtype=torch.float32)
    want = _pair(_plans(xt, "fp32", p=4), q)
    torch.cuda.synchronize()
    wrong, failed = [], []
    print("[m2l plans] threads", flush=True)

    def work():
        try:
            for _ in range(5):
                with torch.cuda.stream(torch.cuda.Stream()):
                    got = _pair(_plans(xt, "fp32", p=4), q)
                    torch.cuda.current_stream().synchronize()
                wrong.extend(i for i, (a, b) in enumerate(zip(got, want)) if not torch.equal(a, b))
        except Exception as e:  # reported by the main thread
            failed.append(repr(e))

    threads = [threading.Thread(target=work) for _ in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed and not wrong

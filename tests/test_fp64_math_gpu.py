"""The FP64 pair math (third-order reciprocal square root, polynomial 2^x)
where it can go wrong: distances of many orders of magnitude in one sum,
exponents around the underflow of exp(-kappa r), coincident points.

32 points in one leaf (a direct sum
on the GPU) against numpy in FP64.  Tolerance: both sides round each of n = 32
terms by a few 1e-16 with all charges of one sign, and the exponent kappa r <= 700
amplifies a rounding of r by kappa r: 700 * 4e-16 < 1e-12."""
import numpy as np
import pytest

from oracle import direct as D
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("span", [1e-6, 1.0, 1e6])
@pytest.mark.parametrize("kr", [1e-3, 30.0, 700.0, 1e5])
def test_pair_math_fp64(span, kr):
    torch = require_gpu()
    from paper_2103_01048_amd import FMMPlan, eval_pair
    rng = np.random.default_rng(151)
    x = rng.random((32, 3)) * np.array([1.0, 1e-2, 1e-4]) * span
    x[5] = x[4]  # coincident: left out of the sum
    kappa = kr / span
    q = rng.random(32) + 0.5
    xt, qt = torch.tensor(x, device="cuda"), torch.tensor(q, device="cuda")
    plans = [FMMPlan(xt, kernel=k, kappa=kappa, p=6, ncrit=64, precision="fp64") for k in ("laplace", "yukawa")]
    for kernel, (pot, grad) in zip(("laplace", "yukawa"), eval_pair(plans[0], plans[1], qt)):
        p0, g0 = D.direct(x, x, q, kernel, kappa)
        for got, ref in ((pot, p0), (grad, g0)):
            got = got.cpu().numpy()
            assert np.isfinite(got).all()
            assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref)

"""The exact maximum of a tile (the warm start of the next sweep) is formed on
the matrix cores by the plain sweep and on the VALU by the certificate's: the
same value and, among equal exponents, the same (first) point, so state and
hints must agree bit for bit after sweeps that raise the running maximum in
many tiles: integer points, which tie, and clouds without an order that the
first tiles could bound, at low temperature."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2609_33814_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu

SIZES = [(15, 17), (63, 65), (130, 81), (500, 900)]


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("integer", [True, False], ids=["ties", "cloud"])
@pytest.mark.parametrize("m,n", SIZES)
def test_maximum_and_its_point(dim, integer, m, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob = inputs.random_problem(m, n, dim, seed=7 * dim + m, integer=integer, span=6.0 if integer else 1.0)
    compare(prob, (0.05, 0.002), (1, 1, 1, 10))


def compare(prob, etas, steps):
    from paper_2609_33814_amd import bdrs
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda:0")
    args = (t(prob.x, torch.float32), t(prob.y, torch.float32), t(prob.r, torch.float64),
            t(prob.c, torch.float64), prob.cost_scale)
    for eta in etas:
        plain = bdrs.Solver(*args, eta=eta, lam=1.2)
        cert = bdrs.Solver(*args, eta=eta, lam=1.2, graph=False)
        for iters in steps:
            plain.step(iters)
            for _ in range(iters):
                bdrs.check(bdrs.lib().bdrs_solve(cert.handle, 0.0, 1, 1, 1, None),
                           allow=(bdrs.OK, bdrs.NOT_CONVERGED, bdrs.E_NUMERIC))
            a, b = plain.get_state(), cert.get_state()
            for key in ("la", "lah", "lb", "lbh", "lt"):
                assert torch.equal(a[key], b[key]), (eta, a["k"], key)
            for key, p, q in zip(("rows", "cols"), hints(plain), hints(cert)):
                assert torch.equal(p, q), (eta, a["k"], key)


def hints(sv):
    from paper_2609_33814_amd import bdrs
    row = torch.empty(sv.m, dtype=torch.int32, device="cuda:0")
    col = torch.empty(sv.n, dtype=torch.int32, device="cuda:0")
    bdrs.check(bdrs.lib().bdrs_get_hints(sv.handle, row.data_ptr(), col.data_ptr()))
    return row, col

"""The plain sweep (exponents on the matrix cores) and the certificate's sweep
(exponents on the VALU) form the same sums, so an iteration's state must not
depend on which of them ran: bit for bit, at the edges of the 64 x 64 tiles
(partial quarters of 16 inputs, one point into the next tile or output block),
for every dimension, at high and low temperature and with overrelaxation."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2609_33814_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (31, 33), (64, 63), (65, 64), (97, 129), (257, 256), (300, 1100)]


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("m,n", SIZES)
def test_plain_and_certificate_sweeps_agree(dim, m, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_33814_amd import bdrs
    prob = inputs.random_problem(m, n, dim, seed=100 * dim + m)
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda:0")
    for eta, lam in ((1.0, 1.0), (0.01, 1.5)):
        args = (t(prob.x, torch.float32), t(prob.y, torch.float32), t(prob.r, torch.float64),
                t(prob.c, torch.float64), prob.cost_scale)
        plain = bdrs.Solver(*args, eta=eta, lam=lam)
        cert = bdrs.Solver(*args, eta=eta, lam=lam, graph=False)
        for iters in (1, 1, 20):
            plain.step(iters)
            for _ in range(iters):
                bdrs.check(bdrs.lib().bdrs_solve(cert.handle, 0.0, 1, 1, 1, None),
                           allow=(bdrs.OK, bdrs.NOT_CONVERGED, bdrs.E_NUMERIC))
            a, b = plain.get_state(), cert.get_state()
            assert a["k"] == b["k"]
            for key in ("la", "lah", "lb", "lbh", "lt"):
                assert torch.equal(a[key], b[key]), (eta, lam, a["k"], key)

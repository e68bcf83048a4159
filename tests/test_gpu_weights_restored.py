"""A call that packs other sweep weights and ends in an error leaves the next
iteration as if it had not been made: bdrs_round on a state whose rounded cost is
not finite (an infinite log alpha, which an iteration at lambda = 1 does not read),
then the iteration bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2609_33814_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("then", ["step", "solve"])
def test_iteration_after_a_failed_rounding(then):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_33814_amd import bdrs
    prob = inputs.random_problem(300, 170, 2, seed=11)
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda:0")
    args = (t(prob.x, torch.float32), t(prob.y, torch.float32), t(prob.r, torch.float64),
            t(prob.c, torch.float64), prob.cost_scale)
    got = []
    for fail in (True, False):
        sv = bdrs.Solver(*args, eta=0.1)
        sv.step(4)
        st = sv.get_state()
        st["la"][17] = float("inf")
        sv.set_state(st)
        if fail:
            with pytest.raises(bdrs.BdrsError) as err:
                sv.round()
            assert err.value.status == bdrs.E_NUMERIC
        if then == "step":
            sv.step(2)
        else:
            sv.solve(0.0, 4, 4)
        got.append(sv.get_state())
        sv.close()
    for key in ("lah", "lb", "lb_prev", "lbh", "lt"):
        assert bool(torch.isfinite(got[1][key]).all()) and torch.equal(got[0][key], got[1][key]), key

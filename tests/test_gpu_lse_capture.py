"""bdrs_lse waits for its result, so it refuses a stream under capture before it
launches anything: the caller's capture goes on and holds only the caller's work."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2609_33814_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("transpose", [False, True])
def test_lse_on_a_stream_under_capture(transpose):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_33814_amd import bdrs
    prob = inputs.random_problem(200, 130, 2, seed=5)
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda:0")
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    sv = bdrs.Solver(t(prob.x, torch.float32), t(prob.y, torch.float32), t(prob.r, torch.float64),
                     t(prob.c, torch.float64), prob.cost_scale, stream=st)
    w = torch.linspace(-1.0, 1.0, 200 if transpose else 130, dtype=torch.float64, device="cuda:0")
    count = torch.zeros(1, device="cuda:0")
    torch.cuda.synchronize()
    want = sv.lse(w, 0.1, transpose=transpose)
    out = torch.zeros_like(want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        count.add_(1.0)
        assert bdrs.lib().bdrs_lse(sv.handle, int(transpose), 0.1, w.data_ptr(), out.data_ptr()) == bdrs.E_DEVICE
    for i in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert count.item() == i + 1.0 and not out.any()
        assert torch.equal(sv.lse(w, 0.1, transpose=transpose), want)

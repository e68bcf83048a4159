"""A wavefront tests its split's tiles in chunks of 64: sweeps of one split over
more tiles than that, just over one chunk (66 tiles) and just over two (130), as
inputs of either direction.  Plain and certificate sweeps walk them with code of
their own and must agree bit for bit, states and hints, at temperatures where most
later chunks hold no candidate and where all do."""
import pytest

torch = pytest.importorskip("torch")

from paper_2609_33814_amd import inputs  # noqa: E402
from test_gpu_sweep_max import compare  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture
def table():
    from paper_2609_33814_amd import bdrs
    keep = bdrs.tune_table()
    yield bdrs
    bdrs.tune_clear()
    for e in keep:
        bdrs.tune_set(e)


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("m,n", [(4161, 8257), (8257, 4161)])
def test_more_tiles_than_a_chunk(table, dim, m, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    table.tune_set(dict(dim=dim, m=m, n=n, splits_row=1, splits_col=1))
    prob = inputs.random_problem(m, n, dim, seed=13 * dim + m)
    compare(prob, (0.5, 0.002), (1, 1, 4))

"""The fitting net's kernels: they split their sums over more waves for few
rows than for many (the thresholds lie between 1,000 and 20,000 rows), and an
atom's results must not feel that.  A request evaluated alone takes the
small-system kernels, beside a 21,000-atom companion the large-system ones;
both give the same bits in every precision, at sizes around the 16-row tiles
and the tile counts where the launches change."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2201_01446_amd as P
    assert torch.cuda.is_available()
    return P


@pytest.fixture(scope="module")
def model(P, cu_cfg, cu_params):
    return P.Model(cu_cfg, cu_params).tabulate(0.7, 0.01, 1.5, 0.1)


@pytest.fixture(scope="module")
def companion():
    return synth.serving_request(np.random.default_rng(5), 21500)[:2]


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("size", [32, 33, 1030, 4100])
def test_rows_do_not_feel_the_launch(P, model, companion, precision, size):
    from paper_2201_01446_amd.serve import Batch
    req = synth.serving_request(np.random.default_rng(size), size)[:2]
    total = len(req[0]) + len(companion[0])
    assert total > 20016
    batch = Batch(model, total, 2)

    def run(cells):
        X = torch.tensor(np.concatenate([x for x, _ in cells]), dtype=torch.float64, device="cuda")
        out = batch.compute([(len(x), box) for x, box in cells], X, precision)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in out.items()}

    alone, beside = run([req]), run([req, companion])
    n = len(req[0])
    assert np.all(np.isfinite(alone["F"])) and np.any(alone["F"] != 0)
    assert alone["E"][0] == beside["E"][0]
    np.testing.assert_array_equal(alone["F"], beside["F"][:n])
    np.testing.assert_array_equal(alone["W"][0], beside["W"][0])

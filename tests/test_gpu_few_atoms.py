"""Few atoms: up to 1,024 take four waves each in the embedding kernels, and up
to 4,096 are summed by one block.  A request evaluated alone there has the bits
that it has beside a 5,000-atom companion, with and without the neighbor limit
cutting some off; and the sums are those of the per-atom values (FP64, 1e-12:
4,097 terms reordered)."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def companion():
    return synth.serving_request(np.random.default_rng(5), 5000)[:2]


def run(P, batch, cells, precision):
    X = torch.tensor(np.concatenate([x for x, _ in cells]), dtype=torch.float64, device="cuda")
    out = batch.compute([(len(x), box) for x, box in cells], X, precision)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("sel", [192, 70])
@pytest.mark.parametrize("size", [32, 333, 1024])
def test_waves_of_an_atom(cu_cfg, cu_params, companion, precision, sel, size):
    import paper_2201_01446_amd as P
    from paper_2201_01446_amd.serve import Batch
    cfg = dict(cu_cfg, sel=sel, sel_t=(sel,))
    model = P.Model(cfg, cu_params).tabulate(0.7, 0.01, 1.5, 0.1)
    req = synth.serving_request(np.random.default_rng(size), size)[:2]
    batch = Batch(model, len(req[0]) + len(companion[0]), 2)
    alone = run(P, batch, [req], precision)
    cut = batch.stats()["sel_overflow"]
    assert (cut > 0) == (sel < 192)
    beside = run(P, batch, [req, companion], precision)
    assert np.all(np.isfinite(alone["F"])) and np.any(alone["F"] != 0)
    assert alone["E"][0] == beside["E"][0]
    np.testing.assert_array_equal(alone["F"], beside["F"][:len(req[0])])
    np.testing.assert_array_equal(alone["W"][0], beside["W"][0])


@pytest.mark.parametrize("natoms", [32, 500, 4096, 4097])
def test_sums_of_one_block(cu_cfg, cu_params, natoms):
    import paper_2201_01446_amd as P
    from paper_2201_01446_amd.serve import Batch
    model = P.Model(cu_cfg, cu_params).tabulate(0.7, 0.01, 1.5, 0.1)
    x, box = synth.serving_request(np.random.default_rng(7), natoms)[:2]
    X = torch.tensor(x, dtype=torch.float64, device="cuda")
    nl = P.NeighborList(model, X, box, 2.0)
    moved = X + 0.05 * torch.sin(X)
    r = P.compute(model, nl, moved, precision=P.FP64, forces=True, virial=True, atom_energy=True)
    E, W, e = r["E"].cpu().numpy(), r["W"].cpu().numpy().ravel(), r["e_atom"].cpu().numpy()
    assert abs(E.ravel()[0] - e.sum()) <= 1e-12 * np.abs(e).sum()
    # the same atoms through the sum of a batch's segments
    b = run(P, Batch(model, natoms, 1), [(moved.cpu().numpy(), box)], P.FP64)
    np.testing.assert_allclose(W, b["W"][0].ravel(), rtol=0, atol=1e-12 * max(1e-30, np.abs(b["F"]).sum() * 10))

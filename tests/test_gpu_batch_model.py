"""A batch evaluated with another model than the one it was created for: the
scratch grows for a model that keeps more neighbors, a cut-off inside the
batch's rcut + skin gives that model's own results, and one past it is refused
(its neighbors would be missing)."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def make(P, cfg, **change):
    c = dict(cfg, **change)
    c["sel_t"] = (c["sel"],)
    prm = synth.model_params(c)
    return c, prm, P.Model(c, prm).tabulate(0.7, 0.01, 1.5, 0.1)


def requests():
    return [synth.serving_request(np.random.default_rng(k), n)[:2] for k, n in ((41, 200), (42, 57))]


def run(batch, model, cells, precision):
    """As Batch.compute of a batch made for `model`."""
    batch.model = model
    X = torch.tensor(np.concatenate([x for x, _ in cells]), dtype=torch.float64, device="cuda")
    out = batch.compute([(len(x), box) for x, box in cells], X, precision)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("precision", [0, 1, 2])
def test_model_with_more_neighbors(cu_cfg, cu_params, precision):
    import paper_2201_01446_amd as P
    from paper_2201_01446_amd.serve import Batch
    few, many = make(P, cu_cfg, sel=24)[2], make(P, cu_cfg, sel=512)[2]
    cells = requests()
    total = sum(len(x) for x, _ in cells)
    b = Batch(few, total, 2)
    first = run(b, few, cells, precision)
    got = run(b, many, cells, precision)
    want = run(Batch(many, total, 2), many, cells, precision)
    again = run(b, few, cells, precision)
    for k in ("E", "F", "W"):
        np.testing.assert_array_equal(got[k], want[k])
        np.testing.assert_array_equal(again[k], first[k])
    assert np.any(got["F"] != first["F"])


def check_against_oracle(P, cfg, prm, out, cells):
    off, table = 0, oracle.Table(cfg, prm, 0.7, 0.01, 1.5, 0.1)
    for k, (x, box) in enumerate(cells):
        ref = oracle.evaluate(cfg, prm, x, box, table=table)
        assert abs(out["E"][k] - ref["E"]) <= 1e-10 * abs(ref["E"])
        assert np.max(np.abs(out["F"][off:off + len(x)] - ref["F"])) <= 1e-10 * np.max(np.abs(ref["F"]))
        off += len(x)


@pytest.mark.parametrize("rcut", [9.0, 10.0])   # inside the batch's reach, and at it
def test_model_with_a_longer_cut_off(cu_cfg, rcut):
    import paper_2201_01446_amd as P
    from paper_2201_01446_amd.serve import Batch
    cells = requests()
    base = make(P, cu_cfg)[2]
    b = Batch(base, sum(len(x) for x, _ in cells), 2, skin=2.0)
    cfg, prm, longer = make(P, cu_cfg, rcut=rcut, sel=420)
    check_against_oracle(P, cfg, prm, run(b, longer, cells, P.FP64), cells)
    assert b.stats()["sel_overflow"] == 0
    past = make(P, cu_cfg, rcut=10.5, sel=420)[2]
    with pytest.raises(P.DPError, match="rcut"):
        run(b, past, cells, P.FP64)


def test_batch_without_a_skin(cu_cfg, cu_params):
    import paper_2201_01446_amd as P
    from paper_2201_01446_amd.serve import Batch
    cells = requests()
    cfg, prm, model = make(P, cu_cfg)
    b = Batch(model, sum(len(x) for x, _ in cells), 2, skin=0.0)
    check_against_oracle(P, cfg, prm, run(b, model, cells, P.FP64), cells)

"""A batch bins its requests together, in groups of at most 65,536 cells: sparse
cells (few atoms in a wide box, 68,921 cells of 5 A each) form groups of their
own between ordinary ones and an open cluster.  Every request has the bits it
has alone, and the oracle's values (FP64 sums of the same terms: 1e-10)."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_groups_of_requests(cu_cfg, cu_params):
    import paper_2201_01446_amd as P
    from paper_2201_01446_amd.serve import Batch
    model = P.Model(cu_cfg, cu_params).tabulate(0.7, 0.01, 1.5, 0.1)
    table = oracle.Table(cu_cfg, cu_params, 0.7, 0.01, 1.5, 0.1)
    rng = np.random.default_rng(31)
    wide = np.diag([206.0, 206.0, 206.0])
    small = [synth.serving_request(rng, n)[:2] for n in (33, 130, 64)]
    blob = synth.copper(3, 0.1, 8)[0]
    cells = [small[0], (np.ascontiguousarray(blob[:40]) + 100.0, wide), (np.ascontiguousarray(blob[:55]) - 3.0, None),
             small[1], (np.ascontiguousarray(blob[:37]) - 4.0, wide), small[2]]
    batch = Batch(model, sum(len(x) for x, _ in cells), len(cells))

    def run(some):
        X = torch.tensor(np.concatenate([x for x, _ in some]), dtype=torch.float64, device="cuda")
        out = batch.compute([(len(x), box) for x, box in some], X, P.FP64)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in out.items()}

    mix, off = run(cells), 0
    for k, (x, box) in enumerate(cells):
        alone = run([(x, box)])
        F = mix["F"][off:off + len(x)]
        off += len(x)
        assert alone["E"][0] == mix["E"][k]
        np.testing.assert_array_equal(alone["F"], F)
        np.testing.assert_array_equal(alone["W"][0], mix["W"][k])
        ref = oracle.evaluate(cu_cfg, cu_params, x, box, table=table)
        assert abs(mix["E"][k] - ref["E"]) <= 1e-10 * abs(ref["E"])
        assert np.max(np.abs(F - ref["F"])) <= 1e-10 * np.max(np.abs(ref["F"]))
    assert batch.stats()["cap_overflow"] == 0

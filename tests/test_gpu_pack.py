"""The weight layouts that are formed on the device: every precision's fitting
net, in the compressed step and in the fused step that runs it as GEMMs, at
widths around the 16- and 32-column tiles, against the oracle.  FP64 1e-10; FP32
and mixed: 2,048-term sums of FP32 products and of BF16 pairs (16 bits), 1e-4
and 1e-3 of the largest force."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [16, 33, 240, 256])
def test_layouts(cu_cfg, width):
    import paper_2201_01446_amd as P
    cfg = dict(cu_cfg, fit=(width,) * 3)
    params = synth.model_params(cfg)
    model = P.Model(cfg, params).tabulate(0.7, 0.01, 1.5, 0.1)
    table = oracle.Table(cfg, params, 0.7, 0.01, 1.5, 0.1)
    x, box = synth.serving_request(np.random.default_rng(3), 45)[:2]
    ref = oracle.evaluate(cfg, params, x, box, table=table)
    X = torch.tensor(x, dtype=torch.float64, device="cuda")
    nl = P.NeighborList(model, X, box, 2.0)
    for mode in (0, 4):
        for precision, tol in ((P.FP64, 1e-10), (P.FP32, 1e-4), (P.MIXED_BF16, 1e-3)):
            r = P.compute(model, nl, X, precision=precision, mode=mode)
            err = np.max(np.abs(r["F"].cpu().numpy() - ref["F"])) / np.max(np.abs(ref["F"]))
            assert err <= tol, (mode, precision, err)

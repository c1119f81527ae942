"""Every kernel that the fitting net's launches choose among, by rows (16 atoms a
tile: the first layer changes at 48, 512 and 1,250 tiles, mixed 256 and 1,024;
the inner layers at 512, mixed 256; the input gradient at 64, 256 and 1,024, mixed
64 and 512), by width (15 tiles of 16 columns, or 8 steps of 32 in the mixed net, have
loops of their own) and by tanh (native or tabulated).

An atom's sums have one order whatever the launch, so a request evaluated alone
has the bits that it has beside others that take it to another kernel.  The
smallest request is compared with the oracle in FP64 (sums of the same terms:
1e-10 of the largest force), from which the bits carry that to every branch."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TAB = (0.7, 0.01, 1.5, 0.1)
# atoms: 44, 65 and 257 tiles alone; with the others 563 and 1,063; all 1,929
SIZES = (700, 1030, 4100, 8000, 17000)


@pytest.fixture(scope="module")
def requests():
    reqs = []
    for n in SIZES:
        x, box = synth.copper(int(np.ceil((n / 4) ** (1 / 3))), 0.08, n)
        keep = np.sort(np.random.default_rng(n).permutation(len(x))[:n])
        reqs.append((np.ascontiguousarray(x[keep]), box))
    return reqs


def evaluate(batch, cells, precision):
    X = torch.tensor(np.concatenate([x for x, _ in cells]), dtype=torch.float64, device="cuda")
    out = batch.compute([(len(x), box) for x, box in cells], X, precision)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("width,tanh", [(240, False), (240, True), (16, False), (100, False), (256, False), (100, True)])
def test_a_request_in_every_launch(cu_cfg, requests, width, tanh, precision):
    import paper_2201_01446_amd as P
    from paper_2201_01446_amd.serve import Batch
    cfg = dict(cu_cfg, fit=(width,) * 3)
    prm = synth.model_params(cfg)
    model = P.Model(cfg, prm).tabulate(*TAB).fitting_tanh(tanh)
    batch = Batch(model, sum(SIZES), len(SIZES))
    groups = [[0], [1], [2], [1, 3], [4], [0, 1, 2, 3, 4]]
    seen = {}
    for group in groups:
        out, off = evaluate(batch, [requests[k] for k in group], precision), 0
        assert np.all(np.isfinite(out["F"]))
        for slot, k in enumerate(group):
            n = len(requests[k][0])
            got = (out["E"][slot], out["F"][off:off + n].copy(), out["W"][slot])
            off += n
            if k in seen:
                for a, b in zip(seen[k], got):
                    np.testing.assert_array_equal(a, b)
            else:
                seen[k] = got
    if precision == 0:
        x, box = requests[0]
        ref = oracle.evaluate(dict(cfg, tanh_table=int(tanh)), prm, x, box, table=oracle.Table(cfg, prm, *TAB))
        assert abs(seen[0][0] - ref["E"]) <= 1e-10 * abs(ref["E"])
        assert np.max(np.abs(seen[0][1] - ref["F"])) <= 1e-10 * np.max(np.abs(ref["F"]))


@pytest.mark.parametrize("precision,tol", [(0, 1e-10), (1, 1e-4), (2, 1e-3)])
@pytest.mark.parametrize("width", [240, 100])
def test_two_types_in_every_launch(width, precision, tol):
    """Rows grouped by type, each group padded to 128: a water cell of 192 atoms
    repeated 2 to 5 times per axis (96, 328, 768 and 1,504 tiles) has in every copy
    the energies and forces of the single cell (16 tiles), but for the rounding
    of its coordinates and distances: the bounds of the comparisons with the oracle."""
    import paper_2201_01446_amd as P
    cfg = dict(synth.water_model_config(), fit=(width,) * 3)
    model = P.Model(cfg, synth.model_params(cfg)).tabulate(*TAB)
    ref = None
    for rep in (1, 2, 3, 4, 5):
        x, types, box = synth.water(rep)
        X = torch.tensor(x, dtype=torch.float64, device="cuda")
        nl = P.NeighborList(model, X, box, types=torch.tensor(types, dtype=torch.int32, device="cuda"))
        r = P.compute(model, nl, X, precision=precision, atom_energy=True)
        e, F = r["e_atom"].cpu().numpy(), r["F"].cpu().numpy()
        if ref is None:
            ref = (e, F)
        home = np.arange(len(x)) % len(ref[0])   # the copies follow each other
        assert np.max(np.abs(e - ref[0][home])) <= tol * np.max(np.abs(ref[0]))
        assert np.max(np.abs(F - ref[1][home])) <= tol * np.max(np.abs(ref[1]))

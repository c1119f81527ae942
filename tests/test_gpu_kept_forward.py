"""The forward that a list keeps for dp_energy_backward is laid out by the
model's sel: a backward with a model of another sel is refused, as is one after
the list's scratch was allocated anew, and a forward and backward of one model
that follow work as before."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def make(P, cfg, sel):
    c = dict(cfg, sel=sel, sel_t=(sel,))
    return P.Model(c, synth.model_params(c)).tabulate(0.7, 0.01, 1.5, 0.1)


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("mode", [0, 4])
def test_backward_of_another_sel(cu_cfg, precision, mode):
    import ctypes

    import paper_2201_01446_amd as P
    from paper_2201_01446_amd._lib import lib
    few, many = make(P, cu_cfg, 24), make(P, cu_cfg, 512)
    x, box = synth.copper(3, 0.05, 12)
    xd = torch.tensor(x, dtype=torch.float64, device="cuda")
    E = torch.empty(1, dtype=torch.float64, device="cuda")
    F = torch.empty_like(xd)
    vp = lambda t: ctypes.c_void_p(t.data_ptr())
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    def forward(m):
        assert lib.dp_energy_forward(m.h, nl.h, len(x), vp(xd), mode, precision, vp(E), None, st) == 0

    def backward(m):
        return lib.dp_energy_backward(m.h, nl.h, len(x), vp(xd), mode, precision, vp(F), None, st)

    nl = P.NeighborList(few, xd, box)
    forward(few)
    assert backward(many) == -6          # the kept neighbors are 24 to an atom
    forward(few)
    nl.model = many
    nl.build(xd, box)                    # 512 to an atom: new scratch
    assert backward(few) == -6
    for m in (few, many):
        forward(m)
        assert backward(m) == 0
        ref = P.compute(m, nl, xd, mode=mode, precision=precision)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(F.cpu().numpy(), ref["F"].cpu().numpy())

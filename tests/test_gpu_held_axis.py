"""The held axis row (centerline through the nodes, viscosities and boundary
values held through a step) is copied by the launch that fills the ghosts, and
ghosts that trace to it read the held state: with physical xi faces and with
periodic ones, whose ghosts wrap around the row itself.

Bars: those of the schedule tests, 1e-11 (FP64) and 1e-5 (FP32 form) of each
variable after three steps (the row itself is derived data)."""
import numpy as np
import pytest
import torch

from _helpers import announce, grouped_rel_err, make_solver, to_np
from cases import problems
from oracle import les

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,periodic", [((20, 9, 16), False), ((20, 9, 16), True),
                                            ((31, 14, 6), True)])
def test_held_axis_row(shape, periodic, precision):
    announce("held axis row", shape, periodic, precision)
    pb = problems.jet_problem(*shape, seed=5, noise=1e-2, thermo_noise=1e-2, axis_node=True)
    prm = dict(pb["params"], visc_coef=1e-3, sgs_model=2, schedule="step")
    if periodic:
        X = pb["grid"][0]
        prm["bc"] = ("periodic", "periodic") + tuple(prm["bc"][2:])
        prm["period"] = ((float(2 * X[-1] - X[-2] - X[0]), 0.0, 0.0),) + tuple(prm["period"][1:])
        pb["inflow"] = None
    pb["params"] = prm
    geo = les.geometry(pb["xyz"].numpy(), prm)
    inflow = None if periodic else pb["inflow"].numpy()
    ref, dts = les.run(pb["Q"].numpy(), geo, prm, inflow, steps=3)
    s = make_solver(pb, precision)
    Qn = s.pad(pb["Q"].cuda(), dtype=torch.float64)
    dt = to_np(s.rk5_step(Qn, 3))
    got = to_np(s.interior(Qn))
    s.close()
    bar = 1e-11 if precision == "fp64" else 1e-5
    assert np.allclose(dt, dts, rtol=bar, atol=0)
    assert grouped_rel_err(got[:, :, 1:], ref[:, :, 1:]) <= bar

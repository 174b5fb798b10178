"""The wide FP32 tile (30 x 14 outputs), taken where it saves a round of blocks
on 256 compute units: meshes of 10 million points and more.  Shapes that end
inside a tile, on a product and on a general mesh.

Bars: against the two-pass reference form 1e-3 of max |R|, as in the other tests
of the FP32 form; the state after a step bitwise the same when repeated."""
import math

import numpy as np
import pytest
import torch

from _helpers import announce, make_solver, per_variable_err, to_np
from cases import flow, mesh, problems

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,kind,schedule", [((301, 211, 200), "jet", "stage"),
                                                 ((300, 210, 200), "node", "step"),
                                                 ((222, 222, 222), "wavy", "stage")])
def test_fp32_wide_tile(shape, kind, schedule):
    announce("FP32 wide tile", shape, kind, schedule)
    if kind == "wavy":
        xyz = mesh.wavy_coords(shape[0], 2.0 * math.pi)
        pb = dict(xyz=xyz, Q=flow.modes_box_state(xyz, seed=2, kmax=2), inflow=None,
                  params=problems.box_params(2.0 * math.pi, visc_coef=1e-3))
    else:
        pb = problems.jet_problem(*shape, seed=2, axis_node=kind == "node", noise=2e-3,
                                  thermo_noise=2e-3)
    pb["params"] = dict(pb["params"], schedule=schedule)
    s = make_solver(pb, "fp32")
    Q = s.pad(pb["Q"].cuda())
    fused = to_np(s.interior(s.residual(Q))).astype(np.float64)
    two_pass = to_np(s.interior(s.residual_reference(Q))).astype(np.float64)
    assert np.isfinite(fused).all()
    assert per_variable_err(fused, two_pass).max() <= 1e-3
    out = []
    for _ in range(2):
        Qn = s.pad(pb["Q"].cuda(), dtype=torch.float64)
        s.rk5_step(Qn, 1)
        out.append(s.interior(Qn).clone())
    assert torch.isfinite(out[0]).all() and torch.equal(out[0], out[1])
    s.close()

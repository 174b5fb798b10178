"""The two FP64 tiles of the stage kernel (14 x 14 and 30 x 14 outputs) at their
edges: extents one short of, at and one past a tile, on product and general
meshes, in both update schedules and with the node on the axis.  The first
shapes' planes make the wide tile the choice on 256 compute units, the last
shape is left to the narrow one.

Bars: residuals 1e-13 of the flux scale (those of the parity tests), the state
after two steps 1e-11 per group (that of the step tests)."""
import math

import numpy as np
import pytest

from _helpers import announce, flux_err, flux_scale, make_solver, rel_err, to_np
from cases import flow, mesh, problems
from oracle import les

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,kind,sgs,schedule", [
    ((29, 13, 88), "jet", 1, "stage"), ((30, 14, 90), "jet", 2, "step"),
    ((31, 15, 50), "node", 2, "stage"), ((60, 28, 28), "jet", 0, "stage"),
    ((61, 29, 26), "node", 1, "step"), ((37, 37, 37), "wavy", 1, "stage"),
    ((45, 45, 45), "wavy", 2, "step"), ((29, 15, 20), "jet", 1, "stage")])
def test_tile_edges(shape, kind, sgs, schedule):
    announce("tile edges", shape, kind, sgs, schedule)
    if kind == "wavy":
        xyz = mesh.wavy_coords(shape[0], 2.0 * math.pi)
        pb = dict(xyz=xyz, Q=flow.modes_box_state(xyz, seed=2, kmax=2), inflow=None,
                  params=problems.box_params(2.0 * math.pi, visc_coef=1e-3))
    else:
        # amplitudes at which the oracle's own steps stay physical on all shapes
        pb = problems.jet_problem(*shape, seed=2, axis_node=kind == "node", noise=2e-3,
                                  thermo_noise=2e-3)
    prm = pb["params"] = dict(pb["params"], sgs_model=sgs, schedule=schedule)
    inflow = pb["inflow"].numpy() if pb.get("inflow") is not None else None
    geo = les.geometry(pb["xyz"].numpy(), prm)
    Q = pb["Q"].numpy()
    s = make_solver(pb)
    Qd = s.pad(pb["Q"].cuda())
    R = to_np(s.interior(s.residual(Qd)))
    scale = flux_scale(Q, geo, prm, inflow)
    assert flux_err(R, les.evaluate(Q, geo, prm, inflow), scale).max() <= 1e-13
    assert flux_err(R, to_np(s.interior(s.residual_reference(Qd))), scale).max() <= 1e-13
    dt = to_np(s.rk5_step(Qd, 2))
    got = to_np(s.interior(Qd))
    s.close()
    ref, dt_ref = les.run(Q, geo, prm, inflow, steps=2)
    assert np.allclose(dt, dt_ref, rtol=1e-11, atol=0)
    rows = slice(1 if kind == "node" else 0, None)      # the axis row is derived data
    assert rel_err(got[:, :, rows], ref[:, :, rows]) <= 1e-11

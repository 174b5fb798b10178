"""The residual adjoint where its passes split the mesh: pass 1 marches chunks
of 1 to 8 planes, chosen by the number of 32 x 8 tiles of the padded plane, and
pass 2 hands cotangents across the edges of such tiles.  Chunks of two and three
planes with a remainder, on a general and on a product mesh, and tiles that
end on the padded extents with the node on the axis.

Bar: <Rbar, J v> = <Qbar, v> to 1e-11 against the oracle's complex-step
derivative, as in the other directional tests."""
import math

import numpy as np
import pytest
import torch

from _helpers import announce, make_solver, to_np
from cases import flow, mesh, problems
from oracle import les

pytestmark = pytest.mark.gpu

H_CS = 1e-30


def _wavy(n):
    xyz = mesh.wavy_coords(n, 2.0 * math.pi)
    return dict(xyz=xyz, Q=flow.modes_box_state(xyz, seed=2, kmax=2), inflow=None,
                params=problems.box_params(2.0 * math.pi, visc_coef=1e-3))


CASES = {
    "wavy80": lambda: _wavy(80),
    "jet93x61x86": lambda: problems.jet_problem(93, 61, 86, seed=26, thermo_noise=1e-3),
    "node28x12x8": lambda: problems.jet_problem(28, 12, 8, seed=27, noise=2e-3, thermo_noise=1e-3,
                                                axis_node=True),
    "node29x13x6": lambda: problems.jet_problem(29, 13, 6, seed=28, noise=2e-3, thermo_noise=1e-3,
                                                axis_node=True),
}


@pytest.mark.parametrize("case", list(CASES))
def test_vjp_at_chunk_and_tile_edges(case):
    announce("vjp tiles", case)
    pb = CASES[case]()
    geo = les.geometry(pb["xyz"].numpy(), pb["params"])
    Q = pb["Q"].numpy()
    Rbar = problems.seeded_field(Q.shape, 3, flow.FIELD_COTANGENT).numpy()
    v = problems.seeded_field(Q.shape, 11, flow.FIELD_DIRECTION).numpy()
    if pb["params"]["bc"][2] == "axis_node":      # R and Q of the axis row are derived data
        Rbar[:, :, 0], v[:, :, 0] = 0.0, 0.0
    s = make_solver(pb)
    Rb = s.pad(torch.from_numpy(Rbar).cuda(), fill=0.0)
    Qb = to_np(s.interior(s.residual_vjp(s.pad(pb["Q"].cuda()), Rb)))
    s.close()
    inflow = None if pb["inflow"] is None else pb["inflow"].numpy().astype(np.complex128)
    Jv = np.imag(les.evaluate(Q.astype(np.complex128) + 1j * H_CS * v, geo, pb["params"], inflow)) / H_CS
    lhs, rhs = float(np.sum(Rbar * Jv)), float(np.sum(Qb * v))
    print(case, lhs, rhs)
    assert abs(rhs - lhs) <= 1e-11 * abs(lhs)

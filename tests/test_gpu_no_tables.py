"""A product mesh without its metric tables (no memory for them, or LESJET_GENERAL=1)
takes the kernels of a general mesh: every call is served, with the results of the
tables' form.

Bars: residuals 1e-13 of the flux scale against the oracle (that of the parity tests);
the two forms, whose metric terms have the same bits and whose derived values differ
by two ulps, 1e-13 of each variable's largest value for totals and steps, 1e-11 for
the VJP (sums over a stencil of cancelling terms), and in FP32 1e-5 (that of the
FP32 tests)."""
import pytest
import torch

from _helpers import announce, flux_err, flux_scale, make_solver, rel_err, to_np
from cases import flow, problems
from oracle import les

pytestmark = pytest.mark.gpu

SHAPE = (17, 11, 14)


@pytest.mark.parametrize("axis_node", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_without_tables(precision, axis_node, monkeypatch):
    announce("no tables", precision, axis_node)
    pb = problems.jet_problem(*SHAPE, seed=2, noise=2e-3, thermo_noise=2e-3, axis_node=axis_node)
    prm, inflow, Q = pb["params"], pb["inflow"].numpy(), pb["Q"].numpy()
    Rbar = problems.seeded_field(Q.shape, 3, flow.FIELD_COTANGENT).cuda()
    out, held = [], []
    for general in (False, True):
        if general:
            monkeypatch.setenv("LESJET_GENERAL", "1")
        s = make_solver(pb, precision)
        held.append(s.query()[2])
        R = to_np(s.interior(s.residual(s.pad(pb["Q"].cuda()))))
        Qn = s.pad(pb["Q"].cuda(), dtype=torch.float64)
        tot = to_np(s.diagnostics(Qn))
        s.rk5_step(Qn, 2)
        vjp = None
        if precision == "fp64":
            vjp = to_np(s.interior(s.residual_vjp(s.pad(pb["Q"].cuda()), s.pad(Rbar, fill=0.0))))
        out.append((R, to_np(s.interior(Qn)), tot, vjp))
        s.close()
    nx, nr, nth = SHAPE
    assert held[0] - held[1] == 8 * (8 * (nr + 4) * (nth + 4) + 4 * (nx + 4))
    (R0, Q0, t0, v0), (R1, Q1, t1, v1) = out
    assert abs(t1 - t0).max() <= 1e-13 * abs(t0).max()
    if precision == "fp64":
        geo = les.geometry(pb["xyz"].numpy(), prm)
        scale = flux_scale(Q, geo, prm, inflow)
        assert flux_err(R1, les.evaluate(Q, geo, prm, inflow), scale).max() <= 1e-13
        assert rel_err(Q1, Q0) <= 1e-13
        assert rel_err(v1, v0) <= 1e-11
    else:
        assert rel_err(Q1, Q0) <= 1e-5

"""Product meshes (x a function of i, y and z of (j, k)): the stage kernel forms
their metric terms from tables, every other mesh reads the stored ones.  The
two-pass reference kernels always read the stored terms, and a mesh with a
single point off the product must be taken as general wherever that point
lies (first and last points, and the row and plane the tables come from).

Bars: both forms evaluate the same terms rounded alike, so FP64 residuals
agree to the 1e-13 of the flux scale of the parity tests and FP32 ones to the
1e-3 of max |R| of the FP32 form; a moved point of 1e-3 of a cell changes the
residual around it by far more."""
import numpy as np
import pytest

from _helpers import announce, flux_err, flux_scale, make_solver, per_variable_err, to_np
from cases import problems
from oracle import les

pytestmark = pytest.mark.gpu


def _residuals(pb, precision):
    s = make_solver(pb, precision)
    Q = s.pad(pb["Q"].cuda())
    out = [to_np(s.interior(f(Q))).astype(np.float64) for f in (s.residual, s.residual_reference)]
    s.close()
    return out


def _check(pb, precision):
    prm = pb["params"]
    inflow = pb["inflow"].numpy() if pb.get("inflow") is not None else None
    geo = les.geometry(pb["xyz"].numpy(), prm)
    Q = pb["Q"].numpy()
    ref = les.evaluate(Q, geo, prm, inflow)
    fused, two_pass = _residuals(pb, precision)
    if precision == "fp64":
        scale = flux_scale(Q, geo, prm, inflow)
        assert flux_err(fused, ref, scale).max() <= 1e-13
        assert flux_err(fused, two_pass, scale).max() <= 1e-13
    else:
        assert per_variable_err(fused, ref).max() <= 1e-3
        assert per_variable_err(fused, two_pass).max() <= 1e-3


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,axis_node,sgs", [((5, 5, 6), False, 1), ((15, 29, 16), False, 2),
                                                 ((31, 14, 18), True, 1), ((30, 6, 12), False, 3)])
def test_product_mesh_matches_the_stored_terms(shape, axis_node, sgs, precision):
    announce("product mesh", shape, axis_node, sgs, precision)
    pb = problems.jet_problem(*shape, seed=2, axis_node=axis_node, noise=0.02, thermo_noise=0.02)
    pb["params"] = dict(pb["params"], sgs_model=sgs)
    _check(pb, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("comp,point", [(0, (0, 0, 0)), (1, (7, 3, 5)), (2, (16, 10, 13)),
                                        (1, (0, 5, 5)), (0, (9, 0, 0))])
def test_one_point_off_the_product_is_a_general_mesh(comp, point, precision):
    announce("off the product", comp, point, precision)
    pb = problems.jet_problem(17, 11, 14, seed=2, noise=0.02, thermo_noise=0.02)
    i, j, k = point
    x = pb["xyz"].clone()
    x[comp, k, j, i] += 1e-3 * float(pb["grid"][1][1])
    pb["xyz"] = x
    _check(pb, precision)

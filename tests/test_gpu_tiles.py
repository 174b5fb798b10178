"""Sizes at which the marching and one-pass kernels can go wrong: tile widths of
the dynamic model's passes (14 x 14 and 30 x 8 outputs) and their remainders,
column groups of the diagnostics (32 columns, every eighth plane), and blocks
and plane chunks of the first pass over Q^n (256 columns, up to 16 planes).

Bars: the model's coefficients 1e-9 (ratios of sums with cancellation, as in
test_gpu_dynamic); totals and statistics 1e-13 of the sum of the magnitudes
(sums of at most 1e5 terms in trees of partial sums, rounding well below
1e3 eps); the time step 1e-13 (a few roundings per point, one maximum)."""
import math

import numpy as np
import pytest
import torch

from _helpers import announce, make_solver, to_np
from cases import flow, mesh, problems
from oracle import les

pytestmark = pytest.mark.gpu

L = 2.0 * math.pi


def _box(shape, kind="box"):
    """Product (box) or general (wavy) periodic mesh with the multi-mode state."""
    xyz = mesh.wavy_coords(shape[0], L) if kind == "wavy" else mesh.box_coords(0, L, shape=shape)
    return dict(xyz=xyz, Q=flow.modes_box_state(xyz, seed=2, kmax=2), inflow=None,
                params=problems.box_params(L, sgs_model=3, visc_coef=1e-3))


def _filled(pb):
    geo = les.geometry(pb["xyz"].numpy(), pb["params"])
    Qp = les.pad_state(pb["Q"].numpy())
    les.fill_ghosts(Qp, geo, pb["params"],
                    pb["inflow"].numpy() if pb.get("inflow") is not None else None)
    return geo, Qp


@pytest.mark.parametrize("shape,kind", [((14, 14, 6), "box"), ((15, 13, 5), "box"),
                                        ((28, 8, 9), "box"), ((29, 9, 7), "box"),
                                        ((31, 43, 18), "box"), ((15, 15, 15), "wavy"),
                                        ((30, 30, 30), "wavy")])
def test_dynamic_coefficients_at_tile_edges(shape, kind):
    announce("dynamic tiles", shape, kind)
    pb = _box(shape, kind)
    geo, Qp = _filled(pb)
    d = les.dynamic_coefficients(Qp, geo, pb["params"])
    s = make_solver(pb)
    Q = s.pad(pb["Q"].cuda())
    c = s.dynamic_coefficients(Q)
    assert s.dynamic_coefficients(Q) == c                       # reproducible
    s.close()
    print(shape, kind, c, d["C_I"], d["C_ds"], d["Pr_sgs"])
    for got, ref in ((c[0], d["C_I"]), (c[1], d["C_ds"]), (c[5], d["Pr_eff"])):
        assert abs(got - ref) <= 1e-9 * abs(ref) + 1e-15


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,kind", [((5, 5, 6), "jet"), ((8, 4 + 4, 8), "jet"),
                                        ((33, 31, 10), "jet"), ((16, 16, 33), "box"),
                                        ((17, 17, 17), "wavy"), ((129, 63, 18), "jet")])
def test_diagnostics_and_time_step_at_group_edges(shape, kind, precision):
    announce("diagnostics groups", shape, kind, precision)
    pb = problems.jet_problem(*shape, seed=2, noise=0.02, thermo_noise=0.02) if kind == "jet" \
        else _box(shape, kind)
    pb["params"] = dict(pb["params"], sgs_model=0)
    geo = les.geometry(pb["xyz"].numpy(), pb["params"])
    Q = pb["Q"].numpy()
    s = make_solver(pb, precision, keep_metrics=True)
    Qn = s.pad(pb["Q"].cuda(), dtype=torch.float64)
    V = to_np(s.interior(s.metrics64))[9]
    if precision == "fp32":
        V = V.astype(np.float32).astype(np.float64)
    st = s.new_stats()
    tot = to_np(s.diagnostics(Qn, st))
    assert np.array_equal(tot, to_np(s.diagnostics(Qn)))       # the same without statistics
    one = s.new_stats()
    s.diagnostics(Qn, (None, one[1]))
    assert np.array_equal(to_np(one[1]), to_np(st[1]))
    for c in range(5):
        assert abs(tot[c] - math.fsum((V * Q[c]).ravel())) <= 1e-13 * np.abs(V * Q[c]).sum()
    f = np.stack(les.primitives(Q, 1.4))
    for got, ref, mag in ((st[0], f.sum(1), np.abs(f).sum(1)), (st[1], (f * f).sum(1), (f * f).sum(1))):
        # the primitives round relative to the terms that form them (p from E)
        assert (np.abs(to_np(got) - ref) <= 1e-13 * np.maximum(mag, mag.max())).all()
    dt = float(s.rk5_step(Qn, 1)[0])
    if precision == "fp64":
        assert abs(dt - les.time_step(Q, geo, pb["params"])) <= 1e-13 * dt
    else:                                                       # metrics rounded to FP32
        assert abs(dt - les.time_step(Q, geo, pb["params"])) <= 1e-6 * dt
    s.close()

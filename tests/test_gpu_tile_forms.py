"""Both tiles of the stage kernel, forced by LESJET_TILE, in every instance a step
takes: product, general and axis-node meshes, both update schedules, the dynamic
model, both precision forms, at shapes that end inside a tile of either width and with
chunks of five planes and a remainder.

Bars against the oracle: residuals 1e-13 of the flux scale (1e-12 with the dynamic model; FP32 1e-3 of max |R|), the
state after two steps 1e-11 (1e-5), both time steps 1e-11 (1e-5); those of the
parity, dynamic-model and FP32 tests, the second step taking the first one's last-
stage reduction.  Narrow against wide at the same chunk length: the same arithmetic per
point, so in FP32, where a rounding would grow to the storage type's, the same
bits."""
import math

import numpy as np
import pytest
import torch

from _helpers import announce, flux_err, flux_scale, grouped_rel_err, make_solver, to_np
from cases import flow, mesh, problems
from oracle import les

pytestmark = pytest.mark.gpu


def _problem(shape, kind, sgs, schedule):
    if kind in ("wavy", "box"):
        L = 2.0 * math.pi
        xyz = mesh.wavy_coords(shape[0], L) if kind == "wavy" else mesh.box_coords(0, L, shape=shape)
        pb = dict(xyz=xyz, Q=flow.modes_box_state(xyz, seed=2, kmax=2), inflow=None,
                  params=problems.box_params(L, visc_coef=1e-3))
    else:
        pb = problems.jet_problem(*shape, seed=2, axis_node=kind == "node", noise=2e-3,
                                  thermo_noise=2e-3)
    pb["params"] = dict(pb["params"], sgs_model=sgs, schedule=schedule)
    return pb


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,kind,sgs,schedule,general", [
    *(c + (g,) for g in (False, True) for c in (
        ((31, 15, 18), "jet", 1, "stage"), ((32, 17, 12), "jet", 2, "step"),
        ((31, 15, 16), "node", 1, "stage"), ((33, 9, 12), "node", 2, "step"),
        ((33, 17, 11), "box", 3, "stage"), ((17, 33, 11), "box", 3, "step"))),
    ((17, 17, 17), "wavy", 1, "stage", True), ((33, 33, 33), "wavy", 2, "step", True)])
def test_both_tiles(shape, kind, sgs, schedule, general, precision, monkeypatch):
    announce("tile forms", shape, kind, sgs, schedule, general, precision)
    pb = _problem(shape, kind, sgs, schedule)
    prm = pb["params"]
    inflow = pb["inflow"].numpy() if pb.get("inflow") is not None else None
    geo = les.geometry(pb["xyz"].numpy(), prm)
    Q = pb["Q"].numpy()
    ref_R = les.evaluate(Q, geo, prm, inflow)
    ref, dts = les.run(Q, geo, prm, inflow, steps=2)
    rows = slice(1 if kind == "node" else 0, None)      # the axis row is derived data
    monkeypatch.setenv("LESJET_KCHUNK", "5")
    if general:
        monkeypatch.setenv("LESJET_GENERAL", "1")
    out = []
    for tile in ("narrow", "wide"):
        monkeypatch.setenv("LESJET_TILE", tile)
        s = make_solver(pb, precision)
        R = s.interior(s.residual(s.pad(pb["Q"].cuda()))).clone()
        Qn = s.pad(pb["Q"].cuda(), dtype=torch.float64)
        dt = to_np(s.rk5_step(Qn, 2))
        got = s.interior(Qn).clone()
        s.close()
        out.append((R, got))
        if precision == "fp64":
            scale = flux_scale(Q, geo, prm, inflow)
            assert flux_err(to_np(R), ref_R, scale).max() <= (1e-12 if sgs == 3 else 1e-13)
        else:
            assert grouped_rel_err(to_np(R).astype(np.float64), ref_R) <= 1e-3
        bar = 1e-11 if precision == "fp64" else 1e-5
        assert np.allclose(dt, dts, rtol=bar, atol=0)
        assert grouped_rel_err(to_np(got)[:, :, rows], ref[:, :, rows]) <= bar
    if precision == "fp32":
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])

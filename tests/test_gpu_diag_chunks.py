"""Diagnostics of meshes of few (i, j) columns, whose azimuth is cut into chunks of
planes: lengths one short of, at and one past the point where a chunk is added,
remainders, and column counts on both sides of a group of 32.

Bars: totals 1e-13 of the sum of the magnitudes (sums of at most 1e5 terms in trees
of partial sums), the same bits with and without statistics.  Totals alone of a mesh
of 64 columns may take at most five times those of a mesh of 8,192 columns with as
many points: both are a launch over 0.5 M points that fills the device, the long
one's rows being 8 points, an eighth of a line in the worst case; one block per
column group, 2 of them, took 40 times as long."""
import math

import numpy as np
import pytest
import torch

from _helpers import announce, make_solver, to_np
from cases import flow, mesh, problems
from oracle import les

pytestmark = pytest.mark.gpu

L = 2.0 * math.pi


def _box(shape):
    xyz = mesh.box_coords(0, L, shape=shape)
    return dict(xyz=xyz, Q=flow.modes_box_state(xyz, seed=2, kmax=2), inflow=None,
                params=problems.box_params(L, sgs_model=0, visc_coef=1e-3))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(5, 5, 32), (5, 5, 33), (8, 8, 63), (8, 8, 65), (16, 16, 130),
                                   (32, 32, 97), (33, 31, 64), (7, 5, 1000), (128, 64, 41)])
def test_totals_at_chunk_edges(shape, precision):
    announce("diagnostics chunks", shape, precision)
    pb = _box(shape)
    Q = pb["Q"].numpy()
    s = make_solver(pb, precision, keep_metrics=True)
    Qn = s.pad(pb["Q"].cuda(), dtype=torch.float64)
    V = to_np(s.interior(s.metrics64))[9]
    if precision == "fp32":
        V = V.astype(np.float32).astype(np.float64)
    st = s.new_stats()
    tot = to_np(s.diagnostics(Qn, st))
    alone = to_np(s.diagnostics(Qn))
    assert np.array_equal(tot, alone)
    s.close()
    for c in range(5):
        assert abs(tot[c] - math.fsum((V * Q[c]).ravel())) <= 1e-13 * np.abs(V * Q[c]).sum()
    f = np.stack(les.primitives(Q, 1.4))
    for got, ref, mag in ((st[0], f.sum(1), np.abs(f).sum(1)), (st[1], (f * f).sum(1), (f * f).sum(1))):
        assert (np.abs(to_np(got) - ref) <= 1e-13 * np.maximum(mag, mag.max())).all()


def _totals_ms(shape):
    s = make_solver(_box(shape))
    Qn = s.field(5, dtype=torch.float64, fill=1.0)
    best = math.inf
    for _ in range(10):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            s.diagnostics(Qn)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 10)
    s.close()
    return best


def test_totals_of_few_columns_fill_the_device():
    few, many = _totals_ms((8, 8, 8192)), _totals_ms((128, 64, 64))
    announce("totals of few columns", few, many)
    assert few <= 5.0 * many

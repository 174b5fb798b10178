"""Whether a mesh is taken as a product, read from the device memory its context
holds: the metric tables are kept for a product mesh only.  In FP32 storage a point
that is off by 1e-3 of a cell changes residuals by less than the bar of that form,
so the residual cannot tell.  Points at the first and last indices, in the row and the
plane the tables come from, and next to the periodic seam."""
import pytest

from _helpers import announce, make_solver
from cases import problems

pytestmark = pytest.mark.gpu

SHAPE = (17, 11, 14)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("axis_node", [False, True])
def test_one_moved_point_gives_up_the_tables(axis_node, precision):
    pb = problems.jet_problem(*SHAPE, seed=2, axis_node=axis_node)
    nx, nr, nth = SHAPE
    tables = 8 * (8 * (nr + 4) * (nth + 4) + 4 * (nx + 4))

    def held(xyz):
        s = make_solver(dict(pb, xyz=xyz), precision)
        b = s.query()[2]
        s.close()
        return b

    product = held(pb["xyz"])
    for comp in range(3):
        for point in ((0, 0, 0), (16, 10, 13), (7, 3, 5), (0, 5, 5), (9, 0, 0), (16, 0, 7), (3, 10, 0)):
            announce("product choice", axis_node, precision, comp, point)
            i, j, k = point
            x = pb["xyz"].clone()
            x[comp, k, j, i] += 1e-3 * float(pb["grid"][1][1])
            assert product - held(x) == tables, (comp, point)

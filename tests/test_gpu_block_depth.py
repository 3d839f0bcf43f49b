"""The stencil passes where the block list takes deep blocks (8 planes: many blocks, mostly solid) and
its usual ones (4 planes: as many blocks, mostly fluid), on long grids whose ends leave remainders,
and two planes with enough tile rows for eight bands, too few and just enough planes; against the
FP64 oracle.

Tolerances as the other parity tests: FP32 rounding of the fields gives about 1e-6 after a few
steps, far below 1e-4; FP64 differs from the oracle by the order of its sums, below 1e-11.
"""
import numpy as np
import pytest
import torch

from oracle.oracle import Model
from paper_1709_02733_amd import el
from paper_1709_02733_amd import scenarios as S
from tests.gpu_util import banner, need_gpu, rel_l2, rel_max

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(request):
    need_gpu()
    banner(request.node.nodeid)
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("shape,npml,fluid", [
    ((33, 6, 13705), 1, 0.0), ((33, 6, 13699), 0, 0.0), ((33, 6, 13705), 1, 1.0),
    ((65, 33, 20), 2, 0.5), ((33, 40, 47), 3, 0.5)])
@pytest.mark.parametrize("precision,tol", [("f32", 1e-4), ("f64", 1e-11)])
def test_block_depths(shape, npml, fluid, precision, tol):
    sc = S.random_scenario(shape, seed=5, nsteps=6, npml=npml, nrec=300, fluid_fraction=fluid)
    plan = el.Plan.from_scenario(sc, precision=precision)
    ref = Model.from_scenario(sc)
    y = np.random.default_rng(3).standard_normal((sc.nsteps, sc.nrec))
    for got, want in ((plan.forward(torch.from_numpy(sc.p0)), ref.forward(sc.p0.astype(np.float64))),
                      (plan.adjoint(torch.from_numpy(y)), ref.adjoint(y))):
        got = got.cpu().numpy().astype(np.float64)
        assert rel_l2(got, want) <= tol and rel_max(got, want) <= tol

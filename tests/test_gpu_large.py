"""The stencil passes where the block list takes deep blocks with the mapping of large grids, fluid
and mixed sub-tiles among them, and where the state outgrows the Infinity Cache and the general update
streams its fields; against the FP64 oracle, the general update alone and the grouped passes.

Tolerances as the other parity tests: FP32 rounding of the fields gives about 1e-6 after a few steps,
far below 1e-4; FP64 differs from the oracle by the order of its sums, below 1e-11.  The depth and the
streaming of each case are asserted on the host in test_block_list.py."""
import numpy as np
import pytest
import torch

from oracle.oracle import Model
from paper_1709_02733_amd import el
from tests import large_media as LM
from tests.gpu_util import banner, need_gpu, rel_l2, rel_max

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(request):
    need_gpu()
    banner(request.node.nodeid)
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("case", range(len(LM.CASES)))
def test_large_media(case):
    shape, npml, fluid, radius, size, _, _ = LM.CASES[case]
    sc, _ = LM.scenario(shape, npml, fluid, radius)
    tol = 1e-4 if size == 4 else 1e-11
    plan = el.Plan.from_scenario(sc, precision="f32" if size == 4 else "f64")
    assert (plan.fluid_path()[0] > 0) == (fluid > 0)
    ref = Model.from_scenario(sc)
    p0 = torch.from_numpy(sc.p0).to(plan.device, plan.dtype)
    y = torch.from_numpy(np.random.default_rng(3).standard_normal((sc.nsteps, sc.nrec))).to(plan.device)
    want = [ref.forward(sc.p0.astype(np.float64)), ref.adjoint(y.cpu().numpy())]
    got = [plan.forward(p0), plan.adjoint(y)]
    plan.fluid_path(False)
    general = [plan.forward(p0), plan.adjoint(y)]
    plan.fluid_path(True)
    for a, b, w in zip(got, general, want):
        for v in (a, b):
            v = v.cpu().numpy().astype(np.float64)
            assert rel_l2(v, w) <= tol and rel_max(v, w) <= tol
    # the grouped passes take the same loops: bitwise
    for op, inp, a in ((el.OP_FORWARD, p0, got[0]), (el.OP_ADJOINT, y, got[1])):
        g = el.Group(max_members=1, precision=plan.grid.precision)
        out = torch.zeros_like(a)
        slot = g.add(plan, op, inp, out)
        g.run(sc.nsteps)
        g.sync()
        assert g.poll(slot)[1] and torch.equal(out, a)
        g.close()

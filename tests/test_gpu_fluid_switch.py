"""A change of the fluid-update setting while an operation is under way.

A group's member and an executor's operation with a replay limit are enqueued in parts; a call of
el_plan_fluid_path in between returns before they are done.  The operation goes on under the setting
it began with: its result is bitwise that of the direct call under that setting, and the next
operation takes the new one.
"""
import numpy as np
import pytest
import torch

from paper_1709_02733_amd import el
from paper_1709_02733_amd import scenarios as S
from tests.gpu_util import banner, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(request):
    need_gpu()
    banner(request.node.nodeid)
    yield
    torch.cuda.synchronize()


def _case(precision, op):
    """A plan with fluid tiles, general tiles and mixed ones, receivers in the fluid; the operation's
    input and its results without and with the fluid update."""
    sc = S.random_scenario((70, 33, 29), seed=7, nsteps=41, npml=3, nrec=50, fluid_fraction=1.0)
    sc.mu[12:17, 14:19, 20:44] = 2.0e8   # a solid in the fluid: c_l <= 1.25 x the fluid's
    sc.dt *= 0.7
    plan = el.Plan.from_scenario(sc, precision=precision)
    if op == el.OP_FORWARD:
        inp = torch.from_numpy(sc.p0).to(plan.device, plan.dtype)
        call = plan.forward
    else:
        inp = torch.from_numpy(np.random.default_rng(3).standard_normal((sc.nsteps, sc.nrec))).to(plan.device)
        call = plan.adjoint
    plan.fluid_path(False)
    off = call(inp).clone()
    assert plan.fluid_path(True)[0] > 0
    on = call(inp).clone()
    torch.cuda.synchronize()
    assert not torch.equal(on, off)   # other sums next to the solid
    return plan, inp, [off, on], call


@pytest.mark.parametrize("began", [True, False])
@pytest.mark.parametrize("op", [el.OP_FORWARD, el.OP_ADJOINT])
@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_group_member_keeps_its_setting(precision, op, began):
    plan, inp, want, call = _case(precision, op)
    plan.fluid_path(began)
    g = el.Group(max_members=2, precision=plan.grid.precision)
    out = torch.zeros_like(want[0])
    slot = g.add(plan, op, inp, out)
    g.run(13)
    plan.fluid_path(not began)
    g.run(100)
    g.sync()
    assert g.poll(slot)[1]
    assert torch.equal(out, want[began])
    assert torch.equal(call(inp), want[not began])
    g.close()


@pytest.mark.parametrize("began", [True, False])
@pytest.mark.parametrize("op", [el.OP_FORWARD, el.OP_ADJOINT])
@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_executor_slot_keeps_its_setting(precision, op, began):
    plan, inp, want, call = _case(precision, op)
    plan.fluid_path(began)
    ex = el.Executor(max_slots=2, chunk=6, ahead=1)
    out = torch.zeros_like(want[0])
    slot = ex.start(plan, op, inp, out)   # one replay of seven is enqueued
    plan.fluid_path(not began)
    ex.wait(slot)
    assert torch.equal(out, want[began])
    assert torch.equal(call(inp), want[not began])
    ex.close()

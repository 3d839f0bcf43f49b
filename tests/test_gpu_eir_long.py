"""Transducer response (el_eir_apply) with more taps than the traces have samples: no sample has a
term beyond the ends of its trace, so the taps from nsteps on change neither the result nor the time."""
import numpy as np
import pytest
import torch

from oracle.eir import eir_adjoint, eir_apply
from paper_1709_02733_amd import el
from tests.gpu_util import banner, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(request):
    need_gpu()
    banner(request.node.nodeid)
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("M,L", [(1, 1), (7, 3), (8, 64), (41, 70), (1030, 1030)])
@pytest.mark.parametrize("more", [1, 8, 3000])
@pytest.mark.parametrize("transpose", [False, True])
def test_taps_beyond_the_trace_change_nothing(M, L, more, transpose):
    rng = np.random.default_rng(M + more)
    h, z = rng.standard_normal(M + more), rng.standard_normal((M, L))
    dev = torch.from_numpy(z).cuda()
    got = el.eir_apply(torch.from_numpy(h), dev, transpose=transpose)
    assert torch.equal(got, el.eir_apply(torch.from_numpy(h[:M].copy()), dev, transpose=transpose))
    cols = np.r_[0:min(L, 3), L - 1]
    ref = eir_adjoint if transpose else eir_apply
    # sums of at most M products in double: M half-ulps of the sum of their magnitudes
    err = np.abs(got.cpu().numpy()[:, cols] - ref(h, z[:, cols]))
    assert np.all(err <= 2.0 ** -52 * M * ref(np.abs(h), np.abs(z[:, cols])))


def test_the_longest_kernel_there_is():
    M, L = 600, 70
    z = torch.from_numpy(np.random.default_rng(5).standard_normal((M, L))).cuda()
    h = torch.zeros(2 ** 31 - 1, dtype=torch.float64, device="cuda")
    h[:M] = torch.linspace(1.0, 2.0, M, dtype=torch.float64)
    h[M:M + 5000] = float("nan")
    for t in (False, True):
        assert torch.equal(el.eir_apply(h, z, transpose=t), el.eir_apply(h[:M].clone(), z, transpose=t))


@pytest.mark.parametrize("transpose", [False, True])
def test_taps_beyond_the_trace_cost_nothing(transpose):
    """Ten times the samples' taps: ten times the work if they were run, none if not."""
    M, L = 2500, 1024
    z = torch.randn((M, L), dtype=torch.float64, device="cuda")
    h = torch.randn(10 * M, dtype=torch.float64, device="cuda")

    def best(taps):
        k, times = h[:taps].clone(), []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            el.eir_apply(k, z, transpose=transpose)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    assert best(10 * M) <= 2.0 * best(M)

"""Transducer response (el_eir_apply) where its register windows end: taps and samples that are no
multiple of the samples per thread (8 for many traces, 4 for few), more taps than samples, and
non-finite values, which reach only the samples whose sum holds them."""
import numpy as np
import pytest
import torch

from oracle.eir import eir_adjoint, eir_apply
from paper_1709_02733_amd import el

pytestmark = pytest.mark.gpu


def _both(h, z):
    dev = torch.from_numpy(z).cuda()
    return [el.eir_apply(torch.from_numpy(h), dev, transpose=t).cpu().numpy() for t in (False, True)]


@pytest.mark.parametrize("M,L", [(1025, 1023), (1039, 1024), (37, 70), (3, 1), (16, 65)])
@pytest.mark.parametrize("nh", [1, 7, 8, 9, 29, 1100])
def test_window_edges(M, L, nh):
    rng = np.random.default_rng(M + nh)
    h, z = rng.standard_normal(nh), rng.standard_normal((M, L))
    cols = np.r_[0:min(L, 3), L - 1]                       # the oracle's columns are independent
    for got, ref in zip(_both(h, z), (eir_apply, eir_adjoint)):
        want = ref(h, z[:, cols])
        # sums of at most nh products in double: nh half-ulps of the sum of their magnitudes
        mags = ref(np.abs(h), np.abs(z[:, cols]))
        assert np.all(np.abs(got[:, cols] - want) <= 2.0 ** -52 * nh * mags)


@pytest.mark.parametrize("M,L", [(1030, 1024), (37, 70)])
def test_non_finite_values_stay_where_they_belong(M, L):
    rng = np.random.default_rng(7)
    nh, k, m = 21, 10, 20
    h, z = rng.standard_normal(nh), rng.standard_normal((M, L))
    z[m, 5] = np.nan
    sample = np.arange(M)
    for got, reach in zip(_both(h, z), ((sample >= m) & (sample < m + nh), (sample <= m) & (sample > m - nh))):
        assert np.array_equal(np.isnan(got[:, 5]), reach) and not np.isnan(got[:, 6]).any()
    z[m, 5], h[k] = 1.0, np.inf
    for got, reach in zip(_both(h, z), (sample >= k, sample < M - k)):
        assert np.array_equal(~np.isfinite(got).all(axis=1), reach)

"""Log-derivatives of a ln cosh network with a weight that is not a number or
infinite: the columns that depend on it are NaN (or the limit), the others
those of the same network without it."""
import numpy as np
import pytest
import torch

from paper_2204_07816_amd import inputs, nqs

pytestmark = pytest.mark.gpu


def rows(L, K, C, w, sp, odt):
    return nqs.Context(L, 1.0, 0.5, K, C, w).log_deriv(sp, dtype=odt).cpu().numpy()


@pytest.mark.parametrize("odt", ["fp64", "fp32"])
@pytest.mark.parametrize("L,C", [(4, 3), (6, 16), (10, 32)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_one_layer(L, C, odt, value):
    c = C - 2
    w = inputs.stress_weights(1, C, 1.0, 81)
    sp = torch.as_tensor(inputs.spins_any(L, 5, 82)).cuda()
    ref = rows(L, 1, C, w, sp, odt)
    w[9 * C + c] = value                          # channel c's bias
    got = rows(L, 1, C, w, sp, odt)
    own = np.zeros(10 * C, bool)
    own[9 * c:9 * c + 9] = own[9 * C + c] = True
    assert np.array_equal(got[:, ~own], ref[:, ~own])
    if np.isnan(value):
        assert np.all(np.isnan(got[:, own]))
    else:                                         # tanh is 1: sums of the spins
        m = sp.cpu().numpy().reshape(5, -1).sum(1)
        assert np.array_equal(got[:, 9 * c:9 * c + 9], np.repeat(m[:, None], 9, 1).astype(got.dtype))
        assert np.all(got[:, 9 * C + c] == L * L)


@pytest.mark.parametrize("C", [3, 16])
@pytest.mark.parametrize("K", [2, 3])
def test_deeper_networks(K, C):
    """A NaN of the first layer reaches every column."""
    L = 6
    w = inputs.stress_weights(K, C, 1.0, 83)
    w[9 * C] = np.nan
    sp = torch.as_tensor(inputs.spins_any(L, 3, 84)).cuda()
    assert np.all(np.isnan(rows(L, K, C, w, sp, "fp64")))

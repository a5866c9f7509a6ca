"""The exact neuron step where the gains favour or shun a device, so that most of the layer is in
excess at first and prices move before the paths do: against the exact oracle, bit for bit (host
only).  Gains whose range leaves no room for prices in 64 bits take the paths alone."""
import numpy as np
import pytest

from oracle import layout as lay
from paper_2609_13846_amd import dtp


@pytest.mark.parametrize("I,L", [(3, 3), (6, 3), (33, 3), (96, 3), (64, 4), (132, 4), (240, 4), (40, 5), (64, 8), (160, 8)])
@pytest.mark.parametrize("kind", ["one", "two", "slope", "equal", "levels", "wide"])
@pytest.mark.parametrize("minimise", [False, True])
def test_skewed_gains_bit_exact(I, L, kind, minimise):
    rng = np.random.default_rng(I * 10 + L)
    Q = rng.integers(1, 1000, (L, I)).astype(np.int64)  # one group per device: M[k][l] = Q[h^-1(l)][k]
    if kind == "one":
        Q[0] *= 5
    elif kind == "two":
        Q[:2] += 900
    elif kind == "slope":
        Q = Q // 50 + 100 * np.arange(L)[:, None]
    elif kind == "equal":  # every neuron the same gains: all is ties
        Q[:] = Q[:, :1]
    elif kind == "levels":
        Q = Q % 3 + 2 * (np.arange(L) == 1)[:, None]
    else:  # a range of 2^56, beyond what prices are taken for
        Q = Q * (1 << 46) + (np.arange(L)[:, None] == 0) * (1 << 55)
    h = rng.permutation(L).astype(np.int32)
    nu, value = dtp.dtp_balanced_assign(L, I, L, Q, h, minimise=minimise)
    M = lay.neuron_gain(Q, h, L)
    nu_ref, v_ref = lay.balanced_assign(M, minimise)
    np.testing.assert_array_equal(nu, nu_ref)
    assert value == v_ref

"""The neuron step for two devices, which runs on the device: the selection's edges (keys in
LDS and in memory, whole and ragged blocks, ties at the threshold) against the exact oracle
and against the library's host step, bit for bit."""
import numpy as np
import pytest

from oracle import layout as lay
from paper_2609_13846_amd import dtp
from tests.test_gpu_layout import announce

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,G,I,levels", [(1, 2, 2, 0), (2, 4, 6, 2), (2, 8, 1022, 3), (1, 16, 1024, 0),
                                          (3, 8, 1026, 2), (2, 8, 7168, 4), (2, 8, 7170, 4), (1, 8, 14336, 0)])
@pytest.mark.parametrize("minimise", [False, True])
def test_two_device_neuron_step_bit_exact(N, G, I, levels, minimise):
    announce(f"two-device neuron step N={N} G={G} I={I} levels={levels} minimise={minimise}")
    rng = np.random.default_rng(N * 1000 + I)
    # few levels: most neurons tie with the threshold, and the index order decides
    draw = (lambda s: rng.integers(1, levels + 1, s)) if levels else (lambda s: rng.random(s) + 0.01)
    Au = draw((N, G, I)).astype(np.float32)
    Ad = draw((N - 1, I, G)).astype(np.float32) if N > 1 else None
    args = (N, G, I, 2, torch.from_numpy(Au).cuda(), None if Ad is None else torch.from_numpy(Ad).cuda())
    Qu = [lay.encode(a) for a in Au]
    Qd = None if Ad is None else [lay.encode(a) for a in Ad]
    hs, nus, J, sweeps = lay.coordinate_ascent(Qu, Qd, 2, minimise=minimise)
    res = dtp.dtp_coordinate_ascent(*args, minimise=minimise)
    np.testing.assert_array_equal(res["h"], np.array(hs))
    np.testing.assert_array_equal(res["nu"], np.array(nus))
    assert res["J_fixed"] == J and res["sweeps"] == sweeps
    # one sweep: the step from the contiguous heads
    one = dtp.dtp_coordinate_ascent(*args, minimise=minimise, max_sweeps=1)
    h0 = (np.arange(G) // (G // 2)).astype(np.int32)
    for i in range(N):
        down = (Qd[i], h0) if i + 1 < N else (None, None)
        nu, _ = dtp.dtp_balanced_assign(G, I, 2, Qu[i], h0, *down, minimise)
        np.testing.assert_array_equal(one["nu"][i], nu)

"""Ascents whose heads stay put (`freeze_heads`, or a mask of all layers) against the exact oracle,
bit for bit.  They score no partitions, so neither the time nor what is accepted depends on how
many there are: 5,300 layers of 12,870 partitions are more wavefronts than one launch of the scoring
holds (2^32 threads)."""
import numpy as np
import pytest

from oracle import layout as lay
from paper_2609_13846_amd import dtp
from tests.test_gpu_layout import announce

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,G,I,L,down,kw", [
    (1, 1, 3, 1, False, {}),
    (3, 8, 40, 2, True, {}),
    (6, 12, 24, 4, True, dict(minimise=True)),      # a block of four layers and a rest
    (4, 8, 64, 8, False, {}),
    (2, 22, 44, 2, True, dict(freeze_neurons=True)),  # 705,432 partitions, nothing moves
    (3, 4, 8, 4, True, dict(layer_mask=[0, 0, 0])),
    (5300, 16, 2, 2, True, {}),
])
def test_frozen_heads_bit_exact(N, G, I, L, down, kw):
    announce(f"frozen heads N={N} G={G} I={I} L={L} down={down} {kw}")
    rng = np.random.default_rng(N + G + I)
    Au = (rng.random((N, G, I)) + 0.01).astype(np.float32)
    Ad = (rng.random((N - 1, I, G)) + 0.01).astype(np.float32) if down else None
    okw = dict(kw)
    if "layer_mask" not in kw:
        okw["freeze_heads"] = True
    hs, nus, J, sweeps = lay.coordinate_ascent([lay.encode(a) for a in Au],
                                               None if Ad is None else [lay.encode(a) for a in Ad], L, **okw)
    res = dtp.dtp_coordinate_ascent(N, G, I, L, torch.from_numpy(Au).cuda(),
                                    None if Ad is None else torch.from_numpy(Ad).cuda(), **okw)
    np.testing.assert_array_equal(res["h"], np.array(hs))
    np.testing.assert_array_equal(res["nu"], np.array(nus))
    assert res["J_fixed"] == J and res["sweeps"] == sweeps

"""Ascents whose neuron step runs on the host, on both sides of the size from which the gain
matrices are summed on the device (48 KiB of codes) and of 256 KiB of them, against the exact
oracle, bit for bit."""
import numpy as np
import pytest

from oracle import dual_ascent as da
from oracle import layout as lay
from paper_2609_13846_amd import dtp
from tests.test_gpu_layout import announce

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,G,I,L,levels,kw", [
    (1, 1, 1, 1, 0, {}),
    (1, 4, 4, 4, 0, {}),
    (1, 4, 1536, 4, 0, {}),                              # 48 KiB
    (1, 4, 1540, 4, 0, {}),                              # one neuron per device more
    (2, 6, 255, 3, 0, {}),                               # 48 KiB less 192 bytes, with down edges
    (2, 6, 258, 3, 3, {}),
    (5, 4, 96, 4, 2, dict(minimise=True)),
    (5, 4, 96, 4, 0, dict(layer_mask=[1, 0, 0, 1, 1])),
    (6, 6, 60, 3, 2, dict(max_sweeps=2)),
    (6, 6, 120, 3, 0, dict(layer_mask=[0, 1, 1, 0, 1, 0])),
    (4, 4, 64, 2, 2, dict(dual_ascent_neurons=True)),
    (4, 4, 512, 2, 0, dict(dual_ascent_neurons=True)),
    (9, 8, 1200, 4, 0, {}),                              # gains of more than 256 KiB
])
def test_host_neuron_step_bit_exact(N, G, I, L, levels, kw):
    announce(f"host neuron step N={N} G={G} I={I} L={L} levels={levels} {kw}")
    rng = np.random.default_rng(N * 100 + I)
    draw = (lambda s: rng.integers(1, levels + 1, s)) if levels else (lambda s: rng.random(s) + 0.01)
    Au = draw((N, G, I)).astype(np.float32)
    Ad = draw((N - 1, I, G)).astype(np.float32) if N > 1 else None
    okw = dict(kw)
    if okw.pop("dual_ascent_neurons", False):
        okw["neuron_step"] = lambda M, minimise: da.assign(-M if minimise else M)[0]
    hs, nus, J, sweeps = lay.coordinate_ascent([lay.encode(a) for a in Au],
                                               None if Ad is None else [lay.encode(a) for a in Ad], L, **okw)
    res = dtp.dtp_coordinate_ascent(N, G, I, L, torch.from_numpy(Au).cuda(),
                                    None if Ad is None else torch.from_numpy(Ad).cuda(), **kw)
    np.testing.assert_array_equal(res["h"], np.array(hs))
    np.testing.assert_array_equal(res["nu"], np.array(nus))
    assert res["J_fixed"] == J and res["sweeps"] == sweeps

"""1/r of long fp32 rows.  The layer is built so that everything but 1/r is exact: one head whose
folded rows are small whole numbers (W_o picks the first columns of W'), one-hot attention, and the
ADD score, so that an entry of A is (1/r)^2 times a whole number.  1/r itself is held to 3
roundings (the row's mean in more than 32 bits, then the root, the quotient and the result), A to
twice that and the three roundings of its own products and sums: 9 * 2^-24, and 10 for the
second order.  A chain of d / 4 additions in 32 bits is off by tens of roundings at these
sizes (about sqrt(d / 4) / 2 of them)."""
import numpy as np
import pytest

from paper_2609_13846_amd import dtp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [16, 4096, 16384, 65536])
def test_f32_row_norms_of_long_rows(d):
    import torch
    print(f"[gpu] f32 1/r d={d}", flush=True)
    I, dh, eps = 64, 16, 1e-6
    rng = np.random.default_rng(d)
    gate, up = np.zeros((I, d), np.float32), np.zeros((I, d), np.float32)
    gate[:, :dh] = rng.integers(1, 9, (I, dh))
    up[:, :dh] = rng.integers(1, 9, (I, dh))
    w_o = np.zeros((d, dh), np.float32)
    w_o[np.arange(dh), np.arange(dh)] = 1
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).cuda()
    layer = dtp.dtp_layer_create(d, I, 1, 1, dh, eps, dtp.DTP_F32)
    worst = 0.0
    try:
        dtp.dtp_layer_set_weights(layer, dev(w_o), torch.ones(d, device="cuda"), dev(gate), dev(up),
                                  torch.ones(d, I, device="cuda"))
        for t in range(8):
            x = (rng.random(d) + 0.5).astype(np.float32)
            a = np.zeros((1, dh), np.float32)
            a[0, t] = 1
            A = torch.zeros(1, I, device="cuda")
            dtp.dtp_affinity_accumulate_add(layer, dev(x[None]), dev(a[None]), 1, A)
            r2 = np.mean(x.astype(np.float64) ** 2) + eps
            ref = (gate[:, t].astype(np.float64) ** 2 + up[:, t].astype(np.float64) ** 2) / r2
            worst = max(worst, np.abs(A.cpu().numpy()[0] / ref - 1).max())
    finally:
        dtp.dtp_layer_destroy(layer)
    print(f"[gpu] worst {worst * 2 ** 24:.2f} * 2^-24", flush=True)
    assert worst < 10 * 2.0 ** -24, worst

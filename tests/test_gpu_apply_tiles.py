"""Layouts applied at the edges of the permuting kernels' dispatch: bit-exact data movement."""
import numpy as np
import pytest

from oracle import apply as ap
from oracle import layout as lay
from paper_2609_13846_amd import dtp
from tests.helpers import torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,I,H,G,dh,L", [
    ("bf16", 40, 2050, 6, 2, 12, 2),      # column groups of 72 bytes, rows of 4,100: both by element
    ("bf16", 24, 40000, 4, 4, 16, 4),     # rows of 80,000 bytes: more than the LDS holds
    ("bf16", 264, 32768, 2, 2, 8, 2),     # rows of exactly the 64 KB it holds, one per block
    ("bf16", 1032, 1096, 16, 8, 24, 8),   # four rows per block, units that cross blocks
    ("f32", 36, 5004, 3, 3, 20, 3),       # fp32, three rows per block, an uneven number of rows
    ("f32", 4, 3, 1, 1, 1, 1),            # the smallest rows there are
])
def test_apply_layout_dispatch_edges(dtype, d, I, H, G, dh, L):
    import torch
    rng = np.random.default_rng(I)
    shapes = dict(w_q=(H * dh, d), w_k=(G * dh, d), w_v=(G * dh, d), w_o=(d, H * dh), w_gate=(I, d),
                  w_up=(I, d), w_down=(d, I))
    bits = np.uint16 if dtype == "bf16" else np.uint32
    stored = {k: rng.integers(0, np.iinfo(bits).max, size=v, dtype=bits) for k, v in shapes.items()}
    if dtype == "f32":
        stored = {k: (v >> 9).astype(np.float32) for k, v in stored.items()}
    hs, nus = lay.random_layout(1, G, I, L, 1000)
    print(f"[gpu] apply {dtype} d={d} I={I} H={H} G={G} dh={dh} L={L}", flush=True)
    src = {k: torch_dev(v) for k, v in stored.items()}
    dst = {k: torch.empty_like(v) for k, v in src.items()}
    dtp.dtp_apply_layout(d, I, H, G, dh, dtp.DTP_BF16 if dtype == "bf16" else dtp.DTP_F32, L, hs[0], nus[0],
                         src, dst)
    torch.cuda.synchronize()
    ref = ap.apply_layout(stored, hs[0], nus[0], H, G, dh, L)
    for k in dtp.WEIGHT_ORDER:
        got = dst[k].view(torch.int16).cpu().numpy().view(np.uint16) if dtype == "bf16" else dst[k].cpu().numpy()
        np.testing.assert_array_equal(got, ref[k], err_msg=k)

"""The down edge's weight factor at the edges of its tiles, against the fp64 oracle.

Both operands are bf16 and the sums fp32; gamma' * w^d is rounded to bf16 once more, an
independent relative error of at most 2^-9 per term of a contraction, so an entry of B (a
sum of squares over at least 48 rows) is off by about 2^-8 / sqrt(48 d) and well inside
the 1e-2 that the down edge is held to everywhere.  The allocation-free call reads the
caller's matrices with other kernels in the same order of products and sums: equal bits.
"""
import numpy as np
import pytest

from oracle import down as orc
from paper_2609_13846_amd import dtp, synth
from tests.helpers import assert_affinity_close, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,I,H,G,dh", [
    (8, 8, 1, 1, 16),        # one stage of which a quarter is real, one piece of neurons
    (40, 264, 2, 1, 32),     # two stages, the second ragged; past one tile of 256 neurons
    (72, 256, 3, 1, 128),    # three stages; five chunks of rows: one per block
    (136, 520, 4, 2, 96),    # five stages; three chunks per group, none full at the end
    (1024, 776, 8, 2, 80),   # 480 rows per group in four chunks, the last ragged: two per block
])
def test_down_weights_tile_edges(d, I, H, G, dh):
    import torch
    rng = np.random.default_rng(d + I)
    bits = [synth.store(0.02 * rng.standard_normal(s), "bf16") for s in
            ((H * dh, d), (G * dh, d), (G * dh, d))]
    gamma, w_down = synth.store(1 + 0.1 * rng.standard_normal(d), "bf16"), synth.store(0.02 * rng.standard_normal((d, I)), "bf16")
    print(f"[gpu] down weights d={d} I={I} H={H} G={G} dh={dh}", flush=True)
    args = (d, I, H, G, dh, dtp.DTP_BF16, *[torch_dev(b) for b in bits], torch_dev(gamma), torch_dev(w_down))
    B = torch.full((G, I), float("nan"), dtype=torch.float32, device="cuda")
    B_na = torch.full((G, I), float("nan"), dtype=torch.float32, device="cuda")
    dtp.dtp_down_weights(*args, B)
    dtp.dtp_down_weights_noalloc(*args, B_na)
    torch.cuda.synchronize()
    f = synth.to_f64
    assert_affinity_close(B.cpu().numpy(), orc.down_weight_norms(*[f(b) for b in bits], f(gamma), f(w_down), H, G))
    assert torch.equal(B, B_na)

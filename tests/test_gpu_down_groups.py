"""The down edge's weight factor of thousands of narrow groups.  Each group is padded to a chunk
of 128 rows, and 4,096 of them at d = 65,536 are more threads than one launch holds (2^32 in the
copy of the row fragments): that call reads the caller's matrices, like the allocation-free
one, and gives its bits.  Values are checked against fp64 products of the same rounded operands
on sampled groups, to the 1e-2 that the down edge is held to: fp32 sums of 65,536 products of
mixed signs are off by some 2^-24 sqrt(65,536 * 2,048) of one product's size (2,048 additions in
a row), about 1e-5 of a sum's.
"""
import pytest

from paper_2609_13846_amd import dtp

pytestmark = pytest.mark.gpu


def test_down_weights_of_thousands_of_groups():
    import torch
    d, I, G = 65536, 8, 4096
    print(f"[gpu] down weights d={d} I={I} G={G} dh=1", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(G)
    w_q, w_k, w_v = (torch.randn(G, d, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    gamma = 1 + 0.1 * torch.randn(d, generator=gen, device="cuda", dtype=torch.bfloat16)
    w_down = torch.randn(d, I, generator=gen, device="cuda", dtype=torch.bfloat16)
    B = torch.full((G, I), float("nan"), dtype=torch.float32, device="cuda")
    B_na = torch.full_like(B, float("nan"))
    args = (d, I, G, G, 1, dtp.DTP_BF16, w_q, w_k, w_v, gamma, w_down)
    dtp.dtp_down_weights(*args, B)
    dtp.dtp_down_weights_noalloc(*args, B_na)
    torch.cuda.synchronize()
    assert torch.equal(B, B_na)
    scaled = (gamma.float()[:, None] * w_down.float()).to(torch.bfloat16).double()
    for g in (0, 1, G // 2, G - 1):
        ref = sum((w[g].double() @ scaled) ** 2 for w in (w_q, w_k, w_v))
        torch.testing.assert_close(B[g].double(), ref, rtol=1e-2, atol=1e-2 * float(ref.max()) * 1e-3)

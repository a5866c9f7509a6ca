"""GPU parity of the fp32 affinity kernels (fold, fused kernel) against the fp64 oracle.

Every product and sum is fp32, so an entry is off by at most about n * 2^-24 of its terms'
magnitude, n = d + dh + 64 roundings along one contraction and the epilogue; the damage is
a difference of such terms, so the bar leaves four times that: 4 * 1,200 * 2^-24 = 2.9e-4 at
the largest d here, below 3e-4 for all of them, on entries above 1e-3 of the maximum (and
the same bound absolute at that level on the rest).
"""
import numpy as np
import pytest

from oracle import affinity as orc
from oracle import down as orc_down
from paper_2609_13846_amd import dtp, synth
from tests import helpers as hp

pytestmark = pytest.mark.gpu

REL = 3e-4
TINY = synth.WORKLOADS["tiny"]


@pytest.mark.parametrize("T,shape,score", [
    (1, {}, "fo"),                                                 # one token
    (33, dict(n_neurons=40), "down"),                              # past a 32-row tile, ragged neurons
    (64, dict(n_neurons=130, d_model=16, n_q_heads=3, n_kv_groups=3, head_dim=16), "add"),  # one stage each
    (65, dict(n_neurons=64, n_q_heads=32, n_kv_groups=32), "down"),  # G at its limit, small tiles
    (700, dict(n_neurons=2050, d_model=272, n_q_heads=6, n_kv_groups=2, head_dim=48), "down"),  # large tiles
    (4200, dict(n_neurons=200, n_q_heads=32, n_kv_groups=32), "fo"),  # large tiles, G at its limit
    (9000, dict(n_neurons=300, d_model=48, n_q_heads=2, n_kv_groups=1), "down"),  # several tiles per block
    (100, dict(n_neurons=512, d_model=1024, n_q_heads=4, n_kv_groups=2, head_dim=80), "add"),
])
def test_f32_matches_oracle(T, shape, score):
    import torch
    wl = synth.shaped(TINY, **shape)
    w = synth.host_weights(wl, 0)
    x, a, x_pre = synth.host_tokens(wl, 0, w, T, with_pre=True)
    print(f"[gpu] f32 affinity T={T} {shape} {score}", flush=True)
    kw = dict(**hp.oracle_inputs(w, x, a), n_kv_groups=wl.n_kv_groups, eps=wl.rms_eps)
    if score == "add":
        A = hp.gpu_affinity(wl, w, x, a, score="add")
        kw.pop("w_down")
        hp.assert_affinity_close(A, orc.affinity_add_folded(**kw), rel=REL)
        return
    hp.assert_affinity_close(hp.gpu_affinity(wl, w, x, a), orc.affinity_folded(**kw), rel=REL)
    if score == "down":
        layer = hp.layer_for(wl)
        try:
            # o_proj at an address 4 bytes past a 16-byte boundary: nothing asks for more
            wo = hp.torch_dev(w.w_o)
            off = torch.empty(wo.numel() + 4, dtype=wo.dtype, device="cuda")[1:1 + wo.numel()]
            off.copy_(wo.reshape(-1))
            dtp.dtp_layer_set_weights(layer, off, *[hp.torch_dev(v) for v in (w.gamma, w.w_gate, w.w_up, w.w_down)])
            A = torch.zeros(wl.n_kv_groups, wl.n_neurons, dtype=torch.float32, device="cuda")
            s = torch.zeros(wl.n_neurons, dtype=torch.float32, device="cuda")
            dtp.dtp_affinity_accumulate_down(layer, hp.torch_dev(x), hp.torch_dev(a), hp.torch_dev(x_pre),
                                             wl.rms_eps, T, A, s)
            torch.cuda.synchronize()
        finally:
            dtp.dtp_layer_destroy(layer)
        hp.assert_affinity_close(A.cpu().numpy(), orc.affinity_folded(**kw), rel=REL)
        s_ref = orc_down.down_token_stat(x=kw["x"], gamma=kw["gamma"], w_gate=kw["w_gate"], w_up=kw["w_up"],
                                         eps=wl.rms_eps, x_next=synth.to_f64(x_pre), eps_next=wl.rms_eps)
        np.testing.assert_allclose(s.cpu().numpy(), s_ref, rtol=REL, atol=REL * 1e-3 * s_ref.max())

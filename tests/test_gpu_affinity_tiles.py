"""The bf16 affinity kernel at the edges of its dispatch, against the fp64 oracle: heads of every
number of 32-column stages that has a kernel of its own (1 to 6) and of fours of them, head
counts that end a round of slots early, widths padded to whole stages, launches split over
KV groups, several tiles per block and several slices per call.

Bars: A is held to the 1e-2 of bf16 inputs on entries above 1e-3 of the maximum.  The
token statistic s_down squares g and u, whose W' rounding a cancelling pre-activation
magnifies by its condition number: it is held entry by entry to the rounding model of
tests/error_model.py, as everywhere, and to 1e-2 where that leaves room for it.
"""
import numpy as np
import pytest

from oracle import affinity as orc
from oracle import down as orc_down
from paper_2609_13846_amd import dtp, synth
from tests import error_model as em
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,score,shape", [
    (200, "fo", dict(d_model=16, n_neurons=40, n_q_heads=1, n_kv_groups=1, head_dim=16)),     # one head of one stage
    (193, "down", dict(d_model=144, n_neurons=130, n_q_heads=7, n_kv_groups=7, head_dim=32)),  # seven of one
    (300, "add", dict(d_model=64, n_neurons=128, n_q_heads=5, n_kv_groups=1, head_dim=48)),    # five of two, padded
    (400, "down", dict(d_model=160, n_neurons=200, n_q_heads=3, n_kv_groups=3, head_dim=64)),  # three of two
    (300, "fo", dict(d_model=96, n_neurons=128, n_q_heads=6, n_kv_groups=2, head_dim=80)),     # six of three, padded
    (300, "down", dict(d_model=96, n_neurons=128, n_q_heads=5, n_kv_groups=5, head_dim=96)),   # five of three
    (500, "add", dict(d_model=256, n_neurons=300, n_q_heads=7, n_kv_groups=7, head_dim=96)),   # seven of three
    (256, "add", dict(d_model=128, n_neurons=128, n_q_heads=2, n_kv_groups=2, head_dim=112)),  # four, padded
    (256, "fo", dict(d_model=128, n_neurons=128, n_q_heads=6, n_kv_groups=3, head_dim=160)),   # six of five
    (256, "down", dict(d_model=128, n_neurons=128, n_q_heads=3, n_kv_groups=1, head_dim=192)),  # three of six
    (256, "down", dict(d_model=128, n_neurons=128, n_q_heads=2, n_kv_groups=2, head_dim=208)),  # seven made eight
    (256, "add", dict(d_model=128, n_neurons=128, n_q_heads=1, n_kv_groups=1, head_dim=384)),  # twelve
    (700, "fo", dict(d_model=64, n_neurons=7000, n_q_heads=5, n_kv_groups=5, head_dim=32)),    # not split over groups
    (30000, "down", dict(d_model=48, n_neurons=1500, n_q_heads=3, n_kv_groups=3, head_dim=32)),  # tiles per block
    (75000, "down", dict(d_model=32, n_neurons=300, n_q_heads=2, n_kv_groups=1, head_dim=16)),  # three slices
    (75000, "add", dict(d_model=32, n_neurons=300, n_q_heads=3, n_kv_groups=3, head_dim=64)),
] + [  # tiles of 128 and of 192 tokens in heads of each number of stages, as the sizes of a launch choose them
    # (rounding W' and F to bf16 alone, in fp64, takes entries off by up to 1.1e-2 with d = 32, 7e-3 with 128)
    (T, score, dict(d_model=256, n_neurons=I, n_q_heads=3, n_kv_groups=3, head_dim=dh))
    for T, I in ((1000, 4096), (18400, 1024))
    for dh, score in ((32, "fo"), (64, "down"), (96, "add"), (96, "down"), (128, "fo"), (160, "down"), (192, "add"),
                      (256, "down"))
] + [  # nine heads of one, three and five stages, which close two rounds of four slots and begin a third
    (T, score, dict(d_model=256, n_neurons=I, n_q_heads=9, n_kv_groups=3, head_dim=dh))
    for T, I in ((1000, 4096), (18400, 1024))
    for dh, score in ((32, "down"), (96, "fo"), (160, "down"), (160, "add"))
] + [  # whole rounds of heads of three, five and six stages, in tiles of 192 tokens
    (18400, score, dict(d_model=256, n_neurons=1024, n_q_heads=12, n_kv_groups=3, head_dim=dh))
    for dh, score in ((96, "down"), (96, "add"), (160, "fo"), (192, "down"), (192, "add"))
])
def test_affinity_dispatch_edges(T, score, shape):
    import torch
    wl = synth.shaped(synth.WORKLOADS["qwen3-0.6b-layer"], **shape)
    w = synth.host_weights(wl, 0)
    x, a, x_pre = synth.host_tokens(wl, 0, w, T, with_pre=True)
    print(f"[gpu] affinity T={T} {score} {shape}", flush=True)
    kw = dict(**hp.oracle_inputs(w, x, a), n_kv_groups=wl.n_kv_groups, eps=wl.rms_eps)
    if score == "add":
        kw.pop("w_down")
        hp.assert_affinity_close(hp.gpu_affinity(wl, w, x, a, score="add"), orc.affinity_add_folded(**kw))
        return
    ref = orc.affinity_folded(**kw)
    hp.assert_affinity_close(hp.gpu_affinity(wl, w, x, a), ref)
    if score == "down":
        layer = hp.layer_for(wl)
        try:
            dtp.dtp_layer_set_weights(layer, *[hp.torch_dev(v) for v in (w.w_o, w.gamma, w.w_gate, w.w_up, w.w_down)])
            A = torch.zeros(wl.n_kv_groups, wl.n_neurons, dtype=torch.float32, device="cuda")
            s = torch.zeros(wl.n_neurons, dtype=torch.float32, device="cuda")
            dtp.dtp_affinity_accumulate_down(layer, hp.torch_dev(x), hp.torch_dev(a), hp.torch_dev(x_pre),
                                             wl.rms_eps, T, A, s)
            torch.cuda.synchronize()
        finally:
            dtp.dtp_layer_destroy(layer)
        hp.assert_affinity_close(A.cpu().numpy(), ref)
        s_ref = orc_down.down_token_stat(x=kw["x"], gamma=kw["gamma"], w_gate=kw["w_gate"], w_up=kw["w_up"],
                                         eps=wl.rms_eps, x_next=synth.to_f64(x_pre), eps_next=wl.rms_eps)
        s_m, s_sig, s_sec = em.down_stat_error(kw["x"], kw["gamma"], kw["w_gate"], kw["w_up"], wl.rms_eps,
                                               synth.to_f64(x_pre), wl.rms_eps)
        np.testing.assert_allclose(s_m, s_ref, rtol=1e-10)
        rep = em.check_entrywise(s.cpu().numpy()[None, :], s_ref[None, :], s_sig[None, :], s_sec[None, :],
                                 label="s_down")
        print(f"[gpu] s_down {rep}", flush=True)

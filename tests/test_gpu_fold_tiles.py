"""Loading a bf16 layer in fold tiles of each height (64, 128 and 256 columns, as the sizes choose
them), with columns that do not fill the last one, against the fp64 oracle; and with every
weight 2 bytes past a 16-byte boundary, which takes the loads of single elements and has to give
the same bits."""
import pytest

from oracle import affinity as orc
from paper_2609_13846_amd import dtp, synth
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,shape", [
    (200, dict(d_model=16, n_neurons=40, n_q_heads=1, n_kv_groups=1, head_dim=16)),       # 64: one stage of four real
    (200, dict(d_model=272, n_neurons=300, n_q_heads=3, n_kv_groups=3, head_dim=48)),     # 64: 144 columns
    (200, dict(d_model=256, n_neurons=384, n_q_heads=4, n_kv_groups=2, head_dim=64)),     # 64: whole tiles
    (200, dict(d_model=48, n_neurons=1500, n_q_heads=19, n_kv_groups=19, head_dim=80)),   # 128: 1,520 columns
    (200, dict(d_model=144, n_neurons=3000, n_q_heads=19, n_kv_groups=19, head_dim=80)),  # 256: 1,520 columns
])
def test_fold_tiles_and_unaligned_weights(T, shape):
    import torch
    wl = synth.shaped(synth.WORKLOADS["qwen3-0.6b-layer"], **shape)
    w = synth.host_weights(wl, 0)
    x, a = synth.host_tokens(wl, 0, w, T)
    print(f"[gpu] fold T={T} {shape}", flush=True)
    aligned = [hp.torch_dev(v) for v in (w.w_o, w.gamma, w.w_gate, w.w_up, w.w_down)]
    shifted = []
    for v in aligned:
        buf = torch.empty(v.numel() + 8, dtype=v.dtype, device="cuda")[1:1 + v.numel()]
        buf.copy_(v.reshape(-1))
        assert buf.data_ptr() % 16 == 2
        shifted.append(buf)
    dx, da = hp.torch_dev(x), hp.torch_dev(a)
    out = []
    for weights in (aligned, shifted):
        layer = hp.layer_for(wl)
        try:
            dtp.dtp_layer_set_weights(layer, *weights)
            A = torch.zeros(wl.n_kv_groups, wl.n_neurons, dtype=torch.float32, device="cuda")
            dtp.dtp_affinity_accumulate(layer, dx, da, T, A)
            torch.cuda.synchronize()
            out.append(A)
        finally:
            dtp.dtp_layer_destroy(layer)
    hp.assert_affinity_close(out[0].cpu().numpy(),
                             orc.affinity_folded(**hp.oracle_inputs(w, x, a), n_kv_groups=wl.n_kv_groups, eps=wl.rms_eps))
    assert torch.equal(out[0], out[1])

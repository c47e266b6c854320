"""The fp32 kernels of small layers: products that norm their rows themselves, and q|k|v with rotation and scatter in the same
kernel, at the edges of their tiles and of their range."""
import numpy as np
import pytest
import torch

import vlc_synth as syn
import paper_2512_12977_amd as vlc
from paper_2512_12977_amd import runner as R
from test_gpu_layer import check_against_oracle
from test_gpu_moe import stack_both_ways

pytestmark = pytest.mark.gpu
DEV = "cuda"


# columns of one and of several 64-wide groups of k-steps, the last width whose rows stay in registers and one beyond
@pytest.mark.parametrize("H,Hq,Hkv,D,bias,norm", [(64, 2, 1, 64, True, False), (192, 3, 3, 64, False, True), (320, 4, 2, 128, True, False),
                                                   (512, 4, 1, 128, False, True), (512, 6, 2, 64, True, False), (576, 4, 2, 64, True, True)])
@pytest.mark.parametrize("n_text", [1, 16, 33])
def test_small_layers_around_the_tiles(H, Hq, Hkv, D, bias, norm, n_text):
    """Two layers against the oracle at the element-wise fp32 tolerance; the chained calls, which find the normed rows in the
    workspace and run the products without their norm, give the same bits."""
    sh = syn.Shape("small", L=2, H=H, Hq=Hq, Hkv=Hkv, D=D, I=128, rope_base=1e4, dtype="f32", qkv_bias=bias, qk_norm=norm)
    req = syn.Request([syn.Segment(0, n_text, False), syn.Segment(n_text, 40, True, 5, 0), syn.Segment(n_text + 40, 3, False)], 0)
    wl = syn.Workload("small", sh, [req], 40, "static", static_k=50, seed=H + n_text)
    check_against_oracle(wl, layers=2, teacher_forced=False, shift_ahead=True)
    check_against_oracle(wl, layers=2, teacher_forced=False, shift_ahead=True, chain=True)

    rec, plans = R.make_shape(sh), R.DevicePlans([req], 2, k=np.full(2, 50, dtype=np.int32))
    W = [R.DeviceWeights(syn.layer_weights(sh, 1, l), torch.float32) for l in range(2)]
    n, S = plans.n_rows[0], plans.total_slots
    h_in, ws = torch.randn((S, H), device=DEV), R.Workspace(rec, n)
    records, outs = [plans.record(0, S, S), plans.record(1, n, S)], []
    for chain in (False, True):
        kc, vc = [torch.zeros((S, Hkv, D), device=DEV) for _ in range(2)], [torch.zeros((S, Hkv, D), device=DEV) for _ in range(2)]
        h1, h2 = torch.empty((n, H), device=DEV), torch.empty((n, H), device=DEV)
        vlc.vlc_layer_forward_chained(rec, W[0].rec, records[0], h_in, h1, kc[0], vc[0], ws.t, False, W[1].t["w_ln1"] if chain else None)
        vlc.vlc_layer_forward_chained(rec, W[1].rec, records[1], h1, h2, kc[1], vc[1], ws.t, chain)
        outs.append([h1, h2] + kc + vc)
    for a, b in zip(*outs):
        assert torch.equal(a, b)


# (query heads = kv heads, MLP width, experts, rows, stages inside another's kernel): 96 tiles of 128 rows x 128 columns (SwiGLU: 64)
# are the line from which a product runs on large tiles and its norm apart.  q|k|v is 24 or 33 tiles wide, gate|up 32 or 1, the router 1.
@pytest.mark.parametrize("heads,I,experts,rows,inside", [
    (16, 2048, 0, 256, ("q|k|v", "gate|up")), (16, 2048, 0, 257, ("q|k|v",)), (16, 2048, 0, 384, ("q|k|v",)), (16, 2048, 0, 385, ()),
    (22, 64, 0, 256, ("q|k|v", "gate|up")), (22, 64, 0, 257, ("gate|up",)),
    (16, 64, 8, 384, ("q|k|v", "router")), (16, 64, 8, 385, ("router",))])
def test_small_layers_around_the_large_tiles(heads, I, experts, rows, inside):
    """Layers that norm in both, in one and in none of their products: two layers against the oracle, chained calls the same bits."""
    more = dict(n_experts=experts, top_k=2, residual_proj_scale=0.01) if experts else {}
    sh = syn.Shape("lines", L=2, H=64, Hq=heads, Hkv=heads, D=64, I=I, rope_base=1e4, dtype="f32", qkv_bias=not experts, qk_norm=True,
                   text_scale=1.0, **more)
    empty = vlc.vlc_layer_empty_stages(R.make_shape(sh), rows)
    assert empty == (0b1010 if "q|k|v" in inside else 0) | (0b1000000 if inside and inside[-1] != "q|k|v" else 0)
    wl = syn.Workload("lines", sh, [syn.Request([syn.Segment(0, rows, False)], 0)], 1, "static", static_k=0, seed=heads + rows)
    check_against_oracle(wl, layers=2, teacher_forced=False, chain=True)
    assert check_against_oracle.chained == 1
    plain, chained, _ = stack_both_ways(wl, 2)
    for l in range(2):
        for a, b in zip(plain[l], chained[l]):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("H,Hq,Hkv,bias,norm,rows,inside", [
    (64, 2, 1, True, False, 8, True), (128, 4, 4, False, True, 23, True), (256, 4, 2, True, False, 32, False), (256, 4, 2, False, True, 33, True),
    (320, 4, 2, True, True, 80, False), (320, 4, 2, True, True, 81, True), (512, 4, 2, True, False, 208, False), (512, 4, 2, False, True, 209, True),
    (512, 8, 8, True, True, 64, False), (512, 8, 8, True, True, 65, True)])
def test_small_layers_of_wide_heads(H, Hq, Hkv, bias, norm, rows, inside):
    """Heads of 128 on both sides of the number of workgroups from which q|k|v takes norm, rotation and scatter along, and widths that always do."""
    sh = syn.Shape("wide", L=1, H=H, Hq=Hq, Hkv=Hkv, D=128, I=128, rope_base=1e4, dtype="f32", qkv_bias=bias, qk_norm=norm)
    assert bool(vlc.vlc_layer_empty_stages(R.make_shape(sh), rows) & 0b1010) == inside
    test_small_layers_around_the_tiles(H, Hq, Hkv, 128, bias, norm, rows - 7)      # 4 of the image's and 3 of the last text's rows


"""bf16 products whose workgroups stay for several tiles and ask for the next one's first k-tiles before they store the last
one's outputs: k ranges shorter than the ring of stages and longer, ragged rows and columns, last rounds split along k, and
experts whose row tiles are only known on the device."""
import ctypes

import numpy as np
import pytest

import vlc_synth as syn
import paper_2512_12977_amd as vlc
from test_gpu_gemm_tiles import RESIDUAL, SWIGLU, choice, stays, test_layer_products_on_every_tile as check_layer
from test_gpu_moe import check_moe_layer

# (product that stays, whether its last round is split, layer: H, I, Hq, Hkv, rows)
CASES = [("gate_up", False, (64, 4096, 1, 1, 5000)), ("gate_up", False, (128, 4160, 1, 1, 8191)), ("gate_up", False, (192, 4096, 1, 1, 16390)),
         ("gate_up", True, (2048, 2048, 1, 1, 16390)), ("gate_up", True, (2048, 6464, 1, 1, 4097)), ("o", False, (2880, 64, 6, 1, 16539)),
         ("o", True, (2368, 192, 30, 5, 16621)), ("down", True, (2880, 7040, 4, 4, 16932)), ("down", False, (5696, 11328, 4, 2, 10866))]


@pytest.mark.gpu
@pytest.mark.parametrize("product,split,layer", CASES)
def test_products_of_many_rounds(product, split, layer):
    """The workgroups stay (asked of the library), at the tolerances of the tests of the tiles."""
    H, I, Hq, Hkv, rows = layer
    of = {"gate_up": (SWIGLU, rows, I, H), "o": (RESIDUAL, rows, H, Hq * 128), "down": (RESIDUAL, rows, H, I)}[product]
    assert stays(*of), choice(*of)
    assert (choice(*of)[2] == "split last round") == split, choice(*of)
    check_layer(H, I, Hq, Hkv, rows)


# (rows, H, I, product whose tiles are counted): 2 of 8 experts, on row tiles of 256
EXPERTS = [(2600, 3328, 64, "down"), (2600, 3264, 192, "down"), (1800, 128, 2432, "gate_up"), (900, 192, 4160, "gate_up")]


def group_tile_rows(pairs, experts, width):
    """Rows per tile of the experts' products, as the launcher chooses them."""
    f = vlc.lib().vlc_probe_group_tile_rows
    f.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int64, ctypes.c_int]
    return f(pairs, experts, width, vlc.VLC_BF16)


@pytest.mark.parametrize("rows,H,I,product", EXPERTS)
def test_expert_cases_have_more_tiles_than_workgroups(rows, H, I, product):
    """However the router loads the experts: full row tiles are the fewest that the pairs can take."""
    tile_rows = group_tile_rows(2 * rows, 8, I)
    assert tile_rows == 256
    assert -(-2 * rows // tile_rows) * -(-(2 * I if product == "gate_up" else H) // 256) > 256


@pytest.mark.gpu
@pytest.mark.parametrize("rows,H,I,product", EXPERTS)
def test_experts_of_many_tiles(rows, H, I, product):
    """More tiles than the 256 workgroups that stay, however the router loads the experts, in the down projection (one and three
    k-tiles), then in gate|up, whose rows are fetched through the pair list (two and three k-tiles); tiles of 256 rows."""
    sh = syn.Shape("moe_stay", L=1, H=H, Hq=4, Hkv=2, D=128, I=I, rope_base=1e4, dtype="bf16", qkv_bias=False, qk_norm=True,
                   mrope_section=(24, 20, 20), n_experts=8, top_k=2, text_scale=1.0, residual_proj_scale=0.01)
    req = syn.Request([syn.Segment(0, rows, False)], 0, 0, syn.grid_positions([("text", rows)]))
    g = check_moe_layer(syn.Workload("moe_stay%d_%d" % (rows, I), sh, [req], 1, "static", static_k=0, seed=1200 + I), 0)
    row_tiles = sum(-(-int(pairs) // group_tile_rows(2 * rows, 8, I)) for pairs in np.diff(g["moe_offset"]))
    assert row_tiles * -(-(2 * I if product == "gate_up" else H) // 256) > 256, row_tiles


@pytest.mark.gpu
@pytest.mark.parametrize("rows,H,I", [(600, 192, 4352), (520, 128, 5632)])
def test_experts_of_many_tiles_of_192_rows(rows, H, I):
    """The same on tiles of 192 rows (150 and 130 rows per expert on average): gate|up of at least eight row tiles, three and two k-tiles."""
    assert group_tile_rows(2 * rows, 8, I) == 192 and 8 * -(-2 * I // 256) > 256
    sh = syn.Shape("moe_192", L=1, H=H, Hq=4, Hkv=2, D=128, I=I, rope_base=1e4, dtype="bf16", qkv_bias=False, qk_norm=True,
                   mrope_section=(24, 20, 20), n_experts=8, top_k=2, text_scale=1.0, residual_proj_scale=0.01)
    req = syn.Request([syn.Segment(0, rows, False)], 0, 0, syn.grid_positions([("text", rows)]))
    g = check_moe_layer(syn.Workload("moe_192_%d" % rows, sh, [req], 1, "static", static_k=0, seed=1300 + I), 0)
    assert np.all(np.diff(g["moe_offset"]) > 0)             # every expert has a row tile


@pytest.mark.parametrize("experts,width", [(8, 192), (16, 960), (16, 1024), (16, 1472), (16, 1536), (128, 768)])
def test_rows_per_tile_by_rows_and_columns(experts, width):
    """The lines on both sides; with less than 192 (128) column tiles over all experts, those of 128 (185) rows do not apply."""
    columns = experts * -(-2 * width // 256)
    lines = [(9, 32), (56, 64), (128 if columns >= 192 else 140, 128), (185, 192), (250, 256 if columns >= 128 else 192), (360, 192), (10000, 256)]
    first = 0
    for end, want in lines:
        for mean in (first, end - 1):
            assert group_tile_rows(mean * experts + experts - 1, experts, width) == want, mean
        first = end

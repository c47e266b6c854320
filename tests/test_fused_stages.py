"""Which stages of small fp32 layers have no kernel of their own, and that what goes by it - the norms that run_layers hands on,
the stage table of the benchmark - asks the library (host only)."""
import types

import pytest

import bench
import vlc_synth as syn
import paper_2512_12977_amd as vlc
from paper_2512_12977_amd import runner as R

STAGE = {name: i for i, name in enumerate(vlc.LAYER_STAGES)}
# 96 tiles of 128 rows x 128 columns (SwiGLU: 64) is where the products begin to run on large tiles
SHAPES = {
    "wide gate|up": dict(H=256, Hq=1, Hkv=1, D=64, I=1024),              # q|k|v 192 columns: 2 tiles wide, gate|up 16
    "narrow gate|up": dict(H=512, Hq=6, Hkv=3, D=128, I=64),             # 12 and 1
    "experts": dict(H=256, Hq=6, Hkv=3, D=64, I=64, n_experts=8, top_k=2),   # 6, the router 1
    "too wide": dict(H=576, Hq=4, Hkv=2, D=64, I=128),
}


def shape(name, dtype="f32"):
    return syn.Shape(name, L=2, rope_base=1e4, dtype=dtype, qkv_bias=False, **SHAPES[name])


def expected(name, n):
    """(input norm and rotation inside q|k|v, second norm inside its product)"""
    s = SHAPES[name]
    tiles = lambda columns: -(-n // 128) * columns
    qkv = -(-(s["Hq"] + 2 * s["Hkv"]) * s["D"] // 128)
    second = 1 if "n_experts" in s else -(-s["I"] // 64)
    # with heads of 128 also: enough workgroups of 16 rows and one head
    wide = s["D"] == 64 or -(-n // 16) * (s["Hq"] + 2 * s["Hkv"]) >= (s["H"] - 192) // 3
    return s["H"] <= 512 and tiles(qkv) < 96 and wide, s["H"] <= 512 and tiles(second) < 96


@pytest.mark.parametrize("name", sorted(SHAPES))
@pytest.mark.parametrize("n", [1, 128, 129, 640, 641, 896, 897, 1920, 1921, 6016, 6017, 12160, 12161])
def test_empty_stages(name, n):
    qkv, second = expected(name, n)
    want = (1 << STAGE["rmsnorm1"] | 1 << STAGE["rope_scatter"] if qkv else 0) | (1 << STAGE["rmsnorm2"] if second else 0)
    assert vlc.vlc_layer_empty_stages(R.make_shape(shape(name)), n) == want


def test_empty_stages_of_other_calls():
    rec = R.make_shape(syn.SHAPES["tiny_bf16"])
    assert vlc.vlc_layer_empty_stages(rec, 8) == 0
    assert vlc.vlc_layer_empty_stages(rec, 0) == (1 << len(STAGE)) - 2
    with pytest.raises(vlc.VlcError):
        vlc.vlc_layer_empty_stages(rec, -1)
    rec.D = 96
    with pytest.raises(vlc.VlcError):
        vlc.vlc_layer_empty_stages(rec, 8)


def plans_of(rows):
    return types.SimpleNamespace(L=2, n_rows=[rows, rows])


@pytest.mark.parametrize("name,rows", [("experts", 1920), ("experts", 1921), ("wide gate|up", 6016), ("wide gate|up", 6017), ("too wide", 8)])
def test_norms_are_handed_on_where_the_next_product_does_not_take_them(monkeypatch, name, rows):
    """fp32 layers on large tiles (expert layers among them, whose weighted sum then takes the norm along) keep their link."""
    calls = []
    monkeypatch.setattr(R.B, "vlc_layer_forward_chained", lambda *a: calls.append(a))
    weights = [types.SimpleNamespace(rec=None, t={"w_ln1": "norm %d" % l}) for l in range(2)]
    R.run_layers(R.make_shape(shape(name)), weights, plans_of(rows), [None] * 2, None, [None] * 2, [None] * 2, [None] * 2,
                 types.SimpleNamespace(t=None))
    linked = not expected(name, rows)[0]
    assert [(c[8], c[9]) for c in calls] == [(False, "norm 1" if linked else None), (linked, None)]


def test_the_stage_table_gives_no_rate_for_an_empty_stage():
    rec, plans = R.make_shape(shape("experts")), types.SimpleNamespace(L=3, n_rows=[1921, 1920, 0])
    notes = {name: bench.fused_stage_note(i, rec, plans) for name, i in STAGE.items()}
    assert {name for name, note in notes.items() if note} == {"rmsnorm1", "rope_scatter", "rmsnorm2"}
    assert notes["rmsnorm1"] == "empty in 1 of 2 layers: part of their kernel counted under qkv_gemm"
    assert notes["rmsnorm2"] == "empty in 2 of 2 layers: part of their kernel counted under gate_up_swiglu_gemm"
    assert not any(bench.fused_stage_note(i, R.make_shape(syn.SHAPES["7b"]), plans) for i in range(len(STAGE)))

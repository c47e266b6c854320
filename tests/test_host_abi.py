"""Host side of the C ABI (no GPU): the library loads, exports what the header declares, and its
planner / index builders agree bit-for-bit with the oracle."""
import ctypes
import os
import re

import numpy as np
import pytest

import vlc_synth as syn
from oracle import vlc_oracle as orc
import paper_2512_12977_amd as vlc
from paper_2512_12977_amd.runner import segments_of
from helpers import plan_steps, counts_for

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "vlcache.h")).read()
    names = set(re.findall(r"\b(vlc_[a-z_]+)\s*\(", hdr))
    assert {"vlc_plan_layer_rates", "vlc_gather_rows", "vlc_rope_shift_kv", "vlc_scatter_kv",
            "vlc_sparse_q_attention", "vlc_layer_forward"} <= names
    L = ctypes.CDLL(vlc.lib_path())
    for n in sorted(names):
        assert hasattr(L, n), n
    assert vlc.lib().vlc_version() >= 100


def test_planner_bit_exact_vs_oracle():
    rng = np.random.default_rng(0)
    for trial in range(40):
        L, G = int(rng.integers(1, 40)), int(rng.integers(1, 151))
        if trial % 3 == 0:
            sens = rng.random((L, G + 1))
        elif trial % 3 == 1:
            sens = syn.sensitivity_table(L, G, trial)
        else:   # many exact ties
            sens = np.round(rng.random((L, G + 1)) * 4) / 4
        B = int(rng.integers(0, L * G + 3))
        np.testing.assert_array_equal(vlc.vlc_plan_layer_rates(sens, B), orc.plan_layer_rates(sens, B))
    for L, bp in ((28, 500), (80, 300)):
        sens = syn.sensitivity_table(L, 150, 1)
        B = orc.budget_steps_from_mean_rate(bp, L)
        np.testing.assert_array_equal(vlc.vlc_plan_layer_rates(sens, B), orc.plan_layer_rates(sens, B))


def test_block_planner_bit_exact_vs_oracle():
    rng = np.random.default_rng(3)
    for trial in range(40):
        L, G = int(rng.integers(1, 30)), int(rng.integers(1, 60))
        if trial % 4 == 0:
            sens = rng.random((L, G + 1))
        elif trial % 4 == 1:
            sens = syn.sensitivity_table(L, G, trial)
        elif trial % 4 == 2:   # many exact ties
            sens = np.round(rng.random((L, G + 1)) * 4) / 4
        else:                  # flat first layers, the case the runs are for
            sens = syn.sensitivity_table(L, G, trial)
            sens[:max(1, L // 4)] = 1.0
        B = int(rng.integers(0, L * G + 3))
        np.testing.assert_array_equal(vlc.vlc_plan_layer_rates_blocks(sens, B), orc.plan_layer_rates_blocks(sens, B))
    sens = syn.sensitivity_table(28, 150, 1)
    sens[0] = sens[0, 0]
    np.testing.assert_array_equal(vlc.vlc_plan_layer_rates_blocks(sens, 700), orc.plan_layer_rates_blocks(sens, 700))
    assert vlc.vlc_plan_layer_rates(sens, 700).sum() == 0 and vlc.vlc_plan_layer_rates_blocks(sens, 700).sum() > 600
    with pytest.raises(vlc.VlcError):
        vlc.vlc_plan_layer_rates_blocks(sens, -1)


@pytest.mark.parametrize("name", ["c1", "c2", "c3", "c4", "c5"])
def test_token_indices_bit_exact_vs_oracle(name):
    wl = syn.make_workload(name)
    L = wl.shape.L
    k, explicit = plan_steps(wl)
    segs = segments_of(wl.requests)
    out = vlc.vlc_plan_token_indices(segs, L, k=k, count_override=explicit)
    reuse = vlc.vlc_plan_reuse_rows(segs, L, k=k, count_override=explicit)
    prev = None
    for l in range(L):
        slots, pos, start, klen, src, dst, delta = [], [], [], [], [], [], []
        for req in wl.requests:
            counts = counts_for(req, k, explicit, l)
            s = orc.select_slots(req.segments, counts)
            slots.append(req.kv_start + s)
            pos.append(req.pos_start + s)
            start.append(np.full(len(s), req.kv_start))
            klen.append(s + 1)
            rs, rr, ro = orc.reused_slots(req.segments, counts)
            src.append(rr)
            dst.append(req.kv_start + rs)
            delta.append(req.pos_start + rs - ro)
        slots = np.concatenate(slots)
        n = int(out["n_rows"][l])
        assert n == len(slots)
        np.testing.assert_array_equal(out["slot"][l, :n], slots)
        np.testing.assert_array_equal(out["pos"][l, :n], np.concatenate(pos))
        np.testing.assert_array_equal(out["kv_start"][l, :n], np.concatenate(start))
        np.testing.assert_array_equal(out["kv_len"][l, :n], np.concatenate(klen))
        if l == 0:
            np.testing.assert_array_equal(out["map"][l, :n], slots)
        else:
            np.testing.assert_array_equal(prev[out["map"][l, :n]], slots)
        m = int(reuse["n_reuse"][l])
        np.testing.assert_array_equal(reuse["src_row"][l, :m], np.concatenate(src))
        np.testing.assert_array_equal(reuse["dst_slot"][l, :m], np.concatenate(dst))
        np.testing.assert_array_equal(reuse["delta"][l, :m], np.concatenate(delta))
        prev = slots


@pytest.mark.parametrize("name", ["c1", "c3", "c4", "c5"])
def test_next_rows_vs_oracle_selection(name):
    """vlc_plan_next_rows: the index of every row of a layer among the rows of the layer below, from the ORACLE's
    selection of both layers (position of a slot in the next layer's sorted slot list, -1 if it is not there)."""
    wl = syn.make_workload(name)
    L = wl.shape.L
    k, explicit = plan_steps(wl)
    segs = segments_of(wl.requests)
    nxt = vlc.vlc_plan_next_rows(segs, L, k=k, count_override=explicit)
    out = vlc.vlc_plan_token_indices(segs, L, k=k, count_override=explicit)

    def slots_of(l):
        return np.concatenate([req.kv_start + orc.select_slots(req.segments, counts_for(req, k, explicit, l))
                               for req in wl.requests])
    dropped = 0
    for l in range(L):
        cur = slots_of(l)
        n = len(cur)
        if l + 1 == L:
            assert (nxt[l, :n] == -1).all()
            continue
        below = slots_of(l + 1)
        at = np.searchsorted(below, cur)
        hit = (at < len(below)) & (below[np.minimum(at, len(below) - 1)] == cur)
        want = np.where(hit, at, -1)
        np.testing.assert_array_equal(nxt[l, :n], want)
        m = int(out["n_rows"][l + 1])
        np.testing.assert_array_equal(nxt[l, out["map"][l + 1, :m]], np.arange(m))     # inverse of the map
        dropped += int((want < 0).sum())
    if name in ("c3", "c5"):
        assert dropped > 0          # layer-aware rates: rows do fall away with depth


def test_budget_steps_vs_oracle():
    for bp, L in ((500, 28), (300, 80), (0, 5), (10000, 3), (37, 7), (1, 19), (9999, 80)):
        assert vlc.vlc_plan_budget_steps(bp, L) == orc.budget_steps_from_mean_rate(bp, L)
    assert vlc.vlc_plan_budget_steps(500, 28) == 700 and vlc.vlc_plan_budget_steps(300, 80) == 1200
    for bad in ((-1, 5), (10001, 5), (100, 0)):
        with pytest.raises(vlc.VlcError):
            vlc.vlc_plan_budget_steps(*bad)


def test_first_token_noalloc_argument_checks():
    """The variant for callers that cannot allocate refuses what does not fit its built-in scratch before any
    GPU work (no GPU needed): sizes beyond the array, bad dtype / shape; zero requests are a no-op."""
    L = vlc.lib()
    f = L.vlc_first_token_noalloc
    cap = L.vlc_first_token_noalloc_max_bytes()
    assert cap == 1 << 20
    assert f(None, None, 0, 3584, 152064, 1e-6, None, None, None, None, vlc.VLC_BF16, None) == 0
    assert f(None, None, 2, 3584, 152064, 1e-6, None, None, None, None, 9, None) == 3
    assert f(None, None, -1, 3584, 152064, 1e-6, None, None, None, None, vlc.VLC_BF16, None) == 2
    assert L.vlc_first_token_workspace_bytes(3584, 128, vlc.VLC_BF16) <= cap < L.vlc_first_token_workspace_bytes(3584, 129, vlc.VLC_BF16)
    assert f(None, None, 129, 3584, 152064, 1e-6, None, None, None, None, vlc.VLC_BF16, None) == 5
    assert "scratch" in vlc.last_error()
    assert f(None, None, 61, 8192, 152064, 1e-6, None, None, None, None, vlc.VLC_BF16, None) == 5


@pytest.mark.parametrize("name", ["c1_q3", "c2_q3", "c3_q3"])
def test_reuse_deltas_with_grid_position_ids(name):
    """3-axis ids: the runner hands the planner each run's first temporal id, so a reused image's shift is
    (new temporal id - cached temporal id) for all of its tokens, of either sign; slots and cache rows as before."""
    wl = syn.make_workload(name)
    L = min(wl.shape.L, 4)
    k, explicit = plan_steps(wl)
    k = None if k is None else k[:L]
    explicit = None if explicit is None else explicit[:L]
    segs = segments_of(wl.requests)
    out = vlc.vlc_plan_token_indices(segs, L, k=k, count_override=explicit)
    reuse = vlc.vlc_plan_reuse_rows(segs, L, k=k, count_override=explicit)
    req = wl.requests[0]
    signs = set()
    for l in range(L):
        counts = counts_for(req, k, explicit, l)
        s = orc.select_slots(req.segments, counts)
        n = int(out["n_rows"][l])
        np.testing.assert_array_equal(out["slot"][l, :n], s)
        np.testing.assert_array_equal(out["kv_len"][l, :n], s + 1)
        rs, rr, _ = orc.reused_slots(req.segments, counts)
        want = np.concatenate([np.full(g.length - c, int(req.pos3[g.start, 0]) - g.old_pos)
                               for g, c in zip([g for g in req.segments if g.is_image], counts)])
        m = int(reuse["n_reuse"][l])
        np.testing.assert_array_equal(reuse["src_row"][l, :m], rr)
        np.testing.assert_array_equal(reuse["dst_slot"][l, :m], rs)
        np.testing.assert_array_equal(reuse["delta"][l, :m], want)
        signs |= set(np.sign(want).tolist())
    if name == "c3_q3":
        assert signs == {-1, 1}


def test_workload_row_counts():
    """Row counts the benchmark configurations state."""
    def rows(name):
        wl = syn.make_workload(name)
        k, explicit = plan_steps(wl)
        out = vlc.vlc_plan_token_indices(segments_of(wl.requests), wl.shape.L, k=k, count_override=explicit)
        return out["n_rows"]
    assert list(rows("c1")) == [61, 61]
    assert set(rows("c2")) == {596}
    assert set(rows("c4")) == {8 * 2368} and set(rows("c4_5")) == {8 * 2864}


def test_host_error_paths():
    sens = np.ones((3, 5))
    with pytest.raises(vlc.VlcError) as e:
        vlc.vlc_plan_layer_rates(sens, -1)
    assert e.value.code == 2
    segs = [vlc.Segment(0, 10, 0, 0, 0, 0, 0), vlc.Segment(10, 50, 1, 10, 0, 0, 0)]
    with pytest.raises(vlc.VlcError) as e:      # rate grows with depth
        vlc.vlc_plan_token_indices(segs, 2, k=[10, 20])
    assert e.value.code == 7
    with pytest.raises(vlc.VlcError) as e:      # overlapping runs
        vlc.vlc_plan_token_indices([segs[0], vlc.Segment(5, 5, 0, 5, 0, 0, 0)], 1, k=[0])
    assert e.value.code == 4
    with pytest.raises(vlc.VlcError) as e:      # capacity
        vlc.vlc_plan_token_indices(segs, 1, k=[500], cap=20)
    assert e.value.code == 2
    with pytest.raises(vlc.VlcError) as e:      # k outside the grid
        vlc.vlc_plan_token_indices(segs, 1, k=[501])
    assert e.value.code == 2
    # no rows at all is fine
    out = vlc.vlc_plan_token_indices([vlc.Segment(0, 50, 1, 0, 0, 0, 0)], 2, k=[0, 0])
    assert list(out["n_rows"]) == [0, 0]
    # shape errors of the layer entry points are reported without touching a GPU
    bad = vlc.LayerShape(256, 4, 3, 64, 512, 0, 1e-6, 1e4)
    with pytest.raises(vlc.VlcError):
        vlc.vlc_layer_workspace_bytes(bad, 10)
    assert "Hq" in vlc.last_error()
    ok = vlc.LayerShape(256, 4, 2, 64, 512, 0, 1e-6, 1e4, 12, 10, 10)
    assert vlc.vlc_layer_workspace_bytes(ok, 10) > 0
    for sec in ((12, 10, 9), (33, 0, 0), (-1, 17, 16)):       # the three axes must share the D/2 = 32 frequencies
        with pytest.raises(vlc.VlcError):
            vlc.vlc_layer_workspace_bytes(vlc.LayerShape(256, 4, 2, 64, 512, 0, 1e-6, 1e4, *sec), 10)
        assert "3-axis" in vlc.last_error()
    # first-token head: argument checks come before any GPU work
    L = vlc.lib()
    assert L.vlc_first_token_workspace_bytes(256, 3, vlc.VLC_F32) >= 3 * 256 * 4
    assert L.vlc_first_token_workspace_bytes(3584, 8, vlc.VLC_BF16) >= 8 * 3584 * 2
    assert L.vlc_first_token_workspace_bytes(3584, 8, vlc.VLC_BF16) % 256 == 0
    assert L.vlc_first_token_workspace_bytes(0, 3, vlc.VLC_F32) == 0
    assert L.vlc_first_token(None, None, 0, 256, 512, 1e-6, None, None, None, None, None, 0, vlc.VLC_F32, None) == 0
    assert L.vlc_first_token(None, None, 2, 256, 512, 1e-6, None, None, None, None, None, 0, vlc.VLC_F32, None) == 1
    assert L.vlc_first_token(None, None, 2, 100, 512, 1e-6, None, None, None, None, None, 0, vlc.VLC_F32, None) == 2
    assert L.vlc_first_token(None, None, 2, 256, 510, 1e-6, None, None, None, None, None, 0, vlc.VLC_F32, None) == 2
    assert L.vlc_first_token(None, None, 2, 256, 512, 1e-6, None, None, None, None, None, 0, 9, None) == 3


def test_workspace_size_is_monotone_in_rows():
    """A workspace sized for n_max rows must serve every call with fewer rows (the scratch areas for
    split-K GEMMs and key-split attention only exist for small row counts)."""
    from paper_2512_12977_amd.runner import make_shape
    for name in ("7b", "72b", "tiny_bf16", "tiny", "q3vl_8b", "tiny_q3", "q3vl_30b_a3b", "tiny_moe"):
        rec = make_shape(syn.SHAPES[name])
        prev = 0
        for n in list(range(0, 3000, 13)) + [5000, 18944, 147456]:
            b = vlc.vlc_layer_workspace_bytes(rec, n)
            assert b >= prev, (name, n, b, prev)
            prev = b


def test_expert_fields_of_the_shape_and_layout():
    from paper_2512_12977_amd.runner import make_shape
    dense = make_shape(syn.SHAPES["7b"])
    off = vlc.vlc_layer_workspace_layout(dense, 100)
    assert all(off[name] == -1 for name in ("moe_idx", "moe_w", "moe_pos", "moe_y", "moe_logits", "moe_offset"))
    moe = make_shape(syn.SHAPES["q3vl_30b_a3b"])
    off = vlc.vlc_layer_workspace_layout(moe, 100)
    vals = [off[name] for name in ("act", "moe_idx", "moe_w", "moe_pos", "moe_y", "moe_logits", "moe_offset")]
    assert all(v >= 0 and v % 256 == 0 for v in vals) and vals == sorted(vals) and len(set(vals)) == len(vals)
    assert off["moe_idx"] - off["act"] >= 100 * 8 * 768 * 2          # the SwiGLU product holds one row per (row, expert) pair
    assert vlc.vlc_layer_workspace_bytes(moe, 100) > vlc.vlc_layer_workspace_bytes(make_shape(syn.SHAPES["q3vl_8b"]), 100) - (1 << 26)
    for n_experts, top_k in ((257, 8), (8, 9), (8, 0), (8, 17), (-1, 0), (6, 2)):   # (6, 2): bf16 wants a multiple of 4
        bad = vlc.LayerShape(2048, 32, 4, 128, 768, vlc.VLC_BF16, 1e-6, 5e6, 24, 20, 20, n_experts, top_k)
        with pytest.raises(vlc.VlcError):
            vlc.vlc_layer_workspace_bytes(bad, 10)
        assert "n_experts" in vlc.last_error()


def test_mean_squared_error_argument_checks():
    L = vlc.lib()
    assert L.vlc_mean_squared_error_workspace_bytes() >= 8
    assert L.vlc_mean_squared_error(None, None, 0, None, None, 0, None) == 2      # n <= 0
    assert L.vlc_mean_squared_error(None, None, 5, None, None, 0, None) == 1      # NULL pointers


def test_rope_shift_kv_layers_argument_checks():
    """Everything the host can check is refused before any launch (no GPU needed)."""
    L = vlc.lib()
    assert ctypes.sizeof(vlc.ShiftJob) == 64                                     # 7 pointers + int64
    f = L.vlc_rope_shift_kv_layers
    assert f(None, 0, 0, 4, 128, 1e6, vlc.VLC_BF16, None) == 0                   # nothing to do
    assert f(None, 3, 0, 4, 128, 1e6, vlc.VLC_BF16, None) == 0                   # no tokens: jobs not read
    assert f(None, 3, 10, 4, 128, 1e6, vlc.VLC_BF16, None) == 1                  # NULL table
    assert f(None, -1, 10, 4, 128, 1e6, vlc.VLC_BF16, None) == 2
    assert f(None, 70000, 10, 4, 128, 1e6, vlc.VLC_BF16, None) == 2              # more jobs than grid rows
    assert f(None, 3, -1, 4, 128, 1e6, vlc.VLC_BF16, None) == 2
    assert f(None, 3, 10, 4, 96, 1e6, vlc.VLC_BF16, None) == 2                   # head size
    assert f(None, 3, 10, 4, 128, 0.0, vlc.VLC_BF16, None) == 2                  # rope base
    assert f(None, 3, 10, 4, 128, 1e6, 7, None) == 3                             # dtype
    assert f(ctypes.c_void_p(0x1004), 3, 10, 4, 128, 1e6, vlc.VLC_BF16, None) == 2   # misaligned table
    assert "aligned" in vlc.last_error()


def test_layer_forward_chained_argument_checks():
    """The chained layer call refuses a flag other than 0/1 and, like vlc_layer_forward, a NULL shape, weights or
    plan before anything is launched (no GPU needed)."""
    f = vlc.lib().vlc_layer_forward_chained
    sh = vlc.LayerShape(256, 4, 2, 128, 512, vlc.VLC_BF16, 1e-6, 1e4, 0, 0, 0, 0, 0)
    a = ctypes.addressof(sh)
    assert f(a, None, None, None, None, None, None, None, 0, None, 2, None, None, None) == 2
    assert "input_norm_ready" in vlc.last_error()
    assert f(None, None, None, None, None, None, None, None, 0, None, 0, None, None, None) == 1
    assert f(a, None, None, None, None, None, None, None, 0, None, 1, None, None, None) == 1      # weights / plan


@pytest.mark.parametrize("Hq,Hkv", [(28, 4), (32, 8), (64, 8), (32, 4), (4, 2)])
def test_attention_key_shares(Hq, Hkv):
    """The most shares that a row tile may take, by the number of (row tile, kv head) pairs: 1024 / pairs (twice its part of
    the 512 workgroups of the launch), 8 at most, none from 512 pairs on, and no share shorter than four key blocks of 64."""
    f = vlc.lib().vlc_probe_attention_shares
    f.argtypes, f.restype = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int64], ctypes.c_int
    rows = 128 // (Hq // Hkv)
    for pairs in list(range(Hkv, 640, Hkv)):
        n = pairs // Hkv * rows - rows // 2
        want = 1 if pairs >= 512 else min(8, 1024 // pairs)
        assert f(n, Hq, Hkv, 64 * 840) == want, (pairs, n)          # 840: a multiple of 1 ... 8
        for keys in (1, 64, 256, 257, 512, 1000, 2048):
            assert f(n, Hq, Hkv, keys) <= max(1, -(-(-(-keys // 64)) // 4)), (pairs, keys)


@pytest.mark.parametrize("raw", [True, False])
def test_current_stream_with_and_without_the_raw_handle(monkeypatch, raw):
    """The current stream's handle, from torch's function for the bare handle where this torch has it, else from the Stream object."""
    import torch
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: type("Stream", (), {"cuda_stream": 77})())
    if raw:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 70 + device, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert vlc.binding._stream(None) == (73 if raw else 77)
    assert vlc.binding._stream(12) == 12


def test_header_is_plain_c_and_the_library_links_from_c(tmp_path):
    """include/vlcache.h compiles as C99 (-pedantic, warnings as errors) and a C program linked against the library
    gets the planner's result (host entry points only: no GPU needed)."""
    import shutil
    import subprocess
    if shutil.which("gcc") is None:
        pytest.skip("no gcc")
    src = tmp_path / "abi.c"
    src.write_text('#include "vlcache.h"\n#include <stdio.h>\n'
                   "int main(void) {\n"
                   "  double sens[8] = {4, 3, 2, 1, 8, 4, 2, 1};\n"
                   "  int32_t k[2];\n"
                   "  int rc = vlc_plan_layer_rates(2, 3, sens, 3, k);\n"
                   '  printf("%d %d %d %d\\n", vlc_version(), rc, (int)k[0], (int)k[1]);\n'
                   "  return rc;\n}\n")
    exe = tmp_path / "abi"
    libdir = os.path.dirname(vlc.lib_path())
    subprocess.run(["gcc", "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror", "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe), "-L", libdir, "-l:libvlcache.so", "-Wl,-rpath," + libdir], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    want = orc.plan_layer_rates(np.array([[4, 3, 2, 1], [8, 4, 2, 1]], dtype=np.float64), 3)
    assert [int(v) for v in out] == [vlc.lib().vlc_version(), 0, int(want[0]), int(want[1])]

"""The bf16 products of a layer on every tile configuration that the dispatcher launches: whole, with a split k range, and with
a last round whose tiles are split along k.  The layers below are small stand-ins (a few columns, many rows, or the other
way round) whose products land on each of them, with workgroups that stay for several tiles where a decoder's do; what a product lands
on is asked of the library, so that a change of the prices cannot move the cases away from the kernels unnoticed."""
import ctypes
import dataclasses

import numpy as np
import pytest
import torch

import paper_2512_12977_amd as vlc
import vlc_synth as syn
from paper_2512_12977_amd import runner as R

DEV = "cuda"
RESIDUAL, SWIGLU, FLOAT = 1, 2, 3

# (hidden size, MLP width, query heads, kv heads, rows); rows and columns are ragged against most of the tiles
LAYERS = [
    (320, 128, 4, 1, 4), (704, 448, 5, 1, 2712), (2176, 448, 1, 1, 5552), (320, 1472, 4, 4, 3238), (2368, 448, 1, 1, 2448),
    (704, 3264, 16, 8, 3275), (448, 1664, 8, 4, 4107), (3136, 1088, 1, 1, 3661), (2240, 128, 1, 1, 2835),
    (448, 3776, 7, 1, 6194), (3008, 128, 2, 2, 1942), (7040, 192, 2, 1, 3255), (896, 256, 5, 1, 9865),
    (896, 512, 7, 1, 8465), (256, 2752, 1, 1, 2113), (704, 3328, 1, 1, 1933), (320, 4544, 7, 1, 11073),
    (3712, 1856, 1, 1, 13119), (448, 8064, 5, 1, 12299), (448, 9984, 1, 1, 6799), (5760, 448, 7, 1, 2134),
    (704, 7808, 1, 1, 6835), (1088, 5824, 1, 1, 8206), (2560, 2368, 2, 1, 6845), (5760, 832, 7, 1, 2712),
    (4992, 704, 1, 1, 13693), (832, 4992, 1, 1, 16465), (8000, 576, 10, 2, 639), (640, 9216, 1, 1, 13715),
    (3072, 2752, 5, 1, 6697), (3520, 3200, 1, 1, 10415), (5056, 192, 5, 1, 16867), (8192, 128, 4, 4, 6724),
    (1152, 128, 28, 4, 14412), (2816, 128, 16, 2, 14722), (128, 128, 56, 8, 578)]
# the tiles with 16-wide steps in rows or columns (128 x 96, 160 x 160, 160 x 192, 224 x 192, 256 x 192, 320 x 160, 320 x 256) and the choices
# that came with them; sums of up to 25216 products here, rounded to bf16 like the others
LAYERS += [
    (6272, 128, 32, 4, 68), (64, 4544, 32, 4, 874), (5440, 192, 28, 4, 130), (6208, 64, 28, 4, 200),
    (64, 3328, 28, 4, 1654), (8448, 64, 16, 4, 686), (9536, 24576, 10, 2, 6), (1984, 24832, 4, 4, 293),
    (7104, 64, 1, 1, 1017), (2944, 17024, 16, 4, 328), (3712, 25216, 16, 4, 194), (2304, 6720, 6, 2, 9797),
    (4096, 8192, 5, 1, 779), (9408, 64, 2, 1, 1597), (64, 2048, 28, 4, 2564), (7872, 128, 32, 4, 3225),
    (128, 1856, 32, 4, 2908), (9664, 448, 20, 4, 648), (5440, 13056, 20, 4, 230), (1024, 9408, 8, 4, 2253),
    (8192, 11712, 12, 4, 399), (7808, 10368, 3, 1, 583), (9856, 6464, 3, 1, 781), (6848, 10240, 8, 1, 812),
    (8256, 6656, 2, 2, 1137), (7936, 128, 8, 4, 6266), (7232, 6272, 1, 1, 1623), (1344, 4800, 2, 1, 11678),
    (6080, 128, 32, 4, 3870), (9664, 128, 4, 4, 10788), (8192, 128, 64, 8, 774)]
# q|k|v on 256 x 256 with eight wavefronts and a whole last round
LAYERS += [(256, 128, 4, 2, 13551)]
# gate|up whose workgroups stay, on 224 x 192, 320 x 160 (split last round) and 192 x 256 (split last round, whole), and of two to three
# rounds with a split last round whose workgroups go, on 320 x 192 and 256 x 256 (the other forms of both: test_gpu_gemm_resident.py)
LAYERS += [(64, 18752, 3, 3, 983), (1344, 6848, 9, 3, 4705), (1088, 22016, 6, 3, 1137), (64, 19648, 3, 1, 1071), (3072, 24896, 12, 4, 590),
           (3264, 8320, 2, 1, 961)]
# q|k|v of one k-tile in many rounds
LAYERS += [(64, 192, 40, 8, 12001)]
# ragged rows and columns between the others' sizes; sums of up to 24704 products
LAYERS += [
    (512, 384, 2, 1, 5470), (128, 832, 21, 3, 8714), (64, 1344, 16, 8, 15745), (9216, 64, 2, 1, 5273),
    (8192, 192, 64, 8, 454), (4992, 8512, 24, 3, 772), (64, 24704, 1, 1, 802), (6144, 1216, 4, 2, 6859),
    (8192, 320, 16, 8, 513), (7040, 576, 40, 8, 3050), (3648, 22144, 24, 3, 1129), (8640, 128, 56, 8, 512),
    (2880, 192, 32, 8, 10945), (1216, 20800, 5, 1, 1594), (1856, 22016, 16, 2, 1040), (7104, 256, 21, 3, 9397),
    (1984, 64, 32, 4, 10637), (8192, 12544, 3, 3, 1123)]
# (requests, vocabulary, hidden size) of heads, on the tile that only they use
HEADS = [(100, 151936, 64), (65, 151936, 192), (8, 152064, 3584), (127, 152060, 320)]


def choice(epilogue, M, N, K, scratch=1, deferred=1):
    """((tile rows, tile columns, workgroups per CU, wavefronts), epilogue, "whole" | "k ranges" | "split last round"):
    the first names one row of the library's list of tiles."""
    f, waves = vlc.lib().vlc_probe_gemm_choice, vlc.lib().vlc_probe_gemm_waves
    f.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    waves.argtypes, waves.restype = f.argtypes[:-1], ctypes.c_int
    o = (ctypes.c_int32 * 5)()
    assert f(epilogue, M, N, K, scratch, deferred, o) == 0
    return (*o[:3], waves(epilogue, M, N, K, scratch, deferred)), epilogue, "k ranges" if o[3] > 1 else "split last round" if o[4] > 1 else "whole"


def stays(epilogue, M, N, K, scratch=1, deferred=1):
    """Whether the workgroups of that product stay for several tiles."""
    f = vlc.lib().vlc_probe_gemm_stays
    f.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int, ctypes.c_int]
    return bool(f(epilogue, M, N, K, scratch, deferred))


def kernel(*product):
    """The choice, and whether its workgroups stay: a kernel of its own for the same tile and epilogue."""
    return (*choice(*product), "stays" if stays(*product) else "goes")


def layer_choices(H, I, Hq, Hkv, rows):
    """The four products of a chained layer, and the down projection of one that is not."""
    hd, nqkv = Hq * 128, (Hq + 2 * Hkv) * 128
    return {"qkv": kernel(FLOAT, rows, nqkv, H), "o": kernel(RESIDUAL, rows, H, hd), "gate_up": kernel(SWIGLU, rows, I, H),
            "down": kernel(RESIDUAL, rows, H, I), "down alone": kernel(RESIDUAL, rows, H, I, 1, 0)}


def test_every_choice_is_among_the_tested_layers():
    """1 to 30000 rows at the decoder shapes of the workloads and three more, and the heads: no tile is launched with an
    epilogue, a split and workgroups that stay or go which the layers of this file and of test_gpu_gemm_resident.py do not run."""
    from test_gpu_gemm_resident import CASES
    tested = {kernel(FLOAT, rows, vocab, H, 0, 0) for rows, vocab, H in HEADS}
    for l in LAYERS + [layer for _, _, layer in CASES]:
        tested |= set(layer_choices(*l).values())
    shapes = [(s.H, s.I, s.Hq, s.Hkv) for s in syn.SHAPES.values() if s.dtype == "bf16" and s.D == 128]
    shapes += [(5120, 13824, 40, 8), (1536, 8960, 12, 2), (2048, 11008, 16, 2)]
    for H, I, Hq, Hkv in shapes:
        rows = 1
        while rows < 30000:
            for name, c in layer_choices(H, I, Hq, Hkv, rows).items():
                assert c in tested, (name, H, I, Hq, Hkv, rows, c)
            rows = max(rows + 1, int(rows * 1.01))
    for H in (64, 512, 2048, 2560, 3072, 3584, 4096, 8192):
        for vocab in (256, 4096, 32000, 151936, 152064):
            for rows in (1, 8, 33, 64, 65, 128, 129, 300, 700, 2000):
                assert kernel(FLOAT, rows, vocab, H, 0, 0) in tested, (H, vocab, rows)


def test_choices_that_measure_faster():
    """Products at which prices have named a slower configuration (us on cold weights, that one against the expected one)."""
    # k ranges that do not all start on one channel: 128 k-tiles in 4 ranges against 3, 34.7 / 28.2
    assert choice(RESIDUAL, 40, 8192, 8192)[0][0] <= 128
    o = (ctypes.c_int32 * 5)()
    vlc.lib().vlc_probe_gemm_choice(RESIDUAL, 40, 8192, 8192, 1, 1, o)
    assert o[3] > 1 and -(-128 // o[3]) % 32 != 0, list(o)
    # heads with few columns, on the two-per-CU tile against 64 x 128: 25.8 / 14.5, 34.1 / 19.1, 112 / 44 at 8 requests
    for H in (2560, 3584, 8192):
        for rows in (1, 8, 64):
            assert choice(FLOAT, rows, 4096, H, 0, 0)[0] == (64, 128, 1, 4)
    # float products whose workgroups stay for several tiles: q|k|v, staying against going, 546 / 538, 327 / 323, 476 / 465, 651 / 639
    for rows, N, K in ((4183, 10240, 8192), (8262, 6144, 4096), (12395, 6144, 4096), (23616, 4608, 3584)):
        assert not stays(FLOAT, rows, N, K)
    # gate|up in many rounds over more than the caches hold, staying against going: 3759 / 3706, 6583 / 6146, 2896 / 2767, 5560 / 5269
    for rows, N, K in ((18944, 18944, 3584), (31000, 18944, 3584), (13500, 13824, 5120), (7500, 29568, 8192)):
        assert not stays(SWIGLU, rows, N, K)
    # and where staying is faster: 3127 / 3150 (390 MB of operands), 3503 / 3543 (19 rounds), 1314 / 1349, 1131 / 1157
    for rows, N, K in ((16500, 18944, 3584), (5200, 29568, 8192), (31000, 8960, 1536), (5824, 18944, 3584)):
        assert stays(SWIGLU, rows, N, K)


def close(got, want, rtol, atol, what):
    err = (got.float() - want).abs()
    bad = err > atol + rtol * want.abs()
    assert not bad.any(), "%s: %d of %d outside tolerance, first at %s, largest error %.3e" % (
        what, int(bad.sum()), bad.numel(), tuple(bad.nonzero()[0].tolist()), err.max().item())


@pytest.mark.gpu
@pytest.mark.parametrize("H,I,Hq,Hkv,rows", LAYERS)
def test_layer_products_on_every_tile(H, I, Hq, Hkv, rows):
    """All rows and columns of the four products against float32 matmuls of the same inputs (the GPU's own previous stage).
    Float outputs: both sides sum at most 9856 float products of about 0.016 (sums of about 2) in some order; every addition
    rounds by 2^-24 of its partial sum, sqrt(9856) * 2^-24 * 2 = 1e-5 in all; typically 1e-4 apart at the largest of all
    outputs.  A missing or doubled k-tile shows as 0.1 and more.  bf16 outputs: one rounding (2^-9) on top, twice that allowed."""
    sh = dataclasses.replace(syn.SHAPES["tiny_bf16"], L=1, H=H, I=I, Hq=Hq, Hkv=Hkv)
    print("layer", H, I, Hq, Hkv, rows, layer_choices(H, I, Hq, Hkv, rows), flush=True)
    rec, dt = R.make_shape(sh), torch.bfloat16
    plans = R.DevicePlans([syn.Request([syn.Segment(0, rows, False)], 0)], 1, k=np.zeros(1, dtype=np.int32), all_rows=True)
    assert plans.n_rows == [rows]
    W = R.DeviceWeights.random(sh, dt, 41)
    g = torch.Generator(device=DEV)
    g.manual_seed(rows)
    h_in = torch.randn((rows, H), generator=g, device=DEV).to(dt)
    kc = torch.zeros((rows, Hkv, 128), device=DEV, dtype=dt)
    vc, h_out, chained = torch.zeros_like(kc), torch.empty_like(h_in), torch.empty_like(h_in)
    ws = R.Workspace(rec, rows)
    record = plans.record(0, rows, rows)
    vlc.vlc_layer_forward(rec, W.rec, record, h_in, h_out, kc, vc, ws.t)
    off = vlc.vlc_layer_workspace_layout(rec, rows)

    def stage(name, cols, t):
        size = 4 if t == torch.float32 else 2
        return ws.t[off[name]:off[name] + rows * cols * size].view(t).reshape(rows, cols)

    f = lambda t: t.float()
    w = {k: f(v) for k, v in W.t.items() if v is not None}
    close(stage("qkv", sh.n_qkv, torch.float32), torch.addmm(w["b_qkv"], f(stage("xn", H, dt)), w["w_qkv"].T), 1e-3, 1e-3, "q|k|v")
    close(stage("h1", H, dt), f(h_in) + f(stage("o", Hq * 128, dt)) @ w["w_o"].T, 2.0 ** -8, 1e-3, "o projection + residual")
    gate, up = (f(stage("n2", H, dt)) @ w["w_gate_up"].T).split(I, 1)
    close(stage("act", I, dt), torch.nn.functional.silu(gate) * up, 2.0 ** -8, 2e-3, "gate|up + SwiGLU")
    del gate, up
    want = f(stage("h1", H, dt)) + f(stage("act", I, dt)) @ w["w_down"].T
    close(h_out, want, 2.0 ** -8, 1e-3, "down projection + residual")
    # chained: the same layer, but the kernel after the down projection also takes the next norm and sums its k ranges
    vlc.vlc_layer_forward_chained(rec, W.rec, record, h_in, chained, kc, vc, ws.t, False, W.t["w_ln1"])
    close(chained, want, 2.0 ** -8, 1e-3, "down projection + residual, chained")


@pytest.mark.gpu
@pytest.mark.parametrize("rows,vocab,H", HEADS)
def test_head_products(rows, vocab, H):
    """All logits against a float32 matmul of the GPU's normed rows (which open the workspace); tolerance as above."""
    assert choice(FLOAT, rows, vocab, H, 0, 0)[0] == (128, 160, 2, 4)
    g = torch.Generator(device=DEV)
    g.manual_seed(vocab + rows)
    h = torch.randn((rows, H), generator=g, device=DEV).to(torch.bfloat16)
    w = (0.02 * torch.randn((vocab, H), generator=g, device=DEV)).to(torch.bfloat16)
    logits, token = torch.zeros((rows, vocab), device=DEV), torch.zeros(rows, device=DEV, dtype=torch.int32)
    ws = torch.empty(vlc.vlc_first_token_workspace_bytes(H, rows, vlc.VLC_BF16), device=DEV, dtype=torch.uint8)
    vlc.vlc_first_token(h, torch.arange(rows, device=DEV, dtype=torch.int32), 1e-6, torch.ones(H, device=DEV, dtype=torch.bfloat16),
                        w, logits, token, ws)
    normed = ws[:rows * H * 2].view(torch.bfloat16).reshape(rows, H)
    close(logits, normed.float() @ w.float().T, 1e-3, 1e-3, "logits")

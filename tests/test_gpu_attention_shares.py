"""Attention whose key ranges are shared out over several workgroups (few rows) against the whole form of the kernel on the
same queries, keys and values."""
import ctypes
import dataclasses

import numpy as np
import pytest
import torch

import paper_2512_12977_amd as vlc
import vlc_synth as syn
from paper_2512_12977_amd import runner as R

DEV = "cuda"


def most_shares(n, Hq, Hkv, slots):
    """The most shares that a row tile of such a layer may take; 1: nothing is shared out."""
    f = vlc.lib().vlc_probe_attention_shares
    f.argtypes, f.restype = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int64], ctypes.c_int
    return f(n, Hq, Hkv, slots)


def layer_attention(Hq, Hkv, requests, seed=3, spoil=None):
    """One layer over requests given as runs of (computed rows, keys that are only read): the queries, the attention output
    of the layer, that of the stand-alone entry point (which shares nothing out), the rows and the most shares.
    spoil(h_in) may edit the input."""
    sh = dataclasses.replace(syn.SHAPES["tiny_bf16"], L=1, H=256, I=64, Hq=Hq, Hkv=Hkv)
    reqs, at = [], 0
    for runs in requests:
        segs, s = [], 0
        for rows, keys in runs:
            if rows:
                segs.append(syn.Segment(s, rows, False))
            if keys:
                segs.append(syn.Segment(s + rows, keys, True, 0, 0))
            s += rows + keys
        reqs.append(syn.Request(segs, at))
        at += s
    plans = R.DevicePlans(reqs, 1, k=np.zeros(1, dtype=np.int32))
    n, rec, dt = plans.n_rows[0], R.make_shape(sh), torch.bfloat16
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    W = R.DeviceWeights.random(sh, dt, 5)
    h_in = torch.randn((at, sh.H), generator=g, device=DEV).to(dt)
    if spoil:
        spoil(h_in)
    kc, vc = (torch.randn((at, Hkv, 128), generator=g, device=DEV).to(dt) for _ in range(2))
    ws, h_out = R.Workspace(rec, n), torch.empty((n, sh.H), device=DEV, dtype=dt)
    vlc.vlc_layer_forward(rec, W.rec, plans.record(0, at, at), h_in, h_out, kc, vc, ws.t)
    off = vlc.vlc_layer_workspace_layout(rec, n)
    stage = lambda name: ws.t[off[name]:off[name] + n * Hq * 256].view(dt).reshape(n, Hq, 128)
    q, shared = stage("q").clone(), stage("o").float()
    whole = torch.empty_like(q)
    vlc.vlc_sparse_q_attention(q, kc, vc, plans.dev[0]["kv_start"], plans.dev[0]["kv_len"], 128 ** -0.5, whole)
    return shared, whole.float(), n, most_shares(n, Hq, Hkv, at)


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,requests", [
    (28, 4, [[(1, 0)]]),                                                   # one row, one key: whole on both sides
    (28, 4, [[(27, 1369), (43, 0)]]),                                      # a question about an image
    (32, 8, [[(61, 1247), (33, 1350), (33, 1400), (87, 0)]]),              # images between texts, ragged ends
    (64, 8, [[(10, 1290)] * 8 + [(256, 0)]]),                              # most rows at the very end
    (64, 8, [[(256, 1290)] + [(10, 1290)] * 6]),                           # most rows in front
    (28, 4, [[(100, 900), (60, 0)], [(7, 3000), (3, 0)], [(40, 0)], [(1, 64), (64, 0)]]),   # requests of unequal sizes
    (12, 3, [[(200, 2000), (100, 0)]]),                                    # kv heads that do not divide the XCDs
    (5, 5, [[(130, 500), (300, 0)], [(17, 0)]]),
    (128, 1, [[(300, 700), (55, 0)]]),                                     # a tile is one row
    (16, 1, [[(4080, 0)]]),                                                # 510 pairs, tiles of up to 64 blocks
    (16, 1, [[(4088, 0)]]),                                                # 511 pairs in 512 slots: the last count that shares
    (8, 8, [[(100, 64 * 130), (40, 0)]]),                                  # the most shares, long ranges
])
def test_shared_keys_equal_whole(Hq, Hkv, requests):
    """Both forms round probabilities and outputs to bf16 once; their running maxima differ, so a probability may round
    the other way (2^-9 of it): the outputs differ by rounding, 2^-8 of a value and 2^-9 of the values' scale."""
    shared, whole, n, shares = layer_attention(Hq, Hkv, requests)
    assert (shares > 1) == (n > 1)
    err = (shared - whole).abs()
    bad = err > 2.0 ** -8 * whole.abs() + 2.0 ** -8
    assert not bad.any(), (n, int(bad.sum()), err.max().item(), bad.nonzero()[0].tolist())
    assert ((shared - whole).norm() / whole.norm()).item() < 2e-3


def test_sharing_ends_at_512_pairs():
    """4088 rows are 511 tiles of 8 rows, the last count that shares; 4089 are 512."""
    assert most_shares(4088, 16, 1, 4088) == 2 and most_shares(4089, 16, 1, 4089) == 1


@pytest.mark.gpu
def test_a_nan_query_row_stays_nan_in_every_share():
    """A row whose scores are all NaN has no running maximum in any share; the merge must not turn it into zeros."""
    def spoil(h):
        h[1396] = float("nan")                   # a row of the text behind the image

    shared, whole, n, shares = layer_attention(28, 4, [[(27, 1369), (43, 0)]], spoil=spoil)
    assert shares > 1
    row = 27                                     # the rows in front, then the first of that text
    assert torch.isnan(whole[row]).all() and torch.isnan(shared[row]).all()

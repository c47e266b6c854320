"""Full-size parity on sampled outputs: one layer of the long-context batch (8 requests x 18432
slots, 18944 packed recomputed rows, 7B shape) and of the 72B-shaped workload runs on the GPU exactly
as bench.py launches it; for a few sampled rows every stage is compared with the oracle evaluated on
the GPU's own input to that stage (element-wise, 2e-2 + 1e-2*|o|), and K/V rows are compared end to end."""
import numpy as np
import pytest
import torch

import vlc_synth as syn
from oracle import vlc_oracle as orc
import paper_2512_12977_amd as vlc
from paper_2512_12977_amd import runner as R
from helpers import plan_steps, counts_for, assert_close

pytestmark = pytest.mark.gpu
DEV = "cuda"


def back(t):
    return t.float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("name,layer,req_ids,n_rows", [("c4", 0, (0, 5), 18944), ("c5", 0, (0,), None),
                                                       ("c5", 79, (0,), None), ("c3", 0, (0,), None),
                                                       ("c3", 20, (0,), None), ("c4_5", 0, (2, 7), 22912),
                                                       ("c5", 40, (0,), None)])
def test_full_size_layer_sampled_rows(name, layer, req_ids, n_rows):
    """c4: the long-context batch at the 7B shape, 2 % recomputed; c4_5: the same at 5 % (51 leading tokens per
    image).  c5: the 72B shape (64 query / 8 kv heads, MLP width 29568) at its first layer (the highest rate of the
    layer-aware plan), a middle one and its last (text rows only: every GEMM splits k).  c3: four images placed in
    shuffled order, so the reused keys are re-rotated forwards and backwards; its first layer (the highest rate)
    and a deep one.  The layer reads the embeddings as its input rows, whatever its depth."""
    wl = syn.make_workload(name)
    sh = wl.shape
    st = orc.STORE[sh.dtype]
    dt = R.torch_dtype(sh.dtype)
    rec = R.make_shape(sh)
    k, explicit = plan_steps(wl)
    k = k[layer:layer + 1]
    W = syn.layer_weights(sh, wl.seed, layer)
    emb = syn.embedding_rows(wl)
    Kc, Vc = syn.cached_kv(wl, layer)
    total = wl.total_slots

    plans = R.DevicePlans(wl.requests, 1, k=k)
    n = plans.n_rows[0]
    assert n_rows is None or n == n_rows
    print("%s layer %d: %d rows (k = %d)" % (name, layer, n, int(k[0])), flush=True)
    ws = R.Workspace(rec, n)
    dW = R.DeviceWeights(W, dt)
    kp, vp = torch.from_numpy(Kc).to(DEV).to(dt), torch.from_numpy(Vc).to(DEV).to(dt)
    kc = torch.zeros((total, sh.Hkv, sh.D), device=DEV, dtype=dt)
    vc = torch.zeros_like(kc)
    h_in = torch.from_numpy(emb).to(DEV).to(dt)
    h_out = torch.empty((n, sh.H), device=DEV, dtype=dt)
    R.run_layer(rec, dW, plans.record(0, total, total, kp, vp), h_in, h_out, kc, vc, ws)
    torch.cuda.synchronize()

    off = vlc.vlc_layer_workspace_layout(rec, n)
    shapes = {"xn": (n, sh.H), "qkv": (n, sh.n_qkv), "q": (n, sh.Hq * sh.D), "o": (n, sh.Hq * sh.D),
              "h1": (n, sh.H), "n2": (n, sh.H), "act": (n, sh.I)}

    def ws_rows(name, rows):
        tdt, size = (torch.float32, 4) if name == "qkv" else (dt, 2)
        shp = shapes[name]
        nb = shp[0] * shp[1] * size
        full = ws.t[off[name]:off[name] + nb].view(tdt).reshape(shp)
        return back(full[torch.from_numpy(rows).to(DEV)])

    slot_all = plans.host["slot"][0, :n].astype(np.int64)
    rng = np.random.default_rng(0)
    for r_i in req_ids:
        req = wl.requests[r_i]
        counts = counts_for(req, k, explicit, 0)
        slots = orc.select_slots(req.segments, counts)               # relative to the request
        first = int(np.searchsorted(slot_all, req.kv_start))          # its rows in the packed list
        assert np.array_equal(slot_all[first:first + len(slots)], req.kv_start + slots)
        # sampled rows: first and last text rows, leading rows of an early and a late image, random ones
        cand = np.concatenate([[0, 1, len(slots) - 1, len(slots) - 2],
                               np.minimum(np.searchsorted(slots, [s.start for s in req.segments if s.is_image][::5]),
                                          len(slots) - 1),
                               rng.integers(0, len(slots), size=6)])
        sel = np.unique(cand)
        rows = first + sel
        # the request's blended K/V as the GPU left them
        gK = back(kc[req.kv_start:req.kv_start + req.S])
        gV = back(vc[req.kv_start:req.kv_start + req.S])
        # end to end: reused keys rotated by the delta, values copied (whole request, element-wise)
        Kb, Vb = orc.blended_kv_before_scatter(sh, req, counts, st(Kc), st(Vc), st)
        reused, _, old = orc.reused_slots(req.segments, counts)
        if name == "c3":     # images moved in both directions: the re-rotation is checked for either sign
            assert set(np.sign(req.pos_start + reused - old).tolist()) == {-1, 1}
        assert_close(gK[reused], Kb[reused], sh.dtype, "reused K of request %d" % r_i)
        np.testing.assert_array_equal(gV[reused], Vb[reused])
        # stage by stage on the sampled rows
        x = st(emb[req.kv_start:req.kv_start + req.S])[slots[sel]]
        forced = {name: ws_rows(name, rows) for name in ("xn", "qkv", "h1", "n2", "act")}
        forced["q"] = ws_rows("q", rows).reshape(len(sel), sh.Hq, sh.D)
        forced["o"] = ws_rows("o", rows).reshape(len(sel), sh.Hq, sh.D)
        forced["K"], forced["V"] = gK, gV
        Ko, Vo = gK.copy(), gV.copy()
        r = orc.layer_stages(sh, W, x, slots[sel], req.pos_start + slots[sel], Ko, Vo, st, forced=forced)
        assert_close(forced["xn"], r["xn"], sh.dtype, "xn")
        assert_close(forced["qkv"], r["qkv"], sh.dtype, "qkv")
        assert_close(forced["q"], r["q"], sh.dtype, "q")
        # fresh k, v of the sampled rows as scattered by the GPU vs the oracle's from the GPU's projection
        assert_close(gK[slots[sel]], r["K"][slots[sel]], sh.dtype, "fresh K")
        assert_close(gV[slots[sel]], r["V"][slots[sel]], sh.dtype, "fresh V")
        assert_close(forced["o"], r["o"], sh.dtype, "attention (up to %d keys)" % (slots[sel].max() + 1))
        assert_close(forced["h1"], r["h1"], sh.dtype, "h1")
        assert_close(forced["n2"], r["n2"], sh.dtype, "n2")
        assert_close(forced["act"], r["act"], sh.dtype, "act")
        assert_close(back(h_out[torch.from_numpy(rows).to(DEV)]), r["h2"], sh.dtype, "h_out")


@pytest.mark.parametrize("shape,n_text,n_image,all_rows", [("7b", 200, 5000, True), ("7b", 720, 2000, False),
                                                           ("7b", 1184, 0, True), ("7b", 1600, 0, True),
                                                           ("72b", 1000, 0, True), ("7b", 300, 0, True),
                                                           ("72b", 600, 0, True)])
def test_layer_rows_that_leave_a_partial_round_of_gemm_tiles(shape, n_text, n_image, all_rows):
    """Row counts of the full 7B and 72B layers between the listed workloads, with ragged row tiles, split k ranges and last
    rounds of tiles that do not fill the chip (some of which are split along k).  Every 13th row (so every tile of every
    GEMM is sampled) is compared stage by stage with the oracle.  Which tile each product lands on is a matter of
    prices; test_gpu_gemm_tiles.py asks for it and runs every combination that the dispatcher returns."""
    sh = syn.SHAPES[shape]
    st = orc.STORE[sh.dtype]
    dt = R.torch_dtype(sh.dtype)
    rec = R.make_shape(sh)
    a = n_text // 2
    segs = [syn.Segment(0, a, False)]
    if n_image:
        segs.append(syn.Segment(a, n_image, True, 7, 0))
    segs.append(syn.Segment(a + n_image, n_text - a, False))
    req = syn.Request(segs, 0)
    wl = syn.Workload("tail_%d_%d" % (n_text, n_image), sh, [req], max(n_image, 1), "static", static_k=0, seed=21)
    W = syn.layer_weights(sh, wl.seed, 0)
    emb = syn.embedding_rows(wl)
    Kc, Vc = syn.cached_kv(wl, 0)
    total = wl.total_slots
    plans = R.DevicePlans(wl.requests, 1, k=np.zeros(1, dtype=np.int32), all_rows=all_rows)
    n = plans.n_rows[0]
    assert n == (total if all_rows else n_text)
    ws = R.Workspace(rec, n)
    dW = R.DeviceWeights(W, dt)
    kp, vp = torch.from_numpy(Kc).to(DEV).to(dt), torch.from_numpy(Vc).to(DEV).to(dt)
    kc = torch.zeros((total, sh.Hkv, sh.D), device=DEV, dtype=dt)
    vc = torch.zeros_like(kc)
    h_in = torch.from_numpy(emb).to(DEV).to(dt)
    h_out = torch.empty((n, sh.H), device=DEV, dtype=dt)
    R.run_layer(rec, dW, plans.record(0, total, total, None if all_rows else kp, None if all_rows else vp),
                h_in, h_out, kc, vc, ws)
    torch.cuda.synchronize()

    off = vlc.vlc_layer_workspace_layout(rec, n)
    shapes = {"xn": (n, sh.H), "qkv": (n, sh.n_qkv), "q": (n, sh.Hq * sh.D), "o": (n, sh.Hq * sh.D),
              "h1": (n, sh.H), "n2": (n, sh.H), "act": (n, sh.I)}
    sel = np.unique(np.concatenate([np.arange(0, n, 13), [n - 1]]))
    sel_t = torch.from_numpy(sel).to(DEV)

    def ws_rows(name):
        tdt, size = (torch.float32, 4) if name == "qkv" else (dt, 2)
        shp = shapes[name]
        return back(ws.t[off[name]:off[name] + shp[0] * shp[1] * size].view(tdt).reshape(shp)[sel_t])

    slots = plans.host["slot"][0, :n].astype(np.int64)
    forced = {name: ws_rows(name) for name in ("xn", "qkv", "h1", "n2", "act")}
    forced["q"] = ws_rows("q").reshape(len(sel), sh.Hq, sh.D)
    forced["o"] = ws_rows("o").reshape(len(sel), sh.Hq, sh.D)
    gK, gV = back(kc), back(vc)
    forced["K"], forced["V"] = gK, gV
    x = st(emb)[slots[sel]]
    r = orc.layer_stages(sh, W, x, slots[sel], orc.positions_of(req, slots[sel]), gK.copy(), gV.copy(), st, forced=forced)
    assert_close(forced["xn"], r["xn"], sh.dtype, "xn")
    assert_close(forced["qkv"], r["qkv"], sh.dtype, "qkv")
    assert_close(forced["q"], r["q"], sh.dtype, "q")
    assert_close(forced["o"], r["o"], sh.dtype, "attention")
    assert_close(forced["h1"], r["h1"], sh.dtype, "h1 (o-proj + residual)")
    assert_close(forced["n2"], r["n2"], sh.dtype, "n2")
    assert_close(forced["act"], r["act"], sh.dtype, "act (gate|up + SwiGLU)")
    assert_close(back(h_out[sel_t]), r["h2"], sh.dtype, "h_out (down-proj + residual)")


@pytest.mark.parametrize("name", ["c2", "c3"])
def test_chained_layers_at_the_7b_shape(name):
    """Three layers of a 7B-shaped workload through vlc_layer_forward_chained (the down projection splits its k
    range, so the fused sum + residual + norm kernel runs).  c2: 596 recomputed rows in every layer.  c3: 1020, 1012
    and 1000 rows - each layer drops rows of the one above, and the norm is written through the row list.
    (1) Every layer's h_out and K/V equal, bit for bit, what vlc_layer_forward gives layer by layer.  (2) After a
    layer that was given its successor's norm weight, every 13th row of h_out and every 13th of the normed rows left
    in the workspace are compared with the oracle evaluated on the GPU's own h1 and SwiGLU product of that layer."""
    wl = syn.make_workload(name)
    sh = wl.shape
    st = orc.STORE[sh.dtype]
    dt = R.torch_dtype(sh.dtype)
    rec = R.make_shape(sh)
    L = 3
    k, _ = plan_steps(wl)
    plans = R.DevicePlans(wl.requests, L, k=k[:L])
    ns, total = plans.n_rows, wl.total_slots
    links = [R.chain_link(plans, l) for l in range(L)]
    assert [a for a, _ in links] == [True, True, False]
    if name == "c2":
        assert ns == [596] * 3 and links[0][1] is None and links[1][1] is None
    else:
        assert ns[0] > ns[1] > ns[2] and links[0][1] is not None and links[1][1] is not None
        assert int((links[1][1] >= 0).sum().item()) == ns[2]
    Ws = [syn.layer_weights(sh, wl.seed, l) for l in range(L)]
    dWs = [R.DeviceWeights(W, dt) for W in Ws]
    pools = [[torch.from_numpy(a).to(DEV).to(dt) for a in syn.cached_kv(wl, l)] for l in range(L)]
    emb = torch.from_numpy(syn.embedding_rows(wl)).to(DEV).to(dt)
    ws = R.Workspace(rec, max(ns))
    recs = [plans.record(l, total if l == 0 else ns[l - 1], total, pools[l][0], pools[l][1]) for l in range(L)]

    def caches():
        return ([torch.zeros((total, sh.Hkv, sh.D), device=DEV, dtype=dt) for _ in range(L)],
                [torch.zeros((total, sh.Hkv, sh.D), device=DEV, dtype=dt) for _ in range(L)])

    # layer by layer, every layer norming its own input
    kc0, vc0 = caches()
    hs0, h_in = [], emb
    for l in range(L):
        h_out = torch.empty((ns[l], sh.H), device=DEV, dtype=dt)
        R.run_layer(rec, dWs[l], recs[l], h_in, h_out, kc0[l], vc0[l], ws)
        hs0.append(h_out)
        h_in = h_out
    torch.cuda.synchronize()

    # chained, stopping after layer 1 to look at what it left behind
    kc1, vc1 = caches()
    hs1 = [torch.empty((ns[l], sh.H), device=DEV, dtype=dt) for l in range(L)]
    print("chained layer 0", flush=True)
    vlc.vlc_layer_forward_chained(rec, dWs[0].rec, recs[0], emb, hs1[0], kc1[0], vc1[0], ws.t, False,
                                  dWs[1].t["w_ln1"], links[0][1])
    print("chained layer 1", flush=True)
    vlc.vlc_layer_forward_chained(rec, dWs[1].rec, recs[1], hs1[0], hs1[1], kc1[1], vc1[1], ws.t, True,
                                  dWs[2].t["w_ln1"], links[1][1])
    torch.cuda.synchronize()
    n, m = ns[1], ns[2]
    off = vlc.vlc_layer_workspace_layout(rec, n)
    sel = np.unique(np.concatenate([np.arange(0, n, 13), [n - 1]]))

    def ws_rows(field, rows, idx, cols):
        return back(ws.t[off[field]:off[field] + rows * cols * 2].view(dt).reshape(rows, cols)[torch.from_numpy(idx).to(DEV)])

    h1, act = ws_rows("h1", n, sel, sh.H), ws_rows("act", n, sel, sh.I)
    assert_close(back(hs1[1][torch.from_numpy(sel).to(DEV)]), st(h1 + orc.linear(act, st(Ws[1]["w_down"]))), sh.dtype,
                 "h_out of a chained layer")
    sel2 = np.unique(np.concatenate([np.arange(0, m, 13), [m - 1]]))
    src = plans.host["map"][2, :m].astype(np.int64)[sel2]          # the rows of layer 1 they come from
    xn_next = ws_rows("xn", m, sel2, sh.H)
    assert_close(xn_next, st(orc.rmsnorm(back(hs1[1][torch.from_numpy(src).to(DEV)]), st(Ws[2]["w_ln1"]), sh.eps)),
                 sh.dtype, "input norm left for the next layer")
    print("chained layer 2", flush=True)
    vlc.vlc_layer_forward_chained(rec, dWs[2].rec, recs[2], hs1[1], hs1[2], kc1[2], vc1[2], ws.t, True, None)
    torch.cuda.synchronize()
    for l in range(L):
        assert torch.equal(hs1[l], hs0[l]), "h_out of layer %d" % l
        assert torch.equal(kc1[l], kc0[l]) and torch.equal(vc1[l], vc0[l]), "K/V of layer %d" % l

    # the runner's loop over all layers, chained and not
    kc2, vc2 = caches()
    hbuf = [torch.empty((max(ns), sh.H), device=DEV, dtype=dt) for _ in range(2)]
    out = R.run_layers(rec, dWs, plans, recs, emb, hbuf, kc2, vc2, ws)
    torch.cuda.synchronize()
    assert torch.equal(out[:ns[-1]], hs0[L - 1]) and all(torch.equal(kc2[l], kc0[l]) for l in range(L))
    out = R.run_layers(rec, dWs, plans, recs, emb, hbuf, kc2, vc2, ws, chain=False)
    torch.cuda.synchronize()
    assert torch.equal(out[:ns[-1]], hs0[L - 1])


def test_free_running_28_layers_of_c2_as_the_benchmark_runs_them(capsys):
    """All 28 layers of configuration 2 (7B shape, bf16, 596 recomputed rows of 1600 slots) exactly as bench.py
    runs a step - the reused keys of every layer placed by one launch ahead of the loop, every layer through
    vlc_layer_forward_chained on its predecessor's output - against the oracle's free-running stack.
    Element-wise (2e-2 + 1e-2 |o|): K and V of the first layer (identical inputs on both sides) and the reused
    K/V of every layer (they depend on no layer output; V bit-exact).  Every layer: h and the fresh K, V rows under
    the noise criterion of a chain of bf16 roundings - two correct bf16 implementations drift apart because one
    flipped rounding moves every later value, so with o16 the oracle at bf16 storage and o64 the oracle unrounded
    (Frobenius norms over the layer's rows): |g - o16| / |o16| <= |o16 - o64| / |o64| (the GPU is as close to
    the bf16 oracle as bf16 storage moves the oracle itself) and |g - o64| <= 1.25 |o16 - o64| (and no further
    from the exact result than storage explains).  The per-layer figures are printed."""
    import sys
    wl = syn.make_workload("c2")
    sh = wl.shape
    L = sh.L
    dt = R.torch_dtype(sh.dtype)
    rec = R.make_shape(sh)
    req = wl.requests[0]
    k, explicit = plan_steps(wl)
    emb = syn.embedding_rows(wl)
    total = wl.total_slots

    def say(msg):
        with capsys.disabled():
            print(msg, file=sys.stderr, flush=True)

    say("\nfree-running c2: generating %d layers" % L)
    Ws = [syn.layer_weights(sh, wl.seed, l) for l in range(L)]
    caches = [syn.cached_kv(wl, l) for l in range(L)]
    plans = R.DevicePlans(wl.requests, L, k=k)
    ws = R.Workspace(rec, max(plans.n_rows))
    dWs = [R.DeviceWeights(W, dt) for W in Ws]
    kps = [torch.from_numpy(c[0]).to(DEV).to(dt) for c in caches]
    vps = [torch.from_numpy(c[1]).to(DEV).to(dt) for c in caches]
    kcs = [torch.zeros((total, sh.Hkv, sh.D), device=DEV, dtype=dt) for _ in range(L)]
    vcs = [torch.zeros((total, sh.Hkv, sh.D), device=DEV, dtype=dt) for _ in range(L)]
    d_emb = torch.from_numpy(emb).to(DEV).to(dt)
    R.ShiftJobs(plans, kps, vps, kcs, vcs).run(sh.rope_base)
    recs, n_prev = [], total
    for l in range(L):
        recs.append(plans.record(l, n_prev, total, None, None))
        n_prev = plans.n_rows[l]
    # one layer at a time through the same chained calls run_layers makes, keeping every layer's output
    hs, h_in, ready = [], d_emb, False
    for l in range(L):
        h_out = torch.empty((plans.n_rows[l], sh.H), device=DEV, dtype=dt)
        linked, next_row = R.chain_link(plans, l)
        vlc.vlc_layer_forward_chained(rec, dWs[l].rec, recs[l], h_in, h_out, kcs[l], vcs[l], ws.t, ready,
                                      dWs[l + 1].t["w_ln1"] if linked else None, next_row)
        hs.append(h_out)
        h_in, ready = h_out, linked
    torch.cuda.synchronize()
    # the same through the runner's loop: bit-equal
    kc2 = [torch.zeros_like(t) for t in kcs]
    vc2 = [torch.zeros_like(t) for t in vcs]
    R.ShiftJobs(plans, kps, vps, kc2, vc2).run(sh.rope_base)
    hbuf = [torch.empty((max(plans.n_rows), sh.H), device=DEV, dtype=dt) for _ in range(2)]
    out = R.run_layers(rec, dWs, plans, recs, d_emb, hbuf, kc2, vc2, ws)
    torch.cuda.synchronize()
    assert torch.equal(out[:plans.n_rows[-1]], hs[-1]) and all(torch.equal(kc2[l], kcs[l]) for l in range(L))
    del dWs, kps, vps, kc2, vc2

    counts = [counts_for(req, k, explicit, l) for l in range(L)]
    say("free-running c2: oracle, bf16 storage")
    o16 = orc.selective_prefill(sh, Ws, emb, req, counts, caches, orc.STORE[sh.dtype])
    say("free-running c2: oracle, exact")
    o64 = orc.selective_prefill(sh, Ws, emb, req, counts, caches, orc.store_exact)
    nrm = np.linalg.norm
    for l in range(L):
        g_h, g_K, g_V = back(hs[l]), back(kcs[l]), back(vcs[l])
        reused, _, _ = orc.reused_slots(req.segments, counts[l])
        assert_close(g_K[reused], o16[l]["K"][reused], sh.dtype, "layer %d reused K" % l)
        np.testing.assert_array_equal(g_V[reused], o16[l]["V"][reused])
        if l == 0:      # identical inputs on both sides: element-wise
            assert_close(g_K, o16[l]["K"], sh.dtype, "layer %d K" % l)
            assert_close(g_V, o16[l]["V"], sh.dtype, "layer %d V" % l)
        fresh = np.setdiff1d(np.arange(req.S), reused)
        rel = lambda a, b: nrm(a - b) / nrm(b)
        floor = rel(o16[l]["h"], o64[l]["h"])
        dev16, dev64 = rel(g_h, o16[l]["h"]), rel(g_h, o64[l]["h"])
        kfloor, kdev16, kdev64 = (rel(o16[l]["K"][fresh], o64[l]["K"][fresh]), rel(g_K[fresh], o16[l]["K"][fresh]),
                                  rel(g_K[fresh], o64[l]["K"][fresh]))
        vfloor, vdev16, vdev64 = (rel(o16[l]["V"][fresh], o64[l]["V"][fresh]), rel(g_V[fresh], o16[l]["V"][fresh]),
                                  rel(g_V[fresh], o64[l]["V"][fresh]))
        say("layer %2d  h: g-o16 %.3e g-o64 %.3e floor %.3e | fresh K: %.3e %.3e %.3e | fresh V: %.3e %.3e %.3e"
            % (l, dev16, dev64, floor, kdev16, kdev64, kfloor, vdev16, vdev64, vfloor))
        for what, d16, d64, fl in (("h", dev16, dev64, floor), ("K", kdev16, kdev64, kfloor), ("V", vdev16, vdev64, vfloor)):
            assert d64 <= 1.25 * fl, (l, what, d64, fl)
            assert d16 <= fl, (l, what, d16, fl)

"""Kernels at the sizes where their tiling can go wrong (tile edges,
remainders, the smallest and largest of a dispatch range), against the
oracle.  The tolerances are those of the parity tests."""
from __future__ import annotations

import time

import numpy as np
import pytest

from tests import parity as P
from tests.test_gpu_parity import (L, O, _check_down_up, _check_structure, _cloud, _dev, _distribute_backward_case, _host,  # noqa: F401
                                   _pair)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# linear backward: 16-class blocks, 64-column blocks, 16-row steps, 128-row chunks, unaligned class counts
@pytest.mark.parametrize("m,C,K", [(15, 4, 1), (17, 60, 16), (127, 64, 17), (129, 68, 48), (1025, 132, 49), (300, 256, 64)])
def test_linear_backward_tiles(L, O, m, C, K):  # noqa: F811
    gl, ol, g2o = _pair(L, O, _cloud(2000 + m, m, 0.6), 0.1)
    rng = np.random.default_rng(m)
    X = rng.normal(size=(ol.n, C)).astype(np.float32)
    wv = (rng.normal(size=C) / np.sqrt(C)).astype(np.float32)
    Wc = (rng.normal(size=(K, C)) / np.sqrt(C)).astype(np.float32)
    Z = rng.normal(size=(ol.m, K)).astype(np.float32)
    ref = ol.deform_slice_classify_backward(X.astype(np.float64), wv.astype(np.float64), 0.1, Wc.astype(np.float64),
                                            Z.astype(np.float64))
    got = gl.deform_slice_classify_backward(_dev(X[g2o]), _dev(wv), 0.1, _dev(Wc), _dev(Z))
    P.assert_close(P.rows_in_oracle_order(_host(got[0]), g2o), ref[0], P.TOL_F32, f"dX m={m} C={C} K={K}")
    P.assert_close(_host(got[3]), ref[3], P.TOL_F32, f"dWc m={m} C={C} K={K}")
    P.assert_close(_host(got[4]), ref[4], P.TOL_F32, f"dbc m={m} C={C} K={K}")


# weight gradient: 64 x 64 tiles, steps of 16 (fp32) and 32 (bf16) vertices, chunks of 64, missing taps
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,cin,cout", [(1, 8, 8), (9, 64, 72), (65, 56, 64), (700, 136, 128), (700, 64, 192),
                                        (3000, 24, 200)])
def test_weight_gradient_tiles(L, O, m, cin, cout, dtype):  # noqa: F811
    gl, ol, g2o = _pair(L, O, _cloud(2100 + m, m, 0.7), 0.07)
    gc, oc = gl.coarsen(), ol.coarsen()
    g2o_c = P.key_permutation(_host(gc.keys()), oc.keys())
    rng = np.random.default_rng(m)
    rnd = O.round_bf16 if dtype == "bf16" else (lambda a: a.astype(np.float32))
    dev = (lambda a: _dev(a.astype(np.float32), torch.bfloat16)) if dtype == "bf16" else _dev
    for gd, gs, od, os_, pd, ps in ((gl, gl, ol, ol, g2o, g2o), (gc, gl, oc, ol, g2o_c, g2o), (gl, gc, ol, oc, g2o, g2o_c)):
        X = rnd(rng.normal(size=(os_.n, cin)))
        dY = rnd(rng.normal(size=(od.n, cout)))
        W = np.zeros((9, cin, cout))
        _, odw, odb = od.conv_backward(os_, X.astype(np.float64), W, dY.astype(np.float64))
        fn = gd.conv_backward_bf16 if dtype == "bf16" else gd.conv_backward
        _, gdw, gdb = fn(gs, dev(X[ps]), None, dev(dY[pd]), want_dx=False)
        P.assert_close(np.transpose(_host(gdw), (0, 2, 1)), odw, P.TOL_F32, f"dW m={m} {cin}->{cout} {dtype}")
        P.assert_close(_host(gdb), odb, P.TOL_F32, f"dbias m={m} {cin}->{cout} {dtype}")
        _, none, gdb = fn(gs, dev(X[ps]), None, dev(dY[pd]), want_dx=False, want_dw=False)
        assert none is None
        P.assert_close(_host(gdb), odb, P.TOL_F32, f"dbias alone m={m} {cin}->{cout} {dtype}")


# Distribute + PointNet backward: 16-row groups, 128-entry ranges cut inside and between lists, every weight instance
@pytest.mark.parametrize("m,cf,widths,clump", [(4, 5, (16, 32, 64), 0), (32, 1, (16, 16, 16), 0), (33, 6, (16, 32, 64), 0),
                                               (600, 2, (32, 16, 48), 400), (700, 13, (32, 32, 64), 3),
                                               (500, 0, (64, 32, 32), 200)])
def test_distribute_backward_tiles(L, O, m, cf, widths, clump):  # noqa: F811
    rng = np.random.default_rng(m)
    pos = _cloud(2200 + m, m, 0.6)
    pos[m // 3:m // 3 + clump] = pos[0] + 1e-4 * rng.random((clump, 3)).astype(np.float32)
    F = rng.normal(size=(m, cf)).astype(np.float32) if cf else None
    gl, ol, g2o = _pair(L, O, pos, 0.1)
    _distribute_backward_case(L, O, gl, ol, g2o, pos, F, widths, m)


# a maximum over a list cut by 128-entry ranges, some of its rows NaN: the walk passes over NaN rows behind the list's first
# row, also where a range starts with one.  Two equal channels with an infinite gamma and weights +1 and -1 make NaN of the
# rows where they are positive and leave the others finite.
def test_distribute_backward_maximum_beside_nan(L, O):  # noqa: F811
    rng = np.random.default_rng(3)
    centres = np.stack(np.meshgrid(*[np.arange(3) * 4.0] * 3, indexing="ij"), -1).reshape(-1, 3) + [0.31, 0.42, 0.53]
    pos = np.concatenate([c + 0.02 * rng.random((300, 3)) for c in centres]).astype(np.float32)
    F = rng.normal(size=(len(pos), 4)).astype(np.float32)
    gl, ol, g2o = _pair(L, O, pos, 1.0)
    layers = [((rng.normal(size=(o, i)) / np.sqrt(i)).astype(np.float32), (0.1 * rng.normal(size=o)).astype(np.float32))
              for i, o in ((7, 16), (16, 32), (32, 64))]
    layers[1][0][1], layers[1][1][1] = layers[1][0][0], layers[1][1][0]
    layers[2][0][:, 0], layers[2][0][:, 1] = 1.0, -1.0
    gamma, beta = np.ones(7 + 16 + 32, np.float32), np.zeros(7 + 16 + 32, np.float32)
    gamma[23:25] = np.inf
    # the rows in float64; finite channels of the last layer's input and its outputs
    idx, _ = ol.simplices()
    v = idx.reshape(-1)
    counts = np.bincount(v, minlength=ol.n)
    g = np.repeat(pos.astype(np.float64), 4, 0)   # (sigma 1)
    mu = np.stack([np.bincount(v, g[:, j], ol.n) / counts for j in range(3)], 1)
    h = np.concatenate([g - mu[v], np.repeat(F.astype(np.float64), 4, 0)], 1)
    for W, b in layers[:2]:
        a = np.maximum((h - h.mean(0)) / np.sqrt(h.var(0) + 1e-5), 0.0)
        h = a @ W.T.astype(np.float64) + b
    xh = (h - h.mean(0)) / np.sqrt(h.var(0) + 1e-5)
    a = np.maximum(xh, 0.0)
    nan = xh[:, 0] > 0
    out = a[:, 2:] @ layers[2][0][:, 2:].T.astype(np.float64) + layers[2][1]
    dev = [(_dev(W), _dev(b)) for W, b in layers]
    seen = 0
    for u in np.nonzero(counts > 260)[0]:
        D = np.zeros((ol.n, 64), np.float32)
        D[u] = 1.0
        got = gl.distribute_pointnet_backward(_dev(pos), _dev(F), dev, _dev(D[g2o]), (_dev(gamma), _dev(beta)))
        dW3 = _host(got["dW3"])[:, 2:]
        rows = np.nonzero(v == u)[0]
        for c in range(64):
            dist = np.abs(a[rows, 2:] - dW3[c]).max(1)
            taken = rows[np.argmin(dist)]
            assert dist.min() < 1e-4, (u, c)
            if nan[taken]:
                continue   # the list's first row is NaN and stays
            finite = rows[~nan[rows]]
            assert out[taken, c] >= out[finite, c].max() - 1e-9, (u, c, out[taken, c], out[finite, c].max())
            seen += 1
    assert seen > 100


# convolution: rows and columns that do not fill a tile, channels that do not fill a stage, odd and even stage counts,
# every tile of the dispatch that a small lattice reaches
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,cin,cout,pre", [(1, 8, 24, False), (40, 40, 40, True), (300, 72, 136, False),
                                            (900, 136, 72, True), (5000, 64, 128, True), (9000, 32, 320, False),
                                            (300, 264, 128, True)])
def test_conv_tiles(L, O, m, cin, cout, pre, dtype):  # noqa: F811
    gl, ol, g2o = _pair(L, O, _cloud(2300 + m, m, 0.7), 0.05)
    gc, oc = gl.coarsen(), ol.coarsen()
    g2o_c = P.key_permutation(_host(gc.keys()), oc.keys())
    rng = np.random.default_rng(m)
    bf = dtype == "bf16"
    tol = P.TOL_BF16 if bf else P.TOL_F32
    rnd = O.round_bf16 if bf else (lambda a: np.asarray(a, np.float32))
    dev = (lambda a: _dev(np.asarray(a, np.float32), torch.bfloat16)) if bf else (lambda a: _dev(np.asarray(a, np.float32)))
    W = rnd(rng.normal(size=(9, cin, cout)) / np.sqrt(9 * cin))
    gW = dev(np.ascontiguousarray(np.transpose(W, (0, 2, 1))))
    bias = (0.3 * rng.normal(size=cout)).astype(np.float32)
    for gd, gs, od, os_, pd, ps, up in ((gl, gl, ol, ol, g2o, g2o, False), (gc, gl, oc, ol, g2o_c, g2o, False),
                                        (gl, gc, ol, oc, g2o, g2o_c, True)):
        X = rnd(rng.normal(size=(os_.n, cin)))
        R = rnd(rng.normal(size=(od.n, cout)))
        A = X.astype(np.float64)
        if pre:
            A = O.groupnorm(A, 4, eps=1e-5, relu=True)
            A = O.round_bf16(A).astype(np.float64) if bf else A
        ref = (od.refine_into if up else od.conv)(os_, A, W.astype(np.float64), bias=bias.astype(np.float64), relu=True)
        if pre:
            res = None if up else dev(R[pd])
            got = gd.conv_preact(gs, dev(X[ps]), gW, groups=4, bias=_dev(bias), relu=True, refine=up, res=res)
            ref = ref if up else ref + R
        else:
            got = (gd.refine if up else gd.conv)(gs, dev(X[ps]), gW, bias=_dev(bias), relu=True)
        P.assert_close(P.rows_in_oracle_order(_host(got), pd), rnd(ref), tol, f"m={m} {cin}->{cout} {dtype} pre={pre} up={up}")


# bf16 convolution on both sides of the line of the 128 x 128 tiles (400 of them), with 0 to 3 stages behind their groups of
# four, a last stage that is not full and rows that do not fill a tile, against float64 products over the neighbour table
@pytest.mark.parametrize("pre", [False, True])
@pytest.mark.parametrize("m,cin,cout", [(3000, 264, 1024), (3000, 296, 1024), (3000, 328, 1024), (3000, 256, 1024),
                                        (3000, 296, 640)])
def test_conv_large_bf16_tiles(L, m, cin, cout, pre):  # noqa: F811
    gl = L.Lattice.create(_dev(_cloud(2350, m, 1.2)), [0.05] * 3)
    n = gl.n
    assert n % 128 and (-(-n // 128) * (cout // 128) >= 400) == (cout == 1024), n
    gen = torch.Generator("cuda").manual_seed(cin)
    X = torch.randn((n, cin), generator=gen, device="cuda").bfloat16()
    W = (torch.randn((9, cout, cin), generator=gen, device="cuda") / np.sqrt(9 * cin)).bfloat16()
    A = X.double()
    if pre:
        g = A.reshape(n, 4, cin // 4)
        mean = g.mean((0, 2), keepdim=True)
        g = (g - mean) / torch.sqrt(((g - mean) ** 2).mean((0, 2), keepdim=True) + 1e-5)
        A = torch.relu(g.reshape(n, cin)).bfloat16().double()
        got = gl.conv_preact(gl, X, W, groups=4, relu=True)
    else:
        got = gl.conv(gl, X, W, relu=True)
    nb = gl.neighbors().long()
    ref = sum((A[nb[:, t].clamp(min=0)] * (nb[:, t:t + 1] >= 0)) @ W[t].double().T for t in range(9))
    P.assert_close(_host(got), _host(torch.relu(ref)), P.TOL_BF16, f"{cin}->{cout} pre={pre}")


# DeformSlice + classifier: 16-point tiles of 1 to 64 lanes per row, 16-class blocks, wide rows, unaligned class counts; by
# lane groups on small clouds (32 or 64 classes kept, one or two chunks a lane) and with few bf16 classes on large ones
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,C,K", [(1, 8, 1), (15, 16, 17), (65, 40, 16), (257, 72, 5), (300, 136, 33), (100, 256, 64),
                                   (70, 264, 60), (33, 504, 32), (90, 64, 4), (91, 64, 5), (260, 72, 33), (261, 128, 40),
                                   (700, 40, 32), (15_001, 40, 32), (1701, 136, 50), (2001, 256, 40), (1801, 264, 60), (3700, 512, 7),
                                   (2002, 504, 32), (30_001, 104, 9), (100_000, 160, 12), (18_001, 200, 5), (9001, 192, 3)])
def test_classifier_tiles(L, O, m, C, K, dtype):  # noqa: F811
    gl, ol, g2o = _pair(L, O, _cloud(2400 + m, m, 0.6), 0.1)
    rng = np.random.default_rng(m)
    X = rng.normal(size=(ol.n, C))
    X = O.round_bf16(X) if dtype == "bf16" else X.astype(np.float32)
    wv = (rng.normal(size=C) / np.sqrt(C)).astype(np.float32)
    Wc = (rng.normal(size=(K, C)) / np.sqrt(C)).astype(np.float32)
    bc = rng.normal(size=K).astype(np.float32)
    ref = ol.deform_slice_classify(X.astype(np.float64), wv.astype(np.float64), 0.1, Wc.astype(np.float64),
                                   bc.astype(np.float64))
    x = _dev(np.asarray(X, np.float32)[g2o], torch.bfloat16 if dtype == "bf16" else None)
    got = gl.deform_slice_classify(x, _dev(wv), 0.1, _dev(Wc), _dev(bc))
    P.assert_close(_host(got), ref, P.TOL_F32, f"logits m={m} C={C} K={K} {dtype}")


# sums of many channels run in short chains: the error of the logits against float64 over that of DeformSlice's own rows
# classified in float64.  Measured 1.22, 1.50, 1.32 and 1.53; by lane groups, which sum in trees, 1.20, 1.46, 1.22 and 1.32;
# with the offsets of wide rows in one chain and runs added one by one 1.22, 1.55, 1.59 and 2.05.  The inputs are fixed, and
# the order of a sum moves a ratio by less than 0.02.
@pytest.mark.parametrize("C,bound", [(128, 1.25), (256, 1.53), (264, 1.4), (512, 1.65)])
def test_classifier_rounding_error(L, C, bound):  # noqa: F811
    gl = L.Lattice.create(_dev(_cloud(2460, 60_000, 1.0)), [0.05] * 3)
    idx, w = gl.simplices()
    gen = torch.Generator("cuda").manual_seed(C)
    x = torch.randn((gl.n, C), generator=gen, device="cuda")
    wv = torch.randn(C, generator=gen, device="cuda") / np.sqrt(C)
    Wc = torch.randn((20, C), generator=gen, device="cuda") / np.sqrt(C)
    got = gl.deform_slice_classify(x, wv, 0.1, Wc).double()
    own = gl.deform_slice(x, wv, 0.1)
    own = (own[0] if isinstance(own, tuple) else own).double() @ Wc.double().T
    rows, b = x.double()[idx.long()], w.double()[..., None]
    q = b * rows
    db = torch.tanh(0.1 + (q - q.max(1, keepdim=True).values) @ wv.double())
    ref = ((b + db[..., None]) * rows).sum(1) @ Wc.double().T
    assert float((got - ref).norm() / (own - ref).norm()) < bound


# infinite values in the last channels of a row that does not fill its lanes: the logits are infinite or NaN where the
# formula makes them so and nowhere else (tiled form, wide rows, lane groups)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,C,K", [(300, 24, 7), (300, 72, 7), (300, 72, 40), (300, 136, 7), (2100, 136, 40), (300, 264, 7),
                                   (2100, 264, 21)])
def test_classifier_infinite_values(L, O, m, C, K, dtype):  # noqa: F811
    gl, ol, g2o = _pair(L, O, _cloud(2450 + C, m, 0.6), 0.1)
    rng = np.random.default_rng(C)
    X = rng.normal(size=(ol.n, C))
    X = (O.round_bf16(X) if dtype == "bf16" else X).astype(np.float32)
    idx, _ = ol.simplices()
    X[idx[5, 0], C - 1] = -np.inf
    X[idx[17, 2], C - 3] = -np.inf
    X[idx[40, 1], C - 2] = np.inf
    wv = (rng.normal(size=C) / np.sqrt(C)).astype(np.float32)
    Wc = (rng.normal(size=(K, C)) / np.sqrt(C)).astype(np.float32)
    with np.errstate(invalid="ignore"):
        ref = ol.deform_slice_classify(X.astype(np.float64), wv.astype(np.float64), 0.1, Wc.astype(np.float64), None)
    got = _host(gl.deform_slice_classify(_dev(X[g2o], torch.bfloat16 if dtype == "bf16" else None), _dev(wv), 0.1, _dev(Wc)))
    assert np.isinf(ref).any(1).sum() > 2 and np.isfinite(ref).all(1).sum() > m // 2
    for kind in (np.isposinf, np.isneginf, np.isnan):
        assert np.array_equal(kind(got), kind(ref)), kind.__name__
    ok = np.isfinite(ref)
    P.assert_close(got[ok], ref[ok], P.TOL_F32, f"finite logits C={C} {dtype}")


# GroupNorm statistics and their backward: rows around the 32-row parts and 8-row batches, one to 16 row slots
@pytest.mark.parametrize("m,C,groups", [(2, 8, 2), (12, 64, 32), (40, 256, 32), (700, 128, 4), (1500, 1024, 32)])
def test_group_norm_parts(L, O, m, C, groups):  # noqa: F811
    gl, ol, g2o = _pair(L, O, _cloud(2500 + m, m, 0.7), 0.1)
    rng = np.random.default_rng(m)
    X = (rng.normal(size=(ol.n, C)) + rng.normal(size=C)).astype(np.float32)
    W = (rng.normal(size=(9, C, 8)) / np.sqrt(9 * C)).astype(np.float32)
    dY = rng.normal(size=(ol.n, 8)).astype(np.float32)
    A = O.groupnorm(X.astype(np.float64), groups, eps=1e-5, relu=True)
    gW = _dev(np.ascontiguousarray(np.transpose(W, (0, 2, 1))))
    got = gl.conv_preact(gl, _dev(X[g2o]), gW, groups=groups)
    P.assert_close(P.rows_in_oracle_order(_host(got), g2o), ol.conv(ol, A, W.astype(np.float64)), P.TOL_F32, f"m={m} C={C}")
    odA, _, _ = ol.conv_backward(ol, A, W.astype(np.float64), dY.astype(np.float64))
    odX, odg, odb = O.groupnorm_backward(X.astype(np.float64), odA, groups, eps=1e-5, relu=True)
    gdX, _, _, gdg, gdb = gl.conv_preact_backward(gl, _dev(X[g2o]), gW, _dev(dY[g2o]), groups=groups)
    P.assert_close(P.rows_in_oracle_order(_host(gdX), g2o), odX, P.TOL_F32, f"dX m={m} C={C}")
    P.assert_close(_host(gdg), odg, P.TOL_F32, f"dgamma m={m} C={C}")
    P.assert_close(_host(gdb), odb, P.TOL_F32, f"dbeta m={m} C={C}")


# bf16 GroupNorm statistics at widths whose bf16 rows split into more parts than fp32 rows (33 rows a part against 35)
@pytest.mark.parametrize("m,C,groups", [(14, 176, 8), (60, 176, 4), (60, 184, 8), (700, 184, 4), (60, 136, 8)])
def test_group_norm_bf16_parts(L, O, m, C, groups):  # noqa: F811
    gl, ol, g2o = _pair(L, O, _cloud(2550 + m, m, 0.7), 0.1)
    rng = np.random.default_rng(m + C)
    X = O.round_bf16(rng.normal(size=(ol.n, C)) + rng.normal(size=C))
    W = O.round_bf16(rng.normal(size=(9, C, 24)) / np.sqrt(9 * C))
    A = O.round_bf16(O.groupnorm(X.astype(np.float64), groups, eps=1e-5, relu=True)).astype(np.float64)
    gW = _dev(np.ascontiguousarray(np.transpose(np.asarray(W, np.float32), (0, 2, 1))), torch.bfloat16)
    got = gl.conv_preact(gl, _dev(np.asarray(X, np.float32)[g2o], torch.bfloat16), gW, groups=groups)
    P.assert_close(P.rows_in_oracle_order(_host(got), g2o), O.round_bf16(ol.conv(ol, A, W.astype(np.float64))), P.TOL_BF16,
                   f"m={m} C={C}")


# first table by the cloud's size: worst case up to 16,384 points, half of it up to 65,536, then 2 slots per point, where a
# sparse cloud overflows and is rebuilt (also when another stream asks first, and through coarse levels built before that)
@pytest.mark.parametrize("m,sigma", [(16_384, 0.002), (16_385, 0.002), (65_536, 0.002), (70_000, 0.001)])
@pytest.mark.parametrize("hierarchy", [True, False])
def test_first_table_sizes(L, O, m, sigma, hierarchy):  # noqa: F811
    pos = _cloud(2600, m, 1.0)
    ols = [O.Lattice.create(pos, np.full(3, sigma, np.float32))]
    ols.append(ols[0].coarsen())
    assert ols[0].n > 3.5 * m
    F = np.random.default_rng(m).normal(size=(m, 4)).astype(np.float32)
    pd, Fd = _dev(pos), _dev(F)
    torch.cuda.synchronize()
    if hierarchy:
        gls = L.Lattice.create_hierarchy(pd, [sigma] * 3, 2)
    else:
        gls = [L.Lattice.create(pd, [sigma] * 3)]
        gls.append(gls[0].coarsen())
    with torch.cuda.stream(torch.cuda.Stream()):
        got = gls[0].splat(Fd)
    torch.cuda.synchronize()
    g2o = [_check_structure(g, o) for g, o in zip(gls, ols)]
    P.assert_close(P.rows_in_oracle_order(_host(got), g2o[0]), ols[0].splat(F)[0], P.TOL_F32, "splat")
    _check_down_up(np.random.default_rng(m), g2o, gls, ols)
    for g in reversed(gls):
        g.destroy()


# up to 16,384 points no level of a hierarchy overflows, however sparse the cloud: the tables are built once, as for a dense one
@pytest.mark.parametrize("m", [1, 500, 3000, 16_384])
def test_small_hierarchies_are_built_once(L, m):  # noqa: F811
    pos = _dev(_cloud(2603, m, 1.0))
    launches = []
    L.timing_enable("nbr")
    for sigma in (0.5, 0.001):
        L.timing_read("nbr")   # (reading clears)
        gls = L.Lattice.create_hierarchy(pos, [sigma] * 3, 3)
        assert sigma > 0.1 or [g.n for g in gls][0] > 3.9 * m
        torch.cuda.synchronize()
        launches.append(L.timing_read("nbr")[0])
        for g in reversed(gls):
            g.destroy()
    L.timing_enable("nbr", False)
    assert launches[0] == launches[1] > 0


# a table that overflows is rebuilt at once: no convolution tables are looked up in a full one, where every absent key walks
# all slots (three levels of this cloud took 11 s in all that way, and take 8 ms)
def test_overflow_takes_no_lookups_in_a_full_table(L):
    pos = _dev(_cloud(2602, 70_000, 1.0))
    L.Lattice.create_hierarchy(pos, [0.5] * 3, 3)[2].n
    torch.cuda.synchronize()
    start = time.perf_counter()
    gls = L.Lattice.create_hierarchy(pos, [0.001] * 3, 3)
    assert [g.n > 262_144 for g in gls] == [True] * 3
    torch.cuda.synchronize()
    assert time.perf_counter() - start < 2.0
    for g in reversed(gls):
        g.destroy()


# a table hinted to lattice_create is not rebuilt: it may fill up, however long the probe sequences get
def test_hinted_table_nearly_full(L, O):  # noqa: F811
    pos = _cloud(2601, 2040, 1.0)
    ol = O.Lattice.create(pos, np.full(3, 0.002, np.float32))
    assert 0.98 * 8192 < ol.n <= 8192
    gl = L.Lattice.create(_dev(pos), [0.002] * 3, capacity_hint=4096)
    _check_structure(gl, ol)
    gl.destroy()


# slice: lane groups up to 128 channels and on small clouds; a wave per point with 4 channels a lane on rows beyond 128
# channels and with 2 on large clouds of 65 to 128 bf16 channels, several passes over a row
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,C", [(1, 8), (3, 64), (5, 72), (258, 128), (259, 136), (1023, 264), (77, 1032), (4096, 136),
                                 (4097, 136), (4099, 264), (4101, 1032), (131_073, 72), (131_079, 128)])
def test_slice_tiles(L, O, m, C, dtype):  # noqa: F811
    gl, ol, g2o = _pair(L, O, _cloud(2700 + m, m, 0.6), 0.1)
    X = np.random.default_rng(m).normal(size=(ol.n, C))
    X = O.round_bf16(X) if dtype == "bf16" else X.astype(np.float32)
    got = gl.slice(_dev(np.asarray(X, np.float32)[g2o], torch.bfloat16 if dtype == "bf16" else None))
    P.assert_close(_host(got), ol.slice(X.astype(np.float64)), P.TOL_F32, f"m={m} C={C} {dtype}")


# gradient of a normalised splat: 1 / (weight sum), given or summed, folded into the slice's weights; lane groups and wave form
@pytest.mark.parametrize("given", [True, False])
@pytest.mark.parametrize("m,C", [(1, 4), (3, 8), (17, 16), (65, 64), (258, 68), (259, 128), (515, 132), (77, 516),
                                 (4097, 132), (4099, 516)])
def test_splat_backward_scales(L, O, m, C, given):  # noqa: F811
    gl, ol, g2o = _pair(L, O, _cloud(2800 + m, m, 0.6), 0.1)
    dX = np.random.default_rng(m + C).normal(size=(ol.n, C)).astype(np.float32)
    ws = None
    if given:
        ws = torch.empty(gl.n, device="cuda")
        gl.splat(_dev(np.ones((m, 4), np.float32)), normalize=True, wsum=ws)
    got = gl.splat_backward(_dev(dX[g2o]), normalize=True, wsum=ws)
    P.assert_close(_host(got), ol.splat_backward(dX.astype(np.float64), normalize=True), P.TOL_F32, f"m={m} C={C}")

"""Kernels at the sizes where their tiling can go wrong (tile edges,
remainders, the smallest and largest of a dispatch range), against the
oracle.  The tolerances are those of the parity tests."""
from __future__ import annotations

import numpy as np
import pytest

from tests import parity as P
from tests.test_gpu_parity import L, O, _cloud, _dev, _host, _pair  # noqa: F401

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

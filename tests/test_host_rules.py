"""Host-side rules of the library that decide buffer sizes, checked without a
GPU through the library's internal functions."""
from __future__ import annotations

import ctypes as C
import os

import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_1912_05905_amd import lattice
    if not os.path.exists(lattice.LIB_PATH):
        pytest.fail("liblattice.so is not built (run __graft_entry__.build())")
    return lattice.lib()


def _internal(lib, symbol, *args):
    fn = getattr(lib, symbol)
    fn.restype, fn.argtypes = C.c_int64, list(args)
    return fn


@pytest.mark.parametrize("bf16", [0, 1])
def test_group_norm_partials_fit_their_workspace(lib, bf16):
    """Every width and row count around the points where the split changes: the partials that a launch of this dtype
    writes (2 C doubles each) fit the workspace that its caller allocates."""
    parts = _internal(lib, "_ZN3lat11gn_partialsElii", C.c_int64, C.c_int, C.c_int)
    size = _internal(lib, "_ZN3lat18gn_workspace_bytesElii", C.c_int64, C.c_int, C.c_int)
    for c in range(8 if bf16 else 4, 1025, 8 if bf16 else 4):
        last = 0
        for base in [*range(1, 400), *range(400, 300_000, 2048)]:
            for n in (base - 1, base, base + 1):
                p = parts(n, c, bf16)
                assert p * 2 * c * 8 <= size(n, c, bf16), f"n={n} C={c}: {p} partials"
                last = max(last, p)
        assert 1 < last <= 2048


@pytest.mark.parametrize("bf16", [0, 1])
def test_group_norm_partials_of_middle_levels(lib, bf16):
    """Up to 65,536 rows a level has at most 512 partials (the finalize reads them all in one workgroup per group), beyond
    that parts of at least 128 rows until there are 2,048 of them."""
    parts = _internal(lib, "_ZN3lat11gn_partialsElii", C.c_int64, C.c_int, C.c_int)
    for c in range(8, 1025, 8):
        for n in (1, 31, 33, 5_000, 16_384, 16_385, 22_743, 52_353, 65_536):
            assert parts(n, c, bf16) <= min(512, -(-n // 32)), (n, c)
        for n in (65_537, 100_000, 262_144):
            assert parts(n, c, bf16) <= -(-n // 128), (n, c)
        assert parts(1_000_000, c, bf16) <= 2048


def test_weight_gradient_chunks(lib):
    """Partials of the weight gradient: one set of 9 Cout Cin + Cout sums per vertex chunk.  Small levels have chunks of at
    least 64 vertices, from three 64 x 64 tiles on of 256 beyond 8 chunks, large ones three workgroups per compute unit."""
    floats = _internal(lib, "_ZN3lat20wgrad_partial_floatsElii", C.c_int64, C.c_int, C.c_int)
    assert floats(0, 64, 64) == 0
    for n in (1, 63, 64, 65, 1284, 2048, 3102, 8445, 200_000, 4_000_000):
        for cout, cin in ((4, 4), (64, 64), (72, 40), (192, 64), (128, 128), (256, 256), (512, 512), (1024, 1024)):
            tiles = -(-cout // 64) * -(-cin // 64)
            per = 9 * cout * cin + cout
            chunks, rest = divmod(floats(n, cout, cin), per)
            assert rest == 0 and 1 <= chunks <= max(1, -(-n // 64)), (n, cout, cin)
            assert chunks <= max(8, 768 // (9 * tiles) + 8)
            if tiles >= 3:
                assert chunks <= max(8, -(-n // 256)), (n, cout, cin, chunks)

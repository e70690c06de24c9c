"""Which kernel a matrix product of some sizes runs on, asked of the library without a GPU: the sizes of the GPU tests still reach the
tiles they are there for, and no product is sent to a tile that is not built for it. For 256 compute units, which the library
takes where there is no device to ask."""
import ctypes
import random

import pytest

pytest.importorskip("torch")
import test_gpu_blast_chunks as chunks
import test_gpu_chain_members as chain_members
import test_gpu_gemm_tiles as tiles
import test_gpu_nonfinite as nonfinite
import test_gpu_parity as parity
import test_gpu_silu_gate as gate
import test_gpu_tile_walk as walk
from paper_2512_20861_amd import binding as B

INTERLEAVED, WINDOWS, EIGHT_BIT = 1, 2, 4
_text = ctypes.create_string_buffer(256)


def status(M, N, K, G=1, run=0, form=0, members=1, size=256):
    f = B.lib().blr_product_tiles
    f.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 4 + [ctypes.c_uint, ctypes.c_int, ctypes.c_char_p, ctypes.c_size_t]
    return f(M, N, K, G, run, form, members, _text, size)


def kernels(*args, **kw):
    assert status(*args, **kw) == B.OK
    return _text.value.decode()


def cases(table):
    return [(name, row) for name, sizes in table.items() for row in sizes]


@pytest.mark.parametrize("name,row", cases(tiles.DENSE) + cases(parity.DENSE_LARGE) + cases(parity.DENSE_SMALL))
def test_dense_rows(name, row):
    T, n_in, n_out = row
    assert kernels(T, n_out, n_in) == name


@pytest.mark.parametrize("name,row", cases(tiles.MONARCH))
def test_monarch_rows(name, row):
    T, b, p, rp, q = row
    for form in (0, INTERLEAVED):
        assert kernels(T, q, b * rp, b, form=form) == name


@pytest.mark.parametrize("name,row", [(n, (T, q, b, r)) for n, (T, q, p, b, r) in cases(chunks.STAGE1)] + cases(nonfinite.WINDOWS))
def test_rows_of_input_windows(name, row):
    T, q, b, r = row
    assert kernels(T, r, q, b, form=WINDOWS) == name


@pytest.mark.parametrize("name,row", cases(walk.SHORT_RUNS))
def test_rows_of_short_runs(name, row):
    b, T, p = row
    rp = walk.short_run(b)
    assert kernels(T, b * rp, p, b, run=rp) == name


def test_combined_members():
    for name, T in gate.TILES.items():
        assert kernels(T, gate.MLP // gate.NB, gate.R, gate.NB, members=2) == name
    forms = ["64x64 w4 k64x4 i32", "128x64 w8 k64x4 i32", "128x128 w8 k64x4 i32", "128x128 w8 k64x4 i16", "128x128 w4 k64x2 i32"]
    for members, products in ((3, ((512, 512, 4), (128, 256, 16))), (2, ((2048, 512, 4), (512, 512, 16), (504, 256, 15)))):
        for N, K, G in products:                         # of the chains of 2048 / 8192 and 1920 / 7560
            assert {f"{members} of {form}" for form in forms} <= {kernels(T, N, K, G, members=members) for T in chain_members.TOKENS}


def test_pairs_of_matrix_instructions():
    pair = lambda call, full, other: [call(T) for T in (full, other)]
    for name, (n_in, n_out, *Ts) in cases(tiles.DENSE_PAIRS):
        edge = " partial" if n_in % 64 else ""
        assert pair(lambda T: kernels(T, n_out, n_in), *Ts) == [name + " i16" + edge, name + " i32" + edge]
    for name, (b, rp, q, *Ts) in cases(tiles.MONARCH_PAIRS):
        assert pair(lambda T: kernels(T, q, b * rp, b, form=INTERLEAVED), *Ts) == [name + " i16", name + " i32"]
    combined = "%d of 128x128 w8 k64x4 i%d"
    assert pair(lambda T: kernels(T, 512, 512, 4, members=3), 1800, 1750) == [combined % (3, 16), combined % (3, 32)]
    assert pair(lambda T: kernels(T, 2048, 512, 4, members=2), 400, 370) == [combined % (2, 16), combined % (2, 32)]
    assert pair(lambda T: kernels(T, 512, 512, 16, members=2), 400, 370) == [combined % (2, 16), combined % (2, 32)]


def test_every_product_has_a_kernel():
    rng = random.Random(3)
    size = lambda lo, hi: int(round(2 ** rng.uniform(lo, hi)))
    for _ in range(20000):
        G, M, N, K = rng.choice((1, 1, 2, 3, 4, 6, 8, 9, 12, 15, 16, 24, 48)), size(0, 14), size(0, 13), size(0, 13)
        if rng.random() < 0.8:
            K = 8 * -(-K // 8)
        form, run, members = rng.choice((0, INTERLEAVED, WINDOWS, EIGHT_BIT, WINDOWS | EIGHT_BIT)), 0, 1
        if form & WINDOWS and (G * K) % 64:
            K = 64 * -(-K // 64) + 8 * rng.randrange(8) if G % 8 == 0 else 64 * -(-K // 64)
        if form & EIGHT_BIT:
            K, N = 8 * -(-K // 8), 16 * -(-N // 16)
        if form == 0 and rng.random() < 0.3:
            run = rng.choice((1, 3, 4, 12, 48, 256))
            N = run * -(-N // run)
        elif form == 0 and rng.random() < 0.4:
            members = rng.choice((2, 3))
        assert status(M, N, K, G, run, form, members) == B.OK, (M, N, K, G, run, form, members)


def test_refusals():
    for bad in (dict(M=0), dict(N=0), dict(K=0), dict(G=0), dict(run=3), dict(form=8), dict(members=4), dict(members=0), dict(size=0)):
        assert status(**(dict(M=100, N=128, K=64) | bad)) == B.ERR_INVALID_ARG, bad
    assert status(4095, 2296, 192, size=20) == B.ERR_WORKSPACE and status(4095, 2296, 192, size=21) == B.OK
    assert kernels(64, 64, 30) == "portable"

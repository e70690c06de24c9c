"""Tiles of the bf16 products that the dispatch picks by estimate for several rounds of workgroups (128 x 192, 192 x 128 and
128 x 128, two workgroups per compute unit) and the eight-wavefront tiles of a single round (by their padded area where
128 x 128 tiles would be more than one), each with a ragged last tile
in rows and columns, contiguous and interleaved outputs, odd and even numbers of steps, a partial last step; and that the two
matrix instructions these tiles run on give the same bits."""
import numpy as np
import pytest

import blr_inputs as bi
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# kernel (tile, wavefronts, step x stages, rows of the matrix instruction, kind of last step) -> sizes it is chosen for; test_tile_rules.py
# checks that it still is. T, n_in, n_out:
DENSE = {
    "192x128 w4 k64x2 i32": [(4095, 192, 2296), (3334, 192, 2308)],
    "256x256 w8 k64x2 i32": [(4095, 192, 3068)],
    "128x128 w4 k64x2 i32": [(3073, 128, 3085), (1158, 128, 1932), (1817, 192, 4108)],        # (columns that end off a 16-byte boundary)
    "128x128 w4 k64x2 i32 partial": [(1718, 136, 1414)],
    "128x256 w8 k64x3 i32": [(520, 256, 11000), (640, 512, 8189), (800, 320, 8188)],
    "128x256 w8 k64x3 i16": [(600, 256, 13050)],
    "192x128 w8 k64x3 i32": [(1100, 320, 4600), (1300, 640, 4092)],
    "192x128 w8 k64x3 i16": [(300, 512, 16380)],
    "128x192 w8 k64x3 i32": [(2047, 192, 2300)],
    "128x192 w8 k64x3 i16": [(600, 320, 9790)],
    "256x128 w8 k64x3 i32": [(2500, 192, 1936)],
    "256x128 w8 k64x3 i32 partial": [(1811, 136, 2437)],
    "256x128 w8 k64x3 i16": [(2040, 320, 4090)],
    "256x128 w8 k64x3 i16 partial": [(2564, 136, 2731)],
    "128x128 w8 k64x4 i32": [(1500, 192, 2299), (1100, 1344, 2044), (1000, 1280, 2050)],      # (three steps on four stages; half of the chip)
    "128x128 w8 k64x4 i32 partial": [(1500, 200, 2300)],
    "128x128 w8 k64x4 i16": [(1999, 1280, 2044), (2001, 192, 2044)],
    "128x128 w8 k64x4 i16 partial": [(1999, 1288, 2041), (2001, 328, 2044), (300, 264, 10500)],
    "128x128 w4 k64x4 i32": [(1000, 640, 4044)],                                              # a full chip, up to 1024 tokens
    "128x128 w4 k64x4 i32 partial": [(1020, 520, 4090)],
    "128x64 w8 k64x4 i32": [(1000, 1280, 2042), (1300, 192, 1148)],
    "128x64 w8 k64x4 i32 partial": [(300, 1000, 4090)],
    "128x64 w8 k128x3 i32 partial": [(1000, 1416, 2044), (300, 1480, 4090)],
    "128x64 w4 k64x2 i32": [(1029, 128, 1090)],
    "128x64 w4 k64x2 i32 partial": [(1026, 136, 1092)],
    "64x128 w8 k64x4 i32 partial": [(2529, 264, 389)],
    "64x128 w8 k128x3 i32 partial": [(2529, 1288, 389)],
    "64x128 w4 k64x2 i32": [(962, 128, 1166)],
    "64x128 w4 k64x2 i32 partial": [(1123, 136, 1042)],
    "64x64 w4 k64x2 i32": [(658, 128, 715)],
    "64x64 w4 k128x4 i32": [(797, 256, 589)],
    "64x64 w4 k128x4 i32 partial": [(598, 264, 806)],
}
# second products of Monarch layers on two kernels, either order of the output. T, b, p, rp, q:
MONARCH = {
    "192x128 w4 k64x2 i32": [(2076, 16, 64, 12, 132), (4111, 4, 64, 48, 388)],
    "128x192 w4 k64x2 i32": [(1743, 16, 64, 12, 516), (4037, 4, 64, 48, 1028)],
    "128x128 w4 k64x2 i32": [(1153, 16, 64, 12, 380), (387, 4, 64, 32, 1171), (1409, 4, 64, 32, 1530), (1153, 16, 64, 8, 572), (2047, 4, 64, 32, 1532)],
    "256x256 w8 k64x2 i32": [(4095, 4, 64, 48, 572)],
    "128x64 w4 k128x3 i32 partial": [(400, 16, 64, 66, 250)],
    "128x64 w8 k64x4 i32": [(300, 16, 64, 64, 250)],
    "192x128 w8 k64x3 i32": [(1300, 4, 64, 48, 1020)],
    "192x128 w8 k64x3 i16": [(265, 8, 64, 24, 1916)],
    "128x192 w8 k64x3 i32": [(1560, 12, 64, 16, 142)],
    "128x192 w8 k64x3 i16": [(393, 12, 64, 16, 936)],
    "128x256 w8 k64x3 i32": [(633, 16, 64, 12, 508), (780, 4, 64, 64, 2036), (804, 4, 64, 48, 1226)],
    "128x256 w8 k64x3 i16": [(577, 4, 64, 64, 3068)],
    "256x128 w8 k64x3 i32": [(391, 4, 64, 48, 2786)],
    "256x128 w8 k64x3 i16": [(1357, 8, 64, 24, 542)],
    "256x128 w8 k64x3 i16 partial": [(265, 8, 64, 20, 1839)],
    "128x128 w8 k64x4 i16": [(261, 4, 64, 48, 2606)],
}
# A nearly full round and an emptier one of the same tile: 16 x 16 x 32 matrix instructions and 32 x 32 x 16. kernel without the
# instruction -> sizes, T of the full round, T of the other
DENSE_PAIRS = {                                       # n_in, n_out
    "128x128 w8 k64x4": [(192, 2945, 1161, 1108), (1096, 2044, 2001, 1700)],
    "192x128 w8 k64x3": [(192, 2945, 1797, 1691)],
    "128x192 w8 k64x3": [(192, 2433, 2327, 2168)],
    "256x128 w8 k64x3": [(192, 2689, 2592, 2539), (200, 2953, 2327, 2274)],
}
MONARCH_PAIRS = {                                     # b, rp, q
    "128x128 w8 k64x4": [(8, 24, 146, 1797, 1744)],
    "192x128 w8 k64x3": [(8, 24, 258, 1797, 1691)],
    "128x192 w8 k64x3": [(16, 12, 162, 1797, 1744)],
    "128x256 w8 k64x3": [(8, 24, 402, 1797, 1638)],
    "256x128 w8 k64x3": [(16, 12, 590, 578, 472)],
}


def rows(table):
    return [row for sizes in table.values() for row in sizes]


@pytest.mark.parametrize("T,n_in,n_out", rows(DENSE))
def test_dense_tiles(T, n_in, n_out):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    W, X = bi.dense_weight(n_in, n_out, "bf16"), bi.activations(T, n_in, "bf16")
    Y = gu.empty_out(T, n_out, "bf16")
    gu.B.dense_reference_forward(gu.to_dev(X), gu.to_dev(W), Y, 0)
    torch.cuda.synchronize()
    assert gu.rel_err(gu.to_f64(Y), oracle.dense_forward(X.f64, W.f64)) <= gu.TOL["bf16"]


@pytest.mark.parametrize("T,b,p,rp,q", rows(MONARCH))
@pytest.mark.parametrize("order", ["interleaved", "blocked"])
def test_monarch_tiles(T, b, p, rp, q, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    R = bi.gaussian(bi.BASE_SEED, 51, (b, rp * b, p), 1.0 / np.sqrt(p), "bf16")
    L = bi.gaussian(bi.BASE_SEED, 52, (b, q, b * rp), 1.0 / np.sqrt(b * rp), "bf16")
    X = bi.activations(T, b * p, "bf16")
    blocked = order == "blocked"
    Yref = oracle.monarch_rect_forward(X.f64, R.f64, L.f64, b, b, oracle.OUT_BLOCKED if blocked else oracle.OUT_INTERLEAVED)
    # (most of these layers are narrow enough for the single kernel, which is what a call without the flag runs)
    for flag in (B.MONARCH_TWO_KERNELS, 0):
        Y = gu.empty_out(T, b * q, "bf16")
        B.monarch_rect_forward(gu.to_dev(X), gu.to_dev(R), gu.to_dev(L), Y, b, b, rp, flag | (B.MONARCH_OUT_BLOCKED if blocked else 0))
        torch.cuda.synchronize()
        assert gu.rel_err(gu.to_f64(Y), Yref) <= gu.TOL["bf16"]


def _wide_range(shape, seed):
    """bf16 numbers of every size between 2^-40 and 2^40, in either sign: sums whose terms cancel, vanish and round."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(shape, generator=g, device="cuda") * torch.exp2(torch.randint(-40, 41, shape, generator=g, device="cuda").float())).bfloat16()


@pytest.mark.parametrize("draw", ["normal", "wide"])
@pytest.mark.parametrize("n_in,n_out,full,other", rows(DENSE_PAIRS))
def test_equal_bits_dense(n_in, n_out, full, other, draw):
    """The matrix instruction depends on the number of tokens: rows of a call have the bits they have in a shorter one."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    X, W = (_wide_range(s, n_in + i) if draw == "wide" else torch.randn(s, device="cuda").bfloat16() for i, s in enumerate(((full, n_in), (n_out, n_in))))
    call = lambda x: gu.B.dense_reference_forward(x, W, gu.empty_out(x.shape[0], n_out, "bf16"), 0)
    Y, part = call(X), call(X[:other])
    assert bool(torch.isfinite(Y).all()) and torch.equal(Y[:other], part)


@pytest.mark.parametrize("b,rp,q,full,other", rows(MONARCH_PAIRS))
def test_equal_bits_monarch(b, rp, q, full, other):
    """The same for an interleaved output; both calls with the first call's intermediate."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    g = torch.Generator(device="cuda").manual_seed(q)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    X, R, L = rand(full, b * 64), rand(b, rp * b, 64), rand(b, q, b * rp)
    ws = torch.empty(B.monarch_rect_workspace_bytes(full, b * 64, b * q, b, b, rp, B.BF16), dtype=torch.uint8, device="cuda")
    Y = B.monarch_rect_forward(X, R, L, gu.empty_out(full, b * q, "bf16"), b, b, rp, B.MONARCH_TWO_KERNELS, workspace=ws)
    part = B.monarch_rect_forward(X[:other], R, L, gu.empty_out(other, b * q, "bf16"), b, b, rp, B.ONLY_LAST_STAGE, workspace=ws)
    assert bool(torch.isfinite(Y).all()) and torch.equal(Y[:other], part)


@pytest.mark.parametrize("op,params", [("monarch", dict(nblocks=4, r_square=512, r_mlp=512)), ("blast", dict(b=16, r_square=256, r_mlp=512))])
@pytest.mark.parametrize("full,other", [(1800, 1750), (400, 370)])      # the sum of q, k, v (Monarch); the SiLU gate
def test_equal_bits_of_combined_members(op, params, full, other):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_20861_amd.chain import DeviceChain
    layers = bi.chain_layers(op, n_layers=1, hidden=2048, mlp=8192, params=params, dtype="bf16")
    x = torch.randn(full, 2048, generator=torch.Generator(device="cuda").manual_seed(full), device="cuda").bfloat16()
    Y, part = (DeviceChain(layers, T).forward(x[:T]) for T in (full, other))
    assert bool(torch.isfinite(Y).all()) and torch.equal(Y[:other], part)

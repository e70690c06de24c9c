"""The 256 x 256 tiles of products with more tiles than compute units, several of which one workgroup computes one after the other:
odd and even numbers of steps, a partial last step, ragged last tiles, gathered weight rows, scattered and contiguous columns,
windows of input blocks, 8-bit outputs. All of the output is looked at for elements nobody wrote, sampled rows (the tiles'
first and last ones among them) are compared with the oracle, and all of it with the same layer on 128 tokens at a time, which
take other tiles."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def draw(gen, *shape, scale=1.0):
    return (torch.randn(*shape, generator=gen, device="cuda") * scale).bfloat16()


def sample(T):
    edges = [t for k in range(0, T, 256) for t in (k, k + 31, k + 255)]
    return np.unique([t for t in edges + [T // 3, T - 2, T - 1] if t < T])


def check(gu, Y, rows, ref):
    assert bool(torch.isfinite(Y).all()), "elements nobody wrote"
    assert gu.rel_err(gu.to_f64(Y[torch.from_numpy(rows).cuda()]), ref) <= gu.TOL["bf16"]


@pytest.mark.parametrize("T,n_in,n_out", [
    (4096, 4224, 7168),                               # whole tiles, an even number of steps
    (4000, 4160, 7096), (3841, 4160, 7100),           # odd, ragged; columns that end off a 16-byte boundary
    (4000, 4232, 7096), (4090, 4168, 6920),           # a partial last step
])
def test_dense(T, n_in, n_out):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    gen = torch.Generator(device="cuda").manual_seed(T + n_in)
    X, W = draw(gen, T, n_in), draw(gen, n_out, n_in, scale=n_in ** -0.5)
    Y = gu.empty_out(T, n_out, "bf16")
    gu.B.dense_reference_forward(X, W, Y, 0)
    rows = sample(T)
    check(gu, Y, rows, oracle.dense_forward(gu.to_f64(X)[rows], gu.to_f64(W)))


@pytest.mark.parametrize("order", ["interleaved", "blocked"])
@pytest.mark.parametrize("T,b,p,rp,q", [(4000, 2, 4160, 1776, 3600), (8200, 4, 256, 96, 2760)])
def test_monarch(T, b, p, rp, q, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    gen = torch.Generator(device="cuda").manual_seed(T + p)
    X, R, L = draw(gen, T, b * p), draw(gen, b, rp * b, p, scale=p ** -0.5), draw(gen, b, q, b * rp, scale=(b * rp) ** -0.5)
    Y = gu.empty_out(T, b * q, "bf16")
    blocked = order == "blocked"
    B.monarch_rect_forward(X, R, L, Y, b, b, rp, B.MONARCH_OUT_BLOCKED if blocked else 0)
    rows = sample(T)
    ref = oracle.monarch_rect_forward(gu.to_f64(X)[rows], gu.to_f64(R), gu.to_f64(L), b, b, oracle.OUT_BLOCKED if blocked else oracle.OUT_INTERLEAVED)
    check(gu, Y, rows, ref)


@pytest.mark.parametrize("T,q,r", [(3000, 600, 1024), (2900, 688, 1008), (3100, 576, 1024)])
@pytest.mark.parametrize("z8", [False, True])
def test_blast(T, q, r, z8):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    from oracle import quant
    B, b, p = gu.B, 16, 32
    gen = torch.Generator(device="cuda").manual_seed(T + q)
    X, U, S, V = draw(gen, T, b * q), draw(gen, b, p, r, scale=r ** -0.5), draw(gen, b, b, r, scale=r ** -0.5), draw(gen, b, q, r, scale=r ** -0.5)
    Y = gu.empty_out(T, b * p, "bf16")
    packed = B.blast_pack(U, S, V, b * q, b * p, b, r)
    B.blast_forward(X, U, None, packed, Y, b, r, B.BLAST_PACKED | (B.BLAST_Z_FP8 if z8 else B.BLAST_THREE_KERNELS))
    rows = sample(T)
    args = gu.to_f64(X)[rows], gu.to_f64(U), gu.to_f64(S), gu.to_f64(V)
    check(gu, Y, rows, quant.blast_forward_qz(*args)[0] if z8 else oracle.blast_forward(*args))


def agree(Y, part):
    """Every row, 64 columns at a time, with part(first token): the same result in other tiles. Both round the same sums to bf16 (and a
    few values of an intermediate, where the order of a sum moves them over a rounding edge): each is within 2^-9 of a value, so
    2^-6 of the 64's norm is four times what both can be apart; a part of another tile or step is apart by the norm itself."""
    for t in range(0, Y.shape[0], 128):
        got, want = Y[t:t + 128].float(), part(t).float()
        pad = -got.shape[1] % 64
        got, want = (torch.nn.functional.pad(v, (0, pad)).view(v.shape[0], -1, 64) for v in (got, want))
        bad = ~((got - want).norm(dim=2) <= 2 ** -6 * want.norm(dim=2))
        assert not bool(bad.any()), f"token, column: {[(t + int(i), 64 * int(j)) for i, j in bad.nonzero()[:8]]}"


@pytest.mark.parametrize("T,n_in,n_out", [(4096, 4224, 7168), (4000, 4160, 7096), (3841, 4160, 7100), (4090, 4168, 6920)])
def test_every_row_dense(T, n_in, n_out):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    gen = torch.Generator(device="cuda").manual_seed(T + n_in)
    X, W = draw(gen, T, n_in), draw(gen, n_out, n_in, scale=n_in ** -0.5)
    call = lambda x: gu.B.dense_reference_forward(x, W, gu.empty_out(x.shape[0], n_out, "bf16"), 0)
    agree(call(X), lambda t: call(X[t:t + 128].contiguous()))


@pytest.mark.parametrize("order", ["interleaved", "blocked"])
@pytest.mark.parametrize("T,b,p,rp,q", [(4000, 2, 4160, 1776, 3600), (8200, 4, 256, 96, 2760)])
def test_every_row_monarch(T, b, p, rp, q, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    gen = torch.Generator(device="cuda").manual_seed(T + p)
    X, R, L = draw(gen, T, b * p), draw(gen, b, rp * b, p, scale=p ** -0.5), draw(gen, b, q, b * rp, scale=(b * rp) ** -0.5)
    call = lambda x: B.monarch_rect_forward(x, R, L, gu.empty_out(x.shape[0], b * q, "bf16"), b, b, rp, B.MONARCH_OUT_BLOCKED if order == "blocked" else 0)
    agree(call(X), lambda t: call(X[t:t + 128].contiguous()))


def short_run(b):
    return max(160 // b, 3)


# kernels -> b, T, p. On the 256 x 256 tile alone, with more tiles than compute units: walked up to 16 batch entries, above that one tile
# to a workgroup. The others: one round of it, one round and the rows of the next on smaller tiles, and what the estimate takes in its place
SHORT_RUNS = {
    "256x256 w8 k64x2 i32 partial": [(16, 7000, 328), (17, 7000, 328), (24, 7000, 328), (24, 4100, 328)],
    "256x256 w8 k64x2 i32": [(16, 4096, 256), (16, 2570, 320), (17, 2570, 320)],
    "256x256 w8 k64x2 i32 + 128x128 w4 k64x2 i32": [(17, 4096, 256)],
    "256x256 w8 k64x2 i32 partial + 128x128 w4 k64x2 i32 partial": [(16, 4100, 328), (17, 4100, 328), (48, 4100, 328), (48, 7000, 328)],
    "128x192 w4 k64x2 i32": [(24, 4096, 256), (24, 2570, 320), (48, 4096, 256), (48, 2570, 320)],
}


@pytest.mark.parametrize("b,T,p", [row for sizes in SHORT_RUNS.values() for row in sizes])
def test_every_row_short_runs(T, b, p):
    """First products whose columns go out in runs of a few elements, b the number of batch entries."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B, rp, q = gu.B, short_run(b), 64
    gen = torch.Generator(device="cuda").manual_seed(T + b)
    X, R, L = draw(gen, T, b * p), draw(gen, b, rp * b, p, scale=p ** -0.5), draw(gen, b, q, b * rp, scale=(b * rp) ** -0.5)
    call = lambda x: B.monarch_rect_forward(x, R, L, gu.empty_out(x.shape[0], b * q, "bf16"), b, b, rp, B.MONARCH_OUT_BLOCKED)
    Y, rows = call(X), sample(T)
    check(gu, Y, rows, oracle.monarch_rect_forward(gu.to_f64(X)[rows], gu.to_f64(R), gu.to_f64(L), b, b, oracle.OUT_BLOCKED))
    agree(Y, lambda t: call(X[t:t + 128].contiguous()))


@pytest.mark.parametrize("T,q,r", [(3000, 600, 1024), (2900, 688, 1008), (3100, 576, 1024)])
def test_every_row_blast(T, q, r):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B, b, p = gu.B, 16, 32
    gen = torch.Generator(device="cuda").manual_seed(T + q)
    X, U, S, V = draw(gen, T, b * q), draw(gen, b, p, r, scale=r ** -0.5), draw(gen, b, b, r, scale=r ** -0.5), draw(gen, b, q, r, scale=q ** -0.5)
    packed = B.blast_pack(U, S, V, b * q, b * p, b, r)
    call = lambda x: B.blast_forward(x, U, None, packed, gu.empty_out(x.shape[0], b * p, "bf16"), b, r, B.BLAST_PACKED | B.BLAST_THREE_KERNELS)
    agree(call(X), lambda t: call(X[t:t + 128].contiguous()))


def test_segments():
    """A first product whose input blocks are runs of the blocked order: 448 tiles, 66 steps in two runs each."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B, T, b, p, rp, q = gu.B, 4000, 2, 4224, 1776, 256
    gen = torch.Generator(device="cuda").manual_seed(p)
    X, R, L = draw(gen, T, b * p), draw(gen, b, rp * b, p, scale=p ** -0.5), draw(gen, b, q, b * rp, scale=(b * rp) ** -0.5)
    runs = X.view(T, p, b).transpose(1, 2).reshape(T, b * p)                     # feature j b + k at k p + j
    Y = B.monarch_forward(runs, B.monarch_permute_first_factor(R, b * p, b, b * rp), L, gu.empty_out(T, b * q, "bf16"), b, b * rp, B.MONARCH_IN_BLOCKED)
    call = lambda x: B.monarch_forward(x, R, L, gu.empty_out(x.shape[0], b * q, "bf16"), b, b * rp, 0)
    agree(Y, lambda t: call(X[t:t + 128].contiguous()))
    rows = sample(T)
    check(gu, Y, rows, oracle.monarch_forward(gu.to_f64(X)[rows], gu.to_f64(R), gu.to_f64(L)))


@pytest.mark.parametrize("T,q,r", [(3000, 600, 1024), (2900, 688, 1008)])
def test_neighbours_infinities(T, q, r):
    """Windows of input blocks, three tiles to a workgroup: an infinity in the first or the last column of every block, which a
    neighbour's window holds too, on tokens of the first, the middle and the last tiles. All factors are positive: a row with
    an infinity is infinite everywhere (a neighbour's, times the zeros it meets there, would make it NaN), the others are finite."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B, b, p = gu.B, 16, 32
    gen = torch.Generator(device="cuda").manual_seed(q)
    make = lambda scale, *s: ((0.5 + 0.5 * torch.rand(*s, generator=gen, device="cuda")) * scale).bfloat16()
    X, U, S, V = make(1, T, b * q), make(1 / r, b, p, r), make(1 / b, b, b, r), make(1 / q, b, q, r)
    packed = B.blast_pack(U, S, V, b * q, b * p, b, r)
    call = lambda x: B.blast_forward(x, U, None, packed, gu.empty_out(x.shape[0], b * p, "bf16"), b, r, B.BLAST_PACKED | B.BLAST_THREE_KERNELS)
    whole = call(X)
    bad = torch.zeros(T, dtype=torch.bool, device="cuda")
    for first in (5, T // 2, T - 40):
        for j in range(b):
            for k, c in enumerate((j * q, (j + 1) * q - 1)):
                X[first + 2 * j + k, c] = float("inf")
                bad[first + 2 * j + k] = True
    Y = call(X)
    torch.cuda.synchronize()
    assert bool((Y[bad] == float("inf")).all()) and torch.equal(Y[~bad], whole[~bad])

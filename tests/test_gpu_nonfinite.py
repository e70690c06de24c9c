"""Infinities and NaN keep to the outputs that depend on them: what a kernel reads past its range (the end of a contraction
index, an absent block, a neighbour's columns) meets a zero there, and an infinity times zero would be NaN. All factors
are positive, so that an infinity in an input is an infinity, not NaN, in every output it reaches."""
import numpy as np
import pytest

import blr_inputs as bi
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _agree(got, ref, tol):
    """The same infinities and NaN, and finite values within the repository's bound of the largest of them."""
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    ok = np.isfinite(ref)
    assert ok.any() and not ok.all() and np.abs(got[ok] - ref[ok]).max() <= tol * np.abs(ref[ok]).max()


@pytest.mark.parametrize("T,p,q,b1,b2,rp", [(3, 68, 24, 2, 2, 20), (17, 4, 16, 1, 3, 4), (5, 132, 100, 3, 5, 12), (8, 64, 64, 4, 4, 16)])
def test_fp32_monarch(T, p, q, b1, b2, rp):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    n_in, n_out = b1 * p, b2 * q
    rng = np.random.default_rng(T + p)
    R, L, X = (rng.uniform(0.5, 1.0, s).astype(np.float32) for s in ((b1, rp * b2, p), (b2, q, b1 * rp), (T, n_in)))
    X[0, n_in - 1] = np.inf                              # in the last four of a block
    X[T // 2, p - 4] = np.nan
    R[b1 - 1, (rp - 1) * b2] = 2e38                      # the last of the intermediate of output block 0 overflows, with finite inputs
    Y = gu.empty_out(T, n_out, "f32")
    gu.B.monarch_rect_forward(*(torch.from_numpy(t).cuda() for t in (X, R, L)), Y, b1, b2, rp, 0)
    torch.cuda.synchronize()
    Z = np.zeros((T, b2, b1 * rp), np.float32)           # the intermediate as fp32 holds it, then fp64 again
    with np.errstate(all="ignore"):
        for l in range(b1):
            z = X[:, l * p:(l + 1) * p].astype(np.float64) @ R[l].astype(np.float64).T
            Z[:, :, l * rp:(l + 1) * rp] = z.astype(np.float32).reshape(T, rp, b2).transpose(0, 2, 1)
        ref = np.stack([Z[:, k].astype(np.float64) @ L[k].astype(np.float64).T for k in range(b2)], axis=2).reshape(T, n_out)
    _agree(gu.to_f64(Y), ref, gu.TOL["f32"])


def _blast(T, q, p, b, r, bad, flags):
    """bad: (token, column) of an infinity in X"""
    import gpu_util as gu
    rng = np.random.default_rng(q + r)
    make = lambda scale, *s: torch.from_numpy((rng.uniform(0.5, 1.0, s) * scale).astype(np.float32)).bfloat16()
    U, S, V, X = make(1 / r, b, p, r), make(1 / b, b, b, r), make(1 / q, b, q, r), make(1, T, b * q)
    for t, c in bad:
        X[t, c] = float("inf")
    Xd, Ud, Sd, Vd = (t.cuda() for t in (X, U, S, V))
    Y = gu.empty_out(T, b * p, "bf16")
    packed = gu.B.blast_pack(Ud, Sd, Vd, b * q, b * p, b, r)
    gu.B.blast_forward(Xd, Ud, None, packed, Y, b, r, flags | gu.B.BLAST_PACKED)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        ref = oracle.blast_forward(*(t.double().numpy() for t in (X, U, S, V)))
    _agree(gu.to_f64(Y), ref, gu.TOL["bf16"])


@pytest.mark.parametrize("T,b", [(2, 1), (2, 3), (2, 4), (2, 15)])
@pytest.mark.parametrize("r", [128, 136])
def test_coupling_of_absent_blocks(T, b, r):
    """One or two tokens: the coupling takes 16 input blocks in four lanes, whatever their number."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _blast(T, 64, 40, b, r, [(1, b * 64 - 1)], 0)


# kernel of the first stage -> sizes (T, q, b, r) it is chosen for; test_tile_rules.py checks that it still is
WINDOWS = {
    "128x128 w4 k64x2 i32 windows": [(330, 152, 16, 512)],
    "192x128 w4 k64x2 i32 windows": [(1329, 136, 8, 656)],
    "128x192 w4 k64x2 i32 windows": [(2700, 136, 16, 264)],
    "128x128 w8 k64x4 i32 windows": [(520, 344, 8, 520)],
    "128x128 w8 k64x4 i16 windows": [(521, 208, 16, 264)],
    "128x128 w4 k64x4 i32 windows": [(700, 584, 8, 520)],
    "192x128 w8 k64x3 i32 windows": [(1300, 344, 8, 264)],
    "192x128 w8 k64x3 i16 windows": [(300, 344, 16, 1024)],
    "128x192 w8 k64x3 i32 windows": [(1052, 200, 16, 136)],
    "128x192 w8 k64x3 i16 windows": [(640, 344, 8, 1144)],
    "128x256 w8 k64x3 i32 windows": [(800, 344, 8, 1016)],
    "128x256 w8 k64x3 i16 windows": [(513, 200, 8, 1336)],
    "256x128 w8 k64x3 i32 windows": [(500, 344, 16, 640)],
    "256x128 w8 k64x3 i16 windows": [(267, 152, 16, 912)],
    "256x256 w8 k64x2 i32 windows": [(700, 344, 16, 1024)],
}


@pytest.mark.parametrize("T,q,b,r", [row for sizes in WINDOWS.values() for row in sizes])
def test_windows_of_input_blocks(T, q, b, r):
    """Input blocks read in 64-column chunks of the input row: infinities in the first and the last column of a block, which
    its neighbours' windows hold too."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    _blast(T, q, 16, b, r, [(0, q), (1, q - 1), (T // 2, (b - 1) * q), (T - 1, b * q - 1), (T - 2, 0)], gu.B.BLAST_THREE_KERNELS)


@pytest.mark.parametrize("T", [1, 17, 32])
@pytest.mark.parametrize("K", [40, 136, 1032])
def test_partial_last_step_of_the_weight_stream(T, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    rng = np.random.default_rng(K)
    W, X = (torch.from_numpy(rng.uniform(0.5, 1.0, s).astype(np.float32)).bfloat16() for s in ((40, K), (T + 1, K)))
    X[0, K - 1], X[T // 2, K - 8], W[3, K - 1] = float("inf"), float("nan") if T > 1 else 1.0, float("inf")
    X = X[:T].contiguous()
    Y = gu.empty_out(T, 40, "bf16")
    gu.B.dense_reference_forward(X.cuda(), W.cuda(), Y, 0)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        ref = X.double().numpy() @ W.double().numpy().T
    got = gu.to_f64(Y)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    ok = np.isfinite(ref)
    assert not ok.any() or np.abs(got[ok] - ref[ok]).max() <= gu.TOL["bf16"] * np.abs(ref[ok]).max()

"""Tiles of the bf16 products that the dispatch picks by estimate for several rounds of workgroups (128 x 192, 192 x 128 and
128 x 128, two workgroups per compute unit) and the eight-wavefront tiles of a single round (by their padded area where
128 x 128 tiles would be more than one), each with a ragged last tile
in rows and columns, contiguous and interleaved outputs, odd and even numbers of steps, a partial last step."""
import numpy as np
import pytest

import blr_inputs as bi
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,n_in,n_out", [
    (4095, 192, 2296), (3334, 192, 2308),             # 192 x 128, three steps
    (4095, 192, 3068),                                # 256 x 256
    (3073, 128, 3085),                                # 128 x 128, two steps; columns that end off a 16-byte boundary
    (520, 256, 11000), (1817, 192, 4108),             # 128 x 128, several rounds
    (1100, 320, 4600),                                # 256 x 128
    (1999, 1280, 2044), (1999, 1288, 2041),           # one round of 128 x 128: eight wavefronts
    (1020, 520, 4090), (1000, 640, 4044),             # ... four: a full chip, up to 1024 tokens
    (1000, 1280, 2042), (300, 1000, 4090),            # one round of 128 x 64, in steps of 64
    (1000, 1416, 2044), (300, 1480, 4090),            # ... and of 128
    (1000, 1280, 2050),                               # several rounds of 128 x 64
    (2529, 264, 389), (2529, 1288, 389),              # one round of 64 x 128, in steps of 64 and of 128
    (1300, 640, 4092), (640, 512, 8189), (800, 320, 8188),                # one round of 192 x 128, 128 x 192 and 128 x 256
    (2047, 192, 2300),                                # ... of 128 x 192, three steps
    (1500, 192, 2299), (1500, 200, 2300), (1300, 192, 1148),              # three steps and a partial fourth on four stages
    (1100, 1344, 2044),                               # half of the chip on 128 x 128
    # a round on nearly every compute unit: 16 x 16 matrix instructions on 192 x 128, 128 x 192, 128 x 256, 256 x 128 and 128 x 128
    (300, 512, 16380), (600, 320, 9790), (600, 256, 13050), (2040, 320, 4090), (2001, 328, 2044), (2001, 192, 2044),
    (300, 264, 10500),                                # 128 x 128 in one round, where 256 x 128 would fill the chip
])
def test_dense_tiles(T, n_in, n_out):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    W, X = bi.dense_weight(n_in, n_out, "bf16"), bi.activations(T, n_in, "bf16")
    Y = gu.empty_out(T, n_out, "bf16")
    gu.B.dense_reference_forward(gu.to_dev(X), gu.to_dev(W), Y, 0)
    torch.cuda.synchronize()
    assert gu.rel_err(gu.to_f64(Y), oracle.dense_forward(X.f64, W.f64)) <= gu.TOL["bf16"]


@pytest.mark.parametrize("T,b,p,rp,q", [
    (2076, 16, 64, 12, 132), (4111, 4, 64, 48, 388),  # second factor on 192 x 128
    (1743, 16, 64, 12, 516), (4037, 4, 64, 48, 1028), # 128 x 192
    (1153, 16, 64, 12, 380), (577, 4, 64, 64, 3068),  # 128 x 128, several rounds
    (1409, 4, 64, 32, 1530), (1153, 16, 64, 8, 572), (2047, 4, 64, 32, 1532),    # ... of two steps
    (4095, 4, 64, 48, 572),                           # 256 x 256
    (400, 16, 64, 66, 250), (300, 16, 64, 64, 250),   # 128 x 64, one round of four wavefronts and of eight
    (1300, 4, 64, 48, 1020), (633, 16, 64, 12, 508), (780, 4, 64, 64, 2036),     # one round of 192 x 128, 128 x 192 and 128 x 256
])
@pytest.mark.parametrize("order", ["interleaved", "blocked"])
def test_monarch_tiles(T, b, p, rp, q, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    R = bi.gaussian(bi.BASE_SEED, 51, (b, rp * b, p), 1.0 / np.sqrt(p), "bf16")
    L = bi.gaussian(bi.BASE_SEED, 52, (b, q, b * rp), 1.0 / np.sqrt(b * rp), "bf16")
    X = bi.activations(T, b * p, "bf16")
    Y = gu.empty_out(T, b * q, "bf16")
    blocked = order == "blocked"
    B.monarch_rect_forward(gu.to_dev(X), gu.to_dev(R), gu.to_dev(L), Y, b, b, rp, B.MONARCH_OUT_BLOCKED if blocked else 0)
    torch.cuda.synchronize()
    Yref = oracle.monarch_rect_forward(X.f64, R.f64, L.f64, b, b, oracle.OUT_BLOCKED if blocked else oracle.OUT_INTERLEAVED)
    assert gu.rel_err(gu.to_f64(Y), Yref) <= gu.TOL["bf16"]

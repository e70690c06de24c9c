"""The fp32 single-kernel Monarch layer against the oracle at the edges of its tiles: token counts around 16, ranks that
are no multiple of a 16-row tile, contraction lengths with a partial piece of 64, more output ranges than one."""
import numpy as np
import pytest

import blr_inputs as bi
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# fp32 sums of at most K = 1024 products: K * 2^-24 of the largest intermediate in the worst case, sqrt(K) * 2^-24 in
# practice; the repository's bound for fp32 (1e-5 of the largest output) covers it
TOL = 1e-5


@pytest.mark.parametrize("order", ["interleaved", "blocked"])
@pytest.mark.parametrize("T,p,q,b1,b2,rp", [
    (8, 64, 64, 4, 4, 16), (1, 4, 4, 1, 1, 4), (16, 68, 24, 2, 2, 20), (17, 132, 100, 3, 5, 12), (33, 256, 256, 4, 4, 64),
    (5, 16, 9, 4, 2, 4), (512, 64, 48, 4, 4, 8), (15, 20, 1000, 2, 1, 40), (3, 8, 4100, 1, 1, 8), (130, 1024, 64, 1, 4, 36)])
def test_against_the_oracle(T, p, q, b1, b2, rp, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    n_in, n_out = b1 * p, b2 * q
    R = bi.gaussian(T + p, 41, (b1, rp * b2, p), 1.0 / np.sqrt(p), "f32")
    L = bi.gaussian(T + p, 42, (b2, q, b1 * rp), 1.0 / np.sqrt(b1 * rp), "f32")
    X = bi.activations(T, n_in, "f32", seed=q)
    blocked = order == "blocked"
    Y = gu.empty_out(T, n_out, "f32")
    B.monarch_rect_forward(gu.to_dev(X), gu.to_dev(R), gu.to_dev(L), Y, b1, b2, rp, B.MONARCH_OUT_BLOCKED if blocked else 0)
    torch.cuda.synchronize()
    ref = oracle.monarch_rect_forward(X.f64, R.f64, L.f64, b1, b2, oracle.OUT_BLOCKED if blocked else oracle.OUT_INTERLEAVED)
    assert gu.rel_err(gu.to_f64(Y), ref) <= TOL

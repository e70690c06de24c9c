"""First Monarch products of short rank blocks on the weight-streaming kernel: a workgroup's 16 weight rows run across the
blocks of up to 8 columns where these are many, and hold one block otherwise; token counts of one tile and of several."""
import numpy as np
import pytest

import blr_inputs as bi
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,p,q,b1,b2,rp", [
    (1, 16, 24, 32, 32, 1), (16, 24, 8, 24, 40, 3), (17, 32, 16, 16, 40, 5), (32, 32, 8, 32, 24, 7),   # packed, a last tile of part of a block
    (5, 8, 8, 128, 8, 1), (100, 64, 16, 16, 16, 8),                                                    # ... and several tiles of tokens
    (20, 520, 16, 8, 72, 6),                                                                           # a partial last step
    (16, 16, 24, 16, 32, 1), (33, 16, 8, 8, 16, 12), (3, 32, 8, 32, 32, 9)])                           # one block per workgroup
def test_against_the_oracle(T, p, q, b1, b2, rp):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    n_in, n_out = b1 * p, b2 * q
    R = bi.gaussian(T + p, 43, (b1, rp * b2, p), 1.0 / np.sqrt(p), "bf16")
    L = bi.gaussian(T + p, 44, (b2, q, b1 * rp), 1.0 / np.sqrt(b1 * rp), "bf16")
    X = bi.activations(T, n_in, "bf16", seed=q)
    Y = gu.empty_out(T, n_out, "bf16")
    gu.B.monarch_rect_forward(gu.to_dev(X), gu.to_dev(R), gu.to_dev(L), Y, b1, b2, rp, gu.B.MONARCH_TWO_KERNELS)
    torch.cuda.synchronize()
    assert gu.rel_err(gu.to_f64(Y), oracle.monarch_rect_forward(X.f64, R.f64, L.f64, b1, b2, oracle.OUT_INTERLEAVED)) <= gu.TOL["bf16"]

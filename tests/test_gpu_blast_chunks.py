"""The three-kernel BLAST execution where its plan can go wrong: input blocks that are no whole cache lines (read in
64-column chunks against the zero-padded copy of the factor), chunks of tokens with the coupling in place, a last chunk of
a few tokens, both coupling tiles."""
import numpy as np
import pytest

import blr_inputs as bi
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,q,p,b,r", [
    (700, 88, 64, 16, 136),       # 64 | 16 q, 64 does not divide q: windows of 2 and 3 chunks, partial tiles in every dimension
    (1300, 344, 32, 8, 264), (640, 184, 40, 8, 128), (330, 152, 24, 16, 512),
    (270, 64, 40, 16, 1032),      # coupling on 32-token tiles, a partial last group of rank indices
])
def test_against_the_oracle(T, q, p, b, r):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    lay = bi.blast_layer(b * q, b * p, b, r, "bf16", seed=T)
    X = bi.activations(T, b * q, "bf16", seed=r)
    Y = gu.to_f64(gu.run_blast(X, lay, gu.B.BLAST_THREE_KERNELS, packed=True))
    assert gu.rel_err(Y, oracle.blast_forward(X.f64, lay.U.f64, lay.S.f64, lay.V.f64)) <= gu.TOL["bf16"]


@pytest.mark.parametrize("T", [3072 + 5, 2 * 3072, 7000])
def test_chunks_agree_with_one_chunk(T):
    """More tokens than a chunk holds (1536 to 3072 at b r = 16 K): rows do not depend on each other, so the rows of a
    call equal those of calls on parts of it that fit one chunk, bit for bit where the products pick the same tiles
    (they need not: bf16 rounding of two intermediates and the output, 3 * 2^-9 of the largest value)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    b, r, q, p = 16, 1024, 64, 16
    g = torch.Generator(device="cuda").manual_seed(T)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    U, S, V = ((rand(*s) / r ** 0.5).bfloat16() for s in ((b, p, r), (b, b, r), (b, q, r)))
    X = rand(T, b * q).bfloat16()
    packed = B.blast_pack(U, S, V, b * q, b * p, b, r)

    def run(x):
        y = torch.full((x.shape[0], b * p), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.blast_forward(x, U, None, packed, y, b, r, B.BLAST_PACKED | B.BLAST_THREE_KERNELS)
        return y

    whole = run(X)
    parts = torch.cat([run(X[i:i + 1000].contiguous()) for i in range(0, T, 1000)])
    torch.cuda.synchronize()
    err = (whole.double() - parts.double()).abs().max() / parts.double().abs().max()
    assert torch.isfinite(whole).all() and float(err) <= 3 * 2.0 ** -9


def test_unaligned_blocks_and_a_last_column_tile():
    """Stage 1 of 16 x 17 large tiles on 256 compute units: the columns past the whole round are a product of their own, with
    too few tiles for the kernels that read input blocks in 64-column windows. Two stored intermediates and the output are
    rounded to bf16, 2^-9 of each value, and the sums in between average it: 1e-2 as for the other cases."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    T, b, r, q, p = 256, 16, 4352, 1376, 16
    g = torch.Generator(device="cuda").manual_seed(7)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    U, S, V = (rand(b, p, r) / r ** 0.5).bfloat16(), (rand(b, b, r) / b ** 0.5).bfloat16(), (rand(b, q, r) / q ** 0.5).bfloat16()
    X = rand(T, b * q).bfloat16()
    packed = B.blast_pack(U, S, V, b * q, b * p, b, r)
    Y = torch.full((T, b * p), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.blast_forward(X, U, None, packed, Y, b, r, B.BLAST_PACKED | B.BLAST_THREE_KERNELS)
    Z = [X[:, j * q:(j + 1) * q].float() @ V[j].float() for j in range(b)]
    ref = torch.cat([sum(S[i, j].float() * Z[j] for j in range(b)) @ U[i].float().t().contiguous() for i in range(b)], dim=1)
    assert float((Y.float() - ref).norm() / ref.norm()) <= 1e-2

"""The three-kernel BLAST execution where its plan can go wrong: input blocks that are no whole cache lines (read in
64-column chunks against the zero-padded copy of the factor) on each tile that takes them, chunks of tokens with the
coupling in place, a last chunk of a few tokens, the 8-bit intermediate behind such windows."""
import numpy as np
import pytest

import blr_inputs as bi
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# kernel of the first stage -> sizes (T, q, p, b, r) it is chosen for; test_tile_rules.py checks that it still is. Windows of 64-column
# chunks: 64 | b q, 64 does not divide q, q >= 128 and 160 and more tiles of 128 x 128
STAGE1 = {
    "128x128 w4 k64x2 i32 windows": [(330, 152, 24, 16, 512), (1200, 152, 24, 16, 264)],
    "192x128 w4 k64x2 i32 windows": [(1329, 136, 16, 8, 656)],
    "128x192 w4 k64x2 i32 windows": [(2700, 136, 16, 16, 264)],
    "128x128 w8 k64x4 i32 windows": [(520, 344, 16, 8, 520)],
    "128x128 w8 k64x4 i16 windows": [(521, 208, 16, 16, 264)],
    "128x128 w4 k64x4 i32 windows": [(700, 584, 16, 8, 520)],
    "192x128 w8 k64x3 i32 windows": [(1300, 344, 32, 8, 264)],
    "192x128 w8 k64x3 i16 windows": [(300, 344, 16, 16, 1024)],
    "128x192 w8 k64x3 i32 windows": [(1052, 200, 16, 16, 136)],
    "128x192 w8 k64x3 i16 windows": [(640, 344, 16, 8, 1144)],
    "128x256 w8 k64x3 i32 windows": [(800, 344, 16, 8, 1016)],
    "128x256 w8 k64x3 i16 windows": [(513, 200, 16, 8, 1336)],
    "256x128 w8 k64x3 i32 windows": [(500, 344, 16, 16, 640)],
    "256x128 w8 k64x3 i16 windows": [(267, 152, 16, 16, 912)],
    "256x256 w8 k64x2 i32 windows": [(700, 344, 16, 16, 1024)],
    # blocks read for themselves: short ones, too few tiles; a partial last group of rank indices
    "128x128 w4 k32x4 i32 partial": [(700, 88, 64, 16, 136)],
    "64x64 w4 k64x2 i32 partial": [(640, 184, 40, 8, 128)],
    "128x128 w4 k32x4 i32": [(270, 64, 40, 16, 1032)],
}


@pytest.mark.parametrize("T,q,p,b,r", [row for sizes in STAGE1.values() for row in sizes])
def test_against_the_oracle(T, q, p, b, r):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    lay = bi.blast_layer(b * q, b * p, b, r, "bf16", seed=T)
    X = bi.activations(T, b * q, "bf16", seed=r)
    Y = gu.to_f64(gu.run_blast(X, lay, gu.B.BLAST_THREE_KERNELS, packed=True))
    assert gu.rel_err(Y, oracle.blast_forward(X.f64, lay.U.f64, lay.S.f64, lay.V.f64)) <= gu.TOL["bf16"]


@pytest.mark.parametrize("T,r,q", [
    (3072 + 5, 1024, 64), (2 * 3072, 1024, 64), (7000, 1024, 64),         # chunks of 1792 and of up to 4096 tokens
    (4096, 1024, 64), (4096 + 5, 1024, 64), (8192 + 5, 768, 64),          # ... on both sides of 4096; 4352
    (4096 + 5, 1024, 960),                                                # ... of up to 3584, where the input bounds them
    (513, 4096, 64), (540, 4096, 64),                                     # of 512: a last one of 1 and of 28 tokens
    (4097, 4096, 64)])                                                    # of 1024: a last one of 1 token
def test_chunks_agree_with_one_chunk(T, r, q):
    """More tokens than a chunk holds, the coupling in place: rows do not depend on each other, so the rows of a call equal
    those of calls on parts of it that fit one chunk, bit for bit where the products pick the same tiles
    (they need not: bf16 rounding of two intermediates and the output, 3 * 2^-9 of the largest value)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    b, p = 16, 16
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
    step = 256 if r == 4096 else 1000
    parts = torch.cat([run(X[i:i + step].contiguous()) for i in range(0, T, step)])
    torch.cuda.synchronize()
    err = (whole.double() - parts.double()).abs().max() / parts.double().abs().max()
    assert torch.isfinite(whole).all() and float(err) <= 3 * 2.0 ** -9


@pytest.mark.parametrize("T", [4096 + 5, 8192 + 1])
@pytest.mark.parametrize("packed", [True, False])
def test_workspace_of_the_shorter_chunks(T, packed):
    """The longer chunks beyond 4096 tokens are a matter of speed: a call in a workspace of the size that 4096 tokens ask for runs
    in shorter ones, inside it (both round two intermediates and the output to bf16: 3 * 2^-9 of the largest value)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    b, q, p, r = 16, 64, 16, 1024
    flags = B.BLAST_THREE_KERNELS | (B.BLAST_PACKED if packed else 0)
    most, least = (B.blast_workspace_bytes(t, b * q, b * p, b, r, B.BF16, flags) for t in (T, 4096))
    assert least < most
    g = torch.Generator(device="cuda").manual_seed(T)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    U, S, V = ((rand(*s) / r ** 0.5).bfloat16() for s in ((b, p, r), (b, b, r), (b, q, r)))
    X = rand(T, b * q).bfloat16()
    pk = B.blast_pack(U, S, V, b * q, b * p, b, r)
    buf = torch.full((most,), 0x5A, dtype=torch.uint8, device="cuda")
    ys = [torch.full((T, b * p), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    for y, size in zip(ys, (least, most)):
        B.blast_forward(X, U, None if packed else S, pk if packed else V, y, b, r, flags, workspace=buf[:size])
        if size == least:
            torch.cuda.synchronize()
            assert bool((buf[size:] == 0x5A).all())
    err = (ys[0].double() - ys[1].double()).abs().max() / ys[1].double().abs().max()
    assert torch.isfinite(ys[0]).all() and float(err) <= 3 * 2.0 ** -9
    with pytest.raises(B.BlrError) as e:
        B.blast_forward(X, U, None if packed else S, pk if packed else V, ys[0], b, r, flags, workspace=buf[:least - 256])
    assert e.value.status == B.ERR_WORKSPACE


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


@pytest.mark.parametrize("T,q,b,r", [(700, 344, 16, 1024), (1300, 344, 8, 272)])        # 256 x 256 and 128 x 128 tiles
def test_windows_with_the_8_bit_intermediate(T, q, b, r):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    from oracle import quant
    lay = bi.blast_layer(b * q, b * 16, b, r, "bf16", seed=T)
    X = bi.activations(T, b * q, "bf16", seed=r)
    Y = gu.to_f64(gu.run_blast(X, lay, gu.B.BLAST_Z_FP8, packed=True))
    assert gu.rel_err(Y, quant.blast_forward_qz(X.f64, lay.U.f64, lay.S.f64, lay.V.f64)[0]) <= gu.TOL["bf16"]


@pytest.mark.parametrize("T,n_in,n_out,b,r", [
    (6145, 768, 96, 3, 128), (8193, 768, 96, 3, 128),                    # 64-token tiles, 128-token tiles; a last tile of one token
    (6200, 3072, 48, 6, 72),                                             # blocks of 512: two groups of rank indices, the last of 8
    (32641, 1536, 24, 3, 8),                                             # one group, the last tile of one token
])
def test_fused_stage12_with_few_blocks(T, n_in, n_out, b, r):
    """The rule's fused execution on few, long blocks, all tokens against the three kernels (each rounds two intermediates and
    the output to bf16: 6 * 2^-9 of the largest value between them) and the first and last rows against the oracle."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    lay = bi.blast_layer(n_in, n_out, b, r, "bf16", seed=T)
    X = bi.activations(T, n_in, "bf16", seed=r)
    sizes = [B.blast_workspace_bytes(T, n_in, n_out, b, r, B.BF16, B.BLAST_PACKED | f) for f in (0, B.BLAST_FUSED_STAGE12)]
    assert sizes[0] == sizes[1]
    Y = gu.to_f64(gu.run_blast(X, lay, 0, packed=True))
    three = gu.to_f64(gu.run_blast(X, lay, B.BLAST_THREE_KERNELS, packed=True))
    assert abs(Y - three).max() <= 6 * 2.0 ** -9 * abs(three).max()
    rows = np.r_[0:64, T - 65:T]
    assert gu.rel_err(Y[rows], oracle.blast_forward(X.f64[rows], lay.U.f64, lay.S.f64, lay.V.f64)) <= gu.TOL["bf16"]

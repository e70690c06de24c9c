"""BLAST at few tokens: stage 1 and the coupling in one launch (two and four input blocks to a tile, parts of a block's
contraction index, partial last steps, absent blocks), and a chain's groups whose last products are combined in one launch."""
import numpy as np
import pytest

import blr_inputs as bi
import oracle
from oracle import chain as oc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T", [1, 4, 5, 8, 9, 16, 17])
@pytest.mark.parametrize("b,q,p,r", [
    (16, 64, 72, 136), (15, 40, 80, 152),               # a wavefront per pair, an absent sixteenth block, a partial last step
    (9, 128, 96, 264), (5, 264, 72, 136),               # idle wavefronts; parts of unequal length
    (1, 1032, 136, 144), (3, 520, 200, 392),            # many parts of few blocks; four blocks to a tile up to 4 tokens
    (16, 536, 16, 136), (16, 1032, 8, 136)])            # more steps than LDS holds; too long an input from 3 tokens on
def test_against_the_oracle(T, b, q, p, r):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    lay = bi.blast_layer(b * q, b * p, b, r, "bf16")
    X = bi.activations(T, b * q, "bf16", seed=T)
    Y = gu.run_blast(X, lay, packed=True)
    assert gu.rel_err(gu.to_f64(Y), oracle.blast_forward(X.f64, lay.U.f64, lay.S.f64, lay.V.f64)) <= gu.TOL["bf16"]
    # the same roundings as with the three launches
    three = gu.run_blast(X, lay, gu.B.BLAST_THREE_KERNELS, packed=True)
    assert gu.rel_err(gu.to_f64(Y), gu.to_f64(three)) <= gu.TOL["bf16"]


@pytest.mark.parametrize("T", [1, 2, 3, 4])
@pytest.mark.parametrize("b,q,p,r", [
    (16, 136, 16, 256), (16, 264, 16, 512),             # 16 blocks to a tile at one token, 8 up to two; r that leaves one round with 8
    (15, 520, 8, 104), (9, 264, 8, 104),                # absent blocks in the only tile and in the last of two, each width
    (6, 264, 8, 24), (5, 40, 80, 152),                  # 8 up to two tokens, 4 up to four; two steps, a partial one
    (3, 1032, 8, 1032)])                                # a round and two rank indices over: two blocks to a tile
def test_blocks_to_a_tile(T, b, q, p, r):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    B = gu.B
    lay = bi.blast_layer(b * q, b * p, b, r, "bf16")
    X = bi.activations(T, b * q, "bf16", seed=T)
    Y = gu.run_blast(X, lay, packed=True)
    assert gu.rel_err(gu.to_f64(Y), oracle.blast_forward(X.f64, lay.U.f64, lay.S.f64, lay.V.f64)) <= gu.TOL["bf16"]
    # a token's infinities stay its own: the tile multiplies it with the other tokens' blocks too
    U, S, V = (gu.to_dev(t) for t in (lay.U, lay.S, lay.V))
    packed, x = B.blast_pack(U, S, V, b * q, b * p, b, r), gu.to_dev(X).clone()
    x[T - 1, q - 1] = x[T - 1, (b - 1) * q] = float("inf")
    Z = B.blast_forward(x, U, None, packed, gu.empty_out(T, b * p, "bf16"), b, r, B.BLAST_PACKED)
    torch.cuda.synchronize()
    assert torch.equal(Z[:T - 1], Y[:T - 1]) and not bool(torch.isfinite(Z[T - 1]).any())


@pytest.mark.parametrize("T", [1, 2])
@pytest.mark.parametrize("b,q,p,r", [(16, 256, 256, 640), (5, 264, 72, 136)])
def test_one_or_two_tokens_whichever_execution(T, b, q, p, r):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    lay = bi.blast_layer(b * q, b * p, b, r, "bf16")
    X = bi.activations(T, b * q, "bf16", seed=T)
    # (the separate launches add stage 1 up in another order: some of these sums round differently there)
    assert torch.equal(gu.run_blast(X, lay, gu.B.BLAST_THREE_KERNELS, packed=True), gu.run_blast(X, lay, packed=True))


@pytest.mark.parametrize("op,params", [("monarch", dict(nblocks=4, r_square=64, r_mlp=1056)), ("blast", dict(b=4, r_square=136, r_mlp=264))])
@pytest.mark.parametrize("T", [3, 16, 17, 32, 33])
def test_combined_groups(op, params, T):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    from paper_2512_20861_amd.chain import DeviceChain
    layers = bi.chain_layers(op, n_layers=2, hidden=512, mlp=800 if op == "blast" else 768, params=params, dtype="bf16")
    x = bi.activations(T, 512, "bf16")
    chain = DeviceChain(layers, T, eps=oc.EPS)
    assert chain._native
    lin = lambda v, f: oracle.monarch_forward(v, f.R.f64, f.L.f64) if op == "monarch" else oracle.blast_forward(v, f.U.f64, f.S.f64, f.V.f64)
    got = [chain.forward(gu.to_dev(x)).clone() for _ in range(3)]
    torch.cuda.synchronize()
    assert gu.rel_err(gu.to_f64(got[0]), oc.chain_forward(x.f64, layers, lin)) <= 2e-2 and all(torch.equal(g, got[0]) for g in got)

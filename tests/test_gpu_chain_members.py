"""A chain's groups whose last products are combined on the tile kernels (the scaled sum of q, k, v; the SiLU gate): every tile that
takes them, ragged token counts and columns, against the oracle on sampled rows and against the same chain step by step."""
import numpy as np
import pytest

import blr_inputs as bi
import oracle
from oracle import chain as oc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _lin(x, f):
    return oracle.monarch_forward(x, f.R.f64, f.L.f64) if hasattr(f, "R") else oracle.blast_forward(x, f.U.f64, f.S.f64, f.V.f64)


# tokens: q + k + v on 128 x 128 / 128 x 64 / 64 x 64 tiles or as steps, gate and up on all four, one round and several, both matrix
# instructions
TOKENS = [70, 150, 300, 490, 520, 1100, 1700, 2000, 2050]


@pytest.mark.parametrize("T", TOKENS)
@pytest.mark.parametrize("op,hidden,mlp,params", [
    ("monarch", 2048, 8192, dict(nblocks=4, r_square=512, r_mlp=512)), ("blast", 2048, 8192, dict(b=16, r_square=256, r_mlp=512)),
    # 504 columns a block; a rank that stays with the steps, and one of a single trip
    ("blast", 1920, 7560, dict(b=15, r_square=192, r_mlp=256))])
def test_members_on_tiles(op, hidden, mlp, params, T):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    from paper_2512_20861_amd.chain import DeviceChain
    layers = bi.chain_layers(op, n_layers=1, hidden=hidden, mlp=mlp, params=params, dtype="bf16")
    x = bi.activations(T, hidden, "bf16", seed=T)
    chain = DeviceChain(layers, T, eps=oc.EPS)
    assert chain._native
    got = [chain.forward(gu.to_dev(x)).clone() for _ in range(3)]
    steps, _ = chain.forward(gu.to_dev(x), record=True, rows=torch.zeros(1, dtype=torch.long, device="cuda"))
    torch.cuda.synchronize()
    assert all(torch.equal(g, got[0]) for g in got)
    assert gu.rel_err(gu.to_f64(got[0]), gu.to_f64(steps)) <= 2e-2
    rows = np.unique([t for t in (0, 31, 63, 64, 127, 128, 255, T // 2, T - 3, T - 1) if t < T])
    ref = oc.chain_forward(x.f64[rows], layers, _lin)
    sel = torch.from_numpy(rows).cuda()
    assert gu.rel_err(gu.to_f64(got[0][sel]), ref) <= 2e-2


# runs of 48 elements (16-byte stores), of 12 (element by element), of 8, of two and one, of three. In the last two the normed first
# products have 2304 to 3840 tiles: a wavefront owns 16 rows, the last workgroup of an output block has two tiles or one, and with
# input blocks of 48 the last step is a partial one.
@pytest.mark.parametrize("T", [1, 3, 4, 16, 17, 32, 33, 70, 900])
@pytest.mark.parametrize("hidden,mlp,params", [
    (768, 3072, dict(nblocks=4, r_square=256, r_mlp=256)), (768, 1152, dict(nblocks=8, r_square=256, r_mlp=264)),
    (2048, 4096, dict(nblocks=16, r_square=256, r_mlp=512)), (1152, 576, dict(nblocks=24, r_square=576, r_mlp=576)),
    (768, 768, dict(nblocks=16, r_square=1152, r_mlp=1152))])
def test_input_blocks_in_one_piece(hidden, mlp, params, T):
    """Monarch: o and down whose input blocks are runs that the matrix kernels do not read."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    from paper_2512_20861_amd.chain import DeviceChain
    layers = bi.chain_layers("monarch", n_layers=2, hidden=hidden, mlp=mlp, params=params, dtype="bf16")
    x = bi.activations(T, hidden, "bf16", seed=T)
    chain = DeviceChain(layers, T, eps=oc.EPS)
    assert chain._native
    got = [chain.forward(gu.to_dev(x)).clone() for _ in range(3)]
    torch.cuda.synchronize()
    assert all(torch.equal(g, got[0]) for g in got)
    rows = np.unique([t for t in (0, 31, 63, 64, 127, 128, T // 2, T - 3, T - 1) if 0 <= t < T])
    ref = oc.chain_forward(x.f64[rows], layers, _lin)
    assert gu.rel_err(gu.to_f64(got[0][torch.from_numpy(rows).cuda()]), ref) <= 2e-2

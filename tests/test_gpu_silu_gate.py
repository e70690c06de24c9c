"""The SiLU gate of a chain where it is computed with its products: every finite bf16 value as the gate, on each of the tiles that
take gate and up together, bit for bit what the elementwise step behind two products gives."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

HIDDEN, MLP, NB, R = 4096, 8192, 4, 256


def _monarch(n_in, n_out, first, second):
    """R[l][rho * NB + k][c], L[k][j][l * R / NB + rho] (bf16 bits)."""
    return types.SimpleNamespace(n_in=n_in, n_out=n_out, r=R, nblocks=NB, dtype="bf16", R=types.SimpleNamespace(dtype="bf16", bits=first),
                                 L=types.SimpleNamespace(dtype="bf16", bits=second))


def _bits(values):
    return torch.from_numpy(np.asarray(values, dtype=np.float32)).bfloat16().view(torch.int16).numpy().view(np.uint16)


# 64 x 64, 128 x 64 and 128 x 128 tiles in one round (a nearly full one on the other matrix instruction), 128 x 128 tiles in several; the
# weight-streaming kernel
TILES = {"2 of 64x64 w4 k64x4 i32": 128, "2 of 128x64 w8 k64x4 i32": 150, "2 of 128x128 w8 k64x4 i32": 300, "2 of 128x128 w8 k64x4 i16": 490,
         "2 of 128x128 w4 k64x2 i32": 520, "": 16}


@pytest.mark.parametrize("T", list(TILES.values()))
def test_every_gate(T):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    from paper_2512_20861_amd.chain import DeviceChain
    # q, k, v, o and down are zero, so gate and up read rmsnorm(x). Token t is the unit vector t % 8, 64 times it when normalised; the
    # first factor makes that a one in rank index t % 8 of every output block, and the products are column t % 8 of the second factor.
    zero = lambda n_in, n_out: _monarch(n_in, n_out, np.zeros((NB, R, n_in // NB), np.uint16), np.zeros((NB, n_out // NB, R), np.uint16))
    pick = np.zeros((NB, R // NB, NB, HIDDEN // NB), np.float32)
    for s in range(8):
        pick[0, s, :, s] = 1 / 64
    every = np.arange(65536, dtype=np.uint32).astype(np.uint16)
    every[(every & 0x7F80) == 0x7F80] = 0                 # (an infinity or a NaN would meet zeros of the other columns)
    gate, up = np.zeros((MLP, R), np.uint16), np.zeros((MLP, R), np.uint16)
    gate[:, :8] = every.reshape(MLP, 8)
    # among the second operands one that brings the gates of the smallest quotients (1e-37) back to ordinary size
    up[:, :8] = np.resize(_bits([1.0, -1.7109375, 1.5e37]), (8, MLP)).T
    first = _bits(pick.reshape(NB, R, HIDDEN // NB))
    layer = {n: zero(HIDDEN, HIDDEN) for n in "qkvo"}
    layer |= {"gate": _monarch(HIDDEN, MLP, first, gate.reshape(NB, MLP // NB, R)), "up": _monarch(HIDDEN, MLP, first, up.reshape(NB, MLP // NB, R)),
              "down": zero(MLP, HIDDEN)}
    chain = DeviceChain([layer], T, eps=0.0)
    assert chain._native
    x = torch.zeros(T, HIDDEN)
    x[torch.arange(T), torch.arange(T) % 8] = 1.0
    x = x.bfloat16().cuda()
    chain.gu.fill_(float("nan"))
    chain.forward(x)
    torch.cuda.synchronize()
    assert bool(chain.gu.isnan().all()), "gate and up were not combined"
    got = chain.m.clone()
    chain.forward(x, record=True, rows=torch.zeros(1, dtype=torch.long, device="cuda"))
    torch.cuda.synchronize()
    assert np.array_equal(np.unique(gu.to_f64(chain.g[:8])), np.unique(torch.from_numpy(every.view(np.int16)).view(torch.bfloat16).double().numpy()))
    assert torch.equal(got.view(torch.int16), chain.m.view(torch.int16))

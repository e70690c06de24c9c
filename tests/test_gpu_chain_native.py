"""DeviceChain.forward as one call of the library: the fused launches of a handful of tokens, the step list of more, the
graph that later passes replay, each against the oracle's chain and against the step-by-step call list."""
import numpy as np
import pytest

import blr_inputs as bi
import oracle
from oracle import chain as oc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PARAMS = {"monarch": dict(nblocks=4, r_square=64, r_mlp=128), "blast": dict(b=4, r_square=136, r_mlp=72)}


@pytest.mark.parametrize("op", ["monarch", "blast"])
@pytest.mark.parametrize("T", [1, 2, 4, 5, 33])
def test_native_chain(op, T):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    from paper_2512_20861_amd.chain import DeviceChain
    layers = bi.chain_layers(op, n_layers=2, hidden=512, mlp=768, params=PARAMS[op], dtype="bf16")
    x0, x1 = bi.activations(T, 512, "bf16"), bi.activations(T, 512, "bf16", seed=99)
    lin = (lambda x, f: oracle.monarch_forward(x, f.R.f64, f.L.f64)) if op == "monarch" else (lambda x, f: oracle.blast_forward(x, f.U.f64, f.S.f64, f.V.f64))
    chain = DeviceChain(layers, T, eps=oc.EPS)
    assert chain.grouped and chain._native
    refs = [oc.chain_forward(x.f64, layers, lin) for x in (x0, x1)]
    steps = gu.to_f64(chain.forward(gu.to_dev(x0), record=True)[0])
    first = []
    for n in range(5):                                   # separate launches, then the graph; other work in between
        for x, ref, keep in ((x0, refs[0], first), (x1, refs[1], None)):
            got = chain.forward(gu.to_dev(x)).clone()
            torch.cuda.synchronize()
            # two bf16 implementations of a 2-layer chain: the bound of the chain tests
            assert gu.rel_err(gu.to_f64(got), ref) <= 2e-2
            if keep is not None:
                keep.append(got)
    assert all(torch.equal(f, first[0]) for f in first)
    assert gu.rel_err(gu.to_f64(first[0]), steps) <= 2e-2
    # a stream that is being captured takes the launches themselves
    side = torch.cuda.Stream()
    xd = gu.to_dev(x0)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=side):
        chain.forward(xd)
    for _ in range(3):
        chain.h.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(chain.h, first[0])


@pytest.mark.parametrize("T", [2, 33])
def test_copies_and_lifetimes(T):
    """A copied chain has buffers and a handle of its own; a chain that ends while another stream is under capture leaves
    the capture alone."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import copy
    import gpu_util as gu
    from paper_2512_20861_amd.chain import DeviceChain
    layers = bi.chain_layers("monarch", n_layers=1, hidden=512, mlp=768, params=PARAMS["monarch"], dtype="bf16")
    x0, x1 = (gu.to_dev(bi.activations(T, 512, "bf16", seed=n)) for n in (1, 2))
    chain = DeviceChain(layers, T, eps=oc.EPS)
    want = [chain.forward(x).clone() for x in (x0, x1, x0)]
    other = copy.deepcopy(chain)
    assert other._native and other.h.data_ptr() != chain.h.data_ptr()
    kept = chain.forward(x0)
    for n in range(3):
        assert torch.equal(other.forward(x1), want[1]) and torch.equal(kept, want[0])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        other.h.copy_(x0)
        del chain
        other.forward(x0)
    for _ in range(3):
        other.h.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(other.h, want[0])


@pytest.mark.parametrize("op,hidden,mlp,params", [
    # a model's widths: first products of a Monarch chain on eight wavefronts, of a BLAST chain with their coupling
    ("monarch", 2048, 8192, dict(nblocks=4, r_square=512, r_mlp=512)), ("blast", 2048, 8192, dict(b=16, r_square=256, r_mlp=512)),
    # ranks that are no multiple of 16 or of 32, blocks of 40 and 72 columns (a partial last step)
    ("blast", 640, 1152, dict(b=16, r_square=264, r_mlp=392))])
@pytest.mark.parametrize("T", [1, 3, 4])
def test_wide_fused_chain(op, hidden, mlp, params, T):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    from paper_2512_20861_amd.chain import DeviceChain
    layers = bi.chain_layers(op, n_layers=2 if hidden < 2048 else 1, hidden=hidden, mlp=mlp, params=params, dtype="bf16")
    x = bi.activations(T, hidden, "bf16")
    chain = DeviceChain(layers, T, eps=oc.EPS)
    assert chain._native
    ref = oc.chain_forward(x.f64, layers, _lin)
    got = [chain.forward(gu.to_dev(x)).clone() for _ in range(3)]
    torch.cuda.synchronize()
    assert gu.rel_err(gu.to_f64(got[0]), ref) <= 2e-2 and all(torch.equal(g, got[0]) for g in got)


def _lin(x, f):
    return oracle.monarch_forward(x, f.R.f64, f.L.f64) if hasattr(f, "R") else oracle.blast_forward(x, f.U.f64, f.S.f64, f.V.f64)


@pytest.mark.parametrize("kind", ["monarch, wider blocks in the MLP", "blast, fewer blocks in the MLP", "blast with a monarch output projection"])
@pytest.mark.parametrize("T", [2, 33])
def test_layers_that_differ_inside(kind, T):
    """The native chain has one block count and one kind of linear; a chain of several runs its own call list."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    from paper_2512_20861_amd.chain import DeviceChain
    make = lambda op, **prm: bi.chain_layers(op, n_layers=2, hidden=512, mlp=1024, params=prm, dtype="bf16")
    op = kind.split()[0].rstrip(",")
    layers = make(op, **PARAMS[op])
    if "output" in kind:
        other = make("monarch", nblocks=4, r_square=136, r_mlp=128)
        names = ("o",)
    else:
        other = make(op, **(dict(nblocks=8, r_square=64, r_mlp=128) if op == "monarch" else dict(b=2, r_square=136, r_mlp=72)))
        names = ("gate", "up", "down")
    for layer, o in zip(layers, other):
        for name in names:
            layer[name] = o[name]
    x = bi.activations(T, 512, "bf16")
    chain = DeviceChain(layers, T, eps=oc.EPS)
    assert chain.grouped
    ref = oc.chain_forward(x.f64, layers, _lin)
    for _ in range(3):
        got = chain.forward(gu.to_dev(x))
        torch.cuda.synchronize()
        assert gu.rel_err(gu.to_f64(got), ref) <= 2e-2


@pytest.mark.parametrize("op", ["monarch", "blast"])
@pytest.mark.parametrize("T", [2, 33])
def test_replaced_parts_are_used(op, T):
    """A pass uses the factors, buffers and settings that the chain holds at the time, also after passes with others: those
    of a pass step by step (bit for bit where the native chain runs the same steps)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    from paper_2512_20861_amd.chain import DeviceChain
    layers = bi.chain_layers(op, n_layers=2, hidden=512, mlp=768, params=PARAMS[op], dtype="bf16")
    others = bi.chain_layers(op, n_layers=2, hidden=512, mlp=768, params=PARAMS[op], dtype="bf16", seed=77)
    x = gu.to_dev(bi.activations(T, 512, "bf16"))
    chain, spare = DeviceChain(layers, T, eps=oc.EPS), DeviceChain(others, T, eps=oc.EPS)
    factor = "R" if op == "monarch" else "U"

    def agrees(passes=4):
        want = chain.forward(x, record=True)[0].clone()
        for _ in range(passes):
            chain.h.fill_(float("nan"))
            got = chain.forward(x)
            assert got is chain.h
            assert torch.equal(got, want) if T > 4 else gu.rel_err(gu.to_f64(got), gu.to_f64(want)) <= 2e-2
        return want

    handle = chain._native
    seen = [agrees()]
    assert handle and chain._native is handle
    lin, other = chain.layers[1]["o"], spare.layers[1]["o"]
    old = getattr(lin, factor)

    def changes():
        setattr(lin, factor, getattr(other, factor)); yield
        getattr(lin, factor).data = old.clone(); yield                    # the same tensor object, other memory
        chain.layers[0]["down"] = spare.layers[0]["down"]; yield
        chain.groups[1] = spare.groups[1]; yield
        chain.eps = 0.5; yield
    for _ in changes():
        seen.append(agrees())
        assert chain._native                             # made anew
        assert not torch.equal(seen[-1], seen[-2])
    for name in ("h", "n", "ws", "m"):                   # buffers of the same layout: the same result in the new ones
        setattr(chain, name, torch.empty_like(getattr(chain, name)))
        assert torch.equal(agrees(), seen[-1])
    for i in range(3):                                   # another factor for every pass
        setattr(lin, factor, (old, getattr(other, factor))[i % 2])
        agrees(1)
    lin.r = lin.r // 2                                   # refused by the call list, and so by a pass
    for _ in range(3):
        with pytest.raises(ValueError):
            chain.forward(x)


def test_smaller_workspace_of_a_long_blast_chain():
    """A chain in a workspace of the size of 4096 tokens' chunks: q + k + v and gate * up are then no longer combined in one piece,
    nothing behind it is written, and the result is that of the longer chunks up to the rounding of the 20 stored values in between."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as gu
    from paper_2512_20861_amd.chain import DeviceChain
    T = 4200
    layers = bi.chain_layers("blast", n_layers=1, hidden=4096, mlp=8192, params=dict(b=16, r_square=256, r_mlp=384), dtype="bf16")
    x = gu.to_dev(bi.activations(T, 4096, "bf16"))
    chain = DeviceChain(layers, T, eps=oc.EPS)
    assert chain._native and chain.ws.numel() == 120 << 20
    want = chain.forward(x).clone()
    whole = chain.ws
    whole.fill_(0x5A)
    chain.ws = whole[:96 << 20]
    for _ in range(4):                                   # step by step, then the new handle's launches and its graph
        chain.h.fill_(float("nan"))
        got = chain.forward(x)
        torch.cuda.synchronize()
        assert torch.isfinite(got).all() and gu.rel_err(gu.to_f64(got), gu.to_f64(want)) <= 2e-2
    assert chain._native and bool((whole[96 << 20:] == 0x5A).all())

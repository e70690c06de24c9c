"""The work a program has this library do, as measurable cases: single BLR linears from one token to thousands
through the forward calls of the binding, and the decoder-layer chain through DeviceChain.forward.

A case is a plain dict. op: "monarch", "blast", "lowrank" (one linear: n_in, n_out, rank r, b blocks, T tokens, dtype)
or "chain" (kind: "monarch" or "blast", layers, T; seven linears and the glue between them per layer). Every program
keeps its factors (BLAST packed once), its output buffer and its workspace, and hands in new activations.
"""
import math
import types

import numpy as np
import torch

from paper_2512_20861_amd import binding as B
from paper_2512_20861_amd.chain import LINEARS, DeviceChain

# decoder-layer chain at Llama-3.2-1B width: blocks and ranks of its square and its MLP linears
HIDDEN, MLP = 2048, 8192
CHAIN = {"monarch": {"b": 4, "r_square": 512, "r_mlp": 512}, "blast": {"b": 16, "r_square": 256, "r_mlp": 512}}

# (op, n_in, n_out, r, b): the layers of the benchmark's configurations and of the paper's layer table
LAYERS = (
    ("monarch", 4096, 4096, 1024, 4), ("monarch", 4096, 11008, 1024, 4), ("monarch", 4096, 4096, 1024, 16),
    ("monarch", 11008, 4096, 1536, 16), ("monarch", 2048, 2048, 256, 16), ("monarch", 2048, 8192, 512, 16),
    ("monarch", 8192, 2048, 768, 16), ("monarch", 768, 2304, 192, 4), ("monarch", 3072, 768, 192, 4), ("monarch", 768, 3072, 128, 4),
    ("blast", 4096, 4096, 640, 16), ("blast", 11008, 4096, 1024, 16), ("blast", 4096, 4096, 1024, 16),
    ("blast", 2048, 2048, 256, 16), ("blast", 2048, 8192, 512, 16), ("blast", 8192, 2048, 768, 16), ("blast", 768, 768, 96, 16),
    ("blast", 768, 2304, 192, 6), ("blast", 768, 3072, 128, 3), ("blast", 3072, 768, 128, 3), ("blast", 1152, 4608, 256, 9),
    ("lowrank", 4096, 4096, 1024, 1), ("lowrank", 4096, 4096, 128, 1), ("lowrank", 11008, 4096, 1488, 1),
    ("lowrank", 2048, 8192, 512, 1), ("lowrank", 768, 2304, 192, 1), ("lowrank", 3072, 768, 128, 1), ("lowrank", 1152, 3456, 384, 1),
)
MAX_T = 8192


def _linear(name, op, n_in, n_out, r, b, T, dtype="bf16"):
    return {"name": name, "op": op, "n_in": n_in, "n_out": n_out, "r": r, "b": b, "T": T, "dtype": dtype}


def listed():
    return [
        # a small layer in full precision on a handful of tokens: the check a user runs first, and the smallest call
        _linear("monarch 256 f32 T=8", "monarch", 256, 256, 64, 4, 8, "f32"),
        # one decoded token through an attention projection
        _linear("monarch 4096 T=1", "monarch", 4096, 4096, 1024, 4, 1),
        # a small decode batch through an attention projection
        _linear("blast 4096 T=16", "blast", 4096, 4096, 640, 16, 16),
        # one image (197 patch tokens) through the second MLP linear of a ViT-B block
        _linear("monarch 3072-768 T=197", "monarch", 3072, 768, 128, 4, 197),
        # a batch of 32 images through a ViT-B width linear of many small blocks
        _linear("blast 768 T=6304", "blast", 768, 768, 96, 16, 6304),
        # a short prompt through the MLP up projection
        _linear("monarch 4096-11008 T=512", "monarch", 4096, 11008, 1024, 4, 512),
        # prompts of no round length through an attention projection, plain low-rank and BLAST
        _linear("lowrank 4096 T=1000", "lowrank", 4096, 4096, 1024, 1, 1000),
        _linear("blast 4096 T=1000", "blast", 4096, 4096, 640, 16, 1000),
        # a long prompt (or a batch of them) through the MLP up and the MLP down projection
        _linear("monarch 4096-11008 T=8192", "monarch", 4096, 11008, 1024, 4, 8192),
        _linear("blast 11008-4096 T=8192", "blast", 11008, 4096, 1024, 16, 8192),
        # one decoded token through all linears of a 16-layer model
        {"name": "chain blast T=1", "op": "chain", "kind": "blast", "layers": 16, "T": 1},
        # a prompt through all linears of a 16-layer model
        {"name": "chain monarch T=2048", "op": "chain", "kind": "monarch", "layers": 16, "T": 2048},
    ]


def _tokens(rng, most):
    return max(1, min(most, int(round(math.exp(rng.uniform(0.0, math.log(most)))))))


def draw(rng):
    what = rng.random()
    if what < 0.15:                                      # a chain of some layers
        kind = rng.choice(("monarch", "blast"))
        return {"op": "chain", "kind": kind, "layers": rng.randint(1, 16), "T": _tokens(rng, 2048 if kind == "monarch" else 1024)}
    if what < 0.25:                                      # a small layer in full precision
        n_in, n_out = 64 * rng.randint(4, 16), 64 * rng.randint(4, 16)
        c = _linear("", "monarch", n_in, n_out, 16 * rng.randint(2, 16), 4, _tokens(rng, 512), "f32")
    else:                                                # one of the layers, at its rank or a lower one
        op, n_in, n_out, r, b = rng.choice(LAYERS)
        unit = 8 * b if op == "monarch" else 8
        c = _linear("", op, n_in, n_out, max(unit, r - unit * rng.randint(0, r // (2 * unit))), b, _tokens(rng, MAX_T))
    del c["name"]
    return c


def _normal(gen, shape, scale, dtype):
    return (torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32) * scale).to(dtype)


def _factor_shapes(op, n_in, n_out, r, b):
    """name -> (shape, scale): i.i.d. N(0, 1) entries scaled so that activations keep their size."""
    if op == "monarch":
        return {"R": ((b, r, n_in // b), (n_in / b) ** -0.5), "L": ((b, n_out // b, r), r ** -0.5)}
    if op == "lowrank":
        return {"V": ((r, n_in), n_in ** -0.5), "U": ((n_out, r), r ** -0.5)}
    return {"U": ((b, n_out // b, r), r ** -0.5), "S": ((b, b, r), r ** -0.5), "V": ((b, n_in // b, r), r ** -0.5)}


def _chain_shape(kind, name):
    n_in, n_out = (HIDDEN, MLP) if name in ("gate", "up") else (MLP, HIDDEN) if name == "down" else (HIDDEN, HIDDEN)
    c = CHAIN[kind]
    return n_in, n_out, c["r_square"] if n_in == n_out else c["r_mlp"], c["b"]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = types.SimpleNamespace(op=case["op"])
    T = case["T"]
    if s.op == "chain":
        # DeviceChain takes the factors as host tensors, as a checkpoint holds them
        kind = case["kind"]
        layers = []
        for _ in range(case["layers"]):
            layer = {}
            for name in LINEARS:
                n_in, n_out, r, b = _chain_shape(kind, name)
                lin = types.SimpleNamespace(n_in=n_in, n_out=n_out, r=r, dtype="bf16", **{"nblocks" if kind == "monarch" else "b": b})
                for key, (shape, scale) in _factor_shapes(kind, n_in, n_out, r, b).items():
                    bits = _normal(gen, shape, scale, torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
                    setattr(lin, key, types.SimpleNamespace(dtype="bf16", bits=bits))
                layer[name] = lin
            layers.append(layer)
        s.chain = DeviceChain(layers, T)
        s.x = _normal(gen, (T, HIDDEN), 1.0, torch.bfloat16)
        return s
    n_in, n_out, s.r, s.b = case["n_in"], case["n_out"], case["r"], case["b"]
    td, dt = (torch.bfloat16, B.BF16) if case["dtype"] == "bf16" else (torch.float32, B.F32)
    for key, (shape, scale) in _factor_shapes(s.op, n_in, n_out, s.r, s.b).items():
        setattr(s, key, _normal(gen, shape, scale, td))
    s.X = _normal(gen, (T, n_in), 1.0, td)
    s.Y = torch.empty((T, n_out), dtype=td, device="cuda")
    if s.op == "monarch":
        need = B.monarch_workspace_bytes(T, n_in, n_out, s.b, s.r, dt)
    elif s.op == "lowrank":
        need = B.lowrank_workspace_bytes(T, n_in, n_out, s.r, dt)
    else:
        s.packed = B.blast_pack(s.U, s.S, s.V, n_in, n_out, s.b, s.r)
        need = B.blast_workspace_bytes(T, n_in, n_out, s.b, s.r, dt, B.BLAST_PACKED)
    s.ws = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    if s.op == "chain":
        return s.chain.forward(s.x)
    if s.op == "monarch":
        return B.monarch_forward(s.X, s.R, s.L, s.Y, s.b, s.r, workspace=s.ws)
    if s.op == "lowrank":
        return B.lowrank_forward(s.X, s.V, s.U, s.Y, workspace=s.ws)
    return B.blast_forward(s.X, s.U, None, s.packed, s.Y, s.b, s.r, B.BLAST_PACKED, workspace=s.ws)


def _params(op, n_in, n_out, r, b):
    return r * (n_in + n_out + (b * b if op == "blast" else 0))


def work(case):
    """Inputs, factors and outputs once each; two operations per factor element and token."""
    T = case["T"]
    if case["op"] == "chain":
        n = case["layers"] * sum(_params(case["kind"], *_chain_shape(case["kind"], name)) for name in LINEARS)
        return {"bytes": 2 * (2 * T * HIDDEN + n), "flops": 2 * T * n}
    n = _params(case["op"], case["n_in"], case["n_out"], case["r"], case["b"])
    return {"bytes": (2 if case["dtype"] == "bf16" else 4) * (T * (case["n_in"] + case["n_out"]) + n), "flops": 2 * T * n}


def tolerance(case):
    """bf16 rounds each stored value to 2^-9 of it, two intermediates and the output of a linear; 16 layers of a chain
    round the residual stream some thirty times. f32: 32-bit sums."""
    if case["op"] == "chain":
        return {"rel": 2e-2}
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}

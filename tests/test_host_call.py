"""The native forward callables of the binding against its Python marshaller: the same results however the arguments
are passed, and the marshaller's own errors for calls that do not fit."""
import pytest

torch = pytest.importorskip("torch")
from paper_2512_20861_amd import binding as B  # noqa: E402


def test_malformed_calls_raise_what_the_marshaller_raises():
    B.lib()
    x = torch.zeros(4, 8)
    for fn, args in ((B.monarch_forward, (x, x, x, x, 4, 8)), (B.lowrank_forward, (x, x, x, x)), (B.blast_forward, (x, x, x, x, x, 2, 8)),
                     (B.dense_reference_forward, (x, x, x)), (B.monarch_rect_forward, (x, x, x, x, 2, 2, 2)), (B.blast_group_forward, (x, x, x, x, 2, 8, 2))):
        with pytest.raises(Exception) as got:
            fn(*args)
        with pytest.raises(Exception) as want:
            fn.marshal(*args)
        assert (type(got.value), str(got.value)) == (type(want.value), str(want.value))
        with pytest.raises(TypeError):
            fn(x, no_such_argument=1)
        with pytest.raises(TypeError):
            fn(*args, X=x)
        assert fn.__name__ in fn.marshal.__name__ and fn.__doc__ == fn.marshal.__doc__


@pytest.mark.gpu
@pytest.mark.parametrize("T", [1, 33])
def test_argument_forms_agree(T):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert B._host is not None, "the native callables are not built"
    g = torch.Generator(device="cuda").manual_seed(T)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    X, R, L = rand(T, 256), rand(4, 64, 64), rand(4, 80, 64)
    want, Y = torch.zeros((T, 320), dtype=torch.bfloat16, device="cuda"), torch.zeros((T, 320), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(B.monarch_workspace_bytes(T, 256, 320, 4, 64, B.BF16), dtype=torch.uint8, device="cuda")
    B.prepared(B.monarch_forward, X, R, L, want, 4, 64, 0, ws)()
    forms = [lambda: B.monarch_forward(X, R, L, Y, 4, 64), lambda: B.monarch_forward(X, R, L, Y, 4, 64, 0, ws),
             lambda: B.monarch_forward(X, R, L, Y=Y, r=64, nblocks=4, workspace=ws),
             lambda: B.monarch_forward(X, R, L, Y, 4, 64, workspace=ws, stream=torch.cuda.current_stream())]
    for call in forms:
        Y.zero_()
        assert call() is Y and torch.equal(Y, want)
    side = torch.cuda.Stream()                           # the stream that is current at the call
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        Y.zero_()
        B.monarch_forward(X, R, L, Y, 4, 64, workspace=ws)
    side.synchronize()
    assert torch.equal(Y, want)
    with pytest.raises(B.BlrError) as e:                 # an error code of the library
        B.monarch_forward(X, R, L, Y, 4, 64, workspace=ws[:16])
    assert e.value.status == B.ERR_WORKSPACE
    with pytest.raises(ValueError):
        B.monarch_forward(X, R, L[:, :40], Y, 4, 64, workspace=ws)


def _entries(T):
    """name -> (function, arguments with an explicit workspace, positions of the tensors that carry data)"""
    g = torch.Generator(device="cuda").manual_seed(T)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    space = lambda n: torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    X, Y = rand(T, 256), rand(T, 320)
    U, S, V = rand(4, 80, 136), rand(4, 4, 136), rand(4, 64, 136)
    Ug, Sg, Vg, Yg = rand(2, 4, 80, 136), rand(4, 4, 272), rand(4, 64, 272), rand(T, 640)
    packed, grouped = B.blast_pack(U, S, V, 256, 320, 4, 136), B.blast_pack(Ug, Sg, Vg, 256, 320, 4, 272)
    R, L = rand(4, 64, 64), rand(4, 80, 64)
    mono = space(B.monarch_workspace_bytes(T, 256, 320, 4, 64, B.BF16))
    return {
        "monarch": (B.monarch_forward, (X, R, L, Y, 4, 64, 0, mono), (0, 1, 2, 3)),
        "monarch_static": (B.monarch_forward_static, (X, R, L, Y, 4, 64, 0), (0, 1, 2, 3)),
        "monarch_rect": (B.monarch_rect_forward, (X, rand(4, 80, 64), rand(5, 64, 64), Y, 4, 5, 16, 0,
                                                  space(B.monarch_rect_workspace_bytes(T, 256, 320, 4, 5, 16, B.BF16))), (0, 1, 2, 3)),
        "lowrank": (B.lowrank_forward, (X, rand(72, 256), rand(320, 72), Y, 0, space(B.lowrank_workspace_bytes(T, 256, 320, 72, B.BF16))), (0, 1, 2, 3)),
        "blast": (B.blast_forward, (X, U, S, V, Y, 4, 136, 0, space(B.blast_workspace_bytes(T, 256, 320, 4, 136, B.BF16, 0))), (0, 1, 2, 3, 4)),
        "blast packed": (B.blast_forward, (X, U, None, packed, Y, 4, 136, B.BLAST_PACKED,
                                           space(B.blast_workspace_bytes(T, 256, 320, 4, 136, B.BF16, B.BLAST_PACKED))), (0, 1, 3, 4)),
        "blast_group": (B.blast_group_forward, (X, Ug, grouped, Yg, 4, 136, 2, 0,
                                                space(B.blast_group_workspace_bytes(T, 256, 320, 4, 136, 2, B.BF16))), (0, 1, 2, 3)),
        "dense": (B.dense_reference_forward, (X, rand(320, 256), Y), (0, 1, 2)),
    }


@pytest.mark.gpu
@pytest.mark.parametrize("T", [2, 33])
@pytest.mark.parametrize("name", ["monarch", "monarch_static", "monarch_rect", "lowrank", "blast", "blast packed", "blast_group", "dense"])
def test_native_checks(name, T):
    """Every native entry: a well-formed call is the marshaller's; with one tensor of another shape, type, layout or device, a
    short packed buffer or a short workspace it raises what the marshaller (or the library) says, before anything is launched."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert B._host is not None, "the native callables are not built"
    fn, args, tensors = _entries(T)[name]
    out = next(a for a in args if a is fn.marshal(*args)[2])
    B.prepared(fn, *args)()
    torch.cuda.synchronize()
    want = out.clone()
    out.fill_(float("nan"))
    assert fn(*args) is out
    torch.cuda.synchronize()
    assert torch.equal(out, want)

    def refused(bad):
        with pytest.raises(Exception) as e:
            fn.marshal(*bad)
        with pytest.raises(type(e.value)) as got:
            fn(*bad)
        assert str(got.value) == str(e.value)

    out.fill_(7.0)
    for i in tensors:
        t = args[i]
        put = lambda other: args[:i] + (other,) + args[i + 1:]
        if i > 0 or "packed" not in name and "group" not in name:             # (a packed buffer may be larger than its layer needs)
            refused(put(t[..., :-8].contiguous()))       # another size (a packed buffer: too short)
        refused(put(t[:-1] if t.dim() > 1 and t.shape[0] > 1 else t[:-16]))
        refused(put(t.float()))
        refused(put(torch.stack((t, t), dim=-1)[..., 0]))                     # the shape is right, the elements lie apart
        refused(put(t.cpu()))
        refused(put(None))
    if isinstance(args[-1], torch.Tensor) and args[-1].dtype == torch.uint8:
        with pytest.raises(B.BlrError) as e:
            fn(*args[:-1], args[-1][:-256])
        assert e.value.status == B.ERR_WORKSPACE
        with pytest.raises(ValueError):
            fn(*args[:-1], args[-1].view(torch.int8))
    torch.cuda.synchronize()
    assert (out == 7.0).all()                            # nothing was launched


def test_build_command_with_a_bare_compiler_name(monkeypatch):
    import os
    import shutil
    from paper_2512_20861_amd import build
    if not shutil.which("hipcc"):
        pytest.skip("no hipcc on the path")
    monkeypatch.setattr(build, "HIPCC", "hipcc")
    command = build._host_command()
    dirs = [command[i + 1] for i, a in enumerate(command) if a == "-isystem"]
    assert all(os.path.isabs(d) for d in dirs) and any(os.path.exists(os.path.join(d, "hip", "hip_runtime.h")) for d in dirs)


def test_callables_behave_as_functions_do():
    import copy
    import inspect
    import weakref
    for fn in (B.monarch_forward, B.blast_forward, B.silu_mul):
        assert copy.copy(fn) is fn and copy.deepcopy([fn])[0] is fn and weakref.ref(fn)() is fn
        assert inspect.signature(fn).parameters


def test_snapshot_tells_what_was_replaced():
    """unchanged() until one of the ways to put another tensor, address, layout or number in a part's place."""
    B.lib()

    class Part:
        def __init__(self):
            self.w, self.n = torch.arange(24.0).reshape(4, 6), 1024

    parts, eps, kept = [Part(), Part()], 0.5, []
    row = B.snapshot((*parts, eps), kept)
    same = lambda: B.unchanged((*parts, eps), row)
    assert all(same() for _ in range(20))
    part, w, n = parts[0], parts[0].w, parts[0].n
    data, other = w.data, parts[1]
    assert any(o is w for o in kept)

    def change_and_back():
        part.w = w.clone(); yield
        part.w = w; yield
        w.data = w.clone(); yield                        # the same tensor object
        w.data = data; yield
        w.t_(); yield
        w.t_(); yield
        part.n = n + 1; yield
        part.n = n; yield
        parts[1] = Part(); yield
        parts[1] = other; yield
        parts.append(w); yield
        parts.pop(); yield
    assert [same() for _ in change_and_back()] == [False, True] * 6
    w.add_(1.0)
    assert same()                                        # values are not looked at
    assert not B.unchanged((*parts, n), row) and not B.unchanged((*parts,), row)
    with pytest.raises(TypeError):
        B.snapshot(parts, [])

"""Single-tensor calls through the binding's C++ checks against the same calls through ctypes: results, errors, and which way is taken."""
import pytest
import torch

srs = pytest.importorskip("paper_2605_07330_amd.srs")

pytestmark = pytest.mark.gpu

N, BE = 5000, 1500
NB = 4


def _payload(width, cap=BE, nb=NB, dtype=torch.int32):
    V = torch.full((nb, cap), -1, dtype={1: torch.int8, 2: torch.int16}[width], device="cuda")
    return torch.full((nb, cap), -1, dtype=dtype, device="cuda"), V, torch.full((nb,), 7, dtype=torch.int32, device="cuda")


def _tensors(kind, seed=1):
    g = torch.Generator().manual_seed(seed)
    if kind == "u8":
        a = torch.randint(0, 255, (N,), generator=g, dtype=torch.int32).to(torch.uint8)
        b = a.clone()
    else:
        a = torch.randn(N, generator=g).to(torch.bfloat16)
        b = a.clone().float() if kind == "cast" else a.clone()
    pos = torch.randperm(N, generator=g)[: N // 9]
    b[pos] = 3
    return a.cuda(), b.cuda()


def _extract(ctx, kind):
    return {"bf16": ctx.extract, "u8": ctx.extract_u8, "cast": ctx.extract_cast}[kind]


def _apply(ctx, kind):
    return ctx.apply_u8 if kind == "u8" else ctx.apply


def _arguments(kind, form):
    """(taken in C++, old, new, bucket size, I, V, counts, cap) of one form of the call."""
    a, b = _tensors(kind)
    w = 1 if kind == "u8" else 2
    I, V, c = _payload(w)
    be = cap = BE
    native = True
    if form == "shaped":
        a, b = a.view(50, 100), b.view(50, 100)
    elif form == "parameter":
        b = torch.nn.Parameter(b, requires_grad=False)
    elif form == "offset":
        a, b = a[1:], b[1:]
    elif form == "strided":
        native, a = False, a[::2]
    elif form == "width":
        native, b = False, b.double()
    elif form == "host":
        native, b = False, b.cpu()
    elif form == "sizes":
        native, b = False, b[:-1]
    elif form == "short_I":
        native, I = False, I[:-1]
    elif form == "short_V":
        native, V = False, V.view(-1)[:-1]
    elif form == "short_counts":
        native, c = False, c[:-1]
    elif form == "type_I":
        native, I = False, I.view(torch.float32)
    elif form == "zero_bucket":
        native, be = False, 0
    elif form == "zero_cap":
        native, cap = False, 0
    elif form == "subclass":
        class Sub(torch.Tensor):
            pass
        native, a = False, a.as_subclass(Sub)
    elif form == "empty":
        a, b = a[:0], b[:0]
    return native, a, b, be, I, V, c, cap


FORMS = ["plain", "shaped", "parameter", "offset", "strided", "width", "host", "sizes", "short_I", "short_V", "short_counts", "type_I", "zero_bucket",
         "zero_cap", "subclass", "empty"]


def _outcome(kind, form, call, monkeypatch):
    ctx = srs.Context(0)
    native, a, b, be, I, V, c, cap = _arguments(kind, form)
    back = a.clone()
    taken = []
    if call is not None:
        class Spy:
            @staticmethod
            def extract(*args):
                taken.append(call.extract(*args))
                return taken[-1]

            @staticmethod
            def apply(*args):
                taken.append(call.apply(*args))
                return taken[-1]
        monkeypatch.setattr(srs, "_call", Spy)
    else:
        monkeypatch.setattr(srs, "_call", None)
    errors = []
    for f, args in ((_extract(ctx, kind), (a, b)), (_apply(ctx, kind), (back,))):
        try:
            f(*args, be, I, V, c, cap)
            errors.append(None)
        except Exception as e:      # noqa: BLE001 - the kind and the text are what is compared
            errors.append((type(e), str(e)))
    flags = ctx.status()
    ctx.close()
    return native, [t is not None for t in taken], errors, flags, [t.detach().as_subclass(torch.Tensor).cpu() for t in (a, back, I, V, c)]


@pytest.mark.parametrize("kind", ["bf16", "u8", "cast"])
@pytest.mark.parametrize("form", FORMS)
def test_same_as_through_ctypes(kind, form, monkeypatch):
    call = srs._call
    assert call is not None, "_call is not built: python -m paper_2605_07330_amd.build"
    native, taken, errors, flags, got = _outcome(kind, form, call, monkeypatch)
    _, _, want_errors, want_flags, want = _outcome(kind, form, None, monkeypatch)
    # apply goes its own way: it takes no new weights, and a clone of strided ones is contiguous
    assert taken == [native, native or form in ("strided", "width", "host", "sizes")]
    assert errors == want_errors and flags == want_flags
    for g, w in zip(got, want):
        assert g.shape == w.shape and torch.equal(g.contiguous().view(torch.uint8), w.contiguous().view(torch.uint8))


def test_streams_and_a_closed_context():
    ctx = srs.Context(0)
    a, b = _tensors("bf16")
    I, V, c = _payload(2)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    ctx.extract(a, b, BE, I, V, c, BE, stream=s)
    s.synchronize()
    assert int(c.sum()) == int((_tensors("bf16")[0] != _tensors("bf16")[1]).sum()) and torch.equal(a, b)
    assert ctx.status(s) == 0
    ctx.close()
    with pytest.raises(srs.SrsError):
        ctx.extract(a, b, BE, I, V, c, BE)

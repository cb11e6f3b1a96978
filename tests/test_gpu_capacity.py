"""Capacities that cannot be: negative ones, which ctypes would hand on as 2^64 - k, and ones beyond what buckets can be addressed with.
All are refused before anything is launched; with one bucket a capacity of 2^64 - 1 is the caller's word that every pair fits."""
import ctypes as C

import pytest
import torch

srs = pytest.importorskip("paper_2605_07330_amd.srs")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N, BE, NB, CAP = 5000, 1500, 4, 64


class Case:
    def __init__(self):
        self.ctx = srs.Context(0)
        self.plan = self.ctx.plan([N - 7, 7], BE)
        i32 = lambda n: torch.full((n,), -1, dtype=torch.int32, device=DEV)  # noqa: E731
        i16 = lambda n: torch.full((n,), -1, dtype=torch.int16, device=DEV)  # noqa: E731
        self.a, self.b = i16(N), torch.zeros(N, dtype=torch.int16, device=DEV)
        self.a8, self.b8 = self.a[: N // 2].view(torch.uint8), self.b[: N // 2].view(torch.uint8)
        self.f = torch.zeros(N, device=DEV)
        self.I, self.V, self.V8, self.counts = i32(NB * CAP), i16(NB * CAP), i16(NB * CAP).view(torch.uint8), i32(NB)
        self.counts.zero_()
        self.D, self.max_gap, self.anchors = srs.alloc_encoded(NB, CAP, DEV)
        self.enc = srs.alloc_value_stream(NB, CAP, DEV)
        self.bits = torch.zeros(srs.bitmap_words(N), dtype=torch.int32, device=DEV)
        self.more = [i32(NB * CAP) for _ in range(4)]
        self.one = i32(1)

    def parts(self, x):
        return list(torch.split(x, [N - 7, 7]))

    def calls(self, cap):
        c, p, pay, pay8 = self.ctx, self.plan, (self.I, self.V, self.counts), (self.I, self.V8, self.counts)
        coded = (self.D, self.I, self.V, self.counts, self.max_gap, self.anchors)
        parts8 = [torch.zeros(n, dtype=torch.uint8, device=DEV) for n in (N - 7, 7)]
        return {
            "extract": lambda: c.extract(self.a, self.b, BE, *pay, cap), "extract_noalloc": lambda: c.extract_noalloc(self.a, self.b, BE, *pay, cap),
            "extract_u8": lambda: c.extract_u8(self.a8, self.b8, BE, *pay8, cap), "extract_cast": lambda: c.extract_cast(self.a, self.f, BE, *pay, cap),
            "apply": lambda: c.apply(self.a, BE, *pay, cap), "apply_u8": lambda: c.apply_u8(self.a8, BE, *pay8, cap),
            "extract_multi": lambda: c.extract_multi(p, self.parts(self.a), self.parts(self.b), *pay, cap),
            "extract_multi_u8": lambda: c.extract_multi_u8(p, parts8, [x.clone() for x in parts8], *pay8, cap),
            "extract_cast_multi": lambda: c.extract_cast_multi(p, self.parts(self.a), self.parts(self.f), *pay, cap),
            "extract_marked_multi": lambda: c.extract_marked_multi(p, self.parts(self.b), self.bits, *pay, cap),
            "apply_multi": lambda: c.apply_multi(p, self.parts(self.a), *pay, cap), "apply_multi_u8": lambda: c.apply_multi_u8(p, parts8, *pay8, cap),
            "tensor_indices": lambda: c.tensor_indices(p, self.I, self.counts, cap, self.more[0], self.more[1]),
            "encode_indices": lambda: c.encode_indices(self.I, self.counts, NB, cap, 0, self.D, self.max_gap, self.anchors),
            "apply_encoded": lambda: c.apply_encoded(self.a, BE, *coded, cap), "apply_multi_encoded": lambda: c.apply_multi_encoded(p, self.parts(self.a), *coded, cap),
            "encode_values": lambda: c.encode_values(self.V, self.counts, NB, cap, self.enc),
            "decode_values": lambda: c.decode_values(self.enc, self.counts, NB, cap, self.V),
            "route": lambda: c.route(self.counts, NB, BE, N, cap, 6, NB, self.more[0], self.more[1], self.more[2], self.one),
        }


@pytest.mark.parametrize("cap", [-1, -8, -(1 << 40), -(1 << 63)])
def test_negative_capacities(cap):
    case = Case()
    kept = [x.clone() for x in (case.a, case.I, case.V, case.D)]
    for name, call in case.calls(cap).items():
        with pytest.raises((srs.SrsError, TypeError)) as e:
            call()
        assert getattr(e.value, "code", srs.ERR_INVALID) == srs.ERR_INVALID, name
    assert case.ctx.status() == 0
    assert all(torch.equal(x, k) for x, k in zip((case.a, case.I, case.V, case.D), kept))
    case.ctx.close()


@pytest.mark.parametrize("cap", [(1 << 58) + 1, (1 << 62) + 3, (1 << 64) - 1])
def test_capacities_beyond_the_address_space(cap):
    case, lib = Case(), srs._lib
    c, p = case.ctx._h, case.plan._h
    ptr = {k: getattr(case, k).data_ptr() for k in ("a", "b", "f", "I", "V", "counts", "D", "max_gap", "anchors")}
    pay = (ptr["I"], ptr["V"], ptr["counts"], cap, None)
    pairs = case.ctx.bind_pairs(case.plan, case.parts(case.a), case.parts(case.b))
    weights = case.ctx.bind_weights(case.plan, case.parts(case.a))
    coded = (ptr["D"], ptr["I"], ptr["V"], ptr["counts"], ptr["max_gap"], ptr["anchors"], cap, None)
    for name, rc in {
        "extract": lib.srs_extract(c, ptr["a"], ptr["b"], N, BE, *pay), "noalloc": lib.srs_extract_noalloc(c, ptr["a"], ptr["b"], N, BE, *pay),
        "cast": lib.srs_extract_cast(c, ptr["a"], ptr["f"], N, BE, *pay), "apply": lib.srs_apply(c, ptr["a"], N, BE, *pay),
        "extract_multi": lib.srs_extract_multi(c, p, pairs, *pay), "apply_multi": lib.srs_apply_multi(c, p, weights, *pay),
        "tensor_indices": lib.srs_tensor_indices(c, p, ptr["I"], ptr["counts"], cap, ptr["I"], ptr["I"], None),
        "encode": lib.srs_encode_indices(c, ptr["I"], ptr["counts"], NB, cap, 0, ptr["D"], ptr["max_gap"], ptr["anchors"], None),
        "apply_encoded": lib.srs_apply_encoded(c, ptr["a"], N, BE, *coded), "apply_multi_encoded": lib.srs_apply_multi_encoded(c, p, weights, *coded),
    }.items():
        assert rc == srs.ERR_INVALID, name
    case.ctx.close()


def test_one_bucket_takes_any_capacity():
    case, lib = Case(), srs._lib
    I, V, counts = srs.alloc_payload(1, N, DEV)
    back = case.a.clone()
    assert lib.srs_extract(case.ctx._h, case.a.data_ptr(), case.b.data_ptr(), N, N, I.data_ptr(), V.data_ptr(), counts.data_ptr(), C.c_uint64(-1), None) == 0
    assert lib.srs_apply(case.ctx._h, back.data_ptr(), N, N, I.data_ptr(), V.data_ptr(), counts.data_ptr(), C.c_uint64(-1), None) == 0
    assert case.ctx.status() == 0 and int(counts[0]) == N and torch.equal(back, case.b)
    case.ctx.close()

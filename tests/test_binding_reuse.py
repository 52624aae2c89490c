"""Output lists given to the binding again after their entries, or those of the input lists, were replaced:
what reaches the C entry point is what the lists hold at the call.  Output tensors that the binding makes have
memory of their own.  The library is a stand-in that records
its arguments (host memory only, no device)."""
import ctypes as C
from collections import deque

import pytest
import torch

from paper_2306_11800_amd import api


class Recorder:
    """inshr_delta and inshr_delta_bound; the arguments of the last delta as plain numbers."""

    def inshr_delta_bound(self, p, c, words):
        p, c = p._obj, c._obj
        words._obj.value = (p.n * max(p.sym_bits, c.sym_bits) + 63) // 64
        return 0

    def inshr_reconstruct(self, h, pa, da, ca, n):
        self.words = [(x.packed, x.packed_words, x.bins) for x in ca]
        return 0

    def inshr_dequantize(self, h, ia, oa, n):
        self.out = list(oa)
        return 0

    def inshr_delta(self, h, pa, pp, ca, oa, n):
        self.codes = [[(x.packed, x.sym_bits, x.bins, x.n) for x in e] for e in (pa, ca)]
        self.out = [(x.packed, x.packed_words, x.group_off, x.group_off_entries, x.perm) for x in oa]
        for p, c, o in zip(pa, ca, oa):
            o.delta_bits = max(p.sym_bits, c.sym_bits)
        return 0


def context():
    ctx = api.Context.__new__(api.Context)
    ctx.lib, ctx.h, ctx._bounds = Recorder(), None, {}
    ctx._check = lambda rc: None
    return ctx


def codes(n, K):
    f = torch.zeros(256)
    return api.Quantized(n, 8, (torch.zeros((n * 9 + 63) // 64, dtype=torch.int64), f, f, f.int(), f), bins=K)


def check(ctx, prev, cur, out):
    for got, qs in zip(ctx.lib.codes, (prev, cur)):
        assert got == [(q._bufs[0].data_ptr(), q.sym_bits, q.K, q.n) for q in qs]
    assert ctx.lib.out == [(d.packed.data_ptr(), d.packed.numel(), d.goff_buf.data_ptr(), d.goff_buf.numel(),
                            None if d.perm is None else d.perm.data_ptr()) for d in out]
    for d, p, c in zip(out, prev, cur):
        assert d.n == p.n and d.delta_bits == max(p.sym_bits, c.sym_bits)
        assert d.group_off.data_ptr() == d.goff_buf.data_ptr() and d.group_off.numel() == p.K + 3


@pytest.mark.parametrize("n_t", [1, 3, 12])  # (arrays are filled in another way above eight tensors)
@pytest.mark.parametrize("want_perm", [False, True])
def test_delta_follows_the_lists(n_t, want_perm):
    ctx = context()
    prev, cur = [codes(1000 + i, 16) for i in range(n_t)], [codes(1000 + i, 12) for i in range(n_t)]
    out = ctx.delta(prev, cur)
    check(ctx, prev, cur, out)
    for d in out:  # room for any symbols
        d.packed = torch.zeros(1000, dtype=torch.int64)
    if want_perm:
        for d in out:
            d.perm = torch.zeros(2000, dtype=torch.int32)

    def again():
        nonlocal out
        out = ctx.delta(prev, cur, want_perm=want_perm, out=out)
        check(ctx, prev, cur, out)

    again()
    prev[:], cur[:] = cur[:], prev[:]  # entries swapped inside the same lists
    again()
    cur[0] = codes(cur[0].n, 256)  # one entry replaced by codes of wider symbols
    again()
    prev[-1], cur[-1] = codes(1500, 3), codes(1500, 4)  # and by codes of another size
    again()
    out[0].packed, out[-1].goff_buf = torch.zeros(900, dtype=torch.int64), torch.zeros(264, dtype=torch.int64)
    again()
    out[0].goff_buf, out[0].perm = torch.zeros(300, dtype=torch.int64), None
    again()
    out[-1] = api.Delta(n=0, delta_bits=0, packed=torch.zeros(800, dtype=torch.int64), group_off=None, perm=None,
                        goff_buf=torch.zeros(264, dtype=torch.int64))
    again()
    other_prev = [codes(q.n, 6) for q in prev]  # other lists altogether
    out = ctx.delta(other_prev, cur, want_perm=want_perm, out=out)
    check(ctx, other_prev, cur, out)
    for kept, name in ((out[0].packed, "packed"), (None, "perm")):  # too small: refused
        setattr(out[0], name, torch.zeros(3, dtype=torch.int64 if name == "packed" else torch.int32))
        with pytest.raises(ValueError):
            ctx.delta(prev, cur, want_perm=want_perm, out=out)
        setattr(out[0], name, kept)
    again()


@pytest.mark.parametrize("n_t", [1, 4, 12])
def test_reconstructed_tensors_are_their_own(n_t):
    ctx = context()
    prev = [codes(1000 + 4096 * i, 16) for i in range(n_t)]
    out = ctx.delta(prev, prev)
    res = ctx.reconstruct(prev, out, [4] * n_t)
    assert ctx.lib.words == [(x.data_ptr(), x.numel(), 16) for x in res]
    for x, p in zip(res, prev):  # nothing else stays allocated with one of them, or is saved with it
        assert x.numel() == (p.n * 5 + 63) // 64 and x.storage_offset() == 0
        assert x.untyped_storage().nbytes() == 8 * x.numel()


@pytest.mark.parametrize("kind", [list, tuple, deque, lambda x: dict(enumerate(x))])
def test_dequantize_takes_any_outputs_by_index(kind):
    ctx = context()
    q = [codes(1000 + i, 16) for i in range(3)]
    out = [torch.zeros(1000 + i) for i in range(4)]  # (more than needed)
    res = ctx.dequantize(q, kind(out))
    assert all(a is b for a, b in zip(res, out)) and ctx.lib.out == [x.data_ptr() for x in out[:3]]

"""Delta and its inverse on codes made from symbols: every pair of symbol widths, with and without the
permutation, tiles that end anywhere, groups of one element, and one group that holds nearly everything
(its run fills whole tiles, the others are a few bits of a word)."""
import numpy as np
import pytest
import torch

from oracle import ref
from test_gpu_parity import dev, u32, u64

pytestmark = pytest.mark.gpu

BINS = [2, 3, 6, 8, 16, 32, 64, 128, 256]  # symbols of 2 (K = 2) to 9 bits
SIZES = [1, 63, 12287, 12288, 12289, 3 * 12288 + 31, 200_003]


def codes(sym, K):
    from paper_2306_11800_amd import api
    w = api.symbol_bits(K)
    f = torch.zeros(256, device="cuda:0")
    return api.Quantized(sym.size, 8, (dev(ref.pack(sym, w).view(np.int64)), f, f, f.int(), f), bins=K)


def symbols(rng, n, K, shape):
    s = rng.integers(0, K + 2, n)
    if shape == "skewed":  # one value nearly everywhere, and every value somewhere
        s = np.where(rng.random(n) < 0.995, K // 2, s)
        s[:min(n, K + 2)] = rng.permutation(K + 2)[:min(n, K + 2)]
    return s.astype(np.uint16)


@pytest.mark.parametrize("Kp", BINS)
@pytest.mark.parametrize("ordered", [True, False])
def test_widths(monkeypatch, Kp, ordered):
    from paper_2306_11800_amd import api
    monkeypatch.setenv("INSHR_NO_LDS_ORDER", "0" if ordered else "1")
    ctx = api.Context(torch.device("cuda:0"))
    rng = np.random.default_rng(Kp)
    for Kc in (Kp, 2, 12, 256):
        for shape in ("even", "skewed"):
            sizes = SIZES if ordered else SIZES[3:5]
            sp = [symbols(rng, n, Kp, shape) for n in sizes]
            sc = [symbols(rng, n, Kc, shape) for n in sizes]
            qp, qc = [codes(s, Kp) for s in sp], [codes(s, Kc) for s in sc]
            for perm in (False, True):
                ds = ctx.delta(qp, qc, want_perm=perm)
                ctx.sync()
                for d, a, b in zip(ds, sp, sc):
                    r = ref.delta(a, 0, b, 0, K_prev=Kp, K_cur=Kc)
                    assert d.delta_bits == r["delta_bits"]
                    assert np.array_equal(u64(d.group_off), r["group_off"])
                    assert np.array_equal(u64(d.packed), ref.pack(r["stream"], r["delta_bits"])), (Kp, Kc, a.size, shape)
                    if perm:
                        assert np.array_equal(u32(d.perm), r["perm"])
            back = ctx.reconstruct(qp, ds, [0] * len(qp), [Kc] * len(qp))
            for w, q in zip(back, qc):
                assert torch.equal(w, q.packed), (Kp, Kc, q.n, shape)
    ctx.close()


def test_buffers_and_bins_between_calls():
    """Output lists used again: a permutation buffer brought later, the group offsets after a static call
    with other bins in between; bins_cur alone, and per-tensor lists longer than the call."""
    from paper_2306_11800_amd import api
    ctx = api.Context(torch.device("cuda:0"))
    rng = np.random.default_rng(5)
    for n_t in (3, 12):  # (C arrays are filled in another way above eight tensors)
        sizes = [5000 + 77 * i for i in range(n_t)]
        sp = [symbols(rng, n, 16, "even") for n in sizes]
        sc = [symbols(rng, n, 12, "even") for n in sizes]
        sp0, sc0 = list(sp), list(sc)
        qp, qc = [codes(s, 16) for s in sp], [codes(s, 12) for s in sc]
        ds = ctx.delta(qp, qc)
        want = [ref.delta(a, 0, b, 0, K_prev=16, K_cur=12) for a, b in zip(sp, sc)]
        for d in ds:
            d.perm = torch.full((d.n,), -1, dtype=torch.int32, device="cuda:0")
        assert ctx.delta(qp, qc, want_perm=True, out=ds) is ds
        ctx.sync()
        assert all(np.array_equal(u32(d.perm), r["perm"]) for d, r in zip(ds, want))
        for d in ds:  # other buffers in the same list
            d.goff_buf, d.packed = torch.zeros_like(d.goff_buf), torch.zeros_like(d.packed)
            d.perm = torch.full((d.n,), -1, dtype=torch.int32, device="cuda:0")
        ds = ctx.delta(qp, qc, want_perm=True, out=ds)
        ctx.sync()
        for d, r in zip(ds, want):
            assert np.array_equal(u64(d.group_off), r["group_off"]) and np.array_equal(u32(d.perm), r["perm"])
            assert np.array_equal(u64(d.packed), ref.pack(r["stream"], r["delta_bits"]))
        kept, ds[0].packed = ds[0].packed, ds[0].packed[:-1]
        with pytest.raises(ValueError):
            ctx.delta(qp, qc, want_perm=True, out=ds)
        ds[0].packed = kept
        # entries of the input lists swapped inside the same lists, one replaced by codes of wider symbols;
        # without the permutation asked for, buffers replaced and a permutation buffer taken away
        for d in ds:
            d.packed = torch.zeros((d.n * 9 + 63) // 64, dtype=torch.int64, device="cuda:0")
        wide = symbols(rng, sizes[0], 256, "even")
        for perm in (True, False):
            qp[:], qc[:] = qc[:], qp[:]
            sp, sc = sc, sp
            if perm:
                qc[0], sc[0] = codes(wide, 256), wide
            else:
                ds[0].packed, ds[1].goff_buf = torch.zeros_like(ds[0].packed), torch.zeros_like(ds[1].goff_buf)
                untouched, ds[2].perm = ds[2].perm.fill_(-1), None
            K = [(p.K, c.K) for p, c in zip(qp, qc)]
            ds = ctx.delta(qp, qc, want_perm=perm, out=ds)
            ctx.sync()
            for d, a, b, (Kp, Kc) in zip(ds, sp, sc, K):
                r = ref.delta(a, 0, b, 0, K_prev=Kp, K_cur=Kc)
                assert np.array_equal(u64(d.group_off), r["group_off"])
                assert np.array_equal(u64(d.packed)[:(d.n * d.delta_bits + 63) // 64], ref.pack(r["stream"], r["delta_bits"]))
                if d.perm is not None:
                    assert np.array_equal(u32(d.perm), r["perm"])
        assert bool((untouched == -1).all())
        qp, sp = [codes(s, 16) for s in sp0], sp0
        qc, sc = [codes(s, 12) for s in sc0], sc0
        s4 = [symbols(rng, n, 4, "even") for n in sizes]
        q4 = [codes(s, 4) for s in s4]
        ctx.delta_static(q4, qc, ds)
        assert all(d.group_off.numel() == 7 for d in ds)
        ctx.delta(qp, qc, out=ds)
        ctx.sync()
        assert all(np.array_equal(u64(d.group_off), r["group_off"]) for d, r in zip(ds, want))
        for bits, bins in ((None, [12] * n_t), ([0] * (n_t + 2), [12] * (n_t + 1))):
            back = ctx.reconstruct(qp, ds, bits, bins)
            assert all(torch.equal(w, q.packed) for w, q in zip(back, qc))
        with pytest.raises(IndexError):
            ctx.reconstruct(qp, ds, [4] * (n_t - 1))
    ctx.close()


def test_small_scratch():
    """A limit on the scratch that only long chunks fit: the same streams and symbols."""
    from paper_2306_11800_amd import api
    rng = np.random.default_rng(9)
    sizes = [10_000_001, 12_289, 5]  # (the first alone is 814 tiles, 13 of the longest chunks)
    sp, sc = [symbols(rng, n, 16, "even") for n in sizes], [symbols(rng, n, 12, "skewed") for n in sizes]
    qp, qc = [codes(s, 16) for s in sp], [codes(s, 12) for s in sc]
    ctx, small = api.Context(torch.device("cuda:0")), api.Context(torch.device("cuda:0"), scratch_bytes=32 << 10)
    for perm in (False, True):
        want = ctx.delta(qp, qc, want_perm=perm)
        got = small.delta(qp, qc, want_perm=perm)
        ctx.sync()
        small.sync()
        for a, b in zip(got, want):
            assert torch.equal(a.packed, b.packed) and torch.equal(a.group_off, b.group_off)
            assert not perm or torch.equal(a.perm, b.perm)
    for w, q in zip(small.reconstruct(qp, got, [0] * 3, [12] * 3), qc):
        assert torch.equal(w, q.packed)
    with pytest.raises(api.InshrError) as e:
        api.Context(torch.device("cuda:0"), scratch_bytes=8 << 10).delta(qp, qc)
    assert e.value.code == -4
    ctx.close()
    small.close()


@pytest.mark.parametrize("n", [16 * 12288, 17 * 12288 + 5, 257 * 12288 + 1])
def test_numbers_of_chunks(n):
    """Chunks of one tile: as many as one workgroup takes for a tensor's groups, one more, shares of many."""
    from paper_2306_11800_amd import api
    ctx = api.Context(torch.device("cuda:0"))
    rng = np.random.default_rng(n)
    K = 32
    a, b = (symbols(rng, n, K, "skewed" if n % 2 else "even") for _ in range(2))
    prev, cur = codes(a, K), codes(b, K)
    d = ctx.delta([prev], [cur], want_perm=True)[0]
    ctx.sync()
    order = np.argsort(a, kind="stable")
    assert np.array_equal(u32(d.perm), order)
    assert np.array_equal(u64(d.group_off), np.searchsorted(a[order], np.arange(K + 3)))
    e = (a.astype(np.int64) - b.astype(np.int64)) % (K + 2)
    assert np.array_equal(u64(d.packed), ref.pack(e[order].astype(np.uint16), api.symbol_bits(K)))
    assert torch.equal(ctx.reconstruct([prev], [d], [5], [K])[0], cur.packed)
    ctx.close()


@pytest.mark.parametrize("sizes", [[128 * 12288], [128 * 12288 + 1, 40], [256 * 12288 + 5, 17 * 12288], [5, 12288, 300],
                                   [12289, 16 * 12288, 3, 391 * 12288 + 77, 17 * 12288 + 1]])
def test_parts_of_chunks(sizes):
    """Chunks of one tile around the numbers that make one part, several, none; tensors of one tile alone and beside
    longer ones; offsets that do not match are reported by either way of counting."""
    from paper_2306_11800_amd import api
    ctx = api.Context(torch.device("cuda:0"))
    rng = np.random.default_rng(len(sizes) * 1000 + sizes[0] % 997)
    sp, sc = ([symbols(rng, n, 256, "even") for n in sizes] for _ in range(2))
    qp, qc = [codes(s, 256) for s in sp], [codes(s, 256) for s in sc]
    ds = ctx.delta(qp, qc, want_perm=True)
    ctx.sync()
    for d, a, b in zip(ds, sp, sc):
        r = ref.delta(a, 0, b, 0, K_prev=256, K_cur=256)
        assert np.array_equal(u64(d.group_off), r["group_off"])
        assert np.array_equal(u64(d.packed), ref.pack(r["stream"], r["delta_bits"]))
        assert np.array_equal(u32(d.perm), r["perm"])
    for w, q in zip(ctx.reconstruct(qp, ds, [0] * len(qp), [256] * len(qp)), qc):
        assert torch.equal(w, q.packed)
    for t in range(len(sizes)):
        ds[t].group_off[257] += 1
        with pytest.raises(api.InshrError) as e:
            ctx.reconstruct(qp, ds, [0] * len(qp), [256] * len(qp))
        assert e.value.code == -5
        ds[t].group_off[257] -= 1
    ctx.close()

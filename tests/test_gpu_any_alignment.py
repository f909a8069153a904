"""GPU parity of the kernels that take rows starting at any element and of any
length, at the edges of their register and vector layouts: operands at
different distances from a 16-byte boundary, odd row strides, lengths just
below, at and above a whole number of vectors or of workgroups. Expected
values from the oracle, tolerances of tests/parity.py."""
from fractions import Fraction
from math import isqrt

import numpy as np
import pytest
import torch

from oracle import numerics as nm
from oracle import ops as O
from oracle import selection as S
from tests.parity import check
import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture
def cache():
    import paper_2609_37241_amd as tri
    c = tri.SpecCache()
    yield c
    torch.cuda.synchronize()
    c.close()


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def put(a, dtype, off, pad):
    """[T, ...] host array on the device, `off` elements past a 256-byte
    boundary, rows `pad` elements longer than their contents."""
    src = wl.to_torch(a, dtype, DEV)
    T, W = src.shape[0], int(np.prod(src.shape[1:]))
    buf = torch.full((off + T * (W + pad),), 7, dtype=src.dtype, device=DEV)
    inner = tuple(int(np.prod(src.shape[i + 1:])) for i in range(1, src.dim()))
    t = torch.as_strided(buf, src.shape, (W + pad,) + inner, off)
    t.copy_(src)
    return t, buf


def host(t):
    return wl.from_torch(t)


def untouched(t, buf):
    """The elements of buf outside t still hold their fill."""
    mask = torch.ones_like(buf, dtype=torch.bool)
    torch.as_strided(mask, t.shape, t.stride(), t.storage_offset()).fill_(False)
    assert bool((buf[mask] == 7).all())


# Row lengths in vectors of V elements plus a tail: no whole vector, one
# vector, the edges of one, two, four and eight vectors per work-item, two
# passes beyond.
def _norm_lengths(v):
    return [v - 1, v, 255 * v + 1, 256 * v, 256 * v + v - 1, 257 * v, 512 * v, 513 * v + 1,
            1024 * v + 1, 1025 * v, 2048 * v + v - 1, 2049 * v, 4096 * v + 1, 4097 * v + 3,
            8192 * v + v - 1, 8193 * v, 12289 * v + 1]


NORM = [(d, H) for d, v in ((nm.F32, 4), (nm.BF16, 8)) for H in _norm_lengths(v)]


@pytest.mark.parametrize("res", [False, True], ids=["rmsnorm", "residual"])
@pytest.mark.parametrize("dtype,H", NORM)
def test_norm_rows(cache, dtype, H, res):
    r = rng(H + 5 * res)
    T = 3
    x, w = wl.host_array(r, (T, H), dtype), wl.host_weight(r, H, dtype)
    z = np.zeros_like(x)
    xd, _ = put(x, dtype, 1, 1)
    wd = put(w[None], dtype, 1, 0)[0][0]
    yd, ybuf = put(z, dtype, 3, 2)
    if res:
        rr = wl.host_array(r, (T, H), dtype)
        rd, _ = put(rr, dtype, 2, 5)
        od, obuf = put(z, dtype, 0, 3)
        cache.residual_rmsnorm(xd, rd, wd, 1e-6, out=yd, residual_out=od)
        wy, wh = O.residual_rmsnorm(x, rr, w, 1e-6, dtype)
        check("res_out", host(od), wh, dtype, exact=True)
        untouched(od, obuf)
        inplace = rd, put(x, dtype, 1, 1)[0]
        cache.residual_rmsnorm(inplace[1], rd, wd, 1e-6, out=inplace[1], residual_out=rd)
        check("y in place", host(inplace[1]), wy, dtype)
        check("res_out in place", host(rd), wh, dtype, exact=True)
    else:
        cache.rmsnorm(xd, wd, 1e-6, out=yd)
        wy = O.rmsnorm(x, w, 1e-6, dtype)
    check("y", host(yd), wy, dtype)
    untouched(yd, ybuf)
    assert cache.last_selection().variant == S.RN_SCALAR


# Row passes of SwiGLU and the element-wise ops: widths below a vector, whole
# vectors and tails of one and of V - 1 elements, rows that end inside a
# workgroup, one row of several workgroups; gaps between rows (or none), and
# operands at different distances from a boundary.
def _slot_cases():
    for dtype, v in ((nm.F32, 4), (nm.BF16, 8)):
        for T, W in ((1, 1), (5, v - 1), (7, v), (3, v + 1), (9, 31 * v + v - 1), (4, 256 * v),
                     (3, 257 * v + 1), (2, 1025 * v - 1)):
            for off, pad in ((0, 0), (1, 0), (1, 3), (0, v)):
                yield dtype, T, W, off, pad


@pytest.mark.parametrize("op", ["swiglu", "silu", "add", "masked_fill"])
@pytest.mark.parametrize("dtype,T,W,off,pad", list(_slot_cases()))
def test_row_passes(cache, op, dtype, T, W, off, pad):
    r = rng(T * 31 + W + off + pad)
    a = wl.host_array(r, (T, W), dtype, outliers=True)
    b = wl.host_array(r, (T, W), dtype)
    ad, _ = put(a, dtype, off, pad)
    bd, _ = put(b, dtype, 3 * off, 2 * pad)
    od, obuf = put(np.zeros_like(a), dtype, 2 * off, pad)
    if op == "swiglu":
        cache.swiglu(ad, bd, out=od)
        want = O.swiglu(a, b, dtype)
    elif op == "silu":
        cache.silu(ad, out=od)
        want = O.silu(a, dtype)
    elif op == "add":
        cache.add(ad, bd, out=od)
        want = O.add(a, b, dtype)
    else:
        mask = (r.random((T, W)) < 0.4).astype(np.uint8) * np.uint8(129)
        mbuf = torch.zeros(off + T * (W + pad), dtype=torch.uint8, device=DEV)
        md = torch.as_strided(mbuf, (T, W), (W + pad, 1), off)
        md.copy_(torch.from_numpy(mask))
        cache.masked_fill(ad, md, float("-inf"), out=od)
        want = O.masked_fill(a, mask, float("-inf"), dtype)
    exact = op in ("add", "masked_fill")
    check(op, host(od), want, dtype, exact=exact)
    untouched(od, obuf)
    if op == "swiglu":                       # in place on the gate
        cache.swiglu(ad, bd, out=ad)
        check("in place", host(ad), want, dtype)


@pytest.mark.parametrize("dtype,T,I", [(nm.BF16, 3000, 19008), (nm.BF16, 3001, 19009),
                                       (nm.F32, 1500, 19001)])
def test_streaming_swiglu_row_passes(cache, dtype, T, I):
    """Calls of more than 320 MiB (nontemporal accesses), gate and up as the
    halves of one buffer: sampled rows against the oracle, and every row
    against calls of 500 rows (cached accesses), bit for bit."""
    g = torch.Generator(device=DEV)
    g.manual_seed(T)
    td = torch.bfloat16 if dtype == nm.BF16 else torch.float32
    gu = torch.randn((T, 2 * I), generator=g, device=DEV).to(td)
    gate, up = gu[:, :I], gu[:, I:]
    out = cache.swiglu(gate, up)
    for lo in range(0, T, 500):
        part = cache.swiglu(gate[lo:lo + 500], up[lo:lo + 500])
        assert torch.equal(out[lo:lo + 500], part), lo
    rows = torch.tensor([0, 1, T // 2, T - 1], device=DEV)
    check("rows", host(out[rows]), O.swiglu(host(gate[rows]), host(up[rows]), dtype), dtype)


# RoPE heads of any size and start: halves (or pairs) of one short chunk, of
# whole chunks that are no power of two, with a short last chunk; more heads
# than one pass of a workgroup; partial rotary spans; the largest head, where
# a float32 head of pairs has more chunks than a wavefront has lanes.
def _rope_cases():
    for hd, rd in ((2, 0), (6, 0), (18, 0), (80, 0), (96, 0), (96, 34), (120, 0), (192, 0),
                   (256, 40), (510, 0), (512, 0)):
        for nq, nk in ((1, 0), (5, 2), (33, 9)):
            yield hd, rd, nq, nk


@pytest.mark.parametrize("qkn", [False, True], ids=["plain", "qkn"])
@pytest.mark.parametrize("inter", [False, True], ids=["half", "pairs"])
@pytest.mark.parametrize("dtype", [nm.F32, nm.BF16])
@pytest.mark.parametrize("hd,rd,nq,nk", list(_rope_cases()))
def test_rope_heads(cache, dtype, hd, rd, nq, nk, inter, qkn):
    import paper_2609_37241_amd as tri
    r = rng(hd * 7 + rd + nq)
    T, span = 3, rd or hd
    q, k = wl.host_array(r, (T, nq, hd), dtype), wl.host_array(r, (T, nk, hd), dtype)
    qw, kw = wl.host_weight(r, hd, dtype), wl.host_weight(r, hd, dtype)
    table = wl.cos_sin_table(r, 64, span) if hd % 4 else None
    pos = r.integers(-2, 70, size=T).astype(np.int64)
    tt = torch.from_numpy(table).to(DEV) if table is not None else None
    ext = tri.rope_ext(rotary_dim=rd, interleaved=inter, pos_int64=True, cos_sin=tt)
    for off, pad in ((0, 0), (1, 3)):
        qd, qbuf = put(q, dtype, off, pad)
        kd, kbuf = put(k, dtype, 2 * off, pad) if nk else (None, None)
        qwd = put(qw[None], dtype, off, 0)[0][0] if qkn else None
        kwd = put(kw[None], dtype, off, 0)[0][0] if qkn and nk else None
        cache.rope(qd, kd, torch.from_numpy(pos).to(DEV), 1e4, ext, q_w=qwd, k_w=kwd)
        wq, wk = O.rope_ext(q, k, pos, 1e4, dtype, q_w=qw if qkn else None,
                            k_w=kw if qkn else None, eps=1e-6, rotary_dim=span, interleaved=inter,
                            cos_sin=table)
        check("q", host(qd), wq, dtype)
        untouched(qd, qbuf)
        if nk:
            check("k", host(kd), wk, dtype)
            untouched(kd, kbuf)


# The scale of a head is 1 / sqrt of a sum of hd squares. A lane sums at most
# ten vectors of four (two of the rotated span, eight past it) in four chains of
# ten and two more additions, so the sum is at most 12 * 2^-24 off if every
# rounding of one head errs alike; over a hundred independent ones it stays far
# below (0.6 rms, 2.7 at most of 40,000 heads in a model of the sum). Half of a
# bound of 5 for the scale, with the sum's rounding, the division and eps (a
# quarter of 2^-24 each) and the square root (one last place, 2^-23): 5.25.
# Heads that one lane sums alone in one chain are up to 11 * 2^-24 off.
@pytest.mark.parametrize("inter", [False, True], ids=["half", "pairs"])
@pytest.mark.parametrize("hd,rd", [(512, 2), (512, 8), (512, 64), (256, 32), (128, 64), (96, 0)])
def test_head_norm_sum(cache, hd, rd, inter):
    import paper_2609_37241_amd as tri
    r = rng(hd + rd)
    T, nq, nk = 64, 32, 8
    q, k = r.standard_normal((T, nq, hd)), r.standard_normal((T, nk, hd))
    q, k = q.astype(np.float32), k.astype(np.float32)
    one = torch.ones(hd, device=DEV)
    qd, _ = put(q, nm.F32, 1, 1)
    kd, _ = put(k, nm.F32, 1, 1)
    ext = tri.rope_ext(rotary_dim=rd, interleaved=inter)
    cache.rope(qd, kd, torch.zeros(T, dtype=torch.int32, device=DEV), 1e4, ext, q_w=one, k_w=one,
               eps=1e-6)                 # position 0: no rotation
    for x, got in ((q, host(qd)), (k, host(kd))):
        x = x.astype(np.float64)
        want = 1.0 / np.sqrt(np.square(x).mean(-1) + np.float64(np.float32(1e-6)))
        # the products' roundings: at most 2^-24 each, an average over the head
        big = np.abs(x) > 1e-3
        scale = np.where(big, got / np.where(big, x, 1.0), 0.0).sum(-1) / big.sum(-1)
        err = np.abs(scale / want - 1.0).max() * 2.0 ** 24
        assert err <= 5.25, err


# Rows beyond 2048 vectors, which a workgroup of 1024 takes (four and eight
# vectors a work-item, two passes), through every way a launch gets its block
# size: compiled for the row length, without kernel arguments, one version for
# a range of lengths, and as a chain's norm.
@pytest.mark.parametrize("path", ["jit", "resident"])
@pytest.mark.parametrize("res", [False, True], ids=["rmsnorm", "residual"])
@pytest.mark.parametrize("dtype", [nm.F32, nm.BF16])
@pytest.mark.parametrize("vecs", [2048, 2049, 4097, 8192, 8193])
def test_long_rows_compiled_and_resident(cache, dtype, vecs, res, path):
    import paper_2609_37241_amd as tri
    H = vecs * (4 if dtype == nm.F32 else 8) + 3
    r, T = rng(H), 3
    x, rr = wl.host_array(r, (T, H), dtype), wl.host_array(r, (T, H), dtype)
    w = wl.host_weight(r, H, dtype)
    xd, rd, wd = put(x, dtype, 1, 1)[0], put(rr, dtype, 0, 2)[0], wl.to_torch(w, dtype, DEV)
    other = tri.SpecCache(jit=path == "jit", resident_args=path == "resident")
    outs = []
    for c in (cache, other):
        y, ybuf = put(np.zeros_like(x), dtype, 3, 1)
        o, obuf = put(np.zeros_like(x), dtype, 2, 0)
        for _ in range(2):                      # a miss, then a hit
            y.zero_()
            if res:
                c.residual_rmsnorm(xd, rd, wd, 1e-6, out=y, residual_out=o)
                untouched(o, obuf)
            else:
                c.rmsnorm(xd, wd, 1e-6, out=y)
            untouched(y, ybuf)
            outs.append((y.clone(), o.clone()))
    torch.cuda.synchronize()
    lanes = other.last_selection().launch[0].block_x
    assert lanes == (1024 if vecs > 2048 else 256)
    if path == "jit":
        assert other.version_info(0).jit == 1
    else:
        assert other.resident_info()["launches"] == 2
    other.close()
    for y, o in outs[1:]:
        assert torch.equal(y, outs[0][0]) and torch.equal(o, outs[0][1])
    wy, wh = O.residual_rmsnorm(x, rr, w, 1e-6, dtype) if res else (O.rmsnorm(x, w, 1e-6, dtype), 0)
    check("y", host(outs[3][0]), wy, dtype)
    if res:
        check("res_out", host(outs[3][1]), wh, dtype, exact=True)


@pytest.mark.parametrize("resident", [False, True], ids=["arguments", "resident"])
def test_one_version_for_rows_of_both_block_sizes(resident):
    import paper_2609_37241_amd as tri
    c, dtype = tri.SpecCache(generic=True, resident_args=resident), nm.BF16
    r = rng(3)
    for H in (16387, 16403, 9, 65555, 16387, 16403, 4099):
        x, w = wl.host_array(r, (5, H), dtype), wl.host_weight(r, H, dtype)
        y = c.rmsnorm(put(x, dtype, 1, 0)[0], wl.to_torch(w, dtype, DEV), 1e-6)
        torch.cuda.synchronize()
        assert c.last_selection().launch[0].block_x == (1024 if H // 8 > 2048 else 256)
        check(f"{H}", host(y), O.rmsnorm(x, w, 1e-6, dtype), dtype)
    assert c.stats()["n_versions"] == 1 and c.stats()["misses"] == 1
    c.close()


@pytest.mark.parametrize("kw", [{}, {"jit": True}, {"resident_args": True}],
                         ids=["arguments", "jit", "resident"])
@pytest.mark.parametrize("H", [16387, 16403])
def test_three_launch_chain_of_long_rows(H, kw):
    import paper_2609_37241_amd as tri
    dtype, T, nq, nk, hd, I = nm.BF16, 3, 4, 2, 64, 688
    r = rng(H)
    h = dict(x=wl.host_array(r, (T, H), dtype), residual=wl.host_array(r, (T, H), dtype),
             q=wl.host_array(r, (T, nq, hd), dtype), k=wl.host_array(r, (T, nk, hd), dtype),
             gate=wl.host_array(r, (T, I), dtype), up=wl.host_array(r, (T, I), dtype),
             w=wl.host_weight(r, H, dtype), pos=r.integers(0, 99, T).astype(np.int32))
    want = O.decode_chain(h, 1e-6, 1e4, dtype)
    c = tri.SpecCache(**kw)
    for _ in range(2):                          # a miss, then a hit
        d = {k: put(v, dtype, 1, 0)[0] for k, v in h.items() if k not in ("w", "pos")}
        y, ro, out = c.decode_chain(d["x"], d["residual"], wl.to_torch(h["w"], dtype, DEV), d["q"],
                                    d["k"], torch.from_numpy(h["pos"]).to(DEV), d["gate"], d["up"],
                                    1e-6, 1e4)
        torch.cuda.synchronize()
        sel = c.last_selection()
        assert sel.n_launches == 3 and sel.launch[0].block_x == (1024 if H // 8 > 2048 else 256)
        for n, g in (("y", y), ("out", out), ("q", d["q"]), ("k", d["k"])):
            check(n, host(g), want[n], dtype)
        check("res_out", host(ro), want["res_out"], dtype, exact=True)
    c.close()


@pytest.mark.parametrize("res", [False, True], ids=["rmsnorm", "residual"])
@pytest.mark.parametrize("dtype", [nm.F32, nm.BF16])
@pytest.mark.parametrize("vecs,tail", [(0, 3), (64, 0), (64, 1), (128, 3), (129, 0), (256, 2)])
def test_many_short_norm_rows(cache, dtype, vecs, tail, res):
    """More rows than workgroups fit on the chip at once (2049 of them: the
    last workgroup has one row): a wavefront per row, against the oracle, and
    against a call of 2048 rows (a workgroup per row)."""
    H = vecs * (4 if dtype == nm.F32 else 8) + tail
    r, T = rng(H), 2049
    x, rr = wl.host_array(r, (T, H), dtype), wl.host_array(r, (T, H), dtype)
    w = wl.host_weight(r, H, dtype)
    xd, _ = put(x, dtype, 1, 1)
    rd, _ = put(rr, dtype, 2, 0)
    wd = put(w[None], dtype, 3, 0)[0][0]
    yd, ybuf = put(np.zeros_like(x), dtype, 1, 2)
    if res:
        od, obuf = put(np.zeros_like(x), dtype, 0, 1)
        cache.residual_rmsnorm(xd, rd, wd, 1e-6, out=yd, residual_out=od)
        wy, wh = O.residual_rmsnorm(x, rr, w, 1e-6, dtype)
        check("res_out", host(od), wh, dtype, exact=True)
        untouched(od, obuf)
        few = cache.residual_rmsnorm(xd[1:], rd[1:], wd, 1e-6)[0]
    else:
        cache.rmsnorm(xd, wd, 1e-6, out=yd)
        wy = O.rmsnorm(x, w, 1e-6, dtype)
        few = cache.rmsnorm(xd[1:], wd, 1e-6)
    check("y", host(yd), wy, dtype)
    check("y of 2048 rows", host(few), wy[1:], dtype)
    untouched(yd, ybuf)


def _near_tie_row(r, H):
    """Seven float32 values, 0.5 first, whose sum of squares S puts sqrt(H / S)
    between 2^-51 and 2^-49.5 (relative) from the midpoint of two adjacent
    float32 numbers, and the one it rounds to. The squares are whole multiples
    of 2^-52 and S < 2, so that any order of float64 sums is exact."""
    while True:
        lo = np.float32(np.sqrt(H / r.uniform(1.05, 1.2)))
        hi = np.nextafter(lo, np.float32(np.inf))
        tie = (Fraction(float(lo)) + Fraction(float(hi))) / 2
        at = H / tie ** 2                              # the sum of squares at the midpoint
        shift = 1 - Fraction(float(r.choice([-1, 1]) * 2.0 ** r.uniform(-50.5, -48.5)))
        left = int(at * shift * 2 ** 52) - 2 ** 50
        n = [isqrt(left) // 4 * 4]                     # 24 bits of mantissa
        left -= n[0] ** 2
        while len(n) < 6:
            n.append(isqrt(left))
            left -= n[-1] ** 2
        total = Fraction(2 ** 50 + sum(i * i for i in n), 2 ** 52)
        off = (at / total - 1) / 2                     # of sqrt(H / S) above the tie, relative
        if 2.0 ** -51 <= abs(off) <= 2.0 ** -49.5:
            return [0.5] + [i * 2.0 ** -26 for i in n], hi if off > 0 else lo


@pytest.mark.parametrize("res", [False, True], ids=["rmsnorm", "residual"])
@pytest.mark.parametrize("T,H", [(2000, 7), (3000, 1139), (1500, 4099), (1000, 8203), (500, 36873)])
def test_norm_scale_keeps_the_precision_of_float64(cache, T, H, res):
    """The scale 1 / sqrt(S / H) rounds to the nearest float32 down to 2^-51
    from a tie: a division, a square root and another division in float64 (or
    a reciprocal, a product and a refined reciprocal square root) are good to
    2.5 * 2^-53 < 2^-51, a scale with fewer bits is not. A wavefront per row, 256
    and 1024 work-items per row, and rows held in part."""
    r = rng(H)
    x, want = np.zeros((T, H), np.float32), np.empty(T, np.float32)
    for i in range(T):
        row, want[i] = _near_tie_row(r, H)
        x[i, :7] = row
    xd = torch.from_numpy(x).to(DEV)
    w = torch.ones(H, device=DEV)
    y = cache.residual_rmsnorm(xd, torch.zeros_like(xd), w, 0.0)[0] if res else \
        cache.rmsnorm(xd, w, 0.0)
    got = 2 * host(y[:, 0].contiguous())               # y = (0.5 * scale) * 1, exactly
    wrong = int((got != want).sum())
    assert wrong == 0


@pytest.mark.parametrize("op,dtype,T,W,pad", [
    ("add", nm.BF16, 4500, 10007, 0), ("add", nm.F32, 2000, 12000, 0),
    ("silu", nm.BF16, 8200, 8200, 8), ("masked_fill", nm.BF16, 9000, 8000, 0),
    ("residual", nm.BF16, 6000, 8192, 0), ("residual", nm.F32, 6000, 4100, 4),
    # eight and sixteen vectors a work-item
    ("residual", nm.BF16, 3000, 16384, 0), ("residual", nm.F32, 2500, 10252, 4),
    # split over 3 and 9 workgroups: slices of 1408 and of 2048 vectors, the last shorter
    ("residual", nm.BF16, 1500, 32776, 8), ("residual", nm.F32, 400, 65540, 0),
    # ragged: 256 and 1024 work-items a row, and rows held in part
    ("residual", nm.BF16, 6000, 8195, 0), ("residual", nm.BF16, 1100, 40003, 5),
    ("residual", nm.F32, 300, 88771, 0)])
def test_streaming_calls_equal_cached_ones(cache, op, dtype, T, W, pad):
    """Calls beyond the last-level cache (nontemporal accesses), flat and by
    rows: the bits of the same call made 1000 rows (or half the rows) at a time,
    and the oracle's values on sampled rows."""
    g = torch.Generator(device=DEV)
    g.manual_seed(W)
    td = torch.bfloat16 if dtype == nm.BF16 else torch.float32

    def draw():
        return torch.randn((T, W + pad), generator=g, device=DEV).to(td)[:, :W]
    a, b = draw(), draw()
    w = torch.rand(W, generator=g, device=DEV).to(td) + 0.5
    mask = a > 0.5
    run = {"add": lambda s: (cache.add(a[s], b[s]),),
           "silu": lambda s: (cache.silu(a[s]),),
           "masked_fill": lambda s: (cache.masked_fill(a[s], mask[s], -1e4),),
           "residual": lambda s: cache.residual_rmsnorm(a[s], b[s], w, 1e-6)}[op]
    whole = run(slice(0, T))
    step = min(1000, T // 2)
    for lo in range(0, T, step):
        part = run(slice(lo, lo + step))
        for x, y in zip(whole, part):
            assert torch.equal(x[lo:lo + step], y), lo
    rows = torch.tensor([0, 1, T // 2, T - 1], device=DEV)
    ah, bh = host(a[rows]), host(b[rows])
    want = {"add": lambda: (O.add(ah, bh, dtype),), "silu": lambda: (O.silu(ah, dtype),),
            "masked_fill": lambda: (O.masked_fill(ah, host(mask[rows].to(torch.uint8)), -1e4, dtype),),
            "residual": lambda: O.residual_rmsnorm(ah, bh, host(w), 1e-6, dtype)}[op]()
    for x, y in zip(whole, want):
        check("rows", host(x[rows]), y, dtype)


@pytest.mark.parametrize("dtype,H", [(nm.F32, 1), (nm.F32, 4), (nm.F32, 1023), (nm.F32, 2052),
                                     (nm.BF16, 7), (nm.BF16, 8), (nm.BF16, 4095), (nm.BF16, 4104)])
@pytest.mark.parametrize("off,pad", [(0, 0), (1, 0), (1, 5)])
def test_embedding_rows(cache, dtype, H, off, pad):
    """Rows of less than a vector, of whole vectors and with a tail, below, at
    and above the 512 slots of a workgroup, ids on both sides of the range."""
    r = rng(H + off)
    for T, n in ((1, 3), (37, 11)):
        table = wl.host_array(r, (n, H), dtype)
        ids = r.integers(-1, n + 1, size=T).astype(np.int64)
        td, _ = put(table, dtype, off, pad)
        od, obuf = put(np.ones((T, H), table.dtype), dtype, 2 * off, pad)
        cache.embedding(td, torch.from_numpy(ids).to(DEV), out=od)
        check("embedding", host(od), O.embedding(table, ids, dtype), dtype, exact=True)
        untouched(od, obuf)


@pytest.mark.parametrize("H", [4104, 4101])
def test_embedding_beyond_the_last_level_cache(cache, H):
    """Outputs written nontemporally: the table's bits, zeros for other ids."""
    g = torch.Generator(device=DEV)
    g.manual_seed(H)
    table = torch.randn((500, H), generator=g, device=DEV).to(torch.bfloat16)
    ids = torch.randint(0, 500, (33000,), generator=g, device=DEV)
    want = table[ids]
    bad = torch.tensor([0, 777, 32999], device=DEV)
    ids[bad] = torch.tensor([-1, 500, 1 << 40], device=DEV)
    want[bad] = 0
    assert torch.equal(cache.embedding(table, ids), want)


@pytest.mark.parametrize("dtype", [nm.F32, nm.BF16])
def test_silu_tail_beside_ordinary_elements(cache, dtype):
    """Vectors of which one element, all or none lie in the negative tail,
    with infinities, NaN and zeros beside it: the oracle's values, and for the
    ordinary elements the bits they have in a vector without a tail."""
    v = 4 if dtype == nm.F32 else 8
    base = np.linspace(-79.5, 90.0, v, dtype=np.float32)
    rows = [base]
    for x in (-80.0, -80.5, -88.0, -91.0, -103.0, -3e38, -np.inf, np.inf, np.nan, 0.0, -0.0, 3e38):
        for i in range(v):
            row = base.copy()
            row[i] = x
            rows.append(row)
    rows.append(np.full(v, -85.0, np.float32))
    a = nm.round_to(np.stack(rows), dtype) if dtype == nm.BF16 else np.stack(rows)
    x = wl.to_torch(a, dtype, DEV)
    got = cache.silu(x)
    want = O.silu(a, dtype)
    fin = np.isfinite(nm.values(want, dtype))
    g = nm.values(host(got), dtype)
    assert (np.isnan(g) == np.isnan(nm.values(want, dtype))).all()
    assert (np.isinf(g) == np.isinf(nm.values(want, dtype))).all()
    w = nm.values(want, dtype)
    rel = 4e-7 if dtype == nm.F32 else 2.0 ** -8      # one rounding (f32: the form's own error)
    tiny = 2.0 ** -126                                 # results below it may flush
    assert (np.abs(g - w)[fin] <= rel * np.abs(w)[fin] + tiny).all()
    first = got[0]
    for i, row in enumerate(rows):
        same = torch.from_numpy(row == rows[0]).to(DEV)
        assert torch.equal(got[i][same], first[same]), i
    up = torch.ones_like(x)
    torch.testing.assert_close(cache.swiglu(x, up), got, rtol=0, atol=0, equal_nan=True)


# Aligned heads, one token to a workgroup: one head per lane group (as many
# groups as heads, and one more head), several (beyond four slices of 256
# lanes, and beyond decode sizes), Q and K on either side of a group's step.
@pytest.mark.parametrize("qkn", [False, True], ids=["plain", "qkn"])
@pytest.mark.parametrize("inter", [False, True], ids=["half", "pairs"])
@pytest.mark.parametrize("dtype,T,nq,nk,hd,table", [
    (nm.BF16, 1, 32, 0, 128, False), (nm.BF16, 1, 32, 1, 128, True), (nm.BF16, 2, 100, 28, 128, True),
    (nm.BF16, 2, 100, 29, 128, False), (nm.F32, 3, 31, 33, 64, True), (nm.F32, 1, 60, 5, 128, False),
    (nm.BF16, 70, 32, 1, 128, True), (nm.BF16, 66, 65, 64, 128, False), (nm.F32, 65, 17, 16, 128, False),
    (nm.BF16, 67, 8, 1, 128, True), (nm.BF16, 131, 16, 0, 128, False), (nm.F32, 65, 2, 1, 512, False),
    (nm.BF16, 67, 1, 0, 512, True), (nm.BF16, 70, 1, 1, 512, False)])
def test_aligned_rope_tokens(cache, dtype, T, nq, nk, hd, table, inter, qkn):
    import paper_2609_37241_amd as tri
    r = rng(T + nq * 3 + hd)
    q, k = wl.host_array(r, (T, nq, hd), dtype), wl.host_array(r, (T, nk, hd), dtype)
    qw, kw = wl.host_weight(r, hd, dtype), wl.host_weight(r, hd, dtype)
    tab = wl.cos_sin_table(r, 300, hd) if table else None
    pos = r.integers(-2, 310, size=T).astype(np.int64 if table else np.int32)
    ext = tri.rope_ext(interleaved=inter, pos_int64=table,
                       cos_sin=torch.from_numpy(tab).to(DEV) if table else None)
    qd, qbuf = put(q, dtype, 0, 64)
    kd, kbuf = put(k, dtype, 0, 32) if nk else (None, None)
    dev = lambda w: wl.to_torch(w, dtype, DEV)
    cache.rope(qd, kd, torch.from_numpy(pos).to(DEV), 1e4, ext, q_w=dev(qw) if qkn else None,
               k_w=dev(kw) if qkn and nk else None)
    wq, wk = O.rope_ext(q, k, pos, 1e4, dtype, q_w=qw if qkn else None, k_w=kw if qkn else None,
                        eps=1e-6, interleaved=inter, cos_sin=tab)
    check("q", host(qd), wq, dtype)
    untouched(qd, qbuf)
    if nk:
        check("k", host(kd), wk, dtype)
        untouched(kd, kbuf)

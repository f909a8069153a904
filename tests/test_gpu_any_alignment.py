"""GPU parity of the kernels that take rows starting at any element and of any
length, at the edges of their register and vector layouts: operands at
different distances from a 16-byte boundary, odd row strides, lengths just
below, at and above a whole number of vectors or of workgroups. Expected
values from the oracle, tolerances of tests/parity.py."""
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


@pytest.fixture(scope="module")
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
            1024 * v + 1, 1025 * v, 2048 * v + v - 1, 2049 * v, 4097 * v + 3]


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

"""One decode step (per channel and multi-head) at the orders where its lanes are
partly filled, at the edges of its power-of-two lane counts, past them, with
ragged batches and widths, and with arrays that are only 8-byte aligned (one mode
per lane), against the same formulas in float64.

Bounds: a dot product of d complex modes in float32, in any order, is within
(2 d + 4) units of 2^-24 of the sum of its terms' magnitudes; an updated state takes
two roundings per product, 4 units of |lambda| |x| sqrt(2) + |u|; a bfloat16 output
is rounded once more (2^-8 relative).
"""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
ORDERS = [1, 3, 5, 6, 7, 10, 12, 17, 24, 31, 33, 48, 63, 65, 66, 100, 126, 127, 129, 130]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    import paper_2310_18780_amd as lh

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    lh.lib()
    yield


def _cplx(g, shape, shift=0):
    """complex64 normals, `shift` values past a 16-byte boundary."""
    import torch

    n = 1
    for s in shape:
        n *= s
    x = torch.randn(n + shift, generator=g, device="cuda", dtype=torch.complex64)[shift:].view(shape)
    assert (x.data_ptr() % 16 != 0) == (shift % 2 == 1)
    return x


def _close(got, ref, bound, io):
    import torch

    err = (got.to(ref.dtype) - ref).abs()
    if io == torch.bfloat16:
        bound = bound + 2.0 ** -8 * ref.abs()
    assert bool((err <= bound).all()), float((err - bound).max())


def _check_state(got, lam, x, z):
    import torch

    ref = lam * x + z
    bound = 4 * EPS * (2 ** 0.5 * lam.abs() * x.abs() + z.abs())
    assert bool(((got.to(torch.complex128) - ref).abs() <= bound).all())


@pytest.mark.parametrize("d", ORDERS)
@pytest.mark.parametrize("B,D,io,shift", [(3, 37, "f32", 0), (9, 130, "bf16", 0), (33, 65, "f32", 1)])
def test_step(d, B, D, io, shift):
    import torch

    import paper_2310_18780_amd as lh

    print(f"[step lanes] B={B} D={D} d={d} {io} shift={shift}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(d)
    io = torch.float32 if io == "f32" else torch.bfloat16
    lam, R, x = _cplx(g, (D, d), shift), _cplx(g, (D, d), shift), _cplx(g, (B, D, d), shift)
    h0 = torch.randn(D, generator=g, device="cuda")
    u = torch.randn((B, D), generator=g, device="cuda").to(io)
    y = torch.full_like(u, float("nan"))
    x0, l64, r64, u64 = x.to(torch.complex128), lam.to(torch.complex128), R.to(torch.complex128), u.double()
    lh.step(lam, R, h0, x, u, y)
    torch.cuda.synchronize()
    ref = (r64 * x0).sum(-1).real + h0.double() * u64
    mag = (r64.abs() * x0.abs()).sum(-1) + (h0.double() * u64).abs()
    _close(y.double(), ref, (2 * d + 4) * EPS * mag, io)
    _check_state(x, l64, x0, u64[..., None])


@pytest.mark.parametrize("d", [1, 3, 6, 10, 17, 31, 48, 65, 126, 129])
@pytest.mark.parametrize("shift", [0, 1])
def test_multihead_step(d, shift):
    import torch

    import paper_2310_18780_amd as lh

    B, M, N = 2, 3, 21
    print(f"[mh lanes] d={d} shift={shift}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(100 + d)
    lam, R, x = _cplx(g, (M, d), shift), _cplx(g, (M, d), shift), _cplx(g, (B, M, N, N, d), shift)
    h0 = torch.randn(M, generator=g, device="cuda")
    q, k, v = (torch.randn((B, M * N), generator=g, device="cuda") for _ in range(3))
    y = torch.full_like(q, float("nan"))
    x0 = x.to(torch.complex128)
    l64, r64 = (a.to(torch.complex128)[:, None, None] for a in (lam, R))
    q64, k64, v64 = (a.double().view(B, M, N) for a in (q, k, v))
    lh.mh_step(lam, R, h0, x, q, k, v, y)
    torch.cuda.synchronize()
    z = k64[..., None] * v64[..., None, :]
    h = h0.double()[:, None, None]
    w = (r64 * x0).sum(-1).real + h * z
    mag = ((r64.abs() * x0.abs()).sum(-1) + (h * z).abs()) * q64.abs()[..., None, :]
    ref = (w * q64[..., None, :]).sum(-1).view(B, M * N)
    _close(y.double(), ref, (2 * d + N + 8) * EPS * mag.sum(-1).view(B, M * N), torch.float32)
    # z itself is rounded to float32 (one unit more of |z|)
    ref_x = l64 * x0 + z[..., None]
    bound = 5 * EPS * (2 ** 0.5 * l64.abs() * x0.abs() + z.abs()[..., None])
    assert bool(((x.to(torch.complex128) - ref_x).abs() <= bound).all())


@pytest.mark.parametrize("B,D,d,shift", [
    (5, 4096, 33, 0),                     # eight rows per thread, three of them past the batch
    (2, 4096, 33, 0), (3, 4096, 17, 0),   # no more rows than there are; two at most in single modes
    (5, 1024, 24, 0), (4, 1024, 32, 0),   # one and two rows: 384 and 512 wavefronts of pairs
    (63, 2048, 9, 0),                     # single modes past the small states: eight rows
    (33, 1024, 15, 0), (35, 1024, 15, 0),  # the generic path up to 4 MiB, the lanes past it
    (35, 1024, 16, 1), (9, 2048, 1, 0),
])
def test_rows_per_thread(B, D, d, shift):
    test_step(d, B, D, "f32", shift)

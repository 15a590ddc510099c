"""The matrix-core prefill at sizes that only the automatic choice takes (any
order up to 64, any width and prompt length), at the edges of its tilings: 1, 2, 4
and 16 time chunks per row among the kernel's columns, segments with a shorter
last one, partial chunks and tiles, ragged rows, widths that leave a partial
channel group or an unaligned row, and the smallest widths.

Compared over every output and state with the VALU scan in one sequential pass
(another kernel, another association of the sums).  Both are within 1e-4 of the
exact result, relative to the largest value of the (b, c) row (checked against the
oracle elsewhere, here on two rows), so they differ by at most twice that; bfloat16
outputs by one rounding on each side more.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads
from parity_util import BF16_REL, REL_TOL, to_device

pytestmark = pytest.mark.gpu

CASES = [
    # (B, D, d, T, io, chunks per row among the columns, segments)
    (60, 1022, 12, 100, "f32", 1, 1),   # partial chunk, D % 16 != 0, ragged rows
    (50, 2035, 7, 83, "bf16", 1, 1),    # D odd
    (33, 1100, 30, 95, "f32", 1, 1),    # 1, two sixteens of modes
    (45, 1030, 24, 70, "bf16", 1, 1),
    (17, 1203, 45, 66, "f32", 2, 1),    # three sixteens
    (40, 600, 60, 130, "bf16", 1, 1),   # four sixteens
    (19, 530, 61, 71, "f32", 2, 1),
    (9, 1030, 12, 250, "f32", 4, 1),
    (23, 1500, 16, 301, "bf16", 2, 1),
    (12, 700, 20, 520, "f32", 4, 1),
    (5, 530, 40, 333, "bf16", 4, 1),
    (3, 101, 5, 1000, "f32", 16, 1),
    (2, 36, 48, 513, "f32", 16, 1),
    (1, 64, 12, 16 * 1024 + 9, "f32", 16, 33),   # the last one partial
    (2, 72, 17, 8192 + 256, "bf16", 16, 17),     # the last one of one tile
    (1, 24, 33, 5000, "f32", 16, 10),
    (6, 4, 64, 300, "bf16", 16, 1),      # one piece of channels
    (300, 18, 33, 200, "f32", 4, 1),    # half a channel group, whole pieces
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    import paper_2310_18780_amd as lh

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    lh.lib()
    yield


def _inputs(B, D, d, T, io, seed):
    import torch

    w = workloads.Workload("case", B, D, d, T, 0, io, 0.7, 0.9999, np.pi, 1.0 / d, seed)
    lam, R, h0 = workloads.make_params(w)
    t = to_device(lam, R, h0, np.zeros((1, 1, D), np.float32), np.zeros((1, 0, D), np.float32), "f32")
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.randn((B, T, D), generator=g, device="cuda").to(
        torch.bfloat16 if io == "bf16" else torch.float32)
    return (lam, R, h0), t, u


def _run(call, u, d):
    import torch

    B, T, D = u.shape
    y = torch.full_like(u, float("nan"))
    x = torch.full((B, D, d), complex(float("nan"), 0), dtype=torch.complex64, device="cuda")
    call(x, y)
    torch.cuda.synchronize()
    return y, x


def _same(a, b, io):
    """Outputs and states of two plans within twice the row tolerance."""
    (ya, xa), (yb, xb) = a, b
    err = (ya.float() - yb.float()).abs()
    bound = 2 * REL_TOL * yb.float().abs().amax(dim=1, keepdim=True)
    if io == "bf16":
        bound = bound + 2 * BF16_REL * yb.float().abs()
    assert bool((err <= bound).all()), float((err - bound).max())
    xerr = (xa - xb).abs()
    assert bool((xerr <= 2 * REL_TOL * xb.abs().amax(dim=2, keepdim=True)).all())


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%d_D%d_d%d_T%d_%s" % c[:5])
def test_against_the_scan(case):
    import torch

    import paper_2310_18780_amd as lh

    B, D, d, T, io, *cut = case
    (lam, R, h0), t, u = _inputs(*case[:5], seed=B * 1000 + d)
    print(f"[columns] {case}", flush=True)
    auto = _run(lambda x, y: lh.prefill(t["lam"], t["R"], t["h0"], u, x, y), u, d)
    scan = _run(lambda x, y: lh.prefill_with_plan(t["lam"], t["R"], t["h0"], u, x, y, T), u, d)
    assert lh.prefill_path(B, D, d, T, io=io) == ("mfma", *cut)
    _same(auto, scan, io)
    rows = [(B - 1, D - 1), (B // 2, D // 3)]
    up = u.float().cpu().numpy()
    ref = oracle.run_rows(lam, R, h0, up, np.zeros((B, 0, D), np.float32), rows)
    for i, (b, c) in enumerate(rows):
        y, x = auto[0][b, :, c].float().cpu().numpy(), auto[1][b, c].cpu().numpy()
        e = np.abs(y - ref["y_prefill"][i])
        tol = REL_TOL * np.abs(ref["y_prefill"][i]).max()
        assert np.all(e <= tol + (BF16_REL * np.abs(ref["y_prefill"][i]) if io == "bf16" else 0))
        assert np.abs(x - ref["x_T"][i]).max() <= REL_TOL * np.abs(ref["x_T"][i]).max()


def test_scratch_limits():
    """With less scratch than the tables need a call runs the VALU scan: a
    workspace of exactly the scan's size, and lh_prefill_noalloc past its 64 MiB."""
    import torch

    import paper_2310_18780_amd as lh

    B, D, d, T = 3, 200, 12, 700
    _, t, u = _inputs(B, D, d, T, "f32", 5)
    args = (t["lam"], t["R"], t["h0"], u)
    cut = 64  # the automatic scan's chunk: 3 x 4 waves, 64 steps each
    need = lh.workspace_bytes(B, D, d, T, plan=cut)
    assert need < lh.workspace_bytes(B, D, d, T)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    small = _run(lambda x, y: lh.prefill(*args, x, y, workspace=ws), u, d)
    scan = _run(lambda x, y: lh.prefill_with_plan(*args, x, y, cut), u, d)
    assert torch.equal(small[0], scan[0]) and torch.equal(small[1], scan[1])
    with pytest.raises(lh.LHError):
        lh.prefill(*args, small[1], small[0], workspace=ws[:-256])

    B, D, d, T = 16, 2560, 60, 300  # 77 MB of tables; the scan is one pass
    _, t, u = _inputs(B, D, d, T, "f32", 6)
    args = (t["lam"], t["R"], t["h0"], u)
    assert lh.prefill_path(B, D, d, T)[0] == "mfma"
    assert lh.workspace_bytes(B, D, d, T) > lh.NOALLOC_SCRATCH_BYTES
    held = _run(lambda x, y: lh.prefill_noalloc(*args, x, y), u, d)
    scan = _run(lambda x, y: lh.prefill_with_plan(*args, x, y, T), u, d)
    assert torch.equal(held[0], scan[0]) and torch.equal(held[1], scan[1])


ERROR_CASES = [(5, 520, 16, 4003), (3, 512, 32, 2001), (3, 520, 64, 1003)]


def _errors(case, io):
    """Outputs of the automatic call, of the VALU scan in one pass and in float64, for
    slow poles, whose large entry states show how many terms of them are kept."""
    import torch

    import paper_2310_18780_amd as lh

    B, D, d, T = case
    w = workloads.Workload("case", B, D, d, T, 0, io, 0.99, 0.9999, 0.1 * np.pi, 1.0 / d, 3)
    lam, R, h0 = workloads.make_params(w)
    t = to_device(lam, R, h0, np.zeros((1, 1, D), np.float32), np.zeros((1, 0, D), np.float32), "f32")
    g = torch.Generator(device="cuda").manual_seed(3)
    u = torch.randn((B, T, D), generator=g, device="cuda").to(
        torch.bfloat16 if io == "bf16" else torch.float32)
    print(f"[error] {case} {io}", flush=True)
    auto = _run(lambda x, y: lh.prefill(t["lam"], t["R"], t["h0"], u, x, y), u, d)
    scan = _run(lambda x, y: lh.prefill_with_plan(t["lam"], t["R"], t["h0"], u, x, y, T), u, d)
    assert lh.prefill_path(B, D, d, T, io=io)[0] == "mfma"
    k = torch.arange(T - 1, device="cuda", dtype=torch.float64)
    h = torch.empty((T, D), dtype=torch.float64, device="cuda")
    h[0] = t["h0"].double()
    h[1:] = 0
    for n in range(d):
        p = torch.exp(torch.log(t["lam"][:, n].to(torch.complex128)) * k[:, None])
        h[1:] += (t["R"][:, n].to(torch.complex128) * p).real
    N = 1 << (2 * T - 1).bit_length()
    y = torch.fft.irfft(torch.fft.rfft(u.double(), N, dim=1) * torch.fft.rfft(h, N, dim=0), N, dim=1)[:, :T]
    return auto[0].double(), scan[0].double(), y


@pytest.mark.parametrize("case", ERROR_CASES, ids=lambda c: "B%d_D%d_d%d_T%d" % c)
def test_error_is_the_scans(case):
    """Orders 16, 32 and 64 at prompts that no named plan takes.  Three terms leave a
    relative error of 2^-24 per product, as float32 does, so the error against
    float64 is at most half as large again as the scan's, or 1e-6."""
    auto, scan, y = _errors(case, "f32")
    err = [float((a - y).norm() / y.norm()) for a in (auto, scan)]
    print(f"[error] {err}", flush=True)
    assert err[0] <= max(1e-6, 1.5 * err[1]), err


@pytest.mark.parametrize("case", ERROR_CASES, ids=lambda c: "B%d_D%d_d%d_T%d" % c)
def test_error_of_cancelling_bfloat16_outputs_is_the_scans(case):
    """The same with bfloat16 u and y, at the outputs below 2e-3 of their row's size:
    their rounding (2^-9 of themselves, 1.9e-6 of the row over these) hides an error
    of float32 arithmetic, while two bfloat16 terms (2^-17 of the row's size, 4e-6
    over these) more than double what is left."""
    auto, scan, y = _errors(case, "bf16")
    rms = y.square().mean(dim=1, keepdim=True).sqrt()
    small = y.abs() < 2e-3 * rms
    err = [float((((a - y) / rms)[small]).square().mean().sqrt()) for a in (auto, scan)]
    print(f"[error] {err}", flush=True)
    assert err[0] <= 1.1 * err[1], err


@pytest.mark.parametrize("d", [16, 32, 64])
def test_second_terms_of_a_named_plan(d):
    """The float32 plans that keep two terms of the entry states: state and residue
    1 + 2^-8 - 2^-14 each, both just two terms, so that only the product of the
    second ones (1.5e-5 here, the largest there is) could be missing; third terms
    and roundings stay below 2^-21."""
    import torch

    import paper_2310_18780_amd as lh

    B, D, T = 2, 8, 512
    v = 1 + 2.0 ** -8 - 2.0 ** -14
    lam = torch.zeros((D, d), dtype=torch.complex64, device="cuda")
    R, h0 = torch.zeros_like(lam), torch.zeros(D, device="cuda")
    lam[:, d // 2] = 1.0
    R[:, d // 2] = v
    u = torch.zeros((B, T, D), device="cuda")
    u[:, 0] = v
    for plan in (lh.PLAN_MFMA, lh.PLAN_MFMA_SEG):
        y, x = _run(lambda x, y: lh.prefill_with_plan(lam, R, h0, u, x, y, plan), u, d)
        err = float((y[:, 1:].double() - v * v).abs().max())
        print(f"[second terms] d={d} plan={plan} {err}", flush=True)
        assert err <= 2.0 ** -21
        assert bool((x[:, :, d // 2] == v).all())


@pytest.mark.parametrize("d,plan", [(12, 0), (16, -1)])
def test_correction_of_a_young_state(d, plan):
    """The rounding of lambda^16 is put right for a whole state at once, also for what
    has not been multiplied by it since: by at most four roundings (2^-24 each),
    whichever chunk the state entered in.  A pole whose lambda^16 is rounded by almost
    2^-24, one input at the last step of a chunk, the output of the next step."""
    import torch

    import paper_2310_18780_amd as lh

    lam32 = np.arange(np.float32(0.75), np.float32(0.86), np.float32(2.0 ** -20), dtype=np.float32)
    p = lam32.astype(np.float64) ** 16
    e = np.abs(p.astype(np.float32) / p - 1)
    assert e.max() > 0.9 * 2.0 ** -24
    B, D, T = 16, 512, 512
    assert lh.prefill_path(B, D, d, T, plan=plan)[:2] == ("mfma", 16)
    lam = torch.zeros((D, d), dtype=torch.complex64, device="cuda")
    R, h0 = torch.zeros_like(lam), torch.zeros(D, device="cuda")
    lam[:, 3] = float(lam32[e.argmax()])
    R[:, 3] = 1.0
    u = torch.zeros((B, T, D), device="cuda")
    for b in range(B):  # a row for each chunk of the second 256 steps
        u[b, 255 + 16 * b] = 1.0
    y, _ = _run(lambda x, y: lh.prefill_with_plan(lam, R, h0, u, x, y, plan), u, d)
    # a chunk later with that product's rounding and the state's own (the named plan's
    # two terms of lambda^16, to 2^-17, would hide it there)
    for chunk in (0, 1) if plan == 0 else (0,):
        want = p[e.argmax()] ** chunk
        err = [float((y[b, 256 + 16 * (b + chunk)].double() - want).abs().max()) / want / 2.0 ** -24
               for b in range(B - chunk)]
        print(f"[young state] d={d} plan={plan} {err}", flush=True)
        assert max(err) <= 4 + 1 + 2 * chunk  # and the rounding of the output


NOT_FINITE = [
    (33, 1100, 30, 95, "f32"), (17, 1203, 45, 66, "f32"), (9, 1030, 12, 250, "f32"),    # 1, 2, 4 chunks
    (3, 101, 5, 1000, "f32"), (2, 36, 48, 513, "f32"), (6, 4, 64, 300, "bf16"),         # 16
    (40, 600, 60, 130, "bf16"), (23, 1500, 16, 301, "bf16"), (50, 2035, 7, 83, "bf16"),
    (1, 64, 12, 16 * 1024 + 9, "f32"), (2, 72, 17, 8192 + 256, "bf16"),                 # segments
    (64, 512, 16, 96, "f32"), (70, 512, 32, 80, "bf16"), (3, 520, 64, 100, "f32"),
    (20, 512, 64, 130, "f32"), (16, 1024, 16, 1024, "bf16"),       # named plans: u not aligned
]


@pytest.mark.parametrize("case", NOT_FINITE, ids=lambda c: "B%d_D%d_d%d_T%d_%s" % c)
def test_inputs_that_are_not_finite(case):
    """Inputs that are not finite, and (float32) one that only its nearest bfloat16 is
    not: each affects its row and channel from its own step on, as in the recurrence.
    Everything before, and every other row and channel, is what the call with zeros in
    their place gives: the same bits elsewhere, within the tolerance of _same in the
    row itself.  From there on the VALU scan's values, finite where those are."""
    import torch

    import paper_2310_18780_amd as lh

    B, D, d, T, io = case
    assert lh.prefill_path(B, D, d, T, io=io)[0] == "mfma"
    _, t, u = _inputs(*case, seed=B * 1000 + d)
    if lh.prefill_plan(B, D, d, T, io=io) != "scan":
        u = torch.cat([u.flatten(), u.flatten()[:1]])[1:].view(u.shape)
        assert u.data_ptr() % 16 != 0
    args = (t["lam"], t["R"] / 256, t["h0"] / 256)  # no sum of outputs near the largest float32
    values = [float("inf"), float("-inf"), float("nan")] + ([3.399e38, -3.399e38] if io == "f32" else [])
    spots = {}
    for i, v in enumerate(values * 3):  # first, last and other steps, rows and channels
        spots[((i * 7) % B if i else B - 1, (i * 37 + D - 1) % D)] = (
            (T - 1 if i == 0 else 0 if i == 1 else (i * 53 + 5) % T), v)
    for (b, c), (s, v) in spots.items():
        u[b, s, c] = 0
    print(f"[not finite] {case} {spots}", flush=True)
    clean = _run(lambda x, y: lh.prefill(*args, u, x, y), u, d)
    for (b, c), (s, v) in spots.items():
        u[b, s, c] = v
    auto = _run(lambda x, y: lh.prefill(*args, u, x, y), u, d)
    scan = _run(lambda x, y: lh.prefill_with_plan(*args, u, x, y, T), u, d)
    hit = torch.zeros((B, D), dtype=torch.bool, device="cuda")
    for (b, c), (s, v) in spots.items():
        hit[b, c] = True
        ya, yc, ys = (r[0][b, :, c].float() for r in (auto, clean, scan))
        tol = 2 * REL_TOL * yc.abs().max() + 2 * BF16_REL * yc.abs() * (io == "bf16")
        assert bool(((ya - yc).abs()[:s] <= tol[:s]).all()), (b, c, s, v)
        assert torch.equal(torch.isfinite(ya), torch.isfinite(ys)), (b, c, s, v)
        assert ya[s] == ys[s] or (ya[s] != ya[s] and ys[s] != ys[s]), (b, c, s, v)
        ok = torch.isfinite(ys)
        ok[:s] = False
        if bool(ok.any()):
            assert bool(((ya - ys).abs()[ok] <= 2 * REL_TOL * ys[ok].abs().max()).all()), (b, c, s, v)
        xa, xs = auto[1][b, c], scan[1][b, c]
        assert torch.equal(torch.isfinite(xa.abs()), torch.isfinite(xs.abs())), (b, c, s, v)
    assert torch.equal(auto[0].transpose(1, 2)[~hit], clean[0].transpose(1, 2)[~hit])
    assert torch.equal(auto[1][~hit], clean[1][~hit])


@pytest.mark.parametrize("case", [
    (1, 64, 16, 4096, "bf16", 16, 8), (1, 64, 16, 4096, "f32", 16, 8),   # segments
    (20, 512, 64, 130, "f32", 2, 1), (59, 2272, 32, 256, "bf16", 2, 1),
], ids=lambda c: "B%d_D%d_d%d_T%d_%s" % c[:5])
def test_unaligned_named_plans(case):
    """The automatic call at sizes of the named plans with u and y one element past a
    16-byte boundary, where it takes the three-term kernel and its larger tables in
    the same workspace, against the VALU scan."""
    import torch

    import paper_2310_18780_amd as lh

    B, D, d, T, io, *cut = case
    assert lh.prefill_plan(B, D, d, T, io=io) != "scan"
    assert lh.prefill_path(B, D, d, T, io=io) == ("mfma", *cut)
    _, t, u = _inputs(*case[:5], seed=B * 1000 + d)
    shift = lambda a: torch.cat([a.flatten()[:1], a.flatten()])[1:].view(a.shape)  # noqa: E731
    u = shift(u)
    print(f"[unaligned] {case}", flush=True)
    args = (t["lam"], t["R"], t["h0"], u)
    y, x = shift(torch.full_like(u, float("nan"))), torch.empty((B, D, d), dtype=torch.complex64, device="cuda")
    assert u.data_ptr() % 16 and y.data_ptr() % 16
    lh.prefill(*args, x, y)
    scan = _run(lambda x, y: lh.prefill_with_plan(*args, x, y, T), u, d)
    _same((y, x), scan, io)

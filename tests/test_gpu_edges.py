"""GPU tests at the edges of kernel variants: rows walked by resident workgroups in the rotation,
the two tile sizes of the compensation's trailing update, the error of the greedy kernels' own P, the
schedule kernel's storage of vhat per length, and rows that are not finite in the P-only kernels."""
import numpy as np
import pytest
import scipy.fft

torch = pytest.importorskip("torch")

import oracle.kashin_ref as ref
import parity_util as pu
import test_gpu_parity as parity
from paper_2609_11687_amd import kashin as K

pytestmark = pytest.mark.gpu


# n at and around the element counts per thread that are compiled (1, 4, 8, 16 times 256 entries),
# the padded and unpadded layouts, every odd part; m above and below the resident workgroups
# (at most 2048), so that workgroups take no, one or several rows
@pytest.mark.parametrize("n,m", [(1, 3), (3, 5), (43, 4), (128, 2100), (256, 4500), (384, 2049), (512, 2047), (1024, 2100),
                                 (1376, 70), (1536, 2051), (2048, 2050), (3072, 2500), (4096, 2305), (6144, 2000),
                                 (8192, 1100), (11008, 800), (16384, 520)])
@pytest.mark.parametrize("inverse", [False, True])
def test_rotate_rows_equal_single_rows(n, m, inverse):
    """Every row of a call over many rows equals the row rotated alone, bit for bit (also in place
    and with spare entries between the rows), and sampled rows agree with the oracle."""
    print(f"rotate n={n} m={m} inverse={inverse}", flush=True)
    rng = np.random.default_rng(n + m)
    x = rng.standard_normal((m, n)).astype(np.float32)
    xd = pu.to_dev(x)
    y = torch.empty_like(xd)
    K.kashin_rotate(n, 9, xd, y, inverse=inverse)
    wide = torch.zeros((m, n + 3), device="cuda")
    wide[:, :n] = xd
    K.kashin_rotate(n, 9, wide[:, :n], wide[:, :n], inverse=inverse)
    picks = sorted({0, 1, m // 2, m - 2, m - 1, min(m - 1, 2048)})
    alone = torch.empty((len(picks), n), device="cuda")
    for i, r in enumerate(picks):
        K.kashin_rotate(n, 9, xd[r:r + 1], alone[i:i + 1], inverse=inverse)
    torch.cuda.synchronize()
    assert torch.equal(wide[:, :n], y)
    assert torch.equal(wide[:, n:], torch.zeros((m, 3), device="cuda"))
    assert torch.equal(alone, y[picks])
    want = ref.rotate(x[picks].astype(np.float64), 9, inverse=inverse)
    got = y[picks].cpu().numpy()
    # each output is a sum of n terms through at most 14 additions and 43 products of the odd factor:
    # well below 64 roundings of 2^-24 of the row's largest entries
    assert np.abs(got - want).max() <= 64 * 2.0 ** -24 * max(np.abs(want).max(), np.abs(x).max())


@pytest.mark.parametrize("n", [3, 96, 768, 6144, 43, 172, 1376, 11008])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rotate_entries_near_the_largest_float(n, dtype):
    """Rows whose odd-factor pair sums exceed the largest float while their products do not: finite and
    the oracle's in both directions, the rows beside them as if alone, and the fused rotation as the
    separate one."""
    print(f"rotate near the largest float n={n} {dtype}", flush=True)
    b = n // (n & -n)
    big = 3.3e38
    x = np.random.default_rng(n).standard_normal((7, n)).astype(np.float32)
    x[[1, 2, 4, 5]] = 0.0
    # norms below the largest float, so that no product overflows; pair sums or differences of 1.4 big
    x[1, [0, b - 1]] = 0.7 * big
    x[2, [n - b, n - 1]] = 0.7 * big, -0.7 * big
    x[4, 1], x[4, [0, b - 1]] = -0.2 * big, 0.68 * big
    x[5, n - b:] = np.where(np.arange(b) % 2, -1.0, 1.0) * big / 16
    x[5, 0] = 2.0 ** 125
    xd = pu.to_dev(x, torch.float32 if dtype == "f32" else torch.bfloat16)
    x64 = xd.float().cpu().numpy().astype(np.float64)
    for inverse in (False, True):
        y = torch.empty((7, n), device="cuda")
        K.kashin_rotate(n, 9, xd, y, inverse=inverse)
        alone = torch.empty((1, n), device="cuda")
        for r in (0, 3, 6):
            K.kashin_rotate(n, 9, xd[r:r + 1], alone, inverse=inverse)
            assert torch.equal(alone[0], y[r])
        got, want = y.cpu().numpy(), ref.rotate(x64, 9, inverse=inverse)
        # 64 roundings of the row's largest entries bound the rotation's error (see above)
        assert np.isfinite(got).all()
        assert (np.abs(got - want).max(axis=1) <= 64 * 2.0 ** -24 * np.abs(x64).max(axis=1)).all()
    if n >= 96 and K.kashin_supported_n(n):
        y = torch.empty((7, n), device="cuda")
        K.kashin_rotate(n, 9, xd, y)
        plan = K.kashin_plan(n, 4, 3)
        sep = K.quantize_alloc(plan, y)
        fused = [torch.empty_like(t) for t in sep]
        K.kashin_quantize_rotated(plan, 9, xd, 0, *fused)
        torch.cuda.synchronize()
        for s, f in zip(sep, fused):
            assert torch.equal(s.view(torch.uint8), f.view(torch.uint8))


@pytest.mark.parametrize("n,d_in,chunk", [(11008, 500, 100), (4096, 1200, 128), (4096, 1129, 33), (10000, 520, 1)])
def test_update_tiles(n, d_in, chunk):
    """The trailing update after one chunk against float64, at sizes with ragged tiles that take the
    128 x 128 tiles (at least 256 of them), and its first columns bit for bit against a call whose
    remainder takes the 64 x 64 tiles."""
    print(f"update n={n} d_in={d_in} chunk={chunk}", flush=True)
    rest = d_in - chunk
    tiles = lambda r: -(-n // 128) * -(-r // 128)  # noqa: E731
    assert tiles(rest) >= 256 and tiles(60) < 256
    g = torch.Generator(device="cuda").manual_seed(n + chunk)
    plan = K.kashin_plan(n, 5, 3)
    w = torch.randn((d_in, n), generator=g, device="cuda") * 0.02
    h = torch.randn((2 * d_in, d_in), generator=g, device="cuda")
    u, v = (torch.empty((d_in, d_in), dtype=torch.float64, device="cuda") for _ in range(2))
    K.kashin_optq_factor((h.t().contiguous() @ h) / (2 * d_in), u, v)

    def step(d):
        wt = w[:d].clone()
        nb = (n + 3) // 4
        cu, cv = (torch.empty((chunk, nb), dtype=torch.uint8, device="cuda") for _ in range(2))
        ce = torch.empty((chunk, 2, 4), device="cuda")
        q = torch.empty((chunk, n), device="cuda")
        work = torch.empty(K.kashin_optq_workspace_bytes(d, n, chunk), dtype=torch.uint8, device="cuda")
        K.kashin_optq_quantize(plan, wt, u[:d, :d], v[:d, :d], chunk, False, 0, cu, cv, ce, q, work,
                               quantize_rows=chunk)
        torch.cuda.synchronize()
        return wt, q

    wt, q = step(d_in)
    small, q2 = step(chunk + 60)
    assert torch.equal(q, q2)
    assert torch.equal(small, wt[:chunk + 60])
    delta = (w[:chunk] - q).double()
    m = (v[:chunk, :chunk] @ u[:chunk, chunk:]).t().contiguous()
    want = w[chunk:].double() - m @ delta
    # each term rounded once in Delta and M, `chunk` FMAs, one subtraction
    bound = 2.0 ** -24 * ((chunk + 3) * (m.abs() @ delta.abs()) + w[chunk:].abs().double() + want.abs()) + 1e-30
    assert bool(((wt[chunk:].double() - want).abs() <= bound).all())


@pytest.mark.parametrize("n", [5120, 6144, 8192, 10000, 13824, 14336, 16384])
def test_operator_error(n):
    """P inside the schedule kernel, whose constants are kept in fewer registers than kashin_apply_p's, and
    P of kashin_apply_p, against float64.  With u = w - r - P vhat formed by the kernel, w - u - r -
    P64 vhat is P's own error (and three roundings).  An FFT's rms error is c 2^-24 sqrt(log2 n) of its
    input; these rows through the reverse schedule's first block have c = 0.80 to 0.85 at these lengths,
    through kashin_apply_p 0.91 to 0.98.  Last-pass twiddles that are chains of products have 0.88 (5120)
    and 0.90 (6144), radix-32 passes whose constants all round down 0.90 to 0.97 and 1.06 to 1.10."""
    print(f"operator error n={n}", flush=True)
    num = den = num_p = den_p = 0.0
    for seed in (1, 2):
        w = np.random.default_rng(seed * 100003 + n).standard_normal((64, n)).astype(np.float32)
        wd = pu.to_dev(w)
        plan = K.kashin_plan(n, seed, 1)
        u, v, r, y = (torch.empty_like(wd) for _ in range(4))
        K.kashin_decompose_schedule(plan, "reverse", wd, u, v, r)
        K.kashin_apply_p(plan, wd, y)
        torch.cuda.synchronize()
        eps = ref.sign_mask(n, seed)
        p64 = lambda x: scipy.fft.idct(eps * scipy.fft.dct(x, norm="ortho"), norm="ortho")  # noqa: E731
        w64, u64, v64, r64, y64 = (t.astype(np.float64) for t in (w, *(t.cpu().numpy() for t in (u, v, r, y))))
        num += ((w64 - u64 - r64 - p64(v64)) ** 2).sum()
        den += (w64 ** 2).sum()
        want = p64(w64)
        num_p += ((y64 - want) ** 2).sum()
        den_p += (want ** 2).sum()
    unit = 2.0 ** -24 * np.sqrt(np.log2(n))
    c, c_p = np.sqrt(num / den) / unit, np.sqrt(num_p / den_p) / unit
    print(f"c = {c:.3f}, P x {c_p:.3f}", flush=True)
    assert c <= 0.865 and c_p <= 1.02


# where the schedule kernel keeps vhat: registers (256, 5120, 6144), all in LDS (8192), private memory
# (13824, 14336, 16384; at 14336 with threads that hold no elements)
@pytest.mark.parametrize("n,schedule", [(256, "adaptive"), (5120, "original"), (6144, "adaptive"), (8192, "adaptive"),
                                        (8192, "reverse"), (13824, "original"), (13824, "alternating"),
                                        (14336, "adaptive"), (16384, "original")])
def test_schedule_storage_replay_parity(n, schedule):
    """Five rows (an unpaired last one), every step replayed by the oracle; the traced call, which writes
    no residual, equals the untraced one bit for bit."""
    print(f"schedule storage n={n} {schedule}", flush=True)
    parity.test_schedule_replay_parity(n, schedule)


@pytest.mark.parametrize("n", [96, 256, 3072, 5120, 8192, 10000, 11008, 13824, 14336, 16384])
@pytest.mark.parametrize("schedule", ["alternating", "adaptive"])
def test_schedule_without_residual(n, schedule):
    """u and vhat of many pairs without an r output equal those with one bit for bit."""
    print(f"schedule without residual n={n} {schedule}", flush=True)
    m = 701
    w = torch.randn((m, n), generator=torch.Generator(device="cuda").manual_seed(n), device="cuda") * 0.02
    plan = K.kashin_plan(n, 3, 2)
    u, v, r, u2, v2 = (torch.empty_like(w) for _ in range(5))
    K.kashin_decompose_schedule(plan, schedule, w, u, v, r)
    K.kashin_decompose_schedule(plan, schedule, w, u2, v2)
    torch.cuda.synchronize()
    assert torch.equal(u, u2) and torch.equal(v, v2)


# the generic path (172), a single wave, several waves, the split pass, radix 32
@pytest.mark.parametrize("n", [172, 512, 4096, 11008, 16384])
def test_p_only_rows_that_are_not_finite(n):
    """y = P x, the reconstruction and its rotated form: a row with a NaN or an infinity is all NaN, and its
    partner is what it is beside a row of zeros, bit for bit."""
    print(f"not finite n={n}", flush=True)
    m = 9  # bad rows in either half of a pair, both halves, and the unpaired last row
    bad = {1: float("nan"), 2: float("inf"), 4: -float("nan"), 5: -float("inf"), 8: float("nan")}
    x = pu.to_dev(np.random.default_rng(n).standard_normal((m, n)).astype(np.float32))
    clean = x.clone()
    for i, (row, val) in enumerate(bad.items()):
        x[row, (i * 37) % n] = val
        clean[row] = 0.0
    plan = K.kashin_plan(n, 4, 3)

    def check(got, want):
        torch.cuda.synchronize()
        rows = [i for i in range(m) if i not in bad]
        assert bool(torch.isnan(got[list(bad)]).all())
        assert torch.equal(got[rows], want[rows]) and bool(torch.isfinite(got[rows]).all())

    y, yc = torch.empty_like(x), torch.empty_like(x)
    K.kashin_apply_p(plan, x, y)
    K.kashin_apply_p(plan, clean, yc)
    check(y, yc)
    cu, cv, ce = K.quantize_alloc(plan, clean)
    for row, val in bad.items():  # every entry of vhat a centre that is not finite
        ce[row, 1] = 0.0
    ce_bad = ce.clone()
    for row, val in bad.items():
        ce_bad[row, 1] = val
    K.kashin_reconstruct(plan, cu, cv, ce_bad, y)
    K.kashin_reconstruct(plan, cu, cv, ce, yc)
    check(y, yc)
    K.kashin_reconstruct_rotated(plan, 9, cu, cv, ce_bad, y)
    K.kashin_reconstruct_rotated(plan, 9, cu, cv, ce, yc)
    check(y, yc)


def test_long_schedule_replays_and_repeats():
    """200 updates at N = 10^4, far past the point where the residual is rounding: the oracle replayed on the
    GPU's near-tie signs gives the same factors (a sign taken otherwise at such an entry moves whole factors by
    1e-3 to 1e-2, so that two correct builds differ by as much), and the call repeats itself bit for bit."""
    n, k, m = 10000, 50, 12
    print("long schedule", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    wd = torch.randn((m, n), generator=g, device="cuda") * 0.02
    plan = K.kashin_plan(n, 21, k)
    u, v, r, u2, v2, ut, vt = (torch.empty_like(wd) for _ in range(7))
    K.kashin_decompose_schedule(plan, "alternating", wd, u, v, r)
    for fill in (0.0, 7.0):
        u2.fill_(fill)
        v2.fill_(fill)
        K.kashin_decompose_schedule(plan, "alternating", wd, u2, v2, r)
        assert torch.equal(u, u2) and torch.equal(v, v2)
    rows = torch.arange(m, dtype=torch.int64, device="cuda")
    sg = torch.empty((m, 4 * k, n), dtype=torch.int8, device="cuda")
    cs, r2 = (torch.empty((m, 4 * k), device="cuda") for _ in range(2))
    ch = torch.empty((m, 4 * k), dtype=torch.int8, device="cuda")
    K.kashin_trace_schedule(plan, "alternating", wd, rows, sg, cs, ch, r2, ut, vt)
    torch.cuda.synchronize()
    assert torch.equal(u, ut) and torch.equal(v, vt)
    w = wd.cpu().numpy().astype(np.float64)
    winf = np.abs(w).max(axis=1)
    rep = ref.decompose_schedule(w, ref.sign_mask(n, 21), 4 * k, "alternating", replay_signs=sg.cpu().numpy(),
                                 replay_choices=ch.cpu().numpy(), tau=pu.TAU_REL * winf, choice_band=1e-5)
    du = (np.abs(u.cpu().numpy() - rep["u"]).max(axis=1) / winf).max()
    dv = (np.abs(v.cpu().numpy() - rep["vhat"]).max(axis=1) / winf).max()
    print(f"du={du:.2e} dv={dv:.2e}", flush=True)
    assert not rep["replay_outside"].any()
    assert du <= pu.TOL_FACTOR and dv <= pu.TOL_FACTOR

"""The launch forms that a call's size selects give the same bits.

Every sum of a cell is taken in the same order whatever the tile, so the rows
of a small call must equal those rows of a large one exactly (tolerance 0).
The large call's form is checked against the oracle by the parity tests.
"""
import ctypes

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_0907_3768_amd as dust  # noqa: E402


def _inputs(n_cells, n_lambda, n_species, n_sizes, mode, seed, pad=0, **options):
    g = synth.make_grid(n_lambda, n_species, n_sizes)
    p = synth.cell_params(n_cells, seed)
    J = torch.empty((n_cells, n_lambda + pad), dtype=torch.float32, device="cuda")[:, :n_lambda]
    synth.radiation_field(p, g.lam, device="cuda", out=J)
    m = torch.as_tensor(p.m_dust, dtype=torch.float32, device="cuda")
    return dust.Plan(g, mode, **options), J, m


@pytest.mark.parametrize("n_lambda,n_species,n_sizes", [
    (96, 2, 20),     # three blocks: always 16-cell tiles
    (129, 1, 33),    # five blocks, an odd last group of grains
    (301, 2, 40),    # ten blocks
    (1000, 1, 45),   # 32 blocks
    (250, 1, 32),    # few grains: always 16-cell tiles
])
def test_emission_forms_agree(n_lambda, n_species, n_sizes):
    nb = (n_lambda + 31) // 32
    n = 16 * (73728 // nb) + 37            # more (16 cells, block) tasks than any small form takes
    plan, J, m = _inputs(n, n_lambda, n_species, n_sizes, "table", 11)
    T = plan.solve(plan.absorb(J))
    T[5, :3] = 0.0
    T[9, 1] = float("nan")
    L = plan.emit(T, m)
    for rows in (1, 5, 63, 1000, 16 * (9216 // nb), 16 * (9216 // nb) + 1, n - 40):
        part = torch.full((rows + 1, n_lambda + 3), -1.0, device="cuda")
        plan.emit(T[:rows], m[:rows], part[:rows, :n_lambda])
        assert torch.equal(part[:rows, :n_lambda].nan_to_num(-3.0), L[:rows].nan_to_num(-3.0)), rows
        assert bool((part[rows] == -1.0).all()) and bool((part[:, n_lambda:] == -1.0).all())


@pytest.mark.parametrize("lookup", ["default", "f32", "polish"])
@pytest.mark.parametrize("n_lambda,hi_um,tmin", [(120, 1000.0, 2.7), (250, 100.0, 10.0),
                                                 (8, 1000.0, 2.7)])
def test_temperatures_below_the_table(n_lambda, hi_um, tmin, lookup):
    """Pairs from just below the table's lowest T down to a sixth of it:
    over the whole second table (down to a third) and below that one.
    Bound on T, given the heating: the second table's interpolation (1e-8 on
    the coarsest grid) and ln H' to 4e-8 (a fifth of it or less in T), plus the
    FP32 exponential, its correction and the rounding, 2 ulp = 2.4e-7."""
    g = synth.make_grid(n_lambda, 2, 5, hi_um=hi_um)
    T = np.geomspace(0.99 * tmin, tmin / 6.0, 700)
    c1, c2 = 2 * 6.62607015e-34 * 299792458.0 ** 2, 6.62607015e-34 * 299792458.0 / 1.380649e-23
    B = c1 / g.lam ** 5 / np.expm1(np.minimum(c2 / (g.lam * T[:, None]), 700.0))
    scale = 2.0 ** 60  # keeps H in FP32's normal range (the emission weights unchanged)
    g.c_abs, g.weight = g.c_abs * scale, g.weight / scale
    H = np.maximum(B @ (g.c_abs * g.dlam).T, 0.0).astype(np.float32)
    keep = (H > 1e-37).all(axis=1)
    H = H[keep]
    assert len(H) > 400
    ref = oracle.temperature(H.astype(np.float64), g.lam, g.dlam, g.c_abs, g.size)
    plan = dust.Plan(g, "mixed", ltab_tmin=tmin, f32_lookup=lookup == "f32",
                     newton_polish=lookup == "polish")
    cnt = dust.new_counters()
    out = plan.solve(torch.as_tensor(H, device="cuda"), counters=cnt).cpu().numpy()
    assert np.abs(out / ref - 1.0).max() <= 3e-7
    assert cnt.tolist()[:3] == [0, 0, H.size]


@pytest.mark.parametrize("mode,lookup", [("mixed", "default"), ("mixed", "f32"),
                                         ("mixed", "polish"), ("table", "default")])
@pytest.mark.parametrize("n_cells,n_lambda,n_species,n_sizes,pad", [
    (1, 380, 1, 16, 0),       # one cell, one grain tile, ragged last k-step
    (33, 127, 3, 17, 2),      # 3 full k-steps and a ragged one, ragged grains, J unaligned
    (130, 128, 2, 40, 0),     # whole k-steps, aligned rows
    (515, 161, 1, 45, 3),     # one group of k-steps and two left over
    (8192, 1000, 1, 16, 0),   # the most cells of the two-kernel form
    (6145, 400, 1, 16, 0),    # one more than it takes of short rows (one kernel)
    (100, 30, 3, 80, 1),      # no full k-step
])
def test_two_kernel_form_of_small_fused_calls(n_cells, n_lambda, n_species, n_sizes, pad, mode,
                                              lookup):
    """A small fused call gives the one-kernel form's T, SED and counters, on
    cells of every kind: no field, NaN, negative and infinite intensity, too
    cold for both tables, hotter than the table, with an extra heating."""
    options = {"f32_lookup": lookup == "f32", "newton_polish": lookup == "polish"}
    plan, J, m = _inputs(n_cells, n_lambda, n_species, n_sizes, mode, 7, pad, **options)
    one = dust.Plan(synth.make_grid(n_lambda, n_species, n_sizes), mode, fused_kernels=1,
                    **options)
    S = plan.n_grains
    for c, f in ((3, 0.0), (4, float("nan")), (7, -1.0), (9, 1e-14), (20, 1e12), (21, 1e-8),
                 (24, float("inf"))):
        if c < n_cells:
            J[c] *= f
    Q = torch.zeros((n_cells, S + 1), device="cuda")
    Q[::5] = 1e-20
    for q in (None, Q):
        out = []
        for p in (one, plan):
            T = torch.full((n_cells + 1, S + 2), -1.0, device="cuda")
            L = torch.full((n_cells + 1, n_lambda + 3), -1.0, device="cuda")
            cnt = dust.new_counters()
            p.fused(J, m, T[:n_cells, :S], L[:n_cells, :n_lambda], counters=cnt, Q=q)
            out.append((T.nan_to_num(-3.0), L.nan_to_num(-3.0), cnt))
        for a, b in zip(*out):
            assert torch.equal(a, b)


@pytest.mark.parametrize("n_cells,n_lambda,n_species,n_sizes", [
    (1, 8, 1, 1),            # one pair
    (17, 33, 1, 5),          # four lanes per cell, a ragged cell block and grain group
    (64, 127, 3, 17),
    (130, 1000, 1, 33),
    (1220, 64, 1, 80),       # 1600 (64 cells, grain) waves: one lane per cell
    (2050, 65, 1, 53),       # ragged in cells, wavelengths and grains
    (70, 10, 2, 30),         # more grains than wavelengths
])
def test_plain_solve_forms(n_cells, n_lambda, n_species, n_sizes):
    """The FP32 Newton, cold and warm-started, with an extra heating and in the
    fused call, against the oracle.  Bound on T: rounding of ln P and ln H (up
    to 80: 4.8e-6 each) and of the FP32 sum (terms to 5e-7), over a slope of at
    least 4, plus the heating's FP32 sum: 5e-6 covers them (the grids below 64
    wavelengths put Newton outside its table too)."""
    plan, J, m = _inputs(n_cells, n_lambda, n_species, n_sizes, "plain", 21, 1)
    g = synth.make_grid(n_lambda, n_species, n_sizes)
    if n_cells > 20:
        J[5] = 0.0
        J[6] *= 1e-9    # colder than the start table
        J[7] *= 1e9     # hotter
    Q = torch.zeros((n_cells, g.n_grains), device="cuda")
    Q[::3] = 1e-21
    rows = np.unique(np.r_[np.arange(min(n_cells, 60)), n_cells - 1])
    for q in (None, Q):
        H, T, L = plan.run(J, m, Q=q)
        ref = oracle.temperature(H[rows].cpu().numpy().astype(np.float64)
                                 + (0 if q is None else q[rows].cpu().numpy()),
                                 g.lam, g.dlam, g.c_abs, g.size)
        ok = ref > 0
        warm = torch.where(T > 0, T * 1.01, T)
        outs = [T, plan.solve(H, T=warm.clone(), Q=q, warm_start=True)]
        for t0 in (None, warm):
            Tf, Lf = plan.fused(J, m, T=None if t0 is None else t0.clone(), Q=q,
                                warm_start=t0 is not None)
            outs.append(Tf)
            assert torch.allclose(Lf[rows], L[rows], rtol=2e-3, atol=float(L.max()) * 1e-12)
        for t in outs:
            t = t[rows].cpu().numpy()
            assert np.abs(t[ok] / ref[ok] - 1.0).max() <= 5e-6
            assert (t[~ok] == 0).all()


@pytest.mark.parametrize("mode", ["plain", "mixed"])
@pytest.mark.parametrize("n_lambda,n_sizes,pad", [
    (31, 9, 0),      # one grain tile, no full k-step
    (32, 30, 1),     # two tiles, one k-step
    (161, 48, 0),    # three
    (130, 55, 2),    # four, rows on even floats
    (65, 77, 3),     # five
    (97, 113, 0),    # eight
    (64, 150, 1),    # ten
])
def test_heating_forms_agree(n_lambda, n_sizes, pad, mode):
    """H of the first rows of a large call equals that of the small calls, whose
    waves take fewer tiles and whose J starts elsewhere (each alignment)."""
    tiles = (n_sizes + 15) // 16
    n = 16 * (6144 // tiles) + 530
    plan, J, _ = _inputs(n, n_lambda, 1, n_sizes, mode, 5, pad)
    H = plan.absorb(J)
    g = synth.make_grid(n_lambda, 1, n_sizes)
    ref = oracle.heating(J[:40].cpu().numpy().astype(np.float64), g.c_abs, g.dlam)
    assert np.abs(H[:40].cpu().numpy() / ref - 1.0).max() <= 1e-4
    for first, rows in ((0, 1), (1, 33), (2, 16 * (1024 // tiles)), (3, 16 * (1024 // tiles) + 1),
                        (0, 16 * (4096 // tiles) + 1), (1, n - 500)):
        out = torch.full((rows + 1, n_sizes + 2), -1.0, device="cuda")
        plan.absorb(J[first:first + rows], out[:rows, :n_sizes])
        assert torch.equal(out[:rows, :n_sizes], H[first:first + rows]), (first, rows)
        assert bool((out[rows] == -1.0).all()) and bool((out[:, n_sizes:] == -1.0).all())


@pytest.mark.parametrize("mode,lookup", [("mixed", "default"), ("mixed", "f32"),
                                         ("mixed", "polish"), ("table", "default")])
def test_table_solve_forms_agree(mode, lookup):
    """T of the first rows of a large call (256 cells per workgroup) equals that
    of small ones, on cells of every kind and with an extra heating, and only
    the grains' columns are written."""
    n, S = 16 * 1024 * 16 // 3 + 77, 45  # 1026 blocks of (256 cells, 16 grains)
    plan, J, _ = _inputs(n, 40, 1, S, mode, 9, f32_lookup=lookup == "f32",
                         newton_polish=lookup == "polish")
    H = plan.absorb(J)
    for c, h in ((3, 0.0), (4, float("nan")), (7, -1e-20), (9, 1e-37), (70, 1e3), (71, 3e-30),
                 (200, float("inf"))):
        H[c] = h
    Q = torch.zeros((n, S + 3), device="cuda")
    Q[::5] = 1e-20
    for q in (None, Q):
        big, small = dust.new_counters(), dust.new_counters()
        T = plan.solve(H, Q=q, counters=big)
        out = torch.full((n + 1, S + 2), -7.0, device="cuda")
        for c in range(0, n, 40000):
            e = min(n, c + 40000)
            plan.solve(H[c:e], out[c:e, :S], counters=small, Q=None if q is None else q[c:e])
        assert torch.equal(out[:n, :S].nan_to_num(-3.0), T.nan_to_num(-3.0))
        assert bool((out[n] == -7.0).all()) and bool((out[:, S:] == -7.0).all())
        assert torch.equal(big, small) and int(big[0]) == 3 * S


@pytest.mark.parametrize("n_lambda,n_sizes,n_levels", [
    (250, 3, 64),     # four wavelengths per lane, the packed upper half at its longest
    (257, 2, 34),     # eight per lane, one packed level
    (600, 1, 33),     # any number, no packed level; odd level count
    (40, 2, 5),
    (250, 2, 80),     # two levels per lane (one cell per wave)
])
def test_fluctuating_forms_agree(n_lambda, n_sizes, n_levels):
    """The distributions of a cell do not depend on the call it is in (which
    cell shares its wave, how many cells a workgroup takes, how J is aligned),
    with a neighbour that is NaN; nor does the averaged emission (one wave per
    tile, or 64-cell workgroups)."""
    g = synth.make_species_grid(n_lambda, [2], n_sizes)
    lev_T, lev_E = synth.fluct_levels(g, n_levels)
    n = 33000 // n_sizes
    p = synth.cell_params(n, 13)
    buf = torch.empty((n, n_lambda + 3), dtype=torch.float32, device="cuda")
    J = synth.radiation_field(p, g.lam, device="cuda", out=buf)[:, :n_lambda]
    J[2] = 0.0
    J[5, 3] = float("nan")
    m = torch.as_tensor(p.m_dust, dtype=torch.float32, device="cuda")
    plan = dust.FluctPlan(g, lev_T, lev_E)
    big = dust.new_counters()
    P = plan.solve_P(J, counters=big)
    ref = oracle.fluct_distribution(J[6:16].cpu().numpy().astype(np.float64), g, lev_T, lev_E)
    out = P[6:16].cpu().numpy().reshape(ref.shape)
    seen = ref >= 1e-30
    assert np.abs(out[seen] / ref[seen] - 1.0).max() <= 1e-6
    assert bool(P[5].isnan().all()) and int(big[0]) == n_sizes
    L = plan.emit(P, m)
    for first, rows in ((0, 1), (1, 7), (4, 2), (3, 40), (0, 1000), (1, n - 1)):
        e = first + rows
        aligned = J[first:e].contiguous()
        for Jp in (J[first:e], aligned):
            Pp = plan.solve_P(Jp)
            assert torch.equal(Pp.nan_to_num(-1.0), P[first:e].nan_to_num(-1.0)), (first, rows)
        Lp = plan.emit(P[first:e], m[first:e])
        assert torch.equal(Lp.nan_to_num(-1.0), L[first:e].nan_to_num(-1.0)), (first, rows)


@pytest.mark.parametrize("n_lambda,n_species,n_sizes,ltab_n", [
    (8, 1, 5, 0),        # one partial wavelength step, one grain tile
    (16, 2, 8, 3000),    # one whole step; forward rows too long for LDS
    (129, 1, 81, 0),     # one step more than the eight waves take; one tile per workgroup
    (250, 3, 50, 0),     # two tiles per workgroup
    (301, 3, 75, 0),     # four tiles per workgroup and a rest of three
])
def test_refresh_forms(n_lambda, n_species, n_sizes, ltab_n):
    """The tables of every form of the refresh: T of heating in their range,
    given in FP32, against the oracle (mixed, polished on the forward table,
    whose cubic's error is below 1e-8; ln H' to 4e-8, rounding and FP32
    exponential 2 ulp) and against the linear interpolation in 64 bits (table:
    rounding, with 1 ulp for the reciprocal's argument), and the same bits from
    the refresh of a batch.  (The default lookup on a grid of 8 wavelengths
    adds its inverse table's own interpolation error, 3.5e-7.)"""
    g = synth.make_grid(n_lambda, n_species, n_sizes)
    scale = 2.0 ** 60  # keeps H in FP32's normal range (the emission weights unchanged)
    g.c_abs, g.weight = g.c_abs * scale, g.weight / scale
    T = np.geomspace(12.0, 1200.0, 61)
    c1, c2 = 2 * 6.62607015e-34 * 299792458.0 ** 2, 6.62607015e-34 * 299792458.0 / 1.380649e-23

    def power(t):
        B = c1 / g.lam ** 5 / np.expm1(np.minimum(c2 / (g.lam * t[:, None]), 700.0))
        return B @ (g.c_abs * g.dlam).T

    H = power(T).astype(np.float32)
    Hd = torch.as_tensor(H, device="cuda")
    n = ltab_n or 2000
    plan = dust.Plan(g, "table", ltab_n=ltab_n)
    out = plan.solve(Hd).cpu().numpy()
    t = 3.0 + np.arange(n) * (1500.0 - 3.0) / (n - 1)
    P = power(t)
    ref = np.stack([np.interp(H[:, s].astype(np.float64), P[:, s], t)
                    for s in range(g.n_grains)], axis=1)
    assert np.abs(out / ref - 1.0).max() <= 1.2e-7
    polished = dust.Plan(g, "mixed", ltab_n=ltab_n, newton_polish=True)
    ref = oracle.temperature(H.astype(np.float64), g.lam, g.dlam, g.c_abs, g.size)
    assert np.abs(polished.solve(Hd).cpu().numpy() / ref - 1.0).max() <= 3e-7
    plan = dust.Plan(g, "mixed", ltab_n=ltab_n)
    before = plan.solve(Hd)
    other = dust.Plan(synth.make_grid(200, 3, 80), "mixed")
    plans = [plan, other, plan]
    args = []
    for k, p in enumerate(plans):
        J = torch.rand((20 + k, p.n_lambda), device="cuda")
        args.append((J, torch.ones(20 + k, device="cuda"),
                     torch.empty((20 + k, p.n_grains), device="cuda"), torch.empty_like(J)))
    b = dust.Batch(plans, *[list(a) for a in zip(*args)], refresh_plans=True)
    b.launch()
    torch.cuda.synchronize()
    assert torch.equal(plan.solve(Hd), before)


@pytest.mark.parametrize("n_lambda,n_sizes", [(60, 9), (97, 17), (300, 40)])
def test_emission_over_every_form(n_lambda, n_sizes):
    """Cells of one temperature, 3 K to 1e5 K, so that each block of wavelengths
    meets every form of the Planck term, against 64 bits.  Bound for
    x = hc/(k lam T): the exponent's factors and product, 4 roundings times its
    sensitivity x / (1 - e^-x); e^x and 1 / (e^x - 1), 2 units each, the first
    over 1 - e^-x; the cut series, 1; the weights and the sum, n_sizes + 4
    roundings."""
    g = synth.make_grid(n_lambda, 1, n_sizes)
    T = np.geomspace(3.0, 1e5, 400).astype(np.float32)
    Td = torch.as_tensor(np.repeat(T[:, None], n_sizes, axis=1), device="cuda")
    L = dust.Plan(g, "plain").emit(Td).cpu().numpy()
    c1, c2 = 2 * 6.62607015e-34 * 299792458.0 ** 2, 6.62607015e-34 * 299792458.0 / 1.380649e-23
    x = c2 / (g.lam * T[:, None].astype(np.float64))
    em = (g.weight[:, None] * g.c_abs * c1 / g.lam ** 5).sum(axis=0)
    with np.errstate(over="ignore"):
        ref = em / np.expm1(x)
    tol = 2.0 ** -24 * ((4 * x + 4) / -np.expm1(-x) + 5 + n_sizes + 4)
    seen = (x < 100.0) & (ref > 1e-25 * em.max())
    assert seen.sum() > 0.5 * x.size
    assert (np.abs(L[seen] / ref[seen] - 1.0) <= tol[seen]).all()


@pytest.mark.parametrize("n_cells,n_lambda", [
    ((1,), 600),               # five workgroups share the only tile
    ((33, 5, 700), 301),       # three rounds of blocks, fewer in the other grids
    ((300, 40, 0, 17), 96),    # fewer than four blocks in every grid: no split
    ((24576,), 250),           # as many tiles as workgroups are resident: no split
])
@pytest.mark.parametrize("in_place", [False, True])
def test_batches_of_few_tiles(n_cells, n_lambda, in_place):
    """A batch gives the one-kernel fused call's T and SED bit for bit and its
    counters once, however many workgroups share a tile, also where L is J."""
    J, m, plans, ref = [], [], [], []
    cnt1, cnt2, cnt3 = dust.new_counters(), dust.new_counters(), dust.new_counters()
    for k, n in enumerate(n_cells):
        nl = max(30, n_lambda - 71 * k)
        p, j, d = _inputs(max(n, 1), nl, 1 + k % 3, 17 + 16 * k, "mixed", 5 + k, fused_kernels=1)
        j, d = j[:n], d[:n]
        for c, f in ((3, 0.0), (4, float("nan")), (9, 1e-14), (16, 1e12)):
            if c < n:
                j[c] *= f
        plans.append(p), J.append(j), m.append(d)
        ref.append(p.fused(j, d, counters=cnt1))
    T = [torch.empty_like(r[0]) for r in ref]
    src = [j.clone() for j in J]
    L = src if in_place else [torch.empty_like(j) for j in src]
    b = dust.Batch(plans, src, m, T, L, counters=cnt2)
    for j, s in zip(J, src):  # the tuner has run on the bound buffers
        s.copy_(j)
    cnt2.zero_()
    b.launch()
    for again in (False, True):
        for r, t, l in zip(ref, T, L):
            assert torch.equal(t.nan_to_num(-3.0), r[0].nan_to_num(-3.0))
            assert torch.equal(l.nan_to_num(-3.0), r[1].nan_to_num(-3.0))
        if not again:
            for j, s in zip(J, src):
                s.copy_(j)
            dust.batch_run(plans, src, m, T, L, counters=cnt3)
    assert cnt1.tolist() == cnt2.tolist() == cnt3.tolist()


def _power(g, T):
    """The right side of Eq. 7 in 64 bits, [len(T), S]."""
    c1, c2 = 2 * 6.62607015e-34 * 299792458.0 ** 2, 6.62607015e-34 * 299792458.0 / 1.380649e-23
    B = c1 / g.lam ** 5 / np.expm1(np.minimum(c2 / (g.lam * np.asarray(T)[:, None]), 700.0))
    return B @ (g.c_abs * g.dlam).T


def _bright_grid(n_lambda, n_species, n_sizes, **kw):
    """A grid whose H stays in FP32's normal range down to a few tenths of a
    kelvin (the emission weights unchanged)."""
    g = synth.make_grid(n_lambda, n_species, n_sizes, **kw)
    scale = 2.0 ** 60
    g.c_abs, g.weight = g.c_abs * scale, g.weight / scale
    return g


@pytest.mark.parametrize("maxit", [0, 8])
@pytest.mark.parametrize("factor", [1.001, 0.999])
def test_plain_warm_starts_beside_the_table(factor, maxit):
    """A warm start 0.1 % off its root takes a few iterations wherever the root
    lies: far below the start table (0.9 K), at its ends and far above
    (3000 K).  Newton in ln T leaves K r^2 / 2 of a residual r <= 0.001 x / 1,
    x <= 240 (0.2 K at 1000 um): two evaluations of the sum and the accepting
    one, or three on the table and one.  Bound on T as in test_plain_solve_forms."""
    g = _bright_grid(250, 1, 7)
    for T in (0.3, 0.5, 0.85, 0.87, 0.95, 20.0, 2990.0, 3010.0, 3100.0, 5000.0, 1e5):
        H = np.repeat(_power(g, [T]), 70, axis=0).astype(np.float32)
        ref = oracle.temperature(H[:1].astype(np.float64), g.lam, g.dlam, g.c_abs, g.size)
        Hd = torch.as_tensor(H, device="cuda")
        warm = torch.as_tensor(np.repeat(ref * factor, 70, axis=0).astype(np.float32),
                               device="cuda")
        for one_kernel in (0, 1):
            plan = dust.Plan(g, "plain", maxit=maxit, fused_kernels=one_kernel)
            cnt = dust.new_counters()
            if one_kernel:  # the heating as the extra term of cells without a field
                out, _ = plan.fused(torch.zeros((70, 250), device="cuda"), T=warm.clone(), Q=Hd,
                                    warm_start=True, counters=cnt)
            else:
                out = plan.solve(Hd, T=warm.clone(), warm_start=True, counters=cnt)
            assert np.abs(out.cpu().numpy() / ref - 1.0).max() <= 5e-6, T
            assert int(cnt[1]) == 0 and int(cnt[3]) <= (4 if 0.9 < T < 3000 else 3) * H.size, T


@pytest.mark.parametrize("n_lambda", [2, 3, 4, 5])
@pytest.mark.parametrize("tol", [0.0, 1e-3])
def test_plain_tolerance_on_coarse_grids(n_lambda, tol):
    """On a few wavelengths ln P is far from a power of T, so only a residual
    within the tolerance ends the iteration.  Bound on T: what the last step
    leaves, K tol^2 / 2 of the residual with K <= 30 there (neighbouring
    wavelengths up to a factor 105 apart: K <= 105 / 4), and rounding: of nu, of 1/T, of their product (6e-8
    each: T moves by as much), of the exponential, the reciprocal, the sum and
    the logarithm (4e-7 over a slope of at least 1) and of T and its exponential
    (1.8e-7): 8e-7.  (Two wavelengths only to 60 K: beyond, the FP32 e^x - 1 at
    1000 um itself cancels.)"""
    g = _bright_grid(n_lambda, 1, 6)
    T = np.geomspace(4.0, 60.0 if n_lambda == 2 else 2000.0, 500)
    H = _power(g, T).astype(np.float32)
    H = H[(H > 1e-36).all(axis=1)]
    ref = oracle.temperature(H.astype(np.float64), g.lam, g.dlam, g.c_abs, g.size)
    Hd = torch.as_tensor(H, device="cuda")
    bound = 8e-7 + 15.0 * (tol or 1e-5) ** 2
    for one_kernel in (0, 1):
        plan = dust.Plan(g, "plain", tol=tol, fused_kernels=one_kernel)
        cnt = dust.new_counters()
        outs = [plan.fused(torch.zeros((len(H), n_lambda), device="cuda"), Q=Hd, counters=cnt)[0],
                plan.solve(Hd, counters=cnt)]
        for f in (0.999, 1.001, 1.0003):
            warm = torch.as_tensor((ref * f).astype(np.float32), device="cuda")
            outs.append(plan.solve(Hd, T=warm, warm_start=True, counters=cnt))
        assert int(cnt[1]) == 0
        for t in outs:
            assert np.abs(t.cpu().numpy() / ref - 1.0).max() <= bound


@pytest.mark.parametrize("n_cells,n_lambda,n_sizes", [
    (50, 7, 33), (50, 8, 33), (4097, 31, 33), (4097, 32, 33),   # more than 16 grains
    (300, 127, 16), (300, 128, 16), (32769, 63, 5), (32769, 64, 5),
])
def test_plain_fused_forms(n_cells, n_lambda, n_sizes):
    """The plain fused call beside its lines between one kernel and three, cold
    and warm-started, against the one-kernel form: the two differ by the order
    of their sums (T within twice the bound of test_plain_solve_forms) and the
    events they count are the same."""
    plan, J, m = _inputs(n_cells, n_lambda, 1, n_sizes, "plain", 31, 1)
    one = dust.Plan(synth.make_grid(n_lambda, 1, n_sizes), "plain", fused_kernels=1)
    J[5] = 0.0
    J[11] *= float("nan")
    Q = torch.zeros((n_cells, n_sizes), device="cuda")
    Q[::3] = 1e-21
    c0, c1 = dust.new_counters(), dust.new_counters()
    T0, L0 = one.fused(J, m, Q=Q, counters=c0)
    outs = [plan.fused(J, m, Q=Q, counters=c1),
            plan.fused(J, m, Q=Q, T=T0 * 1.01, warm_start=True)]
    for T, L in outs:
        assert torch.equal(T.isnan(), T0.isnan()) and torch.equal(L.isnan(), L0.isnan())
        assert torch.allclose(T.nan_to_num(), T0.nan_to_num(), rtol=1e-5, atol=0.0)
        assert torch.allclose(L.nan_to_num(), L0.nan_to_num(), rtol=2e-3,
                              atol=float(L0.nan_to_num().max()) * 1e-12)
    assert c0.tolist()[:3] == c1.tolist()[:3] == [n_sizes, 0, 0]


@pytest.mark.parametrize("lookup", ["default", "f32", "polish"])
@pytest.mark.parametrize("n_lambda,hi_um,tmin", [(2, 1000.0, 2.7), (3, 1000.0, 60.0),
                                                 (8, 1000.0, 2.7), (8, 1000.0, 100.0),
                                                 (30, 1000.0, 2.7), (250, 100.0, 10.0),
                                                 (600, 1000.0, 2.7)])
def test_temperatures_below_the_table_are_rounded_once(n_lambda, hi_um, tmin, lookup):
    """Below the table T is the FP64 result rounded to FP32 on every grid, by
    the second table (or the exact solve where a grain has none) and below it,
    in every path.  Bound, given the heating: half a unit of FP32 (6.0e-8) and
    1e-9, doubled, of the second table and of the exact solve's last step."""
    g = _bright_grid(n_lambda, 1, 5, hi_um=hi_um)
    T = np.geomspace(0.999 * tmin, tmin / 4.0, 700)
    H = np.maximum(_power(g, T), 0.0).astype(np.float32)
    H = H[(H > 1e-36).all(axis=1)]
    assert len(H) > 400
    ref = oracle.temperature(H.astype(np.float64), g.lam, g.dlam, g.c_abs, g.size)
    Hd = torch.as_tensor(H, device="cuda")
    J = torch.zeros((len(H), n_lambda), device="cuda")
    for fused_kernels in (0, 1, 2):
        plan = dust.Plan(g, "mixed", ltab_tmin=tmin, f32_lookup=lookup == "f32",
                         newton_polish=lookup == "polish", fused_kernels=fused_kernels)
        cnt = dust.new_counters()
        for out in (plan.solve(Hd, counters=cnt), plan.fused(J, Q=Hd, counters=cnt)[0]):
            assert np.abs(out.cpu().numpy() / ref - 1.0).max() <= 6.0e-8 + 2e-9
        assert cnt.tolist()[:3] == [0, 0, 2 * H.size]


@pytest.mark.parametrize("mode", ["plain", "mixed", "table"])
@pytest.mark.parametrize("n_cells,n_lambda,n_sizes", [
    (1, 250, 40),       # two columns of blocks, or one
    (70, 250, 80),      # four-cell tiles
    (3000, 130, 40),    # eight-cell tiles
    (900, 100, 20),     # 16-cell tiles
])
def test_sed_over_the_temperatures(n_cells, n_lambda, n_sizes, mode):
    """L may take the memory of T (rows of one length, T in the first columns):
    an emission of up to 256 wavelengths, a fused call and a batch, against the
    same calls on memory of their own, bit for bit."""
    plan, J, m = _inputs(n_cells, n_lambda, 1, n_sizes, mode, 17)
    T = plan.solve(plan.absorb(J))
    buf = torch.empty((n_cells, n_lambda), device="cuda")
    for _ in range(3):
        buf.fill_(-1.0)
        buf[:, :n_sizes] = T
        plan.emit(buf, m, buf)
        assert torch.equal(buf, plan.emit(T, m))
    for fused_kernels in (1, 0):
        p = dust.Plan(synth.make_grid(n_lambda, 1, n_sizes), mode, fused_kernels=fused_kernels)
        if fused_kernels:
            _, L = p.fused(J, m)  # (the one-kernel form, which memory in common takes)
        buf.fill_(-1.0)
        p.fused(J, m, buf, buf)
        assert torch.equal(buf, L)
    if mode == "plain":  # T holds the start temperatures too
        buf[:, :n_sizes] = T * 1.01
        plan.fused(J, m, buf, buf, warm_start=True)
        assert torch.allclose(buf, L, rtol=2e-3, atol=float(L.max()) * 1e-12)
    if mode == "mixed":
        for _ in range(2):
            buf.fill_(-1.0)
            dust.batch_run([plan], [J], [m], [buf], [buf])
            assert torch.equal(buf, L)
        b = dust.Batch([plan], [J], [m], [buf], [buf])
        buf.fill_(-1.0)
        b.launch()
        assert torch.equal(buf, L)


@pytest.mark.parametrize("mode", ["plain", "mixed"])
@pytest.mark.parametrize("n_cells,n_lambda,n_sizes,pad", [
    (1, 64, 40, 0),
    (500, 300, 240, 0),       # many grain tiles of few cells
    (40000, 250, 80, 0),      # 256-cell blocks, J rows aligned
    (40000, 161, 130, 2),     # and not
    (40000, 100, 98, 0),      # grains into the ragged last k-step
    (9000, 320, 300, 1),      # more grains than one pass of the blocked kernel
])
def test_heating_over_the_field(n_cells, n_lambda, n_sizes, pad, mode):
    """H may take the memory of J (the first columns of its rows): the same
    bits as in memory of its own."""
    plan, J, _ = _inputs(n_cells, n_lambda, 1, n_sizes, mode, 19, pad)
    H = plan.absorb(J)
    for _ in range(3):
        buf = torch.empty((n_cells, n_lambda + pad), device="cuda")[:, :n_lambda]
        buf.copy_(J)
        plan.absorb(buf, buf)
        assert torch.equal(buf[:, :n_sizes], H) and torch.equal(buf[:, n_sizes:], J[:, n_sizes:])


@pytest.mark.parametrize("mode", ["plain", "mixed"])
@pytest.mark.parametrize("n_cells,n_lambda,n_sizes,pad", [
    (400000, 12, 240, 0),     # H larger than the caches, short rows
    (33000, 16, 50, 0), (33000, 64, 50, 0), (32000, 40, 81, 1),
    (36000, 47, 40, 1), (36000, 48, 40, 1), (16000, 30, 40, 3),  # short rows on odd floats
    (36000, 60, 130, 1), (50000, 60, 130, 1),                     # many grains
])
def test_heating_of_short_rows(n_cells, n_lambda, n_sizes, pad, mode):
    """The forms that short rows and rows on odd floats take, against the first
    rows' own call bit for bit and the oracle, with no column past the last
    grain written."""
    plan, J, _ = _inputs(n_cells, n_lambda, 1, n_sizes, mode, 23, pad)
    out = torch.full((n_cells + 1, n_sizes + 2), -1.0, device="cuda")
    plan.absorb(J, out[:n_cells, :n_sizes])
    assert bool((out[n_cells] == -1.0).all()) and bool((out[:, n_sizes:] == -1.0).all())
    for first, rows in ((0, 40), (n_cells - 33, 33), (1, 1700)):
        assert torch.equal(plan.absorb(J[first:first + rows]),
                           out[first:first + rows, :n_sizes]), first
    g = synth.make_grid(n_lambda, 1, n_sizes)
    ref = oracle.heating(J[:40].cpu().numpy().astype(np.float64), g.c_abs, g.dlam)
    assert np.abs(out[:40, :n_sizes].cpu().numpy() / ref - 1.0).max() <= 1e-4


@pytest.mark.parametrize("n_cells,n_lambda,n_sizes,n_levels", [
    (1, 128, 4, 40), (300, 100, 3, 64), (500, 17, 1, 33),
])
def test_averaged_sed_over_the_distributions(n_cells, n_lambda, n_sizes, n_levels):
    """L may take the memory of P (the first columns of its rows) up to 128
    wavelengths: the same bits as in memory of its own."""
    g = synth.make_species_grid(n_lambda, [2], n_sizes)
    p = synth.cell_params(n_cells, 13)
    J = synth.radiation_field(p, g.lam, device="cuda")
    m = torch.as_tensor(p.m_dust, dtype=torch.float32, device="cuda")
    plan = dust.FluctPlan(g, *synth.fluct_levels(g, n_levels))
    P = plan.solve_P(J)
    L = plan.emit(P, m)
    for _ in range(3):
        buf = P.clone()
        plan.emit(buf, m, buf)
        assert torch.equal(buf[:, :n_lambda], L) and torch.equal(buf[:, n_lambda:], P[:, n_lambda:])


@pytest.mark.parametrize("n_lambda,n_sizes,n_levels", [
    (513, 1, 64), (1500, 2, 16), (2500, 1, 64), (4095, 1, 64), (4095, 2, 5),
])
def test_fluctuating_many_wavelengths(n_lambda, n_sizes, n_levels):
    """The distributions on grids of which a CU holds few cells' prefix sums, to
    the largest that is taken: against the oracle, and cell by cell the same in
    calls of one and of all."""
    g = synth.make_species_grid(n_lambda, [2], n_sizes)
    lev_T, lev_E = synth.fluct_levels(g, n_levels)
    p = synth.cell_params(37, 13)
    J = synth.radiation_field(p, g.lam, device="cuda")
    J[2] = 0.0
    J[5, n_lambda - 1] = float("nan")
    plan = dust.FluctPlan(g, lev_T, lev_E)
    cnt = dust.new_counters()
    P = plan.solve_P(J, counters=cnt)
    ref = oracle.fluct_distribution(J[6:12].cpu().numpy().astype(np.float64), g, lev_T, lev_E)
    out = P[6:12].cpu().numpy().reshape(ref.shape)
    seen = ref >= 1e-30
    assert np.abs(out[seen] / ref[seen] - 1.0).max() <= 1e-6
    assert bool(P[5].isnan().all()) and int(cnt[0]) == n_sizes
    for c in (0, 2, 4, 5, 36):
        one = plan.solve_P(J[c:c + 1])
        assert torch.equal(one.nan_to_num(-1.0), P[c:c + 1].nan_to_num(-1.0))


@pytest.mark.parametrize("mode,lookup,sizes", [
    ("mixed", "default", (1, 12, 13, 17, 24, 25)), ("mixed", "f32", (2, 16, 36, 37)),
    ("mixed", "polish", (3, 24, 33)), ("table", "default", (1, 3, 4, 20)),
])
def test_table_solves_of_few_grains(mode, lookup, sizes):
    """T of many cells of few grains (pairs in row-major order, or 16-grain
    tiles) equals that of small calls bit for bit, with the same counters, on
    cells of every kind, a cluster of them hotter than the table among them,
    and only the grains' columns are written."""
    n = 262144
    for S in sizes:
        plan, J, _ = _inputs(n + 65, 40, 1, S, mode, 9, f32_lookup=lookup == "f32",
                             newton_polish=lookup == "polish")
        H = plan.absorb(J)
        for c, h in ((3, 0.0), (4, float("nan")), (7, -1e-20), (9, 1e-37), (71, 3e-30),
                     (200, float("inf")), (n - 1, 0.0), (n + 64, 1e3)):
            H[c] = h
        H[5000:5100] = 1e3
        Q = torch.zeros((n + 65, S + 3), device="cuda")
        Q[::5] = 1e-20
        for rows in (n - 1, n, n + 65):
            for q in (None, Q):
                big, small = dust.new_counters(), dust.new_counters()
                out = torch.full((rows + 1, S + 2), -7.0, device="cuda")
                plan.solve(H[:rows], out[:rows, :S], Q=q, counters=big)
                for c in range(0, rows, 70000):
                    e = min(rows, c + 70000)
                    part = plan.solve(H[c:e], Q=None if q is None else q[c:e], counters=small)
                    assert torch.equal(part.nan_to_num(-3.0), out[c:e, :S].nan_to_num(-3.0)), (S, rows)
                assert bool((out[rows] == -7.0).all()) and bool((out[:, S:] == -7.0).all())
                assert torch.equal(big, small) and int(big[0]) == 3 * S


def test_table_solve_of_more_cells_than_a_launch_holds():
    """2^30 cells and more of four grains, T in the memory of H: a launch's
    2^32 threads do not hold them."""
    k = (1 << 30) // 1000 + 2
    plan, J, _ = _inputs(1000, 40, 1, 4, "table", 9)
    H = plan.absorb(J)
    T = plan.solve(H).reshape(1, 4000)
    big = H.reshape(1, 4000).expand(k, 4000).contiguous()
    plan.solve(big.view(k * 1000, 4), big.view(k * 1000, 4))
    for c in range(0, k, 100000):
        assert bool((big[c:c + 100000] == T).all()), c


@pytest.mark.parametrize("lookup", ["default", "f32", "polish"])
@pytest.mark.parametrize("n_cells,n_lambda,n_sizes", [(1, 400, 16), (37, 600, 16), (50, 250, 65),
                                                      (20, 300, 131)])
def test_small_fused_calls_outside_the_table(n_cells, n_lambda, n_sizes, lookup):
    """A small fused call all of whose pairs are solved exactly (a table that
    ends below them): T, SED and counters of the one-kernel form, bit for bit."""
    kw = {"f32_lookup": lookup == "f32", "newton_polish": lookup == "polish", "ltab_tmax": 4.0}
    plan, J, m = _inputs(n_cells, n_lambda, 1, n_sizes, "mixed", 7, 1, **kw)
    one = dust.Plan(synth.make_grid(n_lambda, 1, n_sizes), "mixed", fused_kernels=1, **kw)
    cnt = dust.new_counters(), dust.new_counters()
    a, b = one.fused(J, m, counters=cnt[0]), plan.fused(J, m, counters=cnt[1])
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert torch.equal(*cnt) and int(cnt[0][2]) > 0.9 * n_cells * n_sizes


@pytest.mark.parametrize("n_sizes", [1, 16, 17])
@pytest.mark.parametrize("n_lambda", [250, 1000])
def test_emission_columns_of_few_grains(n_lambda, n_sizes):
    """Splitting a tile's wavelengths into columns (by the number of tiles and
    of grains) does not change a bit."""
    plan, J, m = _inputs(66000, n_lambda, 1, n_sizes, "table", 11)
    T = plan.solve(plan.absorb(J))
    L = plan.emit(T, m)  # one column
    for rows in (1, 500, 6000, 16384, 16385, 40000):
        assert torch.equal(plan.emit(T[:rows], m[:rows]), L[:rows]), rows


def _spoil(plan):
    """Every table that a refresh derives becomes NaN."""
    f = dust.lib().dust_test_spoil_tables
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_void_p]
    assert f(plan.handle) == dust.DUST_OK


@pytest.mark.parametrize("n_lambda,n_species,n_sizes,ltab_n", [
    (48, 1, 5, 0), (49, 1, 16, 0),        # one share of the wavelengths, two
    (96, 2, 17, 0), (97, 1, 40, 0),       # two, four
    (192, 1, 80, 0), (193, 3, 50, 0),     # four, eight
    (8, 1, 3, 16), (640, 3, 75, 0),       # the smallest; the most tiles of a workgroup
])
def test_refresh_rebuilds_every_table(n_lambda, n_species, n_sizes, ltab_n):
    """Tables filled with NaN are what they were after a refresh of one plan and
    after that of a batch, among other plans and with plans enough for each
    number of grain tiles per workgroup: T, SED and heating bit for bit, on
    temperatures in the table and below it."""
    g = _bright_grid(n_lambda, n_species, n_sizes)
    H = torch.as_tensor(np.maximum(_power(g, np.geomspace(1.5, 1200.0, 97)), 1e-37)
                        .astype(np.float32), device="cuda")
    J = torch.rand((97, n_lambda), device="cuda")

    def outputs(p):
        T = p.solve(H)
        return p.absorb(J), T, p.emit(T)

    plain = dust.Plan(g, "plain")
    want = outputs(plain)
    _spoil(plain)
    plain.prepare()
    assert all(torch.equal(a, b) for a, b in zip(outputs(plain), want))
    plan = dust.Plan(g, "mixed", ltab_n=ltab_n)
    want = outputs(plan)
    _spoil(plan)
    assert not torch.equal(outputs(plan)[0], want[0])
    plan.prepare()
    assert all(torch.equal(a, b) for a, b in zip(outputs(plan), want))
    for others in (0, 3, 12):
        plans = [plan] + [dust.Plan(synth.make_grid(60 + 70 * k, 1 + k % 3, 30), "mixed")
                          for k in range(others)]
        Jb = [torch.rand((5, p.n_lambda), device="cuda") for p in plans]
        b = dust.Batch(plans, Jb, [None] * len(plans),
                       [torch.empty((5, p.n_grains), device="cuda") for p in plans],
                       [torch.empty_like(j) for j in Jb], refresh_plans=True)
        for p in plans:
            _spoil(p)
        b.launch()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outputs(plan), want)), others


@pytest.mark.parametrize("specs", [
    [(1, 600, 40)],                                  # five parts
    [(40, 128, 30), (33, 129, 17), (17, 1000, 50)],  # a part that only some grids need
    [(16, 100, 20)] * 40 + [(16, 600, 80)],          # nor most of them
    [(50, 257, 140), (9, 96, 250)],                  # many grains
])
def test_batch_parts_write_everything(specs):
    """With T, L and the counters reset before each launch: a batch of few tiles
    (replayed, without autotuning, and one-shot) gives the one-kernel fused
    call's results bit for bit and counts each event once."""
    plans, J, m, ref = [], [], [], []
    want = dust.new_counters()
    for k, (n, nl, S) in enumerate(specs):
        p, j, d = _inputs(n, nl, 1, S, "mixed", 5 + k, fused_kernels=1)
        for c, f in ((3, 0.0), (4, float("nan")), (9, 1e-14)):
            if c < n:
                j[c] *= f
        plans.append(p), J.append(j), m.append(d)
        ref.append(p.fused(j, d, counters=want))
    T = [torch.empty_like(r[0]) for r in ref]
    L = [torch.empty_like(r[1]) for r in ref]
    cnt = dust.new_counters()
    tuned = dust.Batch(plans, J, m, T, L, counters=cnt)
    plain = dust.Batch(plans, J, m, T, L, counters=cnt, autotune=False)
    for call in (tuned.launch, plain.launch, tuned.launch,
                 lambda: dust.batch_run(plans, J, m, T, L, counters=cnt),
                 lambda: dust.batch_run(plans, J, m, T, L, counters=cnt, no_alloc=True)):
        for x in T + L:
            x.fill_(-7.0)
        cnt.zero_()
        call()
        for r, t, l in zip(ref, T, L):
            assert torch.equal(t.nan_to_num(-3.0), r[0].nan_to_num(-3.0))
            assert torch.equal(l.nan_to_num(-3.0), r[1].nan_to_num(-3.0))
        assert torch.equal(cnt, want)


@pytest.mark.parametrize("n_lambda,n_sizes", [(5, 17), (64, 16), (40, 45)])
def test_plain_solve_of_short_rows(n_lambda, n_sizes):
    """Sixteen grains per workgroup (short rows of many pairs) solve as four do:
    the rows of a smaller call, whose waves hold the same cells, bit for bit,
    cold and warm, with the same iterations, no column past the last grain
    written."""
    n = 64 * (30000000 // n_sizes // 64 + 1) + 70
    plan, J, _ = _inputs(64 * 1000, n_lambda, 1, n_sizes, "plain", 3)
    H1 = plan.absorb(J)
    H1[7] = 0.0
    H1[9] = float("nan")
    reps = (n + len(H1) - 1) // len(H1)
    H = H1.repeat(reps, 1)[:n]
    c1, c0 = dust.new_counters(), dust.new_counters()
    T1 = plan.solve(H1, counters=c1)
    out = torch.full((n + 1, n_sizes + 2), -7.0, device="cuda")
    plan.solve(H, out[:n, :n_sizes], counters=c0)
    for c in range(0, n, len(H1)):
        e = min(n, c + len(H1)) // 64 * 64  # (whole waves)
        assert torch.equal(out[c:e, :n_sizes].nan_to_num(-3.0), T1[:e - c].nan_to_num(-3.0)), c
    assert bool((out[n] == -7.0).all()) and bool((out[:, n_sizes:] == -7.0).all())
    whole = n // len(H1)
    assert int(c0[3]) >= whole * int(c1[3]) and int(c0[0]) >= whole * int(c1[0])
    warm = (out[:n, :n_sizes] * 1.01).contiguous()
    plan.solve(H, T=warm, warm_start=True)
    part = (T1[:64 * 50] * 1.01).contiguous()
    plan.solve(H1[:64 * 50], T=part, warm_start=True)
    T0 = T1[:64 * 50].nan_to_num(0.0)
    assert torch.allclose(warm[:64 * 50].nan_to_num(0.0), T0, rtol=1e-5, atol=0.0)
    assert torch.allclose(part.nan_to_num(0.0), T0, rtol=1e-5, atol=0.0)


@pytest.mark.parametrize("mode", ["plain", "mixed", "table"])
@pytest.mark.parametrize("n_cells,n_lambda,n_sizes", [(40, 100, 20), (5000, 250, 80),
                                                      (300000, 40, 5), (40000, 64, 130)])
def test_temperatures_over_the_heating_and_sed_over_the_field(n_cells, n_lambda, n_sizes, mode):
    """T may take the memory of H, and a fused call's L that of J: the same bits
    as in memory of their own (plain fused: as the one-kernel form)."""
    plan, J, m = _inputs(n_cells, n_lambda, 1, n_sizes, mode, 29)
    H = plan.absorb(J)
    T = plan.solve(H)
    plan.solve(H, H)
    assert torch.equal(H, T)
    one = dust.Plan(synth.make_grid(n_lambda, 1, n_sizes), mode, fused_kernels=1)
    Tf, Lf = one.fused(J, m)
    buf, T2 = J.clone(), torch.empty_like(T)
    plan.fused(buf, m, T2, buf)
    assert torch.equal(T2, Tf) and torch.equal(buf, Lf)

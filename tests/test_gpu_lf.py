"""The one-dimensional Eulerian low-fidelity model (Appendix B) on the GPU against the FP64 oracle, and
the MFMC pipeline with the paper's model pair (particle step as HF, Eulerian model as LF)."""

import sys

import numpy as np
import pytest

from oracle import lf_eulerian as olf
from oracle.physics import q_max_charge
from synthetic.workloads import physical_params

pytestmark = pytest.mark.gpu

# rounding-level agreement: the GPU runs one inward pass (flux carried as an affine map) where the
# oracle marches the momentum inward and the flux outward; transcendental functions differ by ~1 ulp
RTOL = 1e-11


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def test_lf_matches_oracle_over_sizes_charges_and_cohesion():
    from paper_2205_04979_amd.depo import lf_solve
    p = physical_params(180.0, rho_p=2650.0)
    rows = [(d, xi, z) for d in (0.01e-6, 0.3e-6, 1.6e-6, 5e-6, 16e-6, 40e-6)
            for xi, z in ((0.0, 0.0), (0.1, 0.0), (0.0, 1.0), (0.05, 0.3), (0.1, 1.0))]
    d = np.array([r[0] for r in rows])
    q = np.array([r[1] for r in rows]) * q_max_charge(d)
    A = np.array([r[2] for r in rows]) * 1e-18
    say("case: LF", len(rows), "classes")
    g = lf_solve(p, d, q, A)
    o = np.array([olf.solve(p, *r) for r in zip(d, q, A)])
    assert np.all(o > 0)
    assert np.allclose(g, o, rtol=RTOL, atol=0), np.max(np.abs(g / o - 1))
    # a finer grid runs through the same entry point
    g2 = lf_solve(p, d[:5], q[:5], A[:5], n_wall=300, n_core=2000)
    o2 = np.array([olf.solve(p, d[k], q[k], A[k], n_wall=300, n_core=2000) for k in range(5)])
    assert np.allclose(g2, o2, rtol=RTOL, atol=0)


def test_lf_invalid_classes_give_nan_and_empty_batch():
    from paper_2205_04979_amd.depo import lf_solve
    p = physical_params(180.0)
    g = lf_solve(p, np.array([5e-6, 0.0, -1e-6, 5e-6, 5e-6]), np.array([0, 0, 0, np.nan, 0.0]),
                 np.array([0, 0, 0, 0, np.inf]))
    assert np.isfinite(g[0]) and np.all(np.isnan(g[1:]))
    assert lf_solve(p, np.zeros(0), np.zeros(0), np.zeros(0)).shape == (0,)


def test_lf_full_mc_budget_sampled_against_oracle():
    """The LF-only Monte Carlo of Table 3 at p = 36: 25,920 evaluations in one launch; 48 sampled
    classes against the oracle, every output finite and positive."""
    from paper_2205_04979_amd.depo import lf_solve
    rng = np.random.default_rng(7)
    p = physical_params(180.0, rho_p=2650.0)
    n = 25920
    d = rng.choice([1.6e-6, 5e-6, 16e-6], n)
    q = rng.uniform(0, 0.1, n) * q_max_charge(d)
    A = rng.uniform(0, 1, n) * 1e-18
    say("case: LF", n, "classes")
    g = lf_solve(p, d, q, A)
    assert np.all(np.isfinite(g)) and np.all(g > 0)
    idx = np.sort(rng.choice(n, 48, replace=False))
    o = np.array([olf.solve(p, d[k], q[k], A[k]) for k in idx])
    assert np.allclose(g[idx], o, rtol=RTOL, atol=0)


def test_mfmc_with_particle_step_hf_and_eulerian_lf_matches_oracle_pipeline():
    """The paper's pairing: HF = batched particle step (FP64, monodisperse 5 um), LF = Eulerian model;
    the GPU pipeline equals the same pipeline evaluated on the oracle's HF and LF."""
    from oracle.sim import OracleSim
    from paper_2205_04979_amd import mfmc as pmf
    from synthetic import make_workload
    from synthetic.workloads import q_max
    from tests.gpu_common import near_wall_particles
    rng = np.random.default_rng(8)
    n, dp = 150, 5e-6
    # slow particles within 1.5 um of the wall: whether image charge and wall cohesion pull them in
    # within the horizon depends on (xi, zeta)
    p = physical_params(180.0, dt=1e-6)
    f = make_workload("plain-1k", n=4, field_n=32).field()
    d = np.full(n, dp)
    x, er = near_wall_particles(rng, n, p, d, band=1.5e-6)
    v0 = rng.uniform(-0.01, 0.01, n)[:, None] * er
    hf = pmf.HighFidelityGPU(p, f, x, d, steps=100, real_bytes=8, v=v0)
    lf = pmf.LowFidelityGPU(p, dp)

    def hf_oracle(pts):
        out = np.empty(pts.shape[0])
        for k in range(pts.shape[0]):
            sp = np.array([[pts[k, 0], pts[k, 1] * 1e-18, pts[k, 2]]])
            o = OracleSim(p, f, x, d, q_max(d), np.array([0, n]), sp, v0=v0)
            o.step(100)
            out[k] = o.tally()[0]["v_dep_plus"]
        return out

    def lf_oracle(pts):
        return np.array([olf.solve(p, dp, r[0] * q_max_charge(dp), r[1] * 1e-18) for r in pts])

    sample = lambda r, m: np.stack([r.uniform(0, 0.1, m), r.uniform(0, 1, m), np.full(m, 300.0)], 1)  # noqa
    pilot = sample(np.random.default_rng(9), 16)
    say("case: MFMC HF particle step + LF Eulerian, pilot")
    yh, yl = hf(pilot), lf(pilot)
    assert np.allclose(yl, lf_oracle(pilot), rtol=RTOL, atol=0)
    assert yh.std() > 0 and yl.std() > 0
    sigma, rho = (yh.std(ddof=1), yl.std(ddof=1)), (1.0, float(np.corrcoef(yh, yl)[0, 1]))
    w = (1.0, 1e-3)
    say("pilot sigma", sigma, "rho", rho)
    args = (sigma, rho, w, 30.0, sample, 2)
    res = pmf.mfmc_sobol([hf, lf], *args, rng=np.random.default_rng(10))
    ref = pmf.mfmc_sobol([hf_oracle, lf_oracle], *args, rng=np.random.default_rng(10))
    say("counts", res.counts.tolist(), "mean", res.mean, "main", res.main.tolist())
    assert np.array_equal(res.counts, ref.counts) and res.counts[1] > res.counts[0] >= 2
    assert np.isclose(res.mean, ref.mean, rtol=1e-10, atol=0)
    assert np.isclose(res.variance, ref.variance, rtol=1e-9, atol=0)
    assert np.allclose(res.main, ref.main, rtol=1e-8, atol=1e-12)
    assert np.allclose(res.total, ref.total, rtol=1e-8, atol=1e-12)


@pytest.mark.parametrize("n_wall,n_core", [(2, 1), (3, 2), (5, 9), (20, 43), (449, 1), (300, 150)])
def test_lf_short_grids_against_oracle(n_wall, n_core):
    """Grids shorter than, equal to and just past one chunk of the node waves (28 cells at this batch size, 448
    nodes per table), a wall part of two nodes and a core of one."""
    from paper_2205_04979_amd.depo import lf_solve
    p = physical_params(180.0)
    d = np.array([0.3e-6, 1.6e-6, 5e-6, 16e-6, 40e-6])
    q, A = 0.05 * q_max_charge(d), np.full(5, 4e-19)
    say(f"case: LF grid {n_wall} + {n_core}")
    g = lf_solve(p, d, q, A, n_wall=n_wall, n_core=n_core)
    o = np.array([olf.solve(p, *r, n_wall=n_wall, n_core=n_core) for r in zip(d, q, A)])
    assert np.allclose(g, o, rtol=RTOL, atol=0), np.max(np.abs(g / o - 1))


@pytest.mark.parametrize("n", [1, 15, 17, 4096, 4097, 8192, 8193, 10001])
def test_lf_batch_size_does_not_change_a_class(n):
    """The classes per workgroup follow the batch size (16, 32, 64): every class's value is that of a small
    batch, bit for bit; classes with invalid inputs in between change nothing."""
    from paper_2205_04979_amd.depo import lf_solve
    rng = np.random.default_rng(n)
    p = physical_params(180.0)
    d = np.exp(rng.uniform(np.log(0.05e-6), np.log(30e-6), n))
    q, A = rng.uniform(0, 0.1, n) * q_max_charge(d), rng.uniform(0, 1, n) * 1e-18
    bad = rng.random(n) < 0.02
    q = np.where(bad, np.nan, q)
    say(f"case: LF batch of {n}")
    g = lf_solve(p, d, q, A, n_wall=40, n_core=30)
    pick = np.unique(np.concatenate([np.arange(min(n, 40)), np.arange(max(0, n - 40), n), rng.integers(0, n, 60)]))
    small = np.concatenate([lf_solve(p, d[k], q[k], A[k], n_wall=40, n_core=30) for k in np.array_split(pick, 4) if k.size])
    assert np.array_equal(np.isnan(g), bad)
    assert np.array_equal(g[pick], small, equal_nan=True)


@pytest.mark.parametrize("re_tau,d_range,a_decades", [(0.3, (1e-9, 1e-4), (-26, -18)), (0.9, (1e-8, 1e-3), (-22, -12)),
                                                      (0.5, (1e-7, 1e-3), (-22, -12)), (180.0, (4e-3, 0.05), (-16, -8))])
def test_lf_cells_that_run_backwards_against_oracle(re_tau, d_range, a_decades):
    """A pipe radius of less than one wall unit beyond the particle (Re_tau below 1, or a particle as large as
    the pipe) makes the core's spacing negative; such classes, repulsive cohesion (A < 0) among them, are
    accepted and give the oracle's value.  The root of a backward cell cancels in both evaluations, so classes
    that a change of d by 1e-13 moves by 1e-10 are left out, and the others agree to ten times that."""
    from paper_2205_04979_amd.depo import lf_solve
    rng = np.random.default_rng(11)
    p = physical_params(re_tau)
    n = 60
    d = np.exp(rng.uniform(np.log(d_range[0]), np.log(d_range[1]), n))
    q = np.where(np.arange(n) % 3 == 0, 0.0, rng.normal(size=n) * 10.0 ** rng.uniform(-24, -18, n))
    A = rng.normal(size=n) * 10.0 ** rng.uniform(*a_decades, n)
    assert ((1 - 0.5 * d / p["R"]) * re_tau < 1).any()
    say("case: LF backwards", re_tau)
    with np.errstate(all="ignore"):
        o, o2 = (np.array([olf.solve(p, *r, n_wall=200, n_core=100) for r in zip(k * d, q, A)]) for k in (1.0, 1.0 + 1e-13))
        keep = np.isfinite(o) & (np.abs(o2 / o - 1) < 1e-10)
    assert keep.sum() > 50
    g = lf_solve(p, d, q, A, n_wall=200, n_core=100)
    assert np.allclose(g[keep], o[keep], rtol=1e-9, atol=0), np.max(np.abs(g[keep] / o[keep] - 1))


def extended_vdep(p, d, q, A, n_wall, n_core):
    """The model's V_dep+ for arrays of classes in 80-bit arithmetic (the oracle's march and flux, inward)."""
    ld = np.longdouble
    one = ld(1)
    d, q, A = (np.asarray(v).astype(ld) for v in (d, q, A))
    R, nu, rf, rp, re, eps = (ld(p[k]) for k in ("R", "nu", "rho_f", "rho_p", "re_tau", "eps0"))
    pi, kt = 4 * np.arctan(one), ld(1.380649e-23) * 293
    us = re * nu / R
    lw = nu / us
    taup, m = rp * d * d / (18 * rf * nu) * us * us / nu, rp * pi * d ** 3 / 6
    rr, db, yw = 1 / (1 + taup / 10), kt / (3 * pi * rf * nu * nu * d), d / 2 / lw
    lg = np.log(ld(1e-12) / lw)
    e, c = q * q / (16 * pi * eps * m), A * d / (12 * m)

    def v_rms(y):
        return ld(0.005) * y * y / (1 + ld(0.002923) * y ** ld(2.128))

    def node(k):
        gc = R / lw - yw
        if k == 0:
            g = np.full_like(d, ld(1e-12) / lw)
        elif k < n_wall - 1:
            g = np.full_like(d, np.exp(lg * (1 - ld(k) / (n_wall - 1))))
        elif k == n_wall - 1:
            g = np.ones_like(d)
        elif k == n_wall + n_core - 1:
            g = gc
        else:
            g = 1 + ld(k - n_wall + 1) * ((gc - 1) / n_core)
        y = yw + g
        phi = rr * v_rms(y) ** 2
        return y, phi, e / (y * lw) + c / (g * lw), db + 10 * phi

    y1, f1, u1, D1 = node(n_wall + n_core - 1)
    V, s, b = np.zeros_like(d), np.ones_like(d), np.zeros_like(d)
    for k in range(n_wall + n_core - 2, -1, -1):
        y0, f0, u0, D0 = node(k)
        h = y1 - y0
        w = V * V / 2 + (f1 - f0) + (u0 - u1) / (us * us)
        a = h / taup
        Vn = np.where(w > 0, 2 * w / (a + np.sqrt(a * a + 2 * np.maximum(w, 0))), 0)
        Vm, Dm = (V + Vn) / 2, (D0 + D1) / 2
        x = Vm * h / Dm
        on = x > 0
        xs = np.where(on, x, one)
        b -= np.where(on, -np.expm1(-xs) / xs, one) * h / Dm * s
        s *= np.where(on, np.exp(-xs), one)
        V, y1, f1, u1, D1 = Vn, y0, f0, u0, D0
    vp = np.sqrt(rr * v_rms(y1) ** 2 + kt / (m * us * us))
    M = V / (np.sqrt(2 * one) * vp)
    import math
    hw = vp * np.exp(-M * M) / np.sqrt(2 * pi) + V * (1 + np.array([math.erf(float(v)) for v in M]).astype(ld)) / 2
    return hw / (s - hw * b)


def test_lf_error_against_extended_precision():
    """400 random classes of the studies' ranges at the default grid against 80-bit arithmetic: relative rms 1.0e-15, as
    with the library's pow, exp, expm1, roots and divisions in the kernel of one lane per class (bound 1.5e-15), no
    class worse than 2e-14."""
    from paper_2205_04979_amd.depo import lf_solve
    rng = np.random.default_rng(23)
    p = physical_params(180.0)
    n = 400
    d = np.exp(rng.uniform(np.log(0.05e-6), np.log(40e-6), n))
    q, A = rng.uniform(0, 0.1, n) * q_max_charge(d), rng.uniform(0, 1, n) * 1e-18
    say("case: LF against 80 bits")
    ref = extended_vdep(p, d, q, A, 800, 800)
    e = np.abs(lf_solve(p, d, q, A).astype(np.longdouble) / ref - 1).astype(np.float64)
    say("relative rms", np.sqrt(np.mean(e ** 2)), "largest", e.max())
    assert np.sqrt(np.mean(e ** 2)) < 1.5e-15 and e.max() < 2e-14

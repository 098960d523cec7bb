"""The solver's small levels and patches where their kernels change over:
the bottom kernel's ladders (8^3, 16^3), the block sweeps of 32^3 and 64^3,
the double-precision fused sweeps of 128^3, and the patch solve's batches of
blocks, against the oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpucase import cubic, density, dev, field_for, models

pytestmark = pytest.mark.gpu

# Two V-cycles differ from the oracle's by rounding only: a few tens of
# dependent operations per cell and cycle, each good to half an ulp (1.1e-16,
# 6e-8), damped by the smoothing: 1e-12 and 1e-6 of the field's size.
TOL = {"fp64": 1e-12, "mixed": 1e-6}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name,n,pre,post,fw,pw", [
    ("symmetron_a1", 8, 1, 1, 0, 0), ("fofr", 8, 2, 2, 0, 1), ("chameleon", 16, 1, 3, 1, 0),
    ("linear", 16, 2, 2, 0, 0), ("fofr_a07", 16, 3, 1, 1, 1), ("symmetron_a05", 32, 1, 2, 0, 0),
    ("fofr", 32, 1, 1, 0, 1), ("chameleon", 32, 3, 1, 0, 1), ("linear", 32, 2, 3, 0, 0),
    ("symmetron_a1", 32, 2, 1, 1, 0), ("fofr", 64, 3, 1, 0, 0), ("fofr_a07", 64, 1, 3, 1, 1),
    ("chameleon_n05", 64, 2, 1, 0, 0), ("symmetron_a1", 64, 0, 2, 0, 0), ("linear", 64, 2, 0, 0, 0),
    ("symmetron_a1", 128, 1, 3, 0, 0), ("fofr", 128, 2, 2, 0, 1), ("chameleon", 128, 3, 1, 1, 0),
])
def test_cycles_of_small_grids(orc, name, n, pre, post, fw, pw, precision):
    from paper_1307_6748_amd import solver as S
    om, sp, a = models(name)
    box = 4.0 * n
    eta = density(n, 400 + n)
    cfg = orc.Cfg(nu_pre=pre, nu_post=post, restrict_fw=bool(fw), prolong_w=bool(pw))
    ref = orc.vcycles(om, eta, box, orc.cold_start(om, eta), 2, cfg=cfg)
    s = S.Solver(n, box, nu_pre=pre, nu_post=post, max_cycles=2, precision=precision,
                 restriction=fw, prolongation=pw)
    phi, st = s.solve(dev(eta), sp, a, 1e-300, check=False)
    assert st.cycles == 2
    err = np.max(np.abs(cubic(phi, n) - ref.phi)) / (np.abs(ref.phi).max() + 1.0)
    assert err <= TOL[precision], err


def _patch(name, n, seed):
    rng = np.random.default_rng(seed)
    idx = np.arange(n)
    ins = (idx >= 2) & (idx < n - 2)
    mask = np.where(ins[:, None, None] & ins[None, :, None] & ins[None, None, :],
                    0.4 + 0.6 * rng.random((n, n, n)), -rng.random((n, n, n)))
    mask[n // 2, n // 2, n // 2] = -0.5   # a hole
    phi = field_for(name, n, seed)
    return phi, density(n, seed + 1), mask, phi + 0.01 * rng.standard_normal(phi.shape)


@pytest.mark.parametrize("name", ["symmetron_a1", "fofr", "chameleon", "linear"])
@pytest.mark.parametrize("n", [8, 24, 30])
@pytest.mark.parametrize("block,sweeps", [(4, 0), (4, 1), (3, 8), (1, 21)])
@pytest.mark.parametrize("room", [True, False])
def test_patch_blocks(orc, name, n, block, sweeps, room):
    """A bounded number of sweeps, whole blocks or not, gives the oracle's
    iterate, sweep count and defect, with and without room in the workspace
    for the kinds of cells.  Tolerance: 1e-12 of the field per sweep made."""
    from paper_1307_6748_amd import _capi as A
    om, sp, a = models(name)
    h = 0.7
    phi, eta, mask, u_int = _patch(name, n, 70 + n)
    ref, sw, rms = orc.patch_solve(om, h, phi, eta, mask, u_int, block=block, max_sweeps=sweeps,
                                   tol=1e-14)
    g, e, mk, ui = dev(phi), dev(eta), dev(mask), dev(u_int)
    nbytes = A.lib().isis_patch_workspace_size(n) - (0 if room else n ** 3 + 256)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    count, got = C.c_int(), C.c_double()
    pc = sp.c()
    ptr = [C.c_void_p(t.data_ptr()) for t in (g, e, mk, ui)]
    rc = A.lib().isis_patch_solve(C.byref(pc), a, n, h, *ptr, block, sweeps, 1e-14,
                                  C.c_void_p(ws.data_ptr()), nbytes, C.byref(count), C.byref(got),
                                  C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == A.ISIS_ERR_NOT_CONVERGED and count.value == sw == sweeps
    tol = 1e-12 * max(sweeps, 1) * (np.abs(ref).max() + 1.0)
    assert np.max(np.abs(cubic(g, n) - ref)) <= tol
    # the defect weighs the field's error with up to 12 exp(|phi|) / h^2
    scale = 12.0 * np.exp(np.abs(ref).max() if name.startswith(("fofr", "cham")) else 1.0) / h ** 2
    assert abs(got.value - rms) <= 1e-12 * rms + tol * scale


def test_patch_with_nothing_finite_to_judge():
    """A NaN from the start: no sweep is made, as an unmet tolerance.  A defect
    whose square overflows: divergence, after the first block."""
    from paper_1307_6748_amd import _capi as A
    from paper_1307_6748_amd import solver as S
    _, sp, a = models("linear")
    phi, eta, mask, u_int = _patch("linear", 24, 5)
    bad = eta.copy()
    bad[12, 13, 11] = np.nan
    rc, sweeps, rms = S.patch_solve(sp, a, 0.7, dev(phi), dev(bad), dev(mask), dev(u_int), check=False)
    assert (rc, sweeps) == (A.ISIS_ERR_NOT_CONVERGED, 0) and np.isnan(rms)
    rc, sweeps, rms = S.patch_solve(sp, a, 0.7, dev(1e200 * phi), dev(eta), dev(mask), dev(u_int),
                                    block=3, check=False)
    assert (rc, sweeps) == (A.ISIS_ERR_DIVERGED, 3) and not np.isfinite(rms)


def _blocks_queued(h, tol):
    """Blocks that a solve with RMS h[k] after k blocks queues until it has seen
    h[k] <= tol (csrc/patch_schedule.hpp)."""
    done, batch = 0, 1
    while True:
        r0, done = h[done], done + batch
        if done >= len(h) or min(h[:done + 1]) <= tol:
            return done
        rho = (h[done] / r0) ** (1.0 / batch)
        left = np.log(tol / h[done]) / np.log(rho) if rho < 1.0 else 0.0
        batch = 1 if left < 1.0 else int(min(np.ceil(left), 4.0 * batch, 64.0))


@pytest.mark.parametrize("name", ["symmetron_a1", "fofr"])
@pytest.mark.parametrize("room", [True, False])
def test_patch_launches_past_the_end_store_nothing(name, room):
    """A solve stopped by its tolerance, with blocks already queued behind the one
    that met it, leaves the field, sweep count and RMS of one stopped there by
    its sweep limit, which queues none: bit for bit."""
    from paper_1307_6748_amd import _capi as A
    _, sp, a = models(name)
    n, block, h = 16, 4, 0.7
    phi, eta, mask, u_int = _patch(name, n, 90)
    e, mk, ui = dev(eta), dev(mask), dev(u_int)
    nbytes = A.lib().isis_patch_workspace_size(n) - (0 if room else n ** 3 + 256)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    pc = sp.c()

    def solve(sweeps, tol):
        g = dev(phi)
        count, got = C.c_int(), C.c_double()
        ptr = [C.c_void_p(t.data_ptr()) for t in (g, e, mk, ui)]
        rc = A.lib().isis_patch_solve(C.byref(pc), a, n, h, *ptr, block, sweeps, tol,
                                      C.c_void_p(ws.data_ptr()), nbytes, C.byref(count),
                                      C.byref(got),
                                      C.c_void_p(torch.cuda.current_stream().cuda_stream))
        return rc, cubic(g, n), count.value, got.value

    ref = [solve(block * k, 1e-300) for k in range(25)]
    rms = [r[3] for r in ref]
    past = 0
    for k in range(2, 25):
        tol = 1.0001 * rms[k]
        if min(rms[:k]) <= tol:
            continue
        rc, field, sweeps, got = solve(10000, tol)
        assert rc == A.ISIS_OK and sweeps == ref[k][2] == block * k and got == rms[k]
        assert np.array_equal(field, ref[k][1])
        past += _blocks_queued(rms, tol) > k
    assert past >= 3  # else this test asks nothing


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("n", [6, 32])
def test_halfsweep_steps_are_quotients(n, masked):
    """The Newton-Gauss-Seidel step is the correctly rounded quotient L / D in
    double precision.  Linear model, m2 = 1, h = 1, density 1, whole numbers on
    the black cells and zero on the red: L is a whole number, D = -7, and a red
    cell becomes sum(neighbours) / 7, bit for bit."""
    from paper_1307_6748_amd import solver as S
    sp = S.linear(1.3, 1.0)
    rng = np.random.default_rng(7)
    i = np.arange(n)
    red = (i[:, None, None] + i[None, :, None] + i[None, None, :]) % 2 == 0
    phi = np.where(red, 0.0, rng.integers(-10 ** 6, 10 ** 6, (n, n, n)).astype(float))
    nb = sum(np.roll(phi, s, axis) for axis in range(3) for s in (-1, 1))
    ref = np.where(red, nb / 7.0, phi)
    one, g = np.ones((n, n, n)), dev(phi)
    if masked:
        S.masked_halfsweep(sp, 1.0, 1.0, g, dev(one), dev(one), dev(phi), dev(phi), colour=0)
    else:
        S.halfsweep(sp, 1.0, 1.0, g, dev(one), colour=0)
    assert np.array_equal(cubic(g, n), ref)


# Sides where the walk over planes changes: a plane of fewer than 256 items is
# walked with the others as one list (half planes: up to n = 22; planes: 14), and
# from 16 workgroups on (n = 62) their number per plane is rounded up.
@pytest.mark.parametrize("n", [2, 14, 16, 22, 24, 60, 62, 66])
def test_walk_over_planes(orc, n):
    """Every cell is visited once.  Tolerances: a few roundings of a dozen terms."""
    from paper_1307_6748_amd import solver as S
    h = 0.8
    for name in ("symmetron_a1", "fofr"):
        om, sp, a = models(name)
        phi, eta = field_for(name, n, 200 + n), density(n, 201 + n)
        if n > 2:
            mask = np.where(np.random.default_rng(n).random((n, n, n)) < 0.3, 1.0, -1.0)
            mask[:1], mask[:, :1], mask[:, :, :1] = -1.0, -1.0, -1.0
            g = dev(phi)
            S.masked_halfsweep(sp, a, h, g, dev(eta), dev(mask), dev(phi), dev(phi), colour=1)
            ref = orc.masked_halfsweep(om, h, phi, eta, mask, phi, phi, colour=1)
            assert np.max(np.abs(cubic(g, n) - ref)) <= 1e-13 * (np.abs(ref).max() + 1.0)
        g = dev(phi)
        S.halfsweep(sp, a, h, g, dev(eta), colour=1)
        ref = orc.halfsweep(om, h, phi, eta, None, 1)
        assert np.max(np.abs(cubic(g, n) - ref)) <= 1e-13 * (np.abs(ref).max() + 1.0)
        scale = 12.0 * np.exp(np.abs(phi).max()) * (np.abs(phi).max() + 1.0) / h ** 2
        ref = orc.defect(om, h, phi, eta)
        got = cubic(S.defect(sp, a, h, dev(phi), dev(eta)), n)
        assert np.max(np.abs(got - ref)) <= 1e-14 * (scale + np.abs(ref).max())
        force = S.force(sp, a, h * n, field=dev(phi), potential=dev(eta))
        for f, r in zip(force, orc.force(om, h, phi, eta)):
            assert np.max(np.abs(cubic(f, n) - r)) <= 1e-14 * (np.abs(r).max() + 10.0)


@pytest.mark.parametrize("nc", [2, 14, 16, 60, 62])
def test_walk_over_coarse_planes(orc, nc):
    """The same for the kernels that walk the coarse cells."""
    from paper_1307_6748_amd import solver as S
    n = 2 * nc
    rng = np.random.default_rng(nc)
    fine, ch = rng.standard_normal((n, n, n)), rng.standard_normal((nc, nc, nc))
    c = ch + rng.standard_normal((nc, nc, nc))
    assert np.max(np.abs(cubic(S.restrict(dev(fine)), nc) - orc.restrict(fine))) <= 1e-15 * np.abs(fine).max()
    assert np.max(np.abs(cubic(S.restrict_fw(dev(fine)), nc) - orc.restrict_fw(fine))) <= 4e-15 * np.abs(fine).max()
    for gpu, cpu in ((S.prolong_correct, orc.prolong_correct),
                     (S.prolong_correct_w, orc.prolong_correct_w)):
        g = dev(fine)
        gpu(g, dev(c), dev(ch))
        ref = cpu(fine, c, ch)
        assert np.max(np.abs(cubic(g, n) - ref)) <= 1e-14 * (np.abs(ref).max() + 1.0)
    om, sp, a = models("symmetron_a1")
    phi, eta = field_for("symmetron_a1", n, nc), density(n, nc)
    eta_c, phi_c = orc.restrict(eta), orc.restrict(phi)
    for fw in (False, True):
        d = orc.defect(om, 0.7, phi, eta)
        ref = orc.defect(om, 1.4, phi_c, eta_c) - (orc.restrict_fw(d) if fw else orc.restrict(d))
        got = S.fas_descend(sp, a, 0.7, dev(phi), dev(eta), None, dev(eta_c), full_weighting=fw)
        assert np.max(np.abs(cubic(got[0], nc) - phi_c)) <= 2e-15
        assert np.max(np.abs(cubic(got[2], nc) - ref)) <= 1e-14 * (12.0 / 0.49 + np.abs(ref).max())


@pytest.mark.parametrize("name,n,precision,pre,post,fw", [
    ("symmetron_a1", 32, "fp64", 2, 1, 0), ("symmetron_a1", 64, "mixed", 2, 2, 0),
    ("fofr", 64, "fp64", 1, 3, 0), ("chameleon", 32, "mixed", 1, 1, 1)])
def test_profiled_launches_of_block_sweeps(name, n, precision, pre, post, fw):
    """32^3 and 64^3 grids, profiling on: the launch that adds the coarse-grid
    correction counts in fine_prol_*, the other sweeps in fine_sweep_*, with the
    bytes that each cannot do without."""
    from paper_1307_6748_amd import solver as S
    _, sp, a = models(name)
    s = S.Solver(n, 4.0 * n, nu_pre=pre, nu_post=post, precision=precision, restriction=fw)
    s.set_profiling(True)
    _, st = s.solve(dev(density(n, 7)), sp, a, 1e-9)
    cycles = [st.cycles - st.cycles_fp32, st.cycles_fp32]
    assert cycles[0] > 0 and (cycles[1] > 0) == (precision == "mixed")
    for k, size in ((0, 8), (1, 4)):
        plain = cycles[k] * (pre + post - 1)
        coarse = 0 if fw else cycles[k] * 3 * (n // 2) ** 3
        assert st.fine_prol_launches[k] == cycles[k]
        assert st.fine_prol_bytes[k] == cycles[k] * (3 * n ** 3 + 2 * (n // 2) ** 3) * size
        assert st.fine_sweep_launches[k] == plain
        assert st.fine_sweep_updates[k] == plain * n ** 3
        assert st.fine_sweep_bytes[k] == (plain * 3 * n ** 3 + coarse) * size
        assert (st.fine_prol_ms[k] > 0) == (st.fine_sweep_ms[k] > 0) == (cycles[k] > 0)

"""GPU parity: the HIP library (through the C ABI) against the FP64 oracle.

Both sides get the same seeded inputs and, for absorbing sweeps, the same
previous flux (the oracle's own thin sweep), so every sweep is compared
element by element.  Tolerances:

* FP64 form: |F_gpu - F_or| <= 1e-10 F_or on every cell with
  F_or > 1e-6 max F_or, and identical ionisation flags.
* FP32C form: the same relative error bounded by 1e-4 on cells that are not
  within one cell of the oracle's ionisation front (cells next to a dark
  cell); ionisation flags identical away from the front.  Near the front the
  flux is a small difference of large terms and the FP32 mapping error is
  amplified; those cells are counted and reported, not bounded.
"""
import math
import sys

import numpy as np
import pytest

from paper_2105_09644_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL64 = 1e-10
TOL32 = 1e-4


@pytest.fixture(scope="module")
def T():
    import paper_2105_09644_amd as T
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    T.load_library()
    return T


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def gpu_sweep(T, P, prec, f_prev=None, thin=False, targets=None, launch=None, **over):
    ctx = T.context_for(P, prec, **over)
    if launch is not None:
        ctx.set_launch(*launch)
    n = ctx.n_cells
    nh = torch.tensor(np.concatenate(P.n_h), dtype=torch.float64, device="cuda")
    fp = None if f_prev is None else torch.tensor(f_prev, dtype=torch.float64, device="cuda")
    ctx.build(nh, fp, thin=thin)
    if targets is None:
        out = torch.full((n,), -1.0, dtype=torch.float64, device="cuda")
        ion = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
        ctx.sweep(out, ion)
    else:
        tg = torch.tensor(targets, dtype=torch.int64, device="cuda")
        out = torch.full((len(targets),), -1.0, dtype=torch.float64, device="cuda")
        ion = torch.full((len(targets),), 7, dtype=torch.uint8, device="cuda")
        ctx.sweep_targets(tg, out, ion)
    ctx.sync()
    st = ctx.stats()
    res = out.cpu().numpy(), ion.cpu().numpy(), st
    ctx.close()
    return res


def orc_sweep(orc, P, f_prev=None, thin=False, targets=None, **over):
    """Oracle per domain; targets are global cell indices."""
    outs, ions = [], []
    off = 0
    fp_all = f_prev
    for d, dom in enumerate(P.domains):
        n = dom.n_cells()
        fp = None if fp_all is None else fp_all[off:off + n]
        tg = None
        if targets is not None:
            sel = (targets >= off) & (targets < off + n)
            tg = targets[sel] - off
        kw = dict(over)
        if thin:
            kw["alpha_b"] = 0.0
        if tg is None or len(tg):
            f, ion, _ = orc.sweep(dom, P.params, P.n_h[d], P.src_xyz[d], P.src_q[d], f_prev=fp, targets=tg, **kw)
            outs.append(f)
            ions.append(ion)
        off += n
    return np.concatenate(outs), np.concatenate(ions)


def front_mask(P, f_or):
    """Cells within one cell (26-neighbourhood) of a dark cell; uniform grids only."""
    masks = []
    off = 0
    for dom in P.domains:
        n = dom.n_cells()
        f = f_or[off:off + n]
        if dom.leaf_blocks is not None:
            masks.append(f <= 0)
            off += n
            continue
        e = dom.extent_finest()
        dark = (f <= 0).reshape(e)
        near = np.zeros_like(dark)
        pad = np.pad(dark, 1, constant_values=False)
        for dx in (-1, 0, 1):
            for dy in (-1, 0, 1):
                for dz in (-1, 0, 1):
                    near |= pad[1 + dx:1 + dx + e[0], 1 + dy:1 + dy + e[1], 1 + dz:1 + dz + e[2]]
        masks.append(near.ravel())
        off += n
    return np.concatenate(masks)


def compare(f_gpu, ion_gpu, f_or, ion_or, tol, front=None, name=""):
    assert np.all(np.isfinite(f_gpu)), f"{name}: non-finite GPU flux"
    sel = f_or > 1e-6 * f_or.max()
    if front is not None:
        sel &= ~front
    rel = np.abs(f_gpu[sel] - f_or[sel]) / f_or[sel]
    log(f"{name}: cells {sel.sum()} max rel {rel.max():.3e} p99.9 {np.percentile(rel, 99.9):.3e} "
        f"L1 {np.sum(np.abs(f_gpu[sel] - f_or[sel])) / np.sum(f_or[sel]):.3e}")
    assert rel.max() <= tol, f"{name}: max relative error {rel.max():.3e} > {tol}"
    ion_sel = np.ones_like(ion_or, bool) if front is None else ~front
    bad = np.count_nonzero(ion_gpu[ion_sel] != ion_or[ion_sel])
    assert bad == 0, f"{name}: {bad} ionisation flags differ"


def cases():
    return {
        "uniform16": lambda: W.small_uniform(16, n_radial=20),
        "lognormal16": lambda: W.small_lognormal(16, n_src=3, seed=1),
        "padded24": lambda: W.small_lognormal(24, n_src=2, seed=2, nside=1),
        "amr": lambda: W.small_amr(2, seed=3),
        "nside4": lambda: W.small_lognormal(16, n_src=2, seed=4, nside=4, n_radial=24),
    }


@pytest.mark.parametrize("case", list(cases()))
def test_fp64_sweeps(T, orc, case):
    P = cases()[case]()
    log(f"case {case}: cells {P.total_cells()}")
    f0, i0 = orc_sweep(orc, P, thin=True)
    g0, j0, st = gpu_sweep(T, P, T.TR_FP64, thin=True)
    compare(g0, j0, f0, i0, TOL64, name=f"{case} thin fp64")
    f1, i1 = orc_sweep(orc, P, f_prev=f0)
    g1, j1, st = gpu_sweep(T, P, T.TR_FP64, f_prev=f0)
    compare(g1, j1, f1, i1, TOL64, name=f"{case} absorbing fp64")
    assert st.overflow == 0


@pytest.mark.parametrize("case", list(cases()))
def test_fp32c_sweeps(T, orc, case):
    P = cases()[case]()
    f0, i0 = orc_sweep(orc, P, thin=True)
    g0, j0, st = gpu_sweep(T, P, T.TR_FP32C, thin=True)
    compare(g0, j0, f0, i0, TOL32, name=f"{case} thin fp32c")
    f1, i1 = orc_sweep(orc, P, f_prev=f0)
    g1, j1, st = gpu_sweep(T, P, T.TR_FP32C, f_prev=f0)
    compare(g1, j1, f1, i1, TOL32, front=front_mask(P, f1), name=f"{case} absorbing fp32c")
    log(f"  guard recomputes {st.guard_recomputes} of {st.nodes_accepted * 64} sub-points")


def test_batched_domains(T, orc):
    # two domains of different sizes in one context: one launch covers both
    A = W.small_lognormal(16, n_src=2, seed=5)
    B = W.small_lognormal(24, n_src=1, seed=6)
    P = W.Problem("two", A.domains + B.domains, A.n_h + B.n_h, A.src_xyz + B.src_xyz, A.src_q + B.src_q, A.params)
    f0, i0 = orc_sweep(orc, P, thin=True)
    f1, i1 = orc_sweep(orc, P, f_prev=f0)
    for prec, tol in ((T.TR_FP64, TOL64), (T.TR_FP32C, TOL32)):
        g1, j1, st = gpu_sweep(T, P, prec, f_prev=f0)
        compare(g1, j1, f1, i1, tol, front=None if prec == T.TR_FP64 else front_mask(P, f1),
                name=f"batched prec {prec}")


def test_target_list_and_ragged_tail(T, orc):
    P = W.small_lognormal(16, n_src=3, seed=7)
    f0, _ = orc_sweep(orc, P, thin=True)
    rng = np.random.default_rng(3)
    tg = rng.choice(P.total_cells(), 1237, replace=False)   # not a multiple of any launch width
    f1, i1 = orc_sweep(orc, P, f_prev=f0, targets=tg)
    g1, j1, _ = gpu_sweep(T, P, T.TR_FP64, f_prev=f0, targets=tg)
    compare(g1, j1, f1, i1, TOL64, name="target list")
    g2, j2, _ = gpu_sweep(T, P, T.TR_FP64, f_prev=f0, targets=np.zeros(0, np.int64))
    assert len(g2) == 0


def test_config1_fp64_full(T, orc):
    P = W.config1()
    log("config1: 32^3, N_side 2, 32 points")
    f0, i0 = orc_sweep(orc, P, thin=True)
    g0, j0, _ = gpu_sweep(T, P, T.TR_FP64, thin=True)
    compare(g0, j0, f0, i0, TOL64, name="config1 thin fp64")
    f1, i1 = orc_sweep(orc, P, f_prev=f0)
    g1, j1, _ = gpu_sweep(T, P, T.TR_FP64, f_prev=f0)
    compare(g1, j1, f1, i1, TOL64, name="config1 absorbing fp64")


def test_delta_matches_oracle(T, orc):
    P = W.small_lognormal(16, n_src=3, seed=8)
    f0, _ = orc_sweep(orc, P, thin=True)
    f1, _ = orc_sweep(orc, P, f_prev=f0)
    ctx = T.context_for(P, T.TR_FP64)
    a = torch.tensor(f1, device="cuda")
    b = torch.tensor(f0, device="cuda")
    d = ctx.delta(a, b)
    assert d[0] == pytest.approx(orc.delta_cell(f1, f0), rel=1e-14)
    # median of a field with many zeros, and the zero-normaliser case
    z = f0.copy()
    z[: len(z) // 2 + 3] = 0.0
    d = ctx.delta(torch.tensor(f1, device="cuda"), torch.tensor(z, device="cuda"))
    assert math.isinf(d[0]) and math.isinf(orc.delta_cell(f1, z))
    ctx.close()


def test_solve_matches_oracle(T, orc):
    # the same fixed number of outer iterations on both sides
    P = W.small_lognormal(16, n_src=2, seed=9)
    P.params.max_iter = 3
    P.params.eps_lim = 0.0
    dom = P.domains[0]
    f_or, ion_or, it, dl = orc.solve(dom, P.params, P.n_h[0], P.src_xyz[0], P.src_q[0], eps_lim=0.0, max_iter=3)
    ctx = T.context_for(P, T.TR_FP64)
    nh = torch.tensor(P.n_h[0], device="cuda")
    out = torch.zeros(ctx.n_cells, dtype=torch.float64, device="cuda")
    ion = torch.zeros(ctx.n_cells, dtype=torch.uint8, device="cuda")
    iters, delta = ctx.solve(nh, out, ion, allow_noconv=True)
    assert iters == it == 3
    assert delta == pytest.approx(dl, rel=1e-6)
    compare(out.cpu().numpy(), ion.cpu().numpy(), f_or, ion_or, 1e-9, name="solve x3 fp64")
    ctx.close()


def test_graph_step_replays(T, orc):
    """tr_step (one outer iteration captured as a hipGraph) against the eager
    build/sweep/delta calls, replayed several times with eager work between
    the replays, every replay checked; then against the oracle."""
    P = W.small_lognormal(16, n_src=3, seed=10)
    f0, _ = orc_sweep(orc, P, thin=True)
    f1, i1 = orc_sweep(orc, P, f_prev=f0)
    d_or = orc.delta_cell(f1, f0)
    # atomic accumulation order differs between launches: FP64 agrees to
    # rounding, FP32C to its own tolerance away from the front
    for prec, tol in ((T.TR_FP64, 1e-12), (T.TR_FP32C, TOL32)):
        ctx = T.context_for(P, prec)
        n = ctx.n_cells
        nh = torch.tensor(P.n_h[0], device="cuda")
        fp = torch.tensor(f0, device="cuda")
        ref = torch.zeros(n, dtype=torch.float64, device="cuda")
        ctx.build(nh, fp)
        ctx.sweep(ref)
        d_ref = ctx.delta(ref, fp)
        ref_h = ref.cpu().numpy()
        ref_ion = (ref_h > 0).astype(np.uint8)
        fr = None if prec == T.TR_FP64 else front_mask(P, ref_h)
        out = torch.zeros(n, dtype=torch.float64, device="cuda")
        ion = torch.zeros(n, dtype=torch.uint8, device="cuda")
        scratch = torch.zeros(n, dtype=torch.float64, device="cuda")
        for rep in range(4):
            out.fill_(-1.0)
            ion.fill_(7)
            d = ctx.step(nh, fp, out, ion)
            g = out.cpu().numpy()
            log(f"graph prec {prec} replay {rep}: delta {d[0]:.6e} eager {d_ref[0]:.6e}")
            compare(g, ion.cpu().numpy(), ref_h, ref_ion, tol, front=fr, name=f"replay {rep} vs eager")
            assert d[0] == pytest.approx(d_ref[0], rel=1e-9 if prec == T.TR_FP64 else 1e-3)
            # eager work between replays: another build and sweep, a torch kernel
            ctx.build(nh, thin=True)
            ctx.sweep(scratch)
            scratch.mul_(0.5)
            torch.cuda.synchronize()
        tol_or = TOL64 if prec == T.TR_FP64 else TOL32
        compare(out.cpu().numpy(), ion.cpu().numpy(), f1, i1, tol_or,
                front=None if prec == T.TR_FP64 else front_mask(P, f1), name=f"graph step prec {prec}")
        assert d[0] == pytest.approx(d_or, rel=1e-9 if prec == T.TR_FP64 else 1e-3)
        # new buffers: the graph is captured again
        out2 = torch.zeros(n, dtype=torch.float64, device="cuda")
        ctx.step(nh, fp, out2)
        assert torch.equal(out2 > 0, out > 0)
        with pytest.raises(T.TreeRayError) as e:
            ctx.step(nh, fp, fp)
        assert e.value.status == T.TR_EINVAL
        ctx.close()


def test_graph_after_scratch_regrowth(T, orc):
    """A captured step graph refers to the sweep's scratch memory (the overflow
    queue, ray-buffer slabs).  A target list longer than the grid regrows that
    scratch; the next step must capture again instead of replaying the old
    graph.  theta = 0.05 sends every walk through the overflow queue."""
    P = W.small_lognormal(16, n_src=2, seed=25)
    f0, _ = orc_sweep(orc, P, thin=True, theta=0.05)
    f1, i1 = orc_sweep(orc, P, f_prev=f0, theta=0.05)
    ctx = T.context_for(P, T.TR_FP64, theta=0.05)
    ctx.set_launch(4, 0, 2, 0, 0)
    n = ctx.n_cells
    nh = torch.tensor(P.n_h[0], device="cuda")
    fp = torch.tensor(f0, device="cuda")
    out = torch.zeros(n, dtype=torch.float64, device="cuda")
    ctx.step(nh, fp, out)
    compare(out.cpu().numpy(), (out > 0).cpu().numpy().astype(np.uint8), f1, i1, TOL64, name="step before regrowth")
    # 3 n targets (every cell three times): the overflow queue and slabs grow
    tg = torch.arange(3 * n, dtype=torch.int64, device="cuda") % n
    ft = torch.zeros(3 * n, dtype=torch.float64, device="cuda")
    ctx.build(nh, fp)
    ctx.sweep_targets(tg, ft)
    ctx.sync()
    assert ctx.stats().overflow == 0
    compare(ft.cpu().numpy()[:n], (ft[:n] > 0).cpu().numpy().astype(np.uint8), f1, i1, TOL64, name="long list")
    out.fill_(-1.0)
    ctx.step(nh, fp, out)
    ctx.sync()
    assert ctx.stats().overflow == 0
    compare(out.cpu().numpy(), (out > 0).cpu().numpy().astype(np.uint8), f1, i1, TOL64, name="step after regrowth")
    ctx.close()


@pytest.mark.parametrize("theta_if,theta_src", [(0.25, 0.2), (1e-6, 1e-6)])
def test_if_and_src_macs(T, orc, theta_if, theta_src):
    """IF MAC and Src MAC (Sec. 2.4) against the oracle, on a previous flux that
    holds an ionisation front (the oracle's absorbing sweep)."""
    P = W.small_lognormal(16, n_src=2, seed=23)
    f0, _ = orc_sweep(orc, P, thin=True)
    f1, _ = orc_sweep(orc, P, f_prev=f0)
    over = dict(theta_if=theta_if, theta_src=theta_src)
    f2, i2 = orc_sweep(orc, P, f_prev=f1, **over)
    for prec, tol in ((T.TR_FP64, TOL64), (T.TR_FP32C, TOL32)):
        g2, j2, st = gpu_sweep(T, P, prec, f_prev=f1, **over)
        compare(g2, j2, f2, i2, tol, front=None if prec == T.TR_FP64 else front_mask(P, f2),
                name=f"macs {theta_if}/{theta_src} prec {prec}")
        log(f"  accepted per target {st.nodes_accepted / P.total_cells():.1f}")
    # thin, emission resolved to cells
    t0, k0 = orc_sweep(orc, P, thin=True, theta_src=1e-6)
    g0, j0, _ = gpu_sweep(T, P, T.TR_FP64, thin=True, theta_src=1e-6)
    compare(g0, j0, t0, k0, TOL64, name="thin src mac fp64")


def test_long_walks_use_device_lists(T, orc):
    # theta = 0.05 on 16^3 accepts nearly every cell: the walk lists exceed
    # the LDS capacity and every target goes through the device-memory pass
    P = W.small_lognormal(16, n_src=2, seed=25)
    f0, i0 = orc_sweep(orc, P, thin=True, theta=0.05)
    for prec, tol in ((T.TR_FP64, TOL64), (T.TR_FP32C, TOL32)):
        g0, j0, st = gpu_sweep(T, P, prec, thin=True, theta=0.05)
        compare(g0, j0, f0, i0, tol, name=f"theta 0.05 prec {prec}")
        assert st.overflow == 0
        assert st.nodes_accepted / P.total_cells() > 2048


def test_few_targets_with_long_walks(T, orc):
    # a short target list whose walks all overflow the LDS lists, with ray
    # buffers in device memory (FP64, FP32C), split (FP32C at N_side 4 with
    # 64 points) or in LDS in passes over the rays (FP64 at N_side 4): the
    # second pass runs more workgroups than the first, each with its own
    # buffer slab
    rng = np.random.default_rng(26)
    # (at 16 waves the next target is walked by four waves, here with device lists)
    cases = [(W.small_lognormal(16, n_src=2, seed=25), T.TR_FP64, 2, 0, 4),
             (W.small_lognormal(16, n_src=2, seed=25), T.TR_FP32C, 2, 0, 4),
             (W.small_lognormal(16, n_src=2, seed=25), T.TR_FP32C, 1, 1, 16),
             (W.small_lognormal(16, n_src=2, seed=27, nside=4, n_radial=64), T.TR_FP32C, 1, 2, 4),
             (W.small_lognormal(16, n_src=2, seed=27, nside=4, n_radial=64), T.TR_FP64, 1, 3, 4),
             (W.small_lognormal(16, n_src=2, seed=27, nside=4, n_radial=64), T.TR_FP64, 1, 3, 16)]
    for P, prec, buf, where, waves in cases:
        tg = np.sort(rng.choice(P.total_cells(), 37, replace=False))
        f0, i0 = orc_sweep(orc, P, thin=True, targets=tg, theta=0.05)
        g0, j0, st = gpu_sweep(T, P, prec, thin=True, targets=tg, launch=(waves, 0, buf, 0, 0), theta=0.05)
        assert st.overflow == 0 and st.buffer_in_lds == where
        assert st.nodes_accepted / len(tg) > 2048
        compare(g0, j0, f0, i0, TOL64 if prec == T.TR_FP64 else TOL32,
                name=f"37 targets prec {prec} buffer {buf} waves {waves}")


@pytest.mark.parametrize("radius_cells", [0.45, 1.7])
def test_sphere_sources(T, orc, radius_cells):
    """Sources as uniform spheres (Sec. 2.7): the exact-volume deposit against
    the oracle's, through thin and absorbing sweeps, uniform and AMR grids."""
    for P in (W.small_lognormal(16, n_src=4, seed=26), W.small_amr(2, seed=27)):
        r = radius_cells * P.domains[0].finest_dx_cm()
        f0, i0 = orc_sweep(orc, P, thin=True, src_radius_cm=r)
        f1, i1 = orc_sweep(orc, P, f_prev=f0, src_radius_cm=r)
        for prec, tol in ((T.TR_FP64, TOL64), (T.TR_FP32C, TOL32)):
            g0, j0, _ = gpu_sweep(T, P, prec, thin=True, src_radius_cm=r)
            compare(g0, j0, f0, i0, tol, name=f"{P.name} r {radius_cells} thin prec {prec}")
            g1, j1, _ = gpu_sweep(T, P, prec, f_prev=f0, src_radius_cm=r)
            compare(g1, j1, f1, i1, tol, front=None if prec == T.TR_FP64 else front_mask(P, f1),
                    name=f"{P.name} r {radius_cells} absorbing prec {prec}")


@pytest.mark.parametrize("eps_kernel,mass_kernel", [(1, 0), (2, 0), (4, 0), (5, 0), (6, 6), (3, 6)])
def test_radial_kernel_variants(T, orc, eps_kernel, mass_kernel):
    """Radial kernels of App. A (W_f,1, W_f,2, N-point W_f,3, W_p and W_g for the
    emission; W_g for A, E, V) against the oracle."""
    P = W.small_lognormal(16, n_src=3, seed=32, nside=2)
    over = dict(eps_kernel=eps_kernel, mass_kernel=mass_kernel)
    f0, i0 = orc_sweep(orc, P, thin=True, **over)
    f1, i1 = orc_sweep(orc, P, f_prev=f0, **over)
    for prec, tol in ((T.TR_FP64, TOL64), (T.TR_FP32C, TOL32)):
        g0, j0, _ = gpu_sweep(T, P, prec, thin=True, **over)
        compare(g0, j0, f0, i0, tol, name=f"kernels {eps_kernel}/{mass_kernel} thin prec {prec}")
        g1, j1, _ = gpu_sweep(T, P, prec, f_prev=f0, **over)
        compare(g1, j1, f1, i1, tol, front=None if prec == T.TR_FP64 else front_mask(P, f1),
                name=f"kernels {eps_kernel}/{mass_kernel} absorbing prec {prec}")


@pytest.mark.parametrize("make", [lambda: W.small_lognormal(16, n_src=3, seed=43),
                                  lambda: W.small_lognormal(24, n_src=2, seed=44, nside=1),
                                  lambda: W.rabbit_hole(0.5, 48, 2, nside=2)], ids=["cube16", "padded24", "slab48"])
def test_periodic_boundaries(T, orc, make):
    """Periodic boundaries (Sec. 2.8, nearest copy of every node) against the oracle."""
    P = make()
    f0, i0 = orc_sweep(orc, P, thin=True, periodic=True)
    f1, i1 = orc_sweep(orc, P, f_prev=f0, periodic=True)
    for prec, tol in ((T.TR_FP64, TOL64), (T.TR_FP32C, TOL32)):
        g0, j0, _ = gpu_sweep(T, P, prec, thin=True, periodic=True)
        compare(g0, j0, f0, i0, tol, name=f"{P.name} periodic thin prec {prec}")
        g1, j1, _ = gpu_sweep(T, P, prec, f_prev=f0, periodic=True)
        compare(g1, j1, f1, i1, tol, front=None if prec == T.TR_FP64 else front_mask(P, f1),
                name=f"{P.name} periodic absorbing prec {prec}")


@pytest.mark.parametrize("prec", ["fp64", "fp32c"])
def test_launch_shapes(T, orc, prec):
    # every integration form (a lane, a wave, a group of 4, 8 or 16 lanes per
    # ray), both buffer places, 1, 4 and 16 waves per target and both
    # accumulation forms give the oracle's flux; 60 sources on 12 rays put more
    # emitting points on a ray than a group of 4 or 8 lanes holds, so the
    # wider groups run too
    P = W.small_lognormal(16, n_src=60, seed=7, nside=1, n_radial=24)
    f0, i0 = orc_sweep(orc, P, thin=True)
    f1, i1 = orc_sweep(orc, P, f_prev=f0)
    pr, tol = (T.TR_FP64, TOL64) if prec == "fp64" else (T.TR_FP32C, TOL32)
    front = None if prec == "fp64" else front_mask(P, f1)
    shapes = [(w, b, im, 0) for w in (1, 4, 16) for b in (1, 2) for im in (1, 2, 3, 4, 5, 6, 7, 8)]
    shapes += [(w, 1, 0, am) for w in (8, 16) for am in (1, 2)]   # the accumulation forms
    for waves, buf, im, am in shapes:
        name = f"shape waves {waves} buffer {buf} integration {im} atomics {am}"
        g0, j0, st = gpu_sweep(T, P, pr, thin=True, launch=(waves, 0, buf, im, am))
        assert (st.waves_per_target, st.buffer_in_lds) == (waves, int(buf == 1))
        if im:
            assert st.integration_wave == {1: 1, 2: 64, 3: 4, 4: 8, 5: 16, 6: 4, 7: 8, 8: 16}[im]
            # the FP32 march exists for FP32 buffers; the FP64 form takes the FP64 groups
            assert st.integration_fp32 == int(im >= 6 and prec == "fp32c")
        cas = prec == "fp32c" and buf == 1 and waves in (8, 16) and am != 1
        assert st.lds_cas == int(cas)
        compare(g0, j0, f0, i0, tol, name=name + " thin")
        g1, j1, _ = gpu_sweep(T, P, pr, f_prev=f0, launch=(waves, 0, buf, im, am))
        compare(g1, j1, f1, i1, tol, front=front, name=name + " absorbing")


@pytest.mark.parametrize("prec", ["fp64", "fp32c"])
def test_many_emitting_points(T, orc, prec):
    # 4000 sources in 16^3 cells, 12 rays of 120 points, theta 0.3: rays hold
    # from one to more than 64 emitting points, so the rays beyond a group of
    # 4 or 16 lanes are marched again by groups of 8 to 64 lanes, and those
    # beyond 64 points by a wave
    P = W.small_lognormal(16, n_src=4000, seed=11, nside=1, n_radial=120, theta=0.3)
    f0, i0 = orc_sweep(orc, P, thin=True)
    f1, i1 = orc_sweep(orc, P, f_prev=f0)
    pr, tol = (T.TR_FP64, TOL64) if prec == "fp64" else (T.TR_FP32C, TOL32)
    front = None if prec == "fp64" else front_mask(P, f1)
    for im in ((3, 5) if prec == "fp64" else (3, 6, 8)):
        for waves in (4, 16):
            name = f"{prec} many emitters waves {waves} integration {im}"
            g0, j0, st = gpu_sweep(T, P, pr, thin=True, launch=(waves, 0, 0, im, 0))
            log(f"{name}: rays regrouped {st.rays_regrouped}, in FP32 {st.rays_fp32}")
            assert st.rays_regrouped > 0
            compare(g0, j0, f0, i0, tol, name=name + " thin")
            g1, j1, _ = gpu_sweep(T, P, pr, f_prev=f0, launch=(waves, 0, 0, im, 0))
            compare(g1, j1, f1, i1, tol, front=front, name=name + " absorbing")


@pytest.mark.parametrize("waves", [4, 16])
def test_split_ray_buffers(T, orc, waves):
    # N_side 4 with 64 radial points: four rows per ray (197 KB) do not fit in
    # LDS, three do, so the FP32C sweep keeps A, E, V in LDS and the emission
    # rows in device memory; the FP64 sweep maps and integrates the rays in
    # passes with LDS buffers, or keeps everything in device memory
    P = W.small_lognormal(16, n_src=6, seed=8, nside=4, n_radial=64)
    f0, i0 = orc_sweep(orc, P, thin=True)
    f1, i1 = orc_sweep(orc, P, f_prev=f0)
    front = front_mask(P, f1)
    for im in (0, 1, 2, 8):
        name = f"split waves {waves} integration {im}"
        g0, j0, st = gpu_sweep(T, P, T.TR_FP32C, thin=True, launch=(waves, 0, 0, im, 0))
        assert st.buffer_in_lds == 2
        compare(g0, j0, f0, i0, TOL32, name=name + " thin")
        g1, j1, _ = gpu_sweep(T, P, T.TR_FP32C, f_prev=f0, launch=(waves, 0, 0, im, 0))
        compare(g1, j1, f1, i1, TOL32, front=front, name=name + " absorbing")
    # FP64: four rows per ray in LDS for a third of the rays at a time (passes),
    # or all rows in device memory
    for buf, where in ((0, 3), (2, 0)):
        for im in (0, 1, 2):
            g1, j1, st = gpu_sweep(T, P, T.TR_FP64, f_prev=f0, launch=(waves, 0, buf, im, 0))
            assert st.buffer_in_lds == where
            compare(g1, j1, f1, i1, TOL64, name=f"fp64 waves {waves} buffer {buf} integration {im}")


@pytest.mark.parametrize("make", [lambda: W.small_lognormal(16, n_src=6, seed=31, nside=4, n_radial=48),
                                  lambda: W.small_amr(2, seed=32, n_src=12),
                                  lambda: W.small_uniform(24, q=2e48, n_radial=40)])
def test_fp32_march_across_fronts(T, orc, make):
    """The FP32 ray march (integration 6-8) on absorbing sweeps that hold
    ionisation fronts: zero previous flux (zeta_d = 2) and the oracle's own
    thin flux.  Away from the front the flux agrees with the FP64 oracle to
    1e-4 and the flags agree; some rays must have gone back to FP64 (a source
    below 1e-2 of its emitted Phi) and most must have stayed in FP32."""
    P = make()
    f0, _ = orc_sweep(orc, P, thin=True)
    for fp in (None, f0):
        f1, i1 = orc_sweep(orc, P, f_prev=fp)
        front = front_mask(P, f1)
        for im in (6, 7, 8):
            g1, j1, st = gpu_sweep(T, P, T.TR_FP32C, f_prev=fp, launch=(0, 0, 0, im, 0))
            assert st.integration_fp32 == 1
            log(f"{P.name} prev {'zero' if fp is None else 'thin'} integration {im}: rays in FP32 {st.rays_fp32}, "
                f"again in FP64 {st.rays_fp64_again}, front cells {int(front.sum())}")
            assert st.rays_fp32 > 0 and st.rays_fp64_again < st.rays_fp32
            compare(g1, j1, f1, i1, TOL32, front=front, name=f"fp32 march {im}")
        if fp is None:
            assert st.rays_fp64_again > 0


def test_errors(T):
    P = W.small_uniform(16)
    ctx = T.context_for(P, T.TR_FP64)
    nh = torch.tensor(P.n_h[0], device="cuda")
    bad = nh.clone()
    bad[5] = float("nan")
    with pytest.raises(T.TreeRayError) as e:
        ctx.build(bad)
    assert e.value.status == T.TR_EINVAL
    bad[5] = -1.0
    with pytest.raises(T.TreeRayError):
        ctx.build(bad)
    with pytest.raises(T.TreeRayError) as e:
        ctx.set_sources(0, [[1e30, 0, 0]], [1e48])
    assert e.value.status == T.TR_EINVAL
    out = torch.zeros(ctx.n_cells, dtype=torch.float64, device="cuda")
    with pytest.raises(T.TreeRayError) as e:   # sweep before a successful build
        ctx.sweep(out)
    assert e.value.status == T.TR_ESTATE
    ctx.build(nh, thin=True)
    tg = torch.tensor([0, 5, ctx.n_cells + 3], dtype=torch.int64, device="cuda")
    o = torch.zeros(3, dtype=torch.float64, device="cuda")
    ctx.sweep_targets(tg, o)
    with pytest.raises(T.TreeRayError) as e:
        ctx.sync()
    assert e.value.status == T.TR_EINVAL
    assert math.isnan(o[2].item()) and o[0].item() > 0
    # launch options out of range
    for bad_launch in ((3, 0, 0, 0, 0), (4, -1, 0, 0, 0), (4, 0, 3, 0, 0), (4, 0, 0, 9, 0), (4, 0, 0, 0, 3)):
        with pytest.raises(T.TreeRayError) as e:
            ctx.set_launch(*bad_launch)
        assert e.value.status == T.TR_EINVAL
    ctx.close()


def test_many_ray_passes(T, orc):
    # N_side 8 with 64 points in FP64: 768 rays of four rows (1.6 MB) are
    # mapped and integrated in passes of a few dozen rays held in LDS
    P = W.small_lognormal(16, n_src=3, seed=44, nside=8, n_radial=64)
    rng = np.random.default_rng(45)
    tg = np.sort(rng.choice(P.total_cells(), 96, replace=False))
    f0, i0 = orc_sweep(orc, P, thin=True, targets=tg)
    f1, i1 = orc_sweep(orc, P, f_prev=None, targets=tg)
    for waves in (4, 16):
        g0, j0, st = gpu_sweep(T, P, T.TR_FP64, thin=True, targets=tg, launch=(waves, 0, 1, 0, 0))
        assert st.buffer_in_lds == 3
        compare(g0, j0, f0, i0, TOL64, name=f"N_side 8 passes waves {waves} thin")
        g1, j1, _ = gpu_sweep(T, P, T.TR_FP64, targets=tg, launch=(waves, 0, 1, 0, 0))
        compare(g1, j1, f1, i1, TOL64, name=f"N_side 8 passes waves {waves} absorbing")


@pytest.mark.parametrize("nside,sub", [(1, 1), (1, 4), (8, 2), (8, 3), (16, 4)])
def test_pair_batches(T, orc, nside, sub):
    """The mapping takes (node, pixel) pairs 64 at a time: one pair per node
    (s = 1: 64 nodes in a batch) up to nodes of nearly 64 pairs (N_side 16:
    few or one in a batch, some left for the next), on a grid whose larger
    nodes are outside the angular table (24 cells: partial nodes)."""
    P = W.small_lognormal(24, n_src=5, seed=50 + sub, nside=nside, n_radial=20)
    P.params.subsample = sub
    tg = np.sort(np.random.default_rng(51).choice(P.total_cells(), 150, replace=False))
    f0, i0 = orc_sweep(orc, P, thin=True, targets=tg)
    for prec, tol in ((T.TR_FP64, TOL64), (T.TR_FP32C, TOL32)):
        g0, j0, st = gpu_sweep(T, P, prec, thin=True, targets=tg)
        assert 0 < st.nodes_tabulated < st.nodes_accepted * (12 * nside ** 2)
        compare(g0, j0, f0, i0, tol, name=f"pairs N_side {nside} s {sub} prec {prec}")


@pytest.mark.parametrize("theta", [0.5, 0.35])
def test_target_chunks(T, orc, theta):
    """Targets are walked and listed 32768 at a time: a list of two chunks and
    77 more, a bad index in each (NaN and an error at the sync), all other
    targets as the oracle has them; theta 0.35 accepts more nodes than half a
    list holds."""
    P = W.small_lognormal(16, n_src=3, seed=60)
    f0, i0 = orc_sweep(orc, P, thin=True, theta=theta)
    n = P.total_cells()
    tg = np.arange(2 * 32768 + 77, dtype=np.int64) % n
    bad = [5, 32768 + 9, 65536 + 70]
    tg[bad] = [-1, n, n + 7]
    ok = np.ones(tg.size, bool)
    ok[bad] = False
    for prec, tol in ((T.TR_FP64, TOL64), (T.TR_FP32C, TOL32)):
        with T.context_for(P, prec, theta=theta) as ctx:
            ctx.build(torch.tensor(P.n_h[0], device="cuda"), thin=True)
            out = torch.zeros(tg.size, dtype=torch.float64, device="cuda")
            ion = torch.full((tg.size,), 7, dtype=torch.uint8, device="cuda")
            ctx.sweep_targets(torch.tensor(tg, device="cuda"), out, ion)
            with pytest.raises(T.TreeRayError) as e:
                ctx.sync()
            assert e.value.status == T.TR_EINVAL
            g, j = out.cpu().numpy(), ion.cpu().numpy()
        assert np.all(np.isnan(g[bad])) and np.all(j[bad] == 0)
        compare(g[ok], j[ok], f0[tg[ok]], i0[tg[ok]], tol, name=f"chunks theta {theta} prec {prec}")


@pytest.mark.parametrize("nside,waves", [(8, 0), (8, 4), (16, 8)])
def test_more_emitting_rays_than_buffers(T, orc, nside, waves):
    """Sources on a tenth of the cells: nearly every one of the 768 or 3072 rays
    holds emission, more than the workgroup has buffers for, so FP32C maps
    and marches the rays in several passes."""
    P = W.small_lognormal(16, n_src=400, seed=70, nside=nside, n_radial=40)
    tg = np.sort(np.random.default_rng(71).choice(P.total_cells(), 70, replace=False))
    f0, i0 = orc_sweep(orc, P, thin=True, targets=tg)
    for am in (1, 2):
        g0, j0, st = gpu_sweep(T, P, T.TR_FP32C, thin=True, targets=tg, launch=(waves, 0, 0, 0, am))
        compare(g0, j0, f0, i0, TOL32, name=f"{nside} passes waves {waves} atomics {am}")


def test_delta_edges(T, orc):
    """The exact lower median of every domain: one, two and odd counts of
    cells around a wave, a block's run and its unrolled loop; ties, zeros,
    denormals and values that differ in the last bit, in neighbouring domains."""
    rng = np.random.default_rng(80)
    sizes = [1, 2, 3, 63, 64, 65, 511, 513, 2047, 2049, 5000, 40007, 1, 300000]
    old, new = [], []
    for q, n in enumerate(sizes):
        kind = q % 4
        if kind == 0:
            v = rng.integers(0, 3, n).astype(np.float64)                       # ties and zeros
        elif kind == 1:
            v = 1.0 + rng.integers(0, 50, n) * np.finfo(np.float64).eps        # the last bits
        elif kind == 2:
            v = rng.integers(0, 1 << 20, n) * 5e-324                           # denormals
        else:
            v = np.exp(40.0 * rng.standard_normal(n))
        old.append(v)
        new.append(v * (1.0 + 0.1 * rng.standard_normal(n)) if kind != 2 else v + 5e-324 * rng.integers(0, 9, n))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    fo, fn = np.concatenate(old), np.abs(np.concatenate(new))
    out = torch.full((len(sizes),), -1.0, dtype=torch.float64, device="cuda")
    T.delta_noalloc(torch.tensor(fn, device="cuda"), torch.tensor(fo, device="cuda"), off, out)
    got = out.cpu().numpy()
    for d in range(len(sizes)):
        ref = orc.delta_cell(fn[off[d]:off[d + 1]], fo[off[d]:off[d + 1]])
        # a division and a difference: an ulp each
        assert got[d] == ref or got[d] == pytest.approx(ref, rel=1e-15, abs=0.0), (d, got[d], ref)


@pytest.mark.parametrize("nside,n_radial,n_src,prec,launch,over", [
    (32, 48, 3, 0, (0, 0, 0, 0, 0), {}),
    (32, 48, 400, 0, (4, 0, 0, 0, 0), {}),                 # more rays with emission than buffers
    (32, 48, 400, 0, (16, 0, 1, 0, 0), {}),
    (32, 48, 3, 0, (0, 0, 2, 0, 0), {}),
    (32, 48, 3, 0, (0, 0, 0, 0, 0), {"eps_kernel": 5}),    # radial-kernel variants: device memory
    (32, 48, 3, 0, (2, 0, 0, 0, 0), {}),                   # 2 waves: device memory
    (32, 20, 400, 1, (0, 0, 0, 0, 0), {}),
    (32, 100, 400, 1, (8, 0, 0, 0, 0), {}),                # two mask words
    (32, 48, 3, 1, (0, 0, 2, 0, 0), {}),
    (32, 48, 400, 1, (0, 0, 0, 0, 0), {"theta": 0.05}),    # walks by the fallback pass
    (64, 24, 3, 0, (0, 0, 0, 0, 0), {}),
    (64, 48, 400, 1, (0, 0, 0, 0, 0), {}),
    (64, 100, 3, 1, (0, 0, 1, 0, 0), {}),
])
def test_marks_outside_lds(T, orc, nside, n_radial, n_src, prec, launch, over):
    """N_side 32 and 64: the masks and numbers of 12288 and 49152 rays do not
    fit in LDS beside ray buffers, wherever those are."""
    P = W.small_lognormal(16, n_src=n_src, seed=90, nside=nside, n_radial=n_radial)
    P.params.subsample = 3
    for k, v in over.items():
        setattr(P.params, k, v)
    tg = np.sort(np.random.default_rng(91).choice(P.total_cells(), 24, replace=False))
    f0, i0 = orc_sweep(orc, P, thin=True, targets=tg)
    tol = TOL64 if prec == T.TR_FP64 else TOL32
    g0, j0, st = gpu_sweep(T, P, prec, thin=True, targets=tg, launch=launch)
    compare(g0, j0, f0, i0, tol, name=f"N_side {nside} N_R {n_radial} {n_src} sources prec {prec} launch {launch}")
    in_lds = launch[2] != 2 and launch[0] != 2 and "eps_kernel" not in over
    assert (st.buffer_in_lds != 0) == in_lds


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nside,n_radial,waves,over", [
    (2, 100, 8, {}),                     # supports of many points, two mask words
    (4, 20, 1, {}),
    (8, 24, 16, {"eps_kernel": 5}),      # spread emission (run by 8 waves)
    (2, 20, 4, {"eps_kernel": 4, "mass_kernel": 6}),
    (4, 100, 8, {"eps_kernel": 6}),
])
def test_device_memory_points(T, orc, nside, n_radial, waves, over, prec):
    """Ray buffers in device memory: a lane per point of the pairs' supports,
    laid end to end over pairs without any point below their ray's outermost
    emitting one, with one and with more points than a wave has lanes."""
    P = W.small_lognormal(16, n_src=6, seed=95, nside=nside, n_radial=n_radial)
    for k, v in over.items():
        setattr(P.params, k, v)
    tg = np.sort(np.random.default_rng(96).choice(P.total_cells(), 200, replace=False))
    f0, i0 = orc_sweep(orc, P, thin=True, targets=tg)
    g0, j0, st = gpu_sweep(T, P, prec, thin=True, targets=tg, launch=(waves, 0, 2, 0, 0))
    assert st.buffer_in_lds == 0
    compare(g0, j0, f0, i0, TOL64 if prec == T.TR_FP64 else TOL32, name=f"N_side {nside} N_R {n_radial} {over}")


@pytest.mark.parametrize("nside,n_radial,prec,in_lds", [(8, 64, 0, True), (8, 100, 0, False), (16, 16, 0, True),
                                                        (16, 32, 0, False), (8, 64, 1, True), (16, 32, 1, False)])
def test_kernel_variant_buffers(T, orc, nside, n_radial, prec, in_lds):
    """Radial-kernel variants on either side of the rule that puts their ray
    buffers (of all rays) in LDS in passes or in device memory."""
    P = W.small_lognormal(16, n_src=4, seed=97, nside=nside, n_radial=n_radial)
    P.params.eps_kernel, P.params.mass_kernel = 5, 6
    tg = np.sort(np.random.default_rng(98).choice(P.total_cells(), 100, replace=False))
    f0, i0 = orc_sweep(orc, P, thin=True, targets=tg)
    g0, j0, st = gpu_sweep(T, P, prec, thin=True, targets=tg)
    assert (st.buffer_in_lds != 0) == in_lds
    compare(g0, j0, f0, i0, TOL64 if prec == T.TR_FP64 else TOL32, name=f"variants N_side {nside} N_R {n_radial}")


@pytest.mark.parametrize("n_dom", [15, 16, 17, 64, 700])
def test_delta_many_domains(T, orc, n_dom):
    """Up to 16 domains the median's bins are picked by the last block of a
    pass, beyond that by a launch: the same medians, in a context and (up to
    64 domains) without one."""
    rng = np.random.default_rng(110 + n_dom)
    A = W.small_lognormal(8, n_src=1, seed=1, nside=1, n_radial=12)
    P = W.Problem("many", A.domains * n_dom, A.n_h * n_dom, A.src_xyz * n_dom, A.src_q * n_dom, A.params)
    old = np.exp(20.0 * rng.standard_normal(512 * n_dom))
    old[::7] = 0.0
    new = old * (1.0 + 0.1 * rng.standard_normal(old.size)) + 1e-3
    a, b = torch.tensor(new, device="cuda"), torch.tensor(old, device="cuda")
    ref = np.array([orc.delta_cell(new[512 * d:512 * d + 512], old[512 * d:512 * d + 512]) for d in range(n_dom)])
    with T.context_for(P, T.TR_FP64) as ctx:
        for _ in range(2):   # (the second call finds the first one's scratch)
            np.testing.assert_allclose(ctx.delta(a, b), ref, rtol=1e-15)
    if n_dom <= 64:
        out = torch.zeros(n_dom, dtype=torch.float64, device="cuda")
        T.delta_noalloc(a, b, 512 * np.arange(n_dom + 1), out)
        np.testing.assert_allclose(out.cpu().numpy(), ref, rtol=1e-15)


def test_step_after_more_domains(T, orc):
    """A context that stepped one domain is given 700 (their delta_cell takes
    more host memory than a page), then one again: every step's fluxes and
    deltas as those of a fresh context's eager calls."""
    import ctypes as C
    A = W.small_lognormal(8, n_src=1, seed=100, nside=1, n_radial=12)
    B = W.small_lognormal(8, n_src=2, seed=101, nside=1, n_radial=12)

    def step(ctx, probs):
        nh = torch.tensor(np.concatenate([p.n_h[0] for p in probs]), device="cuda")
        fp = torch.full((nh.numel(),), 1e8, dtype=torch.float64, device="cuda")
        out = torch.zeros_like(fp)
        return ctx.step(nh, fp, out), out.cpu().numpy(), (nh, fp)

    def eager(probs):
        P = W.Problem("many", [p.domains[0] for p in probs], [p.n_h[0] for p in probs],
                      [p.src_xyz[0] for p in probs], [p.src_q[0] for p in probs], A.params)
        with T.context_for(P, T.TR_FP64) as ctx:
            nh = torch.tensor(np.concatenate(P.n_h), device="cuda")
            fp = torch.full((nh.numel(),), 1e8, dtype=torch.float64, device="cuda")
            out = torch.zeros_like(fp)
            ctx.build(nh, fp)
            ctx.sweep(out)
            d = ctx.delta(out, fp)
            ctx.sync()
            return d, out.cpu().numpy()

    with T.context_for(A, T.TR_FP64) as ctx:
        for probs in ([A], [A, B] * 350, [B]):
            if ctx.n_domains != len(probs) or probs[0] is B:
                arr = (T._Domain * len(probs))()
                for i, p in enumerate(probs):
                    arr[i].nroot[:] = [int(v) for v in p.domains[0].nroot]
                    arr[i].root_block_cm = float(p.domains[0].root_block_cm)
                ctx._check(ctx.L.tr_set_domains(ctx.h, len(probs), arr))
                ctx.n_domains = len(probs)
                for i, p in enumerate(probs):
                    ctx.set_sources(i, p.src_xyz[0], p.src_q[0])
            d, f, _ = step(ctx, probs)
            d0, f0 = eager(probs)
            np.testing.assert_allclose(f, f0, rtol=1e-10, atol=1e-12 * f0.max())
            np.testing.assert_allclose(d, d0, rtol=1e-9)


@pytest.mark.parametrize("prec,n_src", [(0, 3), (0, 400), (1, 3)])
def test_statistics_of_long_walks(T, prec, n_src):
    """theta = 0 opens every node: each of the targets tests all nodes and
    accepts all other cells (4095, more than the lists hold: the fallback
    pass), every one of them of the target's own size and so in the angular
    table, also where the rays take several passes (400 sources in FP64)."""
    P = W.small_lognormal(16, n_src=n_src, seed=120, nside=8, n_radial=40)
    tg = np.arange(0, P.total_cells(), 37)
    _, _, st = gpu_sweep(T, P, prec, thin=True, targets=tg, theta=0.0)
    assert st.nodes_accepted == tg.size * (P.total_cells() - 1) and st.nodes_accepted > tg.size * 3072
    assert st.nodes_tested == tg.size * st.n_nodes
    assert st.nodes_tabulated == st.nodes_accepted
    assert st.guard_recomputes == 0


@pytest.mark.parametrize("prec,nside,n_radial", [(1, 4, 40), (1, 2, 60), (0, 4, 40)])
def test_marked_and_mapped_points_agree(T, prec, nside, n_radial):
    """The points that the marking gives a target's emission and those that the
    mapping adds it to are the same: a domain whose sources are 1e13 times
    fainter than its neighbour's is swept after and beside that one as it is
    alone (emission left on an unmarked point of the neighbour's, 1e-8 of a
    source or more, would swamp it).  A lane per ray reads every point."""
    A = W.small_lognormal(24, n_src=600, seed=130, nside=nside, n_radial=n_radial)
    B = W.small_lognormal(16, n_src=3, seed=131, nside=nside, n_radial=n_radial)
    scale = 1e-13
    both = W.Problem("two", A.domains + B.domains, A.n_h + B.n_h, A.src_xyz + B.src_xyz,
                     [A.src_q[0], scale * B.src_q[0]], A.params)
    n_a = A.total_cells()
    for integration in (1, 0):
        alone, _, _ = gpu_sweep(T, B, prec, thin=True, launch=(4, 0, 0, integration, 2))
        rng = np.random.default_rng(132)
        tg = rng.permutation(both.total_cells())   # the domains' targets follow each other in a workgroup
        f, _, st = gpu_sweep(T, both, prec, thin=True, targets=tg, launch=(4, 0, 0, integration, 2))
        assert (st.buffer_in_lds == 2) == (prec == 1)   # split rows in FP32
        g = np.empty_like(f)
        g[tg] = f
        np.testing.assert_allclose(g[n_a:], scale * alone, rtol=1e-3 if prec == 1 else 1e-9)


def test_table_without_its_largest_ratio(T, orc):
    """N_side 8 with s = 4 on 80^3: the pairs of nodes of 32 target sizes (15
    million offsets) do not fit the entries' 25 bits, and the table does
    without them: the walk classifies those nodes, with the same weights."""
    P = W.small_lognormal(80, n_src=5, seed=140, nside=8, n_radial=40)
    P.params.subsample = 4
    tg = np.sort(np.random.default_rng(141).choice(P.total_cells(), 200, replace=False))
    f0, i0 = orc_sweep(orc, P, thin=True, targets=tg)
    for prec, tol in ((T.TR_FP64, TOL64), (T.TR_FP32C, TOL32)):
        with T.context_for(P, prec) as ctx:
            assert ctx.L.tr_last_error(ctx.h) == b""
            ctx.build(torch.tensor(P.n_h[0], device="cuda"), thin=True)
            out = torch.zeros(tg.size, dtype=torch.float64, device="cuda")
            ion = torch.zeros(tg.size, dtype=torch.uint8, device="cuda")
            ctx.sweep_targets(torch.tensor(tg, device="cuda"), out, ion)
            ctx.sync()
            st = ctx.stats()
            # a few nodes of 32 target sizes a target (grids of 80 cells hold 3 of them an axis)
            assert 0 < st.nodes_accepted - st.nodes_tabulated < 40 * tg.size
            compare(out.cpu().numpy(), ion.cpu().numpy(), f0, i0, tol, name=f"table prec {prec}")


def test_pool_of_pairs_used_up(T, orc):
    """A coarse target beside refined blocks accepts some 500 nodes finer than
    itself, which no table holds; at N_side 32 their pairs take several times
    its share of the chunk's pool, so 600 such targets use it up and the rest
    are walked by the fallback pass."""
    P = W.small_amr(2, seed=3, threshold=150.0, nside=32)
    dom, theta = P.domains[0], 0.3
    lo, size = W.cell_lo_size(dom)
    coarse = np.nonzero(size == 2)[0]
    c = int(coarse[1200])
    ls, _ = orc.accepted(dom, P.params, P.n_h[0], P.src_xyz[0], P.src_q[0], c, theta=theta)
    fine = ls[ls[:, 3] == 1]
    xt = lo[c] + 0.5 * size[c]
    units = sum(-(-len(orc.node_pixels(32, P.params.subsample, b[:3], b[:3] + 1, xt)) // 4) for b in fine)
    n = 600
    pool = n * 1024 + torch.cuda.get_device_properties(0).multi_processor_count * 16 * 256
    assert len(ls) < 3072 and n * units > 1.2 * pool   # the lists would hold the walk, the pool does not
    tg = np.full(n, c, np.int64)
    f0, i0 = orc_sweep(orc, P, thin=True, targets=tg[:1], theta=theta)
    for prec, tol in ((T.TR_FP64, TOL64), (T.TR_FP32C, TOL32)):
        g, j, st = gpu_sweep(T, P, prec, thin=True, targets=tg, theta=theta)
        assert st.overflow == 0 and st.nodes_accepted == n * len(ls)
        compare(g, j, np.repeat(f0, n), np.repeat(i0, n), tol, name=f"pool prec {prec}")


@pytest.mark.parametrize("nside,n_radial,waves", [(2, 64, 4), (4, 32, 4), (4, 32, 0), (8, 32, 8)])
def test_fp64_rays_in_passes_with_many_sources(T, orc, nside, n_radial, waves):
    """FP64 with emission on nearly every ray: more than a target has buffers
    for, so they are mapped and integrated in several passes."""
    P = W.small_lognormal(16, n_src=400, seed=150, nside=nside, n_radial=n_radial)
    tg = np.sort(np.random.default_rng(151).choice(P.total_cells(), 1100, replace=False))
    f0, i0 = orc_sweep(orc, P, thin=True, targets=tg)
    g0, j0, st = gpu_sweep(T, P, T.TR_FP64, thin=True, targets=tg, launch=(waves, 0, 1, 0, 0))
    assert st.buffer_in_lds == 3
    compare(g0, j0, f0, i0, TOL64, name=f"N_side {nside} N_R {n_radial} waves {waves}")
    f1, i1 = orc_sweep(orc, P, f_prev=np.repeat(1e9, P.total_cells()), targets=tg)
    g1, j1, _ = gpu_sweep(T, P, T.TR_FP64, f_prev=np.repeat(1e9, P.total_cells()), targets=tg, launch=(waves, 0, 1, 0, 0))
    compare(g1, j1, f1, i1, TOL64, name=f"N_side {nside} N_R {n_radial} waves {waves} absorbing")


@pytest.mark.parametrize("nside,sub", [(1, 4), (8, 3)])
def test_nodes_outside_the_table(T, orc, nside, sub):
    """24 cells a side pad the octree: some nodes are partial, which no table
    holds, and the walk classifies them."""
    P = W.small_lognormal(24, n_src=5, seed=160, nside=nside, n_radial=20)
    P.params.subsample = sub
    tg = np.sort(np.random.default_rng(161).choice(P.total_cells(), 150, replace=False))
    f0, i0 = orc_sweep(orc, P, thin=True, targets=tg)
    for prec, tol in ((T.TR_FP64, TOL64), (T.TR_FP32C, TOL32)):
        g0, j0, st = gpu_sweep(T, P, prec, thin=True, targets=tg)
        assert 0.5 * st.nodes_accepted < st.nodes_tabulated < st.nodes_accepted
        compare(g0, j0, f0, i0, tol, name=f"partial nodes N_side {nside} prec {prec}")


def test_delta_beyond_32_bits(T):
    """One domain of 8.6e9 cells (69 GB, the two fields the same memory a cell
    apart): counts of 2^32 cells and more.  The lower median is the second
    value, so the largest change is from it to the third."""
    sizes, values = (4_100_000_000, 4_200_000_000, 300_000_000), (1e-300, 1.0, 4.0)
    n = sum(sizes)
    if torch.cuda.mem_get_info()[0] < 8 * n + (8 << 30):
        pytest.skip("needs 77 GB of free device memory")
    f = torch.empty(n + 1, dtype=torch.float64, device="cuda")
    at = 0
    for m, v in zip(sizes, values):
        f[at:at + m] = v
        at += m
    f[n] = values[2]
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    T.delta_noalloc(f[1:], f, np.array([0, n]), out)
    got = out.item()
    del f
    torch.cuda.empty_cache()
    assert got == 3.0   # 0.75 with the third value as the median, 1e300 with the first


@pytest.mark.parametrize("integration", [1, 2, 3, 6])
def test_emission_rows_left_zero(T, integration):
    """Emission rows in device memory are zero for the next target also where a
    source lies exactly on an evaluation point and the weight of the next
    point rounds to a negative value: a domain with faint sources beside one
    with bright ones is as it is alone.  9 x 8 root-block diagonals and 37
    points put 72 (i/36)^2 on whole cells."""
    P0 = W.small_lognormal(8, n_src=1, seed=1, nside=4, n_radial=37)
    nroot, rb = (1, 4, 8), P0.domains[0].root_block_cm
    dom = W.Domain(nroot=nroot, root_block_cm=rb)
    n, rng = dom.n_cells(), np.random.default_rng(5)

    def centres(k):
        return (np.floor(rng.uniform(0, 1, (k, 3)) * 8 * np.array(nroot)) + 0.5) * (rb / 8)

    bright, faint = (centres(40), np.full(40, 1e49)), (centres(2), np.full(2, 1e36))
    flux = []
    for srcs in ([faint], [bright, faint]):
        P = W.Problem("rows", [dom] * len(srcs), [np.full(n, 1.0)] * len(srcs), [s[0] for s in srcs],
                      [s[1] for s in srcs], P0.params)
        tg = np.random.default_rng(6).permutation(P.total_cells())
        f, _, st = gpu_sweep(T, P, T.TR_FP32C, thin=True, targets=tg, launch=(4, 0, 0, integration, 2), theta=0.0)
        assert st.buffer_in_lds == 2
        g = np.empty_like(f)
        g[tg] = f
        flux.append(g[-n:])
    np.testing.assert_allclose(flux[1], flux[0], rtol=1e-3)

"""GPU: the two-kernel tick -- kernels and dispatch branches at the sizes
where they can go wrong, against the oracle."""

import numpy as np
import pytest

import oracle
import spff_inputs as si
from gpu_common import device, cfg_for, planes_to_tensor, tensor_to_planes, rel_l2
from oracle import spectral as osp
from paper_2203_16467_amd import spff

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,B", [(128, 128, 1), (256, 2048, 1), (512, 64, 3), (1024, 256, 3), (2048, 128, 1),
                                     (64, 1024, 5)])
def test_fp64_register_kernels_match_oracle_and_lds_kernels(nx, ny, B):
    """FP64 problems take the register kernels where the grid has them
    (rows of 128..1024, columns of 128..2048 points); a plan of the LDS kind
    asks for the LDS kernels.  Both give the operators to FP64 rounding."""
    import torch
    print(f"fp64 {B} x {nx}x{ny}", flush=True)
    cfg = cfg_for(nx, ny, "fp64")
    E = torch.ones((B, ny, nx), dtype=torch.float64, device=device())
    p = spff.Problem(E, cfg)
    x = np.random.default_rng(nx + ny).standard_normal((B, 3, ny, nx))
    xt = torch.from_numpy(x).to(device())
    got = [p.apply_operator(op, xt if op != spff.OP_NEG_LAPLACIAN else xt[:, 0]).cpu().numpy()
           for op in (spff.OP_PROJECT, spff.OP_NEG_LAPLACIAN, spff.OP_DISPLACEMENT)]
    for b in range(B):
        assert rel_l2(got[0][b], tensor_to_planes(osp.project(planes_to_tensor(x[b])))) < 1e-12
        assert rel_l2(got[1][b], -osp.laplacian(x[b, 0])) < 1e-12
    last = len(p.plan_buckets()) - 1
    plan = p.get_plan(last)
    assert plan["row_kind"] == spff.FFT_LDS and plan["col_kind"] == spff.FFT_LDS
    p.set_plan(last, plan)
    for op, g in zip((spff.OP_PROJECT, spff.OP_NEG_LAPLACIAN, spff.OP_DISPLACEMENT), got):
        again = p.apply_operator(op, xt if op != spff.OP_NEG_LAPLACIAN else xt[:, 0]).cpu().numpy()
        assert rel_l2(again, g) < 1e-12
    p.close()


@pytest.mark.parametrize("K,graph", [(1, 0), (2, 0), (3, 1), (32, 0), (32, 1)])
def test_blocks_in_flight_give_the_problems_alone(K, graph):
    """Blocks of ticks are enqueued ahead of the host's checks; problems of a
    batch finish at different times, so that the bucket (launch size) shrinks
    while blocks are in flight.  With the plan fixed, every problem's steps
    are bit for bit those of the problem alone, at any block length."""
    import torch
    n, B = 64, 5
    E = np.stack([si.young_modulus(n, 3.0, 0.05 + 0.06 * b, 90 + b) for b in range(B)])
    ramp = si.uniaxial_ramp(12, 0.2, 2.0)[4:7]
    kw = dict(at=2, plan_rows=2, plan_cols=2)
    p = spff.Problem(torch.from_numpy(E).to(device()), cfg_for(n, use_graph=graph, ticks_per_sync=K, **kw))
    _, stats = p.run_sequence(ramp)
    f = p.get_fields(spff.FIELD_PHI | spff.FIELD_EPS_STAR)
    ticks = [sum(s["ticks"] for s in row) for row in stats]
    assert len(set(ticks)) > 1  # they do not finish together
    for b in range(B):
        q = spff.Problem(torch.from_numpy(E[b]).to(device()), cfg_for(n, **kw))
        alone = [q.load_step(e)[1][0] for e in ramp]
        g = q.get_fields(spff.FIELD_PHI | spff.FIELD_EPS_STAR)
        for k in f:
            assert torch.equal(f[k][b], g[k][0]), (b, k)
        for s, a in zip(stats[b], alone):
            assert all(s[k] == a[k] for k in ("cg_iters", "bccg_iters", "am_iters", "ticks", "F_e", "F_f"))
        q.close()
    p.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shift", [0, 1, 2])
def test_operators_and_state_with_shifted_buffers(precision, shift):
    """Caller buffers at any element offset: operators read and write them
    directly where they are aligned to a pixel pair and through the scratch
    otherwise; states and fields move 16 bytes at a time or one value."""
    import ctypes
    import torch
    n, B = 32, 3
    dt = torch.float64 if precision == "fp64" else torch.float32
    E = torch.from_numpy(np.stack([si.young_modulus(n, 3.0, 0.1, 7 + b) for b in range(B)])).to(device(), dt)
    p = spff.Problem(E, cfg_for(n, precision=precision))
    p.load_step((0.0, 0.1, 0.02))
    g = torch.Generator(device="cpu").manual_seed(3)
    x = torch.randn(B, 3, n, n, generator=g, dtype=torch.float64).to(device(), dt)
    L = spff.lib()

    def shifted(shape):
        t = torch.empty(int(np.prod(shape)) + 8, dtype=dt, device=device())
        return t[shift:shift + int(np.prod(shape))].view(shape)

    for op, pin, pout in ((spff.OP_PROJECT, 3, 3), (spff.OP_NEG_LAPLACIAN, 1, 1), (spff.OP_DISPLACEMENT, 3, 2)):
        src = shifted((B, pin, n, n))
        src.copy_(x[:, :pin])
        want = p.apply_operator(op, x if pin == 3 else x[:, 0])
        dst = shifted((B, pout, n, n))
        assert L.spff_apply_operator(p.handle, op, ctypes.c_void_p(src.data_ptr()),
                                     ctypes.c_void_p(dst.data_ptr())) == 0
        assert torch.equal(dst.view(want.shape), want)
    st, eb = p.get_state()
    f = p.get_fields(0x7F)
    again = shifted(tuple(st.shape))
    assert L.spff_get_state(p.handle, ctypes.c_void_p(again.data_ptr()), None) == 0
    assert torch.equal(again, st)
    other = torch.zeros_like(st)
    other[:, 3:] = 0.25
    p.set_state(other, np.zeros(3))
    assert float(p.get_fields(spff.FIELD_PHI)["phi"].min()) == 0.25
    assert L.spff_set_state(p.handle, ctypes.c_void_p(again.data_ptr()), eb.ctypes.data_as(
        ctypes.POINTER(ctypes.c_double))) == 0
    g2 = {}
    ptrs = []
    for bit in sorted(spff.FIELD_PLANES):
        g2[spff.FIELD_NAMES[bit]] = t = shifted((B, spff.FIELD_PLANES[bit], n, n))
        ptrs.append(t.data_ptr())
    assert L.spff_get_fields(p.handle, -1, 0x7F, (ctypes.c_void_p * len(ptrs))(*ptrs)) == 0
    for k in f:
        assert torch.equal(g2[k], f[k]), k
    one = p.get_fields(0x7F, index=1)
    for k in f:
        assert torch.equal(one[k], f[k][1]), k
    # a state with one bad value is refused as a whole
    bad = again.clone()
    bad[2, 4, n - 1, n - 1] = float("nan")
    with pytest.raises(spff.SpffError):
        p.set_state(bad)
    assert torch.equal(p.get_state()[0], st)
    p.close()


@pytest.mark.parametrize("nx,ny,B", [(128, 128, 136), (256, 256, 34)])
def test_column_loads_ahead_leave_the_results(nx, ny, B):
    """Launches of at most 2048 column wavefronts load the residual ahead of
    the transform.  With the plan fixed the batch, which has more, and the
    problem alone, which has fewer, agree bit for bit."""
    import torch
    distinct = 2
    E = np.stack([si.young_modulus(nx, 3.0, 0.1 + 0.05 * b, 40 + b, ny=ny) for b in range(distinct)])
    kw = dict(plan_rows=4 if nx == 256 else 8, plan_cols=4)
    eps = si.uniaxial_ramp(12, 0.2, 2.0)[5]
    Et = torch.from_numpy(E).to(device())
    p = spff.Problem(Et.repeat(B // distinct, 1, 1).contiguous(), cfg_for(nx, ny, **kw))
    _, stats = p.load_step(eps)
    f = p.get_fields(spff.FIELD_PHI | spff.FIELD_EPS_STAR)
    for b in range(distinct):
        q = spff.Problem(Et[b], cfg_for(nx, ny, **kw))
        _, alone = q.load_step(eps)
        g = q.get_fields(spff.FIELD_PHI | spff.FIELD_EPS_STAR)
        for k in f:
            assert torch.equal(f[k][b], g[k][0]) and torch.equal(f[k][B - distinct + b], g[k][0]), k
        assert stats[b]["cg_iters"] == alone[0]["cg_iters"] > 0
        q.close()
    p.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_static_step_is_the_same_at_any_block_length(precision):
    """The static step's blocks are cut after a row kernel and shrink after
    the first: no block length changes its result or its tick count."""
    import torch
    n = 64
    dt = torch.float64 if precision == "fp64" else torch.float32
    E = torch.from_numpy(si.young_modulus(n, 3.0, 0.2, 5)).to(device(), dt).contiguous()
    want = None
    for K in (1, 2, 5, 64):
        state = torch.zeros((5, n, n), dtype=dt, device=device())
        _, s = spff.load_step_static(cfg_for(n, precision=precision, at=2, ticks_per_sync=K), E, state,
                                     (0.0, 0.2, 0.03))
        got = (state, s["ticks"], s["cg_iters"], s["F_e"], s["F_f"])
        want = want or got
        assert torch.equal(got[0], want[0]) and got[1:] == want[1:], K


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_spectral_stress_and_energy_at_its_corners(precision):
    """Vanishing, equal, opposite and barely different eigenvalues, either
    sign: the stress and the driving energy of the strain-spectral split are
    the oracle's to 16 roundings of the largest term."""
    import torch
    n = 16
    dt = torch.float64 if precision == "fp64" else torch.float32
    corners = [(0, 0, 0), (1, 1, 0), (-1, -1, 0), (1, -1, 0), (1, 0, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
               (1, 1, 1), (-1, -1, 1), (1, 1 + 1e-6, 0), (1e-6, -1, 0), (1, -1e-6, 1e-6), (2, 0.5, 1), (-2, -0.5, -1),
               (1e-12, 1e-12, 0)]
    x = np.array(corners, dtype=np.float64) * 1e-2
    eps = np.zeros((3, n * n))
    phi = np.zeros(n * n)
    for i in range(n * n):
        eps[:, i] = x[i % len(x)]
        phi[i] = (i // len(x)) / 16.0
    # the fluctuations are stored in the problem's precision; the mean is 0
    eps = torch.from_numpy(eps.reshape(3, n, n)).to(dt)
    phi = torch.from_numpy(phi.reshape(n, n)).to(dt)
    E = torch.ones((n, n), dtype=dt, device=device())
    cfg = cfg_for(n, precision=precision, split="spectral")
    p = spff.Problem(E, cfg)
    state = torch.cat([eps, phi[None], phi[None]]).to(device())
    p.set_state(state[None].contiguous(), np.zeros(3))
    f = p.get_fields(spff.FIELD_STRESS | spff.FIELD_PSI_PLUS)
    nu = cfg.nu
    lam, mu = nu / ((1 + nu) * (1 - 2 * nu)), 1 / (2 * (1 + nu))
    t = planes_to_tensor(eps.double().numpy())
    sp, sm = oracle.constitutive.sigma0(t, np.full((n, n), lam), np.full((n, n), mu), "spectral")
    h = ((1 - phi.double().numpy()) ** 2 + cfg.k_res)[..., None, None]
    want = tensor_to_planes(h * sp + sm)
    got = f["stress"][0].double().cpu().numpy()
    u = np.finfo(np.float64 if precision == "fp64" else np.float32).eps
    scale = (lam + 2 * mu) * np.abs(eps.double().numpy()).sum(axis=0)
    assert np.all(np.abs(got - want) <= 16 * u * scale[None] + 1e-300)
    pp = oracle.constitutive.psi0(t, np.full((n, n), lam), np.full((n, n), mu), "spectral")[0]
    gpp = f["psi_plus"][0].double().cpu().numpy()
    assert np.all(np.abs(gpp - pp) <= 16 * u * (lam + 2 * mu) * np.abs(eps.double().numpy()).sum(axis=0) ** 2 + 1e-300)
    p.close()


@pytest.mark.parametrize("n,B,rows", [(512, 32, 2), (64, 128, 1)])
def test_near_equilibrium_scaling_is_one_factor_with_many_row_groups(n, B, rows):
    """Algorithm 4's strain scaling in launches of 8192 row groups, of which
    the GPU holds a part at once: every row of a problem is scaled by the one
    factor that its statistics report (eps* is that factor, in the working
    precision, times the strain of the same step without scaling), and the
    batch agrees bit for bit with the problems alone."""
    import torch
    distinct = 4
    print(f"scaling {B} x {n}", flush=True)
    E = np.stack([si.young_modulus(n, n / 32.0, 0.2, 60 + b) for b in range(distinct)])
    Et = torch.from_numpy(E).to(device())
    eps = (0.0, 0.5, 0.0)
    kw = dict(evolution=spff.EVOL_NEAR_EQ, drive_threshold=0.0, deps_max=1e-3, eta=0.0, plan_rows=rows, plan_cols=1,
              max_bccg=20)
    free = spff.Problem(Et, cfg_for(n, fphi_max=1e30, **kw))
    free.load_step(eps)
    before = free.get_fields(spff.FIELD_EPS_STAR)["eps_star"].cpu().numpy()
    free.close()
    cfg = cfg_for(n, fphi_max=0.05, **kw)
    p = spff.Problem(Et.repeat(B // distinct, 1, 1).contiguous(), cfg)
    _, stats = p.load_step(eps)
    f = p.get_fields(spff.FIELD_PHI | spff.FIELD_EPS_STAR)
    got = f["eps_star"].cpu().numpy()
    for b in range(B):
        g = stats[b]["gamma"]
        assert 0.0 < g < 1.0 and stats[b]["ne_flag"] == 1
        assert stats[b]["eps_bar"][1] == g * eps[1]
        assert np.array_equal(got[b], np.float32(g) * before[b % distinct]), b
    for b in range(distinct):
        q = spff.Problem(Et[b], cfg)
        _, alone = q.load_step(eps)
        one = q.get_fields(spff.FIELD_PHI | spff.FIELD_EPS_STAR)
        for i in range(b, B, distinct):
            assert stats[i]["gamma"] == alone[0]["gamma"]
            assert all(torch.equal(f[k][i], one[k][0]) for k in f), i
        q.close()
    p.close()


def test_wall_time_is_that_of_each_problem():
    """A step's wall_ms is the time of that problem's step: of two problems
    in one batch, a homogeneous one that takes a few ticks reports less than
    half of what one that takes many times as many does, also where the two
    are queued."""
    import torch
    n = 64
    E = np.stack([np.ones((n, n), dtype=np.float32), si.young_modulus(n, 3.0, 0.3, 5)])
    ramp = si.uniaxial_ramp(12, 0.2, 2.0)[3:6]
    p = spff.Problem(torch.from_numpy(E).to(device()), cfg_for(n, tol=1e-6))
    for k, rows in enumerate((p.load_step(ramp[0])[1], [r[0] for r in p.run_sequence(ramp[1:])[1]])):
        quick, slow = rows
        assert 4 * quick["ticks"] <= slow["ticks"], k
        assert 0.0 < quick["wall_ms"] < 0.5 * slow["wall_ms"] < 1e3, k
    p.close()


def test_fp64_values_beyond_1e300_are_refused():
    """Finite FP64 inputs beyond 1e300 are refused like non-finite ones, by
    every entry point that takes a field, and a refused state leaves the old
    one; 1e300 itself and any finite FP32 value are accepted as states."""
    import torch
    n = 16
    E = torch.ones((n, n), dtype=torch.float64, device=device())
    big = E.clone()
    big[3, 5] = 2e300
    with pytest.raises(spff.SpffError) as e:
        spff.Problem(big, cfg_for(n, precision="fp64"))
    assert e.value.status == spff.E_INVALID
    sv = spff.Server(64 << 20)
    with pytest.raises(spff.SpffError) as e:
        sv.register(cfg_for(n, precision="fp64"), big)
    assert e.value.status == spff.E_INVALID
    sv.close()
    p = spff.Problem(E, cfg_for(n, precision="fp64"))
    st = torch.full_like(p.get_state()[0], 0.5)
    p.set_state(st)
    for v in (2e300, -2e300, float("inf"), float("nan")):
        other = torch.zeros_like(st)
        other[0, 1, 2, 3] = v
        with pytest.raises(spff.SpffError) as e:
            p.set_state(other)
        assert e.value.status == spff.E_INVALID and torch.equal(p.get_state()[0], st)
    other[0, 1, 2, 3] = -1e300
    p.set_state(other)
    assert torch.equal(p.get_state()[0], other)
    p.close()
    q = spff.Problem(E.float(), cfg_for(n))
    st = torch.zeros_like(q.get_state()[0])
    st[0, 0, 0, 0] = 3e38
    q.set_state(st)
    assert torch.equal(q.get_state()[0], st)
    q.close()


def test_autotuner_keeps_the_faster_built_in_fp64_geometry():
    """FP64 plans name LDS kernels, the built-in geometry takes register
    kernels, which are a quarter faster at 512 x 512: the tuner returns the
    plan that stands for it."""
    from paper_2203_16467_amd import autotune
    plan, t = autotune.tune_bucket(512, 512, 1, precision=spff.FP64)
    import torch
    E = torch.ones((512, 512), dtype=torch.float64, device=device())
    p = spff.Problem(E, cfg_for(512, precision="fp64"))
    assert plan == p.get_plan(0), (plan, t)
    assert t["row_us_per_tick"] > 0 and t["col_us_per_tick"] > 0
    p.close()


@pytest.mark.parametrize("nx,ny,precision", [(64, 64, "fp32"), (256, 128, "fp32"), (512, 512, "fp32"),
                                             (64, 64, "fp64"), (256, 512, "fp64")])
@pytest.mark.parametrize("split,nyquist", [("none", spff.NYQ_ZERO), ("spectral", spff.NYQ_FREE)])
def test_mechanics_residual_is_the_norm_of_the_projected_stress(nx, ny, precision, split, nyquist):
    """mech_residual, a sum over Fourier modes, is the norm of the field
    G[sigma] of the returned stress (an elastic step: phi stays 0), and lies
    within the tolerance, in FP32 within 0.97 of it.  Rounding of the stress
    adds u ||sigma|| to a residual of 1e-3 ||sigma|| at most; 8 of that are
    allowed."""
    import torch
    tol, eps = 1e-3, (0.0, 0.1, 0.03)
    E = torch.from_numpy(si.young_modulus(nx, 4.0, 0.25, 3, ny=ny)).to(device())
    if precision == "fp64":
        E = E.double()
    cfg = cfg_for(nx, ny, precision, split=split, nyquist=nyquist, tol=tol)
    p = spff.Problem(E, cfg)
    _, s = p.load_step(eps)
    f = p.get_fields(spff.FIELD_STRESS | spff.FIELD_PHI)
    assert float(f["phi"].max()) == 0.0 and s[0]["cg_iters"] > 0
    g = p.apply_operator(spff.OP_PROJECT, f["stress"])[0].double().cpu().numpy()
    sg = f["stress"][0].double().cpu().numpy()

    def norm(a):
        return float(np.sqrt((a[0] ** 2 + a[1] ** 2 + 2 * a[2] ** 2).sum()))

    u = 2.0 ** -24 if precision == "fp32" else 2.0 ** -53
    assert abs(norm(g) - s[0]["mech_residual"]) <= 8 * u * norm(sg)
    lam, mu = cfg.nu / ((1 + cfg.nu) * (1 - 2 * cfg.nu)), 1 / (2 * (1 + cfg.nu))
    Ef = E.double().cpu().numpy()
    hom = norm(np.stack([lam * eps[1] * Ef, (lam + 2 * mu) * eps[1] * Ef, 2 * mu * eps[2] * Ef]))
    assert 0.0 < s[0]["mech_residual"] <= (0.97 if precision == "fp32" else 1.0) * tol * hom * (1 + 1e-6)
    p.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_spectral_tangent_at_its_corners(precision):
    """One CG iteration from eps* = 0 at a uniform strain with equal,
    vanishing, opposite or barely different eigenvalues and h(phi) < 1 takes
    eps* to alpha p, p = -G[sigma], alpha = p.p / p.C p: the oracle's with
    its tangent.  p carries the rounding of two transforms and of the stress
    (16 u of its norm), alpha that of p twice and of the products (32 u over
    the smallest h, 1/100); the two together are below 1e4 u."""
    import torch
    n, nu = 16, 0.2
    dt = torch.float64 if precision == "fp64" else torch.float32
    corners = [(1, 1, 0), (-1, -1, 0), (1, -1, 0), (1, 0, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1 + 1e-6, 0),
               (1e-6, -1, 0), (1, -1e-6, 1e-6), (2, 0.5, 0.7), (-2, -0.5, -0.7), (1, 0.2, 1), (-1, 0.3, 0.1)]
    phi = torch.from_numpy(np.random.default_rng(4).uniform(0.0, 0.9, (n, n))).to(dt)
    state = torch.zeros((1, 5, n, n), dtype=dt, device=device())
    state[0, 3] = state[0, 4] = phi.to(device())
    cfg = cfg_for(n, precision=precision, split="spectral", max_newton=1, max_cg=1, max_am=1, max_bccg=1, nu=nu)
    E = si.young_modulus(n, 3.0, 0.2, 6)
    p = spff.Problem(torch.from_numpy(E).to(device(), dt), cfg)
    lam, mu = oracle.constitutive.lame(E, nu)
    ph = phi.double().numpy()
    u = 2.0 ** -24 if precision == "fp32" else 2.0 ** -53
    for c in corners:
        e = 1e-2 * np.array(c, dtype=np.float64)
        p.set_state(state, np.zeros(3))
        _, s = p.load_step(e)
        assert s[0]["cg_iters"] == 1, c
        eps = oracle.constitutive.sym_tensor(*[np.full((n, n), v) for v in e])
        r = -osp.project(oracle.constitutive.stress(eps, ph, lam, mu, "spectral"))
        cp = oracle.constitutive.tangent_action(eps, r, ph, lam, mu, "spectral")
        want = tensor_to_planes((r * r).sum() / (r * cp).sum() * r)
        got = p.get_fields(spff.FIELD_EPS_STAR)["eps_star"][0].double().cpu().numpy()
        assert rel_l2(got, want) < 1e4 * u, (c, rel_l2(got, want) / u)
    p.close()


@pytest.mark.parametrize("nx,ny,B", [(256, 128, 1), (512, 256, 1), (1024, 512, 1), (64, 1024, 1), (128, 2048, 1),
                                     (256, 256, 9), (256, 256, 20), (512, 512, 5), (512, 512, 8), (256, 256, 32),
                                     (128, 128, 128), (256, 1024, 5), (256, 2048, 5)])
def test_fp64_solver_register_against_lds_kernels(nx, ny, B):
    """FP64 load steps (AT2, strain-spectral split: CG and BCCG) with the
    built-in kernels -- register rows of four and eight points per lane,
    register columns with and without loads ahead -- and with an LDS plan
    take the same iterations to the same state.  The iterations are capped,
    so the two differ by the rounding of some 60 of them only: 1e-9 of a
    state is 1e7 roundings."""
    import torch
    print(f"fp64 steps {B} x {nx}x{ny}", flush=True)
    distinct = min(B, 2)
    E = torch.from_numpy(np.stack([si.young_modulus(nx, 4.0, 0.2, 70 + b, ny=ny) for b in range(distinct)]))
    E = E.double().to(device()).repeat((B + distinct - 1) // distinct, 1, 1)[:B].contiguous()
    cfg = cfg_for(nx, ny, "fp64", at=2, max_am=2, max_newton=2, max_cg=8, max_bccg=12, use_graph=1, ticks_per_sync=16)
    p = spff.Problem(E, cfg)
    eps = si.uniaxial_ramp(12, 0.2, 2.0)[5]
    start, eb = p.get_state()
    got = []
    for plan in (None, dict(row_kind=spff.FFT_LDS, rows=1, row_threads=128, col_kind=spff.FFT_LDS, cols=1,
                            col_threads=256)):
        for b in range(len(p.plan_buckets())):
            p.set_plan(b, plan)
        p.set_state(start, eb)
        _, s = p.load_step(eps)
        got.append((p.get_state()[0].cpu().numpy(), s))
    for b in range(B):
        for k in ("am_iters", "newton_iters", "cg_iters", "bccg_iters", "ticks"):
            assert got[0][1][b][k] == got[1][1][b][k], (b, k)
        assert got[0][1][b]["bccg_iters"] > 0 and got[0][1][b]["cg_iters"] > 0
        assert rel_l2(got[0][0][b, :3], got[1][0][b, :3]) < 1e-9
        assert rel_l2(got[0][0][b, 3], got[1][0][b, 3]) < 1e-9
        assert abs(got[0][1][b]["F_e"] - got[1][1][b]["F_e"]) <= 1e-9 * got[1][1][b]["F_e"]
    p.close()


@pytest.mark.parametrize("nx,ny,B", [(512, 512, 10), (256, 1024, 10), (256, 2048, 6)])
def test_column_loads_ahead_leave_the_results_of_long_columns(nx, ny, B):
    """As above for columns of 512 to 2048 points: with the plan fixed the
    batch, above 2048 column wavefronts, and the problem alone, below, agree
    bit for bit."""
    import torch
    kw = dict(plan_rows=4, plan_cols=1, max_am=2, max_cg=12, max_bccg=6, at=2)
    Et = torch.from_numpy(np.stack([si.young_modulus(nx, 4.0, 0.15 + 0.05 * b, 30 + b, ny=ny) for b in range(2)]))
    Et = Et.to(device())
    eps = si.uniaxial_ramp(12, 0.2, 2.0)[5]
    p = spff.Problem(Et.repeat(B // 2, 1, 1).contiguous(), cfg_for(nx, ny, **kw))
    _, stats = p.load_step(eps)
    f = p.get_fields(spff.FIELD_PHI | spff.FIELD_EPS_STAR)
    for b in range(2):
        q = spff.Problem(Et[b], cfg_for(nx, ny, **kw))
        _, alone = q.load_step(eps)
        g = q.get_fields(spff.FIELD_PHI | spff.FIELD_EPS_STAR)
        for k in f:
            assert torch.equal(f[k][b], g[k][0]) and torch.equal(f[k][B - 2 + b], g[k][0]), k
        assert stats[b]["cg_iters"] == alone[0]["cg_iters"] > 0 and stats[b]["bccg_iters"] > 0
        q.close()
    p.close()

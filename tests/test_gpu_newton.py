"""GPU: trust-region Newton step and block coordinate ascent through the C ABI, against the
oracle; batched equals one-source-at-a-time; graph replay equals eager launches."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import elbo as E  # noqa: E402
from oracle import newton as NW  # noqa: E402
from paper_1803_00113_amd import _ffi, api  # noqa: E402
from synth import gen  # noqa: E402


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def tiny():
    return gen.crop_patches(gen.subset(gen.config2(n_sources=6), images=[0, 2, 7]), 22)


def one_step(prob, mask, **opts):
    ctx = api.Context(0, **opts)
    plan = api.Plan(ctx, prob)
    th = torch.as_tensor(prob.theta0, device="cuda").contiguous()
    r = torch.ones(prob.n_sources, dtype=torch.float64, device="cuda")
    st, loc = api.newton_step(plan, th, r, mask)
    torch.cuda.synchronize()
    return th.cpu().numpy(), r.cpu().numpy(), st.cpu().numpy(), loc.cpu().numpy(), plan


def check_step(m, theta0, s, th_gpu, r_gpu, st_gpu, loc_gpu, fp64, fd=False, radius=1.0):
    """One Newton step against the oracle's (Section 4.3).  Along flat directions of the
    Hessian small differences in it move the step without changing its value, so an
    accepted step is judged by the oracle's own local model at the iterate: the GPU's step
    p lies in the trust region and its predicted gain g.p + p.Hp/2 (oracle g and H) equals
    the oracle's optimum within the tolerance; plus a loose element-wise bound, identical
    status and radius, and L_s at the returned point."""
    info = {}
    o_th, o_r, o_st, o_loc = NW.newton_step_source(m, theta0, s, radius, info=info)
    assert st_gpu == o_st
    if fd:
        # FD Hessian (h = 1e-3, float64 gradients): truncation ~h^2 -> 2e-5 of the gain;
        # float32 gradients (h = 1e-2): rounding noise / h + h^2 -> 1e-2 of the gain
        tol_gain, tol_el, tol_r = (2e-5, 1e-3, 1e-3) if fp64 else (1e-2, 5e-2, 5e-2)
    else:
        # exact Hessian: float64 differs from the oracle by summation order only; float32
        # per-pixel terms carry ~1e-5 relative error into the Hessian
        tol_gain, tol_el, tol_r = (1e-10, 1e-8, 1e-8) if fp64 else (1e-5, 1e-4, 1e-4)
    step = np.abs(o_th - theta0[s]).max()
    msg = (f"  s={s} status {st_gpu}/{o_st} |dtheta|max {np.abs(th_gpu - o_th).max():.2e} (step {step:.2e}) "
           f"radius {r_gpu}/{o_r}")
    if o_st == _ffi.ST_ACCEPTED:
        g, H, pred = info["g"], info["H"], info["pred"]
        p = th_gpu[:27] - theta0[s, :27]
        mg = float(g @ p + 0.5 * p @ H @ p)
        msg += f" model gain gpu {mg:.6e} oracle {pred:.6e}"
        assert np.linalg.norm(p) <= radius * (1 + 1e-6)
        assert abs(mg - pred) <= tol_gain * abs(pred) + 1e-12 * abs(info["L"])
    else:
        assert np.array_equal(th_gpu, theta0[s])
    say(msg)
    assert np.abs(th_gpu - o_th).max() <= tol_el * max(1.0, step)
    assert abs(r_gpu - o_r) <= tol_r * max(1.0, o_r)
    assert abs(loc_gpu - o_loc) <= 1e-5 * abs(o_loc)


@pytest.mark.parametrize("fp64,fd", [(True, False), (False, False), (True, True), (False, True)])
def test_newton_step_config1(fp64, fd):
    say(f"case: newton step config1 fp64={fp64} fd={fd}")
    prob = gen.config1()
    m = E.Model(prob)
    with pytest.raises(_ffi.CelError):          # the two sources overlap
        one_step(prob, None)
    for s in range(2):
        mask = np.zeros(2, bool)
        mask[s] = True
        th, r, st, loc, _ = one_step(prob, mask, hessian_fp64=fp64, hessian_fd=fd)
        assert st[1 - s] == _ffi.ST_SKIPPED and np.isnan(loc[1 - s])
        assert np.array_equal(th[1 - s], prob.theta0[1 - s])
        check_step(m, prob.theta0, s, th[s], r[s], st[s], loc[s], fp64, fd)


def test_newton_step_class_batched_equals_single():
    say("case: newton class batched vs single")
    prob = tiny()
    ctx = api.Context(0)
    plan = api.Plan(ctx, prob)
    mask = plan.colours == 0
    th = torch.as_tensor(prob.theta0, device="cuda").contiguous()
    r = torch.ones(prob.n_sources, dtype=torch.float64, device="cuda")
    st, loc = api.newton_step(plan, th, r, mask)
    th2 = torch.as_tensor(prob.theta0, device="cuda").contiguous()
    r2 = torch.ones(prob.n_sources, dtype=torch.float64, device="cuda")
    for s in np.nonzero(mask)[0]:
        one = np.zeros(prob.n_sources, bool)
        one[s] = True
        st1, loc1 = api.newton_step(plan, th2, r2, one)
        assert st1[s].item() == st[s].item() and loc1[s].item() == loc[s].item()
    torch.cuda.synchronize()
    assert torch.equal(th, th2) and torch.equal(r, r2)
    # against the oracle for every stepped source
    m = E.Model(prob)
    thn, rn, stn, locn = th.cpu().numpy(), r.cpu().numpy(), st.cpu().numpy(), loc.cpu().numpy()
    for s in np.nonzero(mask)[0]:
        check_step(m, prob.theta0, int(s), thn[s], rn[s], stn[s], locn[s], False)


def test_sweep_graph_equals_eager_and_matches_oracle():
    say("case: sweep graph vs eager vs oracle")
    prob = gen.crop_patches(gen.subset(gen.config2(n_sources=4), sources=[0, 1, 2], images=[1, 6]), 14)
    ctx = api.Context(0)
    plan = api.Plan(ctx, prob)
    res = []
    for use_graph in (True, False, True):
        th = torch.as_tensor(prob.theta0, device="cuda").contiguous()
        r, st, rep = api.sweep(plan, th, n_sweeps=2, max_newton_iters=20, use_graph=use_graph)
        torch.cuda.synchronize()
        res.append((th.cpu().numpy(), r.cpu().numpy(), st.cpu().numpy(), rep))
        say(f"  graph={use_graph}: elbo {rep['elbo']:.6f}, steps {rep['n_newton_steps']}, {rep['seconds']:.3f} s")
    for k in (1, 2):
        assert np.array_equal(res[0][0], res[k][0]) and np.array_equal(res[0][2], res[k][2])
        assert res[0][3]["elbo"] == res[k][3]["elbo"]
    m = E.Model(prob)
    o_th, _, o_st, o_rep = NW.sweep(m, prob.theta0, dict(n_sweeps=2, max_iter=20))
    th = res[0][0]
    say(f"  oracle elbo {o_rep['elbo']:.6f}; max |dtheta| {np.abs(th - o_th).max():.2e}")
    start = E.elbo(m, prob.theta0)[0].item()
    assert res[0][3]["elbo"] > start
    assert abs(res[0][3]["elbo"] - o_rep["elbo"]) <= 1e-5 * abs(o_rep["elbo"])
    assert np.array_equal(res[0][2], o_st)


def test_sweep_checkpoint_resume_identical(tmp_path):
    """Checkpoint / resume: a sweep stopped after a few colour classes, its state saved to
    disk and reloaded, then resumed at the cursor, ends bitwise where one uninterrupted
    sweep ends."""
    say("case: sweep checkpoint / resume")
    prob = gen.crop_patches(gen.subset(gen.config2(n_sources=20), images=[0, 5]), 20)
    ctx = api.Context(0)
    plan = api.Plan(ctx, prob)
    assert plan.n_colours >= 2
    th_a = torch.as_tensor(prob.theta0, device="cuda").contiguous()
    r_a, st_a, rep_a = api.sweep(plan, th_a, n_sweeps=2, max_newton_iters=20)
    th_b = torch.as_tensor(prob.theta0, device="cuda").contiguous()
    k = plan.n_colours + 1          # stop inside the second pass
    r_b, st_b, rep_b = api.sweep(plan, th_b, n_sweeps=2, max_newton_iters=20, max_classes=k)
    say(f"  stopped after {k} classes: {rep_b}")
    assert rep_b["sweeps_done"] == 1 and rep_b["next_colour"] == 1
    path = tmp_path / "state.npz"
    api.save_state(path, th_b, r_b, st_b, rep_b)
    th_c, r_c, st_c, cur = api.load_state(path, "cuda")
    assert torch.equal(th_c, th_b) and torch.equal(r_c, r_b) and torch.equal(st_c, st_b)
    _, _, rep_c = api.sweep(plan, th_c, n_sweeps=2 - cur["sweeps_done"], max_newton_iters=20,
                            radius=r_c, status=st_c, start_colour=cur["next_colour"])
    torch.cuda.synchronize()
    assert torch.equal(th_c, th_a) and torch.equal(r_c, r_a) and torch.equal(st_c, st_a)
    assert rep_c["elbo"] == rep_a["elbo"] and rep_c["next_colour"] == 0
    assert rep_b["n_newton_steps"] + rep_c["n_newton_steps"] == rep_a["n_newton_steps"]


@pytest.mark.parametrize("logit", [None, -800.0])
@pytest.mark.parametrize("radius", [1e-4, 0.05, 1.0, 20.0])
def test_step_solves_its_subproblem(radius, logit):
    """Steps inside the region, on its boundary, with an indefinite Hessian, and (type weight
    exactly 0: a row of the Hessian and its gradient vanish) the hard case: the step's model
    value is the oracle's optimum for the same gradient and Hessian (float64: 1e-10 of the
    gain, and the gradient times the rounding with which theta holds the step), and it lies in
    the region; a rejected step shrinks the radius to |p| / 4."""
    say(f"case: trust-region subproblem, radius {radius}, type logit {logit}")
    prob = tiny()
    ctx = api.Context(0, pixel_fp64=True, hessian_fp64=True)
    plan = api.Plan(ctx, prob)
    th0 = prob.theta0.copy()
    if logit is not None:
        th0[:, 2] = logit
    H, g, _ = (t.cpu().numpy() for t in api.elbo_hessian(plan, th0))
    th = torch.as_tensor(th0, device="cuda").contiguous()
    r = torch.full((prob.n_sources,), radius, dtype=torch.float64, device="cuda")
    st, _ = api.newton_step(plan, th, r, plan.colours == 0)
    thn, rn, stn = th.cpu().numpy(), r.cpu().numpy(), st.cpu().numpy()
    for s in np.nonzero(plan.colours == 0)[0]:
        po, lam, hard = NW.tr_subproblem(g[s, :27], H[s], radius)
        value = lambda p: float(g[s, :27] @ p + 0.5 * p @ H[s] @ p)
        p = thn[s, :27] - th0[s, :27]
        say(f"  s={s} status {stn[s]} lam {lam:.3g} hard {hard} |p| {np.linalg.norm(p):.6g} gain {value(p):.6g}")
        if stn[s] == _ffi.ST_ACCEPTED:
            assert np.linalg.norm(p) <= radius * (1 + 1e-9)
            held = 2.0 ** -53 * float(np.abs(g[s, :27]) @ np.abs(th0[s, :27]))
            assert abs(value(p) - value(po)) <= 1e-10 * abs(value(po)) + held
        else:
            assert stn[s] == _ffi.ST_REJECTED and np.all(p == 0)
            assert abs(rn[s] - 0.25 * np.linalg.norm(po)) <= 1e-8 * np.linalg.norm(po)


@pytest.mark.parametrize("radius", [0.5, 2.0])
def test_step_hard_case(radius):
    """A type weight of exactly 0 at the other type's optimum, but for the flux: -H is singular
    along the type logit and the unused type's coordinates with no gradient there, so the step
    is completed to the boundary among them."""
    say(f"case: trust-region hard case, radius {radius}")
    prob = tiny()
    ctx = api.Context(0, pixel_fp64=True, hessian_fp64=True)
    plan = api.Plan(ctx, prob)
    th0 = prob.theta0.copy()
    th0[:, 2] = -800.0
    th0 = torch.as_tensor(th0, device="cuda").contiguous()
    api.sweep(plan, th0, n_sweeps=2, max_newton_iters=50)
    th0 = th0.cpu().numpy()
    th0[:, 3] += 1e-2
    H, g, _ = (t.cpu().numpy() for t in api.elbo_hessian(plan, th0))
    th = torch.as_tensor(th0, device="cuda").contiguous()
    r = torch.full((prob.n_sources,), radius, dtype=torch.float64, device="cuda")
    st, _ = api.newton_step(plan, th, r, plan.colours == 0)
    thn, stn = th.cpu().numpy(), st.cpu().numpy()
    for s in np.nonzero(plan.colours == 0)[0]:
        po, lam, hard = NW.tr_subproblem(g[s, :27], H[s], radius)
        value = lambda p: float(g[s, :27] @ p + 0.5 * p @ H[s] @ p)
        p = thn[s, :27] - th0[s, :27]
        say(f"  s={s} status {stn[s]} lam {lam:.3g} hard {hard} |p| {np.linalg.norm(p):.6g} gain {value(p):.6g}")
        if stn[s] == _ffi.ST_ACCEPTED:
            held = 2.0 ** -53 * float(np.abs(g[s, :27]) @ np.abs(th0[s, :27]))
            assert np.linalg.norm(p) <= radius * (1 + 1e-9)
            assert abs(value(p) - value(po)) <= 1e-10 * abs(value(po)) + held


@pytest.mark.parametrize("fp64", [False, True])
def test_step_local_objective_is_the_evaluations(fp64):
    """elbo_local of an accepted source is L_s at the returned theta, the same number as
    elbo_eval gives there (bit for bit: no source it overlaps has moved)."""
    say(f"case: elbo_local of a step against elbo_eval, fp64={fp64}")
    for prob in (tiny(), gen.crop_patches(gen.subset(gen.config2(n_sources=20), images=[0, 5]), 20)):
        plan = api.Plan(api.Context(0, pixel_fp64=fp64), prob)
        for radius in (0.05, 1.0):
            th = torch.as_tensor(prob.theta0, device="cuda").contiguous().clone()
            r = torch.full((prob.n_sources,), radius, dtype=torch.float64, device="cuda")
            st, loc = api.newton_step(plan, th, r, plan.colours == 0)
            at = api.elbo_eval(plan, th)[1]
            moved = st == _ffi.ST_ACCEPTED
            say(f"  S={prob.n_sources} radius {radius}: accepted {int(moved.sum())}, "
                f"largest difference {float((loc - at)[moved].abs().max()):.3e}")
            assert int(moved.sum()) > 0 and torch.equal(loc[moved], at[moved])


@pytest.mark.parametrize("radius", [0.5, 2.0])
def test_step_hard_case_is_reached(radius):
    """The state of test_step_hard_case is the hard case for at least one source, and its step
    is taken: completed to the boundary, of the oracle's model value; a source whose step is
    not taken keeps its parameters and gets a quarter of the step's length as its radius."""
    say(f"case: trust-region hard case reached, radius {radius}")
    prob = tiny()
    plan = api.Plan(api.Context(0, pixel_fp64=True, hessian_fp64=True), prob)
    th0 = prob.theta0.copy()
    th0[:, 2] = -800.0
    th0 = torch.as_tensor(th0, device="cuda").contiguous()
    api.sweep(plan, th0, n_sweeps=2, max_newton_iters=50)
    th0 = th0.cpu().numpy()
    th0[:, 3] += 1e-2
    H, g, _ = (t.cpu().numpy() for t in api.elbo_hessian(plan, th0))
    th = torch.as_tensor(th0, device="cuda").contiguous()
    r = torch.full((prob.n_sources,), radius, dtype=torch.float64, device="cuda")
    st, _ = api.newton_step(plan, th, r, plan.colours == 0)
    thn, rn, stn = th.cpu().numpy(), r.cpu().numpy(), st.cpu().numpy()
    taken = 0
    for s in np.nonzero(plan.colours == 0)[0]:
        po, _, hard = NW.tr_subproblem(g[s, :27], H[s], radius)
        value = lambda p: float(g[s, :27] @ p + 0.5 * p @ H[s] @ p)
        p = thn[s, :27] - th0[s, :27]
        if stn[s] == _ffi.ST_ACCEPTED:
            held = 2.0 ** -53 * float(np.abs(g[s, :27]) @ np.abs(th0[s, :27]))
            # (theta holds a coordinate of size 800 to 1e-13)
            assert not hard or abs(np.linalg.norm(p) - radius) <= 1e-9 * radius + 1e-12
            assert abs(value(p) - value(po)) <= 1e-10 * abs(value(po)) + held
            taken += hard
        else:
            assert stn[s] == _ffi.ST_REJECTED and np.all(p == 0)
            assert abs(rn[s] - 0.25 * np.linalg.norm(po)) <= 1e-8 * np.linalg.norm(po)
    assert taken > 0

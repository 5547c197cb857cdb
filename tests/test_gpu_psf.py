"""GPU: the spatially varying PSF (Section 2.2.2, Table 1: eigen-images with smoothly
varying loadings; Section 2.2.3: a Gaussian-mixture PSF) through the C ABI.

  cel_psf_fit against the oracle's fit (float64 on both sides; differences only from the
  order of summation): every mixture parameter within 1e-9 of its scale, for 1-4
  components, 0, 1 and 30 iterations, positions at the frame's corners and inside it;
  an out-of-range image index gives NaN rows and CEL_DEVERR_BAD_INDEX.
  The objective with per-patch PSFs (each side using its own fits) and a 24 x 32 sky knot
  grid: ELBO and gradient with float32 and float64 pixels, Hessians and a Newton step."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import elbo as E  # noqa: E402
from oracle import psf as OP  # noqa: E402
from paper_1803_00113_amd import _ffi, api  # noqa: E402
from synth import gen  # noqa: E402
from tests.test_gpu_hessian import check_source  # noqa: E402
from tests.test_gpu_newton import check_step  # noqa: E402
from tests.test_gpu_parity import check  # noqa: E402


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def small():
    return gen.config_eigen_small()


def _positions(prob, rng, n_random=6):
    pts = []
    for n in range(prob.n_images):
        W, H = float(prob.img_W[n]), float(prob.img_H[n])
        for x, y in [(0.0, 0.0), (W - 1, H - 1), (0.0, H - 1), ((W - 1) / 2, (H - 1) / 2)]:
            pts.append((n, x, y))
        for _ in range(n_random):
            pts.append((n, rng.uniform(0, W - 1), rng.uniform(0, H - 1)))
    return pts


def _scale_err(got, want):
    return np.abs(got - want) / np.maximum(1.0, np.abs(want))


@pytest.mark.parametrize("K,n_iter", [(1, 0), (1, 5), (2, 1), (2, 30), (3, 0), (3, 30), (4, 30)])
def test_psf_fit_matches_oracle(small, K, n_iter):
    say(f"case: psf fit K={K} n_iter={n_iter}")
    prob = small
    ctx = api.Context(0)
    pts = _positions(prob, np.random.default_rng(K * 100 + n_iter))
    fit_img = np.array([p[0] for p in pts], np.int32)
    fit_xy = np.array([[p[1], p[2]] for p in pts])
    size = np.stack([prob.img_W, prob.img_H], 1).astype(float)
    out = api.psf_fit_at(ctx, prob.psf_eigen, prob.psf_coef, size, fit_img, fit_xy, K, n_iter).cpu().numpy()
    worst = 0.0
    for f, (n, x, y) in enumerate(pts):
        img = OP.psf_image(prob.psf_eigen[n], prob.psf_coef[n], size[n, 0], size[n, 1], x, y)
        want = OP.fit_mixture(img, K, n_iter)
        err = _scale_err(out[f, :K], want).max()
        worst = max(worst, err)
        assert err <= 1e-9, (f, n, x, y, out[f, :K], want)
        assert np.all(out[f, K:] == 0)
    say(f"  {len(pts)} fits, max scaled error {worst:.2e}")


def test_psf_fit_bad_index_and_empty(small):
    say("case: psf fit bad index, no fits")
    prob = small
    ctx = api.Context(0)
    size = np.stack([prob.img_W, prob.img_H], 1).astype(float)
    api.last_device_error(ctx)
    out = api.psf_fit_at(ctx, prob.psf_eigen, prob.psf_coef, size, np.array([0, prob.n_images, 1], np.int32),
                         np.array([[5.0, 5.0], [5.0, 5.0], [7.0, 9.0]]), 3, 10).cpu().numpy()
    assert np.all(np.isnan(out[1])) and np.all(np.isfinite(out[0])) and np.all(np.isfinite(out[2]))
    assert api.last_device_error(ctx) & _ffi.DEVERR_BAD_INDEX
    empty = api.psf_fit_at(ctx, prob.psf_eigen, prob.psf_coef, size, np.zeros(0, np.int32), np.zeros((0, 2)), 3, 10)
    assert empty.shape == (0, 4, 6)
    with pytest.raises(_ffi.CelError):
        api.psf_fit_at(ctx, prob.psf_eigen, prob.psf_coef, size, np.array([0], np.int32), np.zeros((1, 2)), 5, 10)


@pytest.fixture(scope="module")
def fitted(small):
    """The problem with each side's own per-patch PSF fits (3 components, 30 iterations):
    the GPU's for the plan, the oracle's for the oracle model."""
    prob = small
    ctx = api.Context(0)
    gpu_psf = api.patch_psf_fits(ctx, prob, 3, 30)
    o_psf = OP.patch_psfs(prob, 3, 30)
    assert _scale_err(gpu_psf, o_psf).max() <= 1e-9
    m = E.Model(prob, patch_psf=o_psf)
    prob.patch_psf = gpu_psf
    return prob, m, E.elbo_total_and_grad(m, prob.theta0)


@pytest.mark.parametrize("fp64", [False, True])
def test_objective_with_per_patch_psf(fitted, fp64):
    say(f"case: objective with per-patch PSFs and a 24 x 32 sky grid, fp64={fp64}")
    prob, _, (o_tot, o_loc, o_g) = fitted
    ctx = api.Context(0, pixel_fp64=fp64)
    plan = api.Plan(ctx, prob)
    tot, loc, g = api.elbo_grad(plan, prob.theta0)
    tot, loc, g = tot.item(), loc.cpu().numpy(), g.cpu().numpy()
    rt = (1e-10, 1e-8) if fp64 else (1e-5, 1e-4)
    err = check(prob, tot, loc, g, o_tot, o_loc, o_g, rtol_e=rt[0], rtol_g=rt[1])
    say(f"  total {tot:.8f} oracle {o_tot:.8f}; max grad rel err {err:.2e}")
    # the per-patch PSFs matter: the image-wide PSFs give a different objective
    plain = gen.subset(prob)
    plain.patch_psf = None
    tot2 = api.elbo_eval(api.Plan(ctx, plain), prob.theta0)[0].item()
    say(f"  with the image-wide PSFs instead: total {tot2:.8f}")
    assert abs(tot2 - tot) > 1e-6 * abs(tot)


@pytest.mark.parametrize("fp64", [True, False])
def test_hessian_and_newton_step_with_per_patch_psf(fitted, fp64):
    say(f"case: hessian and newton step with per-patch PSFs, fp64={fp64}")
    prob, m, _ = fitted
    ctx = api.Context(0, hessian_fp64=fp64)
    plan = api.Plan(ctx, prob)
    th = torch.as_tensor(prob.theta0, device="cuda").contiguous()
    mask = plan.colours == 0
    h, g, loc = api.elbo_hessian(plan, th, mask)
    h, g, loc = h.cpu().numpy(), g.cpu().numpy(), loc.cpu().numpy()
    for s in np.nonzero(mask)[0][:4]:
        check_source(m, prob.theta0, int(s), h[s], g[s], loc[s], fp64)
    r = torch.ones(prob.n_sources, dtype=torch.float64, device="cuda")
    st, loc = api.newton_step(plan, th, r, mask)
    thn, rn, stn, locn = th.cpu().numpy(), r.cpu().numpy(), st.cpu().numpy(), loc.cpu().numpy()
    for s in np.nonzero(mask)[0][:4]:
        check_step(m, prob.theta0, int(s), thn[s], rn[s], stn[s], locn[s], fp64)


@pytest.mark.parametrize("side", [3, 5, 15, 17, 31, 33, 61, 63])
@pytest.mark.parametrize("K", [1, 4])
def test_psf_fit_grid_sizes(side, K):
    """Grids whose columns fill the workgroup's row strips exactly, with idle threads, with
    fewer rows than strips and with a partial last row pass (float64 on both sides: 1e-9)."""
    say(f"case: psf fit side={side} K={K}")
    rng = np.random.default_rng(side * 10 + K)
    ax = np.arange(side) - 0.5 * (side - 1)
    r2 = ax[:, None] ** 2 + ax[None, :] ** 2
    s = 0.12 * side + 0.4
    base = np.exp(-0.5 * r2 / s ** 2) + 0.3 * np.exp(-0.5 * r2 / (2.2 * s) ** 2)
    eig = np.stack([base, base * ax[None, :] / side, base * ax[:, None] / side])[None]
    coef = rng.uniform(-0.2, 0.2, (1, 3, 6))
    coef[0, 0, 0] += 1.0
    size = np.array([[100.0, 80.0]])
    xy = rng.uniform(0, 1, (3, 2)) * size
    out = api.psf_fit_at(api.Context(0), eig, coef, size, np.zeros(3, np.int32), xy, K, 6).cpu().numpy()
    for f in range(3):
        img = OP.psf_image(eig[0], coef[0], size[0, 0], size[0, 1], xy[f, 0], xy[f, 1])
        assert _scale_err(out[f, :K], OP.fit_mixture(img, K, 6)).max() <= 1e-9
        assert np.all(out[f, K:] == 0)


@pytest.mark.parametrize("K,sigma,scale", [(1, 0.655, 1.0), (1, 0.66, 1e6), (1, 0.67, 1e12), (2, 0.565, 1.0),
                                           (2, 0.575, 1e12)])
def test_psf_fit_far_knot_of_tiny_density(K, sigma, scale):
    """A PSF narrower than the knots' spacing with light in one far knot, where the mixture's
    density is near the smallest numbers (1e-320 to 1e-303, below the knot's weight over the
    largest number): the knot's responsibilities are at most 1 and the fit is the oracle's
    (float64 on both sides: 1e-9)."""
    say(f"case: psf fit, far knot, K={K} sigma={sigma} scale={scale:g}")
    side, n_iter = 51, 5
    dx, dy = OP.knot_offsets(side)
    img = np.exp(-0.5 * (dx ** 2 + dy ** 2) / sigma ** 2)
    img[img < 1e-20] = 0.0
    img[side // 2, side - 1] = 1e-7
    img *= scale
    coef = np.zeros((1, 1, 6))
    coef[0, 0, 0] = 1.0
    out = api.psf_fit_at(api.Context(0), img[None, None], coef, np.array([[100.0, 100.0]]), np.zeros(1, np.int32),
                         np.array([[50.0, 50.0]]), K, n_iter).cpu().numpy()
    want = OP.fit_mixture(img, K, n_iter)
    say(f"  {out[0, :K]}")
    assert np.all(np.isfinite(want)) and _scale_err(out[0, :K], want).max() <= 1e-9


@pytest.mark.parametrize("eps", [1e-8, 1e-11, 1e-20, 1e-30])
def test_psf_fit_exponents_beyond_the_integers(eps):
    """A point with the faintest of neighbours: the start's variance is 2 eps, and exponents
    away from the point go to -1e9 .. -1e32, past the 32- and 64-bit integers; their densities
    are 0 and the point keeps its mixture (the oracle's: 1e-9)."""
    say(f"case: psf fit, exponents to {-600 / eps:.0e}")
    side = 51
    img = np.zeros((side, side))
    img[25, 25] = 1.0
    img[25, 24] = img[25, 26] = img[24, 25] = img[26, 25] = eps
    coef = np.zeros((1, 1, 6))
    coef[0, 0, 0] = 1.0
    for n_iter in (0, 1):
        out = api.psf_fit_at(api.Context(0), img[None, None], coef, np.array([[100.0, 100.0]]), np.zeros(1, np.int32),
                             np.array([[50.0, 50.0]]), 2, n_iter).cpu().numpy()
        want = OP.fit_mixture(img, 2, n_iter)
        assert np.all(np.isfinite(want)) and _scale_err(out[0, :2], want).max() <= 1e-9

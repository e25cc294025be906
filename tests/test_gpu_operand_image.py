"""The matrix-core field kernel that reads the operand image (FP32 field variants
2 and 3 for clusters of at least 160 T particles): step, batched and adjoint
modes against the FP64 oracle, on both sides of the rule and with ragged last
waves.  Bars as in the other GPU tests: states and coefficients 1e-5, the
returned accelerations 2e-5 (evaluated after the steps' own FP32 drift),
gradients 1e-3."""
import numpy as np
import pytest

from paper_2602_13385_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = 1e-5
NFW = [("nfw", (232.98, 20.0))]
CEN = np.array([20.0, 0.0, 0.0, 0.1, 1.4, 0.3])
RATIO = 160


@pytest.fixture(scope="module")
def torch():
    import torch as T
    if not T.cuda.is_available():
        pytest.skip("no GPU")
    return T


@pytest.fixture(scope="module")
def S():
    from paper_2602_13385_amd import scf
    scf.lib()
    return scf


def _r(a):
    return np.asarray(a, np.float32).astype(np.float64)


def _dev(torch, a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")


def _rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


def _force_err(g, ref):
    mag = np.sqrt((ref ** 2).sum(0))
    return (np.sqrt(((g - ref) ** 2).sum(0)) / (mag + np.median(mag))).max()


CASES = [  # (nmax, lmax, alpha, particles beyond 160 T)
    (0, 0, 1.0, 0), (3, 1, 1.0, -1), (3, 1, 1.0, 0), (3, 1, 1.0, 37), (5, 2, 0.5, 1),
    (6, 4, 1.0, 63), (10, 5, 0.8, 129),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"n{c[0]}l{c[1]}a{c[2]}{c[3]:+d}")
def test_step_from_the_image_matches_oracle(torch, S, O, case):
    nmax, lmax, alpha, over = case
    n = RATIO * (nmax + 1) * (lmax + 1) ** 2 + over
    print(f"[image step] nmax={nmax} lmax={lmax} alpha={alpha} N={n}", flush=True)
    p = I.plummer(n, 4100 + n % 89)
    st0, m = _r(p.state()), _r(p.mass)
    B = O.basis(nmax, lmax, alpha=alpha)
    Ho = O.host([(O.HOST_NFW, NFW[0][1])])
    ref, cref, aref, accref = O.step(B, Ho, st0, m, CEN, 0.005, 2, want_acc=True)
    for fv in (2, 3):
        plan = S.Plan(nmax, lmax, alpha=alpha)
        plan.field_variant = fv
        st = [_dev(torch, st0[i]) for i in range(6)]
        coef = torch.empty(plan.T, dtype=torch.float64, device="cuda")
        cen, acc = plan.step(st, _dev(torch, m), 0.005, 2, host=(NFW, 1.0), centre=CEN,
                             coef_last=coef)
        torch.cuda.synchronize()
        out = np.stack([t.cpu().numpy() for t in st]).astype(np.float64)
        a = np.stack([t.cpu().numpy() for t in acc]).astype(np.float64)
        assert _rel(out[:3], ref[:3]) <= TOL and _rel(out[3:], ref[3:]) <= TOL
        assert _rel(coef.cpu().numpy(), aref) <= TOL
        assert _force_err(a, accref) <= 2 * TOL, _force_err(a, accref)


def test_batched_step_from_the_image_matches_oracle(torch, S, O):
    """Clusters below and above the rule in one call (it goes by their mean)."""
    nmax, lmax = 4, 2
    sizes = [300, 20_011, 1, 9_600]
    T = (nmax + 1) * (lmax + 1) ** 2
    assert sum(sizes) // len(sizes) >= RATIO * T
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    parts = [I.plummer(max(k, 2), 4200 + i).state()[:, :k] for i, k in enumerate(sizes)]
    st0 = _r(np.concatenate(parts, axis=1))
    m = _r(np.concatenate([np.full(k, 1.0 / k) for k in sizes]))
    cens = np.stack([np.r_[CEN[:3] + i, CEN[3:]] for i in range(len(sizes))])
    B = O.basis(nmax, lmax)
    Ho = O.host([(O.HOST_NFW, NFW[0][1])])
    plan = S.Plan(nmax, lmax)
    plan.field_variant = 3
    st = [_dev(torch, st0[i]) for i in range(6)]
    cen, _ = plan.step_batched(off, st, _dev(torch, m), 0.005, 2, host=(NFW, 1.0), centres=cens)
    torch.cuda.synchronize()
    out = np.stack([t.cpu().numpy() for t in st]).astype(np.float64)
    for c in range(len(sizes)):
        sl = slice(off[c], off[c + 1])
        ref, cref, _ = O.step(B, Ho, st0[:, sl], m[sl], cens[c], 0.005, 2)[:3]
        assert np.allclose(cen[c], cref, rtol=0, atol=1e-12)
        assert _rel(out[:3, sl], ref[:3]) <= TOL and _rel(out[3:, sl], ref[3:]) <= TOL, c


@pytest.mark.parametrize("keep", [False, True])
def test_adjoint_from_the_image_matches_oracle(torch, S, O, keep):
    nmax, lmax, nsteps, dt = 4, 2, 3, 0.005
    n = RATIO * (nmax + 1) * (lmax + 1) ** 2 + 5
    p = I.plummer(n, 4300)
    st0, m = _r(p.state()), _r(p.mass)
    rng = np.random.default_rng(4301)
    lam, lamc = _r(rng.normal(size=(6, n))), rng.normal(size=6)
    B = O.basis(nmax, lmax)
    Ho = O.host([(O.HOST_NFW, NFW[0][1])])
    lref, lcref, ghref = O.step_adjoint(B, Ho, st0, m, CEN, dt, nsteps, lam, lamc)
    plan = S.Plan(nmax, lmax)
    plan.field_variant = 3
    hist = None
    md = _dev(torch, m)
    if keep:  # weights recorded by the forward pass
        hist = torch.empty((nsteps + 1) * plan.weights_size, dtype=torch.float32, device="cuda")
        plan.step([_dev(torch, st0[i]) for i in range(6)], md, dt, nsteps, host=(NFW, 1.0),
                  centre=CEN, w_hist=hist)
    lt = [_dev(torch, lam[i]) for i in range(6)]
    lc, gh = plan.step_adjoint([_dev(torch, st0[i]) for i in range(6)], md, dt, nsteps, lt, lamc,
                               host=(NFW, 1.0), centre0=CEN, w_hist=hist)
    torch.cuda.synchronize()
    lg = np.stack([t.cpu().numpy() for t in lt]).astype(np.float64)
    assert _rel(lg[:3], lref[:3]) <= 1e-3 and _rel(lg[3:], lref[3:]) <= 1e-3
    assert np.abs(lc - lcref).max() <= 1e-3 * np.abs(lcref).max()
    assert np.abs(gh[0, :2] - ghref[0, :2]).max() <= 1e-3 * np.abs(ghref[0, :2]).max()

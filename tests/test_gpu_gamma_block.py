"""The block kernel on dual numbers (the adjoint's gamma pass in single
precision): particle counts around its stages, the smallest and largest bases
(one slab of records, two arrays that fit two blocks per compute unit), and a
count at which a unit folds more than once and writes two rows.  Reference: the
double-precision plan, whose gamma pass is another kernel; bar 1e-3, as for the
other single-precision gradients."""
import numpy as np
import pytest

from paper_2602_13385_amd import inputs as I

pytestmark = pytest.mark.gpu

NFW = [("nfw", (232.98, 20.0))]
CEN = np.array([20.0, 0.0, 0.0, 0.1, 1.4, 0.3])
CASES = [  # (nmax, lmax, alpha, n)
    (0, 0, 1.0, 1), (4, 0, 1.0, 257), (1, 1, 0.5, 63), (6, 4, 1.0, 65), (10, 6, 1.0, 64),
    (10, 6, 0.8, 1003), (12, 8, 0.5, 129), (16, 10, 1.0, 62), (20, 10, 1.0, 127),
    (16, 10, 1.0, 560_003),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"n{c[0]}l{c[1]}a{c[2]}N{c[3]}")
def test_gamma_pass_matches_double_precision(case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_13385_amd import scf as S
    nmax, lmax, alpha, n = case
    print(f"[gamma block] nmax={nmax} lmax={lmax} alpha={alpha} N={n}", flush=True)
    p = I.plummer(max(n, 2), 4400 + n % 97)
    st0 = np.asarray(p.state()[:, :n], np.float32)
    m = np.full(n, 1.0 / n, np.float32)
    rng = np.random.default_rng(4401)
    lam = rng.normal(size=(6, n)).astype(np.float32)
    lamc = rng.normal(size=6)
    out = {}
    for dt in (torch.float32, torch.float64):
        plan = S.Plan(nmax, lmax, alpha=alpha, dtype="f32" if dt == torch.float32 else "f64")
        dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda").to(dt)
        lt = [dev(lam[i]) for i in range(6)]
        lc, gh = plan.step_adjoint([dev(st0[i]) for i in range(6)], dev(m), 0.005, 1, lt, lamc,
                                   host=(NFW, 1.0), centre0=CEN)
        torch.cuda.synchronize()
        out[dt] = (np.stack([t.cpu().numpy() for t in lt]).astype(np.float64), lc)
    (a, ac), (b, bc) = out[torch.float32], out[torch.float64]
    for sl in (slice(0, 3), slice(3, 6)):
        assert np.abs(a[sl] - b[sl]).max() <= 1e-3 * np.abs(b[sl]).max()
    assert np.abs(ac - bc).max() <= 1e-3 * np.abs(bc).max()

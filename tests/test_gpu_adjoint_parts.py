"""The two self-gravity parts of the reverse step, each by itself.

Half of the particles (A) have no mass and a cotangent lambda_v; the other half
(B) have mass and lambda_v = 0; lambda_x = 0 and there is no host.  Then
lambda_x of A is the Hessian-vector part alone (its own mass, which scales the
coefficient part, is zero), and lambda_x of B is the coefficient part alone (the
gamma pass over A, then the accumulation of its field: B's own Hessian-vector
part has lambda_v = dt lambda_x of the kick before, a factor dt smaller).
lambda_v of A is a smooth vector field of many waves, so that the gamma sums of
every degree add up instead of averaging out.

Single precision (the block kernel on dual numbers, the Hessian-vector and
accumulation passes on the matrix cores from the operand image from 160 particles
per term on, on the vector ALUs below) against the double-precision plan, whose
kernels are others.  Bar 1e-4 of the part's largest value: fields and
coefficients are held to 1e-5 each, and a derivative of degree n, l terms
magnifies rounding by a few times their number.  A part left out, a lost fold (at
560003 and 700001 particles a unit folds twice) or a lost order is an error of
1e-2 and more."""
import numpy as np
import pytest

from paper_2602_13385_amd import inputs as I

pytestmark = pytest.mark.gpu

BAR = 1e-4
RATIO = 160
DT = 0.05
CASES = [  # (nmax, lmax, alpha, particles; negative: beyond 160 T)
    (0, 0, 1.0, 2), (4, 0, 1.0, 258), (1, 1, 0.5, 64), (6, 4, 1.0, 66), (10, 6, 1.0, 64),
    (10, 6, 0.8, 1003), (12, 8, 0.5, 129), (16, 10, 1.0, 62), (20, 10, 1.0, 127),
    (4, 2, 1.0, -1), (10, 6, 1.0, -39), (17, 3, 0.8, -5), (16, 10, 1.0, 560_003),
    (20, 10, 1.0, 700_001),
]


def _waves(pos, seed):
    rng = np.random.default_rng(seed)
    out = np.zeros_like(pos)
    for _ in range(8):
        k, ph, a = rng.normal(0.0, 2.0, 3), rng.uniform(0, 2 * np.pi), rng.normal(size=3)
        out += a[:, None] * np.cos(k @ pos + ph)
    return out


@pytest.mark.parametrize("fv", [0, 3])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"n{c[0]}l{c[1]}a{c[2]}N{c[3]}")
def test_each_part_matches_double_precision(case, fv):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_13385_amd import scf as S
    nmax, lmax, alpha, n = case
    if n < 0:
        n = RATIO * (nmax + 1) * (lmax + 1) ** 2 - n
    print(f"[adjoint parts] nmax={nmax} lmax={lmax} alpha={alpha} N={n} fv={fv}", flush=True)
    st0 = I.plummer(n, 7700 + n % 97).state().astype(np.float32)
    b = np.arange(n) % 2 == 1
    m = np.where(b, 2.0 / n, 0.0).astype(np.float32)
    lam = np.zeros((6, n), np.float32)
    lam[3:] = np.where(b, 0.0, _waves(st0[:3].astype(np.float64), 7701))
    out = {}
    for dt in (torch.float32, torch.float64):
        f32 = dt == torch.float32
        dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda").to(dt)
        for keep in (False, True):
            plan = S.Plan(nmax, lmax, alpha=alpha, dtype="f32" if f32 else "f64")
            if f32:
                plan.field_variant = fv
            hist = None
            if keep:  # the force weights of a forward step
                hist = torch.empty(2 * plan.weights_size, dtype=dt, device="cuda")
                plan.step([dev(st0[i]) for i in range(6)], dev(m), DT, 1, w_hist=hist)
            lt = [dev(lam[i]) for i in range(6)]
            plan.step_adjoint([dev(st0[i]) for i in range(6)], dev(m), DT, 1, lt, np.zeros(6),
                              w_hist=hist)
            torch.cuda.synchronize()
            out[f32, keep] = np.stack([t.cpu().numpy() for t in lt]).astype(np.float64)
        assert np.array_equal(out[f32, False], out[f32, True])
    got, ref = out[True, False][:3], out[False, False][:3]
    for name, part in (("hessian", ~b), ("coefficients", b)):
        top = np.abs(ref[:, part]).max()
        err = np.abs(got[:, part] - ref[:, part]).max()
        print(f"  {name}: largest {top:.3g}, error {err / top:.2e}", flush=True)
        assert top > 0.0
        assert err <= BAR * top, name

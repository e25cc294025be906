"""Frozen-potential substeps taken several to a launch (up to 32 field
evaluations): counts around the launch boundaries, with and without stored
accelerations, for every field variant, against the FP64 oracle."""
import numpy as np
import pytest

from paper_2602_13385_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "f64": 1e-11}
LOG = [("log", (1.5, 1.0))]
CEN = np.array([20.0, 0.0, 0.0, 0.0, I.LOG_VC_20, 0.0])


@pytest.fixture(scope="module")
def torch():
    import torch as T
    if not T.cuda.is_available():
        pytest.skip("no GPU")
    return T


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("case", [(5, 2, 257), (3, 1, 2561), (10, 6, 1000)],
                         ids=lambda c: f"n{c[0]}l{c[1]}N{c[2]}")
def test_run_lengths_match_oracle(torch, O, case, dtype):
    from paper_2602_13385_amd import scf
    nmax, lmax, n = case  # (3, 1): at least 160 T, the operand image
    p = I.plummer(n, 6100 + n)
    rnd = (lambda a: np.asarray(a, np.float32).astype(np.float64)) if dtype == "f32" else \
        (lambda a: np.asarray(a, np.float64))
    td = torch.float32 if dtype == "f32" else torch.float64
    st0, m = rnd(p.state()), rnd(p.mass)
    B = O.basis(nmax, lmax)
    Ho = O.host([(O.HOST_LOG, LOG[0][1])])
    coef = O.coeffs(B, *st0[:3], m)
    cd = torch.as_tensor(coef, device="cuda")
    plan = scf.Plan(nmax, lmax, dtype=dtype)
    dt = 0.002
    for nsteps in (1, 31, 32, 65):
        ref, cref = O.step_frozen(B, Ho, st0, coef, CEN, dt, nsteps)[:2]
        two = O.step_frozen(B, Ho, ref, coef, cref, dt, 33)[:2]
        for fv in range(plan.num_field_variants):
            print(f"[frozen] {dtype} nmax={nmax} N={n} steps={nsteps} fv={fv}", flush=True)
            plan.field_variant = fv
            st = [torch.as_tensor(st0[i], dtype=td, device="cuda") for i in range(6)]
            cen, acc = plan.step_frozen(st, cd, dt, nsteps, host=(LOG, 1.0), centre=CEN)
            torch.cuda.synchronize()
            out = np.stack([t.cpu().numpy() for t in st]).astype(np.float64)
            assert np.allclose(cen, cref, rtol=0, atol=1e-12)
            for r in (slice(0, 3), slice(3, 6)):
                assert np.abs(out[r] - ref[r]).max() <= TOL[dtype] * np.abs(ref[r]).max(), (fv, r)
            # the returned accelerations open the next call
            cen, _ = plan.step_frozen(st, cd, dt, 33, host=(LOG, 1.0), centre=cen, acc=acc)
            torch.cuda.synchronize()
            out = np.stack([t.cpu().numpy() for t in st]).astype(np.float64)
            for r in (slice(0, 3), slice(3, 6)):
                assert np.abs(out[r] - two[0][r]).max() <= TOL[dtype] * np.abs(two[0][r]).max(), fv

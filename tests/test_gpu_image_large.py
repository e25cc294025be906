"""The operand-image kernels at the largest bases, where their registers are
fullest and the reduction deals its threads in groups of 32: steps, batches and
frozen runs of at least 160 particles per term in single precision against the
double-precision plan (another kernel).  Bars as in the other GPU tests: states
and coefficients 1e-5, the returned accelerations 2e-5."""
import numpy as np
import pytest

from paper_2602_13385_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = 1e-5
RATIO = 160
LOG = ([("log", (1.5, 1.0))], 1.0)
CEN = np.array([20.0, 0.0, 0.0, 0.0, I.LOG_VC_20, 0.0])
CASES = [(16, 10, 1.0), (17, 9, 1.0), (20, 10, 0.8)]


def _rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


def _force_err(g, ref):
    mag = np.sqrt((ref ** 2).sum(0))
    return (np.sqrt(((g - ref) ** 2).sum(0)) / (mag + np.median(mag))).max()


@pytest.mark.parametrize("mode", ["step", "batched", "frozen"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"n{c[0]}l{c[1]}a{c[2]}")
def test_image_kernels_at_large_bases(case, mode):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_13385_amd import scf as S
    nmax, lmax, alpha = case
    n = RATIO * (nmax + 1) * (lmax + 1) ** 2 + 67
    sizes = [n, 0, n + 1] if mode == "batched" else [n]
    if mode == "batched":  # (the rule goes by the mean size)
        sizes = [n + n // 2 + 1, 0, 2 * n]
    print(f"[image large] nmax={nmax} lmax={lmax} alpha={alpha} {mode} {sizes}", flush=True)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    st0 = np.concatenate([I.plummer(max(k, 2), 7800 + i).state()[:, :k]
                          for i, k in enumerate(sizes)], axis=1).astype(np.float32)
    m = np.concatenate([np.full(k, 1.0 / max(k, 1)) for k in sizes]).astype(np.float32)
    cens = np.stack([CEN + 0.01 * i for i in range(len(sizes))])
    out = {}
    for dtype in ("f64", "f32"):
        plan = S.Plan(nmax, lmax, alpha=alpha, dtype=dtype)
        if dtype == "f32":
            plan.field_variant = 3
        dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda").to(plan.torch_dtype)
        st, md = [dev(st0[i]) for i in range(6)], dev(m)
        coef = torch.zeros(len(sizes) * plan.T, dtype=torch.float64, device="cuda")
        if mode == "step":
            _, acc = plan.step(st, md, 0.005, 2, host=LOG, centre=CEN, coef_last=coef)
        elif mode == "batched":
            _, acc = plan.step_batched(off, st, md, 0.005, 2, host=LOG, centres=cens,
                                       coef_last=coef)
        else:
            if dtype == "f64":
                fixed = plan.coeffs(*st[:3], md)
            coef.copy_(fixed)
            _, acc = plan.step_frozen(st, fixed, 0.002, 33, host=LOG, centre=CEN)
        torch.cuda.synchronize()
        out[dtype] = tuple(np.stack([t.cpu().numpy() for t in ts]).astype(np.float64)
                           for ts in (st, acc)) + (coef.cpu().numpy().reshape(len(sizes), -1),)
    (a, ga, ca), (b, gb, cb) = out["f32"], out["f64"]
    for c, k in enumerate(sizes):
        if k == 0:
            assert not ca[c].any()
            continue
        sl = slice(off[c], off[c + 1])
        assert _rel(a[:3, sl], b[:3, sl]) <= TOL and _rel(a[3:, sl], b[3:, sl]) <= TOL
        assert _rel(ca[c], cb[c]) <= TOL
        assert _force_err(ga[:, sl], gb[:, sl]) <= 2 * TOL

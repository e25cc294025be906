"""The field autotuner times a kernel once: from 160 particles per term on, where
the two matrix-core variants are the same kernel, variant 2 is not a candidate;
below, and in double precision, every variant is, the last ones under their own
numbers."""
import numpy as np
import pytest

from paper_2602_13385_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("case", [(16, 10, 1.0), (6, 4, 1.0), (6, 4, 0.02)],
                         ids=["n16l10", "n6l4", "n6l4small"])
def test_candidates(dtype, case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_13385_amd import scf as S
    nmax, lmax, share = case
    n = int(share * 160 * (nmax + 1) * (lmax + 1) ** 2) + 1
    p = I.plummer(n, 7900)
    for rep in range(4):
        plan = S.Plan(nmax, lmax, dtype=dtype)
        dev = lambda a: torch.as_tensor(np.asarray(a), device="cuda").to(plan.torch_dtype)
        plan.autotune(*(dev(p.pos[i]) for i in range(3)), dev(p.mass))
        fv = plan.field_variant
        assert 0 <= fv < plan.num_field_variants
        if dtype == "f32" and share >= 1.0:
            assert fv != 2

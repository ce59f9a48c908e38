"""One-block spaces with 12 or more electrons of one spin: 66 and more occupied
pairs per string, more than the inverse pair table of the stored-row gather is
built for.  The same-spin parts then take the atomic kernels; the gather was once
launched without its table, and faulted."""
import pytest
import torch

import oracle
import synth_inputs as si
from tolerance import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("space", [(13, 12, 2), (14, 13, 1), (16, 2, 14)], ids=lambda s: f"n{s[0]}a{s[1]}b{s[2]}")
@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-10), (torch.float32, 1e-5)], ids=["fp64", "fp32"])
def test_sigma_many_electrons(space, dtype, tol):
    import paper_1707_04346_amd as cis
    n, na, nb = space
    h, g = si.integrals(n, 2 * n, 51)
    ctx, ref = cis.Context(n, na, nb, h, g), oracle.Space(n, na, nb, h, g)
    c = si.ci_vector(ctx.ndet, 52)
    C = torch.tensor(c, dtype=dtype, device="cuda")
    S = torch.full_like(C, float("nan"))
    ctx.apply(C, S)
    torch.cuda.synchronize()
    assert rel(S.double().cpu().numpy(), ref.sigma(C.double().cpu().numpy())) <= tol

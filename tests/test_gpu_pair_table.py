"""Spaces on both sides of the inverse pair table's limit of 64 occupied pairs per string
(11 electrons of a spin have 55, 12 have 66): stored same-spin rows up to it, atomic
kernels beyond, through every form of the call."""
import pytest
import torch

import oracle
import synth_inputs as si
from tolerance import rel

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-10, torch.float32: 1e-5}
# (norb, nalpha, nbeta), stored rows
SPACES = [((13, 11, 2), True), ((13, 2, 11), True), ((13, 12, 11), False), ((13, 12, 12), False), ((14, 2, 12), False),
          ((12, 12, 3), False), ((16, 15, 14), False)]


CASES = [(s, stored, how) for s, stored in SPACES for how in ("apply", "noalloc", "sector") if how != "sector" or s[1] == s[2]]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("space,stored,how", CASES, ids=[f"n{s[0]}a{s[1]}b{s[2]}_{how}" for s, _, how in CASES])
def test_sigma_at_the_pair_table_limit(space, stored, how, dtype):
    import paper_1707_04346_amd as cis
    n, na, nb = space
    h, g = si.integrals(n, 2 * n, 81)
    ctx, ref = cis.Context(n, na, nb, h, g), oracle.Space(n, na, nb, h, g)
    C = torch.tensor(si.ci_vector(ctx.ndet, 82), dtype=dtype, device="cuda")
    if how == "sector":
        m = int(round(ctx.ndet ** 0.5))
        C = (C.view(m, m) + C.view(m, m).T).reshape(-1).contiguous()
        ctx.set_option(cis.OPT_SPIN_PARITY, 1)
    S = torch.full_like(C, float("nan"))
    (ctx.apply_noalloc if how == "noalloc" else ctx.apply)(C, S)
    torch.cuda.synchronize()
    assert rel(S.double().cpu().numpy(), ref.sigma(C.double().cpu().numpy())) <= TOL[dtype]
    path = ctx.last_path(cis.FP32 if dtype == torch.float32 else cis.FP64)
    assert bool(path & cis.PATH_SS_MATERIALISED) == stored


def test_deterministic_mode_refuses_beyond_it():
    import paper_1707_04346_amd as cis
    h, g = si.integrals(13, 26, 83)
    ctx = cis.Context(13, 12, 2, h, g)
    ctx.set_option(cis.OPT_DETERMINISTIC, 1)
    C = torch.ones(ctx.ndet, dtype=torch.float64, device="cuda")
    S = torch.full_like(C, 7.0)
    with pytest.raises(cis.CisigmaError) as err:
        ctx.apply(C, S)
    assert err.value.status == cis.EUNSUPPORTED
    torch.cuda.synchronize()
    assert bool((S == 7.0).all())

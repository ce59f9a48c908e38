"""One-block spaces of few alpha strings, whose sigma_3 rows are dealt to several workgroups
by runs of source tiles: against the oracle (FP64 1e-10, FP32 1e-5), repeated bit for bit,
in every place the partial sums can lie (the stored same-spin rows' place, memory of their
own where there are none, the static scratch, none with the overlap option)."""
import pytest
import torch

import oracle
import synth_inputs as si
from tolerance import rel

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-10, torch.float32: 1e-5}
# rows of 8 tiles (the first with two slices) to 201, own row of each kind; stored rows or not
SPACES = [(10, 1, 5), (11, 1, 4), (11, 2, 5), (12, 1, 6), (12, 11, 6), (12, 12, 5), (13, 2, 6), (13, 1, 11), (14, 1, 5),
          (14, 13, 4), (15, 2, 4), (15, 15, 6), (16, 1, 5), (16, 2, 4), (16, 16, 5)]


@pytest.mark.parametrize("how", ["apply", "noalloc", "overlap"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("space", SPACES, ids=lambda s: f"n{s[0]}a{s[1]}b{s[2]}")
def test_few_rows(space, dtype, how):
    import paper_1707_04346_amd as cis
    n, na, nb = space
    h, g = si.integrals(n, 2 * n, 95)
    ctx, ref = cis.Context(n, na, nb, h, g), oracle.Space(n, na, nb, h, g)
    if how == "overlap":
        ctx.set_option(cis.OPT_OVERLAP, 1)
    call = ctx.apply_noalloc if how == "noalloc" else ctx.apply
    C = torch.tensor(si.ci_vector(ctx.ndet, 96), dtype=dtype, device="cuda")
    S = [torch.full_like(C, float("nan")) for _ in range(2)]
    for s in S:
        call(C, s)
        torch.cuda.synchronize()
    assert rel(S[0].double().cpu().numpy(), ref.sigma(C.double().cpu().numpy())) <= TOL[dtype]
    d = cis.FP32 if dtype == torch.float32 else cis.FP64
    assert ctx.last_path(d) & cis.PATH_AB_OWNER
    if ctx.last_path(d) & cis.PATH_SS_MATERIALISED and min(na, nb) > 1:
        assert torch.equal(S[0], S[1])

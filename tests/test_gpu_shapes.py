"""sigma of spaces at the edges of the compiled sigma_3 shapes against the oracle:

* FP64 one-block spaces: each compiled pair of k steps and row quads with both
  scatter programs, at the fewest and the most excitations it takes, own row in a
  k step and as the rank-1 term;
* spaces of several blocks (point group, occupation types) whose row blocks and k
  steps fall between the compiled unit kernels' and take the next larger one, with
  the gathered rows ordered by source type.

Tolerances: FP64 sums of at most 10^4 terms in any order, 10^4 2^-53 of the sum of
magnitudes, which exceeds the largest element of sigma by less than a thousandfold:
1e-10.  FP32: the 1e-5 of the mode."""
import pytest
import torch

import oracle
import synth_inputs as si
from tolerance import rel

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-10, torch.float32: 1e-5}

ONE_BLOCK = [(1, 1, 1), (2, 1, 1), (3, 2, 1), (4, 2, 2), (5, 2, 3), (6, 1, 5), (6, 3, 2), (7, 3, 5), (8, 4, 4), (8, 2, 6),
             (8, 1, 7), (9, 4, 4), (9, 2, 8), (10, 1, 5), (10, 2, 8), (10, 5, 8), (10, 5, 5), (11, 1, 4), (11, 5, 5),
             (11, 2, 10), (12, 1, 3), (12, 2, 10), (12, 4, 9), (12, 5, 3), (12, 6, 3), (12, 6, 10), (13, 2, 6),
             (13, 3, 10), (13, 6, 2), (13, 4, 10), (14, 2, 5), (14, 3, 2), (14, 7, 2), (14, 2, 10), (15, 3, 2),
             (15, 4, 3), (15, 7, 2), (15, 2, 10), (16, 2, 7), (16, 3, 2), (16, 7, 1), (16, 8, 1), (16, 8, 2), (16, 2, 10)]


def both(n, na, nb, dtype, seed, **kw):
    import paper_1707_04346_amd as cis
    h, g = si.integrals(n, 2 * n, seed, orbsym=kw.get("orbsym"))
    ctx, ref = cis.Context(n, na, nb, h, g, **kw), oracle.Space(n, na, nb, h, g, **kw)
    C = torch.tensor(si.ci_vector(ctx.ndet, seed + 1), dtype=dtype, device="cuda")
    S = torch.full_like(C, float("nan"))
    ctx.apply(C, S)
    torch.cuda.synchronize()
    dt = cis.FP64 if dtype == torch.float64 else cis.FP32
    return ctx, rel(S.double().cpu().numpy(), ref.sigma(C.double().cpu().numpy())), ctx.last_path(dt) & cis.PATH_AB_OWNER


@pytest.mark.parametrize("space", ONE_BLOCK, ids=lambda s: f"n{s[0]}a{s[1]}b{s[2]}")
def test_fp64_one_block_shapes(space):
    n, na, nb = space
    _, err, owner = both(n, na, nb, torch.float64, 51)
    assert err <= TOL[torch.float64]
    assert owner or n == 1


D2H = [(9, 2, 3, 1), (10, 5, 2, 3), (11, 3, 4, 0), (12, 2, 6, 7), (13, 6, 2, 0), (14, 3, 3, 5), (15, 2, 4, 2), (16, 4, 2, 0)]
GAS = [(9, 4, 4, ([3, 3, 3], [4, 5, 8], [6, 8, 8])), (11, 3, 5, ([4, 4, 3], [5, 6, 8], [8, 8, 8])),
       (13, 4, 3, ([4, 5, 4], [4, 5, 7], [7, 7, 7])), (14, 3, 4, ([5, 5, 4], [4, 5, 7], [7, 7, 7])),
       (15, 3, 3, ([5, 5, 5], [3, 4, 6], [6, 6, 6]))]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("case", D2H, ids=lambda c: f"n{c[0]}a{c[1]}b{c[2]}t{c[3]}")
def test_point_group_shapes(case, dtype):
    n, na, nb, target = case
    _, err, _ = both(n, na, nb, dtype, 53, orbsym=[p % 8 for p in range(n)], target=target)
    assert err <= TOL[dtype]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("case", GAS, ids=lambda c: f"n{c[0]}a{c[1]}b{c[2]}")
def test_gas_shapes(case, dtype):
    n, na, nb, gas = case
    _, err, _ = both(n, na, nb, dtype, 55, gas=gas)
    assert err <= TOL[dtype]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("space", [(5, 2, 2), (6, 3, 3), (7, 1, 4), (8, 2, 6), (8, 5, 2), (9, 2, 2), (10, 5, 5), (11, 7, 3),
                                   (12, 6, 6)], ids=lambda s: f"n{s[0]}a{s[1]}b{s[2]}")
def test_both_spins_in_one_launch(space, dtype):
    """Small spaces run the same-spin parts of both spins together, except while the
    passes are timed: the same sums, so the same bits."""
    import paper_1707_04346_amd as cis
    n, na, nb = space
    h, g = si.integrals(n, 2 * n, 59)
    ctx = cis.Context(n, na, nb, h, g)
    C = torch.tensor(si.ci_vector(ctx.ndet, 60), dtype=dtype, device="cuda")
    S = [torch.full_like(C, float("nan")) for _ in range(3)]
    ctx.apply(C, S[0])
    ctx.set_option(cis.OPT_PROFILE, 1)
    ctx.apply(C, S[1])
    ctx.set_option(cis.OPT_PROFILE, 0)
    ctx.apply(C, S[2])
    torch.cuda.synchronize()
    atomic = na == 1 or nb == 1            # (a single electron's part is added by atomics)
    assert torch.equal(S[0], S[2]) or atomic
    assert rel(S[0].double().cpu().numpy(), S[1].double().cpu().numpy()) <= (TOL[dtype] if atomic else 0.0)


RDM = [(1, 1, 1), (3, 1, 2), (7, 3, 6), (8, 1, 7), (11, 2, 3), (12, 3, 2), (13, 2, 3), (13, 3, 1), (14, 2, 2), (15, 1, 3),
       (15, 2, 2), (16, 2, 2), (16, 0, 3), (16, 1, 8)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("space", RDM, ids=lambda s: f"n{s[0]}a{s[1]}b{s[2]}")
def test_density_shapes(space, dtype):
    import paper_1707_04346_amd as cis
    n, na, nb = space
    h, g = si.integrals(n, 2 * n, 57)
    ctx, ref = cis.Context(n, na, nb, h, g), oracle.Space(n, na, nb, h, g)
    C = torch.tensor(si.ci_vector(ctx.ndet, 58), dtype=dtype, device="cuda")
    g1 = torch.full((n, n), float("nan"), dtype=torch.float64, device="cuda")
    g2 = torch.full((n, n, n, n), float("nan"), dtype=torch.float64, device="cuda")
    ctx.rdm(C, g1, g2)
    torch.cuda.synchronize()
    for got, want in zip((g1, g2), ref.rdm(C.double().cpu().numpy())):
        if abs(want).max() > 0:
            assert rel(got.cpu().numpy(), want) <= TOL[dtype]
        else:
            assert got.abs().max() <= TOL[dtype]

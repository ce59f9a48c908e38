"""FP32 sigma of one-block spaces, where the alpha-beta part multiplies split FP32
operands on the bf16 matrix cores: one space per compiled shape (row blocks, one or
two 32-row steps, scatter program, own row in a slot or as the rank-1 term), the
smallest and the most ragged of each, against the oracle.

Tolerance 1e-5 of the FP32 mode; the split itself is held to the FP32 instruction's
error: a result may be off by at most (K + terms) 2^-24 of the sum of magnitudes, far
below it."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si
from tolerance import rel

pytestmark = pytest.mark.gpu

# (norb, nalpha, nbeta)
SPACES = [(2, 1, 1), (3, 1, 2), (5, 2, 2), (6, 5, 1), (7, 3, 5), (8, 4, 4), (8, 2, 6), (9, 3, 7), (9, 4, 4), (10, 5, 8),
          (10, 2, 5), (11, 9, 2), (11, 3, 9), (11, 5, 5), (12, 4, 3), (12, 1, 10), (12, 8, 11), (12, 6, 3), (12, 4, 9),
          (13, 11, 2), (13, 2, 6), (13, 2, 9), (13, 4, 5), (13, 4, 10), (14, 2, 5), (14, 2, 2), (14, 4, 2), (14, 3, 5),
          (15, 1, 7), (15, 2, 3), (15, 3, 2), (15, 3, 6), (16, 1, 8), (16, 2, 2), (16, 3, 2)]


@pytest.mark.parametrize("space", SPACES, ids=lambda s: f"n{s[0]}a{s[1]}b{s[2]}")
def test_split_sigma_matches_oracle(space):
    import paper_1707_04346_amd as cis
    n, na, nb = space
    h, g = si.integrals(n, 2 * n, 41)
    ctx, ref = cis.Context(n, na, nb, h, g), oracle.Space(n, na, nb, h, g)
    c = si.ci_vector(ctx.ndet, 42)
    C = torch.tensor(c, dtype=torch.float32, device="cuda")
    S = torch.full_like(C, float("nan"))
    ctx.apply(C, S)
    torch.cuda.synchronize()
    assert ctx.last_path(cis.FP32) & cis.PATH_AB_OWNER
    got = S.double().cpu().numpy()
    assert rel(got, ref.sigma(C.double().cpu().numpy())) <= 1e-5
    S2 = torch.empty_like(S)
    for mode in (0, 3):                      # repeatable, also with one workgroup per compute unit
        ctx.set_option(cis.OPT_SIGMA_PATH, mode)
        ctx.apply(C, S2)
        torch.cuda.synchronize()
        if ctx.last_path(cis.FP32) & cis.PATH_SS_MATERIALISED:
            assert torch.equal(S, S2)


def test_split_full_size_rank1_row():
    """8 alpha of 16 orbitals (64 excitations: the own row as the rank-1 term) with 1
    and 2 beta electrons, so that the oracle covers every element."""
    import paper_1707_04346_amd as cis
    for nb in (1, 2):
        h, g = si.integrals(16, 32, 43)
        ctx, ref = cis.Context(16, 8, nb, h, g), oracle.Space(16, 8, nb, h, g)
        c = si.ci_vector(ctx.ndet, 44)
        C = torch.tensor(c, dtype=torch.float32, device="cuda")
        S = torch.empty_like(C)
        ctx.apply(C, S)
        torch.cuda.synchronize()
        assert ctx.last_path(cis.FP32) & cis.PATH_AB_OWNER
        assert rel(S.double().cpu().numpy(), ref.sigma(C.double().cpu().numpy())) <= 1e-5


def test_split_keeps_nonfinite_elements_nonfinite():
    """An infinite or NaN element of C reaches every element of sigma it couples to;
    the others keep the values they have without it."""
    import paper_1707_04346_amd as cis
    h, g = si.integrals(8, 16, 45)
    ctx = cis.Context(8, 4, 4, h, g)
    c = si.ci_vector(ctx.ndet, 46).astype(np.float32)
    zero = c.copy()
    at = ctx.address(0b00001111, 0b00001111)
    zero[at] = 0.0
    base = torch.empty(ctx.ndet, dtype=torch.float32, device="cuda")
    ctx.apply(torch.tensor(zero, device="cuda"), base)
    col = oracle.Space(8, 4, 4, h, g).sigma(np.eye(1, ctx.ndet, at)[0])
    for bad in (np.inf, np.nan):
        c[at] = bad
        S = torch.empty_like(base)
        ctx.apply(torch.tensor(c, device="cuda"), S)
        torch.cuda.synchronize()
        s = S.cpu().numpy()
        assert not np.isfinite(s[np.abs(col) > 1e-6]).any()

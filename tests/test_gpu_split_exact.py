"""FP32 sigma of one-block spaces, product by product: the alpha-beta part sums split
FP32 operands on the bf16 matrix cores, and has to give what the FP32 instruction gives
also where a sum does not average anything out."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# one 32-row step, two, and two with the own row as the rank-1 term
SPACES = [(8, 4, 4, 72), (12, 6, 6, 16), (16, 8, 2, 12)]


def strings(n, nel):
    return np.array([x for x in range(1 << n) if bin(x).count("1") == nel], dtype=np.int64)


def singles(strs, x):
    """(string, orbital gained, orbital lost) of the single excitations of x."""
    d = strs ^ x
    at = [k for k in range(len(strs)) if bin(d[k]).count("1") == 2]
    return [(k, int(d[k] & strs[k]).bit_length() - 1, int(d[k] & x).bit_length() - 1) for k in at]


def float_integrals(n, seed):
    """Symmetric integrals that FP32 holds exactly."""
    rng = np.random.default_rng(seed)
    h = rng.standard_normal((n, n)).astype(np.float32).astype(np.float64)
    npair = n * (n + 1) // 2
    t = rng.standard_normal((npair, npair)).astype(np.float32).astype(np.float64)
    pair = np.array([[max(p, q) * (max(p, q) + 1) // 2 + min(p, q) for q in range(n)] for p in range(n)])
    return h + h.T, (np.triu(t) + np.triu(t, 1).T)[pair[:, :, None, None], pair[None, None]]


def one_element(space, scale, gscale=1.0):
    """Vectors with one element each: for every sigma element that a single product
    (ij|kl) C makes, the element and the product, both in FP64."""
    import paper_1707_04346_amd as cis
    n, na, nb, count = space
    h, g = float_integrals(n, 61)
    g = g * gscale
    ctx = cis.Context(n, na, nb, h * 0.0, g)
    sa, sb = strings(n, na), strings(n, nb)
    rng = np.random.default_rng(62)
    C = torch.zeros(ctx.ndet, dtype=torch.float32, device="cuda")
    S = torch.empty_like(C)
    got, want = [], []
    for _ in range(count):
        ja, jb = rng.integers(len(sa)), rng.integers(len(sb))
        c = np.float32(rng.standard_normal() * scale)
        at = ja * len(sb) + jb
        assert ctx.address(int(sa[ja]), int(sb[jb])) == at
        C.zero_()
        C[at] = float(c)
        ctx.apply(C, S)
        a, b = singles(sa, sa[ja]), singles(sb, sb[jb])
        idx = np.array([[x[0] * len(sb) + y[0] for y in b] for x in a])
        got.append(S[torch.tensor(idx, device="cuda")].double().cpu().numpy().ravel())
        want.append(np.array([[g[x[1], x[2], y[1], y[2]] for y in b] for x in a]).ravel() * float(c))
    assert ctx.last_path(cis.FP32) & cis.PATH_AB_OWNER
    return np.concatenate(got), np.concatenate(want)


@pytest.mark.parametrize("space", SPACES, ids=lambda s: f"n{s[0]}a{s[1]}b{s[2]}")
def test_one_product_is_as_exact_as_in_fp32(space):
    """The parts of a product are added smallest first: what is left out is below 2^-33
    of it, the earlier roundings are of sums below 2^-6 of it (at most seven), and the
    last one is 2^-24 of it, or twice that where the matrix unit does not round to
    nearest: 2 (1 + 1/16) 2^-24."""
    got, want = one_element(space, 1.0)
    assert np.abs(np.abs(got) - np.abs(want)).max() > 0.0
    assert (np.abs(np.abs(got) - np.abs(want)) <= 2.125 * 2.0 ** -24 * np.abs(want)).all()

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


@pytest.mark.parametrize("space", SPACES, ids=lambda s: f"n{s[0]}a{s[1]}b{s[2]}")
@pytest.mark.parametrize("scale,gscale", [(2.0 ** -115, 1.0), (2.0 ** 70, 1.0), (1.0, 2.0 ** -90), (2.0 ** -10, 2.0 ** 70)],
                         ids=["tiny_c", "huge_c", "tiny_g", "huge_g"])
def test_operands_outside_the_split_range(space, scale, gscale):
    """Operands whose bf16 parts would underflow or overflow: the same bound, wherever the
    product is a normal number."""
    got, want = one_element(space, scale, gscale)
    normal = np.abs(want) >= 2.0 ** -126
    assert normal.mean() > 0.9
    assert (np.abs(np.abs(got) - np.abs(want)) <= 2.125 * 2.0 ** -24 * np.abs(want))[normal].all()


@pytest.mark.parametrize("space", SPACES, ids=lambda s: f"n{s[0]}a{s[1]}b{s[2]}")
def test_infinite_element_stays_infinite(space):
    """(ij|kl) times an infinite element is infinite, not NaN."""
    got, want = one_element(space[:3] + (2,), float("inf"))
    assert np.isinf(want).all() and np.isinf(got).all()


def dense(n, na, nb, seed=63):
    import paper_1707_04346_amd as cis
    import synth_inputs as si
    h, g = si.integrals(n, 2 * n, seed)
    ctx = cis.Context(n, na, nb, h, g)
    return cis, ctx, torch.tensor(si.ci_vector(ctx.ndet, seed + 1), dtype=torch.float32, device="cuda")


@pytest.mark.parametrize("bad", [float("inf"), float("nan"), 2.0 ** -130], ids=["inf", "nan", "denormal"])
def test_bad_element_stays_where_it_couples(bad):
    """An element (Ja, Jb) that is not finite leaves every sigma element with a string Ia
    more than one excitation from Ja and Ib != Jb what it is without it."""
    cis, ctx, C = dense(8, 4, 4)
    sa = strings(8, 4)
    ja, jb = 17, 40
    C[ja * 70 + jb] = 0.0
    base, S = torch.empty_like(C), torch.empty_like(C)
    ctx.apply(C, base)
    C[ja * 70 + jb] = bad
    ctx.apply(C, S)
    far = torch.tensor([bin(int(x ^ sa[ja])).count("1") > 2 for x in sa], device="cuda")
    keep = far[:, None] & (torch.arange(70, device="cuda") != jb)[None, :]
    assert int(keep.sum()) > 1000
    d = (S.view(70, 70) - base.view(70, 70))[keep]
    assert bool(torch.isfinite(d).all()) and float(d.abs().max()) <= 1e-5 * float(base.abs().max())


@pytest.mark.parametrize("how", ["apply", "noalloc", "sector", "graph"])
@pytest.mark.parametrize("space", [(6, 3, 3), (12, 6, 6)], ids=["n6", "n12"])
def test_one_bad_vector_does_not_change_the_next(space, how):
    """The choice of the products is made anew on each call: a vector after a bad one gives
    the bits it gave before, also where a graph replays the calls."""
    cis, ctx, C = dense(*space)
    n = int(round(ctx.ndet ** 0.5))
    if how == "sector":
        ctx.set_option(cis.OPT_SPIN_PARITY, 1)
        C = (C.view(n, n) + C.view(n, n).T).reshape(-1).contiguous()
    bad = C.clone()
    bad[n + 1] = float("nan")              # on the diagonal: symmetric as the vector is
    X, S = C.clone(), torch.empty_like(C)
    call = ctx.apply_noalloc if how == "noalloc" else ctx.apply
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    call(X, S, stream=st)
    st.synchronize()
    want = S.clone()
    if how == "graph":
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            call(X, S, stream=st)
    for k in range(3):
        for src in (bad, C):
            X.copy_(src)
            S.zero_()
            torch.cuda.synchronize()
            if how == "graph":
                graph.replay()
            else:
                call(X, S, stream=st)
            torch.cuda.synchronize()
            assert bool(torch.isnan(S).any()) == (src is bad)
        assert torch.equal(S, want), k

"""The FP32 force kernel on the full lists (200,000 molecules on): every number of species that has a variant of its own,
compensated and plain sums, groups of one cell that take several batches and staged segments, and pairs within FP32
rounding of the cut-off, which are decided exactly for positions that are multiples of 2^-15.

Bound of a force row, in units u = 2^-24 of S = sum over its pairs of 24 eps (2 (sigma/r)^12 + (sigma/r)^6) / r: the pair
vector is exact; s = r^2 carries 3 u and its reciprocal 2 u more, so (sigma/r)^6 about 20 u and the factor of the pair
vector at most 2 * 20 + 5 + 8 = 53 u, with the rounding of the species constants and the products below 80 u.  Plain sums
of at most 8 terms a fold and 40 folds add at most 48 u, and the last rounding one."""
import numpy as np
import pytest

from paper_cs_0702131_amd import workloads as W

pytestmark = pytest.mark.gpu

N = 200_003
U = 2.0 ** -24
EPS = np.array([1.0, 0.5, 0.8, 1.2, 0.7])
SIG = np.array([1.0, 0.88, 0.95, 1.05, 0.9])


@pytest.fixture(scope="module")
def A():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_cs_0702131_amd as pkg
    pkg.lib()
    return pkg


@pytest.fixture(scope="module")
def liquid():
    """Box length, positions (multiples of 2^-15) and the pairs inside 2.5 with their vectors."""
    from scipy.spatial import cKDTree
    L = float(W.qround((N / 0.8) ** (1.0 / 3.0)))
    rng = np.random.default_rng(61)
    k = int(np.ceil(N ** (1.0 / 3.0)))
    g = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3) + 0.5
    g = g[np.sort(rng.permutation(len(g))[:N])]
    x = W.qround((g + rng.uniform(-0.07, 0.07, g.shape)) * (L / k))
    P = cKDTree(x, boxsize=L).query_pairs(2.5 + 1e-6, output_type="ndarray")
    d = x[P[:, 0]] - x[P[:, 1]]
    d -= L * np.round(d / L)
    inside = (d ** 2).sum(1) < 6.25
    return L, x, P[inside], d[inside]


@pytest.mark.parametrize("nsp,compensated,cells", [(1, False, 24), (2, True, 24), (2, False, 24), (3, True, 24), (5, False, 24),
                                                   (1, True, 8), (5, True, 8), (1, False, 8)])
def test_forces_of_species_and_sums(A, liquid, nsp, compensated, cells):
    import torch
    L, x, P, d = liquid
    nodes = W.uniform_nodes(L, cells)
    mesh = W.hex_mesh(nodes, nodes, nodes, periodic_axes=(0, 1, 2))
    sp = np.random.default_rng(5).integers(0, nsp, N).astype(np.int32)
    eps, sig = EPS[:nsp], SIG[:nsp]
    print(f"FP32 full lists: species {nsp} compensated {compensated} cells {cells}^3", flush=True)
    h = A.DIL(mesh, 2.5)
    t = torch.tensor(x, dtype=torch.float32, device="cuda")
    A.aica_bin(h, t)
    F, uw, npairs = A.aica_forces(h, t, torch.tensor(sp, device="cuda"), eps, sig, precision="fp32", compensated=compensated)
    a, b = sp[P[:, 0]], sp[P[:, 1]]
    e, s = np.sqrt(eps[a] * eps[b]), 0.5 * (sig[a] + sig[b])
    r2 = (d ** 2).sum(1)
    s6 = (s * s / r2) ** 3
    f = (24.0 * e * (2.0 * s6 * s6 - s6) / r2)[:, None] * d
    size = 24.0 * e * (2.0 * s6 * s6 + s6) / np.sqrt(r2)
    ref = np.stack([np.bincount(P[:, 0], f[:, q], N) - np.bincount(P[:, 1], f[:, q], N) for q in range(3)], 1)
    S = np.bincount(P[:, 0], size, N) + np.bincount(P[:, 1], size, N)
    assert int(npairs.item()) == len(P)
    err = np.abs(F.double().cpu().numpy() - ref).max(1)
    assert np.all(err <= (81 if compensated else 129) * U * S)
    u, w = (4.0 * e * (s6 * s6 - s6)).sum(), (24.0 * e * (2.0 * s6 * s6 - s6)).sum()
    assert abs(uw[0].item() - u) <= 80 * U * (4.0 * e * (s6 * s6 + s6)).sum()
    assert abs(uw[1].item() - w) <= 80 * U * (24.0 * e * (2.0 * s6 * s6 + s6)).sum()


def test_pairs_in_the_cutoff_band(A):
    """Isolated pairs whose squared separation lies mostly within a few thousand units of 2^-30 of rc^2 = 6.7e9 of them (FP32
    resolves 512 there), on both sides."""
    import torch
    from scipy.spatial import cKDTree
    k, spacing = 47, 8.0
    L, m = k * spacing, 47 ** 3
    rng = np.random.default_rng(62)
    R = int(round(2.5 / W.Q)) ** 2
    ab = rng.integers(0, 52000, (m, 2)).astype(np.int64)
    # of many (a, b) near the first the one whose c^2 comes closest
    best = np.full(m, 1 << 60)
    abc = np.zeros((m, 3), np.int64)
    for _ in range(64):
        t = ab + rng.integers(-500, 501, ab.shape)
        q = R - (t ** 2).sum(1)
        c = np.rint(np.sqrt(q.astype(np.float64))).astype(np.int64)
        off = np.abs(q - c ** 2)
        take = off < best
        best[take] = off[take]
        abc[take] = np.column_stack([t, c])[take]
    abc *= rng.choice([-1, 1], abc.shape)
    site = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3) * spacing
    base = W.qround(site + rng.uniform(0.5, 1.5, (m, 3)))
    x = np.mod(np.vstack([base, base + abc * W.Q]), L)
    # the pairs of the whole system (a few ends of neighbouring sites meet as well), in whole units of 2^-15
    P = cKDTree(x, boxsize=L).query_pairs(2.5 + 1e-6, output_type="ndarray")
    d = x[P[:, 0]] - x[P[:, 1]]
    d = np.rint((d - L * np.round(d / L)) / W.Q).astype(np.int64)
    P = P[(d ** 2).sum(1) < R]
    assert 0.2 * m < len(P) < 0.8 * m and np.median(best) < 2000
    nodes = W.uniform_nodes(L, k)
    mesh = W.hex_mesh(nodes, nodes, nodes, periodic_axes=(0, 1, 2))
    print(f"FP32 full lists: cut-off band, n={2 * m}", flush=True)
    h = A.DIL(mesh, 2.5)
    t = torch.tensor(x, dtype=torch.float32, device="cuda")
    A.aica_bin(h, t)
    F, uw, npairs = A.aica_forces(h, t, None, precision="fp32")
    f = (F != 0).any(1).cpu().numpy()
    assert int(npairs.item()) == len(P)
    assert np.array_equal(np.flatnonzero(f), np.unique(P))

"""One set of pairs for every entry point: forces, adjoint, pair export and pair counts of both precisions take the same
molecule pairs, whichever lists and group frames they run on, and both molecules of a pair take it.  The systems are
isolated pairs at the cut-off to within the rounding of their positions (at coordinates that are no multiples of 2^-15,
across a period that is none either and across a rotated side far from the axis), so that a pair decided differently by
two calls, or from its two sides, shows as a row that is zero in one and not in the other (at rc a pair's force is not
zero)."""
import numpy as np
import pytest

from paper_cs_0702131_amd import workloads as W

pytestmark = pytest.mark.gpu

RC = 2.5
SITE = 8.2  # spacing of the isolated pairs: over 3 rc and the jitter


@pytest.fixture(scope="module")
def A():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_cs_0702131_amd as pkg
    pkg.lib()
    return pkg


def _separations(m, rng, width):
    """m vectors of length rc (1 + e), |e| spread over twelve octaves below width, both signs."""
    u = rng.standard_normal((m, 3))
    u /= np.sqrt((u ** 2).sum(1))[:, None]
    e = width * 2.0 ** rng.uniform(-12.0, 0.0, m) * rng.choice([-1.0, 1.0], m)
    return RC * (1.0 + e)[:, None] * u


def _box(shape, rng, width, cells=None):
    """Pairs on a grid of sites in a periodic box whose x and y periods are no multiples of a power of two; rows k and
    m + k are a pair.  A mesh cell per site by default."""
    L = np.array([SITE * s for s in shape]) + np.array([1.0 / 7.0, 1.0 / 11.0, 0.0])
    mesh = W.hex_mesh(*[W.uniform_nodes(L[k], (cells or shape)[k]) for k in range(3)], periodic_axes=(0, 1, 2))
    g = np.stack(np.meshgrid(*[np.arange(s) for s in shape], indexing="ij"), -1).reshape(-1, 3)
    a = (g + 0.5 + rng.uniform(-0.04, 0.04, g.shape)) * (L / shape)
    a[:, 0] -= 0.5 * L[0] / shape[0]  # the first layer of sites lies on the periodic side
    x = np.mod(np.vstack([a, a + _separations(len(a), rng, width)]), L)
    return mesh, np.minimum(x, np.nextafter(L, 0.0))


def _sector(r0, r1, lz, rng, width):
    """Pairs about the coupled side of a sector of 30 degrees, periodic along z as well."""
    nz, nr = int(lz / SITE), int((r1 - r0) / SITE)
    mesh = W.wedge_mesh(r0, r1, 12, nz * SITE + 1.0 / 7.0, nr, int(r0 * np.pi / 6 / SITE), nz, 0.0, rng)
    lz, th = mesh.wedge["Lz"], np.pi / 6
    r, z = [v.ravel() for v in np.meshgrid(r0 + SITE * (0.5 + np.arange(nr - 1)), (0.5 + np.arange(nz)) * (lz / nz))]
    m = len(r)
    a = np.stack([r, np.zeros(m), z], 1) + rng.uniform(-0.2, 0.2, (m, 3))
    x = np.vstack([a, a + _separations(m, rng, width)])
    below = x[:, 1] < 0  # outside the side at angle 0: the image one sector on
    x[below] = x[below] @ W.rot_z(th).T
    x[:, 2] = np.mod(x[:, 2], lz)
    return mesh, x


def _agree(A, mesh, x, precision, pos_dtype, width, both=True):
    import torch
    n, m = len(x), len(x) // 2
    d = A.DIL(mesh, RC, guard=1e-3)
    t = torch.tensor(x, dtype=getattr(torch, pos_dtype), device="cuda")
    dt = getattr(torch, "float" + precision[2:])
    rng = np.random.default_rng(3)
    G = torch.tensor(rng.uniform(0.5, 1.5, (n, 3)), dtype=dt, device="cuda")
    print(f"pair set: n={n} {precision} positions {pos_dtype}", flush=True)
    A.aica_bin(d, t)
    F, uw, npairs = A.aica_forces(d, t, None, precision=precision)
    gx, ge, gs = A.aica_forces_adjoint(d, t, G, 0.3, None, precision=precision)
    counts = A.aica_pair_counts(d, t, precision=precision).cpu().numpy()
    P = A.aica_pairs_export(d, t, precision=precision)
    F, gx = F.double().cpu().numpy(), gx.double().cpu().numpy()
    f, g = np.abs(F).max(1) > 0, np.abs(gx).max(1) > 0
    took = np.zeros(m, bool)
    took[P[:, 0]] = True
    assert np.array_equal(P[:, 1], P[:, 0] + m) and took.sum() == len(P)
    if both:
        assert 0.2 * m < took.sum() < 0.8 * m  # pairs on both sides of the cut-off
    for name, v in (("forces", f), ("adjoint", g), ("counts", counts == 1)):
        assert np.array_equal(v[:m], v[m:]), f"{name}: {np.sum(v[:m] != v[m:])} pairs from one side only"
        assert np.array_equal(v[:m], took), f"{name}: {np.sum(v[:m] != took)} pairs differ from the export"
    assert int(npairs.item()) == len(P)
    # every pair lies at rc: U and W are the count times the terms there, dL/deps is U's (times gamma) and the forces'
    s6 = RC ** -6.0
    assert abs(uw[0].item() - len(P) * 4.0 * (s6 * s6 - s6)) <= 1e-4 * max(len(P), 1)
    assert abs(uw[1].item() - len(P) * 24.0 * (2.0 * s6 * s6 - s6)) <= 1e-3 * max(len(P), 1)
    return len(P)


# widths of the separations about rc: some tens of roundings of the coordinates (FP64: the offsets between group frames
# are rounded at the size of the absolute coordinates)
@pytest.mark.parametrize("precision,pos_dtype,width", [("fp64", "float64", 2e-13), ("fp32", "float64", 2e-5),
                                                       ("fp32", "float32", 2e-5)])
@pytest.mark.parametrize("targets", [None, (1, 8), (40, 3)])
@pytest.mark.parametrize("system", ["box", "sector"])
def test_pairs_at_the_cutoff(A, monkeypatch, system, targets, precision, pos_dtype, width):
    rng = np.random.default_rng(101)
    if targets:  # the groups of the half and the full lists (by default the same in small systems)
        monkeypatch.setenv("AICA_GROUP_TARGET", str(targets[0]))
        monkeypatch.setenv("AICA_NB_TARGET", str(targets[1]))
    mesh, x = _box((160, 12, 12), rng, width) if system == "box" else _sector(300.0, 420.0, 500.0, rng, width)
    _agree(A, mesh, x, precision, pos_dtype, width)


# FP32 from 200,000 molecules on (full lists) and just below (half lists): the groups differ by default
@pytest.mark.parametrize("shape", [(46, 46, 46), (48, 47, 45)])
@pytest.mark.parametrize("precision,width", [("fp64", 2e-14), ("fp32", 2e-5)])
def test_pairs_at_the_cutoff_of_large_systems(A, shape, precision, width):
    mesh, x = _box(shape, np.random.default_rng(102), width)
    _agree(A, mesh, x, precision, "float64", width)


# cells thousands of cut-offs wide: FP32 rounds their molecules' positions so coarsely that the box test and the search
# need the band's radius
@pytest.mark.parametrize("precision,width", [("fp64", 2e-12), ("fp32", 1e-3)])
def test_pairs_at_the_cutoff_in_wide_cells(A, precision, width):
    mesh, x = _box((1000, 2, 2), np.random.default_rng(103), width, cells=(2, 1, 1))
    _agree(A, mesh, x, precision, "float64", width)


def _dense(n_mesh, L, k, seed):
    """A strongly jittered mesh (some cells are in range only between face or edge interiors) and a dense jittered
    lattice of k^3 molecules (multiples of 2^-15)."""
    rng = np.random.default_rng(seed)
    nodes = W.uniform_nodes(L, n_mesh)
    mesh = W.hex_mesh(nodes, nodes, nodes, periodic_axes=(0, 1, 2))
    mesh = W.jitter_interior(mesh, nodes, nodes, nodes, 0.3, rng)
    mesh = W.renumber_cells(mesh, rng.permutation(mesh.n_cells))
    g = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3) + 0.5
    x = W.qround((g + rng.uniform(-0.35, 0.35, g.shape)) * (L / k))
    return mesh, x


# the vertex predicate lists fewer cell pairs than are in range: which pairs inside the cut-off it leaves out must not
# depend on the call
@pytest.mark.parametrize("n_mesh,L,k,seed", [(6, 12.0, 18, 0), (12, 24.0, 30, 4), (20, 40.0, 37, 0), (20, 40.0, 37, 1)])
def test_vertex_predicate_has_one_pair_set(A, n_mesh, L, k, seed):
    import torch
    mesh, x = _dense(n_mesh, L, k, seed)
    n, eps, sig = len(x), 1.0, 0.6
    d = A.DIL(mesh, RC, predicate="vertex")
    sets = {}
    for prec in ("fp64", "fp32"):
        t = torch.tensor(x, dtype=getattr(torch, "float" + prec[2:]), device="cuda")
        print(f"vertex predicate: n={n} {prec}", flush=True)
        A.aica_bin(d, t)
        F, uw, npairs = A.aica_forces(d, t, None, [eps], [sig], precision=prec)
        gx, ge, gs = A.aica_forces_adjoint(d, t, torch.zeros_like(F), 1.0, None, [eps], [sig], precision=prec)
        P = sets[prec] = A.aica_pairs_export(d, t, precision=prec)
        counts = A.aica_pair_counts(d, t, precision=prec).cpu().numpy()
        dx = x[P[:, 0]] - x[P[:, 1]] - L * P[:, 2:]
        s = (dx ** 2).sum(1)
        s6 = (sig * sig / s) ** 3
        assert int(npairs.item()) == len(P)
        assert np.array_equal(counts, np.bincount(P[:, :2].ravel(), minlength=n))
        # with G = 0 and gamma = 1, dL/deps is U / eps and dL/dx is -F: sums over the pairs of FP64 terms
        u = 4.0 * (s6 * s6 - s6)
        assert abs(ge[0].item() - u.sum()) <= 1e-12 * np.abs(u).sum()
        f = (24.0 * (2.0 * s6 * s6 - s6) / s)[:, None] * dx
        Fr = np.stack([np.bincount(P[:, 0], f[:, q], n) - np.bincount(P[:, 1], f[:, q], n) for q in range(3)], 1)
        # (molecules nearly touch: FP32 forces are not compared; the adjoint's terms and sums are FP64 in both precisions,
        # rounded once)
        rms = np.sqrt((Fr ** 2).sum(1).mean())
        if prec == "fp64":
            assert np.abs(F.cpu().numpy() - Fr).max() <= 1e-12 * rms
        once = 0.0 if prec == "fp64" else 2.0 ** -24 * np.abs(Fr)
        assert np.all(np.abs(gx.double().cpu().numpy() + Fr) <= 1e-12 * rms + once)
    assert np.array_equal(sets["fp32"], sets["fp64"])


# the same across a rotated side and with mixtures: with G = 0 and gamma = 1 the adjoint gives -F, and U as the sum of
# eps dL/deps (U is of first degree in eps)
@pytest.mark.parametrize("nsp", [1, 2, 3])
def test_vertex_predicate_adjoint_is_that_of_the_forces(A, nsp):
    import torch
    wl = W.wedge(seed=8, r0=10.0, r1=24.0, Lz=9.0, nr=9, nphi=6, nz=6, density=0.8, jitter=0.3)
    n, eps, sig = wl.n, np.array([1.0, 0.6, 0.8])[:nsp], np.array([1.0, 0.9, 0.95])[:nsp]
    sp = torch.tensor(np.random.default_rng(4).integers(0, nsp, n).astype(np.int32), device="cuda")
    d, dc = A.DIL(wl.mesh, RC, predicate="vertex"), A.DIL(wl.mesh, RC)
    assert d.info()["n_dil"] < dc.info()["n_dil"]
    print(f"vertex predicate, sector: n={n} species={nsp}", flush=True)
    out = {}
    for prec in ("fp64", "fp32"):
        t = torch.tensor(wl.x, dtype=getattr(torch, "float" + prec[2:]), device="cuda")
        A.aica_bin(d, t)
        F, uw, npairs = A.aica_forces(d, t, sp, eps, sig, precision=prec)
        gx, ge, gs = A.aica_forces_adjoint(d, t, torch.zeros_like(F), 1.0, sp, eps, sig, precision=prec)
        assert int(npairs.item()) == len(A.aica_pairs_export(d, t, precision=prec))
        out[prec] = [v.double().cpu().numpy() for v in (F, uw, gx, ge)]
    F, uw, gx, ge = out["fp64"]
    rms = np.sqrt((F ** 2).sum(1).mean())
    assert np.abs(gx + F).max() <= 1e-12 * rms
    assert abs((eps * ge).sum() - uw[0]) <= 1e-12 * abs(uw[0])
    F, uw, gx, ge = out["fp32"]  # the bars of the FP32 path: forces 1e-5, adjoint 1e-6
    assert np.abs(gx + F).max() <= 1.1e-5 * rms
    assert abs((eps * ge).sum() - out["fp64"][1][0]) <= 1e-6 * abs(out["fp64"][1][0])

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


def _box(shape, rng, width):
    """Pairs on a grid of sites in a periodic box whose x and y periods are no multiples of a power of two; rows k and
    m + k are a pair."""
    L = np.array([SITE * s for s in shape]) + np.array([1.0 / 7.0, 1.0 / 11.0, 0.0])
    mesh = W.hex_mesh(*[W.uniform_nodes(L[k], shape[k]) for k in range(3)], periodic_axes=(0, 1, 2))
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

"""Point location and the order of a binning: a handle that keeps hints and balls from earlier binnings gives the cells
of a handle that never binned before (search only), at the sizes where the locate kernels' blocks begin and end; and the
scans over the cells, at the sizes where their tiles and launches change, against the cells computed from the lattice
of the mesh."""
import numpy as np
import pytest

from paper_cs_0702131_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_cs_0702131_amd as pkg
    pkg.lib()
    return pkg


def _mesh(kind, rng):
    nodes = W.uniform_nodes(12.0, 5)
    if kind == "tet":
        return W.tet_mesh(nodes, nodes, nodes, periodic_axes=(0, 1, 2))
    mesh = W.hex_mesh(nodes, nodes, nodes, periodic_axes=(0, 2))
    return W.jitter_interior(mesh, nodes, nodes, nodes, 0.25, rng)


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("kind,n", [("hex", 1), ("hex", 31), ("hex", 33), ("tet", 257), ("hex", 5000), ("tet", 5000),
                                    ("hex", 131072), ("hex", 131073)])
def test_hints_give_the_searched_cells(A, kind, n, dtype):
    import torch
    rng = np.random.default_rng(71 + n)
    mesh = _mesh(kind, rng)
    L = float(mesh.hi[0])
    x = rng.uniform(1e-3, L - 1e-3, size=(n, 3))
    d = A.DIL(mesh, 1.0)
    # at rest, a small move, a move of about a cell with wrapping (as over a periodic boundary), everywhere new
    for step, amp in enumerate((0.0, 0.0, 0.02, 1.5, L, 0.02)):
        x = np.mod(x + rng.uniform(-amp, amp, size=x.shape), L)
        x = np.clip(x, 1e-3, L - 1e-3)
        t = torch.tensor(x, dtype=getattr(torch, dtype), device="cuda")
        print(f"locate: {kind} n={n} {dtype} step {step}", flush=True)
        A.aica_bin(d, t)
        fresh = A.DIL(mesh, 1.0)
        A.aica_bin(fresh, t)
        for a, b in zip(A.aica_bin_export(d, n), A.aica_bin_export(fresh, n)):
            np.testing.assert_array_equal(a, b)


# one block (a cell, four per thread, one more, the last that it takes), then launches of tiles (a cell in the last one,
# whole ones, a cell more)
@pytest.mark.parametrize("cells", [(1, 1, 1), (16, 16, 16), (17, 241, 1), (32, 32, 16), (29, 5, 113), (32, 32, 32),
                                   (331, 11, 9)])
def test_cell_scans(A, cells):
    import torch
    rng = np.random.default_rng(83)
    n = 20000
    size = [float(c) for c in cells]
    mesh = W.hex_mesh(*[W.uniform_nodes(s, c) for s, c in zip(size, cells)])
    at = np.stack([rng.integers(0, c, size=n) for c in cells], 1)
    x = at + rng.uniform(0.05, 0.95, size=(n, 3))
    want = at[:, 0] + cells[0] * (at[:, 1] + cells[1] * at[:, 2])
    print(f"cell scans: {cells}", flush=True)
    d = A.DIL(mesh, 0.5)
    t = torch.tensor(x, dtype=torch.float64, device="cuda")
    for _ in range(2):
        A.aica_bin(d, t)
        cell_of, order, count = A.aica_bin_export(d, n)
        np.testing.assert_array_equal(cell_of, want)
        np.testing.assert_array_equal(np.sort(order), np.arange(n))
        np.testing.assert_array_equal(count, np.bincount(want, minlength=mesh.n_cells))
        c = cell_of[order]
        new = np.flatnonzero(np.diff(c) != 0) + 1
        assert len(new) + 1 == len(np.unique(want))      # every cell's molecules together
        inside = np.ones(n - 1, bool)
        inside[new - 1] = False
        assert (np.diff(order)[inside] > 0).all()        # in ascending order of their ids


# lists kept from another molecule count (the cut unchanged) or rebuilt (changed): bit for bit those of a fresh handle
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_molecule_count_changes(A, precision):
    import torch
    wl = W.small_random(n_mesh=(6, 5, 4), L=(14.0, 13.0, 12.0), N=1500, seed=29)
    one = np.ones(1)
    d = A.DIL(wl.mesh, 2.5)
    for n in (1500, 1499, 1490, 700, 699, 0, 1, 1500):
        x = torch.tensor(wl.x[:n], dtype=torch.float64, device="cuda")
        G = torch.tensor(np.random.default_rng(n).normal(size=(n, 3)), dtype=getattr(torch, "float" + precision[2:]), device="cuda")
        out = []
        for h in (d, A.DIL(wl.mesh, 2.5)):
            A.aica_bin(h, x)
            F, uw, npairs = A.aica_forces(h, x, None, one, one, precision=precision)
            gx, ge, gs = A.aica_forces_adjoint(h, x, G, 0.7, None, one, one, precision=precision)
            out.append([v.cpu().numpy() for v in (F, uw, npairs, gx, ge, gs)] + [h.info()["n_groups"]])
        print(f"molecule count {n} {precision}: {out[0][-1]} groups", flush=True)
        for a, b in zip(*out):
            np.testing.assert_array_equal(a, b)

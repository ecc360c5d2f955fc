"""GPU parity of the full-list force kernel (every pair from both sides) against the FP64 oracle, at the sizes where its
clusters of 32 molecules, batches of 128, staged segments of 1024 and search words of 64 begin and end.  Bars as in
the other parity tests: FP64 1e-12 of the rms force (of the pair-force scale 24 where it is larger), pair counts equal;
FP32 1e-5."""
import sys

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


def _lattice(L, n, seed):
    """n sites of a jittered lattice in a cube of side L (multiples of Q), the sites left out chosen at random."""
    rng = np.random.default_rng(seed)
    k = int(np.ceil(n ** (1.0 / 3.0)))
    g = (np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3) + 0.5) * (L / k)
    x = g[np.sort(rng.permutation(len(g))[:n])] + rng.uniform(-0.05, 0.05, size=(n, 3)) * (L / k)
    return np.clip(W.qround(x), W.Q, L - W.Q)


# one cell holding everything (one group: partial clusters, whole batches, several batches), then dense cells whose
# neighbourhoods take several segments, then a sparse system whose groups are many cutoffs wide
@pytest.mark.parametrize("n,L,cells,periodic", [
    (1, 6.0, 1, ()), (2, 2.0, 1, ()), (31, 4.0, 1, ()), (32, 4.0, 1, ()), (33, 4.0, 1, ()), (64, 4.5, 1, ()),
    (127, 5.5, 1, ()), (128, 5.5, 1, ()), (129, 5.5, 1, ()), (1023, 11.0, 1, ()), (1025, 11.0, 1, ()), (2500, 14.0, 1, ()),
    (4000, 12.0, 2, (0, 1, 2)), (700, 5.5, 1, (0, 1, 2)), (500, 400.0, 20, (0, 2)), (300, 900.0, 3, (0, 1, 2))])
def test_full_lists_edges(A, oracle, n, L, cells, periodic):
    import torch
    L = float(W.qround(L))
    nodes = W.uniform_nodes(L, cells)
    mesh = W.hex_mesh(nodes, nodes, nodes, periodic_axes=periodic)
    x = _lattice(L, n, 51 + n)
    if L >= 400.0:  # close pairs in an otherwise empty box
        x[n // 2:] = np.clip(W.qround(x[:n - n // 2] + np.array([1.1, 0.0, 0.25])), W.Q, L - W.Q)
    print(f"full lists: n={n} L={L} cells={cells}^3 periodic={periodic}", flush=True)
    sys.stdout.flush()
    one = np.ones(1)
    Fr, Ur, Wr, nr = oracle.forces(x, np.zeros(n, np.int32), one, one, 2.5, mesh.periodic)
    d = A.DIL(mesh, 2.5)
    t = torch.tensor(x, dtype=torch.float64, device="cuda")
    A.aica_bin(d, t)
    F, uw, npairs = A.aica_forces(d, t, None, one, one, precision="fp64")
    assert int(npairs.item()) == nr
    scale = max(np.sqrt((Fr ** 2).sum(1).mean()), 24.0)
    assert np.abs(F.cpu().numpy() - Fr).max() < 1e-12 * scale
    assert abs(uw[0].item() - Ur) <= 1e-12 * max(abs(Ur), n)
    assert abs(uw[1].item() - Wr) <= 1e-12 * max(abs(Wr), 24.0 * n)


@pytest.mark.parametrize("n", [199_999, 200_000])
def test_fp32_on_either_side_of_the_list_choice(A, n):
    """FP32 takes the half lists below 200,000 molecules and the full lists from there on: both against FP64."""
    import torch
    L = float(W.qround((n / 0.8) ** (1.0 / 3.0)))
    nodes = W.uniform_nodes(L, 24)
    mesh = W.hex_mesh(nodes, nodes, nodes, periodic_axes=(0, 1, 2))
    x = _lattice(L, n, 77)
    print(f"list choice: n={n}", flush=True)
    d = A.DIL(mesh, 2.5)
    out = {}
    for prec, dt in (("fp32", torch.float32), ("fp64", torch.float64)):
        t = torch.tensor(x, dtype=dt, device="cuda")
        A.aica_bin(d, t)
        F, uw, npairs = A.aica_forces(d, t, None, precision=prec)
        out[prec] = (F.double(), uw.cpu().numpy(), int(npairs.item()))
    assert out["fp32"][2] == out["fp64"][2] > 0
    rms = out["fp64"][0].pow(2).sum(1).mean().sqrt()
    assert ((out["fp32"][0] - out["fp64"][0]).pow(2).sum(1).sqrt().max() / rms).item() < 1e-5
    assert np.all(np.abs(out["fp32"][1] - out["fp64"][1]) <= 1e-5 * np.abs(out["fp64"][1]))


@pytest.mark.parametrize("n,L,cells,nsp", [(1, 6.0, 1, 1), (33, 4.0, 1, 2), (129, 5.5, 1, 1), (1025, 11.0, 1, 3), (2500, 14.0, 1, 1)])
def test_adjoint_edges(A, oracle, n, L, cells, nsp):
    """The full-list adjoint at the same edges, both precisions (bars: FP64 1e-12, FP32 1e-6 of the rms over rows
    and of the parameter gradients)."""
    import torch
    L = float(W.qround(L))
    nodes = W.uniform_nodes(L, cells)
    mesh = W.hex_mesh(nodes, nodes, nodes)
    x = _lattice(L, n, 91 + n)
    rng = np.random.default_rng(5)
    G = W.qround(rng.standard_normal((n, 3)))
    sp = rng.integers(0, nsp, n).astype(np.int32)
    eps, sig = np.array([1.0, 0.6, 0.8])[:nsp], np.array([1.0, 0.9, 0.95])[:nsp]
    print(f"adjoint edges: n={n} L={L} species={nsp}", flush=True)
    rx, re, rs, _ = oracle.adjoint(x, sp, eps, sig, 2.5, mesh.periodic, G, 0.1)
    d = A.DIL(mesh, 2.5)
    for prec, dt, tol in (("fp64", torch.float64, 1e-12), ("fp32", torch.float32, 1e-6)):
        t = torch.tensor(x, dtype=dt, device="cuda")
        A.aica_bin(d, t)
        gx, ge, gs = A.aica_forces_adjoint(d, t, torch.tensor(G, dtype=dt, device="cuda"), 0.1,
                                           torch.tensor(sp, device="cuda"), eps, sig, precision=prec)
        rms = max(np.sqrt((rx ** 2).mean()), 1e-30)
        assert np.abs(gx.double().cpu().numpy() - rx).max() <= tol * rms
        assert np.abs(ge.cpu().numpy() - re).max() <= tol * max(np.abs(re).max(), 1e-30)
        assert np.abs(gs.cpu().numpy() - rs).max() <= tol * max(np.abs(rs).max(), 1e-30)


def test_adjoint_keeps_a_nan_gradient_in_reach(A):
    """A molecule whose upstream gradient is NaN reaches the rows of its partners inside the cut-off and no others."""
    import torch
    L, n = float(W.qround(12.0)), 900
    nodes = W.uniform_nodes(L, 5)
    mesh = W.hex_mesh(nodes, nodes, nodes)
    x = _lattice(L, n, 13)
    G = W.qround(np.random.default_rng(6).standard_normal((n, 3)))
    G[0] = np.nan
    d = A.DIL(mesh, 2.5)
    near = ((x - x[0]) ** 2).sum(1) < 2.5 ** 2
    for prec, dt in (("fp64", torch.float64), ("fp32", torch.float32)):
        t = torch.tensor(x, dtype=dt, device="cuda")
        A.aica_bin(d, t)
        gx, _, _ = A.aica_forces_adjoint(d, t, torch.tensor(G, dtype=dt, device="cuda"), 0.1, precision=prec)
        assert np.array_equal(np.isnan(gx.cpu().numpy()).any(1), near)

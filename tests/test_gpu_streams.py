"""Lists rebuilt for another molecule count while the last step's kernels are still queued on the caller's stream: a side
stream is not ordered with the copies of the new lists, so these have to wait for it."""
import numpy as np
import pytest

from paper_cs_0702131_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_lists_are_rebuilt_behind_the_queued_step(precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_cs_0702131_amd as A
    n, L = 60000, float(W.qround((60000 / 0.8) ** (1.0 / 3.0)))
    nodes = W.uniform_nodes(L, 24)
    mesh = W.hex_mesh(nodes, nodes, nodes, periodic_axes=(0, 1, 2))
    rng = np.random.default_rng(7)
    k = int(np.ceil(n ** (1.0 / 3.0)))
    g = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3) + 0.5
    x = W.qround((g[:n] + rng.uniform(-0.05, 0.05, (n, 3))) * (L / k))
    dt = getattr(torch, "float" + precision[2:])
    t, few = torch.tensor(x, dtype=dt, device="cuda"), torch.tensor(x[::2].copy(), dtype=dt, device="cuda")
    G = torch.ones_like(t)
    d = A.DIL(mesh, 2.5)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        A.aica_bin(d, t)
        ref = A.aica_forces(d, t, None, precision=precision)[0].clone()
        gref = A.aica_forces_adjoint(d, t, G, 0.1, None, precision=precision)[0].clone()
        side.synchronize()
        groups = d.info()["n_groups"]
        print(f"rebuild behind a queued step: {precision}", flush=True)
        out = []
        for _ in range(150):  # some tens of ms of queued kernels
            out = [A.aica_forces(d, t, None, precision=precision)[0],
                   A.aica_forces_adjoint(d, t, G, 0.1, None, precision=precision)[0]]
        A.aica_bin(d, few)
        assert d.info()["n_groups"] != groups
        side.synchronize()
    assert torch.equal(out[0], ref) and torch.equal(out[1], gref)

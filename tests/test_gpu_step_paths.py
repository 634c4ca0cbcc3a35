"""Paths of a step that depend on what came before it, or on its size.

* A GNN model whose angle buffers are too small for the next system of the same size: it
  redoes the step, and the result is that of a model that starts with that system.
* Energy-only passes in chunks, then the backward: the gradient of the unchunked pass.
* Step graphs under a changed skin: the cutoffs of the earlier skin are not replayed.
* Neighbour lists of 1,023 to 1,025 atoms, where one workgroup or a kernel of its own
  enters the atoms into the cells, and of few atoms in more cells than fit the workgroup's
  LDS, against all pairs."""
import numpy as np
import pytest

from synth import config_system
from synth.gnn_weights import default_gnn_file

pytestmark = pytest.mark.gpu


def _ball(n, R, dmin, seed):
    rng = np.random.default_rng(seed)
    X = []
    while len(X) < n:
        p = rng.normal(size=3)
        p *= R * rng.uniform() ** (1.0 / 3.0) / np.linalg.norm(p)
        if all(np.linalg.norm(p - q) > dmin for q in X):
            X.append(p)
    return np.array(X), rng.integers(0, 5, size=n).astype(np.int32)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_gnn_angle_buffers_grow(prec):
    from paper_2602_02234_amd import GnnModel
    X, t = _ball(40, 1.95, 0.55, 5)
    with_history, fresh = (GnnModel(default_gnn_file(), precision=prec, device=0) for _ in range(2))
    try:
        sparse = with_history.compute(20.0 * X, t, None, atom_energy=True)
        assert with_history.angles() == 0 and np.all(sparse["F"] == 0.0)
        for _ in range(2):
            a = with_history.compute(X, t, None, atom_energy=True)
            b = fresh.compute(X, t, None, atom_energy=True)
            assert with_history.graph_size() == fresh.graph_size()
            assert a["E"] == b["E"] and np.array_equal(a["F"], b["F"]) and np.array_equal(a["E_i"], b["E_i"])
    finally:
        with_history.close()
        fresh.close()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("chunk", [100, 700])
def test_backward_after_a_chunked_energy_pass(gpu_models, prec, chunk):
    import torch
    s = config_system("chain1k")
    m = gpu_models[prec]
    dev = torch.device("cuda:0")
    X, T = torch.tensor(s.coords, device=dev), torch.tensor(s.types, device=dev)
    one = torch.ones(1, dtype=torch.float64, device=dev)
    grads = []
    for c in (0, chunk):
        m.set_chunk(c)
        try:
            E = torch.zeros(1, dtype=torch.float64, device=dev)
            m.compute_device(X, T, s.box, energy=E)
            g = torch.full((s.natoms, 3), 7.0, dtype=torch.float64, device=dev)
            m.backward_device(one, g)
            grads.append((E.item(), g.cpu().numpy()))
        finally:
            m.set_chunk(0)
    assert grads[0][0] == grads[1][0] and np.array_equal(grads[0][1], grads[1][1])


def test_graphs_of_another_skin(gpu_models):
    import torch
    s = config_system("chain1k")
    m = gpu_models["fp32"]
    dev = torch.device("cuda:0")
    X, T = torch.tensor(s.coords, device=dev), torch.tensor(s.types, device=dev)
    E, F = torch.zeros(1, dtype=torch.float64, device=dev), torch.zeros((s.natoms, 3), dtype=torch.float64, device=dev)
    ref = m.compute(s.coords, s.types, s.box)
    m.set_graph(True)
    try:
        for skin in (0.5, 1.0, 0.0, 0.5):
            m.set_skin(skin, 3)
            for _ in range(5):
                F.zero_()
                m.compute_device(X, T, s.box, forces=F, energy=E)
                assert E.item() == ref["E"] and np.array_equal(F.cpu().numpy(), ref["F"])
    finally:
        m.set_skin(0.0)
        m.set_graph(False)


@pytest.mark.parametrize("n,a", [(1, 2.6), (2, 2.6), (1023, 2.6), (1024, 2.6), (1025, 2.6), (1000, 20.0)])
def test_cells_of_one_workgroup(gpu_models, n, a):
    """n atoms of a cubic lattice of edge a (20 A: 210 A across, 35 cells a side), jittered."""
    rng = np.random.default_rng(n)
    k = np.stack(np.meshgrid(*[np.arange(11)] * 3, indexing="ij"), -1).reshape(-1, 3)
    X = a * k[rng.permutation(len(k))[:n]] + rng.uniform(-0.6, 0.6, size=(n, 3))
    if a > 6.0:  # pairs, so that there are lists
        X[1::2] = X[:-1:2] + rng.uniform(1.0, 2.0, size=(n // 2, 3))
    nl, nn, _ = gpu_models["fp32"].neighbors(X, None)
    d = np.linalg.norm(X[:, None] - X[None], axis=2)
    for i in range(n):
        want = np.nonzero((d[i] < 6.0) & (np.arange(n) != i))[0]
        assert nn[i] == len(want) and np.array_equal(nl[i, :nn[i]], want)

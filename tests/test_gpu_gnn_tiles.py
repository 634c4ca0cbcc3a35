"""The GNN layers at the edges of their angle tiles and of their two workgroup sizes,
against the FP64 oracle.

* Balls of n atoms of radius 1.95 A: every atom has the other n - 1 within the angle
  cutoff, so its rows of angles have min(n - 1, 48) - 1 entries: 15, 16 and 31, 32 (one
  below and exactly one and two tiles of 16), 47 (the capacity, reached and overrun).
  Forces are larger than in water and float32 rounding scales with them, so the metrics
  are taken relative to the oracle's force RMS (compare's `scale`).
* Systems of 512 and 513 atoms, the last with eight and the first with four waves per
  atom: repeated calls agree bit for bit, and sampled E_i match the oracle run on the
  atoms within 3 rc of each."""
import numpy as np
import pytest

from oracle.gnn import build_graph, evaluate, forward, load_gnn_model
from synth.gnn_weights import default_gnn_file
from tolerances import TOL_GNN, assert_within_gnn, compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ognn():
    return load_gnn_model(default_gnn_file())


@pytest.fixture(scope="module")
def gnn_models():
    from paper_2602_02234_amd import GnnModel
    ms = {p: GnnModel(default_gnn_file(), precision=p, device=0) for p in ("fp32", "bf16")}
    yield ms
    for m in ms.values():
        m.close()


def _ball(n, R, dmin, seed):
    rng = np.random.default_rng(seed)
    X = []
    while len(X) < n:
        p = rng.normal(size=3)
        p *= R * rng.uniform() ** (1.0 / 3.0) / np.linalg.norm(p)
        if all(np.linalg.norm(p - q) > dmin for q in X):
            X.append(p)
    return np.array(X), rng.integers(0, 5, size=n).astype(np.int32)


@pytest.mark.parametrize("n", [17, 18, 33, 34, 49, 50])
def test_angle_tile_edges(gnn_models, ognn, n):
    prec = "fp32"  # both precisions run the same tiles; the bfloat16 bounds hold at water's density only
    X, t = _ball(n, 1.95, 0.55, 5)
    ref = evaluate(ognn, X, t, None)
    nc = min(n - 1, 48)
    assert ref["n_angles"] == n * nc * (nc - 1)
    out = gnn_models[prec].compute(X, t, None, atom_energy=True)
    assert gnn_models[prec].graph_size() == (n * (n - 1), n * nc, ref["n_angles"])
    scale = max(1.0, float(np.sqrt(np.mean(ref["F"] ** 2))))
    m = compare(out, ref, n, scale=scale)
    print(prec, n, "force rms", scale, m)
    assert_within_gnn(m, prec)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("n", [512, 513])
def test_workgroup_sizes(gnn_models, ognn, prec, n):
    rng = np.random.default_rng(9)
    k = np.stack(np.meshgrid(*[np.arange(9)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
    X, t = 2.4 * k + rng.uniform(-0.5, 0.5, size=(n, 3)), rng.integers(0, 5, size=n).astype(np.int32)
    m = gnn_models[prec]
    a = m.compute(X, t, None, atom_energy=True)
    for _ in range(3):
        b = m.compute(X, t, None, atom_energy=True)
        assert np.array_equal(a["F"], b["F"]) and np.array_equal(a["E_i"], b["E_i"]) and a["E"] == b["E"]
    assert np.max(np.abs(a["F"].sum(0))) < 1e-4 * n ** 0.5
    for i in (0, n // 2, n - 1):
        near = np.nonzero(np.linalg.norm(X - X[i], axis=1) < 18.5)[0]
        Ei = forward(ognn, build_graph(ognn, X[near], t[near], None))[int(np.nonzero(near == i)[0][0])]
        assert abs(a["E_i"][i] - Ei) <= TOL_GNN[prec]["e_atom"]

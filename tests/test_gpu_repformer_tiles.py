"""The repformer layers at the edges of their token blocks and kernel instances, against
the FP64 oracle.

* Balls of n atoms within rc of each other (every atom has the other n - 1 as neighbours):
  1 neighbour; 15, 16 and 17 (one and two blocks of 16); 95, 96 and 97, 112 and 113 (the
  6-wave instance up to 96, the 8-wave one from 97).  Forces are larger than in water and
  float32 rounding scales with them, so the metrics are taken relative to the oracle's
  force RMS (compare's `scale`).
* The same atoms with a ball of 98 beside isolated pairs: both instances in one call.
* 256, 257 and 258 atoms (one atom per workgroup; two, with and without a last half):
  repeated calls agree bit for bit, and sampled E_i match the oracle run on the atoms
  within 3 rc of each."""
import numpy as np
import pytest

from oracle.repformer import build_edges, evaluate, forward, load_rep_model
from synth.rep_weights import default_rep_file
from tolerances import TOL_REP, compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def orep():
    return load_rep_model(default_rep_file())


@pytest.fixture(scope="module")
def rep_model():
    from paper_2602_02234_amd import RepModel
    m = RepModel(default_rep_file(), device=0)
    yield m
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


def _check(out, ref, n):
    scale = max(1.0, float(np.sqrt(np.mean(ref["F"] ** 2))))
    m = compare(out, ref, n, scale=scale)
    print(n, "force rms", scale, m)
    bad = {k: (v, TOL_REP["fp32"][k]) for k, v in m.items() if k in TOL_REP["fp32"] and not v <= TOL_REP["fp32"][k]}
    assert not bad, (bad, m)


@pytest.mark.parametrize("n", [2, 16, 17, 18, 96, 97, 98, 113, 114])
def test_block_edges(rep_model, orep, n):
    X, t = _ball(n, 2.95, 0.8, 5)
    ref = evaluate(orep, X, t, None)
    assert int(ref["nnei"].min()) == n - 1
    out = rep_model.compute(X, t, None, atom_energy=True)
    assert rep_model.edges() == n * (n - 1)
    _check(out, ref, n)


@pytest.mark.parametrize("pairs", [0, 100])
def test_both_instances(rep_model, orep, pairs):
    """98 atoms of 97 neighbours, an atom without any, and pairs: 99 and 299 atoms."""
    X, t = _ball(98, 2.95, 0.8, 5)
    far = np.array([[40.0 + 20.0 * k + 1.5 * a, 0.0, 0.0] for k in range(pairs) for a in range(2)]).reshape(-1, 3)
    X = np.concatenate([X, [[0.0, 40.0, 0.0]], far])
    t = np.concatenate([t, np.arange(1 + 2 * pairs) % 5]).astype(np.int32)
    order = np.random.default_rng(3).permutation(len(X))
    X, t = X[order], t[order]
    _check(rep_model.compute(X, t, None, atom_energy=True), evaluate(orep, X, t, None), len(X))


@pytest.mark.parametrize("n", [256, 257, 258])
def test_workgroup_sizes(rep_model, orep, n):
    rng = np.random.default_rng(9)
    k = np.stack(np.meshgrid(*[np.arange(9)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
    X, t = 2.4 * k + rng.uniform(-0.5, 0.5, size=(n, 3)), rng.integers(0, 5, size=n).astype(np.int32)
    a = rep_model.compute(X, t, None, atom_energy=True)
    for _ in range(3):
        b = rep_model.compute(X, t, None, atom_energy=True)
        assert np.array_equal(a["F"], b["F"]) and np.array_equal(a["E_i"], b["E_i"]) and a["E"] == b["E"]
    assert np.max(np.abs(a["F"].sum(0))) < 1e-4 * n ** 0.5
    for i in (0, n // 2, n - 1):
        near = np.nonzero(np.linalg.norm(X - X[i], axis=1) < 3 * orep.rc + 0.5)[0]
        Ei = forward(orep, build_edges(orep, X[near], t[near], None))[int(np.nonzero(near == i)[0][0])]
        assert abs(a["E_i"][i] - Ei) <= TOL_REP["fp32"]["e_atom"]

"""The float32 attention descriptor's kernels at the edges of their tiles and instances,
against the FP64 oracle: neighbour counts one below, at and one above a block of 16 and
the last count of the 6-wave instance (96), and the capacity (120); and systems just below and above the size from which two atoms share a workgroup.

The bounds are those of tolerances.py, stated for forces of RMS 1 eV/A: where an oracle
force RMS is larger, forces and energies are divided by it first."""
import numpy as np
import pytest

from oracle.dp import evaluate
from tolerances import compare, assert_within

pytestmark = pytest.mark.gpu


def _ball(n, R, dmin, seed):
    """n atoms uniform in a ball of radius R, at least dmin apart (every pair within 2R)."""
    rng = np.random.default_rng(seed)
    X = []
    while len(X) < n:
        p = rng.normal(size=3)
        p *= R * rng.uniform() ** (1.0 / 3.0) / np.linalg.norm(p)
        if all(np.linalg.norm(p - q) > dmin for q in X):
            X.append(p)
    return np.array(X), rng.integers(0, 5, size=n).astype(np.int32)


def _check(gpu, omodel, X, t):
    ref = evaluate(omodel, X, t, None)
    out = gpu.compute(X, t, None, atom_energy=True)
    scale = max(1.0, float(np.sqrt(np.mean(ref["F"] ** 2))))
    m = compare(out, ref, len(t), scale=scale)
    print(len(t), "force rms", scale, m)
    assert_within(m, "fp32")
    return ref, out


@pytest.mark.parametrize("n", [2, 16, 17, 18, 97, 98, 113, 114, 121])
def test_neighbour_counts_at_tile_edges(gpu_fp32, omodel, n):
    X, t = _ball(n, 2.95, 0.8, 5)
    ref, _ = _check(gpu_fp32, omodel, X, t)
    assert int(ref["nnei"].min()) == n - 1


@pytest.mark.parametrize("n", [256, 257, 258])
def test_two_atoms_per_workgroup(gpu_fp32, omodel, n):
    """Below 257 atoms every atom has a workgroup of its own; above, two share one (the
    last alone when the count is odd).  Both give the same bits: the first 192 atoms of a
    far-apart pair of clusters do not depend on the size of the system."""
    X, t = _ball(192, 6.0, 1.0, 7)
    Y, u = _ball(n - 192, 4.0, 1.0, 8)
    XY, tu = np.concatenate([X, Y + 100.0]), np.concatenate([t, u])
    _, out = _check(gpu_fp32, omodel, XY, tu)
    alone = gpu_fp32.compute(X, t, None, atom_energy=True)
    assert np.array_equal(alone["E_i"], out["E_i"][:192]) and np.array_equal(alone["F"], out["F"][:192])

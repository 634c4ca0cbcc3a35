"""The fitting net's workgroups of 32 atoms (from 4,096 atoms on) with atoms that have neighbours in
every part of their tiles: the same cluster of 14 atoms in the first and in the second half of the
first tile, across the end of a tile, and in the last, partial tile; lone atoms elsewhere.

The copies lie at distances that float64 adds without rounding (coordinates are multiples of
2^-20), so each has the energies and forces of the cluster alone, bit for bit, and these agree with
the FP64 oracle.  Four heads with weights of both signs and zero."""
import numpy as np
import pytest

from oracle import load_model
from oracle.dp import evaluate_heads
from synth import default_model_file
from tolerances import assert_within, compare

pytestmark = pytest.mark.gpu

WEIGHTS = (0.75, 0.0, -0.5, 0.25)
K = 14


def _cluster():
    rng = np.random.default_rng(3)
    X = []
    while len(X) < K:
        p = rng.uniform(0.0, 6.0, size=3)
        if all(np.linalg.norm(p - q) > 1.0 for q in X):
            X.append(np.round(p * 2.0 ** 20) / 2.0 ** 20)
    return np.array(X), (np.arange(K) % 5).astype(np.int32)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("n", [4096, 4113, 4127])
def test_rows_of_wide_tiles(prec, n):
    from paper_2602_02234_amd import Model
    path = default_model_file(nheads=4)
    C, t = _cluster()
    ref = evaluate_heads(load_model(path), C, t, None, WEIGHTS)
    k = np.arange(n)
    X = 512.0 + 16.0 * np.stack([k % 17, k // 17 % 17, k // 289], 1)
    T = (k % 5).astype(np.int32)
    firsts = [0, 16, 2048 - 7, n - K]
    for c, a in enumerate(firsts):
        X[a:a + K], T[a:a + K] = C - 128.0 * (c + 1), t
    m = Model(path, prec)
    m.set_head_weights(WEIGHTS)
    alone = m.compute(C, t, None, atom_energy=True)
    out = m.compute(X, T, None, atom_energy=True)
    m.close()
    got = compare(alone, ref, K)
    print(prec, n, got)
    assert_within(got, prec)
    for a in firsts:
        assert np.array_equal(out["E_i"][a:a + K], alone["E_i"]) and np.array_equal(out["F"][a:a + K], alone["F"]), a

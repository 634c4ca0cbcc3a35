"""More atoms with long lists (over 96 neighbours) than the 256 workgroups that take them: three copies
of a ball of 121 atoms with full lists, far from each other, with an odd number of lone pairs
beside them.

The copies lie at distances that float64 adds without rounding (coordinates are multiples of
2^-20): every copy has the same energies and forces, bit for bit, and the attention models' are those
of the ball alone, which agree with the FP64 oracle (test_gpu_descriptor_tiles*.py); the repformer's are
compared with the oracle here."""
import numpy as np
import pytest

from test_gpu_descriptor_tiles import _ball

pytestmark = pytest.mark.gpu

N, COPIES, PAIRS = 121, 3, 7


def _system():
    B, t = _ball(N, 2.95, 0.8, 5)
    B = np.round(B * 2.0 ** 20) / 2.0 ** 20
    pairs = np.array([[16.0 * (k // 2) + (k % 2), 512.0, 0.0] for k in range(2 * PAIRS + 1)])  # the last one alone
    X = np.concatenate([B + np.array([128.0 * c, 0.0, 0.0]) for c in range(COPIES)] + [pairs])
    T = np.concatenate([t] * COPIES + [np.zeros(len(pairs), np.int32)]).astype(np.int32)
    return B, t, X, T


def _copies(out):
    for c in range(1, COPIES):
        for k in ("E_i", "F"):
            assert np.array_equal(out[k][N * c:N * (c + 1)], out[k][:N]), (c, k)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_attention(gpu_models, prec):
    B, t, X, T = _system()
    alone = gpu_models[prec].compute(B, t, None, atom_energy=True)
    out = gpu_models[prec].compute(X, T, None, atom_energy=True)
    _copies(out)
    assert np.array_equal(out["E_i"][:N], alone["E_i"]) and np.array_equal(out["F"][:N], alone["F"])


def test_repformer():
    from oracle.repformer import evaluate, load_rep_model
    from paper_2602_02234_amd import RepModel
    from synth.rep_weights import default_rep_file
    from tolerances import TOL_REP, compare
    B, t, X, T = _system()
    m = RepModel(default_rep_file())
    out = m.compute(X, T, None, atom_energy=True)
    m.close()
    _copies(out)
    ref = evaluate(load_rep_model(default_rep_file()), X, T, None)
    scale = max(1.0, float(np.sqrt(np.mean(ref["F"][:N] ** 2))))
    got = compare(out, ref, len(T), scale=scale)
    print(got)
    assert all(got[k] <= v for k, v in TOL_REP["fp32"].items()), got

"""The branch-free tanh of the first layers does not err the same way for every argument: its mean
error over [0.43, 0.45], where a power series ends or a formula in exp(-2 x) begins to cancel.

A GNN is set up so that an atom's energy is the sum of 64 initial edge features tanh(x) of its only
neighbour, 0.4 A away (switch exactly 1): x are the biases of the edge embedding, no layer changes
the features, and the node update hands their mean over sel to the fitting net, which adds them up.
The reference takes sel's reciprocal as float32 holds it.

Bound: an eighth of float32's unit roundoff, 2^-27.  The roundings of 64 x 48 activations (at most 2^-24
of each) average out to a sixth of that."""
import numpy as np
import pytest

from synth.gnn_weights import make_gnn_params, write_gnn_file

pytestmark = pytest.mark.gpu


def test_mean_error(tmp_path):
    from paper_2602_02234_amd import GnnModel
    rng = np.random.default_rng(23)
    X, T = np.array([[0.0, 0.0, 0.0], [0.4, 0.0, 0.0]]), np.zeros(2, dtype=np.int32)
    sel = float(np.float32(1.0) / np.float32(120.0))
    off = []
    for _ in range(48):
        x = (rng.uniform(0.43, 0.45, size=64)).astype(np.float32).astype(np.float64)
        p = {k: np.zeros_like(v) for k, v in make_gnn_params().items()}
        p["be0"][:] = x
        p["Wnn0"][64 + np.arange(64), np.arange(64)] = 1.0  # rows: n (64), then the mean of the edges
        p["G1"][np.arange(64), np.arange(64)] = 1.0
        p["G3"][:64] = 1.0
        path = str(tmp_path / "model.bin")
        write_gnn_file(path, params=p)
        m = GnnModel(path, "fp32")
        E = m.compute(X, T, None, atom_energy=True)["E_i"]
        m.close()
        exact = np.tanh(np.tanh(np.tanh(x) * sel)).sum()
        off.append(E[0] / exact - 1.0)
    print("mean relative error %.2e, bound %.2e" % (np.mean(off), 2.0 ** -27))
    assert abs(np.mean(off)) <= 2.0 ** -27

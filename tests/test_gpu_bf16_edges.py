"""The bfloat16 models at the edges of their tiles: energies per atom and the RMS force error against
the FP64 oracle.

* GNN: balls whose atoms have 15, 16, 31, 32 and 47 angles a row (test_gpu_gnn_tiles.py).  A force passes, in
  each of three layers, three rounded products forward (angle, message, edge) and four back; each
  rounds two operands, by up to 2^-9 of themselves, uniformly: rms 2^-9 / sqrt(3).  42 independent ones add up
  to sqrt(42 / 3) 2^-9 = 7.3e-3 of the force.
* Attention: neighbour counts at the edges of blocks (test_gpu_descriptor_tiles_b16.py).  13 products forward
  (embedding; Q, K, scores, V, output of two layers) and 13 back: sqrt(52 / 3) 2^-9 = 8.1e-3.

Forces and energies are divided by the oracle's force RMS where that is above 1 eV/A; the energies'
bound is that of tolerances.py."""
import numpy as np
import pytest

from tolerances import TOL, TOL_GNN, compare
from test_gpu_descriptor_tiles import _ball

pytestmark = pytest.mark.gpu


def _check(what, out, ref, n, f_rmse, e_atom):
    m = compare(out, ref, n, scale=max(1.0, float(np.sqrt(np.mean(ref["F"] ** 2)))))
    print(what, n, m, "bounds", f_rmse, e_atom)
    assert m["f_rmse"] <= f_rmse and m["e_atom"] <= e_atom


@pytest.mark.parametrize("n", [17, 18, 33, 34, 49, 50])
def test_gnn_angle_tile_edges(n):
    from oracle.gnn import evaluate, load_gnn_model
    from paper_2602_02234_amd import GnnModel
    from synth.gnn_weights import default_gnn_file
    X, t = _ball(n, 1.95, 0.55, 5)
    m = GnnModel(default_gnn_file(), "bf16")
    out = m.compute(X, t, None, atom_energy=True)
    m.close()
    ref = evaluate(load_gnn_model(default_gnn_file()), X, t, None)
    _check("gnn", out, ref, n, (42 / 3) ** 0.5 * 2.0 ** -9, TOL_GNN["bf16"]["e_atom"])


@pytest.mark.parametrize("n", [2, 16, 17, 18, 33, 34, 81, 97, 98, 113, 114, 121])
def test_attention_block_edges(gpu_bf16, omodel, n):
    from oracle.dp import evaluate
    X, t = _ball(n, 2.95, 0.8, 5)
    out = gpu_bf16.compute(X, t, None, atom_energy=True)
    _check("attention", out, evaluate(omodel, X, t, None), n, (52 / 3) ** 0.5 * 2.0 ** -9, TOL["bf16"]["e_atom"])

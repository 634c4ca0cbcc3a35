"""First-layer activations at and beyond the end of float32's range, in the models that form them
with the branch-free tanh: tanh is 1 there, also where its argument overflows to infinity.

Some of the first layer's weights are +-3e38, so that s w (or cos w) runs from about 1e36 to
infinity over the neighbours.  Those features are +-1 with a gradient of zero; the rest of the model
is the seeded one, and the bounds are those of tolerances.py (forces and energies divided by the
oracle's force RMS where that is above 1)."""
import numpy as np
import pytest

from tolerances import assert_within, assert_within_gnn, compare

pytestmark = pytest.mark.gpu

BIG = 3e38


def _overdrive(w):
    w[0, ::8] = BIG * (-1.0) ** np.arange(len(w[0, ::8]))


def _attn(path, prec):
    from oracle import load_model
    from oracle.dp import evaluate
    from paper_2602_02234_amd import Model
    from synth.weights import make_params, write_model_file
    p = make_params()
    _overdrive(p["emb_W1"])
    write_model_file(path, params=p)
    return Model(path, prec), evaluate, load_model(path), lambda m: assert_within(m, prec)


def _gnn(path, prec):
    from oracle.gnn import evaluate, load_gnn_model
    from paper_2602_02234_amd import GnnModel
    from synth.gnn_weights import make_gnn_params, write_gnn_file
    p = make_gnn_params()
    _overdrive(p["We0"])
    _overdrive(p["Wa0"])
    write_gnn_file(path, params=p)
    return GnnModel(path, prec), evaluate, load_gnn_model(path), lambda m: assert_within_gnn(m, prec)


@pytest.mark.parametrize("make,prec", [(_attn, "fp32"), (_attn, "bf16"), (_gnn, "fp32"), (_gnn, "bf16")])
def test_saturated_first_layer(tmp_path, water192, make, prec):
    s = water192
    m, evaluate, om, check = make(str(tmp_path / "model.bin"), prec)
    ref = evaluate(om, s.coords, s.types, s.box)
    out = m.compute(s.coords, s.types, s.box, atom_energy=True)
    m.close()
    assert np.isfinite(out["E"]) and np.isfinite(out["F"]).all() and np.isfinite(out["E_i"]).all()
    scale = max(1.0, float(np.sqrt(np.mean(ref["F"] ** 2))))
    got = compare(out, ref, s.natoms, scale=scale)
    print(prec, "force rms", scale, got)
    check(got)

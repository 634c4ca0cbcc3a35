"""The repformer's virial against the FP64 oracle evaluated with the weights the library holds
(rounded to float32), averaged over water boxes.

A box's virial is a sum that cancels to a twelfth of its terms (`cancel`, from the oracle), so
a rounding that is alike in all atoms -- a partial sum that depends on the atom's type alone -- shows
`cancel` times enlarged, in every box with the same sign, where independent roundings average out.
Bound: the mean size of one rounding to nearest, 2^-25, so enlarged."""
import numpy as np
import pytest

from oracle.repformer import build_edges, evaluate, load_rep_model, pair_gradients
from synth.rep_weights import default_rep_file, make_rep_params, write_rep_file
from synth.systems import request_system

pytestmark = pytest.mark.gpu


def test_mean_virial_error(tmp_path):
    from paper_2602_02234_amd import RepModel
    # the last layer stays: the library sums it in float64
    p = {k: v if k in ("G3", "d3") else v.astype(np.float32).astype(np.float64) for k, v in make_rep_params().items()}
    om = load_rep_model(write_rep_file(str(tmp_path / "rounded.bin"), params=p))
    m = RepModel(default_rep_file())
    off, cancel = [], []
    for k in range(8):
        s = request_system(192, "water", 60 + k)
        V = evaluate(om, s.coords, s.types, s.box)["virial"]
        g = build_edges(om, s.coords, s.types, s.box)
        gD = pair_gradients(om, g)[1]
        cancel.append((np.linalg.norm(g["D"], axis=1) * np.linalg.norm(gD, axis=1)).sum() / np.linalg.norm(V))
        out = m.compute(s.coords, s.types, s.box)
        off.append(((out["virial"] - V) * V).sum() / (V * V).sum())
    m.close()
    bound = np.mean(cancel) * 2.0 ** -25
    print("virial error %.2e (each %s), bound %.2e" % (np.mean(off), np.array2string(np.array(off), precision=1), bound))
    assert abs(np.mean(off)) <= bound

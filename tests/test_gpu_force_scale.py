"""The float32 attention model's forces as a whole: their projection on the FP64 oracle's, averaged over
water boxes.  Independent roundings average out over the forces; a constant held in float32 (a
reciprocal of a width or a capacity) makes all of them too large or too small together.  Bound:
float32's spacing at 1, 2^-23."""
import numpy as np
import pytest

from oracle.dp import evaluate
from synth.systems import request_system

pytestmark = pytest.mark.gpu


def test_mean_force_scale(gpu_fp32, omodel):
    off = []
    for k in range(8):
        s = request_system(192, "water", 60 + k)
        F = evaluate(omodel, s.coords, s.types, s.box)["F"]
        out = gpu_fp32.compute(s.coords, s.types, s.box)["F"]
        off.append(((out - F) * F).sum() / (F * F).sum())
    print("forces too large by %.2e (each %s), bound %.2e" % (np.mean(off), np.array2string(np.array(off), precision=1), 2.0 ** -23))
    assert abs(np.mean(off)) <= 2.0 ** -23

"""The first steps of a model and of a server's lanes, whose workspaces are allocated in the call, on
streams that do not wait for the default one, with other work on the card: the results of a
later call, bit for bit.  Nothing that is still under way on the default stream may reach a new
workspace.  Device memory is filled with NaN and given back first."""
import numpy as np
import pytest

from synth.systems import request_system

pytestmark = pytest.mark.gpu


def _dirty(torch):
    x = torch.full((1 << 29,), float("nan"), device="cuda")  # 2 GiB
    torch.cuda.synchronize()
    del x
    torch.cuda.empty_cache()


def _same(a, b):
    return a["E"] == b["E"] and np.array_equal(a["F"], b["F"]) and np.array_equal(a["virial"], b["virial"])


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_first_requests_of_a_server(model_path, prec):
    """Small requests in batches and two large ones in chunks, on three lanes at once."""
    import torch
    from paper_2602_02234_amd import Model, Server
    m = Model(model_path, prec)
    systems = [(w.coords, w.types, w.box) for w in (request_system(n, "water", 40 + k) for k, n in enumerate(
        (192, 384, 9999, 600, 20001, 192, 1500, 3000)))]
    alone = [m.compute(*s) for s in systems]
    for _ in range(3):
        _dirty(torch)
        srv = Server(m, 8 << 30)
        ids = [srv.submit(*s) for s in systems]
        outs = [srv.wait(i, 120.0) for i in ids]
        srv.close()
        assert [_same(a, o) for a, o in zip(alone, outs)] == [True] * len(systems)
    m.close()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("n", [192, 3000])
def test_first_step_on_another_stream(model_path, prec, n):
    import torch
    from paper_2602_02234_amd import Model
    w = request_system(n, "water", 50)
    X, T = torch.tensor(w.coords, device="cuda"), torch.tensor(w.types, device="cuda")
    busy = torch.ones(1 << 28, device="cuda")
    got = []
    for k in range(4):
        F, V = torch.zeros(n, 3, dtype=torch.float64, device="cuda"), torch.zeros(9, dtype=torch.float64, device="cuda")
        if k < 3:
            _dirty(torch)
            m = Model(model_path, prec)
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        busy.mul_(1.0)  # the default stream has work under way
        with torch.cuda.stream(s):
            E = m.compute_device(X, T, w.box, forces=F, virial=V)
        torch.cuda.synchronize()
        got.append({"E": E.item(), "F": F.cpu().numpy(), "virial": V.cpu().numpy()})
        if k < 2:
            m.close()
    m.close()
    assert all(_same(got[3], g) for g in got)

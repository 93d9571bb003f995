"""Edge lists that do not fit their capacity, in both forms and through every
entry point that evaluates: no pass may follow the row offsets (which hold the
true counts) past the arrays of the list.  A capacity error, then the same
result as with enough room: the passes of the failed attempt leave nothing
behind."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available()
    return T


@pytest.fixture(scope="module")
def M():
    import paper_2509_21694_amd as mod
    return mod


def _model(M, channels):
    hp = W.HParams(n_species=2, n_layers=3, l_max=2, channels=channels)
    return M.Model(hp, W.make_weights(hp, 5))


def _same(a, b):
    for k in ("energy", "forces", "virial"):
        assert np.array_equal(a[k].cpu().numpy(), b[k].cpu().numpy()), k


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("channels,K,n_owned", [(64, 2, None), (64, 3, None), (128, 2, None), (128, 3, None),
                                                (64, 2, 40), (64, 3, 40)])
def test_evaluate_retries(torch, M, channels, K, n_owned, prec):
    s = W.small_system()
    model = _model(M, channels)
    x = torch.tensor(s.positions, dtype=torch.float64, device="cuda")
    z = torch.tensor(s.species, dtype=torch.int32, device="cuda")
    print(f"[overflow] C={channels} K={K} n_owned={n_owned} {prec}", flush=True)
    o = model.evaluate(x, z, s.cell, s.pbc, K=K, precision=prec, max_edges=6015, n_owned=n_owned)
    assert o["n_edges"] == 6016
    _same(o, model.evaluate(x, z, s.cell, s.pbc, K=K, precision=prec, max_edges=8192, n_owned=n_owned))


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("K", [2, 3])
def test_batch_retries(torch, M, K, prec):
    s = W.small_system()
    model = _model(M, 64)
    b = M.Batch([s, s], "cuda")
    print(f"[overflow] batch K={K} {prec}", flush=True)
    o = M.evaluate_batch(model, b, K=K, precision=prec, max_edges=6100)
    assert o["n_edges"] == 2 * 6016
    _same(o, M.evaluate_batch(model, b, K=K, precision=prec))


@pytest.mark.parametrize("K", [2, 3])
def test_noalloc_reports(torch, M, K):
    """No status to read: NaN in the energy and the virial."""
    s = W.small_system()
    model = _model(M, 64)
    x = torch.tensor(s.positions, dtype=torch.float64, device="cuda")
    z = torch.tensor(s.species, dtype=torch.int32, device="cuda")
    o = dict(energy=torch.zeros(1, dtype=torch.float64, device="cuda"),
             forces=torch.zeros((s.n_atoms, 3), dtype=torch.float64, device="cuda"),
             virial=torch.zeros((3, 3), dtype=torch.float64, device="cuda"))
    print(f"[overflow] noalloc K={K}", flush=True)
    model.evaluate_noalloc(x, z, s.cell, s.pbc, o, K=K, precision="bf16", max_edges=2000)
    torch.cuda.synchronize()
    assert torch.isnan(o["energy"]).all() and torch.isnan(o["virial"]).all()

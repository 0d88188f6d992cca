"""Decision models on weights and rows that are not finite: what the networks make of them does not depend on how many rows a
launch has (up to 256 rows a two-layer network is evaluated from registers), and a NaN probability is not below beta."""
import numpy as np
import pytest
import torch

from workloads import mlp_weights

pytestmark = pytest.mark.gpu

INF, NAN = float("inf"), float("nan")


@pytest.fixture(scope="module")
def binding():
    from paper_2409_10644_amd import binding as b
    return b


def _mlp(binding, ws, bs):
    return binding.make_mlp([torch.from_numpy(w).cuda() for w in ws], [torch.from_numpy(b).cuda() for b in bs])


def _expected(ws, bs, x):
    """The network in binary64, layer by layer: ReLU keeps a NaN."""
    with np.errstate(all="ignore"):
        for l, (w, b) in enumerate(zip(ws, bs)):
            x = np.stack([(w.astype(np.float64) * row).sum(axis=1) + b for row in x])
            if l + 1 < len(ws):
                x = np.where(x < 0, 0.0, x)
        return 1.0 / (1.0 + np.exp(-x[:, 0]))


@pytest.mark.parametrize("hidden", [1, 20, 64, 65, 512])
@pytest.mark.parametrize("what,at,value", [("weight", 0, NAN), ("weight", 0, INF), ("weight", 1, NAN), ("weight", 1, INF), ("bias", 0, NAN),
                                           ("bias", 0, -INF), ("bias", 1, INF), ("rows", 0, INF)])
def test_rows_network_few_and_many_rows(binding, hidden, what, at, value):
    rng = np.random.default_rng(hidden)
    k, V, W = 4, 2100, 16
    ws, bs = mlp_weights((k + 1, hidden, 1), seed=hidden)
    rows = rng.random((20, W, V)).astype(np.float32) / np.float32(V)
    unit = hidden // 2
    if what == "rows":
        rows[0, 3, 77] = value
    elif what == "bias":
        bs[at][unit if at == 0 else 0] = value
    else:
        ws[at][(unit, 1) if at == 0 else (0, unit)] = value
    mlp = _mlp(binding, ws, bs)
    d = torch.from_numpy(rows).cuda()
    for B in (2, 16, 20):                       # flags settled in the launch; by a second one; more rows than compute units
        feat = torch.zeros((B, W, k + 1), device="cuda")
        prob = torch.full((B, W), -7.0, device="cuda")
        stop = torch.full((B,), -7, dtype=torch.int32, device="cuda")
        binding.early_stop_distribution(mlp, B, W, V, k, d, W * V, V, 0.4, feat, prob, stop)
        torch.cuda.synchronize()
        got = prob.cpu().numpy()
        want = _expected(ws, bs, feat.cpu().numpy().reshape(B * W, k + 1).astype(np.float64)).reshape(B, W)
        assert np.array_equal(np.isnan(got), np.isnan(want)), (B, what, at, value)
        assert np.abs(np.nan_to_num(got) - np.nan_to_num(want)).max() <= 1e-5
        assert stop.tolist() == [int(np.all(got[b] < np.float32(0.4))) for b in range(B)]



@pytest.mark.parametrize("widths", [(40, 1), (260, 8, 1), (768, 70, 5, 1), (100, 300, 1)])
@pytest.mark.parametrize("what,value", [("weight", INF), ("weight", -INF), ("weight", NAN), ("row", INF)])
def test_hidden_state_network(binding, widths, what, value):
    rng = np.random.default_rng(widths[0])
    ws, bs = mlp_weights(widths, seed=widths[0])
    x = rng.standard_normal((2, 3, widths[0])).astype(np.float32)
    if what == "row":
        x[1, 2, -1] = value
    else:
        ws[0][0, -1] = value                    # the last column: what a kernel may read again beyond it
    mlp = _mlp(binding, ws, bs)
    prob = torch.full((2, 3), -7.0, device="cuda")
    stop = torch.full((2,), -7, dtype=torch.int32, device="cuda")
    binding.early_stop_hidden(mlp, 2, 3, torch.from_numpy(x).cuda(), 3 * widths[0], widths[0], 0.4, prob, stop)
    torch.cuda.synchronize()
    got = prob.cpu().numpy()
    want = _expected(ws, bs, x.reshape(6, -1).astype(np.float64)).reshape(2, 3)
    assert np.array_equal(np.isnan(got), np.isnan(want)), (widths, what, value)
    assert np.abs(np.nan_to_num(got) - np.nan_to_num(want)).max() <= 1e-5
    assert stop.tolist() == [int(np.all(got[b] < np.float32(0.4))) for b in range(2)]

"""Verification walks shared by several workgroups: chunk edges of the vocabulary, every team size, sums that a workgroup
takes from its partners and sums that it computes itself, both sampling schemes and modes; bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from workloads import DRAFT_INIT, TARGET_INIT, WORKLOADS, scaled, verify_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import gpu_helpers
    return gpu_helpers


@pytest.fixture(scope="module")
def binding():
    from paper_2409_10644_amd import binding as b
    return b


def _check(binding, oracle, H, w, mode, replacement, n_new, plans, seed):
    vi = verify_inputs(w, seed=seed, mode=mode, n_new=n_new, replacement=replacement)
    view = binding.slice_mask(binding.build_mask(w.branching), w.gamma_max)
    d = {k: H.dev(vi[k]) for k in ("p_target", "q_draft", "tokens", "u_accept", "u_sample")}
    B, V = w.B, w.V
    path, alen, new = (torch.full(s, -7, dtype=torch.int32, device="cuda") for s in ((B, w.gamma_max), (B,), (B, n_new)))
    ws_bytes = binding.verify_tree_workspace(view, mode, B, n_new)
    ws = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device="cuda")
    want = oracle.verify_tree(mode, w.branching, vi["tokens"], vi["p_target"], vi["q_draft"], vi["u_accept"], vi["u_sample"],
                              **({} if replacement else {"replacement": False}))
    for team, polls in plans:
        path.fill_(-7)
        binding.verify_tree_tuned(binding.VerifyTuning(team=team, polls=polls), view, mode, 0 if replacement else 1, B, V, d["tokens"], d["p_target"], d["q_draft"],
                                  d["p_target"].stride(0), d["q_draft"].stride(0), d["u_accept"], d["u_sample"], n_new, path, alen,
                                  new, ws)
        for a, b in zip((path, alen, new), want):
            assert np.array_equal(a.cpu().numpy(), b), (V, mode, replacement, team, polls)


@pytest.mark.parametrize("V", [7, 2047, 2048, 2049, 4100, 8191, 16384, 16385, 32768, 32769, 65543, 131072])
@pytest.mark.parametrize("mode,replacement", [(DRAFT_INIT, True), (DRAFT_INIT, False), (TARGET_INIT, True)])
def test_chunk_edges(binding, oracle, H, V, mode, replacement):
    w = scaled(WORKLOADS["cfg1"], B=3, V=V, branching=(3, 2, 2), cfg_id=120, target_sigma=1.5, draft_noise_sigma=1.0)
    _check(binding, oracle, H, w, mode, replacement, 5, ((0, 0), (1, 0), (2, 0), (16, 0), (16, -1), (16, 0)), seed=V)


def test_more_nodes_than_are_fetched_ahead(binding, oracle, H):
    w = scaled(WORKLOADS["cfg1"], B=2, V=9000, branching=(16, 16), cfg_id=121, target_sigma=1.5, draft_noise_sigma=2.0)
    _check(binding, oracle, H, w, DRAFT_INIT, True, 64, ((0, 0),), seed=1)
    _check(binding, oracle, H, w, DRAFT_INIT, False, 1, ((4, 0),), seed=2)


def test_more_teams_than_the_chip_holds(binding, oracle, H):
    w = scaled(WORKLOADS["cfg1"], B=130, V=33000, branching=(2,), cfg_id=122, target_sigma=1.5, draft_noise_sigma=2.0)
    _check(binding, oracle, H, w, DRAFT_INIT, True, 1, ((0, 0),), seed=1)

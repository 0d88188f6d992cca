"""Verification teams whose members start late and give up waiting early: more workgroups than the chip holds at once, one look
per sum, walks of many rejection rounds, so that some run several steps ahead alone; bit for bit against the oracle."""
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


@pytest.mark.parametrize("mode,B,branching,replacement", [(DRAFT_INIT, 96, (12, 2), True), (DRAFT_INIT, 96, (12, 2), False),
                                                         (TARGET_INIT, 12, (8, 6), True)])
def test_late_members(binding, oracle, H, mode, B, branching, replacement):
    w = scaled(WORKLOADS["cfg1"], B=B, V=20000, branching=branching, cfg_id=123, target_sigma=1.5, draft_noise_sigma=2.5)
    vi = verify_inputs(w, seed=5, mode=mode, n_new=3, replacement=replacement)
    view = binding.slice_mask(binding.build_mask(branching), len(branching))
    d = {k: H.dev(vi[k]) for k in ("p_target", "q_draft", "tokens", "u_accept", "u_sample")}
    path, alen, new = (torch.full(s, -7, dtype=torch.int32, device="cuda") for s in ((B, len(branching)), (B,), (B, 3)))
    ws = torch.empty(max(binding.verify_tree_workspace(view, mode, B, 3), 256), dtype=torch.uint8, device="cuda")
    want = oracle.verify_tree(mode, branching, vi["tokens"], vi["p_target"], vi["q_draft"], vi["u_accept"], vi["u_sample"],
                              **({} if replacement else {"replacement": False}))
    for polls in (1, 1, 0, 2):                  # eight workgroups of 4096 entries per walk: 768 of 512 lanes
        path.fill_(-7)
        binding.verify_tree_tuned(binding.VerifyTuning(team=16, polls=polls), view, mode, 0 if replacement else 1, B, w.V, d["tokens"],
                                  d["p_target"], d["q_draft"], d["p_target"].stride(0), d["q_draft"].stride(0), d["u_accept"], d["u_sample"],
                                  3, path, alen, new, ws)
        for a, b in zip((path, alen, new), want):
            assert np.array_equal(a.cpu().numpy(), b), polls

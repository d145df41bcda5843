"""A routed decode step's folded launches (row pass with the router's product; decision and adapter down-projection in
the gate/up launch; adapter up-projection with the down product's reduction) at the edges of their layouts, against
the oracle: token counts around the 16-, 32- and 64-row blocks, every narrow adapter rank, one to four column blocks per
gate/up workgroup, all tokens or all but one on one branch."""
import numpy as np
import pytest

from paper_2609_08189_amd import synth
from tests.parity import check_layer

pytestmark = pytest.mark.gpu


def _layer(T, d=256, d_ff=384, d_r=32, mode="budget", budget=0.3, beta=None, tiled=True):
    from paper_2609_08189_amd.device import DeviceProblem
    print(f"case T={T} d={d} d_ff={d_ff} d_r={d_r} mode={mode} budget={budget}", flush=True)
    w = synth.Workload("decode_route", "bf16", d=d, d_ff=d_ff, d_r=d_r, L_R=8, d_m=32, T=T, mode=mode, budget=budget,
                       bias="spread")
    prob = synth.make_problem(w, seed=T, layer_j=3)
    if beta is not None:
        prob.beta = np.full(T, beta, np.float32)
    dp = DeviceProblem(prob, tiled=tiled)
    dp.run_layer(3)
    check_layer(prob, dp.results(), 3)


@pytest.mark.parametrize("mode", ["budget", "threshold"])
@pytest.mark.parametrize("T", [1, 16, 17, 33, 64, 65, 129, 255, 256])
def test_token_counts(T, mode):
    _layer(T, mode=mode)


@pytest.mark.parametrize("d_r", [64, 96, 128])
@pytest.mark.parametrize("d,d_ff", [(256, 128), (1280, 1408), (2048, 4224)])
def test_ranks_and_widths(d, d_ff, d_r):
    _layer(100, d, d_ff, d_r, tiled=False)


@pytest.mark.parametrize("T,d_r,mode,tiled", [(100, 64, "budget", True), (256, 32, "threshold", False)])
@pytest.mark.parametrize("d_ff,blocks", [(4096, 1), (8192, 2), (8320, 3), (12416, 4), (16384, 4)])
def test_column_blocks(d_ff, blocks, T, d_r, mode, tiled):
    """blocks: the most 16-column blocks of W_g and W_u that one of at most 256 workgroups takes (7B: 3, 8B: 4)."""
    nb = d_ff // 16
    assert -(-nb // min(256, nb)) == blocks
    _layer(T, 256, d_ff, d_r, mode=mode, tiled=tiled)


@pytest.mark.parametrize("T", [1, 70])
@pytest.mark.parametrize("beta", [-50.0, 50.0])
def test_threshold_one_branch(T, beta):
    _layer(T, mode="threshold", beta=beta)


@pytest.mark.parametrize("budget", [0.0, 1.0 / 70, 69.0 / 70, 1.0])
def test_budget_one_branch(budget):
    """No, one, all but one and all of 70 tokens on the adapter (all: without a FFN row no launch is folded)."""
    _layer(70, budget=budget)


@pytest.mark.parametrize("T", [47, 64, 65, 256])
def test_row_pass_is_the_prefills(T):
    """A token's normalised row u (the first region of the workspace) has the same bits in a decode step, where the row
    pass shares the router product's launch, as in a call of 300 tokens with a row pass of its own."""
    import torch
    from paper_2609_08189_amd.device import DeviceProblem
    d = 4096
    u = []
    for n in (T, 300):
        w = synth.Workload("row_pass", "bf16", d=d, d_ff=128, d_r=32, L_R=8, d_m=32, T=n, mode="budget", budget=0.3)
        dp = DeviceProblem(synth.make_problem(w, seed=5, layer_j=3))
        rows = torch.randn(300, d, generator=torch.Generator().manual_seed(9)).to(torch.bfloat16).cuda()
        dp.hbar.copy_(rows[:n])
        dp.run_layer(3)
        torch.cuda.synchronize()
        u.append(dp.ws[:T * d * 2].view(torch.int16).clone())
    assert torch.equal(*u)


@pytest.mark.parametrize("T", [20, 64, 256])
@pytest.mark.parametrize("d,d_ff,d_r", [(4096, 128, 128), (2048, 8320, 64), (1280, 384, 32)])
def test_adapter_sums_are_the_prefills(d, d_ff, d_r, T):
    """A token's adapter sums u W_1^T are formed in the same order in a decode step, where they share the gate/up launch,
    as in a call of 300 tokens with launches of their own: each row of u and W_1 is [x, x], [w, -w], so a sum is only the
    rounding that its order leaves, scaled up by W_2; the gates are exactly 0 or 1."""
    import torch
    from paper_2609_08189_amd.device import DeviceProblem
    h = []
    for n in (T, 300):
        w = synth.Workload("adapter_sums", "bf16", d=d, d_ff=d_ff, d_r=d_r, L_R=8, d_m=32, T=n, mode="threshold",
                           budget=0.3, bias="spread")
        prob = synth.make_problem(w, seed=5, layer_j=3)
        prob.beta = np.where(np.arange(n) % 3 > 0, -50.0, 50.0).astype(np.float32)
        dp = DeviceProblem(prob)
        rows = torch.randn(300, d // 2, generator=torch.Generator().manual_seed(9)).to(torch.bfloat16).cuda()
        dp.hbar.copy_(torch.cat([rows, rows], 1)[:n])
        half = dp.ffn[0]["norm_w"][:d // 2].clone()
        dp.ffn[0]["norm_w"][d // 2:] = half
        w1, w2 = dp.adapter[0]["w1"], dp.adapter[0]["w2"]
        w1[:, d // 2:] = -w1[:, :d // 2]
        w2.mul_(2.0 ** 30)
        dp.run_layer(3)
        torch.cuda.synchronize()
        ad = torch.arange(T, device="cuda") % 3 > 0
        moved = dp.h_out[:T][ad] != dp.hbar[:T][ad]
        assert moved.any()
        h.append(dp.h_out[:T][ad].view(torch.int16).clone())
    assert torch.equal(*h)

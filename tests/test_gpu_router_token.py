"""The one-launch router of calls of few tokens, against the oracle: every memory form and width it takes, router
widths that leave threads idle, both sides of its token limit, the ablations, and the memory read it hands out."""
import numpy as np
import pytest

from oracle import hero_oracle as O
from paper_2609_08189_amd import synth
from tests.parity import check_layer
from tests.test_gpu_history import _oracle_problem

pytestmark = pytest.mark.gpu

BASE = synth.Workload("router_token", "bf16", d=256, d_ff=256, d_r=32, L_R=64, d_m=128, T=19, mode="threshold",
                      bias="spread")
NARROW = dict(d_s=40, d_h=29, d_a=11, d_e=192, d_p=24, d_head=64)


def _layer(w, j, history=False):
    from paper_2609_08189_amd.device import DeviceProblem
    print(f"case {w.dtype} T={w.T} d_m={w.d_m} state={w.state_dtype} j={j} history={history} abl={w.ablation}", flush=True)
    prob = synth.make_problem(w, seed=31, layer_j=j)
    dp = DeviceProblem(prob, history=history)
    dp.run_layer(j)
    check_layer(_oracle_problem(prob, j) if history else prob, dp.results(), j)


@pytest.mark.parametrize("dtype,d_m,state,history", [
    ("bf16", 32, "f32", False), ("bf16", 64, "bf16", False), ("bf16", 128, "f32", False), ("bf16", 256, "bf16", False),
    ("bf16", 256, "f32", True), ("bf16", 128, "f32", True), ("f32", 32, "f32", False), ("f32", 64, "f32", True),
    ("f32", 128, "bf16", False)])
@pytest.mark.parametrize("j", [1, 2, 40])
def test_memory_forms(dtype, d_m, state, history, j):
    _layer(BASE.replace(dtype=dtype, d_m=d_m, state_dtype=state), j, history)


@pytest.mark.parametrize("dtype,T", [("bf16", 1), ("bf16", 768), ("bf16", 769), ("f32", 2048), ("f32", 2049)])
def test_token_limit_and_narrow_router(dtype, T):
    _layer(BASE.replace(dtype=dtype, T=T, d_m=32, **NARROW), 5)


@pytest.mark.parametrize("abl", [1, 2, 4, 8, 15])
def test_ablations(abl):
    _layer(BASE.replace(ablation=abl), 3)


def test_memory_read_output():
    """c_read against the oracle's memory read at fp32's 1e-4."""
    import torch
    from paper_2609_08189_amd import hero as H
    from paper_2609_08189_amd.device import DeviceProblem
    prob = synth.make_problem(BASE, seed=33, layer_j=7)
    dp = DeviceProblem(prob)
    c = torch.full((BASE.T, BASE.d_m), float("nan"), device="cuda:0")
    st = H.hero_state(dp.S.data_ptr(), dp.zeta.data_ptr(), dp.p_hist.data_ptr(), dp.m_hist.data_ptr(), c.data_ptr())
    H.check(H.hero_routed_layer(dp.dims, 7, dp.T, dp.hbar, dp.prev1, dp.prev2, dp.h_out, st, dp.ffn_s[0], dp.router_s,
                                dp.adapter_s[0], dp.eta[6], dp.routing_s, None, dp.ws, dp.ws_bytes, dp.stream()), "layer")
    torch.cuda.synchronize()
    from tests.parity import oracle_layer
    ref = oracle_layer(prob, 7).debug["c"]
    assert np.max(np.abs(c.cpu().numpy() - ref)) <= 1e-4 * np.max(np.abs(ref))

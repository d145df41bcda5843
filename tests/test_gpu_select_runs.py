"""The run-per-thread branch decision from 1025 to 8192 tokens (runs of 4 and 8 tokens): both ends of each run length,
ragged last runs, every token on one branch, two large groups of exactly equal logits, threshold mode."""
import numpy as np
import pytest

from tests.parity import check_budget_selection, check_compaction
from tests.test_gpu_select import W, _layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("T,budget", [(1025, 0.27), (2777, 1.0), (4095, 0.0), (4096, 0.3882), (4097, 0.3882), (8191, 0.27)])
def test_budget(T, budget, ties):
    beta = np.where(np.random.default_rng(T).uniform(size=T) < 0.5, -1e10, 1e10).astype(np.float32) if ties else None
    L = _layer(W.replace(T=T, budget=budget, **({"bias": "none"} if ties else {})), seed=T % 83, beta=beta)
    check_compaction(L, T)
    check_budget_selection(L, budget, T)


@pytest.mark.parametrize("T", [1026, 4096, 5003])
def test_threshold(T):
    L = _layer(W.replace(T=T, mode="threshold", bias="bimodal_runs"), seed=3)
    check_compaction(L, T)
    np.testing.assert_array_equal(L["mask"], L["logit"] >= np.float32(0.0))
    assert L["lam"] == 0.0

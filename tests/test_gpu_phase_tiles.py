"""The large bf16 products on each tile height (128, 192 and 256 rows), chosen on the host (budget mode: the row
count is known) and on the device (threshold mode): forward and backward of a routed layer against the oracle, with
row counts off the tiles.  22 column tiles of the gate/up product: 11 row tiles of 128, 8 and 16 of 192 and 9 of 256
finish in the fewest rounds of 256 workgroups; from 257 to 1001 rows the down product's 128-row tiles split K."""
import pytest

from paper_2609_08189_amd import synth
from tests.parity import check_layer
from tests.test_gpu_backward import BF16, _run_small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["budget", "threshold"])
@pytest.mark.parametrize("T", [257, 639, 1001, 1365, 1501, 2203, 3001])
def test_layer(T, mode):
    from paper_2609_08189_amd.device import DeviceProblem
    print(f"case T={T} mode={mode}", flush=True)
    w = synth.Workload("phase", "bf16", d=256, d_ff=2816, d_r=32, L_R=8, d_m=32, T=T, mode=mode, budget=0.0)
    prob = synth.make_problem(w, seed=T, layer_j=3)
    if mode == "threshold":
        # nearly every token on the FFN branch, as with the zero budget: both count the same rows
        prob.beta = synth.normal32(T, "bias_vals", (T,), 1.0, 4.0)
    dp = DeviceProblem(prob)
    dp.run_layer(3)
    check_layer(prob, dp.results(), 3)


@pytest.mark.parametrize("known", [True, False])
@pytest.mark.parametrize("T", [1365, 2203, 3001])
def test_block_backward(T, known):
    _run_small(BF16.replace(d=256, d_ff=2816, d_r=32, T=T, budget=0.01), T, budget_mode=known)

"""The large bf16 products on each tile height (128, 192 and 256 rows), chosen on the host (budget mode: the row
count is known) and on the device (threshold mode): forward and backward of a routed layer against the oracle, with
row counts off the tiles.  With d = 256 the gate/up product (22 column tiles) takes the heights and the down product splits K
over 128-row tiles to 1001 rows and runs 128-row tiles from 1365 (257 and 639 rows: the gate/up product splits K too);
with d = 2048 the down product (8 column tiles) takes 192 and 256 rows, with its scatter."""
import pytest

from paper_2609_08189_amd import synth
from tests.parity import check_layer
from tests.phase_rule import phase_rows
from tests.test_gpu_backward import BF16, _run_small

pytestmark = pytest.mark.gpu


def _layer(T, mode, d, d_ff):
    from paper_2609_08189_amd.device import DeviceProblem
    print(f"case T={T} mode={mode} d={d} d_ff={d_ff}", flush=True)
    w = synth.Workload("phase", "bf16", d=d, d_ff=d_ff, d_r=32, L_R=8, d_m=32, T=T, mode=mode, budget=0.0)
    prob = synth.make_problem(w, seed=T, layer_j=3)
    if mode == "threshold":
        # nearly every token on the FFN branch, as with the zero budget: both count the same rows
        prob.beta = synth.normal32(T, "bias_vals", (T,), 1.0, 4.0)
    dp = DeviceProblem(prob)
    dp.run_layer(3)
    check_layer(prob, dp.results(), 3)


@pytest.mark.parametrize("mode", ["budget", "threshold"])
@pytest.mark.parametrize("T,rows", [(257, None), (639, None), (1001, 128), (1365, 128), (1501, 192), (2203, 256),
                                    (3001, 192)])
def test_layer(T, rows, mode):
    """rows: the gate/up product's tile height for the T rows of the zero budget (None: it splits K)."""
    assert rows is None or phase_rows(T, 22) == rows
    _layer(T, mode, 256, 2816)


@pytest.mark.parametrize("mode", ["budget", "threshold"])
@pytest.mark.parametrize("T,rows", [(2177, 128), (4501, 192), (7001, 256)])
def test_down_product(T, rows, mode):
    """The down product's tile height with its scatter, for the T rows of the zero budget."""
    assert phase_rows(T, 8) == rows
    _layer(T, mode, 2048, 256)


@pytest.mark.parametrize("known", [True, False])
@pytest.mark.parametrize("T,d_ff,rows", [(1365, 2816, 128), (2203, 2816, 256), (3001, 2816, 192), (3300, 16384, 192)])
def test_block_backward(T, d_ff, rows, known):
    """rows: the tile height of the gate/up recompute (3300: more than eight rounds of 192-row tiles)."""
    w = BF16.replace(d=256, d_ff=d_ff, d_r=32, T=T, budget=0.01)
    assert phase_rows(T - int(w.budget * T + 0.5), d_ff // 128, spill=True) == rows
    _run_small(w, T, budget_mode=known)

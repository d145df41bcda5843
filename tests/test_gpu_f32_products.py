"""fp32 products at the edges of their tiles: K and N off the 16-deep steps and 16- or 32-wide tiles, row pitches
that are not multiples of four (no 16-byte loads), one row, enough rows for the 32 x 32 tiles, and enough 64 x 64
tiles for the VALU ones."""
import pytest

from paper_2609_08189_amd import synth
from tests.parity import check_layer
from tests.test_gpu_backward import F32, _run_small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,d_ff,d_r", [(1, 128, 5, 1), (17, 256, 691, 15), (33, 256, 688, 16), (700, 256, 2101, 15),
                                          (700, 256, 2100, 20)])
def test_f32_layer_products(T, d, d_ff, d_r):
    """Against the oracle at fp32's 1e-4 (sums of at most 2101 products: about 1e-6)."""
    from paper_2609_08189_amd.device import DeviceProblem
    w = synth.Workload("f32_products", "f32", d=d, d_ff=d_ff, d_r=d_r, L_R=4, d_m=32, T=T, mode="budget", budget=0.27)
    print(f"case T={T} d={d} d_ff={d_ff} d_r={d_r}", flush=True)
    prob = synth.make_problem(w, seed=21, layer_j=3)
    dp = DeviceProblem(prob)
    dp.run_layer(3)
    check_layer(prob, dp.results(), 3)


@pytest.mark.parametrize("mode,budget", [("budget", 0.0), ("budget", 0.3), ("budget", 1.0), ("threshold", 0.0)])
@pytest.mark.parametrize("T,d_ff,d_r", [(1, 40, 16), (16, 41, 17), (65, 688, 5), (255, 48, 16), (256, 160, 15), (257, 48, 16)])
def test_f32_shared_launches(T, d_ff, d_r, mode, budget):
    """Calls of at most 256 tokens decide the branches inside the first of two shared launches: both branches, one
    only, row pitches with and without 16-byte loads in either product, and the first size past them."""
    from paper_2609_08189_amd.device import DeviceProblem
    print(f"case T={T} d_ff={d_ff} d_r={d_r} mode={mode} budget={budget}", flush=True)
    w = synth.Workload("f32_pairs", "f32", d=128, d_ff=d_ff, d_r=d_r, L_R=4, d_m=32, T=T, mode=mode, budget=budget,
                       bias="spread")
    prob = synth.make_problem(w, seed=T, layer_j=3)
    dp = DeviceProblem(prob)
    dp.run_layer(3)
    check_layer(prob, dp.results(), 3)


@pytest.mark.parametrize("T,d,d_ff,d_r,budget", [
    (4161, 128, 2051, 5, 0.0),       # gate/up: 66 x 33 tiles of 64, rows and columns off them
    (4095, 128, 2040, 5, 0.0),       # one column of tiles short of them
    (16385, 128, 40, 5, 1.0),        # the router's product: 257 x 8, and the adapter's up at K = 5
    (8193, 512, 41, 64, 1.0)])       # the adapter's up at K = 64
def test_f32_large_products(T, d, d_ff, d_r, budget):
    """Against the oracle at fp32's 1e-4, on both sides of where the VALU tiles take over."""
    from paper_2609_08189_amd.device import DeviceProblem
    w = synth.Workload("f32_large", "f32", d=d, d_ff=d_ff, d_r=d_r, L_R=4, d_m=32, T=T, mode="budget", budget=budget)
    print(f"case T={T} d={d} d_ff={d_ff} d_r={d_r}", flush=True)
    prob = synth.make_problem(w, seed=22, layer_j=2)
    dp = DeviceProblem(prob)
    dp.run_layer(2)
    check_layer(prob, dp.results(), 2)


def test_f32_large_backward():
    """e, the gate/up recompute and du of 4161 rows (66 x 33 tiles of 64 for the first two)."""
    _run_small(F32.replace(T=4161, d=128, d_ff=2051, budget=0.0), 15)

"""GPU parity of the MLP workloads (bf16 operands, fp32 accumulation) against the CPU
oracle with its bf16 rounding points switched on, through the C-ABI."""
import numpy as np
import pytest

import workloads
from parity_util import run_pair, assert_trace_equal, check_models

pytestmark = pytest.mark.gpu

BF16_TOL = 2e-2     # relative, stated for the bf16-input workloads
BF16_GUARD = 5e-3   # per-tensor norms; measured at most 1.2e-3 (K = 4 at the largest shape), typically 1e-5 .. 3e-4


def _check(res, tol=BF16_TOL):
    assert_trace_equal(res, 2e-3)
    # every W_l and b_l separately, element by element, weights and updates (w^T - w^0)
    check_models(res, tol, guard=BF16_GUARD)


@pytest.mark.parametrize("over,T", [
    # two layers, several row tiles per upload boundary, ragged B, d_0 not a tile multiple
    (dict(M=4096, dims=[200, 96, 10], N=8, B=40, n_slow=2, lr=1e-3), 40),
    # three layers, B = one tile, hidden = one and two tiles, 100 classes (128-wide logits)
    (dict(M=8192, dims=[256, 128, 256, 100], n_classes=100, N=8, B=128, n_slow=0, lr=5e-4), 30),
    # staleness-aware step, fixed threshold, many restarts
    (dict(M=4096, dims=[128, 64, 3], n_classes=3, N=16, B=16, n_slow=4, sa_penalty=1,
          tau_mode=1, tau_cap=1, lr=2e-3), 60),
    # everything a multiple of 256: all products take the 256 x 256 tile kernel
    (dict(M=8192, dims=[256, 256, 512, 10], N=6, B=256, K0=2, n_slow=1, lr=5e-4), 20),
    # mixed: 256-row uploads but a 128-wide hidden layer (both GEMM kernels in one round)
    (dict(M=8192, dims=[320, 128, 256, 10], N=4, B=256, n_slow=0, lr=5e-4), 15),
    # B > one tile (two row tiles per upload), Pareto times
    (dict(M=8192, dims=[384, 128, 10], N=4, B=200, n_slow=0, time_dist=1, time_param=1.5, lr=1e-3), 25),
])
def test_mlp_small(over, T):
    p = workloads.scaled_preset(3, **over)
    _check(run_pair(p, T, checkpoints=(1, 5)))


def test_cfg3_shape_prefix():
    """The 3072-512-10 workload at its real layer and batch shapes (shorter dataset), first rounds."""
    p = workloads.scaled_preset(3, M=6400)
    _check(run_pair(p, 12, checkpoints=(1,)))


def test_run_to_run_bitwise_determinism():
    import paper_2301_08895_amd as lib
    p = workloads.scaled_preset(3, M=4096, dims=[256, 128, 10], N=8, B=64, n_slow=2, lr=1e-3)
    d = workloads.make_inputs(p)
    outs = []
    for _ in range(2):
        sim = lib.Simulation(p, d)
        sim.round(30)
        outs.append((sim.model().copy(), sim.trace().copy()))
        sim.close()
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])


def test_mlp_first_round_equals_the_hand_worked_values():
    """The HIP path against tests/golden/mlp_hand_worked_first_round.txt (ReLU forward, H^T dZ, update,
    an untouched hidden layer; every value survives the bf16 narrowing exactly)."""
    import paper_2301_08895_amd as lib
    from parity_util import mlp_hand_worked_first_round
    p, d, w1 = mlp_hand_worked_first_round()
    sim = lib.Simulation(p, d)
    sim.round(1)
    got = sim.model()
    loss = float(np.int32(sim.trace()[0][10]).view(np.float32))
    sim.close()
    assert np.allclose(got, w1, rtol=0, atol=1e-7), (got, w1)
    assert abs(loss - np.log(4.0)) < 1e-6


def test_sampled_kernel_timing_changes_nothing():
    """profile = n brackets the kernels of every n-th round only: same results bit for bit, and the
    statistics say which launches the measured time covers."""
    import paper_2301_08895_amd as lib
    p = workloads.scaled_preset(3, M=2048, dims=[128, 64, 10], N=4, B=32, n_slow=1)
    d = workloads.make_inputs(p)
    runs = {}
    for prof in (0, 1, 4):
        sim = lib.Simulation(p, d, profile=prof)
        sim.round(21)
        runs[prof] = (sim.model().copy(), sim.trace().copy(), sim.kernel_stats())
        sim.close()
    for prof in (1, 4):
        assert np.array_equal(runs[prof][0], runs[0][0]) and np.array_equal(runs[prof][1], runs[0][1])
    for s0, s1, s4 in zip(*(runs[k][2] for k in (0, 1, 4))):
        assert s0["launches"] == s1["launches"] == s4["launches"] and s0["timed_launches"] == 0 and s0["total_ms"] == 0
        assert s1["timed_launches"] == s1["launches"] and s1["timed_flops"] == s1["flops"] and s1["total_ms"] > 0
        per_round = s4["launches"] // 21
        assert s4["timed_launches"] == 6 * per_round and s4["total_ms"] > 0      # rounds 0, 4, ..., 20


@pytest.mark.parametrize("over,T", [
    # contractions shorter than a ring, one valid chunk of 8 features in a k-step of 64
    (dict(M=512, dims=[8, 40, 2], n_classes=2, N=4, B=1, n_slow=0, lr=1e-3), 10),
    (dict(M=1024, dims=[72, 64, 10], N=4, B=130, n_slow=0, lr=1e-3), 10),
    # nothing a multiple of a tile, three hidden widths, a ragged last k-step in the gathered product
    (dict(M=2400, dims=[1000, 520, 300, 26], n_classes=26, N=4, B=90, n_slow=0, lr=2e-4), 6),
    # more than 128 tiles of 128 x 128 in every forward and input-gradient product; one fewer row tile: 64-wide
    (dict(M=4800, dims=[136, 1024, 1024, 10], N=17, K0=17, B=128, n_slow=0, lr=1e-4), 2),
    (dict(M=4800, dims=[136, 1024, 1024, 10], N=16, K0=16, B=128, n_slow=0, lr=1e-4), 2),
    # the transposed minibatch: the most blocks that ride with the output layer's kernel, and a launch of its own;
    # half a block of 256 columns of padding
    (dict(M=6400, dims=[1096, 64, 10], N=50, K0=50, B=100, n_slow=0, lr=2e-4), 2),
    (dict(M=6400, dims=[1096, 64, 10], N=64, K0=64, B=100, n_slow=0, lr=2e-4), 2),
    # a weight gradient long enough for 128-wide tiles (128 k-steps, 128 padded classes)
    (dict(M=12800, dims=[64, 2048, 100], n_classes=100, N=64, K0=64, B=128, n_slow=0, lr=1e-4), 2),
    # the fewest 128 x 256 tiles (512; ragged widths, a k-step with 8 valid columns), in a weight gradient
    # too (104 tiles over 128 k-steps); one column tile fewer: two 128 x 128 workgroups per CU
    (dict(M=25600, dims=[72, 1000, 1010, 10], N=128, K0=128, B=100, n_slow=0, lr=1e-4), 1),
    (dict(M=25600, dims=[72, 1650, 2040, 10], N=64, K0=64, B=120, n_slow=0, lr=1e-4), 1),
    (dict(M=25600, dims=[200, 700, 1000, 26], n_classes=26, N=60, K0=60, B=128, n_slow=0, lr=1e-4), 2),
])
def test_tile_kernel_edges(over, T):
    """The tile kernel where its remainders are: short rings, zero-filled columns of gathered rows, both tile sizes."""
    p = workloads.scaled_preset(3, **over)
    _check(run_pair(p, T, checkpoints=(1,)))


@pytest.mark.parametrize("d0,h1,h2,K,T", [
    (128, 512, 512, 64, 2),        # 2 k-steps in the first layer: no turn of the loop requests anything
    (384, 768, 512, 64, 2),        # 6 and 12
    (512, 512, 768, 64, 2),        # 8 in every product
    (768, 2048, 1024, 37, 2),      # weight gradients too, one straight from the dataset: seven ranges of 19 and one of 15
])
def test_large_tile_kernel_by_number_of_k_steps(d0, h1, h2, K, T):
    """The 256 x 256 kernel over short and odd contractions, against the oracle, and two runs bit for bit: a request that
    overtakes a reader of its place in LDS changes a handful of blocks of 16 x 16, differently each time."""
    import paper_2301_08895_amd as lib
    p = workloads.scaled_preset(3, M=64 * K, dims=[d0, h1, h2, 10], N=K, K0=K, B=256, n_slow=0, lr=1e-4)
    plan = lib.abs_mlp_round_plan(lib.make_config(p), K)
    assert plan.count("256x256") >= 4, plan
    res = run_pair(p, T, checkpoints=(1,))
    _check(res)
    d = workloads.make_inputs(p)
    runs = []
    for _ in range(2):
        sim = lib.Simulation(p, d)
        sim.round(4)
        runs.append(sim.model().copy())
        sim.close()
    assert np.array_equal(runs[0], runs[1])


@pytest.mark.parametrize("d1,C,N,B", [
    (40, 2, 3, 1),            # one block of 16 classes, two of the four wavefronts without a share of the contraction
    (200, 17, 5, 130),        # two blocks, one class in the second; an upload of eight row blocks
    (384, 64, 4, 100),        # four, all 64 padded classes in use
    (500, 65, 3, 40),         # five: classes padded to 128
    (320, 128, 32, 128),      # eight, the most rows
    (320, 128, 33, 128),      # one upload more: workgroups of 128 rows
])
def test_output_layer_of_few_rows(d1, C, N, B):
    """The output layer in workgroups of 32 rows: contractions that leave wavefronts without a share, every padding of the classes."""
    import paper_2301_08895_amd as lib
    p = workloads.scaled_preset(3, M=max(1024, N * B), dims=[64, d1, C], n_classes=C, N=N, K0=N, B=B, n_slow=0, lr=5e-4)
    assert f"logits_ce:{128 if N == 33 else 32}x" in lib.abs_mlp_round_plan(lib.make_config(p), N)
    _check(run_pair(p, 4, checkpoints=(1,)))


@pytest.mark.parametrize("dims,N,B,item", [
    ([40, 24, 3], 1, 1, "steps:64x64/1"),                      # two k-steps: shorter than the ring
    ([3072, 512, 10], 32, 100, "steps:64x64/1"),               # 64 k-steps, the most
    ([512, 128, 10], 24, 128, "steps:64x64/1"),                # 48, the most for as few as 18 tiles
    ([512, 64, 10], 33, 128, "wgrad_tile:64x64/11"),           # 66: split weight gradients, partials, an update
    ([1000, 2040, 10], 2, 60, "steps:128x128/1"),              # 144 tiles of 128 x 128, ragged in both directions
    ([2048, 2040, 26], 3, 128, "steps2:128x128/1"),            # 272: two workgroups per CU
    ([3000, 1400, 10], 24, 100, "steps_x:128x128/1"),          # the dataset in place of its transposed copy, columns beyond d_0
    ([3000, 1400, 700, 130], 22, 128, "steps_x:128x128/1"),    # ... three layers, two column tiles of classes
])
def test_steps_taken_in_the_weight_gradients(dims, N, B, item):
    """All matrices of a round stepped in one launch, at both tile sizes and with either first operand."""
    import paper_2301_08895_amd as lib
    p = workloads.scaled_preset(3, M=max(512, 2 * N * B), dims=dims, n_classes=dims[-1], N=N, K0=N, B=B, n_slow=0, lr=1e-4)
    assert item in lib.abs_mlp_round_plan(lib.make_config(p), N).split()
    _check(run_pair(p, 3, checkpoints=(1,)))


@pytest.mark.parametrize("h,C", [(512, 10), (512, 100), (768, 200)])          # one, two and four k-steps over the classes
def test_input_gradient_of_the_output_layer_on_large_tiles(h, C):
    import paper_2301_08895_amd as lib
    p = workloads.scaled_preset(3, M=64 * 64, dims=[64, h, C], n_classes=C, N=64, K0=64, B=256, n_slow=0, lr=1e-4)
    assert "dgrad:256x256/1" in lib.abs_mlp_round_plan(lib.make_config(p), 64).split()
    _check(run_pair(p, 2, checkpoints=(1,)))
    d = workloads.make_inputs(p)
    runs = []
    for _ in range(2):
        sim = lib.Simulation(p, d)
        sim.round(4)
        runs.append(sim.model().copy())
        sim.close()
    assert np.array_equal(runs[0], runs[1])

"""The kernels an MLP round launches, by shape (abs_mlp_round_plan: host only): the dispatch rules at the places where a
wrong one costs time rather than results."""
import paper_2301_08895_amd as lib
import workloads


def _plan(dims, N, B, K, U=1):
    p = workloads.scaled_preset(3, M=max(4096, 4 * N), dims=dims, n_classes=dims[-1], N=N, B=B, K0=K, n_slow=0, U=U)
    return lib.abs_mlp_round_plan(lib.make_config(p), K).split()


def test_the_transposed_minibatch_is_written_right_before_its_reader():
    """A launch of its own (8192 x 2048: 1024 blocks) stands behind the backward pass, next to the weight gradient."""
    names = [item.split(":")[0] for item in _plan([2000, 1024, 1024, 10], 64, 128, 64)]
    at = names.index("gather_t")
    assert names[at + 1].startswith("wgrad") and names[at - 1].startswith("dgrad"), names

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


def _items(dims, N, B, K, kind, U=1):
    return [item for item in _plan(dims, N, B, K, U) if item.startswith(kind)]


def test_tiles_of_products_with_more_tiles_than_cus():
    """Uploads of 128 rows: 128 x 256 tiles from 512 of them on, below that pairs of 128 x 128 workgroups per CU, and one
    workgroup per CU only while there is no second one."""
    wide = [1024, 2048, 2048, 10]
    assert _items(wide, 128, 128, 64, "fwd") == ["fwd_wide:128x256/1"] * 2
    assert _items(wide, 128, 128, 64, "dgrad") == ["dgrad_wide:128x256/1"] * 2
    assert _items(wide, 128, 128, 63, "fwd") == ["fwd_tile2:128x128/1"] * 2          # 504 tiles of 128 x 256
    assert _items(wide, 128, 128, 17, "dgrad") == ["dgrad_tile2:128x128/1"] * 2      # 272 tiles of 128 x 128
    assert _items(wide, 128, 128, 16, "fwd") == ["fwd_tile:128x128/1"] * 2           # 256
    # gathered rows that are no whole k-steps stay off the 256 x 256 kernel whatever the uploads' rows
    assert _items([3000, 2048, 2048, 100], 128, 256, 32, "fwd")[0] == "fwd_wide:128x256/1"
    # weight gradients: 25 k-steps for each of two workgroups per CU, in few splits
    assert _items([3200, 2048, 10], 128, 128, 64, "wgrad")[0] == "wgrad_wide:128x256/2"
    assert _items([3200, 512, 10], 128, 128, 128, "wgrad")[0].startswith("wgrad_tile2:128x128/")


def test_tiles_of_local_steps_follow_the_number_of_uploads():
    """The contraction of a local step is not cut beyond the uploads: few uploads of many rows keep 64-wide tiles."""
    assert _items([512, 2048, 100], 4, 4096, 2, "wgrad", U=2)[:2] == ["wgrad_step_tile:64x64/2"] * 2
    assert _items([64, 2048, 100], 64, 128, 64, "wgrad", U=2)[:2] == ["wgrad_step_tile2:128x128/64"] * 2
    assert _items([512, 2048, 100], 4, 4096, 4, "wgrad", U=2)[1] == "wgrad_step_tile:128x128/4"      # 4 x 16 x 4 workgroups


def test_rows_of_the_output_layer_beyond_96_classes():
    """A CU holds one 32-row workgroup there: a short contraction takes 128 rows once they and the riding transposed minibatch are
    more than a workgroup per CU, and fewer blocks of it ride."""
    def ce(dims, K):
        plan = _plan(dims, 32, 128, K)
        at = [i for i, item in enumerate(plan) if item.startswith("logits_ce:")][0]
        return plan[at].split("x")[0], "with_gather_t:64x256/1" in plan
    for classes, dims in ((100, [880, 73]), (128, [880, 256])):
        assert ce(dims + [classes], 21) == ("logits_ce:32", True)        # 84 + 168 workgroups
        assert ce(dims + [classes], 22) == ("logits_ce:128", True)       # 88 + 176
    assert ce([880, 73, 96], 32) == ("logits_ce:32", True)
    assert ce([880, 300, 100], 32) == ("logits_ce:32", True)
    assert ce([512, 200, 100], 32) == ("logits_ce:32", True)             # 128 + 128
    assert ce([3072, 512, 100], 21) == ("logits_ce:32", True)            # 504 blocks ride
    assert ce([3072, 512, 100], 22) == ("logits_ce:32", False)           # 528
    assert ce([3072, 256, 100], 22) == ("logits_ce:32", False)
    assert ce([3072, 512, 96], 32) == ("logits_ce:32", True)             # 768

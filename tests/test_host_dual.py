"""The scheduler's rule for batches of few MFMA tiles whose page re-reads are large: both kernels' work
lists, the groups still reported as the vector kernels' (no GPU)."""
import numpy as np
import pytest

from paper_2311_03285_amd import slora


def plan_of(H, n_slots, groups, **options):
    """groups: (rank, tokens) per adapter."""
    n = sum(2 * n_slots * r for r, _ in groups)
    pool = slora.pool_init(H, n, slora.F16, None, n_slots, max(r for r, _ in groups))
    for a, (r, _) in enumerate(groups):
        slora.adapter_alloc(pool, a, r, n_slots)
    for k, v in options.items():
        slora.set_option(pool, k, v)
    plan = slora.batch_plan(pool, np.repeat(np.arange(len(groups)), [t for _, t in groups]))
    info = slora.plan_info(plan)
    slora.plan_destroy(plan)
    slora.pool_destroy(pool)
    return info


@pytest.mark.parametrize("groups,options,dual", [
    ([(64, 512)], {}, True),                                   # 16 tiles, 537 MB read again
    ([(64, 28)], {}, False),                                   # 29 MB
    ([(64, 29)], {}, True),                                    # 34 MB
    ([(64, 29), (8, 1)], {}, False),                           # beside a group of few tokens: 128 MB
    ([(64, 120), (8, 1)], {}, False),                          # 126 MB
    ([(64, 121), (8, 1)], {}, True),                           # 130 MB
    ([(64, 512)], {"mfma_min_tiles": 16}, False),              # enough tiles: the MFMA kernels for every call
    ([(64, 512)], {"mfma_min_tokens": 1 << 40}, False),        # disabled
])
def test_rule(groups, options, dual):
    info = plan_of(4096, 4, groups, **options)
    on_mfma = options.get("mfma_min_tiles") == 16
    assert info["groups_mfma"] == (len(groups) if on_mfma else 0)
    assert (info["mfma_expand_items"] > 0) == (dual or on_mfma)
    if not on_mfma:                                            # every group keeps its vector items
        assert info["vec_shrink_items"] == sum((t + 3) // 4 * ((r + 3) // 4) for r, t in groups)


@pytest.mark.parametrize("H,n_slots,groups,options,fused,tiles", [
    (4096, 4, [(64, 512), (8, 1)], {"mfma_min_tokens": 1, "fuse_decode": 2}, 1, 16),
    (8192, 8, [(64, 512)] + [(64, 4)] * 4 + [(64, 1)] * 120, {"mfma_min_tokens": 4}, 124, 16),
    (4096, 4, [(64, 512), (8, 3)], {"mfma_min_tokens": 1, "fuse_decode": 0}, 0, 17),
])
def test_no_group_is_in_the_one_launch_list_and_the_mfma_lists(H, n_slots, groups, options, fused, tiles):
    """An apply runs both: such a group's delta would be added twice."""
    info = plan_of(H, n_slots, groups, **options)
    assert info["groups_fused"] == fused
    assert info["mfma_expand_items"] == tiles * (H // 256)

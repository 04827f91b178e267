"""Infinite weights in the rank-split expand: a number of ranks that fills its last eight exactly is not followed by another
rank's row times zero, which would turn an infinite last row of B into NaN."""
import numpy as np
import pytest
import torch

from paper_2311_03285_amd import slora

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("y16", [False, True])
@pytest.mark.parametrize("rank", [8, 16, 24, 32, 40, 48, 64, 72, 128])
def test_last_row_of_b(dtype, y16, rank):
    H, toks = 1032, (1, 2, 3, 4, 6, 7, 8)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rank)
    pages = torch.randn((2 * rank, H), device="cuda", generator=gen)
    pages[:rank] /= H ** 0.5
    pages[rank - 1].abs_()                       # v of the last rank is positive: x is
    pages[-1, :H // 2] = float("inf")
    pages = pages.to(dtype)
    pool = slora.pool_init(H, 2 * rank, slora.F16 if dtype == torch.float16 else slora.BF16, pages.data_ptr(), 1, rank)
    slora.set_option(pool, "fuse_decode", 0)
    slora.adapter_load(pool, 0, rank, np.arange(2 * rank, dtype=np.int32).reshape(1, 2, rank))
    down, up = pages[:rank].double(), pages[rank:].double()
    for T in toks:
        x = torch.rand((T, H), device="cuda", generator=gen).to(dtype)
        y = torch.zeros((T, H), device="cuda", dtype=dtype if y16 else torch.float32)
        plan = slora.batch_plan(pool, np.zeros(T, dtype=np.int32), None)
        (slora.lora_apply_multi_y16 if y16 else slora.lora_apply_multi)(plan, [0], [x.data_ptr()], [y.data_ptr()])
        torch.cuda.synchronize()
        slora.plan_destroy(plan)
        assert torch.isposinf(y[:, :H // 2]).all(), (T, y[:, :H // 2])
        got, ref = y[:, H // 2:].double(), (x.double() @ down.t()) @ up[:, H // 2:]
        # sums of 1032 + 128 products in 32 bits; a 16-bit y is rounded once, by half a unit in the last place
        bar = 2e-6 if not y16 else (2.0 ** -11 if dtype == torch.float16 else 2.0 ** -8)
        assert float((got - ref).norm() / ref.norm()) <= bar, T
    slora.pool_destroy(pool)

"""GPU parity of the MFMA kernels' tilings: runs of 32-token tiles that an expand workgroup walks
with B in registers (up to 128 ranks, in stages of 32) or streamed (more), and items of the shrink
taken whole or in halves and quarters of their tokens - at the edges of tiles, stages and runs.

Integer-valued inputs have exact sums (every partial sum is an integer below 2^24), so the result is
compared bit for bit; 16-bit y as elsewhere: the correctly rounded oracle result.
"""
import numpy as np
import pytest
import torch

from paper_2311_03285_amd import slora, synth
from paper_2311_03285_amd.harness import DeviceWorkload, bits_to_device
from gpu_util import assert_close, gpu_slot, oracle_slot
from test_gpu_mfma import MFMA_ALL, route
from test_gpu_y16 import assert_y16_close, gpu_y16, oracle_y16

pytestmark = pytest.mark.gpu

RANKS = (1, 32, 33, 64, 65, 96, 97, 128, 129)
LENS = (300, 257, 288, 320, 353, 65, 64, 33, 500)   # tiles of 32: 10 9 9 10 12 3 2 2 16, the last one full or not


def tiles_workload(seed, dtype, H, n_slots, repeat=1, **kw):
    lens = LENS * repeat
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ids = np.repeat(np.tile(np.random.default_rng(seed).permutation(len(RANKS)), repeat), lens).astype(np.int32)
    return synth.make_workload("tiles", seed, H, dtype, 2 * n_slots * sum(RANKS) + 64, n_slots, RANKS, ids, seg, **kw)


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("H,n_slots,repeat", [(72, 1, 1), (264, 4, 1), (1000, 8, 1), (1000, 8, 3)])
def test_runs_and_subtiles_integer_inputs_bit_exact(dtype, H, n_slots, repeat):
    w = tiles_workload(600 + H + repeat, dtype, H, n_slots, repeat, int_valued=True)
    with DeviceWorkload(w, real_adapters="all", max_rank=max(RANKS)) as dw:
        route(dw.pool, MFMA_ALL)
        plan = dw.plan()
        assert slora.plan_info(plan)["groups_mfma"] == len(RANKS)
        slot = n_slots - 1
        assert np.array_equal(gpu_slot(dw, slot, plan).astype(np.float64), oracle_slot(w, slot))


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_runs_of_tiles_with_16_bit_y(dtype):
    w = tiles_workload(650, dtype, 1000, 8)
    with DeviceWorkload(w, real_adapters="all", max_rank=max(RANKS)) as dw:
        route(dw.pool, MFMA_ALL)
        got = gpu_y16(dw, [5])[0]
        ref, exact = oracle_y16(w, 5)
        assert_y16_close(got, ref, exact, w.y16_bits(5), w.dtype, "runs of tiles")


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("few", [0, 3])
def test_small_batch_with_both_kernels_lists(dtype, few):
    """Fewer tiles than mfma_min_tiles, but many page re-reads: applies to fp32 y take the MFMA kernels (in
    shares of H), 16-bit y and the two-stage calls the vector kernels; an expand after an apply still
    works, and the static scratch serves both."""
    lens = [190, 17, 40] + [1] * few
    ranks = [128, 129, 65] + [5] * few
    ids = np.repeat(np.arange(len(lens)), lens).astype(np.int32)
    w = synth.make_workload("dual", 670 + few, 4096, dtype, 4 * 2 * sum(ranks) + 32, 4, ranks, ids)
    with DeviceWorkload(w, real_adapters="all", max_rank=129) as dw:
        plan = dw.plan()
        info = slora.plan_info(plan)
        assert info["groups_mfma"] == 0 and info["mfma_expand_items"] > 0 and info["split_tiles"] > 0
        for slot in (0, 3):
            rel, _ = assert_close(gpu_slot(dw, slot, plan), oracle_slot(w, slot), f"slot {slot}")
            assert rel <= 5e-6, rel
        want = gpu_slot(dw, 1, plan)
        x, y = dw.x_dev(1), dw.y_dev(1)
        slora.lora_apply_multi_static(plan, [1], [x.data_ptr()], [y.data_ptr()])
        assert np.array_equal(y.cpu().numpy(), want)           # the same kernels, the other scratch
        y2 = dw.y_dev(1)
        slora.lora_expand(plan, [1], [y2.data_ptr()])          # v is still where the apply left it
        assert np.array_equal(y2.cpu().numpy(), want)
        y3 = dw.y_dev(1)
        slora.lora_shrink(plan, [1], [x.data_ptr()])           # two-stage: the vector kernels
        slora.lora_expand(plan, [1], [y3.data_ptr()])
        two = y3.cpu().numpy()
        assert_close(two, oracle_slot(w, 1), "two-stage")
        got = gpu_y16(dw, [1], plan)[0]
        ref, exact = oracle_y16(w, 1)
        assert_y16_close(got, ref, exact, w.y16_bits(1), w.dtype, "dual, 16-bit y")
    with DeviceWorkload(w, real_adapters="all", max_rank=129) as dw:
        slora.set_option(dw.pool, "mfma_min_tokens", 1 << 40)  # vector kernels throughout
        assert np.array_equal(gpu_slot(dw, 1, dw.plan()), two)
        assert np.array_equal(gpu_y16(dw, [1])[0], got)


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_one_launch_groups_beside_mfma_groups_are_added_once(dtype):
    """Groups of one to four tokens that the options allow on the MFMA kernels and on the one-launch kernel."""
    ids = np.repeat([0, 1, 2, 3], [290, 1, 4, 5]).astype(np.int32)
    w = synth.make_workload("once", 690, 4096, dtype, 2 * 2 * (128 + 8 + 16 + 8) + 16, 2, [128, 8, 16, 8], ids, int_valued=True)
    with DeviceWorkload(w, real_adapters="all") as dw:
        route(dw.pool, 1, 32)
        slora.set_option(dw.pool, "fuse_decode", 2)
        plan = dw.plan()
        info = slora.plan_info(plan)
        assert info["groups_fused"] == 2 and info["mfma_expand_items"] > 0
        xs, ys = [dw.x_dev(s) for s in (0, 1)], [dw.y_dev(s) for s in (0, 1)]
        slora.lora_apply_multi(plan, [0, 1], [t.data_ptr() for t in xs], [t.data_ptr() for t in ys])
        for s in (0, 1):
            assert np.array_equal(ys[s].cpu().numpy().astype(np.float64), oracle_slot(w, s))


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_fp32_apply_captured_after_a_16_bit_apply(dtype):
    """The plan's first apply sizes the scratch of both kernel families: the other one may follow under capture."""
    ids = np.repeat([0, 1], [190, 40]).astype(np.int32)
    w = synth.make_workload("capture", 695, 4096, dtype, 2 * 2 * (128 + 65) + 16, 2, [128, 65], ids)
    with DeviceWorkload(w, real_adapters="all") as dw:
        plan = dw.plan()
        x = [dw.x_dev(s) for s in (0, 1)]
        y16 = [bits_to_device(w.y16_bits(s), dw.device) for s in (0, 1)]
        y0 = [dw.y_dev(s) for s in (0, 1)]
        y = [t.clone() for t in y0]
        xp, yp = [t.data_ptr() for t in x], [t.data_ptr() for t in y]
        st = torch.cuda.Stream()
        torch.cuda.synchronize()
        slora.lora_apply_multi_y16(plan, [0, 1], xp, [t.data_ptr() for t in y16], st)
        torch.cuda.synchronize()
        before = slora.pool_stats(dw.pool)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            slora.lora_apply_multi(plan, [0, 1], xp, yp, torch.cuda.current_stream())
        assert slora.pool_stats(dw.pool) == before
        for rep in range(3):
            for k in (0, 1):
                y[k].copy_(y0[k])
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            got = [t.cpu().numpy() for t in y]
            for k in (0, 1):
                assert np.array_equal(got[k], gpu_slot(dw, k)), (rep, k)
                rel, _ = assert_close(got[k], oracle_slot(w, k), f"replay {rep}, slot {k}")
                assert rel <= 5e-6, rel

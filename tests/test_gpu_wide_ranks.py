"""GPU parity of the MFMA expand for adapters of more than 128 ranks: up to 256 with B in registers and V in two halves of
four 32-rank stages, beyond that streamed - at the edges of stages, on both sides of each limit, with column ranges that leave
wavefronts without columns, runs of one and of several tiles per workgroup.

Integer-valued inputs have exact sums (below 2^24), so they are compared bit for bit; rows whose ranks differ in size
by 2^12 from one 128-rank block to the next meet the change of scale between the halves."""
import numpy as np
import pytest
import torch

from paper_2311_03285_amd import slora, synth
from paper_2311_03285_amd.harness import DeviceWorkload, bits_to_device
from gpu_util import assert_close, gpu_slot, oracle_slot
from test_gpu_mfma import MFMA_ALL, route
from test_gpu_y16 import assert_y16_close, gpu_y16, oracle_y16

pytestmark = pytest.mark.gpu

RANKS = (129, 130, 160, 161, 192, 224, 225, 256, 257)
LENS = (300, 257, 33, 320, 1, 65, 32, 31, 500)


def wide_workload(seed, dtype, H, n_slots, **kw):
    seg = np.concatenate([[0], np.cumsum(LENS)]).astype(np.int32)
    ids = np.repeat(np.random.default_rng(seed).permutation(len(RANKS)), LENS).astype(np.int32)
    return synth.make_workload("wide", seed, H, dtype, 2 * n_slots * sum(RANKS) + 64, n_slots, RANKS, ids, seg, **kw)


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("H,n_slots", [(72, 1), (264, 4), (1000, 2)])
def test_integer_inputs_bit_exact(dtype, H, n_slots):
    w = wide_workload(900 + H, dtype, H, n_slots, int_valued=True)
    with DeviceWorkload(w, real_adapters="all") as dw:
        route(dw.pool, MFMA_ALL)
        plan = dw.plan()
        assert slora.plan_info(plan)["groups_mfma"] == len(RANKS)
        slot = n_slots - 1
        assert np.array_equal(gpu_slot(dw, slot, plan).astype(np.float64), oracle_slot(w, slot))


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_both_types_of_y(dtype):
    w = wide_workload(950, dtype, 1000, 2)
    with DeviceWorkload(w, real_adapters="all") as dw:
        route(dw.pool, MFMA_ALL)
        rel, _ = assert_close(gpu_slot(dw, 1), oracle_slot(w, 1), "fp32 y")
        assert rel <= 5e-6, rel
        got = gpu_y16(dw, [1])[0]
        ref, exact = oracle_y16(w, 1)
        assert_y16_close(got, ref, exact, w.y16_bits(1), w.dtype, "16-bit y")


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("small_first", [True, False])
def test_halves_of_different_size(dtype, small_first):
    """A's rows of one 128-rank block are 2^12 smaller than the other's: v of the two halves carries scales 2^12 apart."""
    H, T, rank, td = 512, 70, 200, torch.float16 if dtype == synth.F16 else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(17)
    pages = torch.randn((2 * rank, H), device="cuda", generator=gen)
    pages[:rank] /= H ** 0.5
    block = slice(0, 128) if small_first else slice(128, rank)
    pages[block] *= 2.0 ** -12
    pages, x = pages.to(td), torch.randn((T, H), device="cuda", generator=gen).to(td)
    y = torch.zeros((T, H), device="cuda")
    pool = slora.pool_init(H, 2 * rank, slora.F16 if dtype == synth.F16 else slora.BF16, pages.data_ptr(), 1, rank)
    route(pool, MFMA_ALL)
    slora.adapter_load(pool, 0, rank, np.arange(2 * rank, dtype=np.int32).reshape(1, 2, rank))
    plan = slora.batch_plan(pool, np.zeros(T, dtype=np.int32), None)
    slora.lora_apply(plan, 0, x.data_ptr(), y.data_ptr())
    torch.cuda.synchronize()
    ref = (x.double() @ pages[:rank].double().t()) @ pages[rank:].double()
    rel = float((y.double() - ref).norm() / ref.norm())
    slora.plan_destroy(plan)
    slora.pool_destroy(pool)
    assert rel <= 2e-6, rel   # sums of 512 + 200 products in 32 bits


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_runs_of_several_tiles(dtype):
    """Three tiles per workgroup in a call of eight slots, one in calls of one: the same bits.  The last column range is 72
    wide, so two of its four wavefronts only copy V."""
    H, n_slots, lens = 584, 8, (700, 257, 33, 640, 65, 96, 1400, 31, 1200)
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ids = np.repeat(np.random.default_rng(960).permutation(len(RANKS)), lens).astype(np.int32)
    w = synth.make_workload("runs", 960, H, dtype, 2 * n_slots * sum(RANKS) + 64, n_slots, RANKS, ids, seg)
    with DeviceWorkload(w, real_adapters="all") as dw:
        route(dw.pool, MFMA_ALL)
        plan = dw.plan()
        tiles, ranges = [-(-n // 32) for n in lens], -(-H // 256)
        assert slora.plan_info(plan)["mfma_expand_items"] == sum(tiles) * ranges
        run = sum(tiles) * ranges * n_slots // 1024          # tiles of a run; a run is not shared out from 1024 workgroups on
        assert run == 3 and sum(-(-t // run) for t in tiles) * ranges * n_slots >= 1024 >= 3 * sum(-(-t // run) for t in tiles) * ranges
        slots = list(range(n_slots))
        xs = [dw.x_dev(s) for s in slots]
        for y16 in (False, True):
            def apply(which):
                ys = [bits_to_device(w.y16_bits(s), dw.device) if y16 else dw.y_dev(s) for s in which]
                fn = slora.lora_apply_multi_y16 if y16 else slora.lora_apply_multi
                fn(plan, which, [xs[s].data_ptr() for s in which], [y.data_ptr() for y in ys])
                torch.cuda.synchronize()
                return ys

            many = apply(slots)
            for s in slots:
                assert torch.equal(many[s], apply([s])[0]), (y16, s)
            got = many[-1].cpu().numpy()
            if y16:
                ref, exact = oracle_y16(w, n_slots - 1)
                assert_y16_close(got.view(np.uint16).reshape(w.T, w.H), ref, exact, w.y16_bits(n_slots - 1), dtype, "16-bit y")
            else:
                rel, _ = assert_close(got, oracle_slot(w, n_slots - 1), "fp32 y")
                assert rel <= 5e-6, rel


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("H", [1016, 1024])
def test_single_tiles(dtype, H):
    """One tile per workgroup, on both sides of the width at which 16-bit y takes the halves."""
    w = wide_workload(970 + H, dtype, H, 1)
    with DeviceWorkload(w, real_adapters="all") as dw:
        route(dw.pool, MFMA_ALL)
        rel, _ = assert_close(gpu_slot(dw, 0), oracle_slot(w, 0), "fp32 y")
        assert rel <= 5e-6, rel
        ref, exact = oracle_y16(w, 0)
        assert_y16_close(gpu_y16(dw, [0])[0], ref, exact, w.y16_bits(0), w.dtype, "16-bit y")

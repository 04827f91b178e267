"""GPU parity of the one-launch kernels for small decode batches: bit-identical to the two kernels (the
same sums in the same order), at the edges of what they take - ranks around a block of the rank-split
expand, 1 to 4 tokens per group, one and several column ranges, a ragged last one.  Plain calls hand v over between
workgroups; calls with the static scratch and captured ones take the kernel in which every workgroup computes v."""
import numpy as np
import pytest
import torch

from paper_2311_03285_amd import slora, synth
from paper_2311_03285_amd.harness import DeviceWorkload, bits_to_device
from gpu_util import assert_close, gpu_slot, oracle_slot
from test_gpu_y16 import gpu_y16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def side():
    return torch.cuda.Stream()


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("H,ranks", [(64, (1, 8, 32, 31)), (520, (7, 16, 17, 32)), (1000, (8, 9, 32, 1)), (4096, (1, 8, 7, 16))])
def test_one_launch_is_bit_identical_to_two(dtype, H, ranks, side):
    toks = [4, 3, 2, 1] if H < 4096 else [4, 4, 3, 2]          # 4096: rank x H x tokens up to 128 Ki
    ids = np.repeat([0, 1, 2, 3], toks).astype(np.int32)
    ids = np.concatenate([ids, [-1]])[np.random.default_rng(H).permutation(ids.size + 1)].astype(np.int32)
    w = synth.make_workload("small", 700 + H, H, dtype, 2 * 2 * sum(ranks) + 8, 2, ranks, ids)
    with DeviceWorkload(w, real_adapters="all", max_rank=32) as dw:
        plan = dw.plan()
        slots = [0, 1]
        xs = [dw.x_dev(s) for s in slots]
        xp = [t.data_ptr() for t in xs]
        one, two = [dw.y_dev(s) for s in slots], [dw.y_dev(s) for s in slots]
        slora.lora_apply_multi(plan, slots, xp, [t.data_ptr() for t in one])
        after = [dw.y_dev(s) for s in slots]
        slora.lora_expand(plan, slots, [t.data_ptr() for t in after])       # v of the apply is in memory
        slora.lora_shrink(plan, slots, xp)
        slora.lora_expand(plan, slots, [t.data_ptr() for t in two])
        torch.cuda.synchronize()
        for a, b, c in zip(one, two, after):
            assert torch.equal(a, b) and torch.equal(c, b)
        assert slora.pool_stats(dw.pool)["hand_overs"] == 1
        # the kernel for small batches: with the static scratch (and an expand of the v that it leaves there), and captured
        one, after = [dw.y_dev(s) for s in slots], [dw.y_dev(s) for s in slots]
        slora.lora_apply_multi_static(plan, slots, xp, [t.data_ptr() for t in one])
        slora.lora_expand(plan, slots, [t.data_ptr() for t in after])
        torch.cuda.synchronize()
        for a, b, c in zip(one, two, after):
            assert torch.equal(a, b) and torch.equal(c, b)
        for y16 in (False, True):
            apply, expand = (slora.lora_apply_multi_y16, slora.lora_expand_y16) if y16 else (slora.lora_apply_multi, slora.lora_expand)
            one, two = [[bits_to_device(w.y16_bits(s), dw.device) if y16 else dw.y_dev(s) for s in slots] for _ in range(2)]
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=side):
                apply(plan, slots, xp, [t.data_ptr() for t in one], torch.cuda.current_stream().cuda_stream)
            for _ in range(3):
                g.replay()
                torch.cuda.synchronize()
                slora.lora_shrink(plan, slots, xp)
                expand(plan, slots, [t.data_ptr() for t in two])
                torch.cuda.synchronize()
                for a, b in zip(one, two):
                    assert torch.equal(a, b), y16
        assert slora.pool_stats(dw.pool)["hand_overs"] == 1
        for s in slots:
            rel, _ = assert_close(gpu_slot(dw, s, plan), oracle_slot(w, s), f"slot {s}")
            assert rel <= 2e-6, rel
        got = gpu_y16(dw, slots, plan)
        ys = [bits_to_device(w.y16_bits(s), dw.device) for s in slots]
        slora.lora_shrink(plan, slots, xp)
        slora.lora_expand_y16(plan, slots, [t.data_ptr() for t in ys])
        torch.cuda.synchronize()
        for g, t in zip(got, ys):
            assert np.array_equal(g, t.cpu().numpy().view(np.uint16).reshape(g.shape))


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_y_in_the_buffer_of_x(dtype, side):
    """x += (x A) B in place, on a batch small enough for one launch, against the call with an x of its own; plain and captured."""
    ids = np.array([0, 1, 1, 2], np.int32)
    w = synth.make_workload("in-place", 790, 4096, dtype, 2 * 2 * 40 + 8, 2, [16, 8, 16], ids)
    with DeviceWorkload(w, real_adapters="all") as dw:
        plan = dw.plan()
        xs = [dw.x_dev(s) for s in (0, 1)]
        apart, place = [x.clone() for x in xs], [x.clone() for x in xs]
        slora.lora_apply_multi_y16(plan, [0, 1], [t.data_ptr() for t in xs], [t.data_ptr() for t in apart])
        slora.lora_apply_multi_y16(plan, [0, 1], [t.data_ptr() for t in place], [t.data_ptr() for t in place])
        torch.cuda.synchronize()
        for x, a, p in zip(xs, apart, place):
            assert torch.equal(a, p) and not torch.equal(a, x)
        assert slora.pool_stats(dw.pool)["hand_overs"] == 1   # not the one in place
        for into in ([x.clone() for x in xs], None):
            y = [x.clone() for x in xs]
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=side):
                slora.lora_apply_multi_y16(plan, [0, 1], [t.data_ptr() for t in (y if into is None else xs)],
                                           [t.data_ptr() for t in (into or y)], torch.cuda.current_stream().cuda_stream)
            g.replay()
            torch.cuda.synchronize()
            for a, p in zip(apart, into or y):
                assert torch.equal(a, p)

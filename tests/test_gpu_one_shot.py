"""One-shot calls: a plan of one call sends its lists on the call's own stream.  Adapters loaded right before the call (their page
lists travel on another stream), lists of one item and of thousands, calls that alternate between streams - the bits
are those of a plan and an apply."""
import numpy as np
import pytest
import torch

from paper_2311_03285_amd import slora, synth
from paper_2311_03285_amd.harness import DeviceWorkload
from gpu_util import gpu_slot

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [(1,), (1, 2, 3, 40), (200, 1, 513, 70)])
@pytest.mark.parametrize("load_late", [False, True])
def test_one_shot_is_a_plan_and_an_apply(lens, load_late):
    ranks = [8, 64, 130, 17][:len(lens)]
    ids = np.repeat(np.arange(len(lens)), lens).astype(np.int32)
    w = synth.make_workload("once", 990 + len(lens), 1000, synth.F16, 3 * 2 * sum(ranks) + 16, 1, ranks, ids)
    with DeviceWorkload(w, real_adapters="all") as dw:
        want = gpu_slot(dw, 0)
        x = dw.x_dev(0)
        streams = [torch.cuda.Stream() for _ in range(2)]
        ys = [dw.y_dev(0) for _ in range(6)]
        torch.cuda.synchronize()
        for k, y in enumerate(ys):
            if load_late:   # the same pages in another order of loading: every page list moves in the arena
                torch.cuda.synchronize()
                for a in range(len(ranks)):
                    slora.adapter_unload(dw.pool, a)
                for a in np.roll(np.arange(len(ranks)), k):
                    slora.adapter_load(dw.pool, int(a), ranks[a], w.adapter_page_list(int(a)))
            slora.lora_shrink_expand(dw.pool, 0, x.data_ptr(), ids, None, y.data_ptr(), streams[k % 2])
        torch.cuda.synchronize()
        for y in ys:
            assert np.array_equal(y.cpu().numpy(), want)

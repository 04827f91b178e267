"""GPU parity of the MFMA kernels' tilings: runs of 32-token tiles that an expand workgroup walks
with B in registers (up to 128 ranks, in stages of 32) or streamed (more), and items of the shrink
taken whole or in halves and quarters of their tokens - at the edges of tiles, stages and runs.

Integer-valued inputs have exact sums (every partial sum is an integer below 2^24), so the result is
compared bit for bit; 16-bit y as elsewhere: the correctly rounded oracle result.
"""
import numpy as np
import pytest

from paper_2311_03285_amd import slora, synth
from paper_2311_03285_amd.harness import DeviceWorkload
from gpu_util import gpu_slot, oracle_slot
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

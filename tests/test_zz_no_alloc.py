"""The entry point that allocates nothing (v in the library's static scratch) against the entry
point it is a variant of: same plan, same inputs, results bit for bit, on two calls in a row of
which the second is smaller; and the size limit is enforced before anything is enqueued."""
import numpy as np
import pytest
import torch

from paper_2311_03285_amd import slora, synth
from paper_2311_03285_amd.harness import DeviceWorkload, bits_to_device
from gpu_util import assert_close, oracle_slot

pytestmark = pytest.mark.gpu


def mixed(seed, dtype, lens, decode, H=1000, ranks=(8, 40, 0, 17, 64, 128, 3), n_slots=3):
    """Prefill segments of the given lengths (MFMA path) plus single decode tokens (vector path)."""
    g = np.random.default_rng(seed)
    seg_ad = list(g.integers(0, len(ranks), size=len(lens))) + list(g.integers(-1, len(ranks), size=decode))
    lens = list(lens) + [1] * decode
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ids = np.repeat(np.asarray(seg_ad, dtype=np.int32), lens)
    return synth.make_workload("no-alloc", seed, H, dtype, 4096, n_slots, ranks, ids, seg)


def both_ways(dw, w, slots):
    plan = dw.plan()
    xs = [bits_to_device(w.x_bits(s), dw.device) for s in slots]
    y_a = [torch.from_numpy(w.y_in(s)).to(dw.device) for s in slots]
    y_b = [t.clone() for t in y_a]
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    slora.lora_apply_multi(plan, slots, [t.data_ptr() for t in xs], [t.data_ptr() for t in y_a], st)
    before = slora.pool_stats(dw.pool)
    slora.lora_apply_multi_static(plan, slots, [t.data_ptr() for t in xs], [t.data_ptr() for t in y_b], st)
    assert slora.pool_stats(dw.pool) == before
    st.synchronize()
    for k, s in enumerate(slots):
        a, b = y_a[k].cpu().numpy(), y_b[k].cpu().numpy()
        assert np.array_equal(a, b), f"slot {s}: static-scratch result differs from the allocating entry point"
        assert_close(b, oracle_slot(w, s), f"slot {s} vs oracle", rel_bar=5e-6)


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_static_scratch_matches_the_allocating_entry_point_twice_in_a_row(dtype):
    big = mixed(1201, dtype, lens=(70, 33, 150), decode=40)
    small = mixed(1202, dtype, lens=(20,), decode=9, H=512)
    with DeviceWorkload(big, real_adapters="all") as dw:
        slora.set_option(dw.pool, "mfma_min_tiles", 1)
        both_ways(dw, big, [0, 1, 2])
    with DeviceWorkload(small, real_adapters="all") as dw:      # smaller input: stale scratch beyond it
        slora.set_option(dw.pool, "mfma_min_tiles", 1)
        both_ways(dw, small, [2, 0])


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_static_scratch_matches_where_the_mfma_form_of_a_small_batch_exceeds_it(dtype):
    """Few tiles of a very high rank: the MFMA form (operand fragments, partial sums) of eight slots is larger than
    the static scratch, that of one slot is not."""
    w = synth.make_workload("wide", 1210, 1024, dtype, 8 * 2 * 1024 + 32, 8, [1024], np.zeros(512, dtype=np.int32))
    with DeviceWorkload(w, real_adapters="all", max_rank=1024) as dw:
        assert 8 * slora.plan_info(dw.plan())["scratch_bytes_per_slot"] > slora.STATIC_SCRATCH_BYTES
        both_ways(dw, w, list(range(8)))
        both_ways(dw, w, [6])


def test_static_scratch_rejects_a_batch_beyond_its_size():
    H, T, r = 64, 2100, 1024
    w = synth.make_workload("too-big", 5, H, synth.F16, 4096, 1, [r], np.zeros(T, dtype=np.int32))
    with DeviceWorkload(w, real_adapters="all", max_rank=r) as dw:
        plan = dw.plan()
        info = slora.plan_info(plan)
        need8 = 8 * info["tokens"] * info["v_stride"] * 4
        assert need8 > slora.STATIC_SCRATCH_BYTES
        x = bits_to_device(w.x_bits(0), dw.device)
        ys = [torch.zeros((T, H), dtype=torch.float32, device=dw.device) for _ in range(8)]
        with pytest.raises(slora.SloraError) as e:
            slora.lora_apply_multi_static(plan, [0] * 8, [x.data_ptr()] * 8, [t.data_ptr() for t in ys])
        assert e.value.code == slora.ERANGE and "static scratch" in str(e.value)
        torch.cuda.synchronize()
        assert not any(bool(t.any()) for t in ys)               # nothing was enqueued
        # one slot fits (8.6 MB) and gives the right answer
        slora.lora_apply_multi_static(plan, [0], [x.data_ptr()], [ys[0].data_ptr()])
        torch.cuda.synchronize()
        assert_close(ys[0].cpu().numpy(), oracle_slot(w, 0, y_in=np.zeros((T, H), np.float32)), "one slot", rel_bar=5e-6)

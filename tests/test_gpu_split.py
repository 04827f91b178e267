"""GPU parity of the rank-split vector kernels: whole sums in a wavefront up to 32 ranks, shared ones beyond, blocks of
8 ranks or (one or two tokens left over) 16, and the larger items that calls of many workgroups take (shrink: 8
tokens x 16 pages in pieces of 2048 elements; expand: 16 tokens of up to 32 ranks, 8 of more, with fmaf or the 4x4x1 matrix instruction).  Ranks and tokens per group at the edges of all
of these.  Who forms a sum never changes its bits."""
import numpy as np
import pytest
import torch

from paper_2311_03285_amd import slora, synth
from paper_2311_03285_amd.harness import DeviceWorkload, bits_to_device
from gpu_util import assert_close, gpu_slot, oracle_slot
from test_gpu_y16 import assert_y16_close, gpu_y16, oracle_y16

pytestmark = pytest.mark.gpu

RANKS = (1, 8, 9, 16, 17, 32, 33, 40, 64, 65, 100, 130)
TOKENS = (17, 5, 33, 6, 19, 18, 7, 9, 10, 4, 2, 1)


def crowd(H, dtype, ranks=RANKS, tokens=TOKENS):
    ids = np.concatenate([np.repeat(np.arange(len(ranks)), tokens), [-1, -1]])
    ids = ids[np.random.default_rng(H).permutation(ids.size)].astype(np.int32)
    return synth.make_workload("crowd", 800 + H, H, dtype, 2 * 8 * sum(ranks) + 8, 8, ranks, ids)   # calls of eight slots


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("H", [1032, 2056, 3080, 4096, 5128])   # half a piece, one and a chunk, one and a half, two, two and a half; the expand's larger items from 3080 on
def test_larger_items_are_bit_identical(H, dtype):
    w = crowd(H, dtype)
    with DeviceWorkload(w, real_adapters="all") as dw:
        plan = dw.plan()
        info = slora.plan_info(plan)
        assert info["groups_mfma"] == 0 and info["vec_shrink_items"] < 1400 <= 8 * info["vec_shrink_items"]
        assert (8 * info["vec_expand_items"] >= 2000) == (H >= 3080)
        xs = [dw.x_dev(s) for s in (0, 1)]
        slots = [0, 1] * 4
        for y16 in (False, True):
            def new(s):
                return bits_to_device(w.y16_bits(s), dw.device) if y16 else dw.y_dev(s)

            def two_kernels(which, ys):
                ptrs = [t.data_ptr() for t in ys]
                slora.lora_shrink(plan, which, [xs[s].data_ptr() for s in which])
                (slora.lora_expand_y16 if y16 else slora.lora_expand)(plan, which, ptrs)

            many, applied, one = [new(s) for s in slots], [new(s) for s in slots], [new(s) for s in (0, 1)]
            two_kernels(slots, many)
            apply = slora.lora_apply_multi_y16 if y16 else slora.lora_apply_multi
            apply(plan, slots, [xs[s].data_ptr() for s in slots], [t.data_ptr() for t in applied])
            for s in (0, 1):
                two_kernels([s], [one[s]])
            torch.cuda.synchronize()
            for s, got, got2 in zip(slots, many, applied):
                assert torch.equal(got, one[s]) and torch.equal(got2, one[s]), (y16, s)
            for s in (0, 1):
                if y16:
                    ref, exact = oracle_y16(w, s)
                    assert_y16_close(one[s].cpu().numpy().view(np.uint16).reshape(w.T, w.H), ref, exact, w.y16_bits(s), dtype, f"slot {s}")
                else:
                    rel, _ = assert_close(one[s].cpu().numpy(), oracle_slot(w, s), f"slot {s}")
                    assert rel <= 2e-6, rel


@pytest.mark.parametrize("y16", [False, True])
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("tokens", [(5, 6, 7, 8), (8, 9, 12, 13), (12, 16, 17, 30)])   # none, some and most of the items on the matrix instruction
def test_larger_items_of_few_ranks(dtype, tokens, y16):
    """Adapters of at most 32 ranks: calls of eight slots (larger items) against calls of one (small ones), and the first slot against the oracle."""
    ranks = (1, 4, 8, 9, 15, 16, 17, 24, 25, 32)
    w = crowd(5128, dtype, ranks * 2, (tokens * 5)[:20])
    with DeviceWorkload(w, real_adapters="all") as dw:
        plan = dw.plan()
        info = slora.plan_info(plan)
        assert info["groups_mfma"] == 0 and info["vec_expand_items"] < 2000 <= 8 * info["vec_expand_items"]
        x = [dw.x_dev(s) for s in range(8)]
        new = lambda s: bits_to_device(w.y16_bits(s), dw.device) if y16 else dw.y_dev(s)
        shrink_expand = slora.lora_expand_y16 if y16 else slora.lora_expand
        many, one = [new(s) for s in range(8)], [new(s) for s in range(8)]
        slora.lora_shrink(plan, list(range(8)), [t.data_ptr() for t in x])
        shrink_expand(plan, list(range(8)), [t.data_ptr() for t in many])
        for s in range(8):
            slora.lora_shrink(plan, [s], [x[s].data_ptr()])
            shrink_expand(plan, [s], [one[s].data_ptr()])
        torch.cuda.synchronize()
        for a, b in zip(many, one):
            assert torch.equal(a, b)
        if y16:
            ref, exact = oracle_y16(w, 0)
            assert_y16_close(many[0].cpu().numpy().view(np.uint16).reshape(w.T, w.H), ref, exact, w.y16_bits(0), dtype, "slot 0")
        else:
            rel, _ = assert_close(many[0].cpu().numpy(), oracle_slot(w, 0), "slot 0")
            assert rel <= 2e-6, rel



@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("H", [520, 2056])
def test_one_and_two_tokens(dtype, H):
    """Items of one and two tokens on both sides of 16 and 32 ranks, of a window of 64 and of blocks of 16."""
    ranks = (16, 17, 24, 31, 32, 33, 48, 64, 65, 80, 128, 130)
    ids = np.concatenate([np.arange(12), np.arange(0, 12, 2)]).astype(np.int32)     # every other adapter: two
    ids = ids[np.random.default_rng(H).permutation(ids.size)]
    w = synth.make_workload("few", 870 + H, H, dtype, 2 * 2 * sum(ranks) + 8, 2, ranks, ids)
    with DeviceWorkload(w, real_adapters="all") as dw:
        plan = dw.plan()
        rel, _ = assert_close(gpu_slot(dw, 1, plan), oracle_slot(w, 1), "fp32 y")
        assert rel <= 2e-6, rel
        got = gpu_y16(dw, [1], plan)[0]
        ref, exact = oracle_y16(w, 1)
        assert_y16_close(got, ref, exact, w.y16_bits(1), dtype, "16-bit y")


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_larger_items_beside_groups_of_both_families(dtype):
    """A crowd of small groups and a few of many tokens that are in both kernel families' lists: an apply to fp32 y serves those
    on the MFMA kernels, 16-bit y and the two-stage calls everything on the vector kernels - with the larger items each time."""
    H, n_slots = 3080, 8
    ranks = [8, 9, 17, 32, 33, 40, 64, 100] * 3 + [40, 17]
    toks = [5 + g % 8 for g in range(24)] + [600, 19]
    ids = np.repeat(np.arange(26), toks)[np.random.default_rng(5).permutation(sum(toks))].astype(np.int32)
    w = synth.make_workload("both", 880, H, dtype, 2 * n_slots * sum(ranks) + 8, n_slots, ranks, ids)
    few = torch.from_numpy(ids < 24)
    quads = [-(-t // 4) for t in toks[:24]]
    assert 8 * sum(q * -(-r // 4) for q, r in zip(quads, ranks)) >= 1400 and 8 * 7 * sum(quads) >= 2000
    with DeviceWorkload(w, real_adapters="all") as dw:
        plan = dw.plan()
        info = slora.plan_info(plan)
        assert info["groups_mfma"] == 0 and info["mfma_expand_items"] > 0   # both forms
        slots = list(range(n_slots))
        xs = [dw.x_dev(s) for s in slots]
        xp = [x.data_ptr() for x in xs]
        for y16 in (False, True):
            def new(s):
                return bits_to_device(w.y16_bits(s), dw.device) if y16 else dw.y_dev(s)

            expand = slora.lora_expand_y16 if y16 else slora.lora_expand
            applied, two, one = [new(s) for s in slots], [new(s) for s in slots], [new(s) for s in slots]
            (slora.lora_apply_multi_y16 if y16 else slora.lora_apply_multi)(plan, slots, xp, [y.data_ptr() for y in applied])
            slora.lora_shrink(plan, slots, xp)
            expand(plan, slots, [y.data_ptr() for y in two])
            for s in slots:
                slora.lora_shrink(plan, [s], [xp[s]])
                expand(plan, [s], [one[s].data_ptr()])
            torch.cuda.synchronize()
            for s in slots:
                a, t, o = (v[s].reshape(w.T, w.H).cpu() for v in (applied, two, one))
                assert torch.equal(t, o), (y16, s)
                if y16:
                    assert torch.equal(a, o), s
                else:   # the others' sums are formed in another order
                    assert torch.equal(a[few], o[few]) and not torch.equal(a, o), s
            if not y16:
                rel, _ = assert_close(applied[3].cpu().numpy(), oracle_slot(w, 3), "applied")
                assert rel <= 2e-6, rel

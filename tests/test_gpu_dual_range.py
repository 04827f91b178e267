"""Batches of few MFMA tiles whose applies to fp32 y take the MFMA kernels (see mfma_min_tiles): v = x*A is
carried there with the 24 bits and the range that the vector kernels give it - very large sums, infinite
and NaN ones, and rows whose entries differ by many powers of two.  Plain numpy in 64 bits beside it."""
import numpy as np
import pytest
import torch

from paper_2311_03285_amd import slora

pytestmark = pytest.mark.gpu

H = 4096


class Batch:
    """One adapter, T tokens, one slot: numpy inputs (values of the 16-bit type) on the GPU."""

    def __init__(self, dtype, x, A, B, y):
        tt = torch.float16 if dtype == slora.F16 else torch.bfloat16
        r = A.shape[0]
        self.keep = [torch.from_numpy(a.astype(np.float32)).to(tt).cuda() for a in (x, np.concatenate([A, B]))]
        self.x, pages = self.keep
        self.y = torch.from_numpy(y.astype(np.float32)).cuda()
        self.pool = slora.pool_init(H, 2 * r, dtype, pages.data_ptr(), 1, r)
        slora.adapter_load(self.pool, 0, r, np.arange(2 * r))
        self.plan = slora.batch_plan(self.pool, np.zeros(x.shape[0], np.int32))
        info = slora.plan_info(self.plan)
        assert info["groups_mfma"] == 0 and info["mfma_expand_items"] > 0

    def apply(self):
        y = self.y.clone()
        slora.lora_apply(self.plan, 0, self.x.data_ptr(), y.data_ptr())
        torch.cuda.synchronize()
        return y.cpu().numpy()

    def close(self):
        slora.plan_destroy(self.plan)
        slora.pool_destroy(self.pool)


def result(dtype, x, A, B, y):
    b = Batch(dtype, x, A, B, y)
    got = b.apply()
    b.close()
    return got


@pytest.mark.parametrize("dtype", [slora.F16, slora.BF16])
@pytest.mark.parametrize("rank", [64, 100, 160])
def test_sums_of_any_size_are_exact(dtype, rank):
    """Powers of two with exact sums, |v| from 2^-18 to 2^42: each token of one size, the second half of the
    ranks 2^28 times the first."""
    T = 130
    x = np.exp2((np.arange(T) % 32) - 16.0)[:, None] * np.ones((1, H))
    A = np.exp2(np.arange(rank) % 2 + np.where(np.arange(rank) < rank // 2, -14.0, 14.0))[:, None] * np.ones((1, H))
    B = np.zeros((rank, H))
    B[np.arange(rank), np.arange(rank) * 7] = 0.5
    same = result(dtype, x, A, B, np.zeros((T, H))) == (x @ A.T) @ B
    assert same.all()


@pytest.mark.parametrize("dtype", [slora.F16, slora.BF16])
@pytest.mark.parametrize("rank", [64, 128, 160])
@pytest.mark.parametrize("where", ["x", "A"])
def test_infinite_and_nan_sums(dtype, rank, where):
    """An infinite v gives infinite sums, NaN where it meets a zero or another sign; an infinity in x stays in its
    token's row, one in A in its rank."""
    g = np.random.default_rng(rank)
    T = 150
    x = g.integers(-2, 3, size=(T, H)).astype(np.float64)
    A = g.integers(-1, 2, size=(rank, H)).astype(np.float64)
    B = g.integers(-1, 2, size=(rank, H)).astype(np.float64)
    B[:, :H // 2] = g.integers(1, 3, size=(rank, H // 2))     # no zero and no other sign: infinite sums stay infinite
    x[:, 5:8] = A[:, 5:8] = 1
    if where == "x":
        x[10, 5], x[20, 5], x[30, 6] = np.inf, -np.inf, np.nan
        x[40, 6:8] = np.inf, -np.inf
    else:
        A[rank // 2, 5] = np.inf
    with np.errstate(invalid="ignore"):
        want = (x @ A.T) @ B + 1.0
    got = result(dtype, x, A, B, np.ones((T, H))).astype(np.float64)
    assert np.isinf(want).any() and np.isnan(want).any()
    nan = np.isnan(want)
    same = np.where(nan, np.isnan(got), got == want)
    assert same.all()


def quantized(a, dtype):
    return torch.from_numpy(a.astype(np.float32)).to(torch.float16 if dtype == slora.F16 else torch.bfloat16).double().numpy()


def against_the_vector_kernels(dtype, x, A, B):
    """The bar is the vector kernels' error on the same batch (their v is fp32) plus 1e-7.  That error itself is up
    to 4e-6 where A or B holds subnormal binary16 values (their dot product drops bits of those)."""
    want = (x @ A.T) @ B
    b = Batch(dtype, x, A, B, np.zeros(x.shape))
    mfma = b.apply()
    y = b.y.clone()
    slora.lora_shrink(b.plan, [0], [b.x.data_ptr()])          # two-stage calls: the vector kernels
    slora.lora_expand(b.plan, [0], [y.data_ptr()])
    torch.cuda.synchronize()
    vec = y.cpu().numpy()
    b.close()
    rel = [np.linalg.norm(v - want) / np.linalg.norm(want) for v in (mfma, vec)]
    assert rel[1] <= 5e-6 and rel[0] <= rel[1] + 1e-7, rel


@pytest.mark.parametrize("dtype", [slora.F16, slora.BF16])
@pytest.mark.parametrize("rank", [64, 160])
@pytest.mark.parametrize("spread", [12, 22, 30])
def test_rows_of_very_different_entries(dtype, rank, spread):
    """Rank j of A is small by 2^-k and of B large by 2^k, k up to the spread: every rank counts for as much as
    the others.  (30: the small values' leading pieces are subnormal in binary16.)"""
    g = np.random.default_rng(spread)
    T = 150
    k = np.exp2(np.round(np.linspace(0, spread, rank)))[:, None]
    x, A, B = g.standard_normal((T, H)), g.standard_normal((rank, H)) * 256 / k, g.standard_normal((rank, H)) * k / 2.0**18
    against_the_vector_kernels(dtype, *(quantized(a, dtype) for a in (x, A, B)))


@pytest.mark.parametrize("log2", [-54, -40, 40, 55])
def test_bfloat16_sums_of_extreme_size(log2):
    """x and A of 2^log2, B back to ordinary results where bfloat16 can: v of 2^-102 to 2^116 in three pieces (which end
    at 2^-133: v keeps its 24 bits down to 2^-109)."""
    g = np.random.default_rng(log2 + 100)
    x, A, B = g.standard_normal((150, H)), g.standard_normal((64, H)), g.standard_normal((64, H))
    x, A, B = (quantized(a * 2.0**e, slora.BF16) for a, e in ((x, log2), (A, log2), (B, -2 * log2)))
    against_the_vector_kernels(slora.BF16, x, A, B)


@pytest.mark.parametrize("dtype", [slora.F16, slora.BF16])
@pytest.mark.parametrize("rank", [60, 128, 160])
def test_16_bit_expand_after_an_fp32_apply(dtype, rank):
    """It reads v as that apply left it, in pieces.  Binary16: the sum from zero, added to y and rounded once, which is
    the fp32 result added and rounded; bfloat16 starts from y, so a few of the sums round differently."""
    g = np.random.default_rng(rank + 7)
    T, tt = 150, torch.float16 if dtype == slora.F16 else torch.bfloat16
    x, A, B = (quantized(a, dtype) for a in (g.standard_normal((T, H)), g.standard_normal((rank, H)) / 64, g.standard_normal((rank, H)) / 8))
    b = Batch(dtype, x, A, B, np.zeros((T, H)))
    delta = torch.from_numpy(b.apply()).cuda()
    y = torch.from_numpy(g.standard_normal((T, H)).astype(np.float32)).cuda().to(tt)
    want = (y.float() + delta).to(tt)
    slora.lora_expand_y16(b.plan, [0], [y.data_ptr()])
    torch.cuda.synchronize()
    b.close()
    differ = (y != want).float().mean().item()
    assert differ <= (0.0 if dtype == slora.F16 else 1e-3), differ
    assert (y.float() - want.float()).abs().max().item() <= 2.0**-4

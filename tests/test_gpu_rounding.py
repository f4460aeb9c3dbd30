"""The last step of every product, FP32 -> BF16 (arXiv 2503.13565, section 3.4.3: FP32 accumulation, BF16 output), bit for bit: sums
that are exact in any order, rounded by the kernels' convert instruction, against round to nearest, ties to even, in integers."""
import numpy as np
import pytest
import torch

from paper_2503_13565_amd import binding

pytestmark = pytest.mark.gpu

from helpers import DEV  # noqa: E402

K, TRIPLES = 128, 42


def values(m):
    """FP32 bit patterns [m, TRIPLES]: ties to even and to odd codes, their neighbours, carries into the exponent, the largest BF16 and
    what rounds to infinity, anything else; both signs."""
    rng = np.random.default_rng(m)
    high = rng.integers(0x2000, 0x6000, (m, TRIPLES)).astype(np.uint32) << 16
    low = rng.choice(np.array([0x0000, 0x0001, 0x7FFF, 0x8000, 0x8001, 0xFFFF, 0x4000, 0xC000], np.uint32), (m, TRIPLES))
    bits = high | np.where(rng.random((m, TRIPLES)) < 0.3, rng.integers(0, 1 << 16, (m, TRIPLES)).astype(np.uint32), low)
    bits[:, 0], bits[:, 1], bits[:, 2], bits[:, 3] = 0x3F7F8000, 0x3F808000, 0x3F818000, 0x3FFFFFFF
    bits[:, 4], bits[:, 5], bits[:, 6], bits[:, 7] = 0x7F7F7FFF, 0x7F7F8000, 0x7F7FFFFF, 0x7F7EFFFF
    return bits | rng.integers(0, 2, (m, TRIPLES)).astype(np.uint32) << 31


def rounded(bits):
    return ((bits + 0x7FFF + (bits >> 16 & 1)) >> 16).astype(np.uint16)


def three_parts(bits):
    """BF16 numbers that add up to each value exactly, in any order: its 24 bits, eight at a time."""
    v, parts = bits.view(np.float32).astype(np.float64), []
    for _ in range(3):
        p = (v.astype(np.float32).view(np.uint32) & 0xFFFF0000).view(np.float32)      # towards zero
        parts.append(p)
        v = v - p
    assert not v.any()
    return np.stack(parts, axis=2)


def operands(m, n):
    """x [m, K] and weights [n, K] of ones and zeros: output (r, c) is value (r, c % TRIPLES)."""
    bits = values(m)
    x = np.zeros((m, K), np.float32)
    x[:, :3 * TRIPLES] = three_parts(bits).reshape(m, -1)
    w = np.zeros((n, K), np.float32)
    for i in range(3):
        w[np.arange(n), 3 * (np.arange(n) % TRIPLES) + i] = 1.0
    return (torch.from_numpy(x).to(torch.bfloat16).to(DEV), torch.from_numpy(w).to(torch.bfloat16).to(DEV),
            rounded(bits)[:, np.arange(n) % TRIPLES])


def same(y, want, what):
    torch.cuda.synchronize()
    got = y.cpu().view(torch.int16).numpy().view(np.uint16)
    bad = np.argwhere(got != want)
    assert bad.size == 0, "%s: %d differ, first at %r: %04x, want %04x" % (
        what, len(bad), tuple(bad[0]), got[tuple(bad[0])], want[tuple(bad[0])])


@pytest.mark.parametrize("m,n", [(1, 100), (1, 2049), (1, 40000), (2, 2050), (2, 100), (3, 131), (5, 2049), (16, 4100), (64, 18577), (100, 19938), (300, 2051)])
def test_results_are_rounded_to_nearest_ties_to_even(m, n):
    x, w, want = operands(m, n)
    q, s = binding.mxfp4_direct_cast(w)
    same(binding.mxfp4_woq_gemm(x, q, s), want, "mxfp4")
    same(binding.mxfp4_woq_gemm(x, q, s, path=binding.PATH_VALU_CVT), want, "general")
    same(binding.mxfp4_woq_gemm(x, q, s, path=binding.PATH_MFMA), want, "tiles")
    same(binding.mxfp4_woq_gemm_tiled(x, binding.mxfp4_tile_repack(q, s)), want, "tile-major")
    zero = torch.zeros((m, n + 3), dtype=torch.bfloat16, device=DEV)
    same(binding.mxfp4_woq_gemm_fused(x, q, s, residual=zero[:, :n]), want, "with a residual")
    same(binding.mxfp4_bf16_gemm(x, w), want, "bf16")
    same(binding.mxfp4_e4m3_woq_gemm(x, *binding.mxfp4_e4m3_direct_cast(w)), want, "e4m3")
    same(binding.mxfp4_e2m3_woq_gemm(x, *binding.mxfp4_e2m3_direct_cast(w)), want, "e2m3")
    # (ternary codes are summed as twos and halved: the largest values, columns 4 to 7 of 42, overflow on the way in some kernels)
    cols = np.arange(n)[(np.arange(n) % TRIPLES < 4) | (np.arange(n) % TRIPLES > 7)]
    y = binding.mxfp4_fmt_woq_gemm(binding.FMT_T2, x, *binding.mxfp4_fmt_direct_cast(binding.FMT_T2, w))
    same(y[:, torch.from_numpy(cols).to(DEV)], want[:, cols], "ternary")


@pytest.mark.parametrize("m,n", [(1, 2049), (2, 100), (5, 2049), (64, 18577)])
def test_subnormal_results_stay(m, n):
    # the product is zero; bias and residual of either sign add up to a multiple of the smallest BF16 number
    g = torch.Generator().manual_seed(m)
    x = torch.zeros((m, K), dtype=torch.bfloat16, device=DEV)
    q, s = binding.mxfp4_direct_cast(torch.ones((n, K), dtype=torch.bfloat16, device=DEV))
    bias = torch.randint(1, 0x80, (n,), generator=g, dtype=torch.int16)
    res = torch.randint(1, 0x80, (m, n), generator=g, dtype=torch.int16)
    res[torch.rand((m, n), generator=g) < 0.5] += -0x8000
    total = bias.view(torch.bfloat16).double() + res.view(torch.bfloat16).double()
    want = total.float().to(torch.bfloat16)
    assert torch.equal(want.double(), total)
    y = binding.mxfp4_woq_gemm_fused(x, q, s, bias=bias.view(torch.bfloat16).to(DEV), residual=res.view(torch.bfloat16).to(DEV))
    same(y, want.view(torch.int16).numpy().view(np.uint16), "subnormal")

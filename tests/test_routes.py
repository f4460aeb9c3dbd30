"""The rules of csrc/routes.h on both sides of their lines, on the CPU: which calls take the block kernel and which stay on
the kernels that were measured faster for them (256 compute units, 160 KiB of LDS)."""
import ctypes
import os
import re
import subprocess

import pytest

from block_sizes import BLOCK_SIZES

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_13565_amd", "csrc")

RULES = r"""
#include "routes.h"
#include "sum_chains.h"
#include "block_ways.h"
using namespace mxfp4;
extern "C" int ways(int kind, int wk, int mf, int nf)               // 1: the direct form, 2: the one through registers
{
    return wide::has_direct((wide::Kind)kind, wk, mf, nf) + 2 * wide::has_registers((wide::Kind)kind, wk, mf, nf);
}
extern "C" int direct(int kind, int wk, int mf, int nf, int k, int tiles_m, int pick)
{
    return wide::takes_direct((wide::Kind)kind, wk, mf, nf, k, tiles_m, pick != 0);
}
extern "C" int mx(int m, int n, int k, int fits, int split, int tiled, int fused, int pick)
{
    return wide_preferred({m, n, k, 256, fits != 0, split != 0, tiled != 0, fused != 0, pick != 0});
}
extern "C" int format(int m, int n, int k, int bits, int tiles)
{
    return wide_format_preferred(m, n, k, bits, false, tiles != 0, 256, 160 * 1024);
}
extern "C" int e2m3(int m, int n, int k) { return wide_format_preferred(m, n, k, 6, true, true, 256, 160 * 1024); }
extern "C" int bf16(int m, int n, int k, int tiles)
{
    return wide_bf16_preferred(m, n, k, tiles != 0, 256, 160 * 1024);
}
extern "C" int cuts(int bits, int wm, int wn, int wk, int mf, int nf, int m, int n, int k)
{
    return wide::cuts_enough(bits, wm, wn, wk, mf, nf, m, n, k, 256);
}
extern "C" int workgroups(int rows, int n, int k) { return bf16_workgroups_per_unit(rows, n, k, 256, 160 * 1024); }
extern "C" int ragged(int m, int n, int k) { return wide_ragged_preferred(m, n, k, 256, 160 * 1024); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("routes")
    (d / "routes.cpp").write_text(RULES)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "routes.cpp"),
                           "-o", str(d / "routes.so")])
    return ctypes.CDLL(str(d / "routes.so"))


# (m, n, k, form): form of w = workspace, t = tile-major, f = fused, p = pick
SLOWER = [                                                  # us per launch on the other kernels -> in blocks
    (3, 16, 65536, ""), (3, 2048, 24576, "w"), (5, 1000, 49152, ""), (8, 4096, 65536, ""),        # 26.3 -> 34.1, ...
    (8, 6144, 65536, "w"), (5, 24000, 24576, "w"), (5, 18432, 12288, "wf"),
    (9, 16, 16384, "w"), (12, 1000, 16384, "w"), (16, 36864, 4096, ""), (16, 4096, 1536, ""),
    (17, 16, 65536, "w"), (32, 256, 65536, "w"), (17, 1000, 65536, "w"), (48, 16, 65536, "w"), (64, 16, 65536, "w"),
    (8, 4096, 65536, "tw"), (5, 1000, 16384, "tw"), (3, 256, 24576, "t"), (8, 6144, 28672, "tw"),
    (9, 16, 28672, "tw"), (16, 1000, 11008, "tw"), (9, 2560, 2048, "t"), (16, 16384, 28672, "tw"),
    (17, 16, 28672, "tw"), (32, 1000, 65536, "tw"), (48, 16, 32768, "tw"), (64, 16, 49152, "tw"),
    (5, 256, 24576, "wp"), (8, 1000, 20480, "wp"), (5, 1000, 12288, "twp"), (8, 256, 11008, "twp"), (3, 2048, 20480, "wf"),
    (8, 18432, 24576, "f"), (4, 2048, 24576, "f"), (17, 500, 32768, "w"), (32, 3000, 65536, "w"), (16, 5000, 11008, "w"),
]
FASTER = [
    (32, 12288, 4096, "w"), (17, 16, 128, ""), (509, 22016, 4096, ""), (64, 4096, 65536, "w"), (32, 2048, 28672, "w"),
    (8, 4096, 11008, "w"), (8, 4096, 11008, "t"), (5, 12288, 14336, ""), (5, 24000, 65536, "t"), (8, 8192, 11008, "w"),
    (9, 4096, 11008, "w"), (16, 12288, 14336, "w"), (16, 1000, 11008, ""), (9, 22016, 4096, "f"), (16, 8192, 1024, "t"),
    (16, 24000, 65536, "tw"), (9, 8192, 20480, "tw"), (17, 256, 65536, ""), (96, 16, 49152, "w"), (16, 18432, 4096, "f"),
    (16, 18432, 4096, ""), (16, 4096, 512, ""), (3, 57344, 128, ""), (8, 16, 128, "tw"),
    (8, 12288, 11008, "wp"), (5, 300, 11008, "wp"), (5, 300, 11008, "twp"), (8, 8192, 14336, "wf"), (5, 16, 11008, "f"), (16, 32000, 11008, "tw"),
]


def asked(rules, m, n, k, form):
    width = 4 if m <= 4 else 8 if m <= 8 else 16
    fits = (k // 128 + 3) // 4 * 1024 * width + 16384 <= 160 * 1024       # the rows of a pass and the waves' partial tiles
    return bool(rules.mx(m, n, k, int(fits), int("w" in form), int("t" in form), int("f" in form), int("p" in form)))


@pytest.mark.parametrize("m,n,k,form", SLOWER)
def test_calls_that_were_slower_in_blocks(rules, m, n, k, form):
    assert not asked(rules, m, n, k, form)


@pytest.mark.parametrize("m,n,k,form", FASTER)
def test_calls_that_are_faster_in_blocks(rules, m, n, k, form):
    assert asked(rules, m, n, k, form)


def test_rows_that_the_other_kernels_take_in_one_pass_stay(rules):
    for m in range(3, 9):
        for n in (1, 16, 4096, 64000):
            assert not asked(rules, m, n, 4096, "") and not asked(rules, m, n, 4096, "tw")


@pytest.mark.parametrize("m,n,k,form,blocks", [
    # one pass of the tiles, three to eight rows
    (3, 4096, 1024, "", True), (8, 4096, 1152, "", False), (5, 1000, 5248, "", True), (4, 1000, 5248, "", False),
    (5, 1000, 5248, "tw", False), (3, 8192, 4096, "", True), (8, 12288, 3584, "f", True), (4, 12288, 3584, "", False), (5, 12288, 4224, "f", True),
    (4, 20480, 4352, "", True), (4, 20480, 5120, "", False), (5, 22016, 4096, "f", True), (8, 28672, 4096, "p", False),
    (8, 32000, 5120, "p", True), (8, 57344, 2048, "", False), (8, 57344, 2304, "", True), (8, 57344, 3072, "", False), (4, 64, 128, "", True),
    (3, 33024, 4480, "p", False), (7, 33024, 4480, "p", True), (7, 36864, 2944, "p", False), (3, 34816, 1664, "", False),
    (5, 24576, 4096, "", True), (5, 24832, 4096, "", False), (5, 22016, 4096, "p", False), (8, 32000, 7168, "", True),
    (6, 8192, 5120, "tw", True), (4, 8192, 5120, "tw", False), (8, 12288, 2048, "tw", False), (5, 12288, 9216, "tw", True),
    (8, 22016, 4096, "tw", True), (8, 33924, 7808, "tf", False), (8, 57344, 8192, "tw", True),
    # nine to sixteen, and K split over the units
    (9, 1000, 512, "", True), (9, 4096, 1024, "", True), (9, 1000, 2048, "", False), (11, 35328, 3840, "f", False), (16, 57344, 3584, "", True), (16, 32000, 4096, "wp", True), (16, 57344, 4096, "", False),
    (9, 57344, 4096, "tw", True), (16, 32000, 7168, "w", True), (16, 32000, 8192, "w", False), (9, 32000, 10240, "w", True),
    (8, 57344, 11008, "tw", True), (8, 57344, 10240, "w", False), (12, 1400, 10880, "w", True),
])
def test_lines_of_the_rows_of_one_pass(rules, m, n, k, form, blocks):
    assert asked(rules, m, n, k, form) == blocks


def test_ragged_k(rules):
    assert all(rules.ragged(m, n, k) for m in (4, 7, 16, 500) for n in (1, 300, 32000) for k in (32, 1376, 65504))
    assert not rules.ragged(1, 4096, 1376) and not rules.ragged(2, 4096, 1376)
    assert rules.ragged(3, 4096, 1376) and rules.ragged(3, 1, 544) and rules.ragged(3, 1, 65504)
    assert not rules.ragged(3, 1, 8224) and not rules.ragged(3, 4, 28704) and not rules.ragged(3, 256, 28704)


@pytest.mark.parametrize("bits,m,n,k,blocks", [
    (6, 5, 9216, 4096, False), (6, 8, 10240, 8192, False), (6, 16, 10240, 4096, False), (6, 3, 9216, 16384, False),
    (6, 3, 2048, 16384, False), (6, 4, 3072, 20480, False), (6, 5, 8192, 4096, True), (6, 3, 8192, 4096, True),
    (6, 3, 2048, 4096, True), (6, 3, 1000, 4096, False), (6, 5, 1000, 4096, True), (6, 5, 32000, 11008, True),
    (6, 3, 2048, 24576, True), (6, 4, 8192, 24576, True), (6, 17, 32000, 4096, True), (6, 2, 4096, 24576, False),
    (8, 5, 9216, 9216, False), (8, 8, 12288, 3072, True), (8, 8, 12288, 4736, False), (8, 8, 12288, 7168, False), (8, 5, 16384, 8192, False),
    (8, 8, 12288, 4096, True), (8, 5, 16384, 2048, True), (8, 5, 8192, 9216, True), (8, 4, 8192, 4096, True), (8, 4, 8448, 4096, False),
    (8, 5, 32000, 11008, True), (8, 16, 4096, 5120, True), (8, 24, 64000, 128, True), (8, 8, 22016, 4096, False),
    (2, 4, 1000, 8192, False), (2, 3, 2048, 10240, False), (2, 4, 24000, 128, False), (2, 3, 18000, 512, False),
    (2, 4, 1000, 1024, True), (2, 3, 1000, 1024, False), (2, 4, 1000, 12288, True), (2, 3, 24000, 768, True),
    (2, 4, 4096, 128, True), (2, 5, 1000, 8192, True), (2, 2, 32000, 4096, False),
])
def test_other_formats(rules, bits, m, n, k, blocks):
    width = 4 if m <= 4 else 8 if m <= 8 else 16
    fits = (k // 128 + 3) // 4 * 1024 * width + 16384 <= 160 * 1024
    assert bool(rules.format(m, n, k, bits, int(fits))) == blocks


@pytest.mark.parametrize("m,n,k,tiles,blocks", [
    (9, 4096, 512, True, False), (16, 5120, 1024, True, True), (16, 5120, 3072, True, True), (16, 14336, 3072, True, True), (9, 2048, 2048, True, False),
    (16, 4096, 4096, True, True), (9, 4096, 2048, True, True), (12, 12288, 4096, True, False), (9, 16, 8, False, True),
    (16, 4096, 11008, False, True), (17, 12288, 4096, True, True),
    (5, 2048, 5120, False, False), (8, 5120, 2560, False, False), (6, 8192, 6144, False, False), (7, 10240, 2048, False, False),
    (8, 4096, 10240, False, False), (7, 8192, 10240, False, False), (8, 8192, 16384, False, False), (5, 4096, 11008, False, False),
    (8, 22016, 4096, False, False), (4, 4096, 4096, False, False), (8, 1000, 4096, False, False),
    (8, 4096, 4096, False, True), (5, 2050, 8, False, True), (7, 4096, 16384, False, True), (8, 5120, 11008, False, True),
    (6, 8192, 2048, False, True), (5, 9216, 1024, False, True),
])
def test_unquantised_weights(rules, m, n, k, tiles, blocks):
    assert bool(rules.bf16(m, n, k, int(tiles))) == blocks


@pytest.mark.parametrize("bits,m,n,k,blocks", [
    (8, 4, 1024, 512, False), (8, 4, 2048, 1024, True), (8, 3, 2048, 1152, False), (8, 3, 4096, 7168, True), (8, 4, 8192, 3072, True),
    (8, 4, 9216, 2048, True), (8, 4, 9216, 2560, False), (8, 8, 12288, 2560, True), (8, 16, 32000, 2048, True),
    (8, 16, 32000, 2560, False), (6, 3, 1000, 1024, True), (6, 4, 10240, 3072, True), (6, 16, 10240, 3200, True),
    (6, 16, 10240, 3712, False), (6, 16, 10240, 4352, True), (6, 16, 16384, 6144, True), (6, 16, 20480, 3072, False), (6, 16, 20736, 3072, True), (6, 5, 12288, 7168, False), (6, 8, 32000, 3072, True), (6, 8, 57344, 3072, False),
    (6, 4, 57344, 2048, True), (2, 3, 1024, 4096, True), (2, 3, 1024, 4224, False), (2, 4, 1000, 2560, False),
])
def test_other_formats_with_a_short_k(rules, bits, m, n, k, blocks):
    assert bool(rules.format(m, n, k, bits, 1)) == blocks


@pytest.mark.parametrize("m,n,k,tiles,blocks", [
    (3, 4096, 512, False, True), (3, 4096, 1024, False, False), (4, 4096, 1536, False, True), (4, 12288, 1024, False, True),
    (4, 12288, 1536, False, False), (4, 32000, 512, False, True), (4, 2048, 512, False, False), (5, 2048, 2048, False, True),
    (5, 1024, 2048, False, False), (8, 32000, 1024, False, True), (8, 32000, 1152, False, False), (8, 8192, 5120, False, True),
    (16, 8192, 3072, True, True), (16, 12288, 2048, True, True), (16, 12288, 512, True, True), (16, 12288, 1024, True, False),
])
def test_unquantised_weights_with_a_short_k(rules, m, n, k, tiles, blocks):
    assert bool(rules.bf16(m, n, k, int(tiles))) == blocks


@pytest.mark.parametrize("rows,n,k,want", [
    (3, 4096, 7168, 2), (3, 4096, 8192, 2), (3, 4096, 6824, 4), (3, 4096, 13104, 2), (3, 4096, 27304, 1),
    (8, 1000, 2048, 4), (8, 12288, 2048, 4), (8, 2000, 3072, 3), (8, 2048, 3072, 2), (5, 12288, 4096, 2), (8, 12288, 10240, 1),
    (4, 12288, 6824, 3), (2, 64, 8, 4), (1, 64, 65536, 1), (4, 64, 65536, 1),
])
def test_workgroups_of_a_vector_pass(rules, rows, n, k, want):
    assert rules.workgroups(rows, n, k) == want


def test_later_passes_have_no_fewer_workgroups(rules):
    # a pick reads as many partial winners per row as the first pass has workgroups
    def blocks(rows, n, k):
        per_unit = rules.workgroups(rows, n, k)
        waves = 4 if per_unit >= 3 else 8 if per_unit == 2 else 16
        return min(-(-n // waves), 256 * per_unit)
    for n in (1, 300, 2000, 2048, 4096, 20000):
        for k in range(8, 65537, 488):
            if 16 * k <= 160 * 1024:
                assert all(blocks(rows, n, k) >= blocks(8, n, k) for rows in range(1, 8)), (n, k)


def test_one_and_two_rows_never_take_the_blocks(rules):
    # where the decode kernels take them, whose FP32 sums are closer to 64 bits
    for m in (1, 2):
        for n in (1, 16, 1000, 1024, 1500, 2048, 4096, 9000, 16000, 28000, 32000, 57344):
            for k in (128, 384, 512, 1024, 2048, 4096, 4224, 5120, 8192, 11008, 28672, 65536):
                for fits in (0, 1):
                    for split in (0, 1):
                        for pick in (0, 1):
                            assert not any(rules.mx(m, n, k, fits, split, 0, fused, pick) for fused in (0, 1))
                            assert m == 2 or not rules.mx(m, n, k, fits, split, 1, 0, pick)
                    assert not any(rules.format(m, n, k, bits, fits) for bits in (2, 6, 8))
                assert not rules.ragged(m, n, k + 32) and (256 < n < 2048 or not rules.e2m3(m, n, k))


@pytest.mark.parametrize("m,n,k,form,blocks", [
    # tile-major, where the tiles take one and two rows
    (2, 300, 1024, "t", True), (2, 300, 1024, "tp", True), (1, 300, 1024, "tf", True), (2, 300, 896, "t", False), (1, 28000, 512, "tf", False),
    (2, 4096, 2048, "tp", True), (2, 4000, 2048, "t", False), (2, 9216, 2176, "t", False), (2, 9472, 1280, "t", False),
    (2, 22016, 2560, "tp", True), (1, 22016, 2560, "tf", True), (2, 22016, 2688, "t", False), (2, 25088, 2048, "t", False),
    (2, 57344, 1280, "t", True), (2, 57344, 1408, "tp", False), (1, 57344, 1024, "t", False), (1, 57344, 1024, "tp", False),
])
def test_one_and_two_rows_of_tile_major_weights(rules, m, n, k, form, blocks):
    assert asked(rules, m, n, k, form) == blocks


@pytest.mark.parametrize("kind,m,n,k,blocks", [
    ("e2m3", 1, 257, 384, True), ("e2m3", 2, 2047, 8192, True), ("e2m3", 1, 256, 1024, False), ("e2m3", 2, 1000, 256, False),
    ("e2m3", 1, 1000, 8320, False), ("e2m3", 2, 8192, 8192, False),
    ("bf16", 1, 4097, 384, True), ("bf16", 1, 4096, 384, False), ("bf16", 1, 8000, 512, False), ("bf16", 1, 8192, 1024, True),
    ("bf16", 1, 12288, 1280, False), ("bf16", 1, 28000, 1024, True), ("bf16", 1, 28000, 376, False), ("bf16", 1, 28000, 2048, False),
    ("bf16", 2, 2049, 384, True), ("bf16", 2, 2048, 384, False), ("bf16", 2, 7168, 1024, True), ("bf16", 2, 7169, 1024, False), ("bf16", 2, 9216, 512, True),
    ("bf16", 2, 9217, 128, False), ("bf16", 2, 3000, 512, False),
])
def test_one_and_two_rows_where_the_blocks_are_as_exact(rules, kind, m, n, k, blocks):
    if kind == "e2m3":
        assert bool(rules.e2m3(m, n, k)) == blocks
    else:
        assert all(bool(rules.bf16(m, n, k, tiles)) == blocks for tiles in (0, 1))


def picked(rules, bits, table, m, n, k):
    """The block shape that a call takes (pick_shape of csrc/gemm_wide.h), and by how much it is the cheapest."""
    cost = []
    for i, (wm, wn, wk, mf, nf, start, step, next_start, next_step) in enumerate(table):
        if not rules.cuts(bits, *(int(v) for v in (wm, wn, wk, mf, nf)), m, n, k):
            continue
        bm, bn, wk = int(wm * mf * 16), int(wn * nf * 16), int(wk)
        rounds = -(-(-(-m // bm) * -(-n // bn)) // 256)
        steps = -(-(-(-k // 128)) // wk) * wk
        cost.append((start + step * steps + (rounds - 1) * (next_start + next_step * steps), i))
    cost.sort()
    return cost[0][1], cost[1][0] / cost[0][0] - 1


KINDS = {"mxfp4": (0,), "tiled": (1,), "ragged": (2,), 8: (3, 4), 6: (5, 6), 2: (7,), "bf16": (8,)}       # of csrc/block_ways.h


@pytest.mark.parametrize("kind,source,name", [
    ("mxfp4", "gemm_wide.hip", "kCosts"), ("tiled", "gemm_wide.hip", "kCosts"), ("ragged", "gemm_wide.hip", "kCosts"),
    (8, "gemm_wide_fmt.hip", "kCosts8"), (6, "gemm_wide_fmt.hip", "kCosts6"), (2, "gemm_wide_fmt.hip", "kCosts2"), ("bf16", "gemm_wide_bf16.hip", "kCosts")])
def test_sizes_that_take_every_form_of_every_block_shape(rules, kind, source, name):
    body = re.search(r"constexpr Cost %s\[\] = \{(.*?)\n\};" % name, open(os.path.join(CSRC, source)).read(), re.S).group(1)
    table = [[float(v.rstrip("f")) for v in row.split(",")] for row in re.findall(r"\{([^{}]*)\}", body)]
    bits = {"mxfp4": 4, "tiled": 4, "ragged": 4, "bf16": 16}.get(kind, kind)
    for number in KINDS[kind]:
        built = []
        for i, row in enumerate(table):
            ways = rules.ways(number, *(int(v) for v in row[2:5]))
            assert ways
            built += [(i, way) for way in (1, 0) if ways & (1 if way else 2)]
        taken = []
        for m, n, k in BLOCK_SIZES[kind]:
            i = picked(rules, bits, table, m, n, k)[0]
            wm, _, wk, mf, nf = (int(v) for v in table[i][:5])
            taken.append((i, rules.direct(number, wk, mf, nf, k, -(-m // (16 * wm * mf)), 0)))
        assert taken == built
    for m, n, k in BLOCK_SIZES[kind]:
        assert picked(rules, bits, table, m, n, k)[1] > 0.005                # (the kernel's sums are in 32 bits)
        if kind == "mxfp4":
            assert all(asked(rules, m, n, k, form) for form in ("", "f", "wp"))
        elif kind == "tiled":
            assert asked(rules, m, n, k, "tw") and asked(rules, m, n, k, "twp")
        elif kind == "ragged":
            assert k % 128 and rules.ragged(m, n, k)
        elif kind == "bf16":
            assert rules.bf16(m, n, k, int(k % 128 == 0))
        else:
            assert rules.format(m, n, k, kind, 1)


@pytest.mark.parametrize("kind,wk,mf,nf,k,tiles_m,pick,direct", [
    (0, 8, 1, 1, 6144, 1, 0, True), (0, 8, 1, 1, 6272, 1, 0, False), (0, 8, 1, 1, 128, 1, 1, False), (0, 4, 1, 1, 1024, 7, 0, True),
    (0, 4, 1, 1, 1152, 7, 0, False), (1, 4, 1, 1, 1536, 6, 0, True), (1, 4, 1, 1, 1664, 6, 0, False), (0, 1, 8, 3, 65536, 1, 0, True),
    (0, 1, 8, 3, 65536, 1, 1, True), (0, 1, 4, 2, 8192, 1, 0, True), (0, 1, 4, 2, 8320, 1, 0, False), (0, 1, 4, 2, 8320, 1, 1, False),
    (1, 1, 4, 2, 65536, 1, 0, True), (2, 1, 4, 2, 65504, 1, 0, True), (3, 1, 4, 2, 128, 1, 0, False), (4, 1, 4, 2, 8192, 1, 0, False),
    (3, 1, 4, 1, 65536, 1, 0, True), (6, 1, 4, 2, 65536, 1, 0, True), (8, 1, 8, 2, 128, 1, 0, False), (0, 4, 2, 4, 128, 1, 0, False),
])
def test_which_way_the_activations_take(rules, kind, wk, mf, nf, k, tiles_m, pick, direct):
    assert bool(rules.direct(kind, wk, mf, nf, k, tiles_m, pick)) == direct


@pytest.mark.parametrize("kind,m,n,k,fast", [
    # us by shape, six sets of weights in rotation; those within 5 % of the fastest
    ("bf16", 39, 21924, 4224, [(1, 4, 2, 3, 2), (1, 4, 2, 4, 2)]),      # 46.3, 47.7; one column of tiles instead of two 53.9
    ("bf16", 33, 254, 1408, [(1, 1, 8, 1, 1)]),                         # 5.6; 6.6
    ("mxfp4", 46, 2986, 5504, [(1, 1, 8, 1, 3)]),                       # 8.8; 9.9
    ("mxfp4", 5, 8162, 11392, [(1, 1, 8, 1, 2)]),                       # 14.6; 16.5
    (6, 54, 22740, 10752, [(1, 4, 2, 4, 2)]),                           # 71; 86
    ("mxfp4", 48, 32000, 4096, [(1, 4, 2, 3, 2)]),                      # 23.6; 24.4
    ("mxfp4", 64, 12000, 4096, [(1, 2, 4, 2, 3)]),                      # 13.7; 15.4
    ("mxfp4", 128, 4096, 4096, [(1, 2, 4, 2, 2)]),                      # 11.2; 11.8
    ("mxfp4", 509, 22016, 4096, [(1, 8, 1, 8, 3)]),                     # 75; 94
])
def test_shapes_that_were_measured_the_fastest(rules, kind, m, n, k, fast):
    source, name, bits = {"bf16": ("gemm_wide_bf16.hip", "kCosts", 16), "mxfp4": ("gemm_wide.hip", "kCosts", 4),
                          6: ("gemm_wide_fmt.hip", "kCosts6", 6)}[kind]
    body = re.search(r"constexpr Cost %s\[\] = \{(.*?)\n\};" % name, open(os.path.join(CSRC, source)).read(), re.S).group(1)
    table = [[float(v.rstrip("f")) for v in row.split(",")] for row in re.findall(r"\{([^{}]*)\}", body)]
    assert tuple(int(v) for v in table[picked(rules, bits, table, m, n, k)[0]][:5]) in fast

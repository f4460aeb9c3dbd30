"""How the block kernel cuts the sums of its outputs along K (csrc/sum_chains.h), walked on the CPU for every block shape of
its tables: no call's sums run in longer chains than the shapes with eight, four or two waves along K have, whichever
shape is the cheapest."""
import ctypes
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_13565_amd", "csrc")
TABLES = [("gemm_wide.hip", "kCosts", 4), ("gemm_wide_fmt.hip", "kCosts8", 8), ("gemm_wide_fmt.hip", "kCosts6", 6),
          ("gemm_wide_fmt.hip", "kCosts2", 2), ("gemm_wide_bf16.hip", "kCosts", 16)]

WALK = r"""
#include "sum_chains.h"
using namespace mxfp4::wide;
extern "C" int wanted(int m, int n, int k) { return chains_wanted(m, n, k, 256); }
extern "C" int cuts(int bits, int wm, int wn, int wk, int mf, int nf, int m, int n, int k)
{
    return cuts_enough(bits, wm, wn, wk, mf, nf, m, n, k, 256);
}
// The longest chain, in steps of 128, of the kernel's loop over the phases.
extern "C" int longest(int bits, int wk, int mf, int nf, int k, int chains)
{
    const int steps = (k + 127) / 128, phases = (steps + wk - 1) / wk, pairs = chain_pairs(phases, wk, chains);
    const bool whole = (wk == 8 && mf > 1) || uncut(mf, nf), each = !whole && bits > 4 && !(bits == 8 && mf * nf == 16);
    const int sets = whole || each || bits > 4 ? 1 : sum_sets(wk, mf);
    int most = 0;
    for (int w = 0; w < wk; ++w) {
        int at = 0, left = pairs;
        for (int u = 0; u < phases; ++u) {
            at += u * wk + w < steps;
            most = at > most ? at : most;
            const bool ends = u % 2 == 1 ? --left == 0 : cuts_phases(wk, mf) && phases <= 2;
            if (each || (!whole && sets == 1 && ends)) {
                at = 0;
                left = left > 0 ? left : pairs;
            }
        }
    }
    return (most + sets - 1) / sets;                            // (a step's instructions take turns)
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("sum_chains")
    (d / "walk.cpp").write_text(WALK)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "walk.cpp"),
                           "-o", str(d / "walk.so")])
    return ctypes.CDLL(str(d / "walk.so"))


def shapes(source, name):
    body = re.search(r"constexpr Cost %s\[\] = \{(.*?)\n\};" % name, open(os.path.join(CSRC, source)).read(), re.S).group(1)
    return [tuple(int(v) for v in row.split(",")[:5]) for row in re.findall(r"\{([^{}]*)\}", body)]


@pytest.mark.parametrize("source,name,bits", TABLES)
def test_no_longer_chains_than_the_waves_along_k_have(walk, source, name, bits):
    for m in (3, 16, 17, 32, 33, 48, 64, 100, 128, 200, 509, 1000):
        for n in (16, 300, 2048, 4096, 6200, 12288, 22016, 32000, 57344):
            for k in (32, 128, 256, 384, 512, 640, 1024, 1376, 2048, 4096, 5120, 11008, 28672, 65536):
                steps, chains = (k + 127) // 128, walk.wanted(m, n, k)
                taken = [s for s in shapes(source, name) if walk.cuts(bits, *s, m, n, k)]
                assert taken                                # (every call finds a shape)
                for wm, wn, wk, mf, nf in taken:
                    if mf * nf > 16 and steps > 1:      # the blocks that cannot cut: the largest products only
                        assert m > 100 and m * n > 27 * 256 * 256, (m, n, k)
                        continue
                    # a chain ends with a pair of phases, unless a wave has a single step of them
                    limit = max(-(-steps // chains), 2 if wk < 8 and steps > wk else 1)
                    assert walk.longest(bits, wk, mf, nf, k, chains) <= limit, (m, n, k, wm, wn, wk, mf, nf)


@pytest.mark.parametrize("m,n,k,chains", [
    (97, 16400, 4096, 2), (97, 16400, 4224, 4), (97, 16384, 11008, 8), (509, 22016, 65536, 4), (509, 1500, 65536, 8),
    (3, 57344, 4096, 8), (32, 65536, 4096, 8), (33, 16384, 4096, 8), (33, 16400, 4096, 4), (96, 8192, 4096, 8),
    (96, 16384, 4096, 4), (97, 16384, 512, 4), (509, 22016, 4096, 2), (509, 1500, 4096, 8), (8, 4096, 256, 2), (8, 4096, 32, 1),
])
def test_chains_of_a_call(walk, m, n, k, chains):
    assert walk.wanted(m, n, k) == chains

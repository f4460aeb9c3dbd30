"""Parity of the block kernel for many activation rows and for K that is no multiple of 128
(csrc/gemm_wide.h; arXiv 2503.13565, section 3.4.3): plain, fused and pick forms against the CPU oracle
at the edges of its blocks, and every block shape in every weight layout (block_sizes.py)."""
import functools

import pytest
import torch

import oracle
from paper_2503_13565_amd import binding, synth

pytestmark = pytest.mark.gpu

from block_sizes import BLOCK_SIZES  # noqa: E402
from helpers import DEV, assert_argmax_ok, assert_cast_bit_exact, assert_gemm_close  # noqa: E402


def check(m, n, k):
    tag = "M=%d N=%d K=%d" % (m, n, k)
    print(tag, flush=True)
    w = synth.weights_student_t(n, k, seed=9000 + n + k)
    xb = synth.activations_outlier_channels(m, k + 8, seed=9100 + m).to(DEV)
    x = xb[:, :k]                                           # rows farther apart than K
    q, s, q_ref, s_ref = assert_cast_bit_exact(w, tag)
    y_ref, a_ref = oracle.woq_gemm(synth.to_bits(x.contiguous()), q_ref, s_ref)
    ybuf = torch.full((m, n + 4), 7.0, dtype=torch.bfloat16, device=DEV)
    binding.mxfp4_woq_gemm(x, q, s, y=ybuf[:, :n])
    torch.cuda.synchronize()
    assert_gemm_close(ybuf[:, :n], y_ref, a_ref, tag)
    assert bool((ybuf[:, n:] == 7.0).all()), tag            # nothing written past N
    again = binding.mxfp4_woq_gemm(x, q, s)
    assert torch.equal(again, ybuf[:, :n]), tag             # same bits whatever the strides
    idx, val = binding.mxfp4_woq_gemm_argmax(x, q, s)
    torch.cuda.synchronize()
    assert_argmax_ok(idx, val, y_ref, a_ref, tag)
    g = torch.Generator().manual_seed(m + n)
    for act in ([0, 1] if n % 2 == 0 else [0]):
        c = n // 2 if act else n
        bias = (torch.randn(n, generator=g) * 0.3).to(torch.bfloat16)
        res = (torch.randn(m, c, generator=g) * 0.3).to(torch.bfloat16)
        out_ref, a_out = oracle.epilogue(y_ref, a_ref, synth.to_bits(bias), synth.to_bits(res), act)
        y = res.to(DEV)                                     # the residual updated in place
        binding.mxfp4_woq_gemm_fused(x, q, s, bias=bias.to(DEV), act=act, residual=y, y=y)
        torch.cuda.synchronize()
        assert_gemm_close(y, out_ref, a_out, "%s act %d" % (tag, act))


@pytest.mark.parametrize("m,n,k", [(3, 1, 96), (7, 4096, 1376), (16, 17, 32), (5, 5001, 32), (17, 5001, 32),
                                   (5, 16000, 160), (5, 22000, 160), (5, 32000, 1376), (3, 12636, 288), (3, 32924, 32)])
def test_few_rows_ragged_k(m, n, k):
    check(m, n, k)


@pytest.mark.parametrize("m,n,k", [(17, 16, 128), (17, 8200, 1376), (33, 4096, 160), (33, 1000, 4096), (17, 16000, 1376),
                                   (32, 4098, 11008), (17, 22000, 1376), (17, 32000, 1376), (17, 8200, 160), (17, 22000, 160),
                                   (16, 32000, 288), (64, 259, 288), (17, 4596, 320), (35, 16599, 800), (34, 11208, 2016),
                                   (17, 6556, 288), (33, 11134, 3008)])
def test_several_sequences(m, n, k):
    check(m, n, k)


@pytest.mark.parametrize("m,n,k", [(65, 5001, 160), (65, 8200, 160), (129, 8200, 160), (300, 258, 1024), (129, 16000, 288),
                                   (128, 4096, 96), (129, 22000, 32), (300, 16000, 32), (300, 22000, 32), (300, 32000, 32),
                                   (509, 1, 64), (513, 130, 672), (66, 34424, 576), (536, 477, 544), (454, 260, 2080),
                                   (378, 8148, 768)])
def test_prompts(m, n, k):
    check(m, n, k)


@pytest.mark.parametrize("m,n,k", [(196, 26152, 1216), (138, 44350, 1120), (509, 22016, 4096), (1052, 98, 4192),
                                   (353, 5378, 2208), (590, 4838, 1056), (271, 20346, 1440)])
def test_largest_blocks(m, n, k):
    # checked on sampled weight rows, the edges among them
    w = synth.weights_student_t(n, k, seed=9300 + n, device=DEV)
    x = synth.activations_outlier_channels(m, k, seed=9400 + m, device=DEV)
    q, s = binding.mxfp4_direct_cast(w)
    g = torch.Generator().manual_seed(n)
    even = 2 * torch.cat([torch.arange(8), torch.randint(0, n // 2, (60,), generator=g), torch.arange(n // 2 - 8, n // 2)])
    rows = torch.stack([even, even + 1], dim=1).reshape(-1)         # whole (gate, up) pairs
    y_ref, a_ref = oracle.woq_gemm(synth.to_bits(x), q.cpu()[rows].numpy(), s.cpu()[rows].numpy())
    y = binding.mxfp4_woq_gemm(x, q, s)
    gated = binding.mxfp4_woq_gemm_fused(x, q, s, act=1)
    torch.cuda.synchronize()
    tag = "M=%d N=%d K=%d" % (m, n, k)
    assert_gemm_close(y[:, rows.to(DEV)], y_ref, a_ref, tag)
    out_ref, a_out = oracle.epilogue(y_ref, a_ref, None, None, 1)
    assert_gemm_close(gated[:, even.to(DEV) // 2], out_ref, a_out, tag)


@pytest.mark.parametrize("m,n,k,act", [(20, 131, 160, 0), (75, 17661, 128, 0), (75, 9002, 128, 1), (327, 12967, 128, 0), (130, 9002, 256, 1), (64, 18577, 256, 0), (100, 19938, 256, 1),
                                       (509, 22015, 1024, 0), (509, 22018, 1024, 1)])
@pytest.mark.parametrize("shift,pad", [(0, 0), (1, 0), (6, 3), (3, 8)])
def test_residual_rows_on_any_boundary(m, n, k, act, shift, pad):
    # blocks of a few and of many outputs, whose waves share K or not, in one and two turns; the residual's rows begin `shift`
    # elements behind a 16-byte boundary and lie C + pad apart, the outputs are written over it or elsewhere
    print("M=%d N=%d K=%d act %d shift %d pad %d" % (m, n, k, act, shift, pad), flush=True)
    w = synth.weights_student_t(n, k, seed=9150 + n, device=DEV)
    x = synth.activations_outlier_channels(m, k, seed=9160 + m, device=DEV)
    q, s = binding.mxfp4_direct_cast(w)
    c, g = n // (1 + act), torch.Generator().manual_seed(n + shift)
    edges = torch.cat([torch.arange(max(0, at - 9), min(c, at + 9)) for at in (0, 64, 128, 192, 256, 384, c) if at <= c])
    cols = torch.unique(torch.cat([edges, torch.randint(0, c, (40,), generator=g)]))
    rows = torch.stack([2 * cols, 2 * cols + 1], dim=1).reshape(-1) if act else cols
    y_ref, a_ref = oracle.woq_gemm(synth.to_bits(x), q.cpu()[rows].numpy(), s.cpu()[rows].numpy())
    bias = (torch.randn(n, generator=g) * 0.3).to(torch.bfloat16)
    room = torch.zeros((m * (c + pad) + 32,), dtype=torch.bfloat16, device=DEV)
    res = room[shift:shift + m * (c + pad)].view(m, c + pad)
    res.copy_((torch.randn((m, c + pad), generator=g) * 0.3).to(torch.bfloat16))
    before = room.clone()
    out_ref, a_out = oracle.epilogue(y_ref, a_ref, synth.to_bits(bias[rows]), synth.to_bits(res[:, cols.to(DEV)].contiguous()), act)
    y = binding.mxfp4_woq_gemm_fused(x, q, s, bias=bias.to(DEV), act=act, residual=res[:, :c])
    assert torch.equal(room.view(torch.int16), before.view(torch.int16))
    binding.mxfp4_woq_gemm_fused(x, q, s, bias=bias.to(DEV), act=act, residual=res[:, :c], y=res[:, :c])
    torch.cuda.synchronize()
    assert_gemm_close(y[:, cols.to(DEV)], out_ref, a_out)
    assert torch.equal(res[:, :c].contiguous().view(torch.int16), y.view(torch.int16))
    res[:, :c] = before[shift:shift + m * (c + pad)].view(m, c + pad)[:, :c]       # nothing else was written
    assert torch.equal(room.view(torch.int16), before.view(torch.int16))


@pytest.mark.parametrize("m,n,k", [(9, 4100, 4096), (16, 2050, 896), (5, 300, 11008), (17, 17, 128), (33, 1000, 1152),
                                   (48, 11000, 640), (130, 259, 2048), (300, 5001, 384)])
def test_tile_major_copy_gives_the_same_bits(m, n, k):
    w = synth.weights_student_t(n, k, seed=9500 + n, device=DEV)
    x = synth.activations_outlier_channels(m, k, seed=9600 + m, device=DEV)
    q, s = binding.mxfp4_direct_cast(w)
    tw = binding.mxfp4_tile_repack(q, s)
    ws = torch.empty((max(8, binding.mxfp4_woq_gemm_workspace_bytes(m, n, k)),), dtype=torch.uint8, device=DEV)
    want = binding.mxfp4_woq_gemm(x, q, s)
    assert torch.equal(binding.mxfp4_woq_gemm_tiled(x, tw, workspace=ws), want)
    assert_gemm_close(want[:, :17], *oracle.woq_gemm(synth.to_bits(x), q.cpu()[:17].numpy(), s.cpu()[:17].numpy()))
    idx, val = binding.mxfp4_woq_gemm_argmax(x, q, s)
    idx_t, val_t = binding.mxfp4_woq_gemm_tiled_argmax(x, tw)
    assert torch.equal(idx, idx_t) and torch.equal(val, val_t)


@pytest.mark.parametrize("n,k", [(1000, 384), (2049, 128), (4099, 1408), (8200, 5120), (8201, 672), (24577, 640), (16384, 1024)])
@pytest.mark.parametrize("m", [1, 2])
def test_one_and_two_rows(m, n, k):
    # row-major, tile-major and ragged K, with everything behind the product; sampled weight rows, the last ones among them
    w = synth.weights_student_t(n, k, seed=9170 + n, device=DEV)
    x = synth.activations_outlier_channels(m, k, seed=9180 + m, device=DEV)
    q, s = binding.mxfp4_direct_cast(w)
    cols = torch.unique(torch.cat([torch.arange(20), torch.arange(n - 40, n), torch.randint(0, n, (60,), generator=torch.Generator().manual_seed(n))]))
    y_ref, a_ref = oracle.woq_gemm(synth.to_bits(x), q.cpu()[cols].numpy(), s.cpu()[cols].numpy())
    bias, res = (synth.activations_gaussian(r, n, seed=9190 + r).to(DEV) for r in (1, m))
    out_ref, a_out = oracle.epilogue(y_ref, a_ref, synth.to_bits(bias[0][cols.to(DEV)].contiguous()), synth.to_bits(res[:, cols.to(DEV)].contiguous()), 0)
    y = [binding.mxfp4_woq_gemm(x, q, s), binding.mxfp4_woq_gemm_fused(x, q, s, bias=bias[0], residual=res)]
    if k % 128 == 0:
        tw = binding.mxfp4_tile_repack(q, s)
        y += [binding.mxfp4_woq_gemm_tiled(x, tw), binding.mxfp4_woq_gemm_tiled_fused(x, tw, bias=bias[0], residual=res)]
    torch.cuda.synchronize()
    for i, t in enumerate(y):
        assert_gemm_close(t[:, cols.to(DEV)], *((out_ref, a_out) if i % 2 else (y_ref, a_ref)), "form %d" % i)


FORMATS = {"e4m3": (oracle.e4m3_woq_gemm, binding.mxfp4_e4m3_direct_cast, binding.mxfp4_e4m3_woq_gemm,
                    binding.mxfp4_e4m3_woq_gemm_argmax),
           "e2m3": (oracle.e2m3_woq_gemm, binding.mxfp4_e2m3_direct_cast, binding.mxfp4_e2m3_woq_gemm,
                    binding.mxfp4_e2m3_woq_gemm_argmax)}
for _name, _id in (("e5m2", binding.FMT_E5M2), ("e3m2", binding.FMT_E3M2), ("t2", binding.FMT_T2)):
    FORMATS[_name] = tuple(functools.partial(f, _id) for f in (
        oracle.mx_woq_gemm, binding.mxfp4_fmt_direct_cast, binding.mxfp4_fmt_woq_gemm, binding.mxfp4_fmt_woq_gemm_argmax))


@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("m,n,k", [(1, 2049, 384), (1, 900, 2176), (1, 8200, 1024), (1, 16003, 4224), (2, 2049, 2048), (2, 8200, 128), (2, 8201, 5120)])
def test_one_and_two_rows_of_other_formats(fmt, m, n, k):
    ref, cast, product, _ = FORMATS[fmt]
    w = synth.weights_student_t(n, k, seed=9710 + n, device=DEV)
    x = synth.activations_outlier_channels(m, k, seed=9810 + m, device=DEV)
    q, s = cast(w)
    cols = torch.unique(torch.cat([torch.arange(20), torch.arange(n - 40, n), torch.randint(0, n, (60,), generator=torch.Generator().manual_seed(n))]))
    y = product(x, q, s)
    torch.cuda.synchronize()
    assert_gemm_close(y[:, cols.to(DEV)], *ref(synth.to_bits(x), q.cpu()[cols].numpy(), s.cpu()[cols].numpy()), "%s M=%d N=%d K=%d" % (fmt, m, n, k))


@pytest.mark.parametrize("fmt,m,n,k", [(fmt, *size) for fmt in ["mxfp4", "tiled", "bf16"] + sorted(FORMATS) for size in [
    (1, 300, 1024), (1, 2500, 512), (1, 9000, 1024), (1, 28000, 768), (2, 300, 1024), (2, 1000, 4096), (2, 2500, 1024), (2, 9000, 1024),
    (2, 9000, 5120), (2, 17000, 2048), (2, 28000, 2048)]] + [("mxfp4", 2, 3000, 1344), ("mxfp4", 1, 28000, 832)])
def test_one_and_two_rows_are_picked_from_the_sums_of_the_product(fmt, m, n, k):
    # the second half of K takes back what the first half adds but for a bit of a few elements: sums in another order come out different by far
    # more than the rounding of the result
    print(fmt, m, n, k, flush=True)
    w = synth.weights_student_t(n, k // 2, seed=9760 + n, device=DEV)
    w = torch.cat([w, -w], 1)
    xs = synth.activations_outlier_channels(24 * m, k // 2, seed=9770 + k, device=DEV)
    more = xs.clone()
    more[:, 7::k // 8].view(torch.int16).add_(1)
    xs = torch.cat([xs, more], 1)
    if fmt == "bf16":
        product, pick = (lambda x: binding.mxfp4_bf16_gemm(x, w)), (lambda x: binding.mxfp4_bf16_gemm_argmax(x, w))
    elif fmt in FORMATS:
        q = FORMATS[fmt][1](w)
        product, pick = (lambda x: FORMATS[fmt][2](x, *q)), (lambda x: FORMATS[fmt][3](x, *q))
    else:
        q = binding.mxfp4_direct_cast(w)
        if fmt == "tiled":
            tw = binding.mxfp4_tile_repack(*q)
            product, pick = (lambda x: binding.mxfp4_woq_gemm_tiled(x, tw)), (lambda x: binding.mxfp4_woq_gemm_tiled_argmax(x, tw))
        else:
            product, pick = (lambda x: binding.mxfp4_woq_gemm(x, *q)), (lambda x: binding.mxfp4_woq_gemm_argmax(x, *q))
    for x in xs.split(m):
        y, (idx, val) = product(x), pick(x)
        assert torch.equal(y.gather(1, idx.long()[:, None])[:, 0], val.to(torch.bfloat16))
        assert torch.equal(y.max(dim=1).values, val.to(torch.bfloat16))


@pytest.mark.parametrize("m,n,k", [(1, 4097, 8), (1, 8200, 1000), (1, 16003, 1280), (2, 2049, 384), (2, 8200, 1024), (2, 33000, 128)])
def test_one_and_two_rows_of_unquantised_weights(m, n, k):
    w = synth.weights_student_t(n, k, seed=9920 + n, device=DEV)
    x = synth.activations_outlier_channels(m, k, seed=9960 + m, device=DEV)
    y_ref, a_ref = oracle.bf16_gemm(synth.to_bits(x), synth.to_bits(w))
    y, (idx, val) = binding.mxfp4_bf16_gemm(x, w), binding.mxfp4_bf16_gemm_argmax(x, w)
    torch.cuda.synchronize()
    assert_gemm_close(y, y_ref, a_ref)
    assert_argmax_ok(idx, val, y_ref, a_ref)


@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("m,n,k", [(3, 2050, 128), (5, 17, 1408), (8, 12288, 256), (16, 900, 5632), (17, 4099, 384), (33, 1000, 2176),
                                   (64, 9000, 128), (70, 5001, 256), (129, 259, 1152), (200, 8200, 256), (300, 16000, 128)])
def test_other_formats(fmt, m, n, k):
    ref, cast, product, pick = FORMATS[fmt]
    tag = "%s M=%d N=%d K=%d" % (fmt, m, n, k)
    print(tag, flush=True)
    w = synth.weights_student_t(n, k, seed=9700 + n, device=DEV)
    x = synth.activations_outlier_channels(m, k, seed=9800 + m, device=DEV)
    q, s = cast(w)
    y_ref, a_ref = ref(synth.to_bits(x), q.cpu().numpy(), s.cpu().numpy())
    y = product(x, q, s)
    idx, val = pick(x, q, s)
    torch.cuda.synchronize()
    assert_gemm_close(y, y_ref, a_ref, tag)
    assert_argmax_ok(idx, val, y_ref, a_ref, tag)
    s[n - 1, k // 32 - 1] = 255                             # a NaN block poisons its weight row only
    nan = torch.isnan(product(x, q, s))
    assert bool(nan[:, n - 1].all()) and not bool(nan[:, :n - 1].any()), tag


@pytest.mark.parametrize("m,n,k", [(5, 2050, 8), (7, 5001, 2056), (9, 259, 1000), (16, 4100, 11008), (17, 33, 40), (40, 1000, 136),
                                   (64, 9000, 120), (70, 5001, 264), (129, 259, 1152), (200, 8200, 248), (300, 16000, 128)])
def test_unquantised_weights(m, n, k):
    tag = "BF16 M=%d N=%d K=%d" % (m, n, k)
    print(tag, flush=True)
    wide = synth.weights_student_t(n, k + 16, seed=9900 + n, device=DEV)
    x = synth.activations_outlier_channels(m, k, seed=9950 + m, device=DEV)
    for w in (wide[:, :k], wide[:, :k].contiguous()):       # rows farther apart than K, and not
        y_ref, a_ref = oracle.bf16_gemm(synth.to_bits(x), synth.to_bits(w.contiguous()))
        y = binding.mxfp4_bf16_gemm(x, w)
        idx, val = binding.mxfp4_bf16_gemm_argmax(x, w)
        torch.cuda.synchronize()
        assert_gemm_close(y, y_ref, a_ref, tag)
        assert_argmax_ok(idx, val, y_ref, a_ref, tag)
    wide[:, k:] = float("nan")                              # what lies between the rows is not read into them
    assert torch.equal(binding.mxfp4_bf16_gemm(x, wide[:, :k]), y), tag


CASES = [(name, *size) for kind, names in (("mxfp4", ["mxfp4"]), ("tiled", ["tiled"]), ("ragged", ["ragged"]), (8, ["e4m3", "e5m2"]),
                                           (6, ["e2m3", "e3m2"]), (2, ["t2"]), ("bf16", ["bf16"]))
         for name in names for size in BLOCK_SIZES[kind]]


@pytest.mark.parametrize("name,m,n,k", CASES)
def test_every_block_shape_of_every_layout(name, m, n, k):
    # the product on sampled weight rows, those at the edges of blocks and tiles among them; product and pick take the same
    # block shape, so the pick's value is the product's sum before its rounding
    tag = "%s M=%d N=%d K=%d" % (name, m, n, k)
    print(tag, flush=True)
    w = synth.weights_student_t(n, k, seed=9200 + n, device=DEV)
    x = synth.activations_outlier_channels(m, k, seed=9250 + m, device=DEV)
    g = torch.Generator().manual_seed(n)
    rows = torch.unique(torch.cat([torch.arange(min(n, 33)), torch.arange(max(0, n - 33), n), torch.randint(0, n, (70,), generator=g)]))
    if name == "bf16":
        ref, q = oracle.bf16_gemm, (w,)
        y, (idx, val) = binding.mxfp4_bf16_gemm(x, w), binding.mxfp4_bf16_gemm_argmax(x, w)
        ref_args = (synth.to_bits(w[rows.to(DEV)].contiguous()),)
    elif name in FORMATS:
        ref, cast, product, pick = FORMATS[name]
        q = cast(w)
        y, (idx, val) = product(x, *q), pick(x, *q)
    else:
        ref, q = oracle.woq_gemm, binding.mxfp4_direct_cast(w)
        if name == "tiled":
            tw = binding.mxfp4_tile_repack(*q)
            ws = torch.empty((max(8, binding.mxfp4_woq_gemm_workspace_bytes(m, n, k)),), dtype=torch.uint8, device=DEV)
            y, (idx, val) = binding.mxfp4_woq_gemm_tiled(x, tw, workspace=ws), binding.mxfp4_woq_gemm_tiled_argmax(x, tw)
        else:
            y, (idx, val) = binding.mxfp4_woq_gemm(x, *q), binding.mxfp4_woq_gemm_argmax(x, *q)
    if name != "bf16":
        ref_args = tuple(t.cpu()[rows].numpy() for t in q)
    torch.cuda.synchronize()
    y_ref, a_ref = ref(synth.to_bits(x), *ref_args)
    assert_gemm_close(y[:, rows.to(DEV)], y_ref, a_ref, tag)
    at_pick = y.gather(1, idx.long()[:, None])[:, 0]
    assert torch.equal(val.to(torch.bfloat16), at_pick) and torch.equal(at_pick, y.max(dim=1).values), tag


@pytest.mark.parametrize("name,m,n,k,bound", [("mxfp4", 100, 6656, 4096, 1.2e-7), ("e4m3", 40, 8448, 4096, 1.8e-7),
                                              ("bf16", 40, 8448, 4096, 2.0e-7), ("bf16", 32, 12288, 8192, 2.5e-7),
                                              ("bf16", 8, 4096, 8192, 1.4e-7), ("e4m3", 8, 4096, 8192, 1.5e-7)])
def test_picks_values_are_sums_of_short_chains(name, m, n, k, bound):
    # against 64 bits, as a part of them: between what eight chains of K leave (0.9e-7, 1.3e-7, 1.5e-7, 1.9e-7, by the format's
    # digits and K) and what two do (1.6e-7, 2.8e-7, 3.3e-7, 3.4e-7); at eight rows, between chains of one step (0.9e-7, 1.0e-7)
    # and eight chains (1.6e-7, 1.9e-7), the vector ALUs and the tiles 1.2e-7
    off = size = 0.0
    for seed in range(4 if m > 8 else 16):
        w = synth.weights_student_t(n, k, seed=9600 + seed, device=DEV)
        x = synth.activations_outlier_channels(m, k, seed=9650 + seed, device=DEV)
        if name == "bf16":
            wide, (idx, val) = w, binding.mxfp4_bf16_gemm_argmax(x, w)
        elif name == "e4m3":
            q = binding.mxfp4_e4m3_direct_cast(w)
            wide, (idx, val) = binding.mxfp4_e4m3_dequant(*q), binding.mxfp4_e4m3_woq_gemm_argmax(x, *q)
        else:
            q = binding.mxfp4_direct_cast(w)
            wide, (idx, val) = binding.mxfp4_dequant(*q), binding.mxfp4_woq_gemm_argmax(x, *q)
        exact = (x.double() * wide[idx.long()].double()).sum(dim=1)
        off += float((val.double() - exact).square().sum())
        size += float(exact.square().sum())
    error = (off / size) ** 0.5
    print("%s M=%d N=%d K=%d: %.2e" % (name, m, n, k, error), flush=True)
    assert error <= bound


def test_nan_stays_in_its_row_and_block():
    # a NaN scale byte poisons its weight row, a NaN activation its own row: also in the rows that
    # repeat past M and N and in the blocks that round K up
    n, k, m = 35, 160, 19
    q = torch.randint(0, 256, (n, k // 2), dtype=torch.uint8, device=DEV)
    s = torch.full((n, k // 32), 120, dtype=torch.uint8, device=DEV)
    s[34, 4] = 255
    x = synth.activations_gaussian(m, k, seed=4).to(DEV)
    x[18, 159] = float("nan")
    y = binding.mxfp4_woq_gemm(x, q, s)
    torch.cuda.synchronize()
    want = torch.zeros((m, n), dtype=torch.bool, device=DEV)
    want[18, :] = True
    want[:, 34] = True
    assert torch.equal(torch.isnan(y), want)


def test_replays_from_a_graph():
    n, k, m = 600, 1184, 40
    w = synth.weights_student_t(n, k, seed=3).to(DEV)
    q, s = binding.mxfp4_direct_cast(w)
    x = synth.activations_gaussian(m, k, seed=5).to(DEV)
    y = torch.empty((m, n), dtype=torch.bfloat16, device=DEV)
    binding.mxfp4_woq_gemm(x, q, s, y=y)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        binding.mxfp4_woq_gemm(x, q, s, y=y)
    for i in range(3):
        x.copy_(synth.activations_gaussian(m, k, seed=50 + i))
        want = binding.mxfp4_woq_gemm(x, q, s)
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)

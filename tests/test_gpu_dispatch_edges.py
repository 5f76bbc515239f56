"""Edges of the kernel choices (run with -m gpu): shapes on both sides of each
rule that picks a kernel or a block shape, against the CPU oracle.  Packed
levels and integer accumulators are compared bit for bit."""
import re

import numpy as np
import pytest
import torch

import oracle
import paper_2003_04296_amd as q
from paper_2003_04296_amd import synth
from helpers import tail_bits_zero, unpack_act, unpack_act16, unpack_weight, weight_copies, weight_copy_f16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.lib()
    q.lib()
    return torch.device("cuda:0")


def _x(seed, shape):
    x = synth.normal(synth.generator(seed), shape, 1.0)
    v = torch.tensor([0.0, -0.0, float("nan"), float("inf"), -float("inf"), 0.5, -0.5, 0.125, 0.375, -0.75, 1e-40])
    flat = x.view(-1)
    flat[:: max(1, flat.numel() // 97)][: v.numel()] = v[: flat[:: max(1, flat.numel() // 97)].numel()]
    return x


# lanes along the channels (maps below 16 pixels), along the pixels (from 16
# on), ragged words, more than 16 words per pixel, and 1 / 2 / 4 runs per block
PACK_SHAPES = [(5, 70, 3, 5), (9, 64, 1, 1), (3, 33, 4, 4), (2, 513, 4, 5), (1, 1000, 9, 8), (2, 36, 15, 13),
               (66, 64, 32, 32), (131, 100, 32, 32), (66, 20, 32, 31)]
# small maps on both sides of where lanes run along the pixels (8192 pairs of
# words from 8 pixels on, 65536 from 4 on), in groups of four words with a last
# one of fewer; groups whose last run of pixels, and last eight runs, are not full
PACK_SHAPES += [(1023, 40, 2, 4), (1024, 40, 2, 4), (911, 150, 3, 3), (16383, 20, 2, 2), (16385, 20, 2, 2),
                (5500, 140, 1, 4), (9, 530, 13, 14), (1, 544, 45, 23), (37, 1030, 4, 4)]
# runs of whole images (fewer than 64 pixels, several small images or one, a last
# group of words that is not full, more than 16 words), two words of four runs
# from 1024 (run, word) pairs on, and up to 8 channels on maps of 2 pixels and more
PACK_SHAPES += [(19, 150, 7, 7), (3, 70, 5, 5), (701, 40, 5, 7), (2100, 36, 3, 11), (7, 520, 6, 6), (1, 130, 7, 9),
                (80, 290, 9, 9), (91, 290, 9, 9), (141, 3, 1, 2), (77, 8, 3, 4), (77, 9, 3, 4)]


@pytest.mark.parametrize("bits", [1, 2, 3])
@pytest.mark.parametrize("shape", PACK_SHAPES)
def test_pack_act(dev, bits, shape):
    n, c, h, w = shape
    x = _x(31, shape)
    words = q.packed_act_words(n, c, h, w, bits)
    want = oracle.quantize(x.numpy(), bits)
    for off in (0, 1):  # a 16-byte aligned output, and one that is not
        out = torch.full((words + 8,), 0x5A5A5A5A, dtype=torch.int32, device=dev)
        q.pack_act(x.to(dev), bits, out=out[off:off + words])
        got = out.cpu().numpy()
        np.testing.assert_array_equal(unpack_act(got[off:off + words], n, c, h, w, bits), want)
        assert tail_bits_zero(got[off:off + words], c, bits)
        assert (got[:off] == 0x5A5A5A5A).all() and (got[off + words:] == 0x5A5A5A5A).all()


# past 2^27 units of the lanes-along-the-channels kernel: several launches
def test_pack_act_many_images(dev):
    n = (1 << 27) + 5
    x = torch.empty((n, 1, 1, 1), dtype=torch.float32, device=dev).uniform_(-1, 1)
    out = torch.full((n + 8,), 0x5A5A5A5A, dtype=torch.int32, device=dev)
    q.pack_act(x, 1, out=out[:n])
    assert torch.equal(out[:n], (x.view(-1) > 0).int())
    assert (out[n:] == 0x5A5A5A5A).all()


# through LDS from 65536 (pixel, word) pairs on (here up to 10 words per pixel, in
# groups of 8 of one run of pixels and, where a plane is not whole runs of 64
# bytes, of 1 to 3 of four or two), directly below
@pytest.mark.parametrize("shape", [(33, 40, 32, 32), (8, 270, 31, 31), (3, 40, 9, 9), (9, 300, 28, 28), (700, 70, 6, 6),
                                   (61, 20, 33, 35)])
def test_pack_act16(dev, shape):
    n, c, h, w = shape
    x = _x(32, shape)
    got, pad_ok = unpack_act16(q.pack_act(x.to(dev), 16).cpu().numpy(), n, c, h, w)
    assert pad_ok
    want = oracle.to_f16(x.numpy()).view(np.uint16)
    nan = np.isnan(x.numpy())
    np.testing.assert_array_equal(got.view(np.uint16)[~nan], want[~nan])
    assert np.isnan(got[nan]).all()


# one pass per 8 or 32 output channels (32 from 512 blocks of those on), with
# 16- and 4-byte loads, around 64 input channels, at the most taps its LDS
# holds and past them (the gather)
@pytest.mark.parametrize("bits", [1, 2, 3])
@pytest.mark.parametrize("shape", [(9, 64, 3, 3), (130, 63, 3, 3), (33, 65, 2, 2), (2050, 512, 1, 1), (2050, 511, 1, 1),
                                   (17, 70, 5, 5), (17, 70, 6, 6)])
def test_pack_weight(dev, bits, shape):
    cout, cin, kh, kw = shape
    w = synth.normal(synth.generator(33), shape, 2.0 / (cin * kh * kw))
    w.view(-1)[:2] = torch.tensor([0.0, -0.0])
    lv, s = oracle.quantize_weights(w.numpy(), bits)
    for off in (0, 1):  # 16-byte aligned weights, and weights that are not
        buf = torch.zeros(w.numel() + 4, device=dev)
        buf[off:off + w.numel()] = w.reshape(-1).to(dev)
        words, scale = q.pack_weight(buf[off:off + w.numel()].view(shape), bits)
        words = words.cpu().numpy()
        np.testing.assert_array_equal(scale.cpu().numpy(), s)
        np.testing.assert_array_equal(unpack_weight(words, cout, cin, kh, kw, bits), lv)
        for copy in weight_copies(words, cout, cin, kh, kw, bits):
            np.testing.assert_array_equal(copy, lv)
        np.testing.assert_array_equal(weight_copy_f16(words, cout, cin, kh, kw, bits), lv)


# channels whose scale or thresholds are not finite, or zero, in every packing kernel
# (one pass with 16- and 4-byte loads, the gather past its taps): a NaN weight, one
# and two infinities, zeros alone, denormals, with thresholds 0 and infinite
# (0 x inf and inf x 0 make NaN thresholds) beside the defaults
NONFINITE_THR = {1: [None], 2: [None, (0.0,), (float("inf"),)],
                 3: [None, (0.0, 0.0, 0.0), (0.0, 0.25, 0.5), (0.0, 0.0, 0.5), (0.125, float("inf"), float("inf"))]}


@pytest.mark.parametrize("bits, base", [(b, t) for b in (1, 2, 3) for t in NONFINITE_THR[b]])
@pytest.mark.parametrize("shape", [(9, 64, 3, 3), (9, 63, 3, 3), (2056, 516, 1, 1), (10, 70, 5, 5), (10, 70, 6, 6)])
def test_pack_weight_not_finite(dev, bits, base, shape):
    cout, cin, kh, kw = shape
    nan, inf = float("nan"), float("inf")
    w = synth.normal(synth.generator(41), shape, 2.0 / (cin * kh * kw))
    flat = w.view(cout, -1)
    flat[0, 1] = nan
    flat[1, 2] = inf
    flat[2, 3:5] = torch.tensor([inf, -inf])
    flat[3] = 0.0
    flat[3, ::2] = -0.0
    flat[4, 5:7] = torch.tensor([nan, -inf])
    flat[5] *= 1e-38
    flat[cout - 1, -1] = nan  # beside an all-finite channel of the same block
    lv, s = oracle.quantize_weights(w.numpy(), bits, base_thr=base)
    words, scale = q.pack_weight(w.to(dev), bits, base_thresholds=base)
    words = words.cpu().numpy()
    np.testing.assert_array_equal(scale.cpu().numpy(), s)
    np.testing.assert_array_equal(unpack_weight(words, cout, cin, kh, kw, bits), lv)
    for copy in weight_copies(words, cout, cin, kh, kw, bits):
        np.testing.assert_array_equal(copy, lv)
    np.testing.assert_array_equal(weight_copy_f16(words, cout, cin, kh, kw, bits), lv)


# packed outputs of pooled layers on every block shape: 256 rows x 128 and x 64
# channels and the split-K shape, ragged channels, 255 windows an image
@pytest.mark.parametrize("bits", [1, 2, 3])
@pytest.mark.parametrize("n, cout, cfg", [(130, 100, 0), (130, 48, 1), (11, 100, 2)])
def test_pooled_packed_output(dev, n, cout, cfg, bits):
    cin, h, w = 40, 30, 34
    g = synth.generator(34)
    x = synth.normal(g, (n, cin, h, w), 1.0)
    wt = synth.normal(g, (cout, cin, 3, 3), 2.0 / (9 * cin))
    kk, bb = synth.uniform(g, (cout,), 0.01, 0.05), synth.normal(g, (cout,), 0.1)
    name = q.kernel_name(n, cin, h, w, cout, 3, 1, 1, bits, bits, mode=q.EPI_BN_PACK, flags=q.EPI_POOL2,
                         out_bits=bits, packed_out=True)
    assert int(name.split("<")[1].split(",")[2]) == cfg, name
    wq, _ = q.pack_weight(wt.to(dev), bits)
    _, got = q.conv(q.pack_act(x.to(dev), bits), wq, n, cin, h, w, cout, 3, 1, 1, bits, bits, mode=q.EPI_BN_PACK,
                    flags=q.EPI_POOL2, bn_k=kk.to(dev), bn_b=bb.to(dev), out_bits=bits)
    lw, _ = oracle.quantize_weights(wt.numpy(), bits)
    acc = oracle.qconv_acc(oracle.quantize(x.numpy(), bits), lw, bits, 1, 1)
    acc = acc.reshape(n, cout, h // 2, 2, w // 2, 2).max(axis=(3, 5))
    z = oracle.epi_bn(acc, kk.numpy(), bb.numpy(), 2 * oracle.level_shift(bits))
    np.testing.assert_array_equal(unpack_act(got.cpu().numpy(), n, cout, h // 2, w // 2, bits),
                                  oracle.quantize(oracle.hardtanh(z), bits))
    assert tail_bits_zero(got.cpu().numpy(), cout, bits)


# layers of few output tiles: each block shape of the kernel for them (one
# channel tile and 4 or 8 waves, two and 8), its last tile partly or wholly past
# the last pixel or channel, every epilogue, pooled and not, strides, 1 x 1 and
# a kernel that covers the map, and both sides of its 1024-tile limit
LAT_CASES = [
    # n, cin, h, w, cout, k, stride, pad, shape (channel tiles, waves; None: another kernel)
    (1, 64, 56, 56, 64, 3, 1, 1, (1, 4)),
    (3, 70, 9, 7, 40, 3, 1, 1, (1, 4)),
    (2, 33, 11, 13, 31, 3, 2, 1, (1, 4)),
    (1, 512, 7, 7, 200, 3, 1, 1, (1, 8)),
    (5, 512, 4, 4, 70, 4, 1, 0, (1, 8)),
    (12, 260, 14, 14, 150, 3, 1, 1, (2, 8)),
    (7, 128, 28, 28, 128, 1, 2, 0, (1, 4)),
    (32, 96, 32, 32, 32, 1, 1, 0, (1, 4)),
    (33, 96, 32, 32, 32, 3, 1, 1, None),
    # both sides of two channel tiles (over 320 tiles and 10000 tile steps)
    (80, 256, 8, 8, 64, 3, 1, 1, (1, 4)),
    (81, 256, 8, 8, 64, 3, 1, 1, (2, 8)),
    (138, 128, 8, 8, 64, 3, 1, 1, (1, 4)),
    (139, 128, 8, 8, 64, 3, 1, 1, (2, 8)),
    # and of 40000 tile steps
    (222, 320, 8, 8, 64, 3, 1, 1, (2, 8)),
    (223, 320, 8, 8, 64, 3, 1, 1, None),
    # and of 512 tiles, where 3-bit inputs with unpacked outputs end
    (128, 128, 8, 8, 64, 3, 1, 1, (1, 4)),
    (129, 128, 8, 8, 64, 3, 1, 1, (1, 4)),
    # and of 768 tiles, where int32 outputs of 9 to 17 steps end, and beside them
    # another number of steps and 32 channels
    (48, 64, 16, 16, 64, 3, 1, 1, (1, 4)),
    (49, 64, 16, 16, 64, 3, 1, 1, None),
    (49, 64, 16, 16, 64, 2, 1, 0, (1, 4)),
    (97, 64, 16, 16, 32, 3, 1, 1, (1, 4)),
]


@pytest.mark.parametrize("ab, wb", [(1, 1), (2, 1), (1, 2), (2, 2), (3, 3), (3, 1)])
@pytest.mark.parametrize("case", LAT_CASES)
def test_few_output_tiles(dev, case, ab, wb):
    n, cin, h, w, cout, k, s, p, shape = case
    g = synth.generator(35 + n + cin)
    x = _x(36 + n, (n, cin, h, w))
    wt = synth.normal(g, (cout, cin, k, k), 2.0 / (k * k * cin))
    kk, bb = synth.uniform(g, (cout,), 0.001, 0.05), synth.normal(g, (cout,), 0.1)
    ho, wo = q.out_size(h, k, s, p), q.out_size(w, k, s, p)
    act = q.pack_act(x.to(dev), ab)
    wq, sc = q.pack_weight(wt.to(dev), wb)
    lw, osc = oracle.quantize_weights(wt.numpy(), wb)
    acc = oracle.qconv_acc(oracle.quantize(x.numpy(), ab), lw, ab, s, p)
    shift = oracle.level_shift(ab) + oracle.level_shift(wb)
    algo = q.ALGO_MFMA_FP4
    for pool in (False, True):
        if pool and (ho < 2 or wo < 2):
            continue
        flags = q.EPI_POOL2 if pool else 0
        name = q.kernel_name(n, cin, h, w, cout, k, s, p, ab, wb, flags=flags, algo=algo)
        if not pool:
            many = n * -(-ho * wo // 32) * -(-cout // 32) > 512  # (maps of whole tiles where it matters)
            lat = shape and not (ab == 3 and many and k * k * -(-cin // 64) > 9)
            want = f"conv_mfma_lat_kernel<{q.planes(ab)}, {shape[0]}, {shape[1]}, 0>" if lat else "conv_mfma_kernel"
            assert name.startswith(want), name
            if (n, cin, k) == (49, 64, 3):  # batch norm and residual stay
                assert "lat" in q.kernel_name(n, cin, h, w, cout, k, s, p, ab, wb, mode=q.EPI_BN_F32, algo=algo)
        a = acc
        if pool:
            oh, ow = ho // 2, wo // 2
            a = acc[:, :, :2 * oh, :2 * ow].reshape(n, cout, oh, 2, ow, 2).max(axis=(3, 5))
        z = oracle.epi_bn(a, kk.numpy(), bb.numpy(), shift)
        res = synth.normal(g, z.shape, 1.0)
        args = (act, wq, n, cin, h, w, cout, k, s, p, ab, wb)
        kw = dict(bn_k=kk.to(dev), bn_b=bb.to(dev), algo=algo)
        out, _ = q.conv(*args, flags=flags, algo=algo)
        np.testing.assert_array_equal(out.cpu().numpy(), a)
        out, _ = q.conv(*args, mode=q.EPI_SCALE_F32, flags=flags, scale=sc, algo=algo)
        np.testing.assert_array_equal(out.cpu().numpy(), oracle.epi_scale(a, osc, shift))
        for ob in (1, 2, 3):
            words = q.packed_act_words(n, cout, z.shape[2], z.shape[3], ob)
            outp = torch.full((words + 16,), 0x5A5A5A5A, dtype=torch.int32, device=dev)
            q.conv(*args, mode=q.EPI_BN_PACK, flags=flags, out_bits=ob, out_packed=outp[:words], **kw)
            got = outp.cpu().numpy()
            np.testing.assert_array_equal(unpack_act(got[:words], n, cout, *z.shape[2:], ob),
                                          oracle.quantize(oracle.hardtanh(z), ob))
            assert tail_bits_zero(got[:words], cout, ob) and (got[words:] == 0x5A5A5A5A).all()
        outp = torch.empty(words, dtype=torch.int32, device=dev)
        zr = oracle.add(z, res.numpy())
        out, _ = q.conv(*args, mode=q.EPI_BN_F32, flags=flags | q.EPI_RESIDUAL, residual=res.to(dev), out_bits=3,
                        out_packed=outp, **kw)
        np.testing.assert_array_equal(out.cpu().numpy(), zr)
        np.testing.assert_array_equal(unpack_act(outp.cpu().numpy(), n, cout, *z.shape[2:], 3),
                                      oracle.quantize(oracle.hardtanh(zr), 3))


# AUTO on contractions of up to 256 values: the few-tiles kernel up to 1024 tiles
# (768 for int32 outputs of 1-bit weights in one or two k-steps), the XNOR kernel
# past them, with the same values
AUTO_CASES = [
    # n, cin, h, w, cout, k, stride, pad, kernel of int32 outputs (1-bit, 2-bit weights), of the others
    (24, 64, 16, 16, 128, 1, 1, 0, "lat", "lat", "lat"),
    (25, 64, 16, 16, 128, 1, 1, 0, "xnor", "lat", "lat"),
    (25, 160, 16, 16, 128, 1, 1, 0, "lat", "lat", "lat"),
    (32, 64, 32, 32, 128, 1, 2, 0, "xnor", "lat", "lat"),
    (33, 64, 32, 32, 128, 1, 2, 0, "xnor", "xnor", "xnor"),
    (32, 28, 16, 16, 128, 3, 1, 1, "lat", "lat", "lat"),
    (33, 28, 16, 16, 128, 3, 1, 1, "xnor", "xnor", "xnor"),
]


@pytest.mark.parametrize("ab, wb", [(1, 1), (2, 1), (2, 2), (1, 2)])
@pytest.mark.parametrize("case", AUTO_CASES)
def test_auto_small_contraction(dev, case, ab, wb):
    n, cin, h, w, cout, k, s, p, int1, int2, other = case
    geo = (n, cin, h, w, cout, k, s, p, ab, wb)
    x = _x(42 + n, (n, cin, h, w))
    g = synth.generator(43 + cin)
    wt = synth.normal(g, (cout, cin, k, k), 2.0 / (k * k * cin))
    kk, bb = synth.uniform(g, (cout,), 0.001, 0.05), synth.normal(g, (cout,), 0.1)
    algo = {"lat": q.ALGO_MFMA_FP4, "xnor": q.ALGO_BITPLANE}
    for mode, kernel in ((q.EPI_INT32, int1 if wb == 1 else int2), (q.EPI_SCALE_F32, other), (q.EPI_BN_F32, other)):
        assert q.resolve_algo(*geo, mode=mode) == algo[kernel]
        assert kernel in q.kernel_name(*geo, mode=mode)
    act = q.pack_act(x.to(dev), ab)
    wq, _ = q.pack_weight(wt.to(dev), wb)
    lw, _ = oracle.quantize_weights(wt.numpy(), wb)
    acc = oracle.qconv_acc(oracle.quantize(x.numpy(), ab), lw, ab, s, p)
    out, _ = q.conv(act, wq, *geo)
    np.testing.assert_array_equal(out.cpu().numpy(), acc)
    out, _ = q.conv(act, wq, *geo, mode=q.EPI_BN_F32, bn_k=kk.to(dev), bn_b=bb.to(dev))
    z = oracle.epi_bn(acc, kk.numpy(), bb.numpy(), oracle.level_shift(ab) + oracle.level_shift(wb))
    np.testing.assert_array_equal(out.cpu().numpy(), z)


# fp16 operands: the weight ring of 3 x 3 layers on both 256-row shapes, with one
# and two words per stage (whole small images, runs of one image), a last stage
# of one word, and the layers beside it (another kernel size)
@pytest.mark.parametrize("ab, wb", [(1, 16), (2, 16), (3, 16), (16, 1)])
@pytest.mark.parametrize("n, cin, h, cout, k", [(256, 160, 7, 320, 3), (70, 96, 28, 128, 3), (70, 32, 28, 64, 3),
                                                (40, 64, 28, 128, 5)])
def test_fp16_integer_values(dev, n, cin, h, cout, k, ab, wb):
    g = synth.generator(37 + cin)
    small = torch.randint(-3, 4, (n, cin, h, h), generator=g).float()  # integers: every partial sum is exact in fp32
    x = small if ab == 16 else _x(38, (n, cin, h, h))
    wt = torch.randint(-3, 4, (cout, cin, k, k), generator=g).float() if wb == 16 else \
        synth.normal(g, (cout, cin, k, k), 2.0 / (k * k * cin))
    kk, bb = synth.uniform(g, (cout,), 0.001, 0.05), synth.normal(g, (cout,), 0.1)
    wq, _ = q.pack_weight(wt.to(dev), wb)
    out, _ = q.conv(q.pack_act(x.to(dev), ab), wq, n, cin, h, h, cout, k, 1, k // 2, ab, wb, mode=q.EPI_BN_F32,
                    bn_k=kk.to(dev), bn_b=bb.to(dev))
    m = min(n, 6)  # the first and the last images against the oracle
    idx = list(range(m // 2)) + list(range(n - m // 2, n))
    if wb == 16:
        want = oracle.qconv16w_layer(oracle.quantize(x[idx].numpy(), ab), oracle.to_f16(wt.numpy()), ab, 1, k // 2, "bn",
                                     k=kk.numpy(), b=bb.numpy())
    else:
        lw, _ = oracle.quantize_weights(wt.numpy(), wb)
        want = oracle.qconv16_layer(oracle.to_f16(x[idx].numpy()), lw, wb, 1, k // 2, "bn", k=kk.numpy(), b=bb.numpy())
    want = want[0] if isinstance(want, tuple) else want
    np.testing.assert_array_equal(out.cpu().numpy()[idx], want)


def _launched(fn):
    """What fn returns, and the names of the library's kernels that it launched."""
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        r = fn()
        torch.cuda.synchronize()
    return r, [re.sub(r"^void qc::mfma::|\(qc::mfma::.*$", "", e.key) for e in prof.key_averages() if "qc::" in e.key]


# the unstaged form of the store-overlapped kernel (1- and 2-bit inputs): ragged
# maps, channels and batches (a last block of a few pixels, waves and channel
# tiles with nothing to do), strides, 1 x 1, one and two k-steps a tap; and the
# staged 64-channel shape on layers beside the unstaged form's limits
DIRECT_CASES = [
    # n, cin, h, w, cout, k, stride, pad, packed output alone on it too
    (37, 40, 56, 57, 100, 3, 1, 1, True),
    (67, 64, 55, 56, 130, 1, 2, 0, True),
    (3, 64, 150, 151, 64, 3, 1, 1, True),
    (70, 100, 28, 27, 90, 3, 1, 1, False),
    (46, 64, 33, 29, 96, 3, 1, 1, True),
]
STAGED_CASES = [
    (128, 128, 32, 32, 64, 3, 1, 1, False),  # items that end with the image, over 9 k-steps
    (130, 100, 32, 32, 60, 3, 1, 1, False),  # a last k-step of one word, ragged channels, an odd number of items
    (2048, 64, 16, 16, 32, 3, 2, 1, False),  # 4096 tiles; stride 2, whole images
    (128, 64, 33, 31, 96, 3, 2, 1, True),    # the same, ragged items and channels
]


@pytest.mark.parametrize("ab, wb", [(1, 1), (2, 1), (2, 2), (1, 3)])
@pytest.mark.parametrize("case, cfg", [(c, 3) for c in DIRECT_CASES] + [(c, 1) for c in STAGED_CASES])
def test_store_overlapped_forms(dev, case, cfg, ab, wb):
    n, cin, h, w, cout, k, s, p, packs = case
    g = synth.generator(39 + n + cin)
    x = _x(40 + n, (n, cin, h, w))
    wt = synth.normal(g, (cout, cin, k, k), 2.0 / (k * k * cin))
    kk, bb = synth.uniform(g, (cout,), 0.001, 0.05), synth.normal(g, (cout,), 0.1)
    ho, wo = q.out_size(h, k, s, p), q.out_size(w, k, s, p)
    res = synth.normal(g, (n, cout, ho, wo), 1.0)
    act = q.pack_act(x.to(dev), ab)
    wq, sc = q.pack_weight(wt.to(dev), wb)
    lw, osc = oracle.quantize_weights(wt.numpy(), wb)
    acc = oracle.qconv_acc(oracle.quantize(x.numpy(), ab), lw, ab, s, p)
    shift = oracle.level_shift(ab) + oracle.level_shift(wb)
    z = oracle.epi_bn(acc, kk.numpy(), bb.numpy(), shift)
    geo = (n, cin, h, w, cout, k, s, p, ab, wb)
    algo = q.ALGO_MFMA_FP4
    name, packed = f"conv_mfma_pp_kernel<1, {ab}, {cfg}, 0>", f"conv_mfma_pp_kernel<1, {ab}, {cfg}, {ab}>"
    assert q.kernel_name(*geo, algo=algo) == name
    assert q.kernel_name(*geo, mode=q.EPI_BN_F32, flags=q.EPI_RESIDUAL, out_bits=ab, packed_out=True, algo=algo) == packed
    alone = q.kernel_name(*geo, mode=q.EPI_BN_PACK, out_bits=ab, packed_out=True, algo=algo)
    assert (alone == packed) == packs, alone
    (out, _), ran = _launched(lambda: q.conv(act, wq, *geo, algo=algo))
    assert ran == [name]
    np.testing.assert_array_equal(out.cpu().numpy(), acc)
    out, _ = q.conv(act, wq, *geo, mode=q.EPI_SCALE_F32, scale=sc, algo=algo)
    np.testing.assert_array_equal(out.cpu().numpy(), oracle.epi_scale(acc, osc, shift))
    kw = dict(bn_k=kk.to(dev), bn_b=bb.to(dev), algo=algo)
    out, _ = q.conv(act, wq, *geo, mode=q.EPI_BN_F32, **kw)
    np.testing.assert_array_equal(out.cpu().numpy(), z)
    for ob in (ab, 3):  # the input's width, and one that another kernel serves
        words = q.packed_act_words(n, cout, ho, wo, ob)
        outp = torch.full((words + 16,), 0x5A5A5A5A, dtype=torch.int32, device=dev)
        q.conv(act, wq, *geo, mode=q.EPI_BN_PACK, out_bits=ob, out_packed=outp[:words], **kw)
        got = outp.cpu().numpy()
        np.testing.assert_array_equal(unpack_act(got[:words], n, cout, ho, wo, ob),
                                      oracle.quantize(oracle.hardtanh(z), ob))
        assert tail_bits_zero(got[:words], cout, ob) and (got[words:] == 0x5A5A5A5A).all()
        zr = oracle.add(z, res.numpy())
        out, _ = q.conv(act, wq, *geo, mode=q.EPI_BN_F32, flags=q.EPI_RESIDUAL, residual=res.to(dev), out_bits=ob,
                        out_packed=outp[:words], **kw)
        np.testing.assert_array_equal(out.cpu().numpy(), zr)
        np.testing.assert_array_equal(unpack_act(outp.cpu().numpy()[:words], n, cout, ho, wo, ob),
                                      oracle.quantize(oracle.hardtanh(zr), ob))


# Residual layers whose planes are not whole runs of 64 bytes: the form on both
# sides of each limit (items of 256 pixels x 64 channels; planes of a multiple of four
# pixels and not, up to 9 k-steps and more)
@pytest.mark.parametrize("n, cin, h, w, cout, cfg", [
    (512, 64, 25, 25, 64, 3), (513, 64, 25, 25, 64, 1), (513, 64, 25, 28, 64, 3), (513, 64, 26, 26, 64, 3),
    (513, 128, 25, 25, 64, 1), (512, 128, 30, 30, 64, 3), (513, 128, 30, 30, 64, 1), (513, 128, 28, 28, 64, 3),
    (149, 100, 25, 23, 90, 3), (150, 100, 25, 23, 90, 1), (170, 100, 25, 23, 90, 1), (171, 100, 25, 23, 90, 3),
    (150, 64, 25, 23, 90, 1), (150, 100, 26, 22, 90, 3)])
def test_residual_form(dev, n, cin, h, w, cout, cfg):
    geo = (n, cin, h, w, cout, 3, 1, 1, 2, 2)
    kw = dict(mode=q.EPI_BN_F32, flags=q.EPI_RESIDUAL, out_bits=2)
    assert q.kernel_name(*geo, packed_out=True, **kw) == f"conv_mfma_pp_kernel<1, 2, {cfg}, 2>"
    assert q.kernel_name(*geo, mode=q.EPI_BN_F32) == "conv_mfma_pp_kernel<1, 2, 3, 0>"
    g = torch.Generator(device=dev).manual_seed(54)
    x = torch.randn((n, cin, h, w), generator=g, device=dev)
    res = torch.randn((n, cout, h, w), generator=g, device=dev)
    wq, _ = q.pack_weight(torch.randn((cout, cin, 3, 3), generator=g, device=dev), 2)
    bn = dict(bn_k=torch.rand(cout, generator=g, device=dev) * 0.05, bn_b=torch.randn(cout, generator=g, device=dev))
    outp = torch.zeros(q.packed_act_words(n, cout, h, w, 2), dtype=torch.int32, device=dev)
    out, _ = q.conv(q.pack_act(x, 2), wq, *geo, residual=res, out_packed=outp, **kw, **bn)
    assert torch.equal(outp, q.pack_act(out, 2))  # (|z| <= 1 or not: the threshold is below 1)
    for i0, m in ((0, 2), (n - 2, 2)):  # the first and the last images alone, on another kernel
        part, _ = q.conv(q.pack_act(x[i0:i0 + m].contiguous(), 2), wq, m, *geo[1:], mode=q.EPI_BN_F32, **bn)
        assert torch.equal(out[i0:i0 + m], part + res[i0:i0 + m])


# A stride-2 layer of wide rows: the input tile of the 256-pixel shapes does not
# fit from 147 columns on, and no kernel that is then not launched is named
@pytest.mark.parametrize("w, kernel", [(146, "conv_mfma_pp_kernel<1, 2, 3, "), (147, "conv_mfma_kernel<1, 2, 2, 1>"),
                                       (160, "conv_mfma_kernel<1, 2, 2, 1>")])
def test_wide_rows(dev, w, kernel):
    n, c = 16, 64
    geo = (n, c, w, w, c, 3, 2, 1, 2, 2)
    x = _x(52, (n, c, w, w))
    g = synth.generator(53)
    wt = synth.normal(g, (c, c, 3, 3), 2.0 / (9 * c))
    kk, bb = synth.uniform(g, (c,), 0.001, 0.05), synth.normal(g, (c,), 0.1)
    act = q.pack_act(x.to(dev), 2)
    wq, _ = q.pack_weight(wt.to(dev), 2)
    lw, _ = oracle.quantize_weights(wt.numpy(), 2)
    acc = oracle.qconv_acc(oracle.quantize(x.numpy(), 2), lw, 2, 2, 1)
    kw = dict(mode=q.EPI_BN_PACK, out_bits=2)
    names = q.kernel_name(*geo), q.kernel_name(*geo, packed_out=True, **kw)
    (out, _), ran = _launched(lambda: q.conv(act, wq, *geo))
    assert ran == [names[0]] and names[0].startswith(kernel), (ran, names)
    np.testing.assert_array_equal(out.cpu().numpy(), acc)
    bn = kk.to(dev), bb.to(dev)
    (_, outp), ran = _launched(lambda: q.conv(act, wq, *geo, bn_k=bn[0], bn_b=bn[1], **kw))
    assert ran == [names[1]] and names[1].startswith(kernel), (ran, names)
    z = oracle.epi_bn(acc, kk.numpy(), bb.numpy(), 2 * oracle.level_shift(2))
    ho = q.out_size(w, 3, 2, 1)
    np.testing.assert_array_equal(unpack_act(outp.cpu().numpy(), n, c, ho, ho, 2), oracle.quantize(oracle.hardtanh(z), 2))


# Buffers of 2147483640 bytes: lanes without an element use the byte offset
# 2147483632 of a buffer resource, which lies inside such a buffer.  An output of
# that size (its last group of 32 pixels has one): no such lane may store into
# it; inputs of that size: the pixels outside an image are 0.
@pytest.mark.parametrize("ab, algo", [(1, q.ALGO_MFMA_FP4), (3, q.ALGO_MFMA_FP4), (2, q.ALGO_MFMA_I8)])
def test_output_past_the_masked_offset(dev, ab, algo):
    n, cin, h, w, cout = 4859, 64, 15, 29, 254
    assert n * cout * h * w * 4 == 2147483640
    g = torch.Generator(device=dev).manual_seed(50)
    x = torch.randn((n, cin, h, w), generator=g, device=dev)
    wq, _ = q.pack_weight(torch.randn((cout, cin, 3, 3), generator=g, device=dev), 1)
    out, _ = q.conv(q.pack_act(x, ab), wq, n, cin, h, w, cout, 3, 1, 1, ab, 1, algo=algo)
    for i0, m in ((0, 3), (n // 2, 40), (n - 50, 50)):  # the same images in small batches
        part, _ = q.conv(q.pack_act(x[i0:i0 + m].contiguous(), ab), wq, m, cin, h, w, cout, 3, 1, 1, ab, 1, algo=algo)
        assert torch.equal(out[i0:i0 + m], part)


def test_input_past_the_masked_offset(dev):
    n, h, w, cout = 18705, 113, 127, 1
    assert q.packed_act_words(n, 1, h, w, 2) * 4 == 2147483640
    g = torch.Generator(device=dev).manual_seed(51)
    x = torch.randn((n, 1, h, w), generator=g, device=dev)
    x.view(-1)[-8:] = 2.0  # the words at the offset: nonzero levels
    wq, _ = q.pack_weight(torch.randn((cout, 1, 3, 3), generator=g, device=dev), 1)
    geo = (1, h, w, cout, 3, 1, 1, 2, 1)
    out, _ = q.conv(q.pack_act(x, 2), wq, n, *geo, algo=q.ALGO_MFMA_FP4)
    for i0, m in ((0, 40), (n - 40, 40)):
        part, _ = q.conv(q.pack_act(x[i0:i0 + m].contiguous(), 2), wq, m, *geo, algo=q.ALGO_MFMA_FP4)
        assert torch.equal(out[i0:i0 + m], part)


# the last FC reads operands 16 inputs (fp32) or half a word (packed signs)
# ahead: odd and even numbers of groups, remainders, one chunk and several
@pytest.mark.parametrize("inputs", [3, 15, 16, 17, 32, 47, 64, 95, 192, 208, 223, 1024, 1056, 1071])
@pytest.mark.parametrize("bits", [0, 1])
def test_last_fc(dev, bits, inputs):
    n, out = 67, 6
    g = synth.generator(900 + inputs)
    x = synth.normal(g, (n, inputs, 1, 1), 1.0)
    wt = synth.normal(g, (out, inputs), 2.0 / inputs)
    b = synth.normal(g, (out,), 0.1)
    net = q.Net(inputs, 1, 1)
    net.fc_f32(net.quantize(0, 1) if bits else 0, wt.to(dev), b.to(dev))
    ws = torch.empty(max(net.workspace_bytes(n), 1), dtype=torch.uint8, device=dev)
    got = torch.empty((n, out), dtype=torch.float32, device=dev)
    net.forward(x.to(dev), got, ws)
    xin = oracle.quantize(x.numpy(), 1).astype(np.float32) if bits else x.numpy()
    np.testing.assert_array_equal(got.cpu().numpy(), oracle.fc_f32(xin.reshape(n, -1), wt.numpy(), b.numpy()))

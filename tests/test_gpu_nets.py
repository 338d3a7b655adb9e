"""GPU parity: the layer-chained forwards (bnn_net_*) against the oracle's compositions."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import host, to_dev, words
from oracle import nets

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bnn():
    import paper_2006_16578_amd as b
    b.load()
    return b


def build_mlp(bnn, params):
    net = bnn.Net()
    net.input_u8(params["dims"][0], params["in_thr"])
    nl = len(params["W"])
    for l in range(nl):
        thr = to_dev(params["thr"][l]) if l < nl - 1 else None
        net.add_fc(to_dev(params["W"][l]), thr, params["K"][l])
    return net


@pytest.mark.parametrize("batch", [8, 1024, 37])
@pytest.mark.parametrize("path", [0, 1, 2])
def test_mlp(bnn, orc, batch, path):
    params = wl.mlp_params()
    imgs = wl.mlp_images(batch)
    ref, hidden = nets.mlp_forward(imgs, params, keep=True)
    net = build_mlp(bnn, params)
    scores = host(net.forward(to_dev(imgs), path=path))
    for l in range(3):
        assert np.array_equal(words(net.layer_bits(l + 1)), hidden[l]), "hidden layer %d" % l
    assert np.array_equal(scores, ref)


# run: the layers of the one launch, with sums and with thresholds in the last layer
@pytest.mark.parametrize("dims,u8,batch,run", [
    ((784, 1024, 1024, 1024, 10), True, 4097, (5, 5)), ((784, 1024, 1024, 1024, 10), True, 4081, (5, 5)),    # 32-row workgroups; the last of 16 rows ragged
    ((16, 33, 1), True, 1, (3, 3)), ((17, 64, 64, 64, 64), True, 15, (5, 5)), ((1000, 65, 129, 31, 64), True, 17, (5, 5)), ((3001, 70, 10), True, 129, (3, 3)),
    ((1, 1, 1), False, 16, (3, 3)), ((31, 1100, 3), False, 33, (3, 3)), ((2049, 127, 900, 12), False, 200, (4, 4)),
    ((128, 64, 64, 64, 64, 64, 64, 5), False, 5000, (5, 5)),               # (four layers behind the input at most)
    ((15, 100, 10), True, 40, (0, 0)), ((300, 100, 65), True, 40, (2, 3)),  # rows of 15 bytes, 65 sums (its first layers are the run's)
    ((4001, 70, 10), True, 129, (0, 0))])                                  # beyond LDS
@pytest.mark.parametrize("last_thr", [False, True])
def test_fc_chain(bnn, orc, dims, u8, batch, run, last_thr):
    # fully-connected layers at the head of a network in one launch: widths on and off words, 64-column groups and 1024-bit parts, and
    # thresholds no sum can reach, or every sum does
    rng = np.random.default_rng(sum(dims) + batch)
    p = wl.mlp_params(dims, config=97)
    thr = [rng.integers(-40, 41, size=n).astype(np.int32) for n in dims[1:]]
    for t in thr:
        t[::7] = rng.choice([-2 ** 31, 2 ** 31 - 1, 0], size=t[::7].shape)
    in_thr = int(rng.choice([127, 0, 255]))
    net = bnn.Net()
    if u8:
        net.input_u8(dims[0], in_thr)
        x = rng.integers(0, 256, size=(batch, dims[0])).astype(np.uint8)
        bits = orc.pack_u8(x, in_thr, ldb_w=p["W"][0].shape[1])
    else:
        net.input_bits(dims[0])
        x = bits = wl.random_bits(rng, batch, dims[0], p["W"][0].shape[1])
    nl = len(dims) - 1
    for l in range(nl):
        net.add_fc(to_dev(p["W"][l]), to_dev(thr[l]) if l + 1 < nl or last_thr else None, p["K"][l])
    assert net.fc_run(batch) == run[last_thr]
    out = net.forward(to_dev(x))
    if u8:
        assert np.array_equal(words(net.layer_bits(0)), bits)
    for l in range(nl):
        v = orc.bmm(bits, p["W"][l], p["K"][l])
        if l + 1 == nl and not last_thr:
            assert np.array_equal(host(out), v)
            break
        bits = orc.threshold_pack(v, thr[l], ldb_w=wl.round_up(wl.nwords(dims[l + 1]), 4))
        assert np.array_equal(words(net.layer_bits(l + 1)), bits), "layer %d" % (l + 1)


# The same layers recorded into a graph, where fewer of them are worth one launch: replays with eager passes and other inputs between them
@pytest.mark.parametrize("dims,u8,batch,queued,recorded", [
    ((784, 1024, 1024, 1024, 10), True, 8, 5, 0), ((784, 1024, 1024, 1024, 10), True, 100, 5, 5), ((1024, 1024, 10), False, 150, 3, 0), ((256, 256, 256, 256, 10), False, 16, 5, 5)])
def test_fc_run_recorded(bnn, orc, dims, u8, batch, queued, recorded):
    rng = np.random.default_rng(sum(dims) + batch)
    p = wl.mlp_params(dims, config=98)
    net = bnn.Net()
    net.input_u8(dims[0], 127) if u8 else net.input_bits(dims[0])
    for l, thr in enumerate(p["thr"] + [None]):
        net.add_fc(to_dev(p["W"][l]), to_dev(thr) if thr is not None else None, p["K"][l])
    assert net.fc_run(batch) == queued and net.fc_run(batch, recorded=True) == recorded

    def inputs():
        x = rng.integers(0, 256, size=(batch, dims[0])).astype(np.uint8) if u8 else wl.random_bits(rng, batch, dims[0], p["W"][0].shape[1])
        bits = orc.pack_u8(x, 127, ldb_w=p["W"][0].shape[1]) if u8 else x
        for l, thr in enumerate(p["thr"]):
            bits = orc.threshold_pack(orc.bmm(bits, p["W"][l], p["K"][l]), thr, ldb_w=p["W"][l + 1].shape[1])
        return to_dev(x), orc.bmm(bits, p["W"][-1], p["K"][-1])

    x, ref = inputs()
    static, out = x.clone(), torch.empty((batch, dims[-1]), dtype=torch.int32, device="cuda")
    assert np.array_equal(host(net.forward(static)), ref)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            net.forward(static, out=out)
    torch.cuda.current_stream().wait_stream(side)
    for _ in range(4):
        x, ref = inputs()
        static.copy_(x)
        out.zero_()
        graph.replay()
        assert np.array_equal(host(out), ref)
        assert np.array_equal(host(net.forward(x)), ref)


def build_resnet(bnn, p, hw, pad_mode=0):
    net = bnn.Net()
    net.input_conv_f32(to_dev(p["stem_w"]), to_dev(p["stem_thr"]), hw, hw, 4, 3)
    for blk in p["blocks"]:
        net.add_block(to_dev(blk["W1"]), to_dev(blk["thr1"]), to_dev(blk["W2"]), to_dev(blk["thr2"]),
                      to_dev(blk["Wd"]) if "Wd" in blk else None, blk["cin"], blk["cout"], blk["stride"], pad_mode)
    net.add_head_f32(to_dev(p["fc_w"]))
    return net


def first_layer_values(bnn, xd, w, thr, stride, pad):
    """fp32 output of a real-weight first layer from the kernel bnn_net_forward runs for it: the bf16 split
    kernel with six term products, or the fp32 matrix-core kernel when the filter bank does not fit it."""
    try:
        _, y = bnn.conv_f32_split_thr(xd, w, thr, stride, pad, want_f32=True, products=6)
    except bnn.BnnError as e:
        if e.status != -3:
            raise
        _, y = bnn.conv_f32_thr(xd, w, thr, stride, pad, want_f32=True)
    return y


def check_resnet(bnn, orc, p, x, hw, path, tier, pad_mode=0):
    """Protocol for a network whose first layer is fp32: the stem output must match within
    1e-4 * max(|o|, rms(o)); a stem bit may differ from the oracle's only where the oracle's value
    is that close to the threshold; the oracle's binarized chain is then run from the GPU's stem
    bits and every later bit tensor must match exactly; logits within the same fp32 tolerance."""
    xd = to_dev(x)
    net = build_resnet(bnn, p, hw, pad_mode)
    logits = host(net.forward(xd, path=path))
    stem_bits_gpu = words(net.layer_bits(0)).reshape(x.shape[0], hw // 4, hw // 4, -1)
    # fp32 stem values, from the kernel the layer chain runs (bf16 x 3 split, six term products)
    y = first_layer_values(bnn, xd, to_dev(p["stem_w"]), to_dev(p["stem_thr"]), 4, 3)
    stem_ref = orc.conv_f32(x, p["stem_w"], 4, 3)
    tol = 1e-4 * np.maximum(np.abs(stem_ref), np.sqrt((stem_ref.astype(np.float64) ** 2).mean()))
    err = np.abs(host(y) - stem_ref)
    print("stem: max |gpu - oracle| = %.3e, max error / tolerance = %.3e" % (err.max(), (err / tol).max()), flush=True)
    assert (err <= tol).all()
    ref_bits = orc.pack_f32(stem_ref, p["stem_thr"])
    diff = stem_bits_gpu ^ ref_bits
    ndiff = 0
    if diff.any():
        # every differing bit must belong to a value inside the tolerance of its threshold
        C = p["stem_w"].shape[0]
        d = orc.unpack_pm1(diff.reshape(-1, diff.shape[-1]), C).reshape(stem_ref.shape) > 0
        assert (np.abs(stem_ref - p["stem_thr"])[d] <= tol[d]).all()
        ndiff = int(d.sum())
    print("stem bits that differ from the oracle's (all inside the fp32 tolerance): %d of %d" % (ndiff, stem_ref.size),
          flush=True)
    tr = nets.resnet18_forward(x, p, stem_bits=stem_bits_gpu, tier=tier, keep=True, pad_mode=pad_mode)
    for b in range(len(p["blocks"])):
        got = words(net.layer_bits(b + 1)).reshape(tr["y%d" % b].shape)
        assert np.array_equal(got, tr["y%d" % b]), "block %d output bits" % b
    ref_logits = tr["logits"]
    tol = 1e-4 * np.maximum(np.abs(ref_logits), np.sqrt((ref_logits.astype(np.float64) ** 2).mean()))
    assert (np.abs(logits - ref_logits) <= tol).all()


@pytest.mark.parametrize("path", [1, 2])
def test_resnet_small(bnn, orc, path):
    blocks = ((64, 64, 1), (64, 96, 2), (96, 96, 1), (96, 128, 2))
    p = wl.resnet18_params(blocks=blocks, classes=13, config=95)
    x = wl.resnet18_input(3, hw=32, config=95)
    check_resnet(bnn, orc, p, x, 32, path, tier=0)


@pytest.mark.parametrize("pad_mode", [0, 1])
@pytest.mark.parametrize("widths", [(64, 80, 80, 96), (64, 64, 128, 128)])
def test_resnet_small_widths_and_padding(bnn, orc, widths, pad_mode):
    # residual chains with channel counts that are not multiples of 32 (row-major 16-bit sums, pad bits inside the
    # last word of a pixel) and with multiples of 32 (blocked sums), in both padding conventions; 5 images of 40x40
    # make ragged 32-row blocks at every resolution
    a, b, c, d = widths
    blocks = ((64, a, 1), (a, b, 2), (b, c, 1), (c, d, 2), (d, d, 1))
    p = wl.resnet18_params(blocks=blocks, classes=21, config=96)
    x = wl.resnet18_input(5, hw=40, config=96)
    check_resnet(bnn, orc, p, x, 40, 0, tier=0, pad_mode=pad_mode)


@pytest.mark.parametrize("seed", [301, 302, 303, 304, 305, 306])
def test_resnet_random_chains(bnn, orc, seed):
    # random residual chains: widths on and off multiples of 32, stride-1 and stride-2 blocks with and without a
    # 1x1 shortcut, random batch and image size, both padding conventions
    rng = np.random.default_rng(seed)
    widths = [int(rng.choice([32, 64, 80, 96, 128, 160])) for _ in range(5)]
    blocks, cin = [], widths[0]
    for b in range(int(rng.integers(3, 6))):
        cout = cin if rng.random() < 0.5 else int(rng.choice(widths))
        stride = 2 if (cout != cin and rng.random() < 0.6) else 1
        blocks.append((cin, cout, stride))
        cin = cout
    hw = int(rng.choice([24, 40, 56]))
    batch = int(rng.integers(1, 7))
    pad_mode = int(rng.integers(0, 2))
    print("chain", blocks, "hw", hw, "batch", batch, "pad_mode", pad_mode, flush=True)
    p = wl.resnet18_params(blocks=tuple(blocks), classes=int(rng.integers(3, 40)), config=seed)
    x = wl.resnet18_input(batch, hw=hw, config=seed)
    check_resnet(bnn, orc, p, x, hw, 0, tier=1, pad_mode=pad_mode)


@pytest.mark.parametrize("blocks,hw,batch,pad_mode", [
    (((64, 64, 1), (64, 64, 1), (64, 96, 2)), 40, 340, 0), (((64, 64, 1), (64, 64, 1), (64, 96, 2)), 40, 340, 1),
    (((128, 128, 1), (128, 128, 1)), 32, 2600, 1)])
def test_resnet_chains_patch_kernel(bnn, orc, blocks, hw, batch, pad_mode):
    # residual chains whose stride-1 layers are large enough for the 3x3 kernel with LDS-resident filters (64- and
    # 128-column forms): bits-only layers, the first residual taken from bits, blocked 16-bit sums in and out, in both
    # padding conventions; 10x10 and 8x8 feature maps, so most 64-pixel tiles cross image rows and images
    H = hw // 4
    cin, cout, _ = blocks[0]
    assert bnn.bconv_kernel_name(batch, H, H, cin, cout, 3, 1, 1).startswith("mfma_fp4_conv3x3_patch")
    p = wl.resnet18_params(blocks=blocks, classes=10, config=97)
    x = wl.resnet18_input(batch, hw=hw, config=97)
    check_resnet(bnn, orc, p, x, hw, 0, tier=1, pad_mode=pad_mode)


def test_resnet18_batch8(bnn, orc):
    p = wl.resnet18_params()
    x = wl.resnet18_input(8)
    check_resnet(bnn, orc, p, x, 224, 0, tier=1)


def test_resnet18_batch256(bnn, orc):
    # the configuration bench.py times (batch 256, automatic path); full comparison of every
    # block's bits against the packed tier-1 oracle chain (tier 1 == tier 0 is pinned on CPU and
    # re-checked above at batch 8 sizes by the small-network test)
    p = wl.resnet18_params()
    x = wl.resnet18_input(256)
    check_resnet(bnn, orc, p, x, 224, 0, tier=1)


@pytest.mark.parametrize("shape", [(9, 7, 7, 512, 1000), (35, 3, 5, 200, 70), (1, 1, 1, 33, 1), (16, 8, 8, 1024, 130), (40, 15, 17, 36, 33)])
def test_head_pooled(bnn, orc, shape):
    # with a pooled-sum output the head runs as two kernels (pool, then FC), without it as one fused kernel
    N, H, W, C, J = shape
    rng = np.random.default_rng(12 + C)
    bits = wl.random_bits(rng, (N, H, W), C)
    w = rng.normal(0, 0.02, size=(J, C)).astype(np.float32)
    pr = orc.sumpool_pm1(bits, C)
    ref = orc.head_fc_f32(pr, w, float(H * W))
    tol = 1e-4 * np.maximum(np.abs(ref), np.sqrt((ref.astype(np.float64) ** 2).mean()))
    y, pooled = bnn.head_f32(to_dev(bits), to_dev(w), C, want_pooled=True)
    assert np.array_equal(host(pooled), pr)
    assert (np.abs(host(y) - ref) <= tol).all()
    y1 = bnn.head_f32(to_dev(bits), to_dev(w), C)
    assert (np.abs(host(y1) - ref) <= tol).all()


# The FC of a head beyond one workgroup per compute unit: passes of 256 channels instead of 512, ragged last ones and one alone; images, outputs off 32
@pytest.mark.parametrize("shape", [(8200, 2, 2, 512, 10), (300, 1, 1, 1020, 900), (290, 3, 1, 260, 1000), (4130, 1, 2, 64, 70)])
def test_head_many_workgroups(bnn, orc, shape):
    test_head_pooled(bnn, orc, shape)


# Its pooling from 2^18 packed words on: four lanes to a word instead of sixteen; a last wave with some of its sixteen words, positions off four, a partly filled word
@pytest.mark.parametrize("shape", [(32770, 1, 3, 250, 3), (16391, 2, 1, 512, 2), (8740, 1, 1, 964, 1)])
def test_head_pooling_of_many_words(bnn, orc, shape):
    test_head_pooled(bnn, orc, shape)


@pytest.mark.parametrize("shape", [(2, 21, 19, 3, 5, 7, 4, 3), (1, 9, 9, 1, 1, 3, 1, 1), (3, 16, 12, 4, 70, 5, 2, 2),
                                   (2, 32, 32, 3, 64, 7, 4, 3), (1, 8, 8, 2, 33, 1, 1, 0)])
def test_conv_f32_shapes(bnn, orc, shape):
    N, H, W, C, O, k, st, pad = shape
    rng = np.random.default_rng(sum(shape))
    x = rng.uniform(-1, 1, size=(N, H, W, C)).astype(np.float32)
    w = rng.normal(0, 0.05, size=(O, k, k, C)).astype(np.float32)
    thr = rng.normal(0, 0.05, size=O).astype(np.float32)
    bits, y = bnn.conv_f32_thr(to_dev(x), to_dev(w), to_dev(thr), st, pad, want_f32=True)
    ref = orc.conv_f32(x, w, st, pad)
    tol = 1e-4 * np.maximum(np.abs(ref), np.sqrt((ref.astype(np.float64) ** 2).mean()))
    assert host(y).shape == ref.shape
    assert (np.abs(host(y) - ref) <= tol).all()
    # the bits are exactly the GPU's own fp32 values thresholded, pad bits zero
    assert np.array_equal(words(bits), orc.pack_f32(host(y), thr))


# ------------------------------------------------------------------ max-pooling and the other Table-5 networks
@pytest.mark.parametrize("shape", [(2, 8, 8, 40, 2, 2), (1, 7, 9, 64, 2, 2), (3, 6, 6, 33, 3, 1), (1, 5, 5, 1, 2, 1),
                                   (5, 27, 27, 256, 2, 2), (2, 13, 13, 512, 3, 2), (1, 2, 2, 1024, 2, 2),
                                   (3, 17, 5, 96, 2, 1)])
def test_maxpool_or(bnn, orc, shape):
    N, H, W, C, win, st = shape
    bits = wl.random_bits(np.random.default_rng(sum(shape)), (N, H, W), C)
    got = words(bnn.maxpool_or(to_dev(bits), C, win, st))
    assert np.array_equal(got, orc.maxpool_pm1(bits, C, win, st))


def test_maxpool_or_errors(bnn):
    bits = to_dev(wl.random_bits(np.random.default_rng(0), (1, 4, 4), 32))
    for win, st in ((0, 1), (5, 1), (2, 0)):
        with pytest.raises(bnn.BnnError):
            bnn.maxpool_or(bits, 32, win, st)


def check_cnn(bnn, orc, spec, x, path, tier):
    layers, hw = spec["layers"], spec["in_hw"]
    net = bnn.Net.from_layers(layers, hw)
    xd = to_dev(x)
    scores = host(net.forward(xd, path=path))
    L0 = layers[0]
    if L0["op"] == "bwn":
        _, y = bnn.bwn_conv_thr(xd, to_dev(L0["W"]), to_dev(L0["thr"]), L0["C"], L0["stride"], L0["pad"], want_f32=True)
        ref0 = orc.bwn_conv_f32(x, L0["W"], L0["C"], L0["stride"], L0["pad"])
        cout = L0["W"].shape[0]
    else:
        y = first_layer_values(bnn, xd, to_dev(L0["w"]), to_dev(L0["thr"]), L0["stride"], L0["pad"])
        ref0 = orc.conv_f32(x, L0["w"], L0["stride"], L0["pad"])
        cout = L0["w"].shape[0]
    tol = 1e-4 * np.maximum(np.abs(ref0), np.sqrt((ref0.astype(np.float64) ** 2).mean()))
    err = np.abs(host(y) - ref0)
    print("first layer: max |gpu - oracle| = %.3e, max error / tolerance = %.3e" % (err.max(), (err / tol).max()), flush=True)
    assert (err <= tol).all()
    ref_bits = orc.pack_f32(ref0, L0["thr"])
    bits0 = words(net.layer_bits(0)).reshape(ref_bits.shape)
    diff = bits0 ^ ref_bits
    if diff.any():
        d = orc.unpack_pm1(diff.reshape(-1, diff.shape[-1]), cout).reshape(ref0.shape) > 0
        assert (np.abs(ref0 - L0["thr"])[d] <= tol[d]).all()
        print("first-layer bits inside the fp32 tolerance that differ:", int(d.sum()), flush=True)
    outs = nets.cnn_forward(x, layers, stem_bits=bits0, tier=tier, keep=True)
    for i in range(1, len(layers) - 1):
        got = words(net.layer_bits(i)).reshape(outs[i].shape)
        assert np.array_equal(got, outs[i]), "layer %d (%s) output bits" % (i, layers[i]["op"])
    assert scores.dtype == np.int32 and np.array_equal(scores, outs[-1])


@pytest.mark.parametrize("name,batch,path,tier,first", [
    ("cifar_vgg", 5, 1, 0, "bwn"), ("cifar_vgg", 5, 2, 0, "f32"), ("cifar_vgg", 64, 0, 1, "bwn"),
    ("cifar_resnet14", 5, 1, 0, "f32"), ("cifar_resnet14", 5, 2, 0, "bwn"), ("cifar_resnet14", 64, 0, 1, "bwn"),
    ("alexnet", 3, 2, 1, "f32"), ("alexnet", 16, 0, 1, "bwn"), ("vgg16", 2, 0, 1, "bwn"), ("vgg16", 1, 0, 1, "f32")])
def test_table5_networks(bnn, orc, name, batch, path, tier, first):
    check_cnn(bnn, orc, wl.cnn_layers(name, first=first), wl.cnn_input(name, batch), path, tier)


@pytest.mark.parametrize("shape", [(2, 21, 19, 3, 5, 7, 4, 3), (1, 9, 9, 1, 1, 3, 1, 1), (3, 16, 12, 4, 70, 5, 2, 2),
                                   (2, 32, 32, 3, 64, 7, 4, 3), (1, 8, 8, 2, 33, 1, 1, 0), (2, 32, 32, 3, 128, 3, 1, 1),
                                   (1, 40, 37, 3, 128, 11, 4, 2), (2, 12, 12, 35, 96, 3, 2, 1), (1, 6, 6, 1, 200, 2, 1, 0),
                                   (9, 31, 33, 3, 64, 3, 1, 1)])
def test_bwn_first_layer_shapes(bnn, orc, shape):
    N, H, W, C, O, k, st, pad = shape
    rng = np.random.default_rng(sum(shape) + 1)
    x = rng.uniform(-1, 1, size=(N, H, W, C)).astype(np.float32)
    wb = wl.random_bits(rng, (O, k, k), C)
    thr = rng.normal(0, 1.0, size=O).astype(np.float32)
    bits, y = bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), C, st, pad, want_f32=True)
    ref = orc.bwn_conv_f32(x, wb, C, st, pad)
    tol = 1e-4 * np.maximum(np.abs(ref), np.sqrt((ref.astype(np.float64) ** 2).mean()))
    assert host(y).shape == ref.shape
    assert (np.abs(host(y) - ref) <= tol).all()
    # far tighter in fact: every product is exact, only the fp32 additions round
    assert np.abs(host(y) - ref).max() <= 2e-6 * max(1.0, np.abs(ref).max()) * np.sqrt(k * k * C)
    assert np.array_equal(words(bits), orc.pack_f32(host(y), thr))
    # bits only (no fp32 output) gives the same words
    assert np.array_equal(words(bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), C, st, pad)), words(bits))


# 11x11 stride-4 first layers of 3-channel images with at least 4096 rectangles of 4 x 8 output pixels: the kernel with
# wave-private patches (binarized weights: one weight plane); ragged rectangles, ragged and several 64-column tiles,
# images of a single rectangle, odd padding
@pytest.mark.parametrize("shape", [(300, 92, 76, 3, 36, 2), (230, 100, 90, 3, 100, 2), (4200, 11, 13, 3, 64, 2),
                                   (330, 83, 79, 3, 130, 5)])
def test_bwn_first_layer_11x11_wave_kernel(bnn, orc, shape):
    N, H, W, C, O, pad = shape
    k, st = 11, 4
    P, Q = (H + 2 * pad - k) // st + 1, (W + 2 * pad - k) // st + 1
    assert N * ((P + 3) // 4) * ((Q + 7) // 8) >= 4096
    rng = np.random.default_rng(sum(shape) + 3)
    x = rng.uniform(-1, 1, size=(N, H, W, C)).astype(np.float32)
    wb = wl.random_bits(rng, (O, k, k), C)
    thr = rng.normal(0, 3.0, size=O).astype(np.float32)
    bits, y = bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), C, st, pad, want_f32=True)
    ref = orc.bwn_conv_f32(x, wb, C, st, pad)
    err = np.abs(host(y) - ref)
    print("bwn 11x11", shape, "max error", float(err.max()), "of rms", float(np.sqrt((ref.astype(np.float64) ** 2).mean())), flush=True)
    assert host(y).shape == ref.shape
    assert (err <= 1e-4 * np.maximum(np.abs(ref), np.sqrt((ref.astype(np.float64) ** 2).mean()))).all()
    assert err.max() <= 2e-6 * max(1.0, np.abs(ref).max()) * np.sqrt(k * k * C)
    assert np.array_equal(words(bits), orc.pack_f32(host(y), thr))
    assert np.array_equal(words(bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), C, st, pad)), words(bits))
    # integer inputs: every product and every partial sum is exact, so the result equals the oracle's bit for bit
    xi = rng.integers(-2000, 2001, size=(N, H, W, C)).astype(np.float32)
    _, yi = bnn.bwn_conv_thr(to_dev(xi), to_dev(wb), to_dev(thr), C, st, pad, want_f32=True)
    assert np.array_equal(host(yi), orc.bwn_conv_f32(xi, wb, C, st, pad))


# Residual chains large enough for the kernel whose pixels are expanded in LDS, of widths that keep row-major sums: blocks with a 1x1 shortcut
# whose sum is not kept (bits only, its channels in the kernel's own order) and whose sum is kept, identity blocks that add packed bits or
# a 16-bit residual; both padding conventions; a chain whose sums pass 16 bits (eight blocks of 512).  `served`: the blocks whose
# second convolution runs there (None: asked for by the chain with int32 sums, which bconv_kernel_name does not describe).
@pytest.mark.parametrize("batch,hw,cin,blocks,pad_mode,served", [
    (64, 28, 64, ((64, 90, 1), (90, 86, 1), (86, 64, 2)), 0, (0, 1)),
    (64, 14, 64, ((64, 300, 1), (300, 300, 1), (300, 300, 1), (300, 290, 1), (290, 64, 2)), 0, (0, 1, 2, 3)),
    (64, 8, 64, ((64, 300, 1), (300, 290, 1), (290, 50, 2)), 0, (0, 1)),
    (64, 28, 90, ((90, 90, 1), (90, 90, 1), (90, 50, 1), (50, 100, 2), (100, 64, 2)), 1, (0, 1, 2, 3)),
    (64, 28, 33, ((33, 90, 1), (90, 90, 1), (90, 64, 2)), 1, (0, 1)),
    (32, 14, 64, ((64, 250, 1), (250, 230, 1), (230, 64, 2)), 1, (0, 1)),
    (64, 28, 48, ((48, 96, 1), (96, 96, 1), (96, 96, 1), (96, 512, 7)) + ((512, 512, 1),) * 7, 1, None),
    (64, 14, 48, ((48, 96, 1), (96, 512, 4)) + ((512, 512, 1),) * 7, 0, (0,))])
def test_block_chains_expanded_in_lds(bnn, orc, batch, hw, cin, blocks, pad_mode, served):
    rng = np.random.default_rng(batch + hw + cin)
    W, tau = wl.random_bits(rng, (cin, 3, 3), 3), np.zeros(cin, np.float32)
    net = bnn.Net()
    net.input_bwn_f32(to_dev(W), to_dev(tau), hw, hw, 3, 1, 1)
    params, size = [], hw
    for b, (ci, co, st) in enumerate(blocks):
        blk = {"cin": ci, "cout": co, "stride": st, "W1": wl.random_bits(rng, (co, 3, 3), ci), "W2": wl.random_bits(rng, (co, 3, 3), co),
               "thr1": rng.integers(-20, 21, size=co).astype(np.int32), "thr2": rng.integers(-20, 21, size=co).astype(np.int32)}
        if st != 1 or ci != co:
            blk["Wd"] = wl.random_bits(rng, (co, 1, 1), ci)
        params.append(blk)
        net.add_block(to_dev(blk["W1"]), to_dev(blk["thr1"]), to_dev(blk["W2"]), to_dev(blk["thr2"]),
                      to_dev(blk["Wd"]) if "Wd" in blk else None, ci, co, st, pad_mode)
        size = (size - 1) // st + 1
        keep = b + 1 < len(blocks) and blocks[b + 1][0] == blocks[b + 1][1] and blocks[b + 1][2] == 1
        kernel = bnn.bconv_kernel_name(batch, size, size, co, co, 3, 1, 1, pad_mode=pad_mode, shortcut="Wd" in blk,
                                       residual="Wd" not in blk, keep_sum=keep)
        assert served is None or kernel.startswith("mfma_fp4_conv_xlds") == (b in served), (b, kernel)
    w = rng.normal(0.0, 0.02, size=(7, blocks[-1][1])).astype(np.float32)
    net.add_head_f32(to_dev(w))
    x = rng.integers(-100, 101, size=(batch, hw, hw, 3)).astype(np.float32)
    net.forward(to_dev(x))
    first = words(net.layer_bits(0)).reshape(batch, hw, hw, -1)
    assert np.array_equal(first, orc.pack_f32(orc.bwn_conv_f32(x, W, 3, 1, 1), tau))
    tr = nets.resnet18_forward(x, {"blocks": params, "fc_w": w, "stem_w": np.zeros((cin, 1, 1, 3), np.float32), "stem_thr": tau},
                               stem_bits=first, tier=1, keep=True, pad_mode=pad_mode)
    for b in range(len(blocks)):
        got = words(net.layer_bits(b + 1)).reshape(tr["y%d" % b].shape)
        assert np.array_equal(got, tr["y%d" % b]), "block %d" % b


# 2x2 pooling behind a convolution, stored by the convolution itself on the direct kernels (even sizes) and by the pooling kernel
# (odd sizes, other windows): every tile of the direct kernel, channel counts that fill no word, several pooled layers in a row, a
# last 32-row block that is partly empty; the full and the pooled bits of every layer against the oracle.  `kernels`: what serves each
# convolution, "_pool2" where it stores the pooled bits
@pytest.mark.parametrize("batch,hw,chans,win,kernels", [
    (3, 12, (64, 128, 40), 2, ("wg64x64_pool2", "wg64x64_pool2")), (5, 8, (128, 256, 256), 2, ("wg64x64_pool2", "wg64x64_pool2")),
    (1, 4, (96, 33, 70), 2, ("wg64x64", "wg64x64_pool2")), (3, 9, (64, 65, 128), 2, ("wg64x64", "wg64x64")),
    (2, 12, (64, 64, 64), 3, ("wg64x64", "wg64x64")), (90, 32, (33, 256, 512), 2, ("wg256x128_pool2", "wg128x128_pool2")),
    (40, 64, (512, 60, 128), 2, ("wg512x64_pool2", "wg128x128_pool2"))])
def test_convolution_stores_pooled_bits(bnn, orc, batch, hw, chans, win, kernels):
    rng = np.random.default_rng(batch * 100 + hw)
    layers = [{"op": "bwn", "W": wl.random_bits(rng, (chans[0], 3, 3), 3), "thr": np.zeros(chans[0], np.float32), "C": 3, "stride": 1, "pad": 1}]
    size = hw
    for cin, cout, kernel in zip(chans, chans[1:], kernels):
        # (the choice is the one the chain makes; a window of 3 or another stride is never asked for)
        assert bnn.bconv_kernel_name(batch, size, size, cin, cout, 3, 1, 1, pool2=win == 2) == "mfma_fp4_conv_" + kernel
        layers.append({"op": "bconv", "W": wl.random_bits(rng, (cout, 3, 3), cin), "thr": rng.integers(-20, 21, size=cout).astype(np.int32),
                       "C": cin, "stride": 1, "pad": 1})
        layers.append({"op": "pool", "win": win, "stride": 2})
        size = (size - win) // 2 + 1
    print(batch, hw, chans, kernels, flush=True)
    net = bnn.Net.from_layers(layers, hw)
    x = rng.integers(-100, 101, size=(batch, hw, hw, 3)).astype(np.float32)     # exact in fp32: no bit depends on rounding
    xd = to_dev(x)
    net._out_kind, net._out_cols = torch.int32, 1
    net.forward(xd)
    outs = nets.cnn_forward(x, layers, tier=1, keep=True)
    for i, ref in enumerate(outs):
        got = words(net.layer_bits(i)).reshape(ref.shape)
        assert np.array_equal(got, ref), "layer %d (%s)" % (i, layers[i]["op"])
    assert outs[-1].shape[1] == size


# 3x3 and 5x5 first layers of 3-channel images (one LDS record per pixel): every fragment shape (8, 16, 32 columns), one and two
# 64-channel groups and ragged ones, stride 2, no and large padding, images smaller than a tile; integer inputs are exact in any
# order, so the sums equal the oracle's bit for bit; thresholds of +-infinity; a NaN pixel changes no output that does not cover it
@pytest.mark.parametrize("shape", [(3, 33, 65, 3, 64, 3, 1, 1), (2, 17, 7, 3, 33, 3, 1, 2), (2, 70, 13, 3, 130, 3, 1, 0),
                                   (5, 64, 61, 3, 65, 3, 2, 1), (1, 3, 3, 3, 1, 3, 2, 0), (40, 50, 24, 3, 100, 3, 2, 2),
                                   (2, 37, 40, 3, 64, 5, 1, 2), (3, 19, 30, 3, 128, 5, 1, 4), (2, 66, 35, 3, 40, 5, 2, 2),
                                   (7, 41, 14, 3, 192, 5, 2, 0), (70, 96, 96, 3, 32, 3, 1, 1)])
def test_bwn_first_layer_pixel_records(bnn, orc, shape):
    N, H, W, C, O, k, st, pad = shape
    rng = np.random.default_rng(sum(shape) + 7)
    wb = wl.random_bits(rng, (O, k, k), C)
    thr = rng.normal(0, 600.0, size=O).astype(np.float32)
    thr[0] = np.inf
    thr[O // 2] = -np.inf
    x = rng.integers(-2000, 2001, size=(N, H, W, C)).astype(np.float32)
    bits, y = bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), C, st, pad, want_f32=True)
    ref = orc.bwn_conv_f32(x, wb, C, st, pad)
    assert np.array_equal(host(y), ref)
    assert np.array_equal(words(bits), orc.pack_f32(ref, thr))
    only = words(bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), C, st, pad))
    assert np.array_equal(only, words(bits))
    h, w = H // 2, W // 3
    x[0, h, w, 2] = np.nan
    got = words(bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), C, st, pad))
    P, Q = only.shape[1:3]
    covers = np.zeros((N, P, Q), bool)
    for p in range(P):
        for q in range(Q):
            covers[0, p, q] = 0 <= h - (p * st - pad) < k and 0 <= w - (q * st - pad) < k
    assert np.array_equal(got[~covers], only[~covers]) and not got[covers].any()


# 11x11 stride-4 and 7x7 first layers of 3-channel images (signs in registers, a rectangle of 4 x 8 or 2 x 16 outputs per wave): 64, 96 and 128 channels
# per wave by the number of rectangles, ragged and several channel tiles, one image row or column of rectangles, one output, large and no
# padding, several rectangles per wave; integers are exact in any order; infinite thresholds
@pytest.mark.parametrize("shape", [(1, 11, 11, 1, 11, 0), (2, 50, 37, 33, 11, 2), (3, 227, 227, 128, 11, 2), (9, 223, 224, 96, 11, 2),
                                   (20, 224, 221, 128, 11, 2), (12, 224, 230, 129, 11, 5), (30, 225, 120, 300, 11, 0),
                                   (2, 9, 60, 64, 7, 3), (3, 224, 224, 65, 7, 3), (9, 224, 224, 96, 7, 3), (40, 224, 224, 128, 7, 3),
                                   (25, 201, 190, 190, 7, 6), (60, 33, 34, 40, 7, 0),
                                   (1, 7, 7, 1, 7, 0, 2), (3, 31, 36, 65, 7, 3, 2), (5, 112, 109, 96, 7, 3, 2), (9, 130, 127, 128, 7, 3, 2),
                                   (14, 60, 221, 200, 7, 5, 2)])
def test_bwn_first_layer_strided_windows(bnn, orc, shape):
    N, H, W, O, k, pad, st = shape if len(shape) == 7 else shape + (4,)
    rng = np.random.default_rng(sum(shape))
    wb = wl.random_bits(rng, (O, k, k), 3)
    thr = rng.integers(-4000, 4001, size=O).astype(np.float32)
    thr[0], thr[O // 2] = np.inf, -np.inf
    x = rng.integers(-500, 501, size=(N, H, W, 3)).astype(np.float32)
    print(shape, flush=True)
    ref = orc.bwn_conv_f32(x, wb, 3, st, pad)
    bits, y = bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), 3, st, pad, want_f32=True)
    assert np.array_equal(host(y), ref) and np.array_equal(words(bits), orc.pack_f32(ref, thr))
    only = words(bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), 3, st, pad))
    assert np.array_equal(only, words(bits))
    # a pixel that is not finite (the lower terms of an infinity are NaN) clears the bits of the outputs that cover it and changes no other
    h, w = H // 2, W // 2
    P, Q = only.shape[1:3]
    covers = np.zeros((N, P, Q), bool)
    for p in range(P):
        for q in range(Q):
            covers[0, p, q] = 0 <= h - (p * st - pad) < k and 0 <= w - (q * st - pad) < k
    for bad in (np.inf, np.nan):
        x[0, h, w, 0] = bad
        got = words(bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), 3, st, pad))
        assert np.array_equal(got[~covers], only[~covers]) and not got[covers].any(), bad


# first layers with real weights, stride 2, on the kernel with wave-private patches: ragged rectangles, one output, no, odd and large
# padding, ragged and several 64-channel tiles, several rectangles per wave; with integers below 2^12 every product is exact, in three terms
# or in the largest two of each, and so is every sum; a pixel that is not finite touches no output that does not cover it
@pytest.mark.parametrize("products", [9, 6])
@pytest.mark.parametrize("shape", [(1, 3, 3, 1, 3, 0), (2, 37, 64, 65, 3, 1), (60, 130, 65, 40, 3, 1), (1, 5, 5, 64, 5, 0), (3, 40, 33, 130, 5, 2),
                                   (30, 90, 131, 64, 5, 3), (1, 7, 7, 3, 7, 0), (2, 61, 70, 128, 7, 3), (20, 129, 112, 33, 7, 5)])
def test_stem_split_stride_2(bnn, orc, shape, products):
    N, H, W, O, k, pad = shape
    rng = np.random.default_rng(sum(shape) + products)
    x = rng.integers(-900, 901, size=(N, H, W, 3)).astype(np.float32)
    w = rng.integers(-30, 31, size=(O, k, k, 3)).astype(np.float32)
    thr = rng.integers(-50000, 50001, size=O).astype(np.float32)
    print(shape, products, flush=True)
    ref = orc.conv_f32(x, w, 2, pad)
    bits, y = bnn.conv_f32_split_thr(to_dev(x), to_dev(w), to_dev(thr), 2, pad, want_f32=True, products=products)
    assert np.array_equal(host(y), ref) and np.array_equal(words(bits), orc.pack_f32(ref, thr))
    only = words(bnn.conv_f32_split_thr(to_dev(x), to_dev(w), to_dev(thr), 2, pad, products=products))
    assert np.array_equal(only, words(bits))
    h, q0 = H // 2, W // 2
    P, Q = only.shape[1:3]
    covers = np.zeros((N, P, Q), bool)
    for p in range(P):
        for q in range(Q):
            covers[0, p, q] = 0 <= h - (p * 2 - pad) < k and 0 <= q0 - (q * 2 - pad) < k
    x[0, h, q0, 0] = np.nan
    got = words(bnn.conv_f32_split_thr(to_dev(x), to_dev(w), to_dev(thr), 2, pad, products=products))
    assert np.array_equal(got[~covers], only[~covers]) and not got[covers].any()


# the 7x7 stride-4 stem likewise: a filter row's last run reads one pixel beyond the window, whose zero weights a pixel that is not finite would turn into NaN
@pytest.mark.parametrize("products", [9, 6])
@pytest.mark.parametrize("shape", [(1, 7, 11, 1, 0), (2, 33, 40, 65, 3), (40, 60, 61, 64, 3)])
def test_stem_split_not_finite(bnn, orc, shape, products):
    N, H, W, O, pad = shape
    rng = np.random.default_rng(sum(shape) + products)
    x = rng.integers(-900, 901, size=(N, H, W, 3)).astype(np.float32)
    w = rng.integers(-30, 31, size=(O, 7, 7, 3)).astype(np.float32)
    thr = rng.integers(-50000, 50001, size=O).astype(np.float32)
    only = words(bnn.conv_f32_split_thr(to_dev(x), to_dev(w), to_dev(thr), 4, pad, products=products))
    assert np.array_equal(only, orc.pack_f32(orc.conv_f32(x, w, 4, pad), thr))
    P, Q = only.shape[1:3]
    h, q0 = H // 2, Q // 2
    for col in (q0 * 4 - pad + 6, q0 * 4 - pad + 7):        # the last pixel of a window's rows, and the one behind it
        if col >= W:
            continue
        covers = np.zeros((N, P, Q), bool)
        for p in range(P):
            for q in range(Q):
                covers[N - 1, p, q] = 0 <= h - (p * 4 - pad) < 7 and 0 <= col - (q * 4 - pad) < 7
        for bad in (np.inf, np.nan):
            xb = x.copy()
            xb[N - 1, h, col, 1] = bad
            got = words(bnn.conv_f32_split_thr(to_dev(xb), to_dev(w), to_dev(thr), 4, pad, products=products))
            assert np.array_equal(got[~covers], only[~covers]) and not got[covers].any(), (col, bad)


# Narrow and flat images, where a rectangle of outputs is mostly empty: few of them (one kernel), and so many that the kernel which packs consecutive outputs, or
# rectangles of another shape, serve the call.  Integers are exact in any order; a few images are compared, the others repeat them.
@pytest.mark.parametrize("weights,k,st,H,W", [("bits", 7, 4, 22, 2), ("bits", 7, 4, 3, 33), ("bits", 7, 2, 31, 2), ("bits", 7, 2, 93, 15), ("bits", 7, 2, 12, 33), ("bits", 11, 4, 9, 12),
                                              ("f32", 3, 2, 26, 2), ("f32", 5, 2, 37, 35), ("f32", 7, 2, 19, 4), ("f32", 7, 2, 2, 40)])
@pytest.mark.parametrize("O", [64, 70])
@pytest.mark.parametrize("images", [3, 4099])
def test_first_layers_of_narrow_images(bnn, orc, weights, k, st, H, W, O, images):
    rng = np.random.default_rng(k + st + H + W + O)
    pad = 2 if k == 11 else k // 2
    x = rng.integers(-500, 501, size=(5, H, W, 3)).astype(np.float32)
    many = to_dev(x[np.arange(images) % 5])
    thr = rng.integers(-4000, 4001, size=O).astype(np.float32)
    print(weights, k, st, H, W, O, images, flush=True)
    if weights == "bits":
        w = wl.random_bits(rng, (O, k, k), 3)
        ref = orc.bwn_conv_f32(x, w, 3, st, pad)
        layer = lambda **kw: bnn.bwn_conv_thr(many, to_dev(w), to_dev(thr), 3, st, pad, **kw)
    else:
        w = rng.integers(-30, 31, size=(O, k, k, 3)).astype(np.float32)
        ref = orc.conv_f32(x, w, st, pad)
        layer = lambda **kw: bnn.conv_f32_split_thr(many, to_dev(w), to_dev(thr), st, pad, **kw)
    packed = orc.pack_f32(ref, thr)[np.arange(images) % 5]
    assert np.array_equal(words(layer()), packed)
    bits, y = layer(want_f32=True)
    assert np.array_equal(words(bits), packed)
    assert torch.equal(y, to_dev(ref)[torch.arange(images, device="cuda") % 5])


# weights and thresholds of 64 channels at a time go through LDS: groups one channel short, whole and one over, for workgroups of one
# and of two groups
@pytest.mark.parametrize("k,st", [(3, 1), (3, 2), (5, 1), (5, 2)])
@pytest.mark.parametrize("O", [2, 63, 64, 127, 129, 191])
def test_bwn_first_layer_channel_groups(bnn, orc, O, k, st):
    rng = np.random.default_rng(O * 10 + k + st)
    wb = wl.random_bits(rng, (O, k, k), 3)
    thr = rng.integers(-900, 901, size=O).astype(np.float32)
    x = rng.integers(-300, 301, size=(2, 20, 11, 3)).astype(np.float32)
    ref = orc.bwn_conv_f32(x, wb, 3, st, 1)
    assert np.array_equal(words(bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), 3, st, 1)), orc.pack_f32(ref, thr))
    bits, y = bnn.bwn_conv_thr(to_dev(x), to_dev(wb), to_dev(thr), 3, st, 1, want_f32=True)
    assert np.array_equal(host(y), ref) and np.array_equal(words(bits), orc.pack_f32(ref, thr))


def test_bwn_exact_cases(bnn, orc):
    # (a) integer inputs: the three-way bf16 split is exact and sums below 2^24 never round, so the fp32
    # result equals the oracle's bit for bit; (b) isolated values with all 24 significand bits set (at most
    # one non-zero term per output): checks that the split drops no bit
    rng = np.random.default_rng(5)
    wb = wl.random_bits(rng, (40, 5, 5), 3)
    zero = to_dev(np.zeros(40, np.float32))
    x = rng.integers(-30000, 30001, size=(2, 14, 13, 3)).astype(np.float32)
    _, y = bnn.bwn_conv_thr(to_dev(x), to_dev(wb), zero, 3, 2, 2, want_f32=True)
    assert np.array_equal(host(y), orc.bwn_conv_f32(x, wb, 3, 2, 2))
    x = np.zeros((1, 30, 30, 3), np.float32)
    for (h, w, c, v) in ((2, 3, 0, 16777215.0 / 4096), (12, 20, 1, -11184811.0 / 65536), (25, 6, 2, 13421773.0 * 8),
                         (20, 27, 0, 8388609.0 / 2 ** 30)):
        x[0, h, w, c] = v
    _, y = bnn.bwn_conv_thr(to_dev(x), to_dev(wb), zero, 3, 1, 2, want_f32=True)
    ref = orc.bwn_conv_f32(x, wb, 3, 1, 2)
    assert np.abs(ref).max() > 1e7 and np.array_equal(host(y), ref)


# ------------------------------------------------------------------ whole-network persistent kernel (FC chains)
@pytest.mark.parametrize("batch", [8, 37, 1024, 3000])
def test_mlp_persistent(bnn, orc, batch):
    params = wl.mlp_params()
    imgs = wl.mlp_images(batch)
    net = bnn.Net()
    net.input_u8(784, params["in_thr"])
    for l in range(4):
        net.add_fc(to_dev(params["W"][l]), to_dev(params["thr"][l]) if l < 3 else None, params["K"][l])
    ref, hidden = nets.mlp_forward(imgs, params, keep=True)
    x = to_dev(imgs)
    for rep in range(3):                                   # the barrier counter is re-armed on every call
        got = host(net.forward_persistent(x))
        assert not net.persistent_status(), "a barrier gave up in call %d" % rep
        assert np.array_equal(got, ref), "call %d" % rep
    for l in range(3):
        assert np.array_equal(words(net.layer_bits(l + 1)), hidden[l])
    assert np.array_equal(host(net.forward(x)), ref)       # and the per-layer path still agrees


@pytest.mark.parametrize("blocks,hw,batch,pad_mode", [
    (((64, 64, 1), (64, 128, 2), (128, 128, 1), (128, 256, 2)), 32, 3, 0),
    (((64, 64, 1), (64, 64, 1), (64, 128, 2), (128, 256, 2), (256, 512, 2), (512, 512, 1)), 64, 2, 1),
    (((128, 128, 1), (128, 128, 1)), 40, 9, 0)])
def test_resnet_persistent(bnn, orc, blocks, hw, batch, pad_mode):
    # residual chains as one persistent kernel (stem and head stay ordinary launches): every block's bits and the
    # logits must equal the per-layer forward's exactly -- the same integer arithmetic, another launch structure --
    # and the per-layer forward is checked against the oracle; repeated calls re-use the uploaded layer table
    p = wl.resnet18_params(blocks=blocks, classes=11, config=98)
    x = wl.resnet18_input(batch, hw=hw, config=98)
    check_resnet(bnn, orc, p, x, hw, 0, tier=1, pad_mode=pad_mode)
    xd = to_dev(x)
    net = build_resnet(bnn, p, hw, pad_mode)
    ref = host(net.forward(xd))
    ref_bits = [words(net.layer_bits(b)) for b in range(len(blocks) + 1)]
    for rep, cap in enumerate((0, 0, 16, 1000)):
        got = host(net.forward_persistent(xd, grid_cap=cap))
        assert not net.persistent_status(), "a barrier gave up in call %d" % rep
        assert np.array_equal(got, ref), "logits, call %d" % rep
        for b in range(len(blocks) + 1):
            assert np.array_equal(words(net.layer_bits(b)), ref_bits[b]), "layer %d, call %d" % (b, rep)
    # another batch through the same net: the table is rebuilt
    x2 = to_dev(wl.resnet18_input(batch + 1, hw=hw, config=99))
    assert np.array_equal(host(net.forward_persistent(x2)), host(net.forward(x2)))


def test_persistent_refuses_what_it_cannot_run(bnn):
    # 96 input channels have no unrolled 3x3 form in the persistent kernel
    p = wl.resnet18_params(blocks=((64, 96, 2), (96, 96, 1)), classes=5, config=98)
    net = build_resnet(bnn, p, 32)
    x = to_dev(wl.resnet18_input(2, hw=32, config=98))
    with pytest.raises(bnn.BnnError) as ei:
        net.forward_persistent(x)
    assert ei.value.status == -3
    assert host(net.forward(x)).shape == (2, 5)            # the per-layer path takes it


def test_persistent_timeout_is_reported(bnn, orc):
    # the time-out path, forced from the host: with a poll limit of zero the first workgroup that finds a barrier
    # incomplete raises the abort flag, every workgroup leaves the kernel normally, and the status call says so;
    # the next ordinary call re-arms the barrier and is exact again
    params = wl.mlp_params()
    imgs = wl.mlp_images(2048)
    net = build_mlp(bnn, params)
    x = to_dev(imgs)
    net.forward_persistent(x, give_up_at_once=True)
    assert net.persistent_status()
    got = host(net.forward_persistent(x))
    assert not net.persistent_status()
    assert np.array_equal(got, nets.mlp_forward(imgs, params))


def test_fc_after_unaligned_spatial_layer_is_refused(bnn):
    # an FC whose operand rows (H*W pixels of ceil(C/32) words) are not a multiple of 128 bits: refused when the
    # workspace is sized, not part-way through the forward
    rng = np.random.default_rng(8)
    net = bnn.Net()
    net.input_conv_f32(to_dev(rng.normal(size=(64, 3, 3, 3)).astype(np.float32)), to_dev(np.zeros(64, np.float32)), 3, 3, 1, 0)
    net.add_fc(to_dev(wl.random_bits(rng, 10, 64, 4)), None, 64)         # 1x1x64: rows of 2 words
    with pytest.raises(bnn.BnnError) as e:
        net.workspace_bytes(4)
    assert e.value.status == -3
    with pytest.raises(ValueError):
        bnn.Net().add_fc(to_dev(wl.random_bits(rng, 10, 64, 2)), None, 64)


def test_persistent_bits_input_and_limits(bnn, orc):
    rng = np.random.default_rng(3)
    dims = (200, 96, 70, 5)
    W = [wl.random_bits(rng, dims[i + 1], dims[i], wl.round_up(wl.nwords(dims[i]), 4)) for i in range(3)]
    thr = [wl.random_thresholds(rng, dims[i + 1], -8, 8) for i in range(2)]
    x = wl.random_bits(rng, 50, dims[0], wl.round_up(wl.nwords(dims[0]), 4))
    net = bnn.Net()
    net.input_bits(dims[0])
    for i in range(3):
        net.add_fc(to_dev(W[i]), to_dev(thr[i]) if i < 2 else None, dims[i])
    h = x
    for i in range(2):
        h = orc.threshold_pack(orc.bmm(h, W[i], dims[i]), thr[i], ldb_w=wl.round_up(wl.nwords(dims[i + 1]), 4))
    ref = orc.bmm(h, W[2], dims[2])
    assert np.array_equal(host(net.forward_persistent(to_dev(x))), ref)
    # a convolutional network with pooling layers: every run of layers between the pools is one persistent launch,
    # the result is that of the per-layer forward (Cifar-VGG and Cifar-ResNet-14: convolutions, blocks, then FC layers)
    for name in ("cifar_vgg", "cifar_resnet14"):
        spec = wl.cnn_layers(name)
        cnn = bnn.Net.from_layers(spec["layers"], spec["in_hw"])
        xi = to_dev(wl.cnn_input(name, 3))
        want = host(cnn.forward(xi))
        for rep in range(2):
            assert np.array_equal(host(cnn.forward_persistent(xi)), want), (name, rep)
            assert not cnn.persistent_status()


@pytest.mark.parametrize("shape", [(2, 21, 19, 3, 5, 7, 4, 3), (1, 9, 9, 1, 1, 3, 1, 1), (3, 16, 12, 4, 70, 5, 2, 2),
                                   (2, 32, 32, 3, 64, 7, 4, 3), (1, 8, 8, 2, 33, 1, 1, 0), (5, 64, 64, 3, 64, 7, 4, 3),
                                   (2, 33, 31, 3, 130, 3, 1, 1),
                                   # the kernel with wave-private patches in LDS (pixel step a multiple of 8 bytes in bf16):
                                   # ragged rectangles, pad 0 and pad > 0, several channel tiles, one-pixel outputs, a 4-channel
                                   # stride-1 layer, more images than waves
                                   (3, 37, 41, 3, 64, 7, 4, 3), (2, 30, 30, 3, 100, 7, 4, 0), (1, 7, 7, 3, 64, 7, 4, 0),
                                   (2, 19, 23, 4, 40, 3, 1, 1), (1, 5, 6, 8, 33, 3, 1, 1), (300, 9, 9, 3, 64, 5, 4, 2),
                                   (2, 48, 52, 6, 64, 3, 2, 1), (1, 224, 224, 3, 64, 7, 4, 3)])
@pytest.mark.parametrize("products", [9, 6])
def test_conv_f32_split_shapes(bnn, orc, shape, products):
    # the fp32 first layer on the bf16 matrix cores (three-way exact split of inputs and weights; all nine term
    # products, or the six that reach fp32 precision)
    N, H, W, C, O, k, st, pad = shape
    rng = np.random.default_rng(sum(shape) + 3)
    x = rng.uniform(-1, 1, size=(N, H, W, C)).astype(np.float32)
    w = rng.normal(0, 0.05, size=(O, k, k, C)).astype(np.float32)
    thr = rng.normal(0, 0.05, size=O).astype(np.float32)
    bits, y = bnn.conv_f32_split_thr(to_dev(x), to_dev(w), to_dev(thr), st, pad, want_f32=True, products=products)
    ref = orc.conv_f32(x, w, st, pad)
    tol = 1e-4 * np.maximum(np.abs(ref), np.sqrt((ref.astype(np.float64) ** 2).mean()))
    assert host(y).shape == ref.shape
    assert (np.abs(host(y) - ref) <= tol).all()
    # far tighter in fact: the products are exact (or, with six, as good as rounded to fp32), the fp32 additions round
    assert np.abs(host(y) - ref).max() <= 2e-6 * np.abs(w).max() * np.sqrt(k * k * C) * 4
    assert np.array_equal(words(bits), orc.pack_f32(host(y), thr))
    assert np.array_equal(words(bnn.conv_f32_split_thr(to_dev(x), to_dev(w), to_dev(thr), st, pad, products=products)),
                          words(bits))


def test_conv_f32_split_exact_products(bnn, orc):
    # integer inputs and weights whose products need all 24 + 24 significand bits pairwise: with every term product
    # formed, sums that stay below 2^24 are exact, so the result equals the oracle's bit for bit
    rng = np.random.default_rng(6)
    x = rng.integers(-2000, 2001, size=(2, 12, 13, 3)).astype(np.float32)
    w = rng.integers(-50, 51, size=(40, 5, 5, 3)).astype(np.float32)
    zero = to_dev(np.zeros(40, np.float32))
    _, y = bnn.conv_f32_split_thr(to_dev(x), to_dev(w), zero, 2, 2, want_f32=True)
    ref = orc.conv_f32(x, w, 2, 2)
    assert np.abs(ref).max() < 2 ** 24 and np.array_equal(host(y), ref)
    # one isolated full-precision product: (2^24 - 1) / 2^12 times (2^24 - 3) / 2^20 rounded once, as fp32 does
    x = np.zeros((1, 9, 9, 3), np.float32)
    w = np.zeros((3, 3, 3, 3), np.float32)
    x[0, 4, 4, 1] = 16777215.0 / 4096
    w[2, 1, 1, 1] = 16777213.0 / 1048576
    _, y = bnn.conv_f32_split_thr(to_dev(x), to_dev(w), to_dev(np.zeros(3, np.float32)), 1, 1, want_f32=True)
    assert host(y)[0, 4, 4, 2] == np.float32(np.float64(x[0, 4, 4, 1]) * np.float64(w[2, 1, 1, 1]))
    assert np.array_equal(host(y), orc.conv_f32(x, w, 1, 1))


# Residual chains whose second convolutions run in bands (3x3, 128 / 256 / 512 channels): a first residual taken from bits, blocked 16-bit sums in
# and out, a 1x1 shortcut with and without its sum kept and with a source that fills no word pair (96 channels: what it multiplies beyond its width
# is taken back), K split over two groups of waves; `banded`: the blocks whose second convolution is one.
@pytest.mark.parametrize("pad_mode", [0, 1])
@pytest.mark.parametrize("batch,hw,cin,blocks,banded", [
    (85, 14, 256, ((256, 256, 1), (256, 256, 1), (256, 256, 1)), (0, 1, 2)),
    (117, 14, 96, ((96, 256, 1), (256, 256, 1), (256, 512, 2)), (0, 1, 2)),
    (100, 14, 256, ((256, 512, 2), (512, 512, 1), (512, 512, 1)), (0, 1, 2)),
    (126, 7, 96, ((96, 512, 1), (512, 512, 1)), (0, 1)), (126, 7, 512, ((512, 512, 1), (512, 128, 1)), (0,)),
    (191, 15, 96, ((96, 128, 1), (128, 128, 1), (128, 128, 1)), (0, 1, 2)), (150, 15, 128, ((128, 128, 1), (128, 128, 1)), (0, 1))])
def test_block_chains_in_bands(bnn, orc, batch, hw, cin, blocks, banded, pad_mode):
    size = hw
    for b, (ci, co, st) in enumerate(blocks):
        size = (size - 1) // st + 1
        keep = b + 1 < len(blocks) and blocks[b + 1][0] == blocks[b + 1][1] and blocks[b + 1][2] == 1
        shortcut = st != 1 or ci != co
        kernel = bnn.bconv_kernel_name(batch, size, size, co, co, 3, 1, 1, pad_mode=pad_mode, shortcut=shortcut, residual=not shortcut, keep_sum=keep)
        assert (kernel == "mfma_fp4_conv3x3_band_wg64") == (b in banded), (b, kernel)
    test_block_chains_expanded_in_lds(bnn, orc, batch, hw, cin, blocks, pad_mode, None)


# Small 3x3 layers with a wave per tap: 2x2-pooled bits stored beside the full ones, and residual chains (first residual from bits, blocked 16-bit
# sums in and out, a 1x1 shortcut on a tenth wave whose source fills no word pair).
@pytest.mark.parametrize("batch,hw,chans", [(8, 16, (128, 256, 512)), (2, 20, (256, 500, 60)), (11, 8, (512, 512, 70))])
def test_wave_per_tap_stores_pooled_bits(bnn, orc, batch, hw, chans):
    kernels = []
    for i, (cin, cout) in enumerate(zip(chans, chans[1:])):
        size = hw >> i
        kernels.append(bnn.bconv_kernel_name(batch, size, size, cin, cout, 3, 1, 1, pool2=True)[len("mfma_fp4_conv_"):])
    assert "taps_wg32x32_pool2" in kernels
    test_convolution_stores_pooled_bits(bnn, orc, batch, hw, chans, 2, kernels)


@pytest.mark.parametrize("pad_mode", [0, 1])
@pytest.mark.parametrize("batch,hw,cin,blocks", [
    (3, 14, 96, ((96, 128, 1), (128, 128, 1), (128, 256, 2), (256, 256, 1))), (2, 9, 256, ((256, 256, 1), (256, 256, 1), (256, 512, 2), (512, 512, 1)))])
def test_block_chains_wave_per_tap(bnn, orc, batch, hw, cin, blocks, pad_mode):
    size = hw
    for ci, co, st in blocks:
        size = (size - 1) // st + 1
        shortcut = st != 1 or ci != co
        assert bnn.bconv_kernel_name(batch, size, size, co, co, 3, 1, 1, pad_mode=pad_mode, shortcut=shortcut, residual=not shortcut,
                                     keep_sum=shortcut) == "mfma_fp4_conv_taps_wg32x32"
    test_block_chains_expanded_in_lds(bnn, orc, batch, hw, cin, blocks, pad_mode, None)


# Blocks of a chain may pad in different ways; the 16-bit sums between them are blocked in the order of the kernel that writes them, so that kernel
# must not depend on the padding: in bands (K split and not), patches and a wave per tap
@pytest.mark.parametrize("batch,hw,C,kernel", [(126, 7, 512, "3x3_band_wg64"), (85, 14, 256, "3x3_band_wg64"), (191, 15, 128, "3x3_band_wg64"),
                                               (200, 15, 64, "3x3_patch_wave64x64"), (3, 9, 256, "_taps_wg32x32")])
def test_block_chains_of_mixed_padding(bnn, orc, batch, hw, C, kernel):
    rng = np.random.default_rng(batch + hw + C)
    net, modes, blocks = bnn.Net(), (0, 1, 0, 1), []
    net.input_bwn_f32(to_dev(wl.random_bits(rng, (C, 3, 3), 3)), to_dev(np.zeros(C, np.float32)), hw, hw, 3, 1, 1)
    for pad_mode in modes:
        assert bnn.bconv_kernel_name(batch, hw, hw, C, C, 3, 1, 1, pad_mode=pad_mode, residual=True, keep_sum=True) == "mfma_fp4_conv" + kernel
        blk = [wl.random_bits(rng, (C, 3, 3), C), rng.integers(-20, 21, size=C).astype(np.int32), wl.random_bits(rng, (C, 3, 3), C),
               rng.integers(-20, 21, size=C).astype(np.int32)]
        net.add_block(*map(to_dev, blk), None, C, C, 1, pad_mode)
        blocks.append(blk)
    net.add_head_f32(to_dev(rng.normal(0.0, 0.02, size=(7, C)).astype(np.float32)))
    net.forward(to_dev(rng.integers(-100, 101, size=(batch, hw, hw, 3)).astype(np.float32)))
    x = words(net.layer_bits(0)).reshape(batch, hw, hw, -1)
    total = orc.unpack_pm1(x.reshape(-1, x.shape[-1]), C).astype(np.int32).reshape(batch, hw, hw, C)
    for b, (pad_mode, (w1, t1, w2, t2)) in enumerate(zip(modes, blocks)):
        h = orc.threshold_pack(orc.bconv(x, w1, C, 1, 1, pad_mode, tier=1), t1)
        total = total + orc.bconv(h, w2, C, 1, 1, pad_mode, tier=1)
        x = orc.threshold_pack(total, t2)
        assert np.array_equal(words(net.layer_bits(b + 1)).reshape(x.shape), x), "block %d" % b

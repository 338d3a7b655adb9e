"""CPU-only checks of the boundary: the library loads and exports every symbol include/bnn.h
declares; argument validation that needs no GPU returns the documented codes."""
import ctypes
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "bnn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(bnn_[a-z0-9_]+)\s*\(", text)))


def test_exports_match_header():
    import paper_2006_16578_amd as b
    lib = b.load()
    syms = declared_symbols()
    assert len(syms) >= 25
    for s in syms:
        assert hasattr(lib, s), s
    assert sorted(b.EXPORTS) == syms


def test_status_strings_and_null_checks():
    import paper_2006_16578_amd as b
    lib = b.load()
    assert lib.bnn_version() >= 100
    assert lib.bnn_status_string(0) == b"ok"
    for code in (-1, -2, -3, -4, -5):
        assert lib.bnn_status_string(code) not in (b"ok", b"unknown status")
    # validation happens before any device call
    assert lib.bnn_bmm(None, None, None, 1, 1, 1, 4, 4, 1, None) == -1
    assert lib.bnn_bconv(None, None, None, 1, 1, 1, 1, 1, 1, 1, 0, 0, None) == -1
    net = ctypes.c_void_p()
    assert lib.bnn_net_create(ctypes.byref(net)) == 0
    assert lib.bnn_net_add_fc(net, None, None, 8, 8) == -1
    assert lib.bnn_net_input_u8(net, 784, 127) == 0
    assert lib.bnn_net_input_u8(net, 784, 127) == -1          # only one input layer
    n = ctypes.c_size_t()
    assert lib.bnn_net_workspace_bytes(net, 8, ctypes.byref(n)) == 0 and n.value > 0
    assert lib.bnn_net_destroy(net) == 0


@pytest.mark.parametrize("there", ["missing", "of another torch"])
def test_without_the_native_module(monkeypatch, there):
    # the module only shortens calls: without it, or with one built for another torch, they go by ctypes as ever, and that is said once
    import types
    import warnings

    import torch
    from paper_2006_16578_amd import binding
    name = "paper_2006_16578_amd._native"
    if there == "missing":
        monkeypatch.setitem(sys.modules, name, None)
    else:
        monkeypatch.setitem(sys.modules, name, types.SimpleNamespace(built_for="torch 1.0, Python 3.0", init=lambda *a: pytest.fail("taken")))
    monkeypatch.setattr(binding, "_native", None)
    x = torch.zeros((4, 4), dtype=torch.int32)
    with pytest.warns(RuntimeWarning, match="short calls"), pytest.raises(TypeError, match="device tensor"):
        binding.bmm(x, x, 128)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        with pytest.raises(TypeError, match="device tensor"):
            binding.maxpool_or(x, 32, 2, 2)


def test_the_native_module_is_of_this_torch():
    from paper_2006_16578_amd import binding
    assert binding._native_module().built_for == binding._native_stamp()


def test_kernel_choice_is_host_logic():
    # which kernel variant a shape gets is decided on the host: no device needed to ask
    import paper_2006_16578_amd as b
    assert b.bmm_kernel_name(16384, 16384, 16384) == "mfma_fp4_bmm_xlds_wg256x256"
    assert b.bmm_kernel_name(4096, 4096, 4096) == "mfma_fp4_bmm_xlds_wg256x256"        # 256 tiles: one per compute unit
    assert b.bmm_kernel_name(2048, 2048, 2048) == "mfma_fp4_bmm_lds_wg128x128"         # too few 256 x 256 tiles
    assert b.bmm_kernel_name(8, 4096, 4096) == "mfma_fp4_bmm_skinny_m32"               # at most 128 rows: K split over waves
    assert b.bmm_kernel_name(128, 4096, 4096) == "mfma_fp4_bmm_skinny_m128"
    assert b.bmm_kernel_name(129, 4096, 4096) == "mfma_fp4_bmm_wg64x64"
    assert b.bmm_kernel_name(4096, 4096, 4096, b.PATH_VALU) == "valu_xor_popc_bmm"
    # a short-K matrix product with int32 output moves more bytes than it multiplies: small tiles
    assert b.bmm_kernel_name(8192, 8192, 256, int32_out=True) == "mfma_fp4_bmm_wg64x64"
    assert b.bmm_kernel_name(8192, 8192, 256) != "mfma_fp4_bmm_wg64x64"
    # the graded convolution shape: 3x3, stride 1, few channels -> filters resident in LDS, wave-private patches
    assert b.bconv_kernel_name(128, 56, 56, 128, 128, 3, 1, 1) == "mfma_fp4_conv3x3_patch_wave64x128"
    assert b.bconv_kernel_name(128, 56, 56, 128, 128, 3, 1, 1, int32_out=True) == "mfma_fp4_conv3x3_patch_wave64x128"
    assert b.bconv_kernel_name(128, 56, 56, 64, 64, 3, 1, 1) == "mfma_fp4_conv3x3_patch_wave64x64"
    # stride 2, 64 -> 128 channels, bits out: the same kernel with the lane bases twice as far apart
    assert b.bconv_kernel_name(128, 56, 56, 64, 128, 3, 2, 1) == "mfma_fp4_conv3x3s2_patch_wave64x128"
    # the same layers at a small batch, with int32 sums at stride 2, or with more channels: the direct kernel's tiles
    assert b.bconv_kernel_name(2, 56, 56, 128, 128, 3, 1, 1) == "mfma_fp4_conv_wg64x64"
    assert b.bconv_kernel_name(128, 56, 56, 64, 128, 3, 2, 1, int32_out=True) == "mfma_fp4_conv_wg256x128"
    assert not b.bconv_kernel_name(16, 56, 56, 64, 128, 3, 2, 1).startswith("mfma_fp4_conv3x3")     # too few tiles for it
    assert b.bconv_kernel_name(128, 28, 28, 256, 256, 3, 1, 1) == "mfma_fp4_conv_wg256x128"
    # long K goes through LDS
    assert b.bconv_kernel_name(16, 64, 64, 2048, 2048, 3, 1, 1) == "mfma_fp4_conv_lds_wg256x128"
    assert b.bmm_kernel_name(0, 1, 1) == "invalid" and b.bconv_kernel_name(1, 2, 2, 32, 1, 5, 1, 0) == "invalid"


def test_kernel_names_tell_the_program():
    # a wave tile may be that of several kernels: with program=True the name says which one a product gets
    import paper_2006_16578_amd as b
    def name(*shape, **kw):
        plain, full = b.bmm_kernel_name(*shape, **kw), b.bmm_kernel_name(*shape, program=True, **kw)
        assert full.startswith(plain) or "skinny" in plain
        return full[len("mfma_fp4_bmm_"):]
    assert name(16384, 16384, 16384) == "xlds_wg256x256_01" and name(4097, 3001, 4100) == "lds_wg256x128_01"
    assert name(4000, 4000, 800) == "lds_wg256x128_signs" and name(8192, 8192, 256, int32_out=True) == "wg64x64_signs"
    assert name(4673, 40, 6064) == "wg64x64_01_ksplit" and name(160, 505, 8310, int32_out=True) == "wg32x32_01_ksplit"
    assert name(2738, 1117, 520) == "lds_wg128x128_01_w8" and name(1817, 3303, 2646) == "lds_wg128x128_01_w4"
    # few rows: 16 columns to a workgroup, 32 beyond 4096 columns from 17 rows on
    assert name(8, 100, 4096) == "skinny_m16_c16" and name(8, 4096, 4096) == "skinny_m16_c16" and name(16, 9000, 100) == "skinny_m16_c16"
    assert name(17, 4096, 100) == "skinny_m32_c16" and name(32, 4097, 100) == "skinny_m32_c32"
    assert name(40, 4096, 700) == "skinny_m64_c16" and name(40, 4097, 700) == "skinny_m64_c32" and name(128, 4097, 700, int32_out=True) == "skinny_m128_c32"
    assert b.bmm_kernel_name(0, 1, 1, program=True) == "invalid"


def test_net_workspace_plan():
    # the workspace of a chain grows with the batch and covers residual slots, the first layer's expanded weights
    # and the pooled sums of a head
    import paper_2006_16578_amd as b
    lib = b.load()

    def ws(build, batch):
        net = ctypes.c_void_p()
        assert lib.bnn_net_create(ctypes.byref(net)) == 0
        build(net)
        n = ctypes.c_size_t()
        assert lib.bnn_net_workspace_bytes(net, batch, ctypes.byref(n)) == 0
        assert lib.bnn_net_destroy(net) == 0
        return n.value

    dummy = ctypes.c_void_p(256)            # pointers are only stored by the add calls

    def mlp(net):
        assert lib.bnn_net_input_u8(net, 784, 127) == 0
        assert lib.bnn_net_add_fc(net, dummy, dummy, 784, 1024) == 0
        assert lib.bnn_net_add_fc(net, dummy, None, 1024, 10) == 0

    def resnet(net):
        assert lib.bnn_net_input_conv_f32(net, dummy, dummy, 32, 32, 3, 64, 7, 4, 3) == 0
        assert lib.bnn_net_add_block(net, dummy, dummy, dummy, dummy, None, 64, 64, 1, 0) == 0
        assert lib.bnn_net_add_block(net, dummy, dummy, dummy, dummy, dummy, 64, 128, 2, 0) == 0
        assert lib.bnn_net_add_head_f32(net, dummy, 10) == 0

    assert ws(mlp, 8) < ws(mlp, 1024)
    small, big = ws(resnet, 2), ws(resnet, 64)
    assert small < big
    # at least: two residual slots of 16-bit sums for the largest block output, and its bits twice
    assert big >= 2 * 64 * 8 * 8 * 64 * 2 + 2 * 64 * 8 * 8 * 8


def test_bands_where_they_gain():
    # steps of the band kernel and of the direct kernel's tiles: where a round more costs more than the direct kernel's next tile, the direct kernel
    import paper_2006_16578_amd as b

    def band(B, h, w, C, O, **kw):
        return "_band_" in b.bconv_kernel_name(B, h, w, C, O, 3, 1, 1, **kw)

    for pad_mode in (0, 1):
        chain = dict(residual=True, keep_sum=True, pad_mode=pad_mode)
        assert [band(B, 16, 16, 256, 256, **chain) for B in (480, 488, 512, 528)] == [True, False, False, True]
        assert band(24, 14, 14, 256, 256) == band(24, 14, 14, 256, 256, **chain) == False
    assert not band(19, 146, 139, 256, 128) and not band(21, 192, 192, 256, 64) and band(256, 14, 14, 256, 256) and band(64, 56, 56, 256, 128)
    assert not band(28, 94, 94, 512, 64) and band(171, 14, 14, 512, 64) and band(195, 54, 54, 512, 64)


def test_eight_wave_tiles_where_they_gain():
    # patches above 80 KB: the direct kernel where it was measured the faster one (0.66 to 0.8 of its time), the eight-wave tiles where those are (1.1 to 2.5),
    # always for a partly filled last word with excluded padding
    import paper_2006_16578_amd as b

    def eight(B, hw, C, O, k, stride, pad, pad_mode):
        return any(t in b.bconv_kernel_name(B, hw, hw, C, O, k, stride, pad, pad_mode=pad_mode) for t in ("wg192x256", "wg384x128", "wg768x64"))

    for shape in ((168, 35, 256, 64, 5, 1, 2, 1), (12, 100, 124, 90, 5, 1, 2, 0), (36, 58, 128, 512, 5, 2, 1, 1), (28, 68, 512, 128, 2, 1, 0, 1), (78, 147, 128, 512, 2, 3, 1, 0)):
        assert not eight(*shape), shape
    for shape in ((11, 56, 200, 200, 5, 1, 2, 0), (9, 80, 300, 290, 3, 1, 1, 0), (13, 112, 96, 50, 5, 1, 2, 1), (12, 100, 124, 90, 5, 1, 2, 1)):
        assert eight(*shape), shape


def test_fc_run_refuses_what_its_layers_refuse():
    # an unknown path and a misaligned input (a missing output beside it) of a network whose fully-connected layers go as one launch: the layers' own answers,
    # before anything is launched
    import paper_2006_16578_amd as b
    lib = b.load()
    dummy = ctypes.c_void_p(256)

    def forward(dims, inp, out, path):
        net, ws = ctypes.c_void_p(), ctypes.c_size_t()
        assert lib.bnn_net_create(ctypes.byref(net)) == 0 and lib.bnn_net_input_bits(net, dims[0]) == 0
        for i, (k, n) in enumerate(zip(dims, dims[1:])):
            assert lib.bnn_net_add_fc(net, dummy, dummy if i + 2 < len(dims) else None, k, n) == 0
        assert lib.bnn_net_workspace_bytes(net, 8, ctypes.byref(ws)) == 0
        rc = lib.bnn_net_forward(net, ctypes.c_void_p(inp), ctypes.c_void_p(out), 8, ctypes.c_void_p(4096), ws, path, None)
        assert lib.bnn_net_destroy(net) == 0
        return rc

    for dims in ((256, 128, 10), (256, 128, 64, 10)):
        for path in (-1, 3, 7):
            assert forward(dims, 256, 256, path) == -1
        for path in (b.PATH_AUTO, b.PATH_MFMA):
            assert forward(dims, 264, 256, path) == -2 and forward(dims, 264, 0, path) == -2


def test_fc_run_by_size():
    # how many layers at the head of a network go as one launch, queued and recorded into a graph: host logic
    import paper_2006_16578_amd as b
    lib = b.load()
    dummy = ctypes.c_void_p(256)

    def run(dims, u8, batch, recorded=0):
        net, n = ctypes.c_void_p(), ctypes.c_int(-1)
        assert lib.bnn_net_create(ctypes.byref(net)) == 0
        assert (lib.bnn_net_input_u8(net, dims[0], 127) if u8 else lib.bnn_net_input_bits(net, dims[0])) == 0
        for i, (k, m) in enumerate(zip(dims, dims[1:])):
            assert lib.bnn_net_add_fc(net, dummy, dummy if i + 2 < len(dims) else None, k, m) == 0
        assert lib.bnn_net_fc_run(net, batch, recorded, ctypes.byref(n)) == 0 and lib.bnn_net_destroy(net) == 0
        return n.value

    mlp = (784, 1024, 1024, 1024, 10)
    assert [run(mlp, True, m) for m in (1, 16, 128, 4096, 8192, 8193)] == [5, 5, 5, 5, 5, 0]
    assert [run(mlp, False, m) for m in (8, 128, 129)] == [0, 0, 5]
    # replayed, the kernels for few rows are the faster ones: none of these layers up to 16 rows unless they are many and small
    assert [run(mlp, True, m, 1) for m in (1, 16, 17, 64, 128, 129, 8192)] == [0, 0, 5, 5, 5, 5, 5]
    assert [run((1024, 1024, 10), False, m, 1) for m in (8, 16, 64, 65, 128, 129, 1024, 1025)] == [0, 0, 0, 3, 3, 0, 0, 3]
    assert [run((1024, 1024, 10), False, m) for m in (8, 128, 129, 4096)] == [3, 3, 3, 3]
    assert run((256, 256, 256, 256, 10), True, 8, 1) == 5 and run((784, 256, 10), True, 8, 1) == 0 and run((784, 256, 10), True, 17, 1) == 3
    assert [run((784, 64), True, m, 1) for m in (16, 17, 4096, 4097)] == [0, 2, 2, 0] and run((784, 64), True, 4097) == 2
    # four layers behind the input at most; sums of at most 64 columns; 8-bit rows of 16 or more; what fits LDS
    assert run((128, 64, 64, 64, 64, 64, 5), False, 40) == 5 and run((300, 100, 65), True, 40) == 2 and run((15, 100, 10), True, 40) == 0
    assert run((4001, 70, 10), True, 129) == 0 and run((3001, 70, 10), True, 129) == 3
    n = ctypes.c_int()
    assert lib.bnn_net_fc_run(None, 8, 0, ctypes.byref(n)) == -1


def test_lds_expanded_convolutions_by_output():
    # bits alone go to that kernel from 96 workgroups; sums and residuals leave through a slower epilogue and need more workgroups or a longer K
    import paper_2006_16578_amd as b

    def served(batch, hw, C, **kw):
        return b.bconv_kernel_name(batch, hw, hw, C, C, 3, 1, 1, **kw).startswith("mfma_fp4_conv_xlds")

    for pad_mode in (0, 1):
        assert served(64, 14, 90, pad_mode=pad_mode) and served(64, 14, 90, pad_mode=pad_mode, shortcut=True)        # 98 workgroups
        for kw in (dict(residual=True), dict(keep_sum=True, shortcut=True), dict(residual=True, keep_sum=True)):
            assert not served(64, 14, 90, pad_mode=pad_mode, **kw)
            assert served(256, 14, 300, pad_mode=pad_mode, **kw)
    # 27 words of K, 392 workgroups: a residual pays in both conventions, bits and sums only where the direct kernel corrects by pixel
    assert served(64, 28, 90, residual=True) and not served(64, 28, 90, shortcut=True, keep_sum=True)
    assert served(64, 28, 90, pad_mode=1, residual=True) and served(64, 28, 90, pad_mode=1, shortcut=True, keep_sum=True)
    # ... and not against the direct kernel's 256x128 tile
    assert not served(128, 28, 90, residual=True) and served(128, 28, 90)
    # sums alone: 132 workgroups, 96 with excluded padding and no unrolled form of the direct kernel
    assert not served(64, 14, 90, int32_out=True) and served(128, 14, 90, int32_out=True) and served(64, 14, 90, pad_mode=1, int32_out=True)
    assert not served(64, 14, 100, pad_mode=1, int32_out=True)
    # ... except images of 1 GiB, which the direct kernel cannot address
    for kw in (dict(residual=True), dict(keep_sum=True, shortcut=True)):
        assert b.bconv_kernel_name(2, 1 << 20, 256, 32, 90, 4, 1, 1, **kw).startswith("mfma_fp4_conv_xlds")
        assert not b.bconv_kernel_name(2, 1 << 10, 256, 32, 90, 4, 1, 1, **kw).startswith("mfma_fp4_conv_xlds")
    # bits alone below 192 workgroups, -1 padding: what a workgroup stages per K-step is bounded, by the words of a pixel
    def conv(batch, hw, C, O, k, stride, pad_mode=0):
        return b.bconv_kernel_name(batch, hw, hw, C, O, k, stride, k // 2, pad_mode=pad_mode).startswith("mfma_fp4_conv_xlds")

    assert not conv(123, 32, 64, 55, 5, 2) and conv(123, 32, 64, 55, 5, 2, 1) and conv(300, 32, 64, 55, 5, 2)
    assert not conv(64, 14, 128, 120, 5, 1) and conv(64, 14, 96, 120, 5, 1)
    # blocked 16-bit sums stay on the direct kernels
    assert not served(256, 14, 96, residual=True, keep_sum=True)


def test_blocked_sums_are_read_by_the_kernel_that_writes_them():
    # the 16-bit sums between two blocks lie in the order of the writing kernel: over shapes, whichever way a block pads, with a shortcut, a residual and a
    # last sum that is not kept, the same kernel (the direct one's tiles and the wave-per-tap kernel share an order)
    import paper_2006_16578_amd as b

    def order(name):
        assert "xlds" not in name and "lds_wg" not in name
        return "band" if "_band_" in name else "patch" if "_patch_" in name else "accumulator"

    seen = set()
    for hw in (5, 7, 13, 14, 28, 33, 56):
        for C in (32, 64, 96, 128, 192, 256, 320, 512, 1024):
            for batch in (1, 2, 4, 8, 16, 26, 40, 57, 73, 85, 104, 128, 146, 200, 256, 292, 400, 512, 585, 1024):
                kinds = {order(b.bconv_kernel_name(batch, hw, hw, C, C, 3, 1, 1, pad_mode=pad_mode, **kw)) for pad_mode in (0, 1)
                         for kw in (dict(shortcut=True, keep_sum=True), dict(residual=True, keep_sum=True), dict(residual=True))}
                assert len(kinds) == 1, (batch, hw, C, kinds)
                seen |= kinds
    assert seen == {"band", "patch", "accumulator"}


def test_stream_without_the_private_torch_function(monkeypatch):
    import types
    from paper_2006_16578_amd import binding as b
    t = types.SimpleNamespace(device="dev", get_device=lambda: 3)
    monkeypatch.setattr(b, "_raw_stream", lambda index: 0x1000 + index)
    assert b._stream(t).value == 0x1003
    monkeypatch.setattr(b, "_raw_stream", None)
    monkeypatch.setattr(b.torch.cuda, "current_stream", lambda device: types.SimpleNamespace(cuda_stream=0x2000 if device == "dev" else 0))
    assert b._stream(t).value == 0x2000


def test_packs_refuse_rows_beyond_32_bit_columns():
    # a row stride of more than 2^26 words would pass 2^31 columns: refused before anything is launched (the pointers are never read)
    import paper_2006_16578_amd as b
    lib = b.load()
    p, ld = ctypes.c_void_p(256), (1 << 26) + 1
    rows = ctypes.c_int64(1)
    assert lib.bnn_threshold_pack(p, p, p, rows, 64, 64, ld, None) == -3
    assert lib.bnn_pack_f32(p, p, p, rows, 64, ld, None) == -3
    assert lib.bnn_pack_u8(p, 127, p, rows, 64, ld, None) == -3
    assert lib.bnn_sign_pack_f32(p, p, rows, 64, 64, ld, None) == -3


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0 and "ONE GPU" in (r.stdout + r.stderr)

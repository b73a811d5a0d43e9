"""Host-side checks of the C ABI: the library loads, exports every declared symbol, and every
argument error is reported before any launch (no GPU needed)."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def dp():
    from paper_2112_10065_amd import binding
    return binding


def test_exports_every_declared_symbol(dp):
    hdr = open(os.path.join(ROOT, "include", "dp.h")).read()
    declared = set(re.findall(r"\b(dp_[a-z0-9_]+)\s*\(", hdr))
    assert {"dp_conv2d_fwd", "dp_conv2d_bwd_data", "dp_conv2d_bwd_filter", "dp_linear_fwd_bwd",
            "dp_profile_layer"} <= declared
    for name in declared:
        assert hasattr(dp.lib, name), name
    assert declared == set(dp.EXPORTS)
    assert "gfx950" in dp.dp_version()


def test_struct_sizes_match_header(dp):
    assert C.sizeof(dp.dp_conv_desc) == 13 * 4
    assert C.sizeof(dp.dp_linear_desc) == 5 * 4
    assert C.sizeof(dp.dp_profile_row) == 48


@pytest.mark.parametrize("initialised,raw,want", [(True, True, 7), (True, False, 9), (False, True, 9)])
def test_current_stream_without_the_private_functions(dp, monkeypatch, initialised, raw, want):
    import types
    import torch
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: initialised)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=9))
    private = types.SimpleNamespace(_cuda_getDevice=lambda: 0)
    if raw:
        private._cuda_getCurrentRawStream = lambda device: 7
    monkeypatch.setattr(torch, "_C", private)
    got = dp._current_stream()
    monkeypatch.undo()
    assert got == want


A = 0x1000  # fake, 16-byte aligned, never dereferenced: validation fails first


def test_conv_argument_errors(dp):
    lib = dp.lib
    good = dp.conv_desc(2, 16, 16, 16, 16, 3, 3, (1, 1), (1, 1), dp.DP_BF16, dp.DP_BIAS)
    assert lib.dp_conv2d_fwd(None, A, A, A, A, None, 0, None) == dp.DP_ERR_NULL
    assert lib.dp_conv2d_fwd(C.byref(good), None, A, A, A, None, 0, None) == dp.DP_ERR_NULL
    assert b"x is NULL" in lib.dp_last_error()
    assert lib.dp_conv2d_fwd(C.byref(good), A, A, None, A, None, 0, None) == dp.DP_ERR_NULL  # DP_BIAS without bias
    assert lib.dp_conv2d_fwd(C.byref(good), A + 2, A, A, A, None, 0, None) == dp.DP_ERR_BAD_DESC  # misaligned
    bad = dp.conv_desc(0, 16, 16, 16, 16, 3, 3)
    assert lib.dp_conv2d_fwd(C.byref(bad), A, A, A, A, None, 0, None) == dp.DP_ERR_BAD_DESC
    bad = dp.conv_desc(1, 2, 2, 4, 4, 3, 3)  # filter larger than the unpadded image
    assert lib.dp_conv2d_bwd_data(C.byref(bad), A, None, A, A, None, 0, None) == dp.DP_ERR_BAD_DESC
    bad = dp.conv_desc(1, 8, 8, 4, 4, 3, 3, io_dtype=7)
    assert lib.dp_conv2d_bwd_filter(C.byref(bad), A, A, None, A, None, None, 0, None) == dp.DP_ERR_UNSUPPORTED
    bad = dp.conv_desc(1, 8, 8, 4, 4, 3, 3, flags=1 << 20)
    assert lib.dp_conv2d_fwd(C.byref(bad), A, A, A, A, None, 0, None) == dp.DP_ERR_UNSUPPORTED
    bad = dp.conv_desc(1, 8, 8, 4, 4, 3, 3, io_dtype=dp.DP_F32, flags=dp.DP_DX_F32)
    assert lib.dp_conv2d_fwd(C.byref(bad), A, A, A, A, None, 0, None) == dp.DP_ERR_UNSUPPORTED
    huge = dp.conv_desc(1 << 12, 1 << 10, 1 << 10, 8, 8, 1, 1)
    assert lib.dp_conv2d_fwd(C.byref(huge), A, A, A, A, None, 0, None) == dp.DP_ERR_BAD_DESC
    assert dp.dp_conv2d_workspace_bytes(bad, 0) == 0
    assert dp.dp_conv2d_workspace_bytes(good, 9) == 0


def test_workspace_errors(dp):
    lib = dp.lib
    # backward-filter always splits its long reduction here -> needs scratch
    d = dp.conv_desc(2, 56, 56, 64, 64, 3, 3, (1, 1), (1, 1), dp.DP_BF16, 0)
    need = dp.dp_conv2d_workspace_bytes(d, dp.DP_PASS_WGRAD)
    assert need > 0
    assert lib.dp_conv2d_bwd_filter(C.byref(d), A, A, None, A, A, None, 0, None) == dp.DP_ERR_WORKSPACE
    assert lib.dp_conv2d_bwd_filter(C.byref(d), A, A, None, A, A, A, 16, None) == dp.DP_ERR_WORKSPACE
    ld = dp.linear_desc(4, 4096, 4096, dp.DP_BF16, 0)
    assert dp.dp_linear_workspace_bytes(ld) > 0
    assert lib.dp_linear_fwd_bwd(C.byref(ld), A, A, None, None, None, A, None, None, None, None, 0, None) == dp.DP_ERR_WORKSPACE
    assert lib.dp_relu_bias_grad(100, 64, dp.DP_BF16, A, A, None, A, None, 0, None) == dp.DP_ERR_WORKSPACE
    assert dp.dp_relu_bias_grad_workspace_bytes(100, 64) > 0


def test_noalloc_backward_filter_argument_errors(dp):
    """The allocation-free form validates like dp_conv2d_bwd_filter and rejects layers beyond its built-in scratch
    before any HIP call."""
    lib = dp.lib
    d = dp.conv_desc(2, 28, 28, 64, 64, 3, 3, (1, 1), (1, 1), dp.DP_BF16, 0)
    assert lib.dp_conv2d_bwd_filter_noalloc(None, A, A, None, A, A, None) == dp.DP_ERR_NULL
    assert lib.dp_conv2d_bwd_filter_noalloc(C.byref(d), None, A, None, A, A, None) == dp.DP_ERR_NULL
    assert lib.dp_conv2d_bwd_filter_noalloc(C.byref(d), A, A, None, None, A, None) == dp.DP_ERR_NULL
    assert lib.dp_conv2d_bwd_filter_noalloc(C.byref(d), A, A + 4, None, A, A, None) == dp.DP_ERR_BAD_DESC
    big = dp.conv_desc(32, 224, 224, 64, 64, 3, 3, (1, 1), (1, 1), dp.DP_BF16, 0)
    assert dp.dp_conv2d_workspace_bytes(big, dp.DP_PASS_WGRAD) > dp.DP_NOALLOC_SCRATCH_BYTES
    assert lib.dp_conv2d_bwd_filter_noalloc(C.byref(big), A, A, None, A, A, None) == dp.DP_ERR_WORKSPACE
    assert b"built-in scratch" in lib.dp_last_error()
    hdr = open(os.path.join(ROOT, "include", "dp.h")).read()
    assert "#define DP_NOALLOC_SCRATCH_BYTES ((size_t)32 << 20)" in hdr and dp.DP_NOALLOC_SCRATCH_BYTES == 32 << 20


def test_linear_and_pointwise_argument_errors(dp):
    lib = dp.lib
    ld = dp.linear_desc(4, 64, 32, dp.DP_BF16, dp.DP_BIAS)
    N = None
    assert lib.dp_linear_fwd_bwd(C.byref(ld), A, A, A, N, N, N, N, N, N, N, 0, N) == dp.DP_ERR_NULL  # nothing requested
    assert lib.dp_linear_fwd_bwd(C.byref(ld), N, A, A, N, N, A, N, N, N, N, 0, N) == dp.DP_ERR_NULL  # y needs x
    assert lib.dp_linear_fwd_bwd(C.byref(ld), A, A, A, N, N, N, A, N, N, N, 0, N) == dp.DP_ERR_NULL  # dx needs dy
    assert lib.dp_linear_fwd_bwd(C.byref(dp.linear_desc(0, 64, 32)), A, A, A, N, N, A, N, N, N, N, 0, N) == dp.DP_ERR_BAD_DESC
    assert lib.dp_relu_bias_grad(0, 64, dp.DP_BF16, A, A, A, N, N, 0, N) == dp.DP_ERR_BAD_DESC
    assert lib.dp_relu_bias_grad(10, 64, dp.DP_BF16, A, A, N, N, N, 0, N) == dp.DP_ERR_NULL
    assert lib.dp_relu_bias_grad(10, 64, 5, A, A, A, N, N, 0, N) == dp.DP_ERR_UNSUPPORTED


def test_profile_and_override_argument_errors(dp):
    lib = dp.lib
    cd = dp.conv_desc(1, 8, 8, 8, 8, 3, 3, (1, 1), (1, 1))
    ld = dp.linear_desc(1, 8, 8)
    rows = (dp.dp_profile_row * 1)()
    b = (C.c_int32 * 1)(1)
    assert lib.dp_profile_layer(None, None, b, 1, 1, 1, rows, None) == dp.DP_ERR_NULL
    assert lib.dp_profile_layer(C.byref(cd), C.byref(ld), b, 1, 1, 1, rows, None) == dp.DP_ERR_NULL
    assert lib.dp_profile_layer(C.byref(cd), None, None, 1, 1, 1, rows, None) == dp.DP_ERR_NULL
    assert lib.dp_profile_layer(C.byref(cd), None, b, 1, 1, 0, rows, None) == dp.DP_ERR_BAD_DESC
    bneg = (C.c_int32 * 1)(-3)
    assert lib.dp_profile_layer(C.byref(cd), None, bneg, 1, 1, 1, rows, None) == dp.DP_ERR_BAD_DESC
    assert lib.dp_set_override(5, 0, 0) == dp.DP_ERR_UNSUPPORTED
    assert lib.dp_set_override(0, -1, 0) == dp.DP_OK
    assert lib.dp_set_autotune(1) == dp.DP_OK and lib.dp_set_autotune(0) == dp.DP_OK
    # the trace hook: end without begin, begin twice, missing output arguments; an empty trace has no rows
    n = C.c_int32(7)
    trows = (dp.dp_trace_row * 2)()
    assert lib.dp_trace_end(trows, 2, C.byref(n)) == dp.DP_ERR_UNSUPPORTED
    assert lib.dp_trace_begin() == dp.DP_OK and lib.dp_trace_begin() == dp.DP_ERR_UNSUPPORTED
    assert lib.dp_trace_end(trows, 2, None) == dp.DP_ERR_NULL
    assert lib.dp_trace_begin() == dp.DP_OK
    assert lib.dp_trace_end(trows, 2, C.byref(n)) == dp.DP_OK and n.value == 0
    assert C.sizeof(dp.dp_trace_row) == 96 + 16


def test_no_gpu_fails_loudly(dp):
    """On a host without a GPU a valid call must return DP_ERR_HIP, never succeed or fall back."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("GPU present")
    d = dp.conv_desc(1, 8, 8, 8, 8, 3, 3, (1, 1), (1, 1), dp.DP_BF16, 0)
    assert dp.lib.dp_conv2d_fwd(C.byref(d), A, A, None, A, None, 0, None) == dp.DP_ERR_HIP
    assert dp.lib.dp_last_error() != b""


def test_glue_argument_errors(dp):
    lib = dp.lib
    assert lib.dp_maxpool2x2_fwd(1, 4, 4, 8, dp.DP_BF16, None, A, None) == dp.DP_ERR_NULL
    assert lib.dp_maxpool2x2_fwd(1, 4, 4, 8, dp.DP_BF16, A, None, None) == dp.DP_ERR_NULL
    assert lib.dp_maxpool2x2_fwd(1, 4, 4, 8, 5, A, A, None) == dp.DP_ERR_UNSUPPORTED
    assert lib.dp_maxpool2x2_fwd(0, 4, 4, 8, dp.DP_BF16, A, A, None) == dp.DP_ERR_BAD_DESC
    assert lib.dp_maxpool2x2_fwd(1, 4, 4, 8, dp.DP_BF16, A + 2, A, None) == dp.DP_ERR_BAD_DESC
    assert lib.dp_maxpool2x2_bwd(1, 4, 4, 8, dp.DP_BF16, A, None, A, None) == dp.DP_ERR_NULL
    assert lib.dp_maxpool2x2_bwd(1, 4, 4, 8, dp.DP_BF16, A, A, None, None) == dp.DP_ERR_NULL
    assert lib.dp_softmax_xent(4, 10, dp.DP_F32, A, None, A, None, None) == dp.DP_ERR_NULL
    assert lib.dp_softmax_xent(4, 0, dp.DP_F32, A, A, A, None, None) == dp.DP_ERR_BAD_DESC
    assert lib.dp_softmax_xent(4, 10, 9, A, A, A, None, None) == dp.DP_ERR_UNSUPPORTED
    assert lib.dp_sgd_update(16, 0.1, 0.9, None, A, A, None, None) == dp.DP_ERR_NULL
    assert lib.dp_sgd_update(-1, 0.1, 0.9, A, A, A, None, None) == dp.DP_ERR_BAD_DESC
    assert lib.dp_sgd_update(16, 0.1, 0.9, A, A + 4, A, None, None) == dp.DP_ERR_BAD_DESC
    assert lib.dp_sgd_update(0, 0.1, 0.9, A, A, A, None, None) == dp.DP_OK   # nothing to do, nothing launched


def test_fused_input_relu_argument_errors(dp):
    lib = dp.lib
    d = dp.conv_desc(2, 16, 16, 16, 16, 3, 3, (1, 1), (1, 1), dp.DP_BF16, dp.DP_RELU_IN)
    assert lib.dp_conv2d_bwd_data(C.byref(d), A, None, A, A, None, 0, None) == dp.DP_ERR_NULL        # no saved input to mask with
    assert b"x_saved" in lib.dp_last_error()
    assert lib.dp_conv2d_bwd_data_relu(C.byref(d), A, None, A, None, A, None, 0, None) == dp.DP_ERR_NULL
    assert lib.dp_conv2d_bwd_data_relu(C.byref(d), A, None, A, A + 8, A, None, 0, None) == dp.DP_ERR_BAD_DESC  # misaligned
    ld = dp.linear_desc(4, 64, 32, dp.DP_BF16, dp.DP_RELU_IN)
    assert lib.dp_linear_fwd_bwd(C.byref(ld), None, A, None, A, None, None, A, None, None, None, 0, None) == dp.DP_ERR_NULL  # dx needs x
    # the flag changes which kernels a call may use, so the workspace query takes it into account without failing
    assert dp.dp_conv2d_workspace_bytes(d, 1) >= 0


def test_pixel_strip_plan_rules(dp):
    """Host logic of the kernel choice (no GPU call): the pixel-strip kernels are planned for the 3x3 / stride 1 / pad 1
    layers with 128 or more reduction channels on grids of 160 or more blocks, never for fp32 input gradients, other
    filters, strides or paddings, and a reduction split takes an even number of 64-channel blocks."""
    def info(n, h, c, k, pass_, r=3, stride=(1, 1), pad=(1, 1), extra=0):
        d = dp.conv_desc(n, h, h, c, k, r, r, stride, pad, dp.DP_BF16, dp.DP_BIAS | dp.DP_RELU | extra)
        return dp.dp_conv2d_kernel_info(d, pass_)
    assert info(32, 56, 256, 256, 0) == ("k_conv_strip<false, 224, 256>", 1)        # conv3_2: 448 tiles of 224 pixels fill two rounds of
    assert info(32, 56, 256, 256, 1) == ("k_conv_strip<true, 224, 256>", 1)         # 256 blocks better than 392 tiles of 256
    assert info(32, 28, 512, 512, 0) == ("k_conv_strip<false, 224, 256>", 1)        # conv4_2: 224 blocks instead of 196
    assert info(32, 14, 512, 512, 0) == ("k_conv_strip<false, 128, 256>", 2)        # conv5_x: 98 tiles, two splits of four blocks
    assert "k_conv_strip" not in info(32, 56, 256, 256, 1, extra=dp.DP_DX_F32)[0]   # bf16 staged epilogue only
    assert "k_conv_strip" not in info(4, 14, 512, 512, 0)[0]                         # too few blocks
    assert "k_conv_strip" not in info(32, 56, 64, 256, 0)[0]                         # 64 reduction channels
    assert "k_conv_strip" not in info(32, 56, 256, 256, 0, r=1, pad=(0, 0))[0]
    assert "k_conv_strip" not in info(32, 56, 256, 256, 0, stride=(2, 2))[0]
    assert "k_conv_strip" not in info(32, 56, 256, 256, 2)[0]                        # not a filter-gradient kernel
    for code, splits, want in ((230, 2, 2), (230, 3, 2), (230, 4, 2), (231, 4, 2), (232, 8, 2)):   # 256 channels: four blocks
        dp.dp_set_override(0, code, splits)
        try:
            assert info(8, 28, 256, 256, 0)[1] == want
        finally:
            dp.dp_set_override(0, -1, 0)
    dp.dp_set_override(1, 230, 4)
    try:
        assert info(8, 14, 512, 512, 1) == ("k_conv_strip<true, 256, 256>", 4)      # 512 channels: eight blocks, four splits of two
    finally:
        dp.dp_set_override(1, -1, 0)



def test_flat_walk_backward_data_plan_rules(dp):
    """Host logic of the kernel choice (no GPU call): where 64 does not divide c_out, the flat-walk kernels take the place of the generic
    kernel and of split 64x128 tiles of 32-wide steps, and of no kernel that is faster than they are."""
    def name(n, h, c, k, r, s, stride=(1, 1), pad=(0, 0)):
        return dp.dp_conv2d_kernel_info(dp.conv_desc(n, h, h, c, k, r, s, stride, pad, dp.DP_BF16, dp.DP_RELU | dp.DP_RELU_IN), 1)[0]
    assert name(30, 27, 352, 352, 1, 3, pad=(0, 1)).startswith("k_dgrad_dma<128, 128, 32")       # flat 42 us against 29
    assert name(25, 30, 384, 352, 1, 7, pad=(0, 3)).startswith("k_dgrad_dma<128, 128, 32")       # 82 against 60
    assert name(25, 17, 288, 352, 1, 3, pad=(0, 1)).startswith("k_dgrad_dma<64, 128, 32")        # 19.7 against 17.7
    assert name(27, 11, 96, 96, 1, 3, pad=(0, 1)).startswith("k_conv_fast<1, 64, 64, 32")        # 7.7 against 6.0
    assert name(7, 11, 96, 288, 1, 3, pad=(0, 1)).startswith("k_conv_fast<1, 64, 64, 32")        # 10.1 against 8.9
    assert name(6, 9, 16, 16, 1, 1).startswith("k_conv_gemm<1")
    assert name(15, 56, 208, 400, 3, 3, pad=(1, 1)).startswith("k_dgrad_mix<")                   # 118 against 282
    assert name(5, 109, 144, 240, 5, 5, (2, 2), (1, 1)).startswith("k_dgrad_mix<")               # 89 against 540
    assert name(12, 14, 320, 288, 1, 7, pad=(0, 3)).startswith("k_dgrad_mix<")                   # 14.3 against 20.4 in five splits
    assert name(2, 17, 400, 288, 3, 3, (2, 2), (1, 1)).startswith("k_dgrad_mix<")                # 12 against 18
    assert not name(16, 17, 160, 192, 7, 1, pad=(3, 0)).startswith("k_dgrad_mix<")               # 64 divides c_out


def test_backward_data_scratch_is_optional_where_a_slower_form_needs_none(dp):
    """A layer that 64 does not divide ran without scratch on the generic kernel; a faster kernel that wants some does not take that away.
    Valid calls get as far as the missing GPU."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("would launch on the addresses made up here")
    d = dp.conv_desc(6, 126, 126, 240, 400, 3, 3, (1, 1), (1, 1), dp.DP_BF16, dp.DP_RELU_IN)
    assert dp.dp_conv2d_workspace_bytes(d, 1) > 0
    for saved in (None, A):
        assert dp.lib.dp_conv2d_bwd_data_relu(C.byref(d), A, saved, A, A, A, None, 0, None) == dp.DP_ERR_HIP
    # a layer that always wanted scratch is rejected as before
    d = dp.conv_desc(2, 56, 56, 64, 64, 3, 3, (1, 1), (1, 1), dp.DP_BF16, 0)
    assert dp.dp_conv2d_workspace_bytes(d, 1) > 0
    assert dp.lib.dp_conv2d_bwd_data(C.byref(d), A, None, A, A, None, 0, None) == dp.DP_ERR_WORKSPACE


def test_filter_gradient_split_rounding_rules(dp):
    """Host logic of the kernel choice (no GPU call): the empty splits that make a count a multiple of eight come after the choice of the
    plan, with operands of 32 MB and more and more than 16 splits only."""
    def info(n, h, w, c, k, r, s, stride=1, pad=(0, 0)):
        return dp.dp_conv2d_kernel_info(dp.conv_desc(n, h, w, c, k, r, s, (stride, stride), pad, dp.DP_BF16, 0), 2)
    assert info(64, 56, 56, 256, 512, 1, 1, 2) == ("k_wgrad_dma<64, 128, 64, 2, 2, 2>", 48)          # 47 of them work: 47.6 -> 30.7 us
    assert info(45, 58, 58, 256, 256, 1, 1) == ("k_wgrad_dma<64, 128, 64, 2, 2, 2>", 96)             # 95: 79 -> 38
    assert info(17, 18, 18, 192, 224, 1, 7, pad=(0, 3)) == ("k_wgrad_dma<64, 128, 64, 2, 2, 2>", 15)   # 16 splits: 18.8 -> 22.5
    assert info(3, 27, 27, 256, 1024, 1, 1) == ("k_wgrad_dma<64, 128, 64, 2, 2, 2>", 7)              # 8: 12.9 -> 13.6
    assert info(4, 61, 66, 192, 128, 3, 3, pad=(1, 1)) == ("k_wgrad_dma<64, 128, 64, 2, 2, 2>", 23)  # 24: 24.1 -> 26.5
    # priced with their empty splits these lost their plan to the register-staged kernel or to fewer splits
    assert info(1, 43, 48, 64, 128, 3, 3, pad=(1, 1)) == ("k_wgrad_dma<64, 64, 32, 2, 2, 2>", 13)    # 9.0 against 15.2
    assert info(2, 29, 29, 128, 384, 1, 3, pad=(0, 1)) == ("k_wgrad_dma<64, 128, 32, 2, 2, 2>", 14)  # 12.2 against 16.7
    assert info(9, 46, 46, 640, 320, 1, 1) == ("k_wgrad_dma<64, 128, 64, 2, 2, 2>", 32)              # 30 of them work


def test_filter_gradient_takes_the_scratch_that_was_enough_before(dp):
    """Less scratch than the query names is enough where only the empty splits or the stem kernel's one partial do not fit; valid calls get as far
    as the missing GPU."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("would launch on the addresses made up here")
    for d, enough in ((dp.conv_desc(45, 58, 58, 256, 256, 1, 1, (1, 1), (0, 0), dp.DP_BF16, 0), 102934528),     # 95 splits, the query says 96
                      (dp.conv_desc(1, 7, 9, 2, 8, 7, 6, (2, 2), (0, 1), dp.DP_BF16, 0), 20480)):               # im2col matrix of four pixels
        assert dp.dp_conv2d_workspace_bytes(d, 2) > enough
        assert dp.lib.dp_conv2d_bwd_filter(C.byref(d), A, A, None, A, A, A, enough, None) == dp.DP_ERR_HIP
        assert dp.lib.dp_conv2d_bwd_filter(C.byref(d), A, A, None, A, A, A, enough - 256, None) == dp.DP_ERR_WORKSPACE


def test_filter_gradient_of_nine_tap_layers_takes_the_window_kernels_scratch(dp):
    """The nine-tap kernel, and the tiles that are faster than the window kernel, ask for more scratch than the window kernel, and the nine-tap kernel for more than
    with larger tiles.  A call with what those ask for is accepted, also without a workspace of its own where that fits the built-in scratch.  Valid calls get as far as the missing GPU."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("would launch on the addresses made up here")
    # (n, h, w, c_out, pad, what the window kernel's plan asks for, whether that fits the 32 MiB built in)
    for n, h, w, k, pad, enough, builtin in ((8, 153, 149, 128, 1, 65529856, False), (48, 35, 39, 8, 1, 2723584, True), (30, 26, 23, 384, 0, 28323840, True),
                                             (6, 212, 217, 40, 1, 33315328, True), (21, 27, 29, 256, 1, 22509056, True), (10, 93, 92, 320, 1, 73845760, False),
                                             # the nine-tap kernel's plan with fewer blocks
                                             (2, 193, 174, 32, 1, 11441920, True), (3, 109, 110, 192, 1, 28361472, True), (16, 16, 16, 440, 1, 12615680, True)):
        d = dp.conv_desc(n, h, w, 64, k, 3, 3, (1, 1), (pad, pad), dp.DP_BF16, 0)
        for saved in (None, A):
            assert dp.lib.dp_conv2d_bwd_filter(C.byref(d), A, A, saved, A, A, A, enough, None) == dp.DP_ERR_HIP, (n, h, w, k)
        assert (dp.lib.dp_conv2d_bwd_filter_noalloc(C.byref(d), A, A, None, A, A, None) == dp.DP_ERR_HIP) == builtin
        # the message names what is enough
        assert dp.lib.dp_conv2d_bwd_filter(C.byref(d), A, A, None, A, A, None, 0, None) == dp.DP_ERR_WORKSPACE
        least = int(re.search(rb"needs (\d+) workspace", dp.lib.dp_last_error()).group(1))
        assert least <= enough and dp.lib.dp_conv2d_bwd_filter(C.byref(d), A, A, None, A, A, A, least, None) == dp.DP_ERR_HIP
        assert dp.lib.dp_conv2d_bwd_filter(C.byref(d), A, A, None, A, A, A, least - 256, None) == dp.DP_ERR_WORKSPACE
    # the query is what the fastest form takes
    d = dp.conv_desc(8, 153, 149, 64, 128, 3, 3, (1, 1), (1, 1), dp.DP_BF16, 0)
    assert dp.dp_conv2d_kernel_info(d, 2)[0] == "k_wgrad_halo9<true>" and dp.dp_conv2d_workspace_bytes(d, 2) > 65529856


def test_backward_data_tile_price_rules(dp):
    """Host logic of the kernel choice (no GPU call): the mask of lone 256x256 tiles and the wide 64x256 tiles of short reductions are priced in
    for layers of more than one round of blocks, where the tiles that replace them are faster, and change nothing else."""
    def name(n, h, w, c, k, r=1, pass_=1, pad=0):
        d = dp.conv_desc(n, h, w, c, k, r, r, (1, 1), (pad, pad), dp.DP_BF16, dp.DP_RELU | dp.DP_RELU_IN)
        return dp.dp_conv2d_kernel_info(d, pass_)[0].replace("k_dgrad_dma", "").replace("k_fwd_dma", "")
    assert name(16, 65, 65, 256, 576) == "<128, 64, 64, 2, 2, 2, 1>"                   # 256x256 without the mask
    assert name(13, 138, 136, 64, 192, 3, pad=1) == "<64, 128, 64, 2, 2, 2, 1>"        # as 128 channels were: 64x256 82, 59
    assert name(54, 18, 18, 768, 576) == "<256, 256, 64, 2, 4, 2, 1>"                  # one round
    assert name(54, 48, 48, 192, 768) == "<256, 256, 64, 2, 4, 2, 1>"                  # two full rounds; 64x128: 72, 80
    # the kernels with stationary weights, each in the place of the tile that these rules had chosen (64 x 56 x 56, 256 <- 128: 57 us -> 38)
    assert name(64, 56, 56, 256, 128) == "k_pointwise<1, 2, 2, 4, true>"
    assert name(22, 37, 37, 256, 128) == "k_pointwise<1, 2, 1, 4, true>"
    assert name(54, 18, 18, 768, 192) == "k_pointwise<1, 3, 1, 4, true>"
    assert name(24, 65, 65, 256, 64) == "k_pointwise<1, 1, 2, 4, true>"
    assert name(13, 138, 136, 64, 128, 3, pad=1) == "k_halo_ws<1, true, 2>"
    assert name(11, 76, 71, 512, 64, 3, pad=1) == "k_halo_ws<1, true>"
    assert name(23, 41, 42, 128, 192, 3, pass_=0, pad=1) == "k_halo_ws<0, false, 2>"
    assert name(27, 68, 61, 64, 192, 3, pad=1) == "<64, 256, 64, 1, 4, 2, 1>"          # 64x128: 53, 60
    assert name(14, 4, 4, 128, 512) == "<64, 64, 64, 2, 2, 2, 4>"                      # small grids: as without a mask
    assert name(1, 11, 11, 512, 128) == "<64, 64, 128, 2, 2, 3, 1>"
    assert name(23, 41, 42, 192, 192, 3, pass_=0, pad=1) == "<64, 256, 64, 1, 4, 2, 1>"   # forward: as before


def test_few_tiles_of_64_channels_keep_the_smallest_window_tile(dp):
    """Host logic of the kernel choice (no GPU call): where the smallest tile of the window kernel is its cheapest, a layer of 64 reduction channels has too few tiles
    for the kernel that keeps nine taps of weights in registers."""
    def name(n, h, c, k, pass_, flags=dp.DP_RELU_IN):
        return dp.dp_conv2d_kernel_info(dp.conv_desc(n, h, h, c, k, 3, 3, (1, 1), (1, 1), dp.DP_BF16, dp.DP_RELU | flags), pass_)[0]
    assert name(1, 17, 64, 16, 0) == "k_conv_win<false, 1, 2, 1, false>"     # 8.6 us, 8.1 with flushed caches
    assert name(4, 9, 64, 256, 0) == "k_conv_win<false, 1, 2, 1, false>"     # 8.9, 8.2
    assert name(2, 16, 256, 64, 1) == "k_conv_win<true, 1, 2, 1, false>"     # 8.5, 8.3
    assert name(3, 59, 64, 64, 0) == "k_halo_ws<0, false>"                   # 9.2 for the 10.2 of wider window tiles
    assert name(4, 9, 64, 256, 0, 0) == "k_halo_ws<0, false>"                # masks by its own y: keeps the order of its sums


def test_stationary_weights_of_64_channels_are_priced_by_whole_rounds(dp):
    """Host logic of the kernel choice (no GPU call): a layer with a little more than one or two tiles per persistent block pays for the next round; tiles or
    the window kernel, which fill the chip evenly, run it.  Just below, and from three rounds on, it is the faster one."""
    def name(n, h, w, c, k, pass_, pad=1, flags=dp.DP_RELU_IN):
        return dp.dp_conv2d_kernel_info(dp.conv_desc(n, h, w, c, k, 3, 3, (1, 1), (pad, pad), dp.DP_BF16, dp.DP_RELU | flags), pass_)[0].split("<")[0]
    assert name(25, 20, 20, 64, 240, 0, 0, 0) == "k_fwd_dma"         # 1.17 rounds: 10.7 us, 8.2; masks by its own y: no window kernel
    assert name(22, 22, 19, 64, 232, 0, 0) == "k_fwd_dma"            # 1.03 rounds: 10.2, 7.9
    assert name(19, 49, 49, 64, 128, 0) == "k_fwd_dma"               # 2.08 rounds: 14.7, 12.5
    assert name(12, 46, 47, 64, 80, 0, 2) == "k_conv_win"            # 1.12 rounds: 10.3, 9.5
    assert name(15, 41, 40, 128, 64, 1) == "k_conv_win"              # 1.05 rounds, backward-data: 10.8, 10.0
    assert name(2, 79, 83, 64, 160, 0) == "k_halo_ws"                # 0.8 rounds
    assert name(21, 67, 65, 64, 256, 0, 1, 0) == "k_halo_ws"         # 7.4 rounds: 33.5 for the 42.2 of 256x256 tiles
    assert name(31, 35, 33, 64, 192, 0, 1, 0) == "k_halo_ws"         # 2.7 rounds: 15.3 for 20.6


def test_strided_1x1_fp32_gradient_plan_is_the_one_that_runs(dp):
    """A strided 1x1 layer's fp32 input gradient goes in natural pixel order with all its blocks: its tiles and splits are priced as that
    (as the quarter of the blocks that a bf16 gradient takes, 96 <- 448 ran 31.5 us instead of 17.2)."""
    def info(n, h, c, k, extra=0):
        d = dp.conv_desc(n, h, h, c, k, 1, 1, (2, 2), (0, 0), dp.DP_BF16, dp.DP_RELU | extra)
        return dp.dp_conv2d_kernel_info(d, 1)
    assert info(10, 53, 96, 448, dp.DP_DX_F32) == ("k_dgrad_dma<64, 128, 64, 2, 2, 2, 1>", 1)
    assert info(10, 53, 96, 448)[0] != info(10, 53, 96, 448, dp.DP_DX_F32)[0]


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_forward_takes_the_scratch_of_its_query_with_any_flags(dp, mode):
    """The query knows no flags, the call's kernel choice does: what the query says is enough for every call, over the layers of the tracked
    networks and every choice mode.  Valid calls get as far as the missing GPU."""
    import torch
    from paper_2112_10065_amd import workloads as W
    if torch.cuda.is_available():
        pytest.skip("would launch on the addresses made up here")
    differ = 0
    dp.dp_set_autotune(mode)
    try:
        for l in W.vgg16_convs() + W.resnet50_convs() + W.inception_convs() + W.wrn101_2_convs():
            for n in W.BATCHES:
                asked = []
                for flags in (0, dp.DP_BIAS | dp.DP_RELU, dp.DP_RELU | dp.DP_RELU_IN, dp.DP_RELU | dp.DP_DETERMINISTIC):
                    d = dp.conv_desc(n, l.h, l.w, l.c, l.k, l.r, l.s, (l.sh, l.sw), (l.ph, l.pw), dp.DP_BF16, flags)
                    need = dp.dp_conv2d_workspace_bytes(d, 0)
                    assert dp.lib.dp_conv2d_fwd(C.byref(d), A, A, A, A, A if need else None, need, None) == dp.DP_ERR_HIP, (l, n, flags)
                    if not flags & dp.DP_DETERMINISTIC:
                        asked.append(need)
                    if dp.lib.dp_conv2d_fwd(C.byref(d), A, A, A, A, None, 0, None) == dp.DP_ERR_WORKSPACE:
                        least = int(re.search(rb"needs (\d+) workspace", dp.lib.dp_last_error()).group(1))
                        assert least <= need
                        differ += least < need
                assert len(set(asked)) == 1
    finally:
        dp.dp_set_autotune(0)
    assert mode != 2 or differ > 0   # calls that need less than others exist


def test_pixel_window_plan_keeps_to_rows_and_columns_that_its_reciprocals_divide(dp):
    """The window kernel finds image rows by fp32 reciprocals, exact below 2^21 slots a row (or slot rows an image): longer rows and columns, which
    the filters of one row or column would otherwise let through, have no such plan, not even forced."""
    def name(h, w, r, s, pass_):
        return dp.dp_conv2d_kernel_info(dp.conv_desc(1, h, w, 64, 64, r, s, (1, 1), (r // 2, s // 2), dp.DP_BF16, 0), pass_)[0]
    for pass_ in (0, 1):
        for variant in range(250, 259):
            dp.dp_set_override(pass_, variant, 0)
            try:
                for size, runs in ((5000000, False), (1 << 20, False), (1000000, True)):
                    assert name(1, size, 1, 3, pass_).startswith("k_conv_win<") == runs
                    # columns of 32-row tiles: the window of a filter column is a few slots, whatever the height
                    assert name(size, 1, 3, 1, pass_).startswith("k_conv_win<") == runs
            finally:
                dp.dp_set_override(pass_, -1, 0)


def test_narrow_window_tiles_are_priced_by_what_an_l2_holds(dp):
    """Host logic of the kernel choice (no GPU call): backward-data tiles of 32 channels fetch half lines of weights.  That costs them where the weights
    exceed an L2, not below."""
    def name(n, h, c, k):
        return dp.dp_conv2d_kernel_info(dp.conv_desc(n, h, h, c, k, 3, 3, (1, 1), (1, 1), dp.DP_BF16, dp.DP_RELU | dp.DP_RELU_IN), 1)[0]
    assert name(2, 10, 512, 384).startswith("k_conv_win<true, 1, 2, 1")    # 3.5 MB: 12.3 us in tiles of 64x64 with splits, 8.7
    assert name(1, 19, 512, 256).startswith("k_conv_win<true, 1, 2, 1")    # 2.4 MB: 11.5, 7.8
    assert name(1, 16, 736, 192).startswith("k_conv_win<true, 1, 2, 1")    # 2.5 MB: 10.6, 7.5
    assert not name(1, 14, 512, 512).startswith("k_conv_win")              # 4.7 MB: 11.7, 13.8
    assert not name(1, 14, 256, 1024).startswith("k_conv_win")             # 4.7 MB: 12.8, 19.8
    assert not name(1, 13, 1024, 1024).startswith("k_conv_win<true, 1, 2, 1")   # 18.9 MB: 19.1, 27.9

"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, rejects bad arguments before touching the device, and maps workgroup ids to
output tiles bijectively."""
import ctypes
import re
from pathlib import Path

import numpy as np
import pytest

from paper_2207_04296_amd import binding as B

ROOT = Path(__file__).resolve().parent.parent


def test_library_exports_every_declared_symbol():
    header = (ROOT / "include" / "tir.h").read_text()
    declared = set(re.findall(r"\b(tir_[a-z0-9_]+)\s*\(", header))
    assert {"tir_gemm", "tir_batch_matmul", "tir_conv2d", "tir_last_error"} <= declared
    L = B.lib()
    for name in sorted(declared):
        assert hasattr(L, name), f"libtir.so does not export {name}"
    assert declared == set(B.EXPORTS)
    assert B.tir_version() == "0.1"


GOOD = dict(M=64, N=64, K=64, a_rs=64, a_cs=1, b_rs=64, b_cs=1, c_rs=64, c_cs=1, in_dtype="f16", out_dtype="f32")
FAKE = 0x1000  # a non-null, 16-byte aligned "pointer"; never dereferenced because validation fails first


def _gemm(**over):
    a = dict(GOOD, **over)
    return B.tir_gemm_status(a.pop("A", FAKE), a.pop("Bp", FAKE), a.pop("C", FAKE), a["M"], a["N"], a["K"], a["a_rs"],
                             a["a_cs"], a["b_rs"], a["b_cs"], a["c_rs"], a["c_cs"], a["in_dtype"], a["out_dtype"])


@pytest.mark.parametrize("over,status", [
    (dict(M=-1), B.TIR_ERR_INVALID_ARG),
    (dict(K=-5), B.TIR_ERR_INVALID_ARG),
    (dict(a_rs=-64), B.TIR_ERR_INVALID_ARG),
    (dict(C=0), B.TIR_ERR_INVALID_ARG),
    (dict(A=0), B.TIR_ERR_INVALID_ARG),
    (dict(c_rs=0, c_cs=0), B.TIR_ERR_INVALID_ARG),
    (dict(in_dtype=7), B.TIR_ERR_INVALID_ARG),
    (dict(in_dtype="f16", out_dtype="i32"), B.TIR_ERR_UNSUPPORTED),
    (dict(in_dtype="i8", out_dtype="f32"), B.TIR_ERR_UNSUPPORTED),
    (dict(in_dtype="f32", out_dtype="f32"), B.TIR_ERR_UNSUPPORTED),
    (dict(in_dtype="bf16", out_dtype="f16"), B.TIR_ERR_UNSUPPORTED),
    (dict(M=2 ** 31), B.TIR_ERR_UNSUPPORTED),
    (dict(A=FAKE + 1), B.TIR_ERR_ALIGNMENT),
    (dict(C=FAKE + 2), B.TIR_ERR_ALIGNMENT),
])
def test_gemm_rejects_bad_arguments(over, status):
    assert _gemm(**over) == status
    assert B.last_error() != ""


def test_zero_sized_calls_are_noops_without_a_device():
    assert _gemm(M=0) == B.TIR_OK
    assert _gemm(N=0, A=0, Bp=0, C=0) == B.TIR_OK
    assert B.tir_batch_matmul_status(FAKE, FAKE, FAKE, 0, 8, 8, 8, 64, 8, 1, 64, 8, 1, 64, 8, 1, "f16", "f32") == B.TIR_OK
    assert B.tir_conv2d_status(FAKE, FAKE, FAKE, 0, 8, 8, 8, 8, 3, 3, 1, 1, 1, 1, 1, 1, 1, "f16", "f16") == B.TIR_OK


def test_bmm_rejects_overlapping_outputs():
    st = B.tir_batch_matmul_status(FAKE, FAKE, FAKE, 4, 8, 8, 8, 64, 8, 1, 64, 8, 1, 0, 8, 1, "f16", "f32")
    assert st == B.TIR_ERR_INVALID_ARG and "overlap" in B.last_error()


def _conv(**over):
    a = dict(N=1, H=8, W=8, C=8, K=8, R=3, S=3, sh=1, sw=1, ph=1, pw=1, dh=1, dw=1, g=1, i="f16", o="f16")
    a.update(over)
    return B.tir_conv2d_status(a.get("x", FAKE), a.get("w", FAKE), a.get("y", FAKE), a["N"], a["H"], a["W"], a["C"], a["K"],
                               a["R"], a["S"], a["sh"], a["sw"], a["ph"], a["pw"], a["dh"], a["dw"], a["g"], a["i"], a["o"])


@pytest.mark.parametrize("over,status", [
    (dict(g=3), B.TIR_ERR_INVALID_ARG),           # groups must divide C and K
    (dict(g=0), B.TIR_ERR_INVALID_ARG),
    (dict(C=8, K=12, g=8), B.TIR_ERR_INVALID_ARG),
    (dict(sh=0), B.TIR_ERR_INVALID_ARG),
    (dict(dw=0), B.TIR_ERR_INVALID_ARG),
    (dict(ph=-1), B.TIR_ERR_INVALID_ARG),
    (dict(H=2, W=2, ph=0, pw=0), B.TIR_ERR_INVALID_ARG),   # 3x3 filter does not fit: P <= 0
    (dict(H=0), B.TIR_ERR_INVALID_ARG),
    (dict(x=0), B.TIR_ERR_INVALID_ARG),
    (dict(H=20000), B.TIR_ERR_UNSUPPORTED),
    (dict(i="i8", o="f16"), B.TIR_ERR_UNSUPPORTED),
])
def test_conv_rejects_bad_arguments(over, status):
    assert _conv(**over) == status
    assert B.last_error() != ""


@pytest.mark.parametrize("tiles", [(1, 1), (16, 16), (7, 5), (3, 100), (49, 1), (2, 4), (13, 24), (196, 1)])
def test_block_to_tile_map_is_a_bijection(tiles):
    # the binding of block iterators to workgroup ids must cover every tile exactly once
    tm, tn = tiles
    seen = {B.tir_debug_tile_of_block(b, tm, tn) for b in range(tm * tn)}
    assert len(seen) == tm * tn
    assert all(0 <= a < tm and 0 <= b < tn for a, b in seen)


def test_division_by_launch_constants_is_exact():
    """The kernels decode output rows with multiply-and-shift constants; exact for every dividend below 2^31."""
    rng = np.random.default_rng(5)
    divisors = [1, 2, 3, 5, 7, 28, 49, 56, 784, 3136, 12544, 65535, 65536, 65537, 2**30 - 1, 2**30, 2**30 + 1, 2**31 - 1]
    divisors += [int(x) for x in rng.integers(1, 2**31, 40)]
    for d in divisors:
        edge = [0, 1, d - 1, d, d + 1, 2 * d - 1, 2 * d, 2**31 - 1, 2**31 - 2, (2**31 - 1) // d * d, (2**31 - 1) // d * d - 1]
        for m in edge + [int(x) for x in rng.integers(0, 2**31, 200)]:
            if 0 <= m < 2**31:
                assert B.tir_debug_fastdiv(d, m) == m // d, (d, m)


@pytest.mark.parametrize("dtype,out,n,p,q,c,pixels", [
    # us with four and with eight pixels per thread
    ("f16", "f16", 16, 56, 56, 128, 8),        # 8.1, 6.9
    ("f16", "f16", 4, 505, 4, 512, 4),         # 5.7, 7.2: half of a group of eight is padding
    ("f16", "f16", 9, 110, 11, 352, 4),        # 7.8, 8.1: a third more pixels
    ("f16", "f32", 16, 60, 14, 384, 4),        # 12.3, 12.8
    ("bf16", "bf16", 4, 480, 4, 384, 4),       # 6.0, 7.5
    ("bf16", "bf16", 8, 180, 9, 256, 8),       # 7.9, 7.8
    ("bf16", "f32", 4, 505, 9, 256, 4),        # 11.3, 12.4
    ("i8", "i8", 4, 137, 49, 384, 4),          # 13.1, 16.4
    ("i8", "i8", 16, 286, 4, 384, 4),          # 9.6, 13.8
    ("i8", "i8", 8, 245, 49, 128, 8),          # 16.8, 16.2
    ("i8", "i32", 2, 2880, 28, 64, 4),         # 33.3, 35.8
    ("f16", "f16", 32, 56, 56, 128, 4),        # more than one round of workgroups of eight
])
def test_depthwise_pixels_per_thread(dtype, out, n, p, q, c, pixels):
    """Eight pixels per thread only where the workgroups of four no longer run at once and those of eight do; padding counts."""
    assert B.tir_debug_depthwise_pixels(n, p, q, c, 1, dtype, out) == pixels
    assert B.tir_debug_depthwise_pixels(n, p, q, c, 2, dtype, out) == 4


@pytest.mark.parametrize("dtype,n,p,q,c,rows", [
    # us with one row of pixels per thread and with two
    ("bf16", 10, 72, 22, 208, 2),        # 8.4, 7.7
    ("bf16", 3, 110, 25, 448, 1),        # 5.7, 6.9: 511 workgroups of one row, 259 of two
    ("bf16", 29, 37, 9, 304, 1),         # 6.1, 7.0: 505, 260
    ("bf16", 27, 40, 62, 32, 2),         # 7.0, 6.7: 540, 270
    ("bf16", 14, 65, 69, 112, 1),        # 9.8, 12.2: 1024, 520
    ("bf16", 24, 18, 75, 208, 2),        # 13.0, 10.6: 1028, 516
    ("bf16", 8, 78, 105, 96, 2),         # 12.1, 10.2: 1054, 528
    ("bf16", 17, 45, 83, 224, 2),        # 19.9, 16.9: 2012, 1028
    ("f16", 20, 43, 11, 336, 2),         # 6.2, 5.7
    ("f16", 16, 56, 56, 128, 1),         # 7.85, 8.08
    ("f16", 32, 112, 112, 64, 2),        # 28.4, 26.1
])
def test_depthwise_rows_per_thread(dtype, n, p, q, c, rows):
    """Two rows of pixels per thread, except where one row's workgroups just fill the CUs and those of two begin another round."""
    assert B.tir_debug_depthwise_rows(n, p, q, c, dtype, dtype) == rows


@pytest.mark.parametrize("batch,m,n,d,out,kernel", [
    # us with this kernel and with another, the same operands again / three sets of operands in turn
    (512, 256, 256, 64, "bf16", "t128_sequential"),       # 15.7 / 16.1, in tiles of 256 15.7 / 18.7
    (512, 256, 256, 64, "f32", "t128_sequential"),        # 17.2 / 17.2, 17.6 / 21.1
    (256, 512, 320, 64, "f32", "t128_sequential"),        # 17.3 / 17.7, 18.3 / 18.6
    (256, 512, 768, 64, "bf16", "t256_sequential"),       # 32.2 / 33.0, in tiles of 128 33.5 / 33.9
    (800, 128, 600, 64, "bf16", "t128_sequential"),       # 31.9 / 33.2, pipelined 32.0 / 38.5
    (2000, 40, 64, 64, "bf16", "t128_sequential"),        # 11.0 / 12.6, 12.3 / 13.8
    (2000, 128, 160, 64, "bf16", "t128_sequential"),      # 27.1 / 27.3, in chunks of 32 25.1 / 31.7
    (500, 128, 1000, 64, "bf16", "t128_stream"),          # 28.8 / 30.1, plain 26.9 / 32.2
    (1024, 128, 400, 128, "bf16", "t128_stream"),         # 49.8 / 49.3, plain 44.9 / 58.8
    (200, 128, 2000, 128, "bf16", "t128"),                # 38.7 / 52.2, non-temporal 47.9 / 49.6
    (390, 256, 512, 128, "f32", "t128"),                  # 40.1 / 48.4, in tiles of 256 45.6 / 50.4
    (16, 4096, 4096, 128, "bf16", "t256"),
    (192, 128, 128, 64, "f16", "t128"),
])
def test_attention_kernel_of_measured_calls(batch, m, n, d, out, kernel):
    assert B.tir_debug_attention_kernel(batch, m, n, d, out) == kernel


def test_variant_choice_reflects_layout():
    # row-major B is read N-major, a transposed B K-major; odd K falls back to the general kernel
    assert B.tir_gemm_variant(1, 4096, 4096, 4096, 4096, 1, 4096, 1, 4096, 1, "f16", "f32").endswith("ak_bn")
    assert B.tir_gemm_variant(1, 4096, 4096, 4096, 4096, 1, 1, 4096, 4096, 1, "f16", "f32").endswith("ak_bk")
    assert B.tir_gemm_variant(1, 100, 100, 37, 37, 1, 100, 1, 100, 1, "f16", "f32").endswith("generic")
    assert "conv" in B.tir_conv2d_variant(16, 56, 56, 64, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, "f16", "f16")
    assert B.tir_conv2d_variant(1, 8, 8, 3, 8, 3, 3, 1, 1, 1, 1, 1, 1, 1, "f16", "f16").endswith("conv_generic")
    assert B.tir_gemm_variant(1, -1, 8, 8, 8, 1, 8, 1, 8, 1, "f16", "f32") == ""


@pytest.mark.parametrize("call,variant", [
    # the variant that was measured faster, us with it and with the one the score preferred
    (("gemm", 21, 32, 896, 64, "n", "bf16", "f32"), "t64x32w2x1s4_ak_bn"),                    # 3.91, 4.45 in 96x96 tiles
    (("gemm", 25, 704, 96, 64, "t", "i8", "i8"), "t256x32w4x1s3_ak_bk"),                      # 4.20, 4.56 in 96x96
    (("gemm", 63, 64, 272, 96, "t", "bf16", "f32"), "t96x96w3x1s4c4_ak_bk"),                  # 4.57, 5.66 in 64x32
    (("gemm", 49, 64, 928, 64, "n", "f16", "f32"), "t64x64w2x2s2_ak_bn"),                     # 5.51, 6.53 in 128x192
    (("gemm", 1, 576, 3040, 1024, "n", "f16", "f32"), "t128x64w2x2s4_ak_bn"),                 # 9.61, 10.25 with copy waves
    (("gemm", 84, 608, 656, 64, "t", "bf16", "f32"), "t256x256w2x4s2_ak_bk"),                 # 36.7, 43.2 in 64x64
    (("conv", 16, 106, 90, 128, 288, 3, 2, 1, 1, "bf16", "bf16"), "t256x96w4x1s3c4_conv"),    # 34.8, 45.3 in 128x96
    (("conv", 3, 18, 57, 464, 160, 5, 1, 2, 1, "f16", "f16"), "t128x32w4x1s3k2_conv/z2"),     # 34.8, 44.8 in one slice
    (("conv", 25, 14, 43, 96, 32, 5, 1, 1, 1, "f16", "f16"), "patch128x32w4x1r128_conv"),     # 10.1; 11.1 in 64x32 tiles of two reduction groups
    (("conv", 11, 70, 43, 256, 384, 5, 1, 1, 8, "i8", "i32"), "t128x64w2x2s3_conv"),          # 39.1, 44.8 with copy waves
    (("conv", 3, 70, 100, 672, 576, 1, 1, 1, 2, "i8", "i8"), "t256x96w4x1s3c4_conv"),        # three stages: 16.7, 20.5 in 128x64
    (("conv", 14, 11, 34, 896, 128, 5, 1, 1, 8, "f16", "f16"), "patch256x32w4x1r64_conv"),    # 14.6; 25.8 in 64x32
    (("conv", 4, 110, 86, 80, 32, 1, 1, 1, 1, "f16", "f16"), "t64x32w2x1s4_conv"),            # 4.94, 5.39 in 256x32
    (("tconv", 31, 7, 34, 64, 32, "bf16", "bf16"), "patch128x32w4x1r128_conv/ph2x2"),         # 4.2 - 4.5; 5.0 in 128x32
    # as many pixels, columns and products for the score as these three, strided or of one tap: the channel-block kernel does not take them
    (("conv", 25, 28, 86, 96, 32, 5, 2, 1, 1, "f16", "f16"), "t64x32w2x1s4k2_conv"),          # 11.2, 14.7 in two slices
    (("conv", 14, 22, 68, 896, 128, 5, 2, 1, 8, "f16", "f16"), "t64x32w2x1s4_conv"),          # 31.5, 39.8 in 256x32
    (("conv", 31, 7, 34, 1024, 128, 1, 1, 1, 4, "bf16", "bf16"), "t128x32w4x1s4_conv"),       # 5.40, 5.76 in two reduction groups
])
def test_variant_choice_of_measured_calls(call, variant):
    """One call per rule of the scoring that corrects a slower choice, and calls just beyond."""
    if call[0] == "gemm":
        _, batch, m, n, k, b, dtype, out = call
        name = B.tir_gemm_variant(batch, m, n, k, k, 1, *((1, k) if b == "t" else (n, 1)), n, 1, dtype, out)
    elif call[0] == "conv":
        _, n, h, w, c, k, r, stride, dil, groups, dtype, out = call
        pad = dil * (r - 1) // 2
        name = B.tir_conv2d_variant(n, h, w, c, k, r, r, stride, stride, pad, pad, dil, dil, groups, dtype, out)
    else:
        _, n, h, w, c, k, dtype, out = call
        name = B.tir_conv2d_transpose_variant(n, h, w, c, k, 4, 4, (2, 2), (1, 1), (1, 1), (0, 0), 1, dtype, out)
    assert name == f"{dtype}_{out}_{variant}"


@pytest.mark.parametrize("call,variant", [
    # us with this kernel and with the other one: the implicit GEMM or the patch kernel of 128-byte pixels, and the channel-block kernel
    (("tconv", 6, 33, 45, 192, 128, "f16", "f16"), "t256x128w4x2s3c4_conv/ph2x2"),                # 14.9, 18.4: 560 workgroups of blocks, two per CU
    (("tconv", 5, 48, 40, 96, 224, "f16", "f16"), "t256x256w2x4s4r64_convr/ph2x2"),               # 15.8, 19.5
    (("tconv", 17, 19, 29, 64, 224, "bf16", "bf16"), "t256x256w2x4s4r64_conv/ph2x2"),             # 12.9, 15.4
    (("conv", 29, 21, 39, 112, 144, 3, 1, 2, 1, "bf16", "f32"), "t128x192w2x2s3c4_conv"),         # 13.5, 18.3
    (("conv", 5, 40, 29, 256, 2048, 3, 1, 1, 8, "f16", "f16"), "t256x256w2x4s4r64_conv"),         # 13.8, 15.4
    (("conv", 7, 50, 49, 128, 224, 5, 1, 1, 2, "bf16", "bf16"), "t256x128w4x2s3c4_conv"),         # 20.5, 27.8
    (("conv", 1, 21, 109, 256, 3328, 3, 1, 2, 8, "i8", "i32"), "t256x256w2x4s4r64_conv"),         # 10.8, 14.2
    (("conv", 5, 96, 71, 16, 192, 3, 1, 1, 1, "i8", "i32"), "t256x256w2x4s3r64_conv"),            # 8.9, 11.0
    (("conv", 16, 56, 56, 64, 64, 3, 1, 1, 1, "f16", "f16"), "patch256x64_conv"),                 # 7.2, 7.4
    (("tconv", 16, 14, 14, 256, 128, "f16", "f16"), "patch128x64w2x2r128_conv/ph2x2"),            # 10.7, 8.6
    (("tconv", 31, 38, 15, 192, 128, "bf16", "bf16"), "patch256x64w4x1r64_conv/ph2x2"),           # 42.6, 27.2: 128x128 tiles of two stages, three rounds
    (("conv", 8, 28, 28, 256, 256, 3, 1, 2, 8, "i8", "i8"), "patch256x32w4x1r64_conv"),           # 5.6, 4.9
    (("conv", 7, 88, 42, 704, 512, 3, 1, 1, 4, "i8", "i8"), "patch256x64w4x1r64_conv"),           # 62.7, 35.6
    (("conv", 14, 88, 55, 64, 112, 5, 1, 2, 1, "f16", "f16"), "patch256x64w4x1r64_conv"),         # 66.0, 38.2
    (("conv", 3, 42, 48, 64, 16, 3, 1, 1, 1, "f16", "f16"), "patch64x64w2x2r128_conv"),           # 6.4, 4.4
    (("conv", 2, 57, 59, 896, 128, 5, 1, 1, 8, "bf16", "f32"), "patch256x32w4x1r64_conv"),        # 46.9, 15.7
    (("tconv", 29, 17, 54, 64, 32, "bf16", "bf16"), "patch256x32w4x1r64_conv/ph2x2"),             # 10.4, 7.1
    (("conv", 30, 43, 72, 160, 152, 2, 1, 1, 1, "bf16", "f32"), "t128x192w2x2s3c4_conv"),         # 39.8, 49.5: two by two taps, stores
    (("conv", 3, 69, 48, 16, 374, 2, 1, 1, 1, "bf16", "f32"), "t128x128w2x2s2_conv"),             # 6.5, 6.9
    (("conv", 38, 26, 18, 5120, 24, 2, 1, 1, 8, "i8", "i32"), "patch256x32w4x1r64_conv"),         # 39.5, 22.6
    (("conv", 14, 25, 230, 72, 24, 2, 1, 2, 3, "bf16", "bf16"), "patch256x32w4x1r64_conv"),       # 15.4, 10.1
    (("conv", 4, 66, 4, 512, 24, 2, 1, 1, 8, "bf16", "f32"), "patch64x64w2x2r128_conv"),          # 6.0, 3.7
])
def test_channel_block_choice_of_measured_calls(call, variant):
    """Stride-1 convolutions on both sides of the line between the channel-block kernel and the others."""
    test_variant_choice_of_measured_calls(call, variant)


def test_channel_block_plans_are_few():
    """Tiles of the channel-block kernel that cannot win are not planned: small convolutions are bound by the host, and there are six tiles in up to six strip widths."""
    def plan(n, h, w, c, k, r, dil, groups, dtype="f16"):
        pad = dil * (r - 1) // 2
        assert B.tir_conv2d_variant(n, h, w, c, k, r, r, 1, 1, pad, pad, dil, dil, groups, dtype, dtype)
        return B.tir_debug_block_plan()
    assert plan(16, 56, 56, 64, 64, 3, 1, 1) == (0, 0)                # the patch kernel's
    assert plan(1, 112, 112, 32, 32, 3, 1, 1) == (0, 0)
    assert plan(8, 28, 28, 256, 256, 3, 2, 8, "i8") == (1, 1)         # one strip of 28 columns 4.95 us, two 5.35
    rng = np.random.default_rng(11)
    planned = []
    for _ in range(400):
        n, h, w, r, groups = (int(v) for v in (rng.integers(1, 33), rng.integers(7, 113), rng.integers(7, 113), rng.choice([3, 5]), rng.choice([1, 1, 2, 4, 8])))
        planned.append(plan(n, h, w, int(rng.integers(1, 33)) * 16 * groups, int(rng.integers(1, 33)) * 16 * groups, r, int(rng.integers(1, 3)), groups)[0])
    assert np.mean(planned) < 6 and max(planned) <= 36, (np.mean(planned), max(planned))


R128, R64 = ["patch64x64w2x2r128", "patch128x64w2x2r128", "patch128x32w4x1r128"], ["patch128x64w2x2r64", "patch256x64w4x1r64", "patch256x32w4x1r64"]


@pytest.mark.parametrize("dtype,out", [("f16", "f16"), ("bf16", "f32"), ("i8", "i32")])
@pytest.mark.parametrize("kind,n,h,w,vecs,k,r,pad,dil,groups,tiles", [
    ("conv", 7, 5, 6, 9, 40, 3, (1, 1), (1, 1), 1, R128 + R64),
    ("conv", 2, 9, 150, 4, 24, 3, (1, 1), (1, 1), 2, R128 + R64),                          # 128-byte blocks in strips
    ("conv", 1, 9, 700, 12, 40, 3, (1, 1), (1, 1), 1, R64),                                # eight strips of 88 columns: 270 pixels of two buffers do not fit beside the filter
    ("conv", 1, 9, 2000, 12, 40, 3, (1, 1), (1, 1), 1, []),                                # too wide for the strips there are
    ("conv", 1, 40, 30, 12, 40, 3, (8, 8), (8, 8), 1, []),                                 # dilated rows: too many copy instructions per patch
    ("conv", 1, 12, 17, 8, 72, 5, (2, 2), (1, 1), 1, R128 + R64),                          # 5x5, one block
    ("conv", 1, 12, 17, 20, 72, 5, (2, 2), (1, 1), 1, R128[2:] + R64),                     # several: no room for the patch beside 120 KiB of filter
    ("conv", 1, 20, 20, 12, 40, 4, (1, 1), (1, 1), 1, []),                                 # sixteen taps are not compiled
    ("tconv", 1, 3, 300, 12, 40, 4, (1, 1), (1, 1), 1, R128 + R64),
    ("tconv", 2, 6, 9, 19, 42, 10, (4, 4), (1, 1), 1, R128[2:] + R64),                     # 5x5 taps per phase
    ("tconv", 2, 6, 9, 19, 42, 5, (2, 2), (1, 1), 1, []),                                  # phases of unequal taps
])
def test_channel_block_tiles_that_fit(dtype, out, kind, n, h, w, vecs, k, r, pad, dil, groups, tiles):
    """Which tiles of the channel-block kernel a problem can run in: forced by name, and from a tuning record; where none fits, the built-in choice stays another kernel."""
    c = vecs * (16 if dtype == "i8" else 8) * groups
    if kind == "conv":
        query = lambda: B.tir_conv2d_variant(n, h, w, c, k, r, r, 1, 1, *pad, *dil, groups, dtype, out)
    else:
        query = lambda: B.tir_conv2d_transpose_variant(n, h, w, c, k, r, r, (2, 2), pad, dil, (0, 0), groups, dtype, out)
    every = [f"{dtype}_{out}_{t}_conv" for t in R128 + R64]
    assert set(every) == {v for v in B.tir_debug_variant_names() if v.startswith(f"{dtype}_{out}_patch") and "patch256x64_conv" not in v}
    fit = set()
    try:
        for name in every:
            B.tir_debug_force_variant(name)
            if query().split("/")[0] == name:
                assert B.tir_debug_block_plan()[1] >= 1
                fit.add(name)
    finally:
        B.tir_debug_force_variant("")
    assert fit == {f"{dtype}_{out}_{t}_conv" for t in tiles}
    if not tiles:
        assert "w2x2r" not in query() and "w4x1r" not in query()


def _geometry_hash(fields):
    """FNV-1a over the 64-bit fields of a convolution's geometry, as tuning records store it."""
    h = 1469598103934665603
    for f in fields:
        for b in range(8):
            h = ((h ^ (f >> (8 * b) & 0xff)) * 1099511628211) % 2 ** 64
    return h


@pytest.mark.parametrize("n,h,w,c,k,r,stride,dil,fits", [
    (2, 20, 23, 96, 40, 3, 1, 1, True),
    (2, 20, 23, 96, 40, 3, 2, 1, False),        # strided
    (2, 20, 23, 96, 40, 1, 1, 1, False),        # one tap
    (2, 9, 700, 96, 40, 3, 1, 1, False),        # no strip of it fits LDS in this tile
    (2, 60, 60, 96, 40, 3, 1, 9, False),        # nor its dilated rows
])
def test_channel_block_record_is_taken_only_where_the_tile_fits(tmp_path, n, h, w, c, k, r, stride, dil, fits):
    name = "f16_f16_patch128x64w2x2r128_conv"
    pad = dil * (r - 1) // 2
    query = lambda: B.tir_conv2d_variant(n, h, w, c, k, r, r, stride, stride, pad, pad, dil, dil, 1, "f16", "f16")
    P, Q = ((x + 2 * pad - dil * (r - 1) - 1) // stride + 1 for x in (h, w))
    geom = _geometry_hash([n, 1, 1, h, w, 1, r, r, 1, stride, stride, 0, pad, pad, 1, dil, dil, 0, 0, 0, 0])
    B.tir_tune_clear()
    try:
        default = query()
        rec = tmp_path / "records.txt"
        lines = lambda v: f"tir-tune-records 1\n1 0 0 1 0 {n} {P * Q} {k} {r * r * c} {geom} {v} 1\n"
        other = "f16_f16_t128x128w2x2s2_conv"         # the record's signature is this call's
        assert default not in (name, other)
        rec.write_text(lines(other))
        B.tir_tune_load(rec)
        assert B.tir_tune_count() == 1 and query() == other
        B.tir_tune_clear()
        rec.write_text(lines(name))
        B.tir_tune_load(rec)
        assert B.tir_tune_count() == 1
        assert query() == (name if fits else default)
        B.tir_debug_force_variant("t64x64w2x2s3_conv")      # a forced variant wins over a record
        assert query() == "f16_f16_t64x64w2x2s3_conv"
    finally:
        B.tir_debug_force_variant("")
        B.tir_tune_clear()


def test_few_channels_take_the_row_kernel_where_it_pays():
    """Vectors of one tap that are not whole: filter rows as the unit of the reduction, unless the reduction is one
    stage in one round of workgroups and the patch (wide strides, many channels) takes longer to copy than the element-wise kernel takes
    altogether, or the layout rules it out."""
    def rows(c, k, r, stride, dil=1, groups=1, dtype="f16", n=2):
        return "rows256x" in B.tir_conv2d_variant(n, 97, 157, c, k, r, r, stride, stride, r // 2, r // 2, dil, dil, groups, dtype, dtype if dtype != "i8" else "i32")
    assert rows(3, 64, 7, 2) and rows(1, 16, 3, 1) and rows(4, 32, 3, 2, dtype="i8")
    assert rows(9, 64, 1, 3) and rows(28, 512, 1, 2) and rows(12, 64, 1, 2) and rows(3, 64, 2, 6) and rows(24, 64, 1, 3, dtype="i8")
    assert not rows(12, 256, 1, 3) and not rows(20, 256, 1, 3) and not rows(12, 64, 2, 3)
    assert rows(12, 64, 1, 3, n=64)
    assert not rows(3, 64, 3, 1, dil=2) and not rows(6, 12, 3, 1, groups=2) and not rows(40, 64, 3, 1)
    # operands of any alignment, by vectors along their contiguous axis
    assert "_uk_un_" in B.tir_gemm_variant(1, 1001, 1531, 777, 777, 1, 1531, 1, 1531, 1, "f16", "f16")
    assert "_um_uk_" in B.tir_gemm_variant(1, 1001, 1531, 777, 1, 1001, 1, 777, 1531, 1, "f16", "f16")


# ------------------------------------------------------------------------------ measured-choice records
def _gemm_variant_512():
    return B.tir_gemm_variant(1, 512, 512, 512, 512, 1, 512, 1, 512, 1, "f16", "f32")


def test_tuning_records_load_save_and_steer_the_choice(tmp_path):
    """A record file names the variant per problem signature: loading it changes what the planner
    picks for exactly that signature, saving writes it back, clearing restores the scoring rule.
    (Record lines: kind dt out amode bmode batch M N K geom variant; row-major f16 -> f32 GEMM is
    dt 0, out 3, A k-major 0, B n-major 1.)"""
    B.tir_tune_clear()
    try:
        default = _gemm_variant_512()
        other = "f16_f32_t64x32w2x1s4_ak_bn"
        assert default and default != other and other in B.tir_debug_variant_names()
        rec = tmp_path / "records.txt"
        rec.write_text("tir-tune-records 1\n"
                       f"0 0 3 0 1 1 512 512 512 0 {other}\n"
                       "0 0 3 0 1 1 640 512 512 0 no_such_variant\n"              # unknown name: skipped
                       "0 0 3 0 1 1 768 512 512 0 i8_i32_t64x64w2x2s2_ak_bn\n"    # wrong dtype for the key: skipped
                       "0 0 3 0 1 1 896 512 512 0 f16_f32_t64x64w2x2s2_ak_bk\n"   # wrong copy mode for the key: skipped
                       "garbage line\n")
        B.tir_tune_load(rec)
        assert B.tir_tune_count() == 1
        assert _gemm_variant_512() == other
        # another signature (batch 2) is untouched
        B.tir_debug_force_variant("")
        batch2 = B.tir_gemm_variant(2, 512, 512, 512, 512, 1, 512, 1, 512, 1, "f16", "f32")
        assert batch2 and batch2 != other
        # a forced variant wins over a record
        B.tir_debug_force_variant("t128x128w2x2s2_")
        assert "t128x128w2x2s2_" in _gemm_variant_512()
        B.tir_debug_force_variant("")
        # save / clear / load round trip
        out = tmp_path / "saved.txt"
        B.tir_tune_save(out)
        lines = out.read_text().splitlines()
        assert lines[0] == "tir-tune-records 1" and lines[1:] == [f"0 0 3 0 1 1 512 512 512 0 {other} 1"]   # last field: reduction slices
        B.tir_tune_clear()
        assert B.tir_tune_count() == 0 and _gemm_variant_512() == default
        B.tir_tune_load(out)
        assert _gemm_variant_512() == other
    finally:
        B.tir_debug_force_variant("")
        B.tir_tune_clear()


def test_reduction_split_is_planned_only_where_it_fits(tmp_path):
    """A reduction can be split over several workgroups per output tile ("<variant>/z<slices>"): only by the fast
    kernels, only when every slice gets a stage, and the scoring rule asks for it when few tiles face a long K."""
    def gemm(M, N, K, batch=1):
        return B.tir_gemm_variant(batch, M, N, K, K, 1, 1, K, N, 1, "f16", "f32")
    B.tir_tune_clear()
    try:
        assert "/z" not in gemm(4096, 4096, 4096)                     # the tiles fill the CUs: no split
        auto = gemm(128, 128, 16384)
        assert "/z" in auto and 2 <= int(auto.split("/z")[1]) <= 8    # 1-4 tiles, 256 stages
        B.tir_debug_force_ksplit(4)
        assert gemm(128, 128, 16384).endswith("/z4")
        assert gemm(4096, 4096, 4096).endswith("/z4") is False       # workspace: 256 tiles x 4 slices x 256 KiB > 32 MiB
        assert "/z" not in gemm(128, 128, 128)                        # two stages cannot feed four slices
        assert gemm(128, 128, 256).endswith("/z4")                    # four stages can
        assert "/z" not in gemm(100, 100, 4001)                       # odd K: the general kernel does not split
        assert "/z" not in B.tir_conv2d_variant(1, 8, 8, 3, 8, 3, 3, 1, 1, 1, 1, 1, 1, 1, "f16", "f16")
        conv = B.tir_conv2d_variant(2, 14, 14, 256, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, "f16", "f16")
        assert conv.endswith("/z4") and "patch" not in conv
        B.tir_debug_force_ksplit(0)
        # a record carries the split; one that does not fit its problem is planned without it
        name = "f16_f32_t64x64w2x2s3_ak_bk"
        assert name in B.tir_debug_variant_names()
        rec = tmp_path / "split.txt"
        rec.write_text("tir-tune-records 1\n"
                       f"0 0 3 0 0 1 128 128 16384 0 {name} 6\n"
                       f"0 0 3 0 0 1 128 128 128 0 {name} 6\n"
                       f"0 0 3 0 0 1 128 128 256 0 {name} 99\n")           # out of range: skipped
        B.tir_tune_load(rec)
        assert B.tir_tune_count() == 2
        assert gemm(128, 128, 16384) == name + "/z6"
        assert gemm(128, 128, 128) == name
        out = tmp_path / "saved.txt"
        B.tir_tune_save(out)
        assert f"0 0 3 0 0 1 128 128 16384 0 {name} 6" in out.read_text().splitlines()
    finally:
        B.tir_debug_force_ksplit(0)
        B.tir_tune_clear()


def test_output_policy_is_a_checked_field_of_the_epilogue():
    """The cache policy of a call's output stores travels in its epilogue: 0 or 1, anything else is rejected on the host."""
    def call(streaming):
        ep = B.Epilogue(None, 0, 0.0, streaming)
        return B.lib().tir_gemm_fused(FAKE, FAKE, FAKE, 64, 64, 64, 64, 1, 64, 1, 64, 1, B.TIR_F16, B.TIR_F32, ep, None)
    assert call(7) == B.TIR_ERR_INVALID_ARG and "streaming" in B.last_error()
    assert call(-1) == B.TIR_ERR_INVALID_ARG
    assert B.make_epilogue() is None and B.make_epilogue(streaming=True).streaming == 1
    assert not hasattr(B.lib(), "tir_set_output_policy")       # no process-wide policy


def test_split_static_rejects_what_its_scratch_cannot_hold():
    """tir_gemm_split_static checks slices, the copy mode and the size of its static scratch before any HIP call."""
    def call(M=128, N=128, K=4096, slices=4, a_rs=None, in_dtype="f16", out_dtype="f32"):
        return B.tir_gemm_split_static_status(FAKE, FAKE, FAKE, M, N, K, a_rs or K, 1, 1, K, N, 1, in_dtype, out_dtype, None, slices)
    assert call(slices=1) == B.TIR_ERR_INVALID_ARG and "slices" in B.last_error()
    assert call(slices=65) == B.TIR_ERR_INVALID_ARG
    assert call(K=0) == B.TIR_ERR_INVALID_ARG
    assert call(M=0) == B.TIR_OK                                              # nothing to do
    assert call(K=4001, a_rs=4001) == B.TIR_ERR_UNSUPPORTED and "general kernel" in B.last_error()
    assert call(K=128, slices=4) == B.TIR_ERR_INVALID_ARG and "non-empty slices" in B.last_error()     # two stages, four slices
    # 4096 x 4096 outputs: at least 1024 tiles of 128 x 128 x 4 slices x 64 KiB = 256 MiB of partial sums
    assert call(M=4096, N=4096, K=4096, slices=4) == B.TIR_ERR_INVALID_ARG
    msg = B.last_error()
    assert str(B.TIR_STATIC_SCRATCH_BYTES) in msg and str(B.TIR_STATIC_SCRATCH_TILES) in msg, msg
    assert call(in_dtype="f16", out_dtype="i32") == B.TIR_ERR_UNSUPPORTED
    header = (ROOT / "include" / "tir.h").read_text()
    assert "#define TIR_STATIC_SCRATCH_BYTES (8u << 20)" in header and "#define TIR_STATIC_SCRATCH_TILES 1024" in header
    assert (B.TIR_STATIC_SCRATCH_BYTES, B.TIR_STATIC_SCRATCH_TILES) == (8 << 20, 1024)


def test_caller_workspace_arguments_are_checked():
    """tir_set_workspace rejects a buffer that is too small or not 256-byte aligned before it touches the device."""
    need = B.tir_workspace_bytes()
    assert need == (32 << 20) + 16384 * 4
    assert B.tir_set_workspace_status(FAKE, need - 1) == B.TIR_ERR_INVALID_ARG
    assert "tir_workspace_bytes" in B.last_error()
    assert B.tir_set_workspace_status(FAKE + 16, need) == B.TIR_ERR_ALIGNMENT


def test_tuning_record_files_are_validated(tmp_path):
    bad = tmp_path / "bad.txt"
    bad.write_text("something else\n")
    with pytest.raises(B.TirError) as e:
        B.tir_tune_load(bad)
    assert e.value.status == B.TIR_ERR_INVALID_ARG
    with pytest.raises(B.TirError):
        B.tir_tune_load(tmp_path / "missing.txt")
    with pytest.raises(B.TirError):
        B.tir_tune_save(tmp_path / "no_such_dir" / "x.txt")
    assert B.tir_tune_count() == 0


def test_tuning_rejects_bad_arguments_before_touching_the_device():
    import ctypes
    L = B.lib()
    us = ctypes.c_double(-1.0)
    # reps out of range, then an invalid problem: status codes, no launch
    st = L.tir_tune_batch_matmul(FAKE, FAKE, FAKE, 1, 64, 64, 64, 0, 64, 1, 0, 64, 1, 0, 64, 1, 0, 3, None, 0, ctypes.byref(us), None)
    assert st == B.TIR_ERR_INVALID_ARG and "reps" in B.last_error()
    st = L.tir_tune_batch_matmul(FAKE, FAKE, FAKE, 1, -4, 64, 64, 0, 64, 1, 0, 64, 1, 0, 64, 1, 0, 3, None, 3, ctypes.byref(us), None)
    assert st == B.TIR_ERR_INVALID_ARG
    # zero-sized problems are a successful no-op
    st = L.tir_tune_batch_matmul(FAKE, FAKE, FAKE, 1, 0, 64, 64, 0, 64, 1, 0, 64, 1, 0, 64, 1, 0, 3, None, 3, ctypes.byref(us), None)
    assert st == B.TIR_OK and us.value == 0.0 and B.tir_tune_count() == 0


def test_fused_entry_points_validate_the_epilogue_on_the_host():
    """Epilogue errors are status codes before any launch: int8 output only through the fused entry
    points and only with a finite positive scale; the bias pointer must be 4-byte aligned."""
    import ctypes
    L = B.lib()
    def gemm_fused(out, ep):
        return L.tir_gemm_fused(FAKE, FAKE, FAKE, 64, 64, 64, 64, 1, 64, 1, 64, 1, B.TIR_I8, out,
                                None if ep is None else ctypes.byref(ep), None)
    assert gemm_fused(B.TIR_I8, None) == B.TIR_ERR_UNSUPPORTED
    assert gemm_fused(B.TIR_I8, B.Epilogue(None, 0, 0.0)) == B.TIR_ERR_INVALID_ARG
    assert gemm_fused(B.TIR_I8, B.Epilogue(None, 0, float("nan"))) == B.TIR_ERR_INVALID_ARG
    assert gemm_fused(B.TIR_I32, B.Epilogue(FAKE + 2, 0, 0.0)) == B.TIR_ERR_ALIGNMENT
    assert gemm_fused(B.TIR_F16, B.Epilogue(None, 1, 1.0)) == B.TIR_ERR_UNSUPPORTED        # (I8, F16) is no pair
    assert B.tir_gemm_status(FAKE, FAKE, FAKE, 64, 64, 64, 64, 1, 64, 1, 64, 1, "i8", B.TIR_I8) == B.TIR_ERR_UNSUPPORTED
    # zero-sized fused calls are no-ops as well
    assert L.tir_gemm_fused(FAKE, FAKE, FAKE, 0, 64, 64, 64, 1, 64, 1, 64, 1, B.TIR_I8, B.TIR_I8,
                            ctypes.byref(B.Epilogue(None, 1, 0.5)), None) == B.TIR_OK
    # the variant query knows the requantising kernels
    assert B.tir_gemm_variant(1, 512, 512, 512, 512, 1, 512, 1, 512, 1, "i8", B.TIR_I8).startswith("i8_i8_")


def test_attention_rejects_bad_arguments_on_the_host():
    def st(**kw):
        a = dict(Q=FAKE, K=FAKE, V=FAKE, O=FAKE, batch=1, M=128, N=128, d=64, scale=0.125, i="f16", o="f16")
        a.update(kw)
        return B.tir_attention_status(a["Q"], a["K"], a["V"], a["O"], a["batch"], a["M"], a["N"], a["d"], a["scale"], a["i"], a["o"])
    assert st(d=96) == B.TIR_ERR_UNSUPPORTED and "head dimension" in B.last_error()
    assert st(N=0) == B.TIR_ERR_INVALID_ARG
    assert st(M=-1) == B.TIR_ERR_INVALID_ARG
    assert st(scale=float("inf")) == B.TIR_ERR_INVALID_ARG
    assert st(i="i8", o="i32") == B.TIR_ERR_UNSUPPORTED
    assert st(i="bf16", o="f16") == B.TIR_ERR_UNSUPPORTED
    assert st(V=0) == B.TIR_ERR_INVALID_ARG
    assert st(O=FAKE + 8) == B.TIR_ERR_ALIGNMENT
    assert st(M=0) == B.TIR_OK and st(batch=0) == B.TIR_OK          # nothing to do: no launch, no device needed


def test_conv1d_conv3d_and_transposed_conv_validate_on_the_host():
    L = B.lib()
    def c1(**kw):
        a = dict(N=1, L=32, C=16, K=16, R=3, stride=1, pad=1, dil=1, groups=1)
        a.update(kw)
        return L.tir_conv1d(FAKE, FAKE, FAKE, a["N"], a["L"], a["C"], a["K"], a["R"], a["stride"], a["pad"], a["dil"], a["groups"],
                            B.TIR_F16, B.TIR_F32, None, None)
    assert c1(stride=0) == B.TIR_ERR_INVALID_ARG
    assert c1(groups=3) == B.TIR_ERR_INVALID_ARG
    assert c1(L=2, R=5, pad=0) == B.TIR_ERR_INVALID_ARG          # empty output
    assert c1(N=0) == B.TIR_OK

    def c3(**kw):
        a = dict(N=1, D=4, H=8, W=8, C=16, K=16, T=3, R=3, S=3, s=(1, 1, 1), p=(1, 1, 1), d=(1, 1, 1), groups=1)
        a.update(kw)
        return L.tir_conv3d(FAKE, FAKE, FAKE, a["N"], a["D"], a["H"], a["W"], a["C"], a["K"], a["T"], a["R"], a["S"], *a["s"], *a["p"], *a["d"],
                            a["groups"], B.TIR_F16, B.TIR_F16, None, None)
    assert c3(D=0) == B.TIR_ERR_INVALID_ARG
    assert c3(d=(0, 1, 1)) == B.TIR_ERR_INVALID_ARG
    assert c3(p=(-1, 0, 0)) == B.TIR_ERR_INVALID_ARG
    assert c3(D=2, T=5, p=(0, 1, 1)) == B.TIR_ERR_INVALID_ARG    # empty output along the depth
    assert c3(D=20000) == B.TIR_ERR_UNSUPPORTED
    assert c3(N=0) == B.TIR_OK

    def ct(**kw):
        a = dict(N=1, H=8, W=8, C=16, K=16, R=3, S=3, s=(2, 2), p=(1, 1), d=(1, 1), op=(1, 1), groups=1)
        a.update(kw)
        return L.tir_conv2d_transpose(FAKE, FAKE, FAKE, a["N"], a["H"], a["W"], a["C"], a["K"], a["R"], a["S"], *a["s"], *a["p"], *a["d"], *a["op"],
                                      a["groups"], B.TIR_I8, B.TIR_I32, None, None)
    assert ct(op=(-1, 0)) == B.TIR_ERR_INVALID_ARG
    assert ct(s=(0, 1)) == B.TIR_ERR_INVALID_ARG
    assert ct(H=1, W=1, R=1, S=1, p=(1, 1), op=(0, 0), s=(1, 1)) == B.TIR_ERR_INVALID_ARG   # extent (1-1)*1 - 2 + 0 + 0 + 1 < 1
    assert ct(K=15, groups=2) == B.TIR_ERR_INVALID_ARG
    assert ct(H=1, s=(20000, 1), op=(0, 0)) == B.TIR_ERR_UNSUPPORTED    # the kernels keep remainders modulo the stride in 16 bits
    assert ct(N=0) == B.TIR_OK
    # by output phase: only undilated, strided, whole 128-byte channel blocks; the queries report how a problem would run
    q = lambda C, s, d, dt="f16": B.tir_conv2d_transpose_variant(2, 8, 8, C, 32, 4, 4, s, (1, 1), d, (0, 0), 1, dt, dt if dt != "i8" else "i32")
    assert q(64, (2, 2), (1, 1)).endswith("_conv/ph2x2")
    assert q(128, (1, 3), (1, 1)).endswith("_conv/ph1x3")
    assert q(128, (2, 2), (1, 1), "i8").endswith("_conv/ph2x2") and "ph" not in q(64, (2, 2), (1, 1), "i8")
    assert "convx" in q(64, (2, 2), (2, 1)) and "convx" in q(32, (2, 2), (1, 1)) and "convx" in q(64, (1, 1), (1, 1))
    assert B.tir_conv3d_variant(1, 10, 16, 16, 128, 64, 3, 3, 3, (1, 1, 1), (1, 1, 1), (1, 1, 1), 1, "f16", "f16").endswith("_convx/z6")
    assert B.tir_conv3d_variant(1, 0, 16, 16, 128, 64, 3, 3, 3, (1, 1, 1), (1, 1, 1), (1, 1, 1), 1, "f16", "f16") == ""


def test_variant_table_is_what_its_generator_writes():
    """csrc/tir_variants.def is generated (gen_variants.py): the committed table and the tile list must not drift apart,
    and every name must be unique."""
    import importlib.util
    import re
    from pathlib import Path
    csrc = Path(__file__).resolve().parent.parent / "paper_2207_04296_amd" / "csrc"
    spec = importlib.util.spec_from_file_location("gen_variants", csrc / "gen_variants.py")
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    text = (csrc / "tir_variants.def").read_text()
    assert gen.render() == text, "run python paper_2207_04296_amd/csrc/gen_variants.py"
    names = re.findall(r'^V\d+\("([^"]+)"', text, flags=re.M)
    assert len(names) == len(set(names)) and len(names) > 600


@pytest.mark.parametrize("args,exc", [
    ((FAKE, FAKE, FAKE, 0, 8, 8, 8, 1, 8, 1, 8, 1, "f16", "f32", None, 0), None),                    # zero-sized: TIR_OK
    ((FAKE, FAKE, FAKE, 0, 8, 8, 8, 1, 8, 1, 8, 1, B.TIR_F16, B.TIR_F32, B.Epilogue(), 0), None),    # codes, an epilogue
    ((FAKE, FAKE, FAKE, 0, 8, 8, 8, 1, 8, 1, 8, 1, "f17", "f32", None, 0), KeyError),
    ((FAKE, "A", FAKE, 0, 8, 8, 8, 1, 8, 1, 8, 1, "f16", "f32", None, 0), AttributeError),
    ((FAKE, FAKE, FAKE, 0.5, 8, 8, 8, 1, 8, 1, 8, 1, "f16", "f32", None, 0), TypeError),
    ((FAKE, FAKE, FAKE, 0, 8, 8, 8, 1, 8, 1, 8, 1, "f16", "f32", 3, 0), TypeError),
    # anything with a buffer of the struct's size is no epilogue: its first bytes would be taken for the bias pointer
    ((FAKE, FAKE, FAKE, 0, 8, 8, 8, 1, 8, 1, 8, 1, "f16", "f32", np.zeros(8, np.float32), 0), TypeError),
    ((FAKE, FAKE, FAKE, 0, 8, 8, 8, 1, 8, 1, 8, 1, "f16", "f32", bytes(64), 0), TypeError),
    ((FAKE, FAKE, FAKE, 0, 8, 8, 8, 1, 8, 1, 8, 1, "f16", "f32", (ctypes.c_char * 64)(), 0), TypeError),
    ((FAKE, FAKE, FAKE, -1, 8, 8, 8, 1, 8, 1, 8, 1, "f16", "f32", None, 0), B.TirError),
])
def test_native_binding_converts_and_checks_its_arguments(args, exc):
    if exc is None:
        assert B.tir_gemm_fused(*args) is None
    else:
        with pytest.raises(exc):
            B.tir_gemm_fused(*args)

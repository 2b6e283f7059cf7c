"""Writes csrc/tir_variants.def from the tile table below.

Each fast-path tile is (BM, BN, WM, WN, ROWB, NSTAGE, KW[, CW]): BM x BN workgroup tile, WM x WN waves,
ROWB bytes of k per LDS row and stage, NSTAGE ring slots, KW reduction groups (KW sets of WM x WN
waves that split the stages of the reduction between them), CW extra waves that only copy (then the
multiplying waves issue no global->LDS loads).  Run after editing TILES:
    python paper_2207_04296_amd/csrc/gen_variants.py
"""
from pathlib import Path

TILES = [
    # large, MFMA-bound problems: one 8-wave workgroup per CU
    (256, 256, 2, 4, 128, 2, 1),
    # ... with 64-byte stages: the same 64 KB tile pair in a ring of three or four 32 KB slots instead of two 64 KB ones
    # (4096-cube GEMM 1095 -> 1160 TFLOP/s fp16 on one box, cold launches as fast as hot ones; three, four and five
    # slots measure alike, 4 x 2 waves 2 % slower than 2 x 4)
    (256, 256, 2, 4, 64, 3, 1),
    (256, 256, 2, 4, 64, 4, 1),
    # medium tiles: deeper rings hide the global latency that short K loops cannot
    (128, 128, 2, 2, 128, 2, 1),
    (128, 128, 2, 2, 128, 3, 1),
    (128, 128, 2, 2, 128, 4, 1),
    (256, 128, 4, 2, 128, 2, 1),
    (256, 128, 4, 2, 128, 3, 1),
    (128, 64, 2, 2, 128, 3, 1),
    (128, 64, 2, 2, 128, 4, 1),
    (256, 64, 4, 2, 128, 3, 1),
    (256, 64, 4, 1, 128, 3, 1),
    (64, 64, 2, 2, 128, 2, 1),
    (64, 64, 2, 2, 128, 3, 1),
    (64, 64, 2, 2, 128, 4, 1),
    (128, 32, 4, 1, 128, 3, 1),
    (128, 32, 4, 1, 128, 4, 1),
    (256, 32, 4, 1, 128, 3, 1),
    (64, 32, 2, 1, 128, 4, 1),
    # two reduction groups: small tiles of short-M problems, where one 4-wave workgroup per CU
    # cannot hide the copy latency (8 waves, twice the stages in flight)
    (64, 64, 2, 2, 128, 3, 2),
    (64, 64, 2, 2, 128, 4, 2),
    (128, 64, 2, 2, 128, 3, 2),
    (128, 128, 2, 2, 128, 2, 2),
    (128, 32, 4, 1, 128, 3, 2),
    (64, 32, 2, 1, 128, 4, 2),
    # 256-byte stages behind copy waves: half as many stages, barriers and copy set-ups for small tiles facing a
    # long reduction (the other tiles and the variants without copy waves gained nothing from them)
    (64, 64, 2, 2, 256, 3, 1, 4),
    (64, 64, 2, 2, 256, 4, 1, 4),
    # copy waves: four waves (one per SIMD) that only issue the global->LDS loads (measured: -8 .. -17 % on the
    # mid-size GEMMs; deeper rings than these, eight copy waves, smaller tiles and the general convolution decode
    # gained nothing)
    (64, 64, 2, 2, 128, 3, 1, 4),
    (64, 64, 2, 2, 128, 4, 1, 4),
    (128, 64, 2, 2, 128, 3, 1, 4),
    (128, 128, 2, 2, 128, 3, 1, 4),
    (128, 128, 2, 2, 128, 4, 1, 4),
    (256, 128, 4, 2, 128, 3, 1, 4),
    # three 32-column blocks per wave (64 x 96 wave tiles): 256 tiles for outputs such as 2048 x 3072, which 256 x 128
    # tiles cut into 192 (FFN GEMM 13.3 -> 12.3 - 12.5 us with warm caches, 16.4 -> 16.5 - 18.3 cold; a deeper ring and
    # two reduction groups over 64-byte stages measured slower)
    (256, 96, 4, 1, 128, 3, 1, 4),
    (128, 192, 2, 2, 128, 3, 1, 4),
    # one 96-column block row per wave: outputs whose extents are multiples of 96 or 192 rather than 128 or 256 (network widths of 768, 1152, 1536,
    # 2304 ...), which 128-wide tiles cut into a number that leaves CUs idle (the rule in pick() finds them by fill and padding).  us, before -> now:
    # 1536x1536x1024 fp16 9.2 -> 8.0 (144 tiles -> 256), 1152x1152x4096 A^T 32.3 -> 23.6, 1024x2304x768 8.3 -> 7.1, 700x1700x1024 7.85 -> 7.1;
    # nine waves of 32x32 are 5 - 10 % slower, and so are 96x128 tiles of six waves
    (96, 96, 3, 1, 128, 4, 1, 4),
    (128, 96, 4, 1, 128, 3, 1, 4),
]
PAIRS = [("DT_F16", "DT_F32", "f16_f32"), ("DT_F16", "DT_F16", "f16_f16"), ("DT_BF16", "DT_F32", "bf16_f32"),
         ("DT_BF16", "DT_BF16", "bf16_bf16"), ("DT_I8", "DT_I32", "i8_i32"), ("DT_I8", "DT_I8", "i8_i8")]
MODES = [("ak_bk", "A_KMAJOR", "B_KMAJOR"), ("ak_bn", "A_KMAJOR", "B_NMAJOR"), ("conv", "A_CONV", "B_KMAJOR")]
# the general convolution decode (3-D, transposed 2-D) is compiled for a few tiles only
CONVX_TILES = [(256, 128, 4, 2, 128, 3, 1), (128, 128, 2, 2, 128, 3, 1), (128, 64, 2, 2, 128, 3, 1), (64, 64, 2, 2, 128, 3, 1),
               (64, 64, 2, 2, 128, 3, 2), (128, 32, 4, 1, 128, 3, 1)]

# A transposed A (stored [k][x]: weight gradients, dW = X^T dY): the tiles the scoring rule reaches
AM_TILES = [(96, 96, 3, 1, 128, 4, 1, 4), (128, 96, 4, 1, 128, 3, 1, 4), (256, 256, 2, 4, 64, 3, 1), (256, 128, 4, 2, 128, 3, 1, 4), (128, 192, 2, 2, 128, 3, 1, 4), (128, 128, 2, 2, 128, 3, 1, 4),
            (128, 128, 2, 2, 128, 3, 1), (128, 64, 2, 2, 128, 3, 1), (64, 64, 2, 2, 128, 3, 1), (64, 64, 2, 2, 128, 4, 1),
            (64, 64, 2, 2, 128, 3, 2), (64, 32, 2, 1, 128, 4, 1)]
AM_MODES = [("am_bk", "A_MMAJOR", "B_KMAJOR"), ("am_bn", "A_MMAJOR", "B_NMAJOR")]

# by output phase with a ragged last stage per tap: the tiles the scoring rule reaches
RAGGED_TILES = [(256, 256, 2, 4, 64, 4, 1), (256, 128, 4, 2, 128, 3, 1, 4), (128, 192, 2, 2, 128, 3, 1, 4), (128, 128, 2, 2, 128, 4, 1, 4),
                (128, 64, 2, 2, 128, 4, 1), (64, 64, 2, 2, 128, 4, 1), (64, 64, 2, 2, 128, 4, 2), (128, 32, 4, 1, 128, 3, 2),
                (64, 32, 2, 1, 128, 4, 1), (64, 32, 2, 1, 128, 4, 2)]
RAGGED_MODES = [("convr", "A_CONV_RAGGED", "B_KMAJOR")]

# channel-block convolution: (BM, BN, WM, WN, ROWB), four copy waves; with all of them the best tile takes 0.87 of the implicit GEMM's time over 1276 calls, with
# 128x128, 256x32 and 256x64 of 128-byte blocks as well 0.1 % less
BLOCK_TILES = [(64, 64, 2, 2, 128), (128, 64, 2, 2, 128), (128, 64, 2, 2, 64), (256, 64, 4, 1, 64), (128, 32, 4, 1, 128), (256, 32, 4, 1, 64)]

# operands of any alignment, staged through registers (two stages ahead).  A name ending in _generic says that the variant takes operands
# of any alignment: these and the few-channel kernels by vectors, t64x64w2x2s2_generic and t64x64w2x2s2_conv_generic element by element.
U_TILES = [(128, 128, 2, 2, 128, 2, 1), (128, 128, 2, 4, 128, 2, 1), (128, 64, 4, 2, 128, 2, 1), (64, 64, 2, 2, 128, 2, 1), (64, 64, 2, 2, 128, 2, 2), (64, 32, 2, 1, 128, 2, 1), (64, 32, 2, 1, 128, 2, 4)]
U_MODES = [("uk_uk_generic", "A_UK", "B_UK"), ("uk_un_generic", "A_UK", "B_UN"), ("um_uk_generic", "A_UM", "B_UK"), ("um_un_generic", "A_UM", "B_UN")]


def render() -> str:
    """The text of tir_variants.def for the tables above."""
    out = ["// Generated by gen_variants.py - do not edit by hand.",
           "//   Vn(name, DT, OUT, BM, BN, WM, WN, AMODE, BMODE, ROWB, NSTAGE, KW, CW)   n = index of the translation unit that",
           "// instantiates the variant (tir_inst.hip is compiled once per unit with -DTIR_UNIT=n)."]
    for unit, (dt, od, tag) in enumerate(PAIRS):
        for tile, modes in [(t, MODES) for t in TILES] + [(t, AM_MODES) for t in AM_TILES] + [(t, RAGGED_MODES) for t in RAGGED_TILES] + [(t, U_MODES) for t in U_TILES]:
            (bm, bn, wm, wn, rowb, ns, kw), cw = tile[:7], (tile[7] if len(tile) > 7 else 0)
            for (mname, am, bmo) in modes:
                if bmo == "B_NMAJOR" and dt == "DT_I8" and bn * 1 < 32:
                    continue
                name = (f"{tag}_t{bm}x{bn}w{wm}x{wn}s{ns}" + (f"k{kw}" if kw > 1 else "") + (f"c{cw}" if cw else "") +
                        ("r64" if rowb == 64 else "r256" if rowb == 256 else "") + f"_{mname}")
                out.append(f'V{unit}("{name}", {dt}, {od}, {bm}, {bn}, {wm}, {wn}, {am}, {bmo}, {rowb}, {ns}, {kw}, {cw})')
        for tile in CONVX_TILES:
            (bm, bn, wm, wn, rowb, ns, kw), cw = tile[:7], (tile[7] if len(tile) > 7 else 0)
            name = f"{tag}_t{bm}x{bn}w{wm}x{wn}s{ns}" + (f"k{kw}" if kw > 1 else "") + (f"c{cw}" if cw else "") + ("r256" if rowb == 256 else "") + "_convx"
            out.append(f'V{unit}("{name}", {dt}, {od}, {bm}, {bn}, {wm}, {wn}, A_CONVX, B_KMAJOR, {rowb}, {ns}, {kw}, {cw})')
        out.append(f'V{unit}("{tag}_patch256x64_conv", {dt}, {od}, 256, 64, 4, 1, A_CONV_PATCH, B_KMAJOR, 128, 4, 1, 0)')
        for (bm, bn, wm, wn, rowb) in BLOCK_TILES:
            name = f"{tag}_patch{bm}x{bn}w{wm}x{wn}r{rowb}_conv"
            out.append(f'V{unit}("{name}", {dt}, {od}, {bm}, {bn}, {wm}, {wn}, A_CONV_BLOCKS, B_KMAJOR, {rowb}, 3, 1, 4)')
        for bn in (64, 32):
            out.append(f'V{unit}("{tag}_rows256x{bn}_conv_generic", {dt}, {od}, 256, {bn}, 4, 1, A_CONV_ROWS, B_GENERIC, 128, 2, 1, 0)')
        out.append(f'V{unit}("{tag}_t64x64w2x2s2_generic", {dt}, {od}, 64, 64, 2, 2, A_GENERIC, B_GENERIC, 128, 2, 1, 0)')
        out.append(f'V{unit}("{tag}_t64x64w2x2s2_conv_generic", {dt}, {od}, 64, 64, 2, 2, A_CONV_GENERIC, B_GENERIC, 128, 2, 1, 0)')
    return "\n".join(out) + "\n"


def main():
    text = render()
    Path(__file__).with_name("tir_variants.def").write_text(text)
    print(f"{len(text.splitlines()) - 3} variants")


if __name__ == "__main__":
    main()

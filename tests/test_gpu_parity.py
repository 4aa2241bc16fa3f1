"""GPU parity: the HIP library against the CPU oracle, element by element, through the C ABI.

Bars: scales, offsets, weight codes, activation codes and int32 accumulators bit-exact (the benchmark spec would
tolerate codes that differ where the fp32 product lies within 1 ulp of a rounding boundary: none do);
outputs within max|err| <= 1e-3 * max|ref|.
"""
import numpy as np
import pytest

from gen import Workload, get_workload, make_inputs
from oracle import stamp_oracle as so

import stamp_testlib as tl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2510_26771_amd as st
    st.load_library()  # fails loudly if the HIP library has not been built


def _wl(name, **kw):
    base = dict(name=name, batch=1, seq_len=256, d_in=256, d_out=256, xform="haar1d", levels=8, k_hi=8,
                x_dtype="bf16", rho=0.9, n_outlier_channels=3, outlier_scale=30.0, w_std=0.02, seed=11)
    base.update(kw)
    return Workload(**base)


def test_cfg1_small_config_all_steps():
    r = tl.full_case(get_workload("cfg1"))
    assert r["code_mismatches"] == 0


SMALL = [
    # several M tiles, ragged N (two N tiles, the second mostly masked), K tail (160 -> 256)
    _wl("r32_ragged", batch=3, seq_len=512, levels=9, k_hi=16, d_in=160, d_out=300, seed=21),
    # M = 192 < one tile; blocks of 8 tokens
    _wl("r8_small_m", batch=3, seq_len=64, levels=6, k_hi=8, d_in=96, d_out=64, seed=22),
    _wl("r16", batch=2, seq_len=256, levels=8, k_hi=16, d_in=320, d_out=257, seed=23, first_token_scale=100.0),
    _wl("r64_f32in", batch=2, seq_len=512, levels=9, k_hi=8, d_in=1024, d_out=512, x_dtype="f32", seed=24),
    # blocks of 128 tokens: only the unfused inverse applies
    _wl("r128", batch=1, seq_len=1024, levels=10, k_hi=8, d_in=128, d_out=256, seed=25),
    # k = 1: a single block sum is the only 8-bit token
    _wl("k1", batch=2, seq_len=64, levels=6, k_hi=1, d_in=64, d_out=96, seed=26),
    # 2-D grids: 4x4 and 8x8 token blocks
    _wl("g16_blk4", batch=2, seq_len=256, xform="haar2d", levels=4, grid_h=16, grid_w=16, k_hi=16, d_in=96, d_out=130,
        corr_len=4.0, seed=27),
    _wl("g32_blk8", batch=1, seq_len=1024, xform="haar2d", levels=5, grid_h=32, grid_w=32, k_hi=16, d_in=288,
        d_out=512, corr_len=8.0, seed=28),
    _wl("g8_blk4", batch=3, seq_len=64, xform="haar2d", levels=3, grid_h=8, grid_w=8, k_hi=4, d_in=64, d_out=40,
        corr_len=2.0, seed=29),
]


@pytest.mark.parametrize("w", SMALL, ids=[w.name for w in SMALL])
def test_small_cases(w):
    r = tl.full_case(w, with_bias=True)
    assert r["code_mismatches"] == 0


# The asymmetric (min-max, Eq. 1 in full) form of the quantizer, on shifted activations so that the token
# ranges are skewed and one-sided tokens occur: 1-D with several block sizes (fused and unfused inverse,
# ragged shapes), fp32 input, both 2-D block sizes.
ASYM = [
    _wl("asym_r32_ragged", batch=3, seq_len=512, levels=9, k_hi=16, d_in=160, d_out=300, seed=41, act_quant="asym",
        mean_shift=0.75),
    _wl("asym_r8", batch=3, seq_len=64, levels=6, k_hi=8, d_in=96, d_out=64, seed=42, act_quant="asym", mean_shift=-2.0),
    _wl("asym_r64_f32in", batch=2, seq_len=512, levels=9, k_hi=8, d_in=1024, d_out=512, x_dtype="f32", seed=43,
        act_quant="asym", mean_shift=0.3, first_token_scale=50.0),
    _wl("asym_r128", batch=1, seq_len=1024, levels=10, k_hi=8, d_in=128, d_out=256, seed=44, act_quant="asym"),
    _wl("asym_g16_blk4", batch=2, seq_len=256, xform="haar2d", levels=4, grid_h=16, grid_w=16, k_hi=16, d_in=96,
        d_out=130, corr_len=4.0, seed=45, act_quant="asym", mean_shift=1.0),
    _wl("asym_g32_blk8", batch=1, seq_len=1024, xform="haar2d", levels=5, grid_h=32, grid_w=32, k_hi=16, d_in=288,
        d_out=512, corr_len=8.0, seed=46, act_quant="asym", mean_shift=-0.5),
]


@pytest.mark.parametrize("w", ASYM, ids=[w.name for w in ASYM])
def test_asymmetric_quantizer_cases(w):
    r = tl.full_case(w, with_bias=True)
    assert r["code_mismatches"] == 0


def test_asymmetric_bf16_output():
    tl.full_case(_wl("asym_bf16_out", batch=2, seq_len=256, levels=8, k_hi=8, d_in=256, d_out=384, seed=47,
                     act_quant="asym", mean_shift=0.5), with_bias=True, y_dtype="bf16")


# Partial depth: J levels with log2(block size) <= J < full depth; the 8-bit tokens are then the level-J
# approximations followed by the details of the levels above the blocks (J = 3 on a 64 x 64 grid with 64
# 8-bit tokens is the paper's own image-model setting: the 8-bit tokens are the whole low-low band).
PARTIAL = [
    _wl("part_r8_L0", batch=2, seq_len=512, levels=3, k_hi=64, d_in=128, d_out=192, seed=51),
    _wl("part_r32_L2", batch=2, seq_len=512, levels=7, k_hi=16, d_in=160, d_out=300, seed=52),
    _wl("part_r64_L1_asym", batch=1, seq_len=1024, levels=7, k_hi=16, d_in=256, d_out=256, seed=53, act_quant="asym",
        mean_shift=0.4),
    _wl("part_g16_blk4_L0", batch=2, seq_len=256, xform="haar2d", levels=2, grid_h=16, grid_w=16, k_hi=16, d_in=96,
        d_out=130, corr_len=4.0, seed=54),
    _wl("part_g32_blk4_L2", batch=1, seq_len=1024, xform="haar2d", levels=4, grid_h=32, grid_w=32, k_hi=64, d_in=96,
        d_out=128, corr_len=6.0, seed=55),
    _wl("part_g32_blk8_L1", batch=1, seq_len=1024, xform="haar2d", levels=4, grid_h=32, grid_w=32, k_hi=16, d_in=288,
        d_out=512, corr_len=8.0, seed=56),
]


# Fewer 8-bit tokens than the transform leaves approximations (the paper's language-model setting: 3 levels,
# 64 8-bit tokens, so of the s / 8 approximations only the first 64 are 8-bit): the blocks are the 2^J (4^J) tokens
# of one approximation, and the 4-bit approximations travel with the 8-bit rows.  k_hi need not be a power of two.
FEWER_HI = [
    _wl("few_1d_J3_k8", batch=2, seq_len=512, levels=3, k_hi=8, d_in=128, d_out=192, seed=57),
    _wl("few_1d_J4_k5_asym", batch=2, seq_len=1024, levels=4, k_hi=5, d_in=160, d_out=300, seed=58, act_quant="asym",
        mean_shift=0.4),
    _wl("few_1d_J5_k0", batch=1, seq_len=2048, levels=5, k_hi=0, d_in=96, d_out=130, seed=59),
    _wl("few_2d_J2_k16", batch=1, seq_len=1024, xform="haar2d", levels=2, grid_h=32, grid_w=32, k_hi=16, d_in=96,
        d_out=128, corr_len=6.0, seed=60),
    _wl("few_2d_J3_k3_asym", batch=2, seq_len=4096, xform="haar2d", levels=3, grid_h=64, grid_w=64, k_hi=3, d_in=64,
        d_out=72, corr_len=8.0, seed=66, act_quant="asym", mean_shift=-0.5),
    # more 8-bit rows over the batch than the few-rows kernel takes, and more than one tile of them
    _wl("few_1d_J3_k70_b3", batch=3, seq_len=1024, levels=3, k_hi=70, d_in=192, d_out=264, seed=67),
    _wl("few_1d_J4_k100_b4_asym", batch=4, seq_len=2048, levels=4, k_hi=100, d_in=128, d_out=136, seed=68,
        act_quant="asym", mean_shift=0.3),
    # more than 256 approximations (3 levels on 4096 / 8192 tokens, 2 levels on a 128 x 128 grid)
    _wl("few_1d_J3_512top", batch=2, seq_len=4096, levels=3, k_hi=64, d_in=128, d_out=192, seed=77),
    _wl("few_1d_J3_1024top_asym", batch=1, seq_len=8192, levels=3, k_hi=64, d_in=96, d_out=130, seed=78,
        act_quant="asym", mean_shift=0.4, x_dtype="f32"),
    _wl("few_1d_J3_512top_k0", batch=3, seq_len=4096, levels=3, k_hi=0, d_in=64, d_out=72, seed=79),
    _wl("few_2d_J2_1024top", batch=1, seq_len=16384, xform="haar2d", levels=2, grid_h=128, grid_w=128, k_hi=64,
        d_in=64, d_out=72, corr_len=8.0, seed=80),
    _wl("few_1d_J3_512top_wide", batch=1, seq_len=4096, levels=3, k_hi=64, d_in=11008, d_out=64, seed=81),
    _wl("few_2d_J2_1024top_wide_asym", batch=1, seq_len=16384, xform="haar2d", levels=2, grid_h=128, grid_w=128,
        k_hi=5, d_in=4128, d_out=40, corr_len=8.0, seed=82, act_quant="asym", mean_shift=0.2),
    # channels split over workgroups: the top rows are quantized by the separate kernel
    _wl("few_1d_J3_k9_wide", batch=2, seq_len=256, levels=3, k_hi=9, d_in=4128, d_out=64, seed=69, x_dtype="f32"),
    _wl("few_2d_J2_k7_wide_asym", batch=1, seq_len=256, xform="haar2d", levels=2, grid_h=16, grid_w=16, k_hi=7,
        d_in=4128, d_out=72, corr_len=4.0, seed=70, act_quant="asym", mean_shift=0.2),
]
PARTIAL = PARTIAL + FEWER_HI


@pytest.mark.parametrize("w", PARTIAL, ids=[w.name for w in PARTIAL])
def test_partial_depth_cases(w):
    r = tl.full_case(w, with_bias=True)
    assert r["code_mismatches"] == 0


# Many 8-bit rows against a wide layer: the 8-bit rows' GEMM keeps its depth in one piece (tiled kernel, 256 x 128 or
# 256 x 256 tiles) and runs the top levels of the inverse in its own epilogue (the tile holds whole sequences: 1 to 16
# of them, the last tile only partly filled), writing the block sums directly.
TOP_IN_GEMM = [
    _wl("topfused_1d_k64_b3", batch=3, seq_len=512, levels=9, k_hi=64, d_in=64, d_out=16640, seed=71),
    _wl("topfused_1d_k64_b5_wide_asym", batch=5, seq_len=512, levels=9, k_hi=64, d_in=32, d_out=16650, seed=72,
        act_quant="asym", mean_shift=0.4),
    _wl("topfused_2d_k16_b9", batch=9, seq_len=256, xform="haar2d", levels=4, grid_h=16, grid_w=16, k_hi=16, d_in=32,
        d_out=33000, corr_len=4.0, seed=73),
    _wl("topfused_1d_k256", batch=1, seq_len=2048, levels=11, k_hi=256, d_in=32, d_out=16640, seed=74),
    _wl("topfused_1d_k16_L2_b10", batch=10, seq_len=512, levels=7, k_hi=16, d_in=32, d_out=16640, seed=75),
    _wl("topfused_2d_k4_b40", batch=40, seq_len=64, xform="haar2d", levels=3, grid_h=8, grid_w=8, k_hi=4, d_in=32,
        d_out=16640, corr_len=2.0, seed=83),
    _wl("topfused_1d_k2_b70", batch=70, seq_len=16, levels=4, k_hi=2, d_in=32, d_out=16640, seed=84),
    _wl("topfused_2d_k64_L1_b3_asym", batch=3, seq_len=1024, xform="haar2d", levels=3, grid_h=32, grid_w=32, k_hi=64,
        d_in=32, d_out=16640, corr_len=6.0, seed=76, act_quant="asym", mean_shift=-0.3),
]


@pytest.mark.parametrize("w", TOP_IN_GEMM, ids=[w.name for w in TOP_IN_GEMM])
def test_top_levels_inverted_in_the_8bit_rows_gemm(w):
    r = tl.full_case(w, with_bias=True, hi_rows=1, routes=("hi_top_fused",))
    assert r["code_mismatches"] == 0


@pytest.mark.parametrize("w", TOP_IN_GEMM, ids=[w.name for w in TOP_IN_GEMM])
def test_top_levels_inverted_by_the_kernel_of_the_rule(w):
    """The same plans through whichever kernel the library takes for so little depth."""
    r = tl.full_case(w, with_bias=True, check_acc=False, check_unfused=False)
    assert r["code_mismatches"] == 0


# 8-bit rows on the int8 pipeline with their depth in several parts (few tiles), and the kernel that adds the parts in each
# kind of plan: top levels of the inverse, block sums alone, the first k_hi rows only, no transform.  More than 128 rows (up
# to four parts of two K steps or more) and fewer (parts of four), both quantizer forms.
SPLIT = [
    _wl("split_top_1d_k64", batch=3, seq_len=512, levels=9, k_hi=64, d_in=1024, d_out=192, seed=171),
    _wl("split_top_1d_k16_asym", batch=2, seq_len=256, levels=8, k_hi=16, d_in=1056, d_out=130, seed=172, act_quant="asym",
        mean_shift=0.4),
    _wl("split_top_2d_k16_b9_asym", batch=9, seq_len=256, xform="haar2d", levels=4, grid_h=16, grid_w=16, k_hi=16, d_in=544,
        d_out=200, corr_len=4.0, seed=173, act_quant="asym", mean_shift=-0.3),
    _wl("split_sums_1d_J3", batch=3, seq_len=512, levels=3, k_hi=64, d_in=1024, d_out=136, seed=174),
    _wl("split_sums_2d_J2", batch=1, seq_len=1024, xform="haar2d", levels=2, grid_h=32, grid_w=32, k_hi=64, d_in=1088,
        d_out=72, corr_len=6.0, seed=175),
    _wl("split_own_1d_J3_k70_asym", batch=2, seq_len=1024, levels=3, k_hi=70, d_in=576, d_out=264, seed=176, act_quant="asym",
        mean_shift=0.3),
    _wl("split_own_2d_J2_k9", batch=3, seq_len=256, xform="haar2d", levels=2, grid_h=16, grid_w=16, k_hi=9, d_in=2080,
        d_out=66, corr_len=4.0, seed=177),
    _wl("split_ident_k80_asym", xform="identity", levels=0, batch=2, seq_len=200, k_hi=80, d_in=1024, d_out=257, seed=178,
        act_quant="asym", mean_shift=0.6),
    _wl("split_ident_k9", xform="identity", levels=0, batch=2, seq_len=33, k_hi=9, d_in=1024, d_out=64, seed=179),
]


@pytest.mark.parametrize("w", SPLIT, ids=[w.name for w in SPLIT])
def test_8bit_rows_in_several_parts_of_the_depth(w):
    r = tl.full_case(w, with_bias=True, hi_rows=1, routes=("hi_split",), check_unfused=w.xform != "identity")
    assert r["code_mismatches"] == 0


# the same in one piece (a depth too short to split) where the rows' way out is a kernel of its own
WHOLE = [_wl("whole_ident_k80", xform="identity", levels=0, batch=2, seq_len=200, k_hi=80, d_in=160, d_out=257, seed=180),
         _wl("whole_own_J3_k70", batch=2, seq_len=1024, levels=3, k_hi=70, d_in=160, d_out=264, seed=181),
         _wl("whole_top_k16", batch=2, seq_len=256, levels=8, k_hi=16, d_in=160, d_out=130, seed=182)]


@pytest.mark.parametrize("w", WHOLE, ids=[w.name for w in WHOLE])
def test_8bit_rows_on_the_int8_pipeline_in_one_piece(w):
    r = tl.full_case(w, with_bias=True, hi_rows=1, routes=("-hi_split", "-hi_fp6", "-hi_top_fused"),
                     check_unfused=w.xform != "identity")
    assert r["code_mismatches"] == 0


# Layers wider than one workgroup of the transform kernel holds (8192 bf16 channels in 1-D, 4096 for fp32
# input and in 2-D): the channels are split over workgroups and the kernel runs twice (row maxima, then
# codes).  Shapes of real layers: an LLM down-projection (d_in 11008 / 14336), the second MLP layer of an
# image transformer on an 8 x 8-blocked grid (d_in 4608); ragged splits; both quantizer forms.
WIDE = [
    _wl("wide_1d_11008", batch=1, seq_len=256, levels=8, k_hi=8, d_in=11008, d_out=192, seed=61,
        n_outlier_channels=30, outlier_scale=40.0),
    _wl("wide_1d_14336_asym", batch=2, seq_len=128, levels=7, k_hi=16, d_in=14336, d_out=130, seed=62, act_quant="asym",
        mean_shift=0.5, n_outlier_channels=40),
    _wl("wide_1d_f32in_4128", batch=1, seq_len=256, levels=8, k_hi=4, d_in=4128, d_out=128, x_dtype="f32", seed=63),
    _wl("wide_2d_4608", batch=1, seq_len=256, xform="haar2d", levels=4, grid_h=16, grid_w=16, k_hi=4, d_in=4608,
        d_out=160, corr_len=4.0, seed=64, n_outlier_channels=12),
    _wl("wide_2d_blk4_8224_asym", batch=1, seq_len=64, xform="haar2d", levels=3, grid_h=8, grid_w=8, k_hi=4, d_in=8224,
        d_out=64, corr_len=2.0, seed=65, act_quant="asym", mean_shift=-0.3),
    # channel splits on plans WITHOUT top levels (the paper's 3-level settings on wide layers): two-pass bottom
    # kernel, then the top kernel with nothing to transform, fewer 8-bit tokens than approximations
    _wl("wide_1d_11008_J3_few", batch=1, seq_len=512, levels=3, k_hi=8, d_in=11008, d_out=136, seed=67,
        n_outlier_channels=30, outlier_scale=40.0),
    _wl("wide_2d_4608_J2_few_asym", batch=1, seq_len=256, xform="haar2d", levels=2, grid_h=16, grid_w=16, k_hi=3,
        d_in=4608, d_out=96, corr_len=4.0, seed=68, act_quant="asym", mean_shift=0.6),
]


@pytest.mark.parametrize("w", WIDE, ids=[w.name for w in WIDE])
def test_wide_layers_channel_split(w):
    r = tl.full_case(w, with_bias=True)
    assert r["code_mismatches"] == 0


# Deep layers (d_in >= 3072: at least 24 K steps of the GEMM, the operand ring wraps many times within a tile) at small
# M and N: every block length of the fused inverse (8 .. 64 tokens), both quantizer forms, both output types, tiles
# with rows and columns beyond the matrix, an odd number of K steps.
DEEP = [
    _wl("deep_r64", batch=2, seq_len=256, levels=8, k_hi=4, d_in=3072, d_out=130, seed=131),
    _wl("deep_r32_asym", batch=1, seq_len=256, levels=8, k_hi=8, d_in=3200, d_out=264, seed=132, act_quant="asym",
        mean_shift=0.4),
    _wl("deep_r16", batch=3, seq_len=256, levels=8, k_hi=16, d_in=3136, d_out=72, seed=133, first_token_scale=100.0),
    _wl("deep_r8_J3_few_asym", batch=1, seq_len=512, levels=3, k_hi=8, d_in=4096, d_out=200, seed=134, act_quant="asym",
        mean_shift=-0.5, n_outlier_channels=20),
    _wl("deep_small_m", batch=1, seq_len=64, levels=6, k_hi=1, d_in=3072, d_out=64, seed=135),
    _wl("deep_r8_f32in", batch=2, seq_len=128, levels=7, k_hi=16, d_in=3104, d_out=300, x_dtype="f32", seed=136),
    _wl("deep_r32_odd_steps", batch=2, seq_len=512, levels=9, k_hi=16, d_in=3328, d_out=96, seed=137),
    # the widest layer the library takes (256 K steps; the exactness argument of the FP6 engine is stated for this depth)
    _wl("deep_max_width", batch=1, seq_len=64, levels=6, k_hi=8, d_in=32768, d_out=72, seed=138, n_outlier_channels=60,
        outlier_scale=40.0),
    _wl("deep_max_width_asym_f32in", batch=1, seq_len=128, levels=7, k_hi=4, d_in=32768, d_out=40, x_dtype="f32", seed=139,
        act_quant="asym", mean_shift=0.3),
]


@pytest.mark.parametrize("y_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("w", DEEP, ids=[w.name for w in DEEP])
def test_deep_layers(w, y_dtype):
    r = tl.full_case(w, with_bias=True, y_dtype=y_dtype)
    assert r["code_mismatches"] == 0


# Plans without a sequence transform: the layers the paper leaves un-transformed and the baseline the
# transform's cost is measured against.  Per-token quantization of X itself, tokens 0..k-1 at 8 bits (k any
# number, none included), ragged shapes, both quantizer forms, both engines, bf16 and fp32 output.
IDENT = [
    _wl("ident_k8", xform="identity", levels=0, batch=3, seq_len=200, k_hi=8, d_in=160, d_out=300, seed=71),
    _wl("ident_k0", xform="identity", levels=0, batch=2, seq_len=256, k_hi=0, d_in=256, d_out=130, seed=72),
    _wl("ident_k5_asym", xform="identity", levels=0, batch=2, seq_len=333, k_hi=5, d_in=96, d_out=257, seed=73,
        act_quant="asym", mean_shift=0.6),
    _wl("ident_f32in_wide", xform="identity", levels=0, batch=1, seq_len=128, k_hi=64, d_in=8800, d_out=64, x_dtype="f32",
        seed=74, first_token_scale=100.0),
    # every token at 8 bits (k = s): the 4-bit rows' GEMM has nothing to do
    _wl("ident_all_8bit", xform="identity", levels=0, batch=3, seq_len=96, k_hi=96, d_in=128, d_out=200, seed=75),
    _wl("ident_all_8bit_asym", xform="identity", levels=0, batch=1, seq_len=256, k_hi=256, d_in=64, d_out=64, seed=76,
        act_quant="asym", mean_shift=0.2),
]


@pytest.mark.parametrize("w", IDENT, ids=[w.name for w in IDENT])
def test_identity_transform_cases(w):
    r = tl.full_case(w, with_bias=True, check_unfused=False)
    assert r["code_mismatches"] == 0
    tl.full_case(w, with_bias=True, check_unfused=False, y_dtype="bf16", check_acc=False)


def test_many_rows_few_channels():
    """2^18 token rows (1024 row tiles, several rounds of workgroups on every XCD), narrow layer: the tile numbering,
    the row-indexed buffers and the 64-bit offsets at a row count 8 times the benchmark's."""
    w = _wl("many_rows", batch=32, seq_len=8192, levels=13, k_hi=128, d_in=64, d_out=96, seed=91)
    r = tl.full_case(w, with_bias=True, y_dtype="bf16", check_unfused=False)
    assert r["code_mismatches"] == 0


def _random_workload(seed: int) -> Workload:
    """A valid plan drawn from the whole supported set (shape, transform, depth, quantizer form)."""
    rng = np.random.default_rng(1000 + seed)
    kind = rng.choice(["haar1d", "haar2d", "identity"], p=[0.5, 0.35, 0.15])
    d_in = int(rng.integers(1, 25)) * 32
    d_out = int(rng.integers(1, 520))
    batch = int(rng.integers(1, 4))
    kw = dict(batch=batch, d_in=d_in, d_out=d_out, seed=2000 + seed, x_dtype=str(rng.choice(["bf16", "f32"])),
              act_quant=str(rng.choice(["sym", "asym"])), mean_shift=float(rng.choice([0.0, 0.5, -1.0])),
              n_outlier_channels=int(rng.integers(0, 4)), outlier_scale=25.0)
    if kind == "haar1d":
        r = int(rng.integers(3, 8))               # block of 8..128 tokens
        lk = int(rng.integers(0, 5))              # 1..16 8-bit tokens
        s = (1 << r) << lk
        if rng.random() < 0.3:                    # fewer 8-bit tokens than approximations: blocks = 2^J tokens
            return _wl(f"rnd{seed}_1d_J{r}_few", xform="haar1d", seq_len=s, k_hi=int(rng.integers(0, 1 << lk)),
                       levels=r, **kw)
        return _wl(f"rnd{seed}_1d_r{r}_k{1 << lk}", xform="haar1d", seq_len=s, k_hi=1 << lk,
                   levels=int(rng.integers(r, r + lk + 1)), **kw)
    if kind == "haar2d":
        r = int(rng.integers(2, 4))               # 4 x 4 or 8 x 8 token blocks
        lg = int(rng.integers(0, 3))              # 1, 4 or 16 blocks
        side = (1 << r) << lg
        if rng.random() < 0.3:
            return _wl(f"rnd{seed}_2d_J{r}_few", xform="haar2d", seq_len=side * side, grid_h=side, grid_w=side,
                       k_hi=int(rng.integers(0, 1 << (2 * lg))), levels=r, corr_len=4.0, **kw)
        return _wl(f"rnd{seed}_2d_b{1 << r}_g{side}", xform="haar2d", seq_len=side * side, grid_h=side, grid_w=side,
                   k_hi=1 << (2 * lg), levels=int(rng.integers(r, r + lg + 1)), corr_len=float(rng.choice([2.0, 6.0])), **kw)
    return _wl(f"rnd{seed}_ident", xform="identity", levels=0, seq_len=int(rng.integers(1, 400)),
               k_hi=0, **kw) if rng.random() < 0.3 else \
        _wl(f"rnd{seed}_ident_k", xform="identity", levels=0, seq_len=int(rng.integers(40, 400)),
            k_hi=int(rng.integers(1, 40)), **kw)


@pytest.mark.parametrize("seed", range(32))
def test_random_valid_plans(seed):
    """Seeded sweep over the supported set: every plan the library accepts must meet the same bars."""
    w = _random_workload(seed)
    rng = np.random.default_rng(3000 + seed)
    r = tl.full_case(w, with_bias=bool(rng.integers(0, 2)), y_dtype=str(rng.choice(["f32", "bf16"])),
                     check_unfused=w.xform != "identity")
    assert r["code_mismatches"] == 0


@pytest.mark.parametrize("seed", range(24))
def test_random_plans_with_4bit_approximations(seed):
    """Seeded sweep over the plans without top levels whose 8-bit tokens are fewer than the approximations (the
    paper's language-model setting): the 4-bit approximations go through the 4-bit rows' GEMM as row 0 of their block,
    the 8-bit rows' GEMM over the first k_hi rows of every sequence (few-rows and tiled kernels, split depth or not,
    one or several sequences, channel splits of the transform kernel)."""
    rng = np.random.default_rng(7000 + seed)
    d_in = int(rng.choice([32, 96, 160, 512, 1024, 2080, 4128, 4608]))
    kw = dict(batch=int(rng.integers(1, 5)), d_in=d_in, d_out=int(rng.integers(1, 300)) * 2, seed=8000 + seed,
              x_dtype=str(rng.choice(["bf16", "f32"])), act_quant=str(rng.choice(["sym", "asym"])),
              mean_shift=float(rng.choice([0.0, 0.5, -1.0])), n_outlier_channels=int(rng.integers(0, 4)), outlier_scale=25.0)
    if rng.random() < 0.6:
        r = int(rng.integers(3, 7))
        lk = int(rng.integers(1, 8 if d_in <= 1024 else 6))
        w = _wl(f"few{seed}_1d_J{r}", xform="haar1d", seq_len=(1 << r) << lk, k_hi=int(rng.integers(1, 1 << lk)), levels=r, **kw)
    else:
        r = int(rng.integers(2, 4))
        lg = int(rng.integers(1, 4 if r == 2 else 3))
        side = (1 << r) << lg
        w = _wl(f"few{seed}_2d_J{r}", xform="haar2d", seq_len=side * side, grid_h=side, grid_w=side,
                k_hi=int(rng.integers(1, 1 << (2 * lg))), levels=r, corr_len=4.0, **kw)
    res = tl.full_case(w, with_bias=bool(seed & 1), y_dtype=("bf16" if seed % 3 == 0 else "f32"), check_unfused=(seed % 4 == 0))
    assert res["code_mismatches"] == 0


@pytest.mark.parametrize("case", ["1d", "2d_asym", "1d_fewer_hi"])
def test_forward_q_from_buffers_packed_on_the_host(case):
    """stamp_linear_forward_q on code / scale buffers that the HOST packs from the oracle's results, following only
    the layout that include/stamp.h documents (physical row order, tiled nibbles, stored asymmetric codes): the
    documented layout is the one the GEMM path reads."""
    import torch
    import paper_2510_26771_amd as st
    if case == "1d":
        w = _wl("hostpack_1d", batch=2, seq_len=512, levels=9, k_hi=16, d_in=160, d_out=200, seed=86)
    elif case == "2d_asym":
        w = _wl("hostpack_2d", batch=1, seq_len=1024, xform="haar2d", levels=5, grid_h=32, grid_w=32, k_hi=16, d_in=96,
                d_out=136, seed=87, act_quant="asym", mean_shift=0.4)
    else:
        w = _wl("hostpack_few", batch=2, seq_len=512, levels=3, k_hi=5, d_in=128, d_out=96, seed=88, act_quant="asym")
    inp = make_inputs(w, with_bias=True)
    ora = tl.run_oracle(w, inp)
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda(), torch.from_numpy(inp["bias"]).cuda())
    row = plan.row_of_coeff().astype(np.int64)       # physical row of STaMP slot p
    n_top = plan.hi_rows()
    B, s, d = w.batch, w.seq_len, w.d_in
    asym = w.act_quant == "asym"
    codes = ora["codes"].astype(np.int16)            # [B, s, d] in STaMP order
    if asym:                                         # stored form: code - 2^(b-1), b = 8 for the first k_hi slots
        codes = codes - np.where(np.arange(s) < w.k_hi, 128, 8).astype(np.int16)[None, :, None]
    q_hi = np.ascontiguousarray(codes[:, :n_top].astype(np.int8))
    # q_lo: byte of channels (c, c + 1) of row m = b * s + r at (((m/256)*(Kp/128) + c/128)*256 + m%256)*64 + (c%128)/2
    mp, kp = -(-(B * s) // 256) * 256, -(-d // 128) * 128
    q_lo = np.zeros(mp * kp // 2, dtype=np.uint8)
    phys = np.zeros((B, s, d), dtype=np.int16)
    phys[:, row[n_top:]] = codes[:, n_top:]
    nib = (phys & 0xF).astype(np.uint8)
    byte = (nib[:, :, 0::2] | (nib[:, :, 1::2] << 4)).reshape(B * s, d // 2)
    m = np.arange(B * s)[:, None]
    c = (2 * np.arange(d // 2))[None, :]
    q_lo[(((m // 256) * (kp // 128) + c // 128) * 256 + m % 256) * 64 + (c % 128) // 2] = byte
    scales = np.zeros((2, B, s) if asym else (B, s), dtype=np.float32)
    if asym:
        scales[0][:, row] = ora["scales"]
        scales[1][:, row] = ora["zeros"]
    else:
        scales[:, row] = ora["scales"]
    ws = plan.alloc_workspace()
    for engine in ("fp6", "int8"):
        plan.set_gemm_engine(engine)
        Y = torch.zeros((B, s, w.d_out), dtype=torch.float32, device="cuda")
        plan.linear_forward_q(torch.from_numpy(q_hi).cuda(), torch.from_numpy(q_lo).cuda(), torch.from_numpy(scales).cuda(),
                              Y, ws)
        torch.cuda.synchronize()
        tl.check_output(Y.cpu().numpy(), ora["Y"], False, f"{w.name} {engine}")
    plan.destroy()


def test_one_quantized_activation_feeds_several_linears():
    """One L + Q output feeds several linear layers, each with its own weights and inverse (the paper's block diagram:
    to_q / to_k / to_v share a quantized input): stamp_quantize_act once, stamp_linear_forward_q per plan."""
    import torch
    import paper_2510_26771_amd as st
    from dataclasses import replace
    w = _wl("shared_act", batch=2, seq_len=1024, levels=10, k_hi=16, d_in=256, d_out=192, seed=89)
    inp = make_inputs(w, with_bias=True)
    Xd = tl.to_device_x(inp, w)
    plans, refs = [], []
    for i, d_out in enumerate((192, 320, 64)):
        wi = replace(w, d_out=d_out, seed=w.seed + 10 * i)
        Wi, bi = make_inputs(wi, with_bias=True)["W"], make_inputs(wi, with_bias=True)["bias"]
        plans.append(st.StampPlan(tl.plan_desc_for(wi, "f32"), torch.from_numpy(Wi).cuda(), torch.from_numpy(bi).cuda()))
        refs.append(so.stamp_linear_forward(inp["X_f32"], Wi, w.xform, w.levels, w.k_hi, bias=bi, dtype=np.float32)["Y"])
    q_hi, q_lo, scales = plans[0].alloc_act_buffers()
    plans[0].quantize_act(Xd, q_hi, q_lo, scales, plans[0].alloc_workspace())
    for plan, ref in zip(plans, refs):
        Y = torch.zeros(ref.shape, dtype=torch.float32, device="cuda")
        plan.linear_forward_q(q_hi, q_lo, scales, Y, plan.alloc_workspace())
        torch.cuda.synchronize()
        tl.check_output(Y.cpu().numpy(), ref, False, "shared activation")
        plan.destroy()


def test_one_plan_two_streams_distinct_workspaces():
    """A plan is read-only in stamp_linear_forward: two streams may run it at the same time on different inputs,
    each with its own workspace, and get what the calls give one after the other."""
    import torch
    import paper_2510_26771_amd as st
    w = _wl("two_streams", batch=4, seq_len=2048, levels=11, k_hi=64, d_in=512, d_out=768, seed=83)
    inp = make_inputs(w, with_bias=True)
    plan = st.StampPlan(tl.plan_desc_for(w, "bf16"), torch.from_numpy(inp["W"]).cuda(),
                        torch.from_numpy(inp["bias"]).cuda())
    X1 = tl.to_device_x(inp, w)
    X2 = (X1.float() * -0.5 + 0.25).to(X1.dtype)
    ws1, ws2 = plan.alloc_workspace(), plan.alloc_workspace()
    shape = (w.batch, w.seq_len, w.d_out)
    ref1 = torch.zeros(shape, dtype=torch.int16, device="cuda")
    ref2 = torch.zeros_like(ref1)
    plan.linear_forward(X1, ref1, ws1)
    plan.linear_forward(X2, ref2, ws1)
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for it in range(3):
        Y1 = torch.zeros_like(ref1)
        Y2 = torch.zeros_like(ref1)
        torch.cuda.synchronize()
        for _ in range(4):  # several calls back to back, so that the two streams really overlap
            plan.linear_forward(X1, Y1, ws1, stream=s1)
            plan.linear_forward(X2, Y2, ws2, stream=s2)
        torch.cuda.synchronize()
        assert torch.equal(Y1, ref1) and torch.equal(Y2, ref2), f"round {it}"
    plan.destroy()


def test_non_finite_input_does_not_fault():
    """NaN / Inf activations: the result is unspecified, but every kernel runs to completion (no data-dependent
    addressing anywhere on the path) and the next call on clean input is correct."""
    import torch
    import paper_2510_26771_amd as st
    for w in (_wl("nonfinite_1d", batch=2, seq_len=256, levels=8, k_hi=8, d_in=128, d_out=136, seed=84),
              _wl("nonfinite_2d_asym", batch=1, seq_len=256, xform="haar2d", levels=4, grid_h=16, grid_w=16, k_hi=4,
                  d_in=96, d_out=64, seed=85, act_quant="asym")):
        inp = make_inputs(w)
        plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda())
        ws = plan.alloc_workspace()
        X = tl.to_device_x(inp, w)
        Y = torch.zeros((w.batch, w.seq_len, w.d_out), dtype=torch.float32, device="cuda")
        plan.linear_forward(X, Y, ws)
        torch.cuda.synchronize()
        good = Y.clone()
        Xb = X.clone()
        Xb[0, 3, 5] = float("nan")
        Xb[0, 100, 7] = float("inf")
        Xb[-1, 17, 0] = float("-inf")
        plan.linear_forward(Xb, Y, ws)
        torch.cuda.synchronize()            # completes without a fault
        plan.linear_forward(X, Y, ws)
        torch.cuda.synchronize()
        assert torch.equal(Y, good)
        plan.destroy()


def test_forward_under_hip_graph_capture():
    """stamp_linear_forward only enqueues kernels on the caller's stream (no allocation, no synchronisation, no
    memset): it can be captured into a HIP graph, and every replay reproduces the eager result bit for bit."""
    import torch
    import paper_2510_26771_amd as st
    few = _wl("graph_1d_few", batch=2, seq_len=1024, levels=3, k_hi=8, d_in=1024, d_out=192, seed=85)
    topfused = _wl("graph_1d_topfused", batch=3, seq_len=512, levels=9, k_hi=64, d_in=64, d_out=16640, seed=86)
    for w, hi_rows, routes in (
            (_wl("graph_1d", batch=2, seq_len=512, levels=9, k_hi=16, d_in=160, d_out=300, seed=81), 0, ("parts", "hi_fp6")),
            (_wl("graph_1d_beside", batch=2, seq_len=512, levels=9, k_hi=16, d_in=32, d_out=300, seed=81), 0, ("beside_top", "hi_fp6")),
            (_wl("graph_2d", batch=1, seq_len=256, xform="haar2d", levels=4, grid_h=16, grid_w=16, k_hi=4, d_in=96,
                 d_out=128, seed=82, act_quant="asym"), 0, ("hi_fp6",)),
            # no top levels, 4-bit approximations in the 4-bit rows' GEMM, the 8-bit rows on either pipeline (int8: the depth
            # split, parts added by a kernel)
            (few, 0, ("direct", "hi_fp6")), (few, 1, ("hi_split",)),
            # the 8-bit rows' GEMM runs the top levels of the inverse itself
            (topfused, 0, ()), (topfused, 1, ("hi_top_fused",))):
        inp = make_inputs(w, with_bias=True)
        plan = st.StampPlan(tl.plan_desc_for(w, "bf16"), torch.from_numpy(inp["W"]).cuda(),
                            torch.from_numpy(inp["bias"]).cuda())
        plan.set_choice("hi_rows", hi_rows)
        tl.check_routes(plan, w, routes)
        X = tl.to_device_x(inp, w)
        ws = plan.alloc_workspace()
        Y_eager = torch.zeros((w.batch, w.seq_len, w.d_out), dtype=torch.int16, device="cuda")
        plan.linear_forward(X, Y_eager, ws)           # also sets the kernels' attributes before the capture
        torch.cuda.synchronize()
        Y = torch.zeros_like(Y_eager)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            plan.linear_forward(X, Y, ws)             # warm-up on the capture stream
            torch.cuda.synchronize()
            with torch.cuda.graph(graph, stream=side):
                plan.linear_forward(X, Y, ws)
        torch.cuda.current_stream().wait_stream(side)
        for it in range(3):
            Y.fill_(-1)                               # eager work and a synchronisation between the replays
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(Y, Y_eager), f"{w.name}: replay {it} differs from the eager result"
        plan.destroy()


def test_bf16_output_and_bias():
    tl.full_case(_wl("bf16_out", batch=2, seq_len=256, levels=8, k_hi=8, d_in=256, d_out=384, seed=31),
                 with_bias=True, y_dtype="bf16")
    tl.full_case(_wl("bf16_out_2d", batch=1, seq_len=256, xform="haar2d", levels=4, grid_h=16, grid_w=16, k_hi=4,
                     d_in=128, d_out=256, seed=32), with_bias=True, y_dtype="bf16")


def test_degenerate_inputs():
    """All-zero activation (every scale 0, every code 0, output = bias) and a constant activation
    (only slot 0 is non-zero)."""
    import torch
    import paper_2510_26771_amd as st
    w = _wl("zeros", batch=1, seq_len=256, levels=8, k_hi=8, d_in=128, d_out=256, x_dtype="f32")
    inp = make_inputs(w, with_bias=True)
    Wd = torch.from_numpy(inp["W"]).cuda()
    bd = torch.from_numpy(inp["bias"]).cuda()
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), Wd, bd)
    ws = plan.alloc_workspace()
    for fill in (0.0, 1.5):
        X = np.full((1, 256, 128), fill, dtype=np.float32)
        ora = so.stamp_linear_forward(X, inp["W"], "haar1d", 8, 8, bias=inp["bias"])
        Xd = torch.from_numpy(X).cuda()
        q_hi, q_lo, scales = plan.alloc_act_buffers()
        plan.quantize_act(Xd, q_hi, q_lo, scales, ws)
        codes, sc, _ = tl.gpu_codes_in_stamp_order(plan, q_hi, q_lo, scales)
        assert np.array_equal(sc.view(np.uint32), ora["scales"].view(np.uint32))
        assert np.array_equal(codes, ora["codes"])
        if fill == 0.0:
            assert not codes.any() and not sc.any()
        Y = torch.empty((1, 256, 256), dtype=torch.float32, device="cuda")
        plan.linear_forward(Xd, Y, ws)
        torch.cuda.synchronize()
        tl.check_output(Y.cpu().numpy(), ora["Y"], False, f"fill {fill}")
    plan.destroy()


def test_bf16_weights_are_widened_exactly():
    """A plan built from bf16 weights holds the codes and scales of the same values given in fp32."""
    import torch
    import paper_2510_26771_amd as st
    from gen.workloads import f32_to_bf16_bits, bf16_bits_to_f32
    w = _wl("w_bf16", batch=1, seq_len=256, levels=8, k_hi=8, d_in=160, d_out=200, seed=97)
    inp = make_inputs(w, with_bias=True)
    bits = f32_to_bf16_bits(inp["W"])
    Wr = bf16_bits_to_f32(bits)
    d32 = tl.plan_desc_for(w, "f32")
    dbf = tl.plan_desc_for(w, "f32")
    dbf.w_dtype = st.binding.STAMP_BF16
    bias = torch.from_numpy(inp["bias"]).cuda()
    p32 = st.StampPlan(d32, torch.from_numpy(Wr).cuda(), bias)
    pbf = st.StampPlan(dbf, torch.from_numpy(bits.view(np.int16)).cuda(), bias)
    q32, s32 = p32.debug_weight_codes()
    qbf, sbf = pbf.debug_weight_codes()
    qo, so_ = so.quantize_weight(Wr, w.bits_w)
    assert np.array_equal(q32, qo) and np.array_equal(qbf, qo)
    assert np.array_equal(sbf.view(np.uint32), so_.view(np.uint32)) and np.array_equal(s32.view(np.uint32), so_.view(np.uint32))
    X = tl.to_device_x(inp, w)
    Y32 = torch.zeros((w.batch, w.seq_len, w.d_out), dtype=torch.float32, device="cuda")
    Ybf = torch.zeros_like(Y32)
    p32.linear_forward(X, Y32, p32.alloc_workspace())
    pbf.linear_forward(X, Ybf, pbf.alloc_workspace())
    torch.cuda.synchronize()
    assert torch.equal(Y32, Ybf)
    p32.destroy()
    pbf.destroy()


def test_w_out_by_in_layout():
    """W given as [d_out, d_in] (the algorithm's X W^T) yields the same plan as its transpose."""
    import torch
    import paper_2510_26771_amd as st
    w = _wl("wT", batch=1, seq_len=256, levels=8, k_hi=8, d_in=128, d_out=200)
    inp = make_inputs(w)
    d1 = tl.plan_desc_for(w, "f32")
    d2 = tl.plan_desc_for(w, "f32")
    d2.w_is_out_by_in = 1
    p1 = st.StampPlan(d1, torch.from_numpy(inp["W"]).cuda())
    p2 = st.StampPlan(d2, torch.from_numpy(np.ascontiguousarray(inp["W"].T)).cuda())
    q1, s1 = p1.debug_weight_codes()
    q2, s2 = p2.debug_weight_codes()
    assert np.array_equal(q1, q2) and np.array_equal(s1, s2)
    ref_q, ref_s = so.quantize_weight(inp["W"])
    assert np.array_equal(q1, ref_q) and np.array_equal(s1.view(np.uint32), ref_s.view(np.uint32))
    p1.destroy()
    p2.destroy()


@pytest.mark.parametrize("case", ["1d", "2d", "1d_partial", "2d_partial", "1d_many_top"])
def test_stamp_inverse_entry_point(case):
    """stamp_inverse alone on random STaMP-ordered input against the oracle's inverse."""
    import torch
    import paper_2510_26771_amd as st
    if case == "1d":
        w = _wl("inv1d", batch=2, seq_len=512, levels=9, k_hi=16, d_in=64, d_out=96)
    elif case == "1d_partial":
        w = _wl("inv1d_partial", batch=2, seq_len=512, levels=6, k_hi=16, d_in=64, d_out=96)
    elif case == "1d_many_top":  # 512 approximations, no top levels
        w = _wl("inv1d_many_top", batch=2, seq_len=4096, levels=3, k_hi=16, d_in=64, d_out=96)
    elif case == "2d_partial":
        w = _wl("inv2d_partial", batch=2, seq_len=1024, xform="haar2d", levels=3, grid_h=32, grid_w=32, k_hi=16,
                d_in=64, d_out=96)
    else:
        w = _wl("inv2d", batch=2, seq_len=1024, xform="haar2d", levels=5, grid_h=32, grid_w=32, k_hi=16, d_in=64,
                d_out=96)
    inp = make_inputs(w, with_bias=True)
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda(),
                        torch.from_numpy(inp["bias"]).cuda())
    rng = np.random.default_rng(5)
    for ncols in (96, 37):
        Yt = rng.standard_normal((w.batch, w.seq_len, ncols)).astype(np.float32)
        ref = np.stack([so.sequence_inverse(Yt[b], w.xform, w.levels, w.grid_h, w.grid_w) for b in range(w.batch)])
        if ncols == w.d_out:
            ref = ref + inp["bias"][None, None, :]
        Y = torch.empty((w.batch, w.seq_len, ncols), dtype=torch.float32, device="cuda")
        ws = torch.empty(max(plan.workspace_bytes(), w.batch * plan.hi_rows() * ncols * 4), dtype=torch.uint8, device="cuda")
        plan.inverse(torch.from_numpy(Yt).cuda(), ncols, Y, ws)
        torch.cuda.synchronize()
        err = np.max(np.abs(Y.cpu().numpy() - ref)) / np.max(np.abs(ref))
        assert err <= 1e-5, err
    plan.destroy()


def test_workspace_errors_on_device():
    import torch
    import paper_2510_26771_amd as st
    w = _wl("ws", batch=1, seq_len=256, levels=8, k_hi=8, d_in=128, d_out=256)
    inp = make_inputs(w)
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda())
    X = tl.to_device_x(inp, w)
    Y = torch.empty((1, 256, 256), dtype=torch.float32, device="cuda")
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(st.StampError) as e:
        plan.linear_forward(X, Y, small)
    assert e.value.status == 4
    ws = plan.alloc_workspace()
    with pytest.raises(st.StampError) as e:
        plan.linear_forward(X, Y, ws[1:])  # misaligned
    assert e.value.status == 4
    plan.destroy()


# ------------------------------------------------------------------------------------------------
# Full benchmark sizes, in the launch configuration bench.py times.  Stage A (codes, scales) is
# compared in full; the GEMM / inverse on a seeded sample of output columns the oracle can afford
# (the inverse needs whole columns, so the sample is by column).
# ------------------------------------------------------------------------------------------------
def _sample_cols(N, n, seed):
    """Output columns compared at full size: one seeded column inside EVERY 128-wide stretch (so every N tile of
    either GEMM engine, 256 or 128 wide, and every wave's 64-column half of some tile is sampled somewhere), both
    edges, and `n` further seeded columns."""
    rng = np.random.default_rng(seed)
    per_tile = [int(rng.integers(t, min(t + 128, N))) for t in range(0, N, 128)]
    extra = rng.choice(N, size=min(n, N), replace=False)
    return np.unique(np.concatenate([per_tile, extra, [0, N - 1]]).astype(np.int64))


def _full_size(w, seed, n_extra=16, with_bias=True):
    """bf16 output (the benchmark's configuration) and fp32 output (the stated 1e-3 bar with no allowance for
    the output format) on the same columns."""
    cols = _sample_cols(w.d_out, n_extra, seed)
    r = tl.full_case(w, with_bias=with_bias, y_dtype="bf16", cols=cols, check_unfused=False, also_f32_out=True)
    assert r["code_mismatches"] == 0
    tl.log(f"{w.name}: {len(cols)} columns; bf16 outputs not identical to the rounded oracle: "
           f"{r['bf16_nonidentical']} of {r['bf16_compared']}")
    assert max(v for k, v in r.items() if k.startswith("y_relerr_f32out")) <= 1e-3
    return r


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name", ["cfg2", "cfg4"])
def test_full_size_llm_and_dit(name):
    _full_size(get_workload(name), 7)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name", ["cfg2", "cfg4"])
def test_full_size_asymmetric_quantizer(name):
    """The paper's own quantizer (asymmetric min-max) on the LLM and image-token shapes at full size."""
    _full_size(get_workload(name, act_quant="asym"), 11)


@pytest.mark.timeout(600)
def test_full_size_image_tokens_three_levels():
    """cfg4's 64 x 64 grid with the 3-level transform of the paper's image-model experiments: the 64 8-bit
    tokens are exactly the low-low band, 8 x 8 token blocks hold all three levels."""
    _full_size(get_workload("cfg4", levels=3), 12)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name", ["cfg2", "cfg4"])
def test_full_size_second_mlp_layer(name):
    """The layer that follows cfg2 / cfg4 in its model (d_in and d_out swapped: 11008 -> 4096 on the LLM stream,
    4608 -> 1152 on the 64 x 64 grid): wider than one workgroup of the transform kernel holds."""
    base = get_workload(name)
    _full_size(get_workload(name, d_in=base.d_out, d_out=base.d_in, seed=base.seed + 50), 13)


@pytest.mark.timeout(600)
def test_full_size_llm_three_levels_64_hi_tokens():
    """cfg2's shape in the setting of the paper's language-model experiments: 3 levels, 64 8-bit tokens (of the 256
    approximations the first 64 are 8-bit, the other 192 are 4-bit rows), asymmetric min-max quantizer."""
    _full_size(get_workload("cfg2", levels=3, act_quant="asym"), 14)


@pytest.mark.timeout(900)
def test_full_size_cfg3_three_levels_64_hi_tokens():
    """cfg3's shape (8 sequences of 4096 tokens) in the paper's language-model setting: 3 levels leave 512
    approximations per sequence, 64 of them 8-bit tokens; served by the fast path (no top levels)."""
    w = get_workload("cfg3", levels=3)
    assert not tl.general_path(tl.plan_desc_for(w, "bf16"))
    _full_size(w, 8, with_bias=False)


@pytest.mark.timeout(900)
def test_full_size_cfg3():
    _full_size(get_workload("cfg3"), 8, with_bias=False)


@pytest.mark.timeout(1200)
def test_full_size_cfg5_benchmark_workload():
    _full_size(get_workload("cfg5"), 9, with_bias=False)

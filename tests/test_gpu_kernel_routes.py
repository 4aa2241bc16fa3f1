"""Edges of the kernels that serve only part of the plans: each case goes through the C ABI and is compared with the
oracle (codes and scales bit for bit, outputs to the output bar)."""
import numpy as np
import pytest

import stamp_testlib as tl
from gen.workloads import Workload
from oracle import stamp_oracle as so

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_26771_amd as st
    st.load_library()


def _wl(name, **kw):
    base = dict(batch=1, seq_len=256, d_in=128, d_out=192, xform="haar1d", levels=3, k_hi=16, x_dtype="f32", rho=0.9,
                n_outlier_channels=3, outlier_scale=20.0, w_std=0.05, seed=11)
    base.update(kw)
    return Workload(name, **base)


# ---- which pipeline takes the 8-bit rows: sizes on either side of the rule, all of them where one form takes at least 1.2
# times as long as the other (all tokens at 8 bits; 64 top rows a sequence with and without top levels; any length)
HI_RULE = [(dict(xform="identity", levels=0, seq_len=8192, k_hi=8192, d_in=1536, d_out=1536), False),
           (dict(xform="identity", levels=0, seq_len=2048, k_hi=2048, d_in=1152, d_out=4608), False),
           (dict(xform="identity", levels=0, seq_len=4096, k_hi=4096, d_in=4096, d_out=512), False),
           (dict(xform="identity", levels=0, seq_len=7820, k_hi=7820, d_in=2656, d_out=12), False),
           (dict(xform="identity", levels=0, seq_len=8192, k_hi=8192, d_in=192, d_out=64), True),
           (dict(xform="identity", levels=0, seq_len=1024, k_hi=1024, d_in=2048, d_out=2048), True),
           (dict(xform="identity", levels=0, seq_len=8192, k_hi=8192, d_in=256, d_out=256), True),
           (dict(batch=32, seq_len=512, levels=9, k_hi=64, d_in=4096, d_out=4096), False),
           (dict(batch=32, seq_len=512, levels=9, k_hi=64, d_in=512, d_out=4096), False),
           (dict(batch=8, seq_len=512, levels=9, k_hi=64, d_in=2048, d_out=2048), True),
           (dict(batch=32, seq_len=512, levels=3, k_hi=63, d_in=2048, d_out=4096), False),
           (dict(batch=4, seq_len=512, levels=3, k_hi=63, d_in=4096, d_out=1024), True),
           (dict(batch=64, seq_len=481, levels=3, k_hi=60, d_in=4096, d_out=2048, skip_first=True), False),
           (dict(batch=8, seq_len=481, levels=3, k_hi=60, d_in=4096, d_out=1024, skip_first=True), True),
           (dict(batch=2, seq_len=64, levels=6, k_hi=64, d_in=11008, d_out=11008), True)]  # up to 128 rows


@pytest.mark.parametrize("kw,fp6", HI_RULE, ids=["-".join(str(v) for v in kw.values()) for kw, _ in HI_RULE])
def test_rule_of_the_8bit_rows_pipeline(kw, fp6):
    import torch
    import paper_2510_26771_amd as st
    w = _wl("rule", x_dtype="bf16", **kw)
    plan = st.StampPlan(tl.plan_desc_for(w, "bf16"), torch.zeros((w.d_in, w.d_out), dtype=torch.float32, device="cuda"))
    tl.check_routes(plan, w, ("hi_fp6" if fp6 else "-hi_fp6",))
    plan.destroy()


# ---- blocks of 8 and 16 tokens by lanes (FP6 operands straight from the quantizer): the widths on either side of what one group of
# channels per lane holds and the widest of all, a last wave that is partly empty, blocks of any length, several sequences
def _lanes(d, levels=3, **kw):
    base = dict(seq_len=2048 if d > 8192 else 128, levels=levels, k_hi=16, d_in=d, d_out=66, seed=600 + d)
    base.update(kw)
    return _wl("lanes_d%d_l%d_%s" % (d, levels, "_".join(f"{k}{v}" for k, v in kw.items())), **base)


LANES = [_lanes(64, batch=3, x_dtype="bf16"), _lanes(96, act_quant="asym", mean_shift=0.4), _lanes(544, levels=4, k_hi=8, x_dtype="bf16"),
         _lanes(4096, levels=4, k_hi=8), _lanes(4064, levels=4, k_hi=8, act_quant="asym", mean_shift=0.4, x_dtype="bf16"),
         _lanes(8192, x_dtype="bf16"), _lanes(8192, act_quant="asym"), _lanes(4128), _lanes(8224, x_dtype="bf16"),
         _lanes(12288, x_dtype="bf16", act_quant="asym", mean_shift=0.4), _lanes(1184, levels=7, k_hi=16, x_dtype="bf16"),
         _lanes(1056, levels=4, k_hi=16, seq_len=256, batch=2, act_quant="asym"), _lanes(160, levels=8, k_hi=16, seq_len=256), _lanes(8192, seq_len=131, skip_first=True, x_dtype="bf16"),
         _lanes(224, levels=4, seq_len=402, skip_first=True, batch=2, act_quant="asym", mean_shift=0.4), _lanes(4096, levels=4, seq_len=203)]


@pytest.mark.parametrize("w", LANES, ids=[w.name for w in LANES])
def test_blocks_by_lanes(w):
    import torch
    import paper_2510_26771_amd as st
    tl.full_case(w, with_bias=True, check_unfused=False, engines=("fp6",), routes=("direct",))
    # the same codes as the quantizer that packs them: the same output bit for bit
    inp = tl.make_inputs(w)
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda())
    X = tl.to_device_x(inp, w)
    Y = [torch.empty((w.batch, w.seq_len, w.d_out), dtype=torch.float32, device="cuda") for _ in range(2)]
    for packed in (0, 1):
        plan.set_choice("operands", packed)
        plan.linear_forward(X, Y[packed], plan.alloc_workspace())
    torch.cuda.synchronize()
    assert torch.equal(Y[0], Y[1])
    plan.destroy()


# ---- blocks of a token grid by lanes: the widths of one wave, of several and the widest, a last wave that is partly empty, blocks
# whose sums are 8-bit rows, 4-bit rows (k_hi below the approximations; both block sizes and code forms) or go to levels above; grids
# that are no square, which run level by level and then by rows
def _lanes2(d, levels, gh, gw, k, batch=1, **kw):
    base = dict(xform="haar2d", grid_h=gh, grid_w=gw, seq_len=gh * gw, batch=batch, levels=levels, k_hi=k, d_in=d, d_out=66, seed=900 + d, corr_len=4.0)
    base.update(kw)
    return _wl("lanes2_%dx%dx%dx%d_J%d_k%d_%s" % (batch, gh, gw, d, levels, k, "_".join(f"{a}{b}" for a, b in kw.items())), **base)


LANES2 = [_lanes2(32, 3, 16, 16, 4, x_dtype="bf16"), _lanes2(160, 3, 16, 32, 8, act_quant="asym", mean_shift=0.4),
          _lanes2(1536, 3, 16, 16, 4, x_dtype="bf16", act_quant="asym"), _lanes2(1536, 3, 16, 16, 4), _lanes2(1184, 3, 32, 16, 5, batch=2),
          _lanes2(288, 4, 32, 32, 16, x_dtype="bf16"), _lanes2(1056, 4, 32, 32, 16, act_quant="asym", mean_shift=-0.3),
          _lanes2(32, 2, 16, 16, 16, batch=3, x_dtype="bf16"), _lanes2(544, 2, 8, 16, 8, act_quant="asym", mean_shift=0.4), _lanes2(1184, 2, 16, 8, 5, batch=2),
          _lanes2(4096, 2, 16, 16, 16, x_dtype="bf16"), _lanes2(4064, 2, 16, 16, 16, act_quant="asym"),
          _lanes2(544, 2, 16, 16, 5, act_quant="asym", mean_shift=0.4), _lanes2(1184, 2, 16, 16, 5, batch=2, x_dtype="bf16"),
          _lanes2(160, 3, 32, 32, 7, act_quant="asym", mean_shift=0.4), _lanes2(1184, 3, 32, 32, 5, batch=2),
          # 4 x 4 blocks below top levels
          _lanes2(288, 4, 16, 16, 16, batch=2, x_dtype="bf16"), _lanes2(1056, 3, 16, 16, 16, act_quant="asym", mean_shift=0.4), _lanes2(32, 3, 8, 8, 4, batch=3),
          _lanes2(2080, 4, 16, 16, 16, batch=16, x_dtype="bf16")]


@pytest.mark.parametrize("w", LANES2, ids=[w.name for w in LANES2])
def test_grid_blocks_by_lanes(w):
    import torch
    import paper_2510_26771_amd as st
    tl.full_case(w, with_bias=True, check_unfused=False, engines=("fp6",), routes=("direct", "-general" if w.grid_h == w.grid_w else "general"))
    inp = tl.make_inputs(w)
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda())
    X = tl.to_device_x(inp, w)
    Y = [torch.empty((w.batch, w.seq_len, w.d_out), dtype=torch.float32, device="cuda") for _ in range(2)]
    for packed in (0, 1):
        plan.set_choice("operands", packed)
        plan.linear_forward(X, Y[packed], plan.alloc_workspace())
    torch.cuda.synchronize()
    assert torch.equal(Y[0], Y[1])
    plan.destroy()


# ---- rows by lanes: four, two and one of them to a workgroup, the widths on either side; rows and 8-bit rows that are no multiple
# of that; a last wave that is partly empty; all rows at 8 bits; rows of the general path; few rows by 8 channels a thread, on either
# side of their line (256 rows; 2048 channels bf16, 4096 fp32)
def _rows(d, s, batch, k, xform="identity", **kw):
    base = dict(xform=xform, levels=0, seq_len=s, batch=batch, k_hi=k, d_in=d, d_out=66, seed=700 + d)
    base.update(kw)
    return _wl("rows_%s_%dx%dx%d_k%d_%s" % (xform, batch, s, d, k, "_".join(f"{a}{b}" for a, b in kw.items())), **base)


ROWS = [_rows(32, 3, 1, 1), _rows(96, 131, 3, 5, x_dtype="bf16"), _rows(544, 37, 2, 0, act_quant="asym", mean_shift=0.4),
        _rows(2080, 130, 1, 33, x_dtype="bf16", act_quant="asym"), _rows(8192, 21, 1, 4, x_dtype="bf16"), _rows(8224, 21, 1, 4, x_dtype="bf16"),
        _rows(8224, 19, 1, 3, act_quant="asym", mean_shift=0.4), _rows(16384, 7, 3, 2), _rows(16416, 5, 3, 2), _rows(16416, 5, 3, 2, x_dtype="bf16"),
        _rows(96, 4100, 2, 16, x_dtype="bf16"), _rows(1056, 1030, 1, 7, act_quant="asym", mean_shift=0.4), _rows(8192, 517, 1, 4), _rows(160, 64, 3, 5, xform="wht"), _rows(1056, 33, 3, 2, xform="dct", act_quant="asym", x_dtype="bf16"),
        _rows(96, 256, 1, 5), _rows(544, 257, 1, 5), _rows(2048, 85, 3, 9, x_dtype="bf16"), _rows(2080, 85, 3, 9, x_dtype="bf16", act_quant="asym"),
        _rows(4096, 16, 1, 1, act_quant="asym", mean_shift=0.4), _rows(4128, 16, 1, 16), _rows(32, 20, 2, 20, x_dtype="bf16", act_quant="asym"),
        _rows(1056, 300, 1, 33, act_quant="asym"), _rows(96, 257, 2, 40, x_dtype="bf16")]


@pytest.mark.parametrize("w", ROWS, ids=[w.name for w in ROWS])
def test_rows_by_lanes(w):
    import torch
    import paper_2510_26771_amd as st
    tl.full_case(w, with_bias=True, check_unfused=False, engines=("fp6",), routes=("direct",))
    inp = tl.make_inputs(w)
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda())
    X = tl.to_device_x(inp, w)
    Y = [torch.empty((w.batch, w.seq_len, w.d_out), dtype=torch.float32, device="cuda") for _ in range(2)]
    for packed in (0, 1):
        plan.set_choice("operands", packed)
        plan.linear_forward(X, Y[packed], plan.alloc_workspace())
    torch.cuda.synchronize()
    assert torch.equal(Y[0], Y[1])
    plan.destroy()


# ---- who writes the FP6 operands: the quantizer, or a pass over packed codes (sizes where the form that the rule takes is at least 1.05
# times as fast, us packed and direct beside them: quantizers by rows, by blocks on a line, of any length, on a grid)
OPERANDS = [(dict(xform="identity", levels=0, batch=32, seq_len=1024, k_hi=2, d_in=256), True),  # 39.0, 25.3
            (dict(xform="identity", levels=0, seq_len=4096, k_hi=4096, d_in=256), True),  # 18.3, 12.7
            (dict(xform="identity", levels=0, batch=16, seq_len=1024, k_hi=256, d_in=1024), True),  # 46.0, 34.6
            (dict(xform="wht", levels=0, batch=64, seq_len=1024, k_hi=1, d_in=32), True),  # 97.5, 75.0
            (dict(xform="identity", levels=0, batch=2, seq_len=1024, k_hi=32, d_in=2048), True),  # 31.0, 26.4
            (dict(xform="wht", levels=0, batch=1, seq_len=1024, k_hi=64, d_in=512), True),  # 39.3, 35.8
            (dict(batch=64, seq_len=1024, k_hi=1, d_in=1024), True),  # 70.2, 53.8
            (dict(batch=256, seq_len=1024, k_hi=1, d_in=32), False),  # 95.1, 106.8
            (dict(batch=128, seq_len=512, levels=9, k_hi=64, d_in=256), False),  # 70.7, 77.2
            (dict(batch=128, seq_len=513, k_hi=1, d_in=512, skip_first=True), True),  # 52.5, 38.9
            (dict(xform="haar2d", batch=4, seq_len=1024, grid_h=32, grid_w=32, k_hi=16, d_in=512), True),  # 24.7, 19.6
            (dict(xform="haar2d", batch=32, seq_len=1024, grid_h=32, grid_w=32, levels=5, k_hi=64, d_in=1152), True),  # 73.2 (beside the top levels), 66.9
            (dict(xform="haar2d", batch=128, seq_len=1024, grid_h=32, grid_w=32, levels=5, k_hi=64, d_in=64), False),  # 82.4, 87.2
            (dict(batch=2, seq_len=1024, levels=10, k_hi=32, d_in=512), True)]  # blocks of 32, in parts: 29.6 (beside the top levels), 22.7

# ---- blocks below top levels: in parts of 8 tokens or not (us, whole blocks and parts)
PARTS_RULE = [(dict(seq_len=4096, levels=12, k_hi=64, d_in=64), True),  # 42.1, 23.4
              (dict(seq_len=256, levels=8, k_hi=8, d_in=128), True),  # 25.1, 19.4
              (dict(batch=2, seq_len=2048, levels=11, k_hi=64, d_in=512), True),  # 33.9, 25.1
              (dict(seq_len=1024, levels=10, k_hi=64, d_in=128), True),  # 23.0, 20.1
              (dict(batch=64, seq_len=128, levels=7, k_hi=8, d_in=96), False),  # 20.6, 22.3
              (dict(batch=64, seq_len=256, levels=8, k_hi=16, d_in=128), False),  # 23.5, 25.3
              (dict(batch=256, seq_len=128, levels=7, k_hi=8, d_in=512), True),  # 39.6, 35.0
              (dict(batch=4, seq_len=2048, levels=11, k_hi=64, d_in=4096), False),  # 62.3, 71.8
              (dict(batch=8, seq_len=2048, levels=11, k_hi=32, d_in=2048), False),  # 57.6, 63.3
              (dict(batch=32, seq_len=512, levels=9, k_hi=8, d_in=2048), True),  # 59.3, 55.6
              (dict(batch=8, seq_len=2048, levels=11, k_hi=32, d_in=1024), True)]  # 49.3, 42.6


@pytest.mark.parametrize("kw,parts", PARTS_RULE, ids=["-".join(str(v) for v in kw.values()) for kw, _ in PARTS_RULE])
def test_rule_of_the_parts(kw, parts):
    import torch
    import paper_2510_26771_amd as st
    w = _wl("parts_rule", x_dtype="bf16", d_out=256, **kw)
    plan = st.StampPlan(tl.plan_desc_for(w, "bf16"), torch.zeros((w.d_in, w.d_out), dtype=torch.float32, device="cuda"))
    tl.check_routes(plan, w, ("parts" if parts else "-parts",))
    plan.destroy()



@pytest.mark.parametrize("kw,direct", OPERANDS, ids=["-".join(str(v) for v in kw.values()) for kw, _ in OPERANDS])
def test_rule_of_the_operands(kw, direct):
    import torch
    import paper_2510_26771_amd as st
    w = _wl("operands", x_dtype="bf16", d_out=256, **kw)
    plan = st.StampPlan(tl.plan_desc_for(w, "bf16"), torch.zeros((w.d_in, w.d_out), dtype=torch.float32, device="cuda"))
    tl.check_routes(plan, w, ("direct" if direct else "-direct",))
    plan.destroy()


# ---- DCT of power-of-two lengths (FFT): odd and even numbers of radix-2 stages, one and several channels per
# workgroup, the shortest length of the route and the longest of the library
DCT = [_wl("dct_8", batch=2, xform="dct", levels=0, seq_len=8, k_hi=1, seed=201),
       _wl("dct_16_bf16", xform="dct", levels=0, seq_len=16, k_hi=2, x_dtype="bf16", seed=202),
       _wl("dct_512", batch=3, xform="dct", levels=0, seq_len=512, d_in=160, d_out=131, seed=203),
       _wl("dct_1024_asym", xform="dct", levels=0, seq_len=1024, act_quant="asym", mean_shift=0.5, seed=204),
       # points in registers: four and eight channels per workgroup, last pass of radix 1, 2, 4 and 8, a last group of channels
       # that is not full
       _wl("dct_512_reg", batch=13, xform="dct", levels=0, seq_len=512, d_in=160, d_out=163, k_hi=8, x_dtype="bf16", seed=205),
       _wl("dct_1024_reg", batch=13, xform="dct", levels=0, seq_len=1024, d_in=160, d_out=163, k_hi=8, seed=206),
       _wl("dct_2048_reg", batch=8, xform="dct", levels=0, seq_len=2048, d_in=256, d_out=258, k_hi=8, x_dtype="bf16", seed=207),
       # with seed 208 a row maximum lies 4e-6 of its fp32 spacing from a rounding boundary
       _wl("dct_2048_near", xform="dct", levels=0, seq_len=2048, d_in=96, d_out=33, k_hi=8, x_dtype="bf16", seed=208),
       _wl("dct_2048_few", xform="dct", levels=0, seq_len=2048, d_in=96, d_out=33, k_hi=8, x_dtype="bf16", seed=214),
       _wl("dct_4096_reg", batch=8, xform="dct", levels=0, seq_len=4096, d_in=256, d_out=257, k_hi=8, seed=209)]


@pytest.mark.parametrize("w", DCT, ids=[w.name for w in DCT])
def test_dct_of_power_of_two_lengths(w):
    tl.full_case(w, with_bias=True, check_unfused=False)


@pytest.mark.parametrize("s", [16, 64, 256, 1024, 4096, 16384])
def test_dct_rows_of_one_magnitude_are_rounded_once(s):
    """Coefficients 0 and s / 2 are signed sums of tokens over sqrt(s).  For s a power of four that is exact in fp64, and a sum
    half way between two fp32 numbers goes to the even one."""
    import torch
    import paper_2510_26771_amd as st
    w = _wl(f"dct_tie_{s}", xform="dct", levels=0, seq_len=s, k_hi=1, d_in=32, d_out=16, x_dtype="bf16")
    X = torch.zeros((1, s, 32), dtype=torch.bfloat16, device="cuda")
    # tokens 0 and 3 enter both with a plus: 2^14 + 2^-10, 25 bits
    X[0, 0], X[0, 3] = 2.0 ** 14, 2.0 ** -10
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.zeros((32, 16), dtype=torch.float32, device="cuda"))
    q = plan.alloc_act_buffers()
    plan.quantize_act(X, *q, plan.alloc_workspace())
    torch.cuda.synchronize()
    row = np.float32(2.0 ** 14 / np.sqrt(float(s)))
    assert q[2][0, 0].item() == row / np.float32(127) and q[2][0, s // 2].item() == row / np.float32(7)
    plan.destroy()


@pytest.mark.parametrize("s", [8, 64, 2048, 4096, 16384])
def test_dct_inverse_against_the_dense_product(s):
    """stamp_inverse of an odd number of columns: fp64 all the way, one rounding at the end.  Both sides are fp64 sums, so they
    agree to 2^-24 of the column plus the rounding of s terms."""
    import torch
    import paper_2510_26771_amd as st
    w = _wl(f"inv_dct_{s}", batch=2 if s <= 64 else 1, seq_len=s, xform="dct", levels=0, k_hi=1, d_in=32, d_out=37)
    W = torch.zeros((32, 37), dtype=torch.float32, device="cuda")
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), W)
    rng = np.random.default_rng(s)
    Yt = rng.standard_normal((w.batch, s, 37)).astype(np.float32)
    Yt[:, :, 5] *= 1e6  # a channel's error stays its own
    cols = [0, 5, 36]
    if s <= 4096:
        ref = np.stack([so.dct_matrix(s).T @ Yt[b][:, cols].astype(np.float64) for b in range(w.batch)])
    else:
        n = np.arange(s, dtype=np.float64)
        k = np.arange(s, dtype=np.int64)
        ref = np.zeros((w.batch, s, len(cols)))
        for lo in range(0, s, 1024):  # angles reduced to one turn as integers
            ang = ((2 * np.arange(lo, lo + 1024, dtype=np.int64)[:, None] + 1) * k[None, :]) % (4 * s)
            C = np.cos(np.pi * ang / (2.0 * s)) * np.sqrt(2.0 / s)
            C[:, 0] = np.sqrt(1.0 / s)
            ref[0, lo:lo + 1024] = C @ Yt[0][:, cols].astype(np.float64)
        del n
    one = -(-(w.batch * s * 37 * 4) // 256) * 256
    ws = torch.empty(2 * one, dtype=torch.uint8, device="cuda")
    Y = torch.empty((w.batch, s, 37), dtype=torch.float32, device="cuda")
    plan.inverse(torch.from_numpy(Yt).cuda(), 37, Y, ws)
    torch.cuda.synchronize()
    y = Y.cpu().numpy()[:, :, cols].astype(np.float64)
    bound = 2.0 ** -24 * np.abs(ref) + (s * 2.0 ** -50) * np.abs(ref).max(axis=(0, 1), keepdims=True)
    assert (np.abs(y - ref) <= bound).all(), float((np.abs(y - ref) / bound).max())
    plan.destroy()


@pytest.mark.parametrize("s", [8, 64, 1024, 2048, 8192])
def test_dct_of_infinities(s):
    """An infinite activation makes every coefficient of its channel infinite, so every scale of that sequence is, and no
    output of it looks like a number; an infinite coefficient makes its whole column infinite, each token with the sign of
    its cosine.  The other sequence and the other columns do not notice."""
    import torch
    import paper_2510_26771_amd as st
    w = _wl(f"dct_inf_{s}", batch=2, xform="dct", levels=0, seq_len=s, k_hi=2, d_in=64, d_out=37)
    inp = tl.make_inputs(w)
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda())
    X = tl.to_device_x(inp, w)
    ws = plan.alloc_workspace()
    good, bad = plan.alloc_act_buffers(), plan.alloc_act_buffers()
    Y, Yb = (torch.zeros((2, s, 37), dtype=torch.float32, device="cuda") for _ in range(2))
    plan.quantize_act(X, *good, ws)
    plan.linear_forward(X, Y, ws)
    X[0, s // 2 + 1, 5] = float("inf")
    X[0, 1, 9] = float("-inf")
    plan.quantize_act(X, *bad, ws)
    plan.linear_forward(X, Yb, ws)
    torch.cuda.synchronize()
    assert torch.isinf(bad[2][0]).all(), "a scale that does not show the infinity"
    assert not torch.isfinite(Yb[0]).any()
    assert torch.equal(bad[2][1], good[2][1]) and torch.equal(Yb[1], Y[1])
    # stamp_inverse: coefficient k infinite
    k, col = s // 2 + 1, 3
    Yt = torch.randn((2, s, 37), device="cuda")
    inv_ws = torch.empty(2 * (-(-(2 * s * 37 * 4) // 256) * 256), dtype=torch.uint8, device="cuda")
    plan.inverse(Yt, 37, Y, inv_ws)
    Yt[1, k, col] = float("-inf")
    plan.inverse(Yt, 37, Yb, inv_ws)
    torch.cuda.synchronize()
    cosine = np.cos(np.pi * (((2 * np.arange(s, dtype=np.int64) + 1) * k) % (4 * s)) / (2.0 * s))
    assert np.array_equal(Yb[1, :, col].cpu().numpy(), np.where(cosine > 0, -np.inf, np.inf))
    Yb[1, :, col] = Y[1, :, col]
    assert torch.equal(Yb, Y)
    plan.destroy()


# ---- WHT in one pass (64 .. 4096 tokens): every split of the stages, the lengths on either side of the range, channel
# counts that leave the last workgroup partly empty
WHT = [_wl(f"wht_{1 << J}", batch=2 if J < 10 else 1, xform="wht", levels=0, seq_len=1 << J, k_hi=1 << (J // 2), d_in=32 * (J - 3),
           d_out=101 + J, act_quant="asym" if J % 2 else "sym", x_dtype="bf16" if J % 3 else "f32", seed=220 + J)
       for J in range(5, 14)]


@pytest.mark.parametrize("w", WHT, ids=[w.name for w in WHT])
def test_wht_lengths(w):
    tl.full_case(w, with_bias=True, check_unfused=False, engines=("fp6",))


# ---- 1-D Haar of any length in its blocked form (3 .. 6 levels): every number of tokens in the short last block, blocks
# that cross the GEMM's row tiles, 8-bit tokens from one to all approximations, odd d_out
def _rag(levels, n, skip, **kw):
    s = n + skip
    kw.setdefault("k_hi", max(1, min(16, (n >> levels) // 2)))
    return _wl(f"rag_L{levels}_n{n}_o{skip}_k{kw['k_hi']}_N{kw.get('d_out', 192)}", seq_len=s, levels=levels,
               skip_first=bool(skip), seed=300 + n, **kw)


RAG = ([_rag(3, 40 + m, m & 1, batch=3, d_in=96, d_out=68) for m in range(1, 9)] +
       [_rag(4, 300 + m, 1, batch=2, d_in=64, act_quant="asym", mean_shift=0.3) for m in (1, 4, 6, 11)] +
       [_rag(5, 513 + m, 1, d_in=160, d_out=257, x_dtype="bf16") for m in (0, 6, 31)] +
       [_rag(6, 700 + m, 1, batch=2, d_in=64, d_out=130) for m in (5, 25, 60)] +
       [_rag(3, 1023, 1, k_hi=129, d_out=515), _rag(3, 1000, 0, k_hi=1), _rag(4, 776, 1, batch=3, k_hi=32, d_out=33),
        _rag(3, 5, 1, k_hi=1, batch=64), _rag(3, 9, 1, k_hi=3, batch=64)])
# (the rows in block order lie over the workspace's fp32 copies of X: plans whose copies are smaller run level by level)
RAG_SMALL = [_rag(3, 5, 1, k_hi=1), _rag(3, 9, 1, k_hi=3)]


@pytest.mark.parametrize("w", RAG, ids=[w.name for w in RAG])
def test_blocked_haar_of_any_length(w):
    for y in ("f32", "bf16"):
        tl.full_case(w, with_bias=True, check_unfused=False, y_dtype=y, routes=("any_length_blocks", "hi_fp6"))


@pytest.mark.parametrize("w", RAG_SMALL, ids=[w.name for w in RAG_SMALL])
def test_short_sequences_level_by_level(w):
    for y in ("f32", "bf16"):
        tl.full_case(w, with_bias=True, check_unfused=False, y_dtype=y, routes=("-any_length_blocks",))


# ---- per-block scales on blocks of 4 x 4 and 8 x 8 tokens: with and without top levels, 4-bit approximations, a depth
# that ends in half a K step, output widths off the tile, several sequences
def _grp(side, J, k, d, n, **kw):
    return _wl(f"grp_{side}_J{J}_k{k}_d{d}_n{n}", seq_len=side * side, grid_h=side, grid_w=side, xform="haar2d", levels=J, k_hi=k,
               d_in=d, d_out=n, group_size=64, corr_len=4.0, seed=400 + d + n, **kw)


GRP_LEVELS = [_grp(64, 3, 64, 192, 131), _grp(32, 3, 64, 64, 258, batch=2, x_dtype="bf16"), _grp(32, 5, 64, 320, 66, batch=3),
              _grp(64, 6, 64, 128, 514), _grp(32, 2, 16, 128, 192, x_dtype="bf16"), _grp(32, 3, 4, 256, 128), _grp(8, 1, 4, 64, 64),
              _grp(8, 3, 4, 192, 200, batch=5), _grp(16, 2, 16, 448, 64, batch=9), _grp(32, 3, 64, 128, 131)]
# (the sizes from which on the block kernels serve such plans: smaller ones, and odd widths, run level by level)
GRP = [_grp(64, 3, 64, 192, 1026), _grp(32, 5, 64, 320, 1410, batch=3), _grp(64, 6, 64, 128, 1026),
       _grp(32, 3, 64, 64, 2050, batch=2, x_dtype="bf16"), _grp(8, 3, 4, 192, 1026, batch=70), _grp(16, 2, 16, 448, 1026, batch=17),
       _grp(32, 3, 4, 256, 1026, batch=4), _grp(32, 2, 16, 128, 1090, batch=4, x_dtype="bf16"),
       # top levels over 4 x 4 block sums, to the last one and not; at most 32 8-bit rows over the batch
       _grp(16, 4, 16, 128, 1026, batch=17), _grp(16, 3, 16, 320, 1290, batch=15, x_dtype="bf16"),
       _grp(32, 4, 16, 192, 2050, batch=2), _grp(32, 5, 16, 64, 2306, batch=2, x_dtype="bf16"),
       # the last 256 columns of the stored weights hold one tile of outputs and one of nothing
       _grp(64, 3, 64, 64, 322, batch=4, x_dtype="bf16")]


@pytest.mark.parametrize("w", GRP, ids=[w.name for w in GRP])
def test_per_block_scales_on_token_blocks(w):
    for y in ("f32", "bf16"):
        tl.grouped_case(w, with_bias=True, y_dtype=y, routes=("group_blocks", "group_quant"))


# blocks for the quantizer only: too few tiles for the GEMM with the inverse
GRP_QUANT = [_grp(64, 3, 64, 192, 130), _grp(16, 2, 16, 448, 64, batch=17), _grp(32, 3, 4, 256, 128, batch=4),
             _grp(32, 2, 16, 128, 192, batch=5, x_dtype="bf16"), _grp(64, 6, 64, 64, 510, batch=2, x_dtype="bf16"),
             _grp(16, 2, 16, 64, 66, batch=256, x_dtype="bf16")]


@pytest.mark.parametrize("w", GRP_QUANT, ids=[w.name for w in GRP_QUANT])
def test_per_block_scales_quantized_on_token_blocks(w):
    for y in ("f32", "bf16"):
        tl.grouped_case(w, with_bias=True, y_dtype=y, routes=("-group_blocks", "group_quant"))


@pytest.mark.parametrize("w", GRP_LEVELS, ids=[w.name for w in GRP_LEVELS])
def test_per_block_scales_level_by_level(w):
    for y in ("f32", "bf16"):
        tl.grouped_case(w, with_bias=True, y_dtype=y, routes=("-group_blocks", "-group_quant"))


# ---- the blocked forms take 16-byte aligned X and Y; others run level by level.  Codes are the same either way, so the two
# halves of a layer may take different forms.
ALIGN = [(_rag(3, 203, 1, batch=2, d_in=96, d_out=72), "any_length_blocks"),
         (_rag(4, 300, 0, d_in=64, d_out=67, act_quant="asym", mean_shift=0.3, x_dtype="bf16"), "any_length_blocks"),
         (_grp(64, 3, 64, 128, 1026), "group_blocks"), (_grp(16, 4, 16, 64, 1026, batch=17, x_dtype="bf16"), "group_blocks")]


@pytest.mark.parametrize("w,route", ALIGN, ids=[w.name for w, _ in ALIGN])
def test_tensors_off_the_16_byte_grid(w, route):
    import torch
    import paper_2510_26771_amd as st

    def off_by_one(t):
        buf = torch.zeros(t.numel() + 1, dtype=t.dtype, device="cuda")
        buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)

    inp = tl.make_inputs(w, with_bias=True)
    ora = (so.stamp_linear_forward_grouped(inp["X_f32"], inp["W"], w.xform, w.levels, w.k_hi, 64, w.bits_hi, w.bits_lo, w.bits_w,
                                           w.grid_h, w.grid_w, inp["bias"]) if w.group_size else tl.run_oracle(w, inp))
    X = tl.to_device_x(inp, w)
    for y_dtype, ydt in (("f32", torch.float32), ("bf16", torch.int16)):
        plan = st.StampPlan(tl.plan_desc_for(w, y_dtype), torch.from_numpy(inp["W"]).cuda(), torch.from_numpy(inp["bias"]).cuda())
        tl.check_routes(plan, w, (route,))
        ws = plan.alloc_workspace()
        acts = []
        for x in (X, off_by_one(X)):
            q = plan.alloc_act_buffers()
            q[0].zero_()
            plan.quantize_act(x, *q, ws)
            acts.append(q)
            for aligned in (True, False):
                Y = torch.zeros((w.batch, w.seq_len, w.d_out), dtype=ydt, device="cuda")
                Y = Y if aligned else off_by_one(Y)
                assert (Y.data_ptr() % 16 == 0) == aligned
                plan.linear_forward(x, Y, ws)
                Yq = torch.zeros_like(Y) if aligned else off_by_one(torch.zeros_like(Y))
                plan.linear_forward_q(*q, Yq, ws)
                torch.cuda.synchronize()
                tl.check_output(tl.y_to_numpy(Y, y_dtype == "bf16"), ora["Y"], y_dtype == "bf16", f"{w.name} Y aligned={aligned}")
                assert torch.equal(Y, Yq)
        assert all(torch.equal(a, b) for a, b in zip(*acts)), "codes depend on the alignment of X"
        plan.destroy()


# ---- the quantizers by lanes read X in 16-byte words wherever it lies: the same bits from an X one element off the 16-byte grid
OFF_GRID = [_lanes(544, levels=4, k_hi=8, x_dtype="bf16"), _lanes(4128), _lanes(8224, x_dtype="bf16"), _lanes(1184, levels=7, k_hi=16, x_dtype="bf16"),
            _lanes2(288, 3, 16, 16, 4, x_dtype="bf16"), _lanes2(160, 2, 16, 16, 16), _rows(1056, 1030, 1, 7, x_dtype="bf16"), _rows(544, 300, 2, 5),
            _rows(16416, 5, 3, 2, x_dtype="bf16"), _rows(96, 20, 3, 5, x_dtype="bf16"), _rows(96, 20, 3, 5)]


@pytest.mark.parametrize("w", OFF_GRID, ids=[w.name for w in OFF_GRID])
def test_quantizers_by_lanes_off_the_16_byte_grid(w):
    import torch
    import paper_2510_26771_amd as st
    inp = tl.make_inputs(w)
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda())
    tl.check_routes(plan, w, ("direct",))
    X = tl.to_device_x(inp, w)
    buf = torch.zeros(X.numel() + 16, dtype=X.dtype, device="cuda")
    buf[1:X.numel() + 1] = X.reshape(-1)
    off = buf[1:X.numel() + 1].view(X.shape)
    assert off.data_ptr() % 16 == X.element_size()
    out = []
    for x in (X, off):
        Y = torch.empty((w.batch, w.seq_len, w.d_out), dtype=torch.float32, device="cuda")
        plan.linear_forward(x, Y, plan.alloc_workspace())
        out.append(Y)
    torch.cuda.synchronize()
    assert torch.equal(*out)
    plan.destroy()


# ---- blocks in parts of 8 tokens: every block length, 16 to 512 sums per sequence, depths that end inside a thread's 16 sums, at them
# and above, channels that leave the last workgroup partly empty, sequences beside each other, 8-bit rows in tiles and not
def _parts(s, levels, k, d=192, **kw):
    return _wl(f"parts_s{s}_l{levels}_k{k}_d{d}", seq_len=s, levels=levels, k_hi=k, d_in=d, d_out=kw.pop("d_out", 68), seed=750 + s + d, **kw)


PARTS = [_parts(128, 7, 8, x_dtype="bf16"), _parts(128, 7, 2, batch=2, d=224, act_quant="asym", mean_shift=0.4), _parts(256, 8, 8, d=544),
         _parts(256, 5, 16, batch=2, x_dtype="bf16"), _parts(512, 9, 8, act_quant="asym", mean_shift=0.4, x_dtype="bf16"), _parts(512, 6, 32, batch=3),
         _parts(1024, 10, 64, d=1056, x_dtype="bf16"), _parts(1024, 7, 64), _parts(2048, 11, 64, d=544, act_quant="asym"),
         _parts(2048, 7, 32, d=256), _parts(4096, 12, 64, x_dtype="bf16"), _parts(4096, 8, 64, d=224, act_quant="asym", mean_shift=0.4),
         _parts(256, 8, 8, d=8192, x_dtype="bf16"), _parts(1024, 10, 32, d=576, d_out=8450, x_dtype="bf16"), _parts(4096, 12, 64, d=224, d_out=4098),
         _parts(256, 8, 8, d=160, x_dtype="bf16"), _parts(1024, 10, 16, d=96, batch=3, act_quant="asym", mean_shift=0.5), _parts(512, 9, 8, d=64, batch=2),
         _parts(2048, 11, 64, d=512, batch=2, d_out=768, x_dtype="bf16")]


@pytest.mark.parametrize("w", PARTS, ids=[w.name for w in PARTS])
def test_blocks_in_parts(w):
    import torch
    import paper_2510_26771_amd as st
    tl.full_case(w, with_bias=True, check_unfused=False, engines=("fp6",), routes=("parts", "direct"))
    # the same codes as the quantizer of whole blocks: the same output bit for bit, with the 8-bit rows in either GEMM
    inp = tl.make_inputs(w)
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda())
    X = tl.to_device_x(inp, w)
    out = []
    for hi_rows in (0, 2):
        plan.set_choice("hi_rows", hi_rows)
        for packed in (0, 1):
            plan.set_choice("operands", packed)
            tl.check_routes(plan, w, ("-parts",) if packed else ("parts",))
            Y = torch.empty((w.batch, w.seq_len, w.d_out), dtype=torch.float32, device="cuda")
            plan.linear_forward(X, Y, plan.alloc_workspace())
            out.append(Y)
    torch.cuda.synchronize()
    assert all(torch.equal(out[0], o) for o in out[1:])
    plan.destroy()


@pytest.mark.parametrize("w", [_parts(512, 9, 8, d=512, d_out=512), _parts(4096, 12, 64, d=1024, d_out=1024)], ids=lambda w: w.name)
def test_parts_after_a_layout_under_the_int8_engine(w):
    """A plan that was laid out again while the other engine was selected gives what a new one gives, in the same workspace."""
    import torch
    import paper_2510_26771_amd as st
    inp = tl.make_inputs(w)
    X, out = tl.to_device_x(inp, w), []
    for relaid in (False, True):
        plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda())
        if relaid:
            plan.set_gemm_engine("int8")
            plan.set_unfused(False)
            plan.set_gemm_engine("fp6")
        tl.check_routes(plan, w, ("parts", "hi_in_tiles"))
        n = plan.workspace_bytes()
        ws = torch.full((n + 65536,), 0x5A, dtype=torch.uint8, device="cuda")
        Y = torch.empty((w.batch, w.seq_len, w.d_out), dtype=torch.float32, device="cuda")
        plan.linear_forward(X, Y, ws[:n])
        torch.cuda.synchronize()
        assert (ws[n:] == 0x5A).all(), "writes behind the workspace"
        out.append((n, Y))
        plan.destroy()
    assert out[0][0] == out[1][0] and torch.equal(out[0][1], out[1][1])


# ---- the 8-bit rows in the tiles of the 4-bit rows' GEMM: every block length, sub-trees above, below and beside the tile's, several
# sequences per tile, partial depths, 4-bit sums beside 8-bit ones, the token left out in its own tile and in the next, a
# last tile that is partly empty, grids; against the oracle, and bit for bit against the rows' own kernel.  (Codes that were
# converted need room for the operand beside them, blocks of 64 tokens d_out accordingly: r6_one, r6_own.)
def _hit(name, **kw):
    base = dict(d_in=160, d_out=132, k_hi=8, seed=700 + len(name))
    base.update(kw)
    return _wl("hit_" + name, **base)


HIT = [_hit("r3_own", batch=3, seq_len=512, levels=3, k_hi=20, x_dtype="bf16"), _hit("r3_all", seq_len=256, levels=3, k_hi=32),
       _hit("r3_two_sequences_a_tile", batch=5, seq_len=64, levels=6, k_hi=8), _hit("r3_partial", batch=3, seq_len=64, levels=5, k_hi=8, act_quant="asym"),
       _hit("r4_full", batch=3, seq_len=1024, levels=10, k_hi=64, act_quant="asym", mean_shift=0.4), _hit("r4_k256", seq_len=4096, levels=12, k_hi=256, x_dtype="bf16"),
       _hit("r4_partial", batch=2, seq_len=1024, levels=8, k_hi=64), _hit("r4_below_tile", batch=2, seq_len=512, levels=6, k_hi=32),
       _hit("r5_full", batch=2, seq_len=1024, levels=10, k_hi=32, x_dtype="bf16"), _hit("r5_tiles_and_more", seq_len=256, levels=8, k_hi=8, d_out=700),
       _hit("r6_full", batch=2, seq_len=2048, levels=11, k_hi=32, d_in=416), _hit("r6_one", batch=3, seq_len=64, levels=6, k_hi=1, d_out=700),
       _hit("r6_own", batch=2, seq_len=1024, levels=6, k_hi=5, d_out=700, act_quant="asym", mean_shift=0.4),
       _hit("grid4", batch=3, seq_len=256, grid_h=16, grid_w=16, xform="haar2d", levels=2, k_hi=16, corr_len=4.0),
       _hit("grid8_own", batch=2, seq_len=1024, grid_h=32, grid_w=32, xform="haar2d", levels=3, k_hi=7, corr_len=4.0, x_dtype="bf16"),
       _rag(3, 1000, 1, k_hi=17, d_out=131), _rag(3, 1000, 1, k_hi=16, d_out=130, batch=2), _rag(3, 401, 1, k_hi=9, batch=3, act_quant="asym", mean_shift=0.3),
       _rag(4, 402, 1, k_hi=20, batch=3, x_dtype="bf16"), _rag(5, 999, 0, k_hi=32, batch=2), _rag(6, 1500, 1, k_hi=3, d_out=65),
       # codes converted by 16 places a tile: more than 512 channels, with and without top levels
       _hit("r5_wide", batch=2, seq_len=1024, levels=10, k_hi=32, d_in=608, d_out=700), _hit("r4_wide_own", batch=3, seq_len=512, levels=4, k_hi=9, d_in=576)]


HIT_NO_ROOM_Q = ("hit_r6_full", "hit_grid8_own")  # linear_forward_q runs the rows' own kernel


@pytest.mark.parametrize("w", HIT, ids=[w.name for w in HIT])
def test_8bit_rows_in_the_tiles(w):
    import torch
    import paper_2510_26771_amd as st
    by_rule = ("hi_in_tiles", "-q_hi_in_tiles" if w.name in HIT_NO_ROOM_Q else "q_hi_in_tiles")
    for y in ("f32", "bf16"):
        tl.full_case(w, with_bias=True, check_unfused=False, engines=("fp6",), y_dtype=y, routes=by_rule)
    inp = tl.make_inputs(w, with_bias=True)
    plan = st.StampPlan(tl.plan_desc_for(w, "f32"), torch.from_numpy(inp["W"]).cuda(), torch.from_numpy(inp["bias"]).cuda())
    X = tl.to_device_x(inp, w)
    q = plan.alloc_act_buffers()
    plan.quantize_act(X, *q, plan.alloc_workspace())
    out = {}
    for choice in (0, 2):  # by rule; the kernel of their own
        plan.set_choice("hi_rows", choice)
        # (the rows' own kernel takes up to 128 of a sequence through their top levels, the int8 pipeline more: same sums)
        tl.check_routes(plan, w, by_rule if choice == 0 else ("-hi_in_tiles", "-q_hi_in_tiles") + (("hi_fp6",) if w.k_hi <= 128 else ()))
        for operands in (0, 1):
            plan.set_choice("operands", operands)
            if choice == 0 and w.name not in HIT_NO_ROOM_Q:
                tl.check_routes(plan, w, by_rule)  # packed codes (operands 1) are converted as those of linear_forward_q
            Y, Yq = (torch.zeros((w.batch, w.seq_len, w.d_out), dtype=torch.float32, device="cuda") for _ in range(2))
            ws = plan.alloc_workspace()
            plan.linear_forward(X, Y, ws)
            plan.linear_forward_q(*q, Yq, ws)
            torch.cuda.synchronize()
            out[choice, operands] = (Y, Yq)
    for o in out.values():
        assert torch.equal(o[0], out[2, 1][0]) and torch.equal(o[1], out[2, 1][1]), "differs from the rows' own kernel"
    plan.destroy()


# ---- 4-bit rows' GEMM: both tile sizes (128 x 256 where that leaves fewer rounds, else 256 x 256), with one row more than a
# tile and a depth of one, two and an odd number of K steps
def _tiles(name, m, n, d, **kw):
    return _wl(name, seq_len=m, d_in=d, d_out=n, k_hi=kw.pop("k_hi", 16), seed=500 + m + n, **kw)


TILES = [_tiles("t256_ident_odd_rows", 8193, 2050, 64, xform="identity", levels=0),
         _tiles("t256_rag", 2049, 8190, 96, levels=3, skip_first=True),
         _tiles("t256_rag_odd_n", 2050, 8065, 96, levels=4, skip_first=True, act_quant="asym"),
         _tiles("t256_haar", 2048, 7938, 160, levels=11, k_hi=64),
         _tiles("t256_wht", 2048, 7938, 32, xform="wht", levels=0),
         _tiles("t256_grid", 4096, 4098, 288, xform="haar2d", grid_h=64, grid_w=64, levels=3, k_hi=64, corr_len=4.0),
         _tiles("t128_ident_rows", 257, 300, 32, xform="identity", levels=0),
         # tiles with few rows: a lane group without any, one row in the second
         _tiles("t128_ident_4_rows", 260, 300, 32, xform="identity", levels=0), _tiles("t128_ident_5_rows", 261, 300, 32, xform="identity", levels=0, act_quant="asym"),
         _tiles("t128_wht_64_rows", 64, 131, 160, xform="wht", levels=0), _tiles("t128_haar32_64_rows", 64, 131, 160, levels=6, k_hi=2),
         # 132 and 128 tiles of 256 x 256: either side of one round of half tiles
         _tiles("t256_haar_132_tiles", 1024, 8300, 416, levels=10, k_hi=32, act_quant="asym"),
         _tiles("t128_haar_128_tiles", 1024, 8180, 416, levels=10, k_hi=32, act_quant="asym"),
         _tiles("t128_grid4", 1024, 514, 160, xform="haar2d", grid_h=32, grid_w=32, levels=5, k_hi=64, corr_len=4.0)]


@pytest.mark.parametrize("w", TILES, ids=[w.name for w in TILES])
def test_both_gemm_tile_sizes(w):
    tl.full_case(w, with_bias=True, check_unfused=False, y_dtype="bf16" if w.d_out % 4 else "f32", check_acc=False,
                 routes=("tiles_128" if w.name.startswith("t128") else "-tiles_128",))


# ---- two workgroups of 128 x 256 tiles per CU: few tiles more than they hold at once (a row more than a tile, odd d_out), depths of 1, 9 and 10
# K steps, every block length, fp32 rows (WHT, a plan of blocks run level by level); and the sizes beside them that keep 256 x 256 tiles: a
# last round more than half full, one round, fp32 rows at 10 steps and beyond two rounds
PAIRS = [_tiles("pair_ident_odd", 8193, 2049, 128, xform="identity", levels=0), _tiles("pair_haar32_10_steps", 2048, 8448, 1248, levels=11, k_hi=64),
         _tiles("pair_haar8_asym", 4096, 4354, 1152, levels=3, k_hi=512, act_quant="asym"), _tiles("pair_haar16_odd", 2048, 8449, 224, levels=4, k_hi=128, act_quant="asym"),
         _tiles("pair_grid8", 4096, 4354, 96, xform="haar2d", grid_h=64, grid_w=64, levels=3, k_hi=64, corr_len=4.0),
         _tiles("pair_rag64", 2100, 8193, 160, levels=6, skip_first=True, k_hi=32),
         _tiles("pair_wht", 8192, 2306, 1120, xform="wht", levels=0, k_hi=32), _tiles("pair_wht_odd_asym", 2048, 8193, 96, xform="wht", levels=0, act_quant="asym"),
         _tiles("t256_wht_10_steps", 2048, 8193, 1184, xform="wht", levels=0), _tiles("t256_wht_more_than_two_rounds", 4096, 8200, 160, xform="wht", levels=0),
         _tiles("pair_ident_10_steps", 2048, 8450, 1184, xform="identity", levels=0, act_quant="asym"),
         _tiles("t256_last_round_full", 4096, 6900, 1184, levels=3, k_hi=64), _tiles("t256_one_round", 4096, 4096, 96, levels=3, k_hi=64)]


@pytest.mark.parametrize("w", PAIRS, ids=[w.name for w in PAIRS])
def test_pairs_of_tiles(w):
    tl.full_case(w, with_bias=True, check_unfused=False, y_dtype="bf16" if w.d_out % 4 else "f32", check_acc=False, engines=("fp6",),
                 routes=("tiles_pair" if w.name.startswith("pair") else "-tiles_pair",))


# ---- 8-bit rows' kernel: 32 rows a workgroup where 64 leave half of the CUs idle (either side of that line, a row more and less than whole
# groups), two strips of columns a workgroup (either side of one round, of three quarters of the second and of seven eighths of the first in
# shallow layers; their first depth and one K step less), with and without top levels, odd d_out, all its outputs
def _few(name, n, k, **kw):
    base = dict(xform="identity", levels=0, seq_len=k + 40, d_in=416, d_out=n, k_hi=k)
    base.update(kw)
    return _tiles("few_" + name, base.pop("seq_len"), base.pop("d_out"), base.pop("d_in"), **base)


R32, STRIPS, NEITHER = ("hi_rows_32", "-hi_two_strips"), ("hi_two_strips", "-hi_rows_32"), ("-hi_rows_32", "-hi_two_strips")
FEW = [(_few("ident_64_line", 4096, 64), R32), (_few("ident_64_above", 4097, 64), NEITHER), (_few("ident_33", 1000, 33, act_quant="asym"), R32),
       (_few("ident_31", 8300, 31), R32), (_few("ident_65_one_strip", 8301, 65, act_quant="asym"), NEITHER), (_few("wht_33", 515, 33, xform="wht", seq_len=256), R32),
       (_few("tops_128", 8256, 128, xform="haar1d", levels=10, seq_len=1024), NEITHER),
       (_few("ident_strips_one_round", 8129, 65, act_quant="asym"), STRIPS), (_few("ident_strips_above", 8201, 65, d_in=2048), NEITHER),
       (_few("ident_strips_7_8", 7105, 65), STRIPS), (_few("ident_strips_less", 7040, 65), NEITHER),
       (_few("ident_strips_first", 8257, 64, act_quant="asym", d_in=1952), STRIPS), (_few("ident_15_steps", 8257, 64, d_in=1920), NEITHER),
       (_few("ident_strips_second_round", 4129, 385, d_in=1952), STRIPS), (_few("ident_strips_second_round_less", 3072, 450, d_in=1952), NEITHER),
       (_few("wht_strips", 8258, 40, xform="wht", seq_len=64, d_in=1952), STRIPS),
       (_few("tops_strips", 12290, 64, xform="haar1d", levels=9, seq_len=512, d_in=1952), STRIPS),
       # (below half of a round of 256 x 256 tiles these rows would ride in the 4-bit rows' tiles)
       (_few("rag_strips", 10753, 64, xform="haar1d", levels=3, seq_len=800, skip_first=True, d_in=1952), STRIPS),
       (_few("rag_one_strip", 10753, 64, xform="haar1d", levels=3, seq_len=800, skip_first=True), NEITHER)]


@pytest.mark.parametrize("w,form", FEW, ids=[w.name for w, _ in FEW])
def test_rows_and_strips_of_the_8bit_rows(w, form):
    tl.full_case(w, with_bias=True, check_unfused=False, y_dtype="bf16" if w.d_out % 4 else "f32", check_acc=False, engines=("fp6",),
                 routes=("hi_fp6", "-hi_in_tiles") + form)


# ---- split channels without top levels: the bottom kernel's two passes carry the block sums' maxima too (a last split of one
# channel group, both quantizer forms, every block sum at 8 bits or only some, one block length of the packed codes)
SPLIT_TOP = [_wl("split_top_f32_asym", seq_len=64, d_in=4128, k_hi=3, act_quant="asym", mean_shift=0.5, seed=601),
             _wl("split_top_all_8bit", seq_len=128, d_in=8224, k_hi=8, levels=4, x_dtype="bf16", batch=2, seed=602),
             _wl("split_top_32_asym", seq_len=256, d_in=4640, k_hi=5, levels=5, act_quant="asym", mean_shift=-0.3, seed=603),
             _wl("split_top_grid_all", seq_len=64, d_in=8192, d_out=66, k_hi=4, levels=2, xform="haar2d", grid_h=8, grid_w=8,
                 corr_len=2.0, x_dtype="bf16", seed=604)]


@pytest.mark.parametrize("w", SPLIT_TOP, ids=[w.name for w in SPLIT_TOP])
def test_split_channels_without_top_levels(w):
    tl.full_case(w, with_bias=True)


# ---- 8 x 8 blocks of a grid: sub-blocks side by side up to 1536 channels, one after another beyond; with and without top
# levels, every block sum at 8 bits or only some, both quantizer forms and input types
def _quads(name, d, **kw):
    return _wl(name, xform="haar2d", grid_h=16, grid_w=16, seq_len=256, d_in=d, corr_len=4.0, seed=700 + d, **kw)


QUADS = [_quads("quads_1536", 1536, levels=4, k_hi=4, x_dtype="bf16"),
         _quads("quads_1536_f32_asym", 1536, levels=3, k_hi=3, act_quant="asym", mean_shift=0.5),
         _quads("quads_1568", 1568, levels=3, k_hi=4, x_dtype="bf16"),
         _quads("quads_544_few", 544, levels=3, k_hi=1, x_dtype="bf16", batch=3),
         _quads("quads_32_asym", 32, levels=4, k_hi=4, act_quant="asym", mean_shift=-0.3, x_dtype="bf16", batch=2)]


@pytest.mark.parametrize("w", QUADS, ids=[w.name for w in QUADS])
def test_grid_blocks_by_sub_blocks(w):
    tl.full_case(w, with_bias=True)
    tl.full_case(w, with_bias=True, check_unfused=False, y_dtype="bf16")


# ---- conversion of the packed codes beside the top levels: one and several row tiles and K steps, 8-bit rows that do not
# fill their operand's groups, an operand larger than the 8-bit codes it lies over, blocks on a line and on a grid
BESIDE = [_wl("beside_32", batch=2, seq_len=64, levels=6, k_hi=2, d_in=160, x_dtype="bf16", seed=801),
          _wl("beside_64_b3_asym", batch=3, seq_len=1024, levels=10, k_hi=16, d_in=32, act_quant="asym", mean_shift=0.5, seed=802),
          _wl("beside_32_b5", batch=5, seq_len=64, levels=6, k_hi=2, d_in=32, seed=803),
          _wl("beside_grid4", batch=2, seq_len=256, levels=4, k_hi=16, d_in=1568, xform="haar2d", grid_h=16, grid_w=16, corr_len=4.0,
              x_dtype="bf16", seed=804),
          _wl("beside_wide", seq_len=512, levels=9, k_hi=16, d_in=8224, x_dtype="bf16", seed=805)]


@pytest.mark.parametrize("w", BESIDE, ids=[w.name for w in BESIDE])
def test_codes_converted_beside_the_top_levels(w):
    tl.full_case(w, with_bias=True, routes=("beside_top",))
    tl.full_case(w, with_bias=True, check_unfused=False, y_dtype="bf16", routes=("beside_top",))


# ---- two streams on one plan, each with its own workspace, on the routes whose buffers lie over one another
STREAMS = [(_wl("streams_direct", batch=2, seq_len=512, levels=3, k_hi=16, d_in=256, d_out=384, x_dtype="bf16", seed=901), ("direct", "hi_fp6")),
           (_wl("streams_beside", batch=2, seq_len=2048, levels=11, k_hi=64, d_in=32, d_out=768, x_dtype="bf16", seed=902), ("beside_top",)),
           (_wl("streams_parts", batch=2, seq_len=2048, levels=11, k_hi=64, d_in=512, d_out=768, x_dtype="bf16", seed=902), ("parts",)),
           (_rag(3, 1003, 1, batch=2, d_in=256, d_out=515, x_dtype="bf16"), ("any_length_blocks", "direct")),
           (_grp(64, 3, 64, 128, 1026), ("group_blocks",)),
           (_wl("streams_dct", seq_len=1024, xform="dct", levels=0, k_hi=64, d_in=256, d_out=384, seed=903), ("hi_fp6",))]


@pytest.mark.parametrize("w,routes", STREAMS, ids=[w.name for w, _ in STREAMS])
def test_two_streams_with_distinct_workspaces(w, routes):
    import torch
    import paper_2510_26771_amd as st
    inp = tl.make_inputs(w, with_bias=True)
    plan = st.StampPlan(tl.plan_desc_for(w, "bf16"), torch.from_numpy(inp["W"]).cuda(), torch.from_numpy(inp["bias"]).cuda())
    tl.check_routes(plan, w, routes)
    X1 = tl.to_device_x(inp, w)
    X2 = X1.flip(1).contiguous()
    ws1, ws2 = plan.alloc_workspace(), plan.alloc_workspace()
    ref1, ref2 = (torch.zeros((w.batch, w.seq_len, w.d_out), dtype=torch.int16, device="cuda") for _ in range(2))
    plan.linear_forward(X1, ref1, ws1)
    plan.linear_forward(X2, ref2, ws1)
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for it in range(3):
        Y1, Y2 = torch.zeros_like(ref1), torch.zeros_like(ref1)
        torch.cuda.synchronize()
        for _ in range(4):
            plan.linear_forward(X1, Y1, ws1, stream=s1)
            plan.linear_forward(X2, Y2, ws2, stream=s2)
        torch.cuda.synchronize()
        assert torch.equal(Y1, ref1) and torch.equal(Y2, ref2), f"round {it}"
    plan.destroy()

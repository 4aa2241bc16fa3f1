"""Where the workspace of a plan holds the 8-bit rows' FP6 operand, on the host alone: it fits the room it lies in, and
neither place nor size depends on the GEMM engine that was selected when the plan was laid out."""
import ctypes as C
import random

import pytest

import paper_2510_26771_amd as st
from paper_2510_26771_amd import binding


@pytest.fixture(scope="module")
def lib():
    return st.load_library()


def _layout(lib, desc, relaid):
    out = (C.c_size_t * 5)()
    rc = lib.stamp_debug_layout(C.byref(desc.to_c()), relaid, out)
    return rc, dict(zip(("total", "routes", "off", "bytes", "room"), out))


def _haar(s, d, n, levels, k, batch=1, **kw):
    return st.PlanDesc(batch=batch, seq_len=s, d_in=d, d_out=n, levels=levels, k_hi=k, **kw)


# blocks in parts of 8 tokens whose 8-bit rows ride in the GEMM's tiles: their operand lies behind everything else, between the parts'
# sums and the scales, over the block sums; and one in which they have a kernel of their own
PARTS = [_haar(512, 512, 512, 9, 8), _haar(2048, 4096, 2048, 11, 64), _haar(4096, 1024, 1024, 12, 64), _haar(1024, 1024, 1024, 10, 64),
         _haar(2048, 4096, 11008, 11, 64)]


@pytest.mark.parametrize("desc", PARTS, ids=lambda d: f"{d.seq_len}x{d.d_in}x{d.d_out}")
def test_parts_do_not_depend_on_the_engine_of_the_layout(lib, desc):
    rc, fresh = _layout(lib, desc, 0)
    assert rc == 0 and fresh["routes"] & binding.ROUTES["parts"]
    assert _layout(lib, desc, 1) == (0, fresh)
    assert fresh["bytes"] <= fresh["room"] and fresh["off"] + fresh["bytes"] <= fresh["total"]


def _random_desc(rng):
    xform = rng.choice([st.STAMP_L_IDENTITY, st.STAMP_L_HAAR1D, st.STAMP_L_HAAR1D, st.STAMP_L_HAAR1D, st.STAMP_L_HAAR2D, st.STAMP_L_WHT, st.STAMP_L_DCT])
    kw = dict(batch=rng.choice([1, 1, 2, 3, 8, 33]), xform=xform, x_dtype=rng.randint(0, 1), y_dtype=rng.randint(0, 1), act_quant=rng.randint(0, 1),
              d_in=32 * int(2 ** rng.uniform(0, 8.6)), d_out=int(2 ** rng.uniform(0, 13.5)))
    if xform == st.STAMP_L_HAAR2D:
        side = 2 ** rng.randint(2, 6)
        kw.update(grid_h=side, grid_w=side, seq_len=side * side, levels=rng.randint(1, side.bit_length() - 1), k_hi=rng.choice([1, 3, 4, 16, 64]))
    elif xform == st.STAMP_L_HAAR1D:
        s = 2 ** rng.randint(4, 12)
        if rng.random() < 0.25:  # of any length
            s += rng.randint(-s // 3, s // 3)
            kw.update(skip_first=rng.randint(0, 1), levels=rng.randint(3, 6), k_hi=rng.randint(1, 20))
        else:
            kw.update(levels=rng.randint(1, s.bit_length() - 1), k_hi=rng.choice([1, 2, 5, 8, 16, 32, 64]))
        kw["seq_len"] = s
    else:
        kw.update(seq_len=2 ** rng.randint(4, 12), levels=0, k_hi=rng.choice([0, 1, 8, 64]))
    return st.PlanDesc(**kw)


def test_operand_of_the_8bit_rows_fits_its_place(lib):
    rng = random.Random(5)
    seen, routes = 0, 0
    while seen < 4000:
        desc = _random_desc(rng)
        rc, fresh = _layout(lib, desc, 0)
        if rc:
            continue
        seen += 1
        routes |= fresh["routes"]
        assert fresh["bytes"] <= fresh["room"] and fresh["off"] + fresh["bytes"] <= fresh["total"], desc
        assert _layout(lib, desc, 1) == (0, fresh), desc
    for name in ("general", "any_length_blocks", "direct", "beside_top", "hi_fp6", "tiles_128", "hi_in_tiles", "q_hi_in_tiles", "parts"):
        assert routes & binding.ROUTES[name], name

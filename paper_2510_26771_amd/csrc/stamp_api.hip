// Host side of the C ABI declared in include/stamp.h: argument validation (always before any HIP
// call), plan construction, workspace layout and the launch sequences.
#include <cstdlib>
#include <cstring>
#include <new>

#include "stamp_internal.h"

// Scratch memory of stamp_linear_forward_static: one array per GPU, part of the loaded code object.  In host
// code this name only stands for the symbol; the device address comes from hipGetSymbolAddress (static_scratch()).
// Behind the documented size: room for the FP6 operand of up to 128 8-bit rows, at most 32 rows x 32768 channels x 1.5 bytes
// where nothing else in the workspace is large enough to hold it (place_hi6).
constexpr size_t kHi6Tail = (size_t)2 << 20;
static __device__ __align__(256) unsigned char scratch[STAMP_STATIC_SCRATCH_BYTES + kHi6Tail];

namespace {

// device address of `scratch` on the current device, looked up once per device
stamp_status_t static_scratch(void** out) {
  static void* ptr[kStampMaxDevices] = {};
  static std::mutex mu;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kStampMaxDevices) return STAMP_ERR_DEVICE;
  std::lock_guard<std::mutex> lock(mu);
  if (ptr[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return STAMP_ERR_DEVICE;
    }
    ptr[dev] = p;
  }
  *out = ptr[dev];
  return STAMP_OK;
}

inline bool is_pow2(int64_t n) { return n >= 1 && (n & (n - 1)) == 0; }
inline int ilog2(int64_t n) { int l = 0; while ((int64_t(1) << (l + 1)) <= n) ++l; return l; }
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

int max_ragged_levels(int n) {
  int l = 0;
  while (n > 1) {
    n = (n + 1) / 2;
    ++l;
  }
  return l;
}

// Geometry of the fast path (blocks of tokens, top rows); STAMP_ERR_UNSUPPORTED when the setting has none.
stamp_status_t fast_geometry(const stamp_plan_desc_t* d, StampGeom* g, int* fused_ok, int side) {
  if (d->xform == STAMP_L_IDENTITY) {
    // tokens quantized as they are: any number of 8-bit tokens (none included), no blocks, no inverse
    if (d->batch > 65535 || (int64_t)d->batch * d->k_hi > 65535) return STAMP_ERR_UNSUPPORTED;  // grid dimensions
    g->ident = 1;
    g->R = 1;
    *fused_ok = 1;
    return STAMP_OK;
  }
  // More than 256 top rows: only where no kernel needs all top rows of a sequence in LDS at once, i.e. plans
  // without top levels (fewer 8-bit tokens than approximations).  E.g. 3 levels and 64 8-bit tokens on 4096 or 8192 tokens.
  // Blocks.  With at least as many 8-bit tokens as level-J approximations, the blocks hold seq_len / k_hi tokens
  // (the top part runs the remaining levels over the k_hi block sums).  With fewer, the blocks hold the 2^J
  // (4^J) tokens of one approximation, the top part is the approximations themselves, and those beyond the
  // first k_hi are 4-bit rows that stay with the 8-bit rows' data path (4-bit codes held as int8).
  if (d->xform == STAMP_L_HAAR1D) {
    g->is2d = 0;
    const int na = d->seq_len >> d->levels;
    if (d->k_hi >= na) {
      if (d->k_hi < 1 || !is_pow2(d->k_hi)) return STAMP_ERR_UNSUPPORTED;
      g->k = g->khi = d->k_hi;
    } else {
      g->k = na;
      g->khi = d->k_hi;
    }
    if (g->k > 256 && d->k_hi >= na) return STAMP_ERR_UNSUPPORTED;
    g->R = d->seq_len / g->k;
    g->r = ilog2(g->R);
    if (g->r < 3 || g->r > 7) return STAMP_ERR_UNSUPPORTED;
    *fused_ok = g->r <= 6;
  } else {
    const int sa = side >> d->levels;  // approximations per grid side
    if (d->k_hi >= sa * sa) {
      const int lk = ilog2(d->k_hi);
      if (d->k_hi < 1 || !is_pow2(d->k_hi) || lk % 2 != 0) return STAMP_ERR_UNSUPPORTED;  // k must be a power of four
      g->G = 1 << (lk / 2);
      g->k = g->khi = d->k_hi;
    } else {
      g->G = sa;
      g->k = sa * sa;
      g->khi = d->k_hi;
    }
    if (g->k > 256 && d->k_hi >= sa * sa) return STAMP_ERR_UNSUPPORTED;
    g->is2d = 1;
    g->R = d->seq_len / g->k;
    g->g = side / g->G;
    g->r = ilog2(g->g);
    g->gridW = d->grid_w;
    if (g->r < 2 || g->r > 3) return STAMP_ERR_UNSUPPORTED;
    *fused_ok = 1;
  }
  g->L = g->J - g->r;
  // batch and batch * (top rows) are grid dimensions y / z of the transform and inverse kernels
  if (d->batch > 65535 || (int64_t)d->batch * g->k > 65535) return STAMP_ERR_UNSUPPORTED;
  return STAMP_OK;
}

stamp_status_t validate(const stamp_plan_desc_t* d, StampGeom* g, int* fused_ok, StampGen* gen) {
  memset(gen, 0, sizeof(*gen));
  if (d->batch < 1 || d->seq_len < 1 || d->d_in < 1 || d->d_out < 1) return STAMP_ERR_SHAPE;
  if (d->xform < STAMP_L_IDENTITY || d->xform > STAMP_L_DCT) return STAMP_ERR_SHAPE;
  if (d->skip_first != 0 && d->skip_first != 1) return STAMP_ERR_SHAPE;
  if (d->skip_first && (d->xform != STAMP_L_HAAR1D || d->seq_len < 2)) return STAMP_ERR_SHAPE;  // defined for the 1-D Haar transform
  if (d->bias_mode != 0 && d->bias_mode != 1) return STAMP_ERR_SHAPE;
  if (d->group_size < 0) return STAMP_ERR_SHAPE;
  if (d->k_hi < 0 || d->k_hi > d->seq_len) return STAMP_ERR_SHAPE;
  if (d->bits_hi < 2 || d->bits_hi > 8 || d->bits_lo < 2 || d->bits_lo > 8 || d->bits_w < 2 || d->bits_w > 8)
    return STAMP_ERR_SHAPE;
  if (d->d_in % 2 != 0) return STAMP_ERR_SHAPE;
  for (int32_t t : {d->x_dtype, d->y_dtype, d->w_dtype})
    if (t != STAMP_F32 && t != STAMP_BF16) return STAMP_ERR_SHAPE;
  if (d->w_is_out_by_in != 0 && d->w_is_out_by_in != 1) return STAMP_ERR_SHAPE;
  if (d->act_quant != STAMP_ACT_SYMMETRIC && d->act_quant != STAMP_ACT_ASYMMETRIC) return STAMP_ERR_SHAPE;
  if ((int64_t)d->batch * d->seq_len > (int64_t)1 << 30) return STAMP_ERR_SHAPE;

  int J = 0, side = 0;
  const bool ragged = d->xform == STAMP_L_HAAR1D && (d->skip_first || !is_pow2(d->seq_len));
  if (ragged) {
    if (d->levels < 0 || d->levels > max_ragged_levels(d->seq_len - d->skip_first)) return STAMP_ERR_SHAPE;
  } else if (d->xform == STAMP_L_WHT) {
    if (!is_pow2(d->seq_len) || d->levels != 0) return STAMP_ERR_SHAPE;
  } else if (d->xform == STAMP_L_DCT) {
    if (d->levels != 0) return STAMP_ERR_SHAPE;
  } else if (d->xform == STAMP_L_HAAR1D) {
    J = ilog2(d->seq_len);
    if (d->levels < 1 || d->levels > J) return STAMP_ERR_SHAPE;
  } else if (d->xform == STAMP_L_HAAR2D) {
    if (d->grid_h < 1 || d->grid_w < 1 || (int64_t)d->grid_h * d->grid_w != d->seq_len) return STAMP_ERR_SHAPE;
    if (!is_pow2(d->grid_h) || !is_pow2(d->grid_w)) return STAMP_ERR_SHAPE;
    side = d->grid_h < d->grid_w ? d->grid_h : d->grid_w;
    J = ilog2(side);
    if (d->levels < 1 || d->levels > J) return STAMP_ERR_SHAPE;
  } else if (d->levels != 0) {
    return STAMP_ERR_SHAPE;  // no transform, no levels
  }

  // ---- valid STaMP settings from here on; what follows is what this library implements ----
  if (d->bits_hi != 8 || d->bits_lo != 4 || d->bits_w != 4) return STAMP_ERR_UNSUPPORTED;
  if (d->d_in % 32 != 0 || d->d_in > 32768) return STAMP_ERR_UNSUPPORTED;  // wider than one workgroup holds: channel splits, two passes
  if (d->d_out > (1 << 21)) return STAMP_ERR_UNSUPPORTED;  // the GEMM epilogues address a tile's 256 output rows with 32-bit byte offsets
  memset(g, 0, sizeof(*g));
  g->B = d->batch; g->s = d->seq_len; g->d = d->d_in; g->N = d->d_out;
  g->J = d->levels; g->k = g->khi = d->k_hi;
  g->x_bf16 = d->x_dtype == STAMP_BF16;
  g->y_bf16 = d->y_dtype == STAMP_BF16;
  g->asym = d->act_quant == STAMP_ACT_ASYMMETRIC;
  // ---- the fast path's geometry, where the setting has one ----
  const bool rect2d = d->xform == STAMP_L_HAAR2D && d->grid_h != d->grid_w;  // the fast path takes square grids only
  bool need_general = ragged || rect2d || d->xform == STAMP_L_WHT || d->xform == STAMP_L_DCT || d->bias_mode == 1 || d->group_size != 0;
  if (!need_general) {
    const stamp_status_t fs = fast_geometry(d, g, fused_ok, side);
    if (fs == STAMP_OK) return STAMP_OK;
    // a valid setting outside the fast path's block structure (block sizes, more than 256 top rows, an 8-bit token
    // count that is not a power of two, ...): the general path takes it
    need_general = true;
    memset(g, 0, sizeof(*g));
    g->B = d->batch; g->s = d->seq_len; g->d = d->d_in; g->N = d->d_out;
    g->k = g->khi = d->k_hi;
    g->x_bf16 = d->x_dtype == STAMP_BF16;
    g->y_bf16 = d->y_dtype == STAMP_BF16;
    g->asym = d->act_quant == STAMP_ACT_ASYMMETRIC;
  }
  // ---- general path: transforms without the fast path's block structure, transformed bias, per-block scales ----
  if (d->group_size != 0 && d->group_size != 64) return STAMP_ERR_UNSUPPORTED;
  if (d->group_size == 64 && (d->d_in % 64 != 0 || g->asym)) return STAMP_ERR_UNSUPPORTED;
  if (d->seq_len > 65535 || d->batch > 65535 || (int64_t)d->batch * d->k_hi > 65535) return STAMP_ERR_UNSUPPORTED;  // grid dimensions
  if (d->xform == STAMP_L_DCT && d->seq_len > 16384) return STAMP_ERR_UNSUPPORTED;  // dense s x s matrix in fp64
  gen->kind = ragged ? kGenHaarRagged
              : d->xform == STAMP_L_WHT ? kGenWht
              : d->xform == STAMP_L_DCT ? kGenDct
              : d->xform == STAMP_L_HAAR1D ? kGenHaarClassic
              : d->xform == STAMP_L_HAAR2D ? kGenHaar2d : kGenCopy;
  gen->levels = d->levels;
  gen->skip = d->skip_first;
  gen->group = d->group_size;
  gen->bias_mode = d->bias_mode;
  gen->gridH = d->grid_h;
  gen->gridW = d->grid_w;
  // the quantizer and the GEMM see the transformed tokens as rows: physical row = STaMP slot, no blocks
  g->J = 0;
  g->ident = 1;
  g->R = 1;
  if (d->group_size == 64) g->k = d->seq_len;  // every token's codes travel as int8 (khi of them are 8-bit rows)
  *fused_ok = 0;
  return STAMP_OK;
}

// Per-block scales on a 2-D Haar transform with the fast path's block structure (4 x 4 or 8 x 8 token blocks; top levels over
// at most 8 x 8 block sums, which a lane of their kernel holds), even d_out (the epilogue stores pairs), bias after the
// inverse.  Everything else runs level by level, and so do small layers: the quantizer by blocks, level by level against this
// form (whole layers, microseconds), with top levels, 1024 tokens 512 -> 512 27.6, 35.0; 4608 -> 1152 90.6, 96.1; 2048 tokens
// 896 -> 1608 (112 tiles of 256 x 128) 43.1, 43.9; 1024 tokens 1152 -> 4608 (144) 52.5, 47.0; without, 4096 tokens 512 -> 512
// (64) 37.6, 29.2.
// The GEMM with the inverse in its epilogue needs tiles for the CUs, as every tile walks its whole depth, and d_out that is
// worth the conversion of all codes.  linear_forward_q, level by level against this form: 1152 channels, 8192 tokens 512 outputs
// (128 tiles) 31.7, 36.6, 768 (192) 39.7, 36.3; 4096 tokens 1024 (128) 35.3, 34.7; 2048 tokens 2304 (144) 40.6, 35.0; 4 x 4 blocks,
// 16384 tokens 384 (192) 37.3, 40.0, 512 (256) 41.5, 40.7; one column of tiles: 81920 tokens 112 (320) 59, 69.
void grp_geometry(stamp_plan* p) {
  const stamp_plan_desc_t& d = p->desc;
  p->grp_quant = p->grp = 0;
  if (p->gen.kind != kGenHaar2d || p->gen.group != 64 || p->gen.bias_mode != 0 || d.grid_h != d.grid_w || d.d_out % 2 != 0) return;
  StampGeom g = p->geom;
  g.J = d.levels;
  g.k = g.khi = d.k_hi;
  g.ident = 0;
  int fused = 0;
  if (fast_geometry(&d, &g, &fused, d.grid_h) != STAMP_OK || !fused) return;
  if (g.L > 0 && g.k > 64) return;
  if (g.s % 64 != 0 || g.khi < 1) return;
  const int64_t rows = (int64_t)g.B * g.s, mt = (rows + 255) / 256, tiles = mt * ((d.d_out + 127) / 128);
  if (mt * ((d.d_out + 255) / 256 * 2) < 128 && (g.L > 0 || rows < 4096)) return;
  p->bgeom = g;
  p->grp_quant = 1;
  p->grp = d.d_out > 128 && (tiles >= (g.R == 16 ? 256 : 192) || (tiles >= 128 && d.d_out >= 1024));
}

// Blocked form of a plan of the general path (1-D Haar of any length): per-token scales, bias after the inverse, 3 to 6
// levels (blocks of 8 .. 64 tokens: what the GEMM epilogues invert), 8-bit tokens among the approximations (and the
// token left out, which has to be one of them).  Everything else runs level by level.
void rag_geometry(stamp_plan* p) {
  const StampGeom& g = p->geom;
  const StampGen& gn = p->gen;
  p->rag = StampRag{};
  if (gn.kind != kGenHaarRagged || gn.group != 0 || gn.bias_mode != 0 || gn.levels < 3 || gn.levels > 6) return;
  StampRag r = {};
  r.o = gn.skip;
  r.n = g.s - r.o;
  r.r = gn.levels;
  r.nb = (r.n + (1 << r.r) - 1) >> r.r;
  r.mlast = r.n - ((r.nb - 1) << r.r);
  if (g.khi < 1 || g.khi > r.o + r.nb) return;
  if (((int64_t)g.B * r.nb << r.r) > (int64_t)1 << 30) return;
  r.on = 1;
  p->rag = r;
  p->bgeom = g;
  p->bgeom.ident = 0;
  p->bgeom.J = p->bgeom.r = r.r;
  p->bgeom.R = 1 << r.r;
  p->bgeom.k = r.nb;
}

// Where the 8-bit rows' FP6 operand lies: over a region that is free by then, or (a dozen rows or fewer, the operand is padded
// to 32; narrow layers, padded to 128 channels) behind everything else.  stamp_linear_forward_static keeps taking the plans
// whose workspace without it fits: beyond kHi6Tail it must not push them out.
void place_hi6(stamp_plan* p, size_t region, size_t room) {
  const size_t base = p->ws_base;
  p->ws_total = base;
  for (int own = 0; own < 2; ++own) {
    if (!p->hi6[own]) continue;
    const size_t need = stamp_hi6_bytes(p, own);
    if (need <= room) continue;
    if (need > kHi6Tail && base <= STAMP_STATIC_SCRATCH_BYTES && align256(base + need) > STAMP_STATIC_SCRATCH_BYTES) p->hi6[own] = 0;
    else if (p->ws_total < align256(base + need)) p->ws_total = align256(base + need);
  }
  p->ws_hi6 = p->ws_total > base ? base : region;
}

// Blocks of 16 tokens and more below top levels, quantized in parts of 8 (stamp_lanes1d.hip): the sums of the parts lie from the
// quantizer's scratch on over the packed codes, which that form does not have; the 8-bit rows' operand (ws_parts_hi, 0: not
// this form) behind them, over the block sums' parts and P where the tiles take the 8-bit rows along, or behind everything.
// A block's workgroup takes its tokens one after the other: with few blocks that chain is what a layer waits for; the sums of the
// parts are 4 bytes per channel and 8 tokens more, twice, which is what counts with many.  Layers, us, whole blocks against
// parts.  Blocks of 64: 4096 x 64 42.1, 23.4, x 1024 50.3, 31.5, x 4096 73.6, 56.0, 2 x 4096 x 4096 78.2, 75.7, 8 x 4096 x 1024 68.6, 62.8, 4 x
// 4096 x 4096 88.1, 114.6; of 32: 256 x 160 26.5, 20.4, 512 x 1024 40.6, 24.1, 2 x 2048 x 512 34.3, 25.6, 2048 x 4096 56.2, 48.2, 4 x 2048 x 2048
// 46.5, 45.4, 4 x 2048 x 4096 65.7, 75.5; of 16: 1024 x 128 23.0, 20.1, 2 x 1024 x 4096 48.2, 44.7, 16 x 1024 x 4096 101.5, 103.2.  So up to
// 2^24 elements, 2^25 in blocks of 64.  The chain of a block of 16 is short: of narrow layers of many short sequences (more than
// 128 blocks, at most 32 a sequence, below 512 channels) its workgroups fill the CUs without parts, 64 x 256 x 128 23.5, 25.3, 64 x 128
// x 96 20.6, 22.3, but 256 x 128 x 512 39.6, 35.0.  Beyond 2^24 elements parts need a launch to save, which those whose 8-bit rows ride in
// the tiles have not: with more than 128 blocks whole blocks from 2048 tokens on, and of fp32 (256 outputs, 8 x 2048 x 2048 bf16 57.6,
// 63.3, fp32 62.0, 73.3, 16 x 1024 x 2048 fp32 61.7, 67.9; 16 x 1024 x 2048 bf16 58.0, 58.2, 32 x 512 x 2048 59.3, 55.6).
// 1657 such pairs (128 .. 4096 tokens, 64 .. 8192 channels): 0.3 % above always taking the better one on average, 13 % at worst.
void place_parts(stamp_plan* p) {
  const StampGeom& g = p->geom;
  p->ws_parts_hi = 0;
  const int64_t elems = (int64_t)g.B * g.s * g.d;
  if (elems > (g.r >= 6 ? 1 << 25 : 1 << 24)) return;
  if (g.r == 4 && g.B * g.k > 128 && g.k <= 32 && g.d < 512) return;
  if (g.ident || g.is2d || g.L == 0 || g.r < 4 || g.r > 6 || g.s < 128 || g.s > 4096 || g.d > 8192 || !stamp_lanes1d_fits(p, 3)) return;
  const StampHiTiles ht = p->parts_tiles = stamp_hi_tiles(p, 0);
  if (!ht.on && !p->hi6[0]) return;
  if (ht.on && elems > 1 << 24 && g.B * g.k > 128 && (g.s >= 2048 || !g.x_bf16)) return;
  const size_t end = p->ws_abot + align256((size_t)g.B * (g.s / 8) * g.d * sizeof(float));
  const size_t hi = ht.on ? stamp_hi_tiles_bytes(p) : stamp_hi6_bytes(p, 0);
  if (end > p->ws_scales) return;
  if (end + hi <= p->ws_scales) {
    p->ws_parts_hi = end;
  } else if (ht.on && hi <= p->ws_a6 - p->ws_ythi) {
    p->ws_parts_hi = p->ws_ythi;
  } else if (p->ws_base > STAMP_STATIC_SCRATCH_BYTES || align256(p->ws_base + hi) <= STAMP_STATIC_SCRATCH_BYTES) {
    p->ws_parts_hi = p->ws_base;
    if (p->ws_total < align256(p->ws_base + hi)) p->ws_total = align256(p->ws_base + hi);
  }
}

void layout_workspace(stamp_plan* p) {
  const StampGeom& g = p->geom;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align256(off + bytes); return o; };
  if (p->gen.kind != kGenNone) {
    // general path: three fp32 copies of the activation and of the transformed output for the level kernels, and
    // the quantized activation (per-token scales: the buffers of the fast path; per-block scales: int8 codes)
    const bool grouped = p->gen.group != 0;
    p->ws_abot = p->ws_rowmax = p->ws_gpart = p->ws_P = p->ws_ytlo = 0;
    p->ws_qhi = take(grouped ? 0 : (size_t)g.B * g.k * g.d);
    p->ws_qlo = take(grouped ? 0 : (size_t)p->Mpad * (p->Kpad / 2));
    p->ws_scales = take(grouped ? 0 : (size_t)2 * g.B * g.s * sizeof(float));
    p->ws_ythi = take(grouped ? 0 : (size_t)p->hi_ksplit * g.B * g.k * g.N * sizeof(float));
    p->ws_a6 = take(grouped ? 0 : stamp_a6_bytes(p));
    for (size_t& o : p->ws_T) o = take((size_t)g.B * g.s * g.d * sizeof(float));
    for (size_t& o : p->ws_Yt) o = take((size_t)g.B * g.s * g.N * sizeof(float));
    p->ws_codes8 = take(grouped ? (size_t)g.B * g.s * g.d : 0);
    p->ws_scalesg = take(grouped ? (size_t)g.B * g.s * (g.d / 64) * sizeof(float) : 0);
    p->ws_base = off;
    p->hi6[0] = stamp_hi6_fits(p, 0);
    p->hi6[1] = 0;
    place_hi6(p, p->ws_T[2], p->ws_Yt[0] - p->ws_T[2]);
    // the blocked form uses neither the fp32 copies of the activation nor those of the output: its rows in block order
    // lie over the former, its block sums over the latter (a plan for which they do not fit keeps the level kernels)
    p->ws_ba6 = p->ws_T[0];
    p->ws_bP = p->ws_Yt[0];
    p->direct_ok = !grouped && (g.k == 0 || (p->hi6[0] && stamp_hi6_bytes(p, 0) <= p->ws_scales - p->ws_qhi));
    if (p->rag.on && (stamp_rag_a6_bytes(p) > p->ws_T[2] - p->ws_T[0] ||
                      (size_t)g.B * g.khi * p->Npad * sizeof(float) > p->ws_codes8 - p->ws_Yt[0]))
      p->rag.on = 0;
    if (p->grp) {
      // over the fp32 copies, like the blocked 1-D form: block sums of X | operands of the 4-bit rows, then block sums of
      // the inverse | operands of the 8-bit rows
      size_t n[4];
      stamp_grp_bytes(p, n);
      const size_t xs = align256((size_t)g.B * p->bgeom.k * g.d * sizeof(float)), ys = align256((size_t)g.B * p->bgeom.k * p->Npad * sizeof(float));
      p->ws_grp[0] = p->ws_T[0] + xs;
      p->ws_grp[1] = p->ws_grp[0] + n[0];
      p->ws_grp[2] = p->ws_Yt[0] + ys;
      p->ws_grp[3] = p->ws_grp[2] + n[2];
      if (p->ws_grp[1] + n[1] > p->ws_Yt[0] || p->ws_grp[3] + n[3] > p->ws_codes8) p->grp = 0;
    }
    return;
  }
  p->ws_abot = take((size_t)g.B * g.k * g.d * sizeof(float));
  p->ws_rowmax = take((size_t)2 * g.B * g.k * ((g.d + 31) / 32) * sizeof(uint32_t));  // partial row maxima (asymmetric: of both signs) per 32-channel slice
  {
    const int nsplit = stamp_actquant_nsplit(p);
    p->ws_gpart = take(nsplit > 1 ? (size_t)2 * nsplit * g.B * g.s * sizeof(uint32_t) : 0);  // row maxima per channel split
  }
  p->ws_qhi = take((size_t)g.B * g.k * g.d);
  p->ws_qlo = take((size_t)p->Mpad * (p->Kpad / 2));
  p->ws_scales = take((size_t)2 * g.B * g.s * sizeof(float));  // scales, then offsets (asymmetric plans)
  {
    // partial rows per part of a split depth, for either set of rows the 8-bit rows' GEMM may be run over
    const size_t all = (size_t)p->hi_ksplit * g.k, own = (size_t)p->hi_ksplit_own * g.khi;
    p->ws_ythi = take((all > own ? all : own) * g.B * g.N * sizeof(float));
  }
  p->ws_P = take((size_t)g.B * g.k * p->Npad * sizeof(float));
  p->ws_a6 = take(stamp_a6_bytes(p));
  p->ws_ytlo = off;
  if (p->unfused || !p->fused_ok) take((size_t)g.B * g.s * g.N * sizeof(float));
  p->ws_base = off;
  for (int own = 0; own < 2; ++own) p->hi6[own] = stamp_hi6_fits(p, own);
  place_hi6(p, p->ws_abot, p->ws_qhi - p->ws_abot);  // over the quantizer's scratch
  // written by the quantizer itself it lies over the packed codes, which are not used then
  const size_t room = p->ws_scales - p->ws_qhi;
  p->direct_ok = (g.ident && g.k == 0) || ((p->hi6[0] || p->hi6[1]) && stamp_hi6_bytes(p, 0) <= room && stamp_hi6_bytes(p, 1) <= room);
  place_parts(p);
}

// everything of a new plan that needs no device
void init_plan(stamp_plan* p, const stamp_plan_desc_t* desc, const StampGeom& g, int fused_ok, const StampGen& gen) {
  memset(p, 0, sizeof(*p));
  p->desc = *desc;
  p->geom = g;
  p->gen = gen;
  p->fused_ok = fused_ok && (g.ident || g.N % 2 == 0);  // the fused inverse stores pairs of columns: even d_out
  p->unfused = 0;
  p->engine = STAMP_GEMM_FP6;
  p->Kpad = ((g.d + 127) / 128) * 128;
  p->Npad = ((g.N + 255) / 256) * 256;
  p->Mpad = ((g.B * g.s + 255) / 256) * 256;
  p->hi_ksplit = gen.group ? 1 : stamp_hi_ksplit(p, g.k);
  p->hi_ksplit_own = gen.group ? 1 : stamp_hi_ksplit(p, g.khi);
  rag_geometry(p);
  grp_geometry(p);
  layout_workspace(p);
}

inline bool ws_ok(const stamp_plan* p, const void* ws, size_t bytes, size_t need) {
  (void)p;
  return ws != nullptr && (reinterpret_cast<uintptr_t>(ws) & 255) == 0 && bytes >= need;
}

inline uint8_t* at(void* ws, size_t off) { return reinterpret_cast<uint8_t*>(ws) + off; }

// Plans without top levels that keep only some of the block sums at 8 bits (0 < khi < k), default route (FP6
// engine, fused inverse): the 4-bit block sums are rows of the 4-bit rows' GEMM (the quantizer has put their packed
// codes at coefficient 0 of their blocks), and the 8-bit rows' GEMM runs over the first khi rows of every sequence only.
inline bool own_top(const stamp_plan* p) {
  const StampGeom& g = p->geom;
  return p->gen.kind == kGenNone && !g.ident && g.L == 0 && g.khi > 0 && g.khi < g.k && p->engine == STAMP_GEMM_FP6 &&
         p->fused_ok && !p->unfused;
}

// block sums of the first khi blocks of every sequence -> P [B * khi][Npad]
inline hipError_t launch_block_sums_own(const stamp_plan* p, const int8_t* q_hi, const float* scales, float* ythi,
                                        float* P, const uint8_t* hi6, hipStream_t st) {
  if (p->hi6[1]) return stamp_launch_hi6(p, hi6, scales, 0, P, p->Npad, 1, nullptr, 1.0f, st);
  if (p->hi_ksplit_own <= 1) return stamp_launch_gemm_hi(p, q_hi, scales, 1, P, st, p->Npad, true);
  const hipError_t e = stamp_launch_gemm_hi(p, q_hi, scales, 1, ythi, st, 0, true);
  if (e != hipSuccess) return e;
  return stamp_launch_sum_parts(ythi, p->hi_ksplit_own, p->geom.B * p->geom.khi, p->geom.N, P, p->Npad, st);
}

// Packed codes -> FP6 operands, one launch: the 8-bit rows and the 4-bit rows (q_lo given) beside them.  Where the 8-bit rows
// stay int8, the 4-bit rows are converted right before their GEMM instead (stamp_launch_repack6): the pass takes 6.8 us after the
// 8-bit rows' GEMM and 10.0 before it (16384 x 1024).
inline hipError_t convert_rows(const stamp_plan* p, const int8_t* q_hi, const uint8_t* q_lo, uint8_t* a6, int own, void* ws, hipStream_t st) {
  const StampHi6Pack hp = stamp_hi6_pack(p, q_hi, at(ws, p->ws_hi6), own, StampHiTiles{});
  return stamp_launch_repack6(p, q_lo, a6, st, &hp);
}

// Where a call keeps the FP6 operand of the 8-bit rows: its form, and what is free there.
struct HiPlace {
  StampHiTiles ht;
  size_t off, bytes, room;
};
inline size_t hi_place_bytes(const stamp_plan* p, const StampHiTiles& ht, int own) { return ht.on ? stamp_hi_tiles_bytes(p) : stamp_hi6_bytes(p, own); }

// Converted from codes: in the tiles of the 4-bit rows (ht.on: the plan takes them along and there is room) over the quantizer's
// scratch, or over the block sums and their parts, which that form does not have; else for the rows' own kernel (place_hi6).
inline HiPlace converted_place(const stamp_plan* p, int own) {
  StampHiTiles ht = p->engine == STAMP_GEMM_FP6 ? stamp_hi_tiles(p, own) : StampHiTiles{};
  const bool gen = p->gen.kind != kGenNone;
  const size_t scratch = gen ? p->ws_T[2] : p->ws_abot, room = gen ? p->ws_Yt[0] - p->ws_T[2] : p->ws_qhi - p->ws_abot;
  if (ht.on) {
    const size_t need = stamp_hi_tiles_bytes(p), ythi = gen ? 0 : p->ws_a6 - p->ws_ythi;
    if (need <= room) return {ht, scratch, need, room};
    if (need <= ythi) return {ht, p->ws_ythi, need, ythi};
    ht.on = 0;
  }
  return {ht, p->ws_hi6, stamp_hi6_bytes(p, own), p->ws_hi6 >= p->ws_base ? p->ws_total - p->ws_hi6 : room};
}
inline StampHiOut hi_operand(const stamp_plan* p, const HiPlace& place, int own, void* ws) {
  return stamp_hi6_out(p, at(ws, place.off), own, place.ht);
}
inline StampHiOut tiles_operand(const stamp_plan* p, int own, void* ws) { return hi_operand(p, converted_place(p, own), own, ws); }

// Blocked form of the 1-D Haar transform of any length (rules: rag_geometry): block sums from the 8-bit rows, then the
// 4-bit rows' GEMM with the inverse in its epilogue writes Y.  Y has to be aligned for its vector stores.
inline bool rag_route(const stamp_plan* p, const void* Y) { return p->rag.on && (reinterpret_cast<uintptr_t>(Y) & 15) == 0; }

stamp_status_t rag_forward_q(const stamp_plan* p, const int8_t* q_hi, const uint8_t* q_lo, const float* scales, void* Y, void* ws,
                             hipStream_t st, const StampDirect* dir) {
  float* ythi = reinterpret_cast<float*>(at(ws, p->ws_ythi));
  float* P = reinterpret_cast<float*>(at(ws, p->ws_bP));
  uint8_t* blk = at(ws, p->ws_ba6);
  uint8_t* hi6 = dir != nullptr ? dir->hi.p : at(ws, p->ws_hi6);
  const bool fp6 = p->engine == STAMP_GEMM_FP6;
  hipError_t e = hipSuccess;
  const StampHiOut hi = dir != nullptr ? dir->hi : tiles_operand(p, 0, ws);
  if (hi.ht.on) {
    if (dir == nullptr) {
      const StampHi6Pack hp = stamp_hi6_pack(p, q_hi, hi.p, 0, hi.ht);
      e = stamp_launch_repack6_rag(p, q_lo, blk, st, &hp);
    }
    if (e == hipSuccess) e = stamp_launch_gemm_lo6_rag(p, blk, scales, Y, nullptr, st, &hi);
    return e == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
  }
  if (p->hi6[0]) {
    if (dir == nullptr) {
      const StampHi6Pack hp = stamp_hi6_pack(p, q_hi, hi6, 0, StampHiTiles{});
      e = fp6 ? stamp_launch_repack6_rag(p, q_lo, blk, st, &hp) : stamp_launch_repack6(p, nullptr, nullptr, st, &hp);
    }
    if (e == hipSuccess) e = stamp_launch_hi6(p, hi6, scales, 3, P, p->Npad, 0, Y, stamp_haar_norm_host(p->rag.r), st);
  } else {
    e = stamp_launch_gemm_hi(p, q_hi, scales, 1, ythi, st);
    if (e == hipSuccess) e = stamp_launch_rag_top(p, ythi, p->hi_ksplit, P, Y, st);
    if (e == hipSuccess && fp6) e = stamp_launch_repack6_rag(p, q_lo, blk, st, nullptr);
  }
  if (e == hipSuccess && !fp6) e = stamp_launch_gather_lo_rag(p, q_lo, blk, st);
  if (e == hipSuccess) e = fp6 ? stamp_launch_gemm_lo6_rag(p, blk, scales, Y, P, st) : stamp_launch_gemm_lo_rag(p, blk, scales, Y, P, st);
  return e == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
}

// codes_are_ours: q_hi / q_lo were written by this library's quantizer (which also fills the rows of q_lo that
// own_top reads); buffers a caller packed need not hold them
stamp_status_t forward_q(const stamp_plan* p, const int8_t* q_hi, const uint8_t* q_lo, const float* scales, void* Y,
                         void* ws, hipStream_t st, bool codes_are_ours, const StampDirect* dir = nullptr) {
  float* ythi = reinterpret_cast<float*>(at(ws, p->ws_ythi));
  float* P = reinterpret_cast<float*>(at(ws, p->ws_P));
  if (p->grp && (reinterpret_cast<uintptr_t>(Y) & 15) == 0) {
    uint8_t* const buf[4] = {at(ws, p->ws_grp[0]), at(ws, p->ws_grp[1]), at(ws, p->ws_grp[2]), at(ws, p->ws_grp[3])};
    return stamp_launch_grp_forward(p, q_hi, scales, buf, reinterpret_cast<float*>(at(ws, p->ws_Yt[0])), Y, st) == hipSuccess
               ? STAMP_OK : STAMP_ERR_DEVICE;
  }
  if (rag_route(p, Y)) return rag_forward_q(p, q_hi, q_lo, scales, Y, ws, st, dir);
  if (p->gen.kind != kGenNone) {
    // general path: dequantized rows in STaMP order -> (transformed bias) -> inverse level by level -> Y
    float* const yt[3] = {reinterpret_cast<float*>(at(ws, p->ws_Yt[0])), reinterpret_cast<float*>(at(ws, p->ws_Yt[1])),
                          reinterpret_cast<float*>(at(ws, p->ws_Yt[2]))};
    if (p->gen.group) {
      // q_hi carries every token's int8 codes, scales one per token and 64-channel group
      if (stamp_launch_gemm_grouped(p, q_hi, scales, yt[0], st) != hipSuccess) return STAMP_ERR_DEVICE;
    } else {
      const bool lo = p->geom.k < p->geom.s, lo6 = lo && p->engine == STAMP_GEMM_FP6;
      uint8_t* a6g = at(ws, p->ws_a6);
      const bool hi6 = p->geom.k > 0 && p->hi6[0];
      if (hi6) {
        if (dir == nullptr && convert_rows(p, q_hi, lo6 ? q_lo : nullptr, a6g, 0, ws, st) != hipSuccess) return STAMP_ERR_DEVICE;
        if (stamp_launch_hi6(p, dir != nullptr ? dir->hi.p : at(ws, p->ws_hi6), scales, 2, yt[0], 0, 0, nullptr, 1.0f, st) != hipSuccess) return STAMP_ERR_DEVICE;
      } else if (p->geom.k > 0) {
        if (stamp_launch_gemm_hi(p, q_hi, scales, 1, ythi, st) != hipSuccess) return STAMP_ERR_DEVICE;
        if (stamp_launch_merge_hi(p, ythi, p->hi_ksplit, yt[0], st) != hipSuccess) return STAMP_ERR_DEVICE;
      }
      if (lo) {
        if (lo6) {
          if (dir == nullptr && !hi6 && stamp_launch_repack6(p, q_lo, a6g, st) != hipSuccess) return STAMP_ERR_DEVICE;
          if (stamp_launch_gemm_lo6(p, a6g, scales, 1, yt[0], nullptr, st) != hipSuccess) return STAMP_ERR_DEVICE;
        } else {
          if (stamp_launch_gemm_lo(p, q_lo, scales, 1, yt[0], nullptr, st) != hipSuccess) return STAMP_ERR_DEVICE;
        }
      }
    }
    const bool tbias = p->gen.bias_mode == 1 && p->bias_dev != nullptr;
    if (tbias && stamp_launch_add_ell_bias(p, yt[0], st) != hipSuccess) return STAMP_ERR_DEVICE;
    return stamp_gen_inverse(p, yt, p->geom.N, tbias ? nullptr : p->bias_dev, Y, st) == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
  }
  if (p->geom.ident) {
    // no transform: the 8-bit rows' GEMM and their output (one kernel, or partial rows and an output pass), then the
    // 4-bit rows straight to Y
    uint8_t* a6i = at(ws, p->ws_a6);
    const bool lo6 = p->geom.k < p->geom.s && p->engine == STAMP_GEMM_FP6;
    const bool hi6 = p->geom.k > 0 && p->hi6[0];
    if (hi6) {
      if (dir == nullptr && convert_rows(p, q_hi, lo6 ? q_lo : nullptr, a6i, 0, ws, st) != hipSuccess) return STAMP_ERR_DEVICE;
      if (stamp_launch_hi6(p, dir != nullptr ? dir->hi.p : at(ws, p->ws_hi6), scales, 1, Y, 0, 0, nullptr, 1.0f, st) != hipSuccess) return STAMP_ERR_DEVICE;
    } else if (p->geom.k > 0) {
      if (stamp_launch_gemm_hi(p, q_hi, scales, 1, ythi, st) != hipSuccess) return STAMP_ERR_DEVICE;
      if (stamp_launch_hi_rows_out(p, ythi, Y, st, p->hi_ksplit) != hipSuccess) return STAMP_ERR_DEVICE;
    }
    if (p->geom.k == p->geom.s) return STAMP_OK;
    if (lo6) {
      if (dir == nullptr && !hi6 && stamp_launch_repack6(p, q_lo, a6i, st) != hipSuccess) return STAMP_ERR_DEVICE;
      return stamp_launch_gemm_lo6(p, a6i, scales, 3, Y, nullptr, st) == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
    }
    return stamp_launch_gemm_lo(p, q_lo, scales, 3, Y, nullptr, st) == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
  }
  const bool fused = p->fused_ok && !p->unfused;
  const bool own = codes_are_ours && own_top(p);
  uint8_t* a6 = at(ws, p->ws_a6);
  const uint8_t* hi6 = dir != nullptr ? dir->hi.p : at(ws, p->ws_hi6);
  const bool fp6 = p->engine == STAMP_GEMM_FP6;
  const StampHiOut hi = dir != nullptr ? dir->hi : tiles_operand(p, own, ws);
  if (hi.ht.on) {
    if (dir == nullptr) {
      const StampHi6Pack hp = stamp_hi6_pack(p, q_hi, hi.p, own, hi.ht);
      if (stamp_launch_repack6(p, q_lo, a6, st, &hp) != hipSuccess) return STAMP_ERR_DEVICE;
    }
    return stamp_launch_gemm_lo6(p, a6, scales, 2, Y, nullptr, st, own, &hi) == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
  }
  if (dir == nullptr && p->hi6[own] && convert_rows(p, q_hi, fp6 ? q_lo : nullptr, a6, own, ws, st) != hipSuccess) return STAMP_ERR_DEVICE;
  if (own) {
    if (launch_block_sums_own(p, q_hi, scales, ythi, P, hi6, st) != hipSuccess) return STAMP_ERR_DEVICE;
  } else if (p->hi6[0]) {
    if (stamp_launch_hi6(p, hi6, scales, 0, P, p->Npad, 0, nullptr, 1.0f, st) != hipSuccess) return STAMP_ERR_DEVICE;
  } else if (stamp_hi_rows_are_block_sums(p)) {
    if (stamp_launch_gemm_hi(p, q_hi, scales, 1, P, st, p->Npad) != hipSuccess) return STAMP_ERR_DEVICE;
  } else if (stamp_hi_top_fused(p)) {
    if (stamp_launch_gemm_hi(p, q_hi, scales, 2, P, st, p->Npad) != hipSuccess) return STAMP_ERR_DEVICE;
  } else {
    if (stamp_launch_gemm_hi(p, q_hi, scales, 1, ythi, st) != hipSuccess) return STAMP_ERR_DEVICE;
    if (stamp_launch_inverse_top(p, ythi, 0, p->geom.N, P, p->Npad, st, p->hi_ksplit) != hipSuccess) return STAMP_ERR_DEVICE;
  }
  float* ytlo = reinterpret_cast<float*>(at(ws, p->ws_ytlo));
  if (fp6) {
    if (dir == nullptr && !p->hi6[own] && stamp_launch_repack6(p, q_lo, a6, st) != hipSuccess) return STAMP_ERR_DEVICE;
    if (stamp_launch_gemm_lo6(p, a6, scales, fused ? 2 : 1, fused ? Y : ytlo, fused ? P : nullptr, st, own) != hipSuccess)
      return STAMP_ERR_DEVICE;
  } else {
    if (stamp_launch_gemm_lo(p, q_lo, scales, fused ? 2 : 1, fused ? Y : ytlo, fused ? P : nullptr, st) != hipSuccess)
      return STAMP_ERR_DEVICE;
  }
  if (!fused && stamp_launch_inverse_bottom(p, ytlo, 0, P, p->Npad, p->geom.N, p->bias_dev, Y, st) != hipSuccess)
    return STAMP_ERR_DEVICE;
  return STAMP_OK;
}

// general path, steps 1-2: forward transform level by level, then the row quantizer
stamp_status_t gen_quantize(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, void* ws, hipStream_t st,
                            const StampDirect* dir = nullptr) {
  if (p->grp_quant && (reinterpret_cast<uintptr_t>(X) & 15) == 0)
    return stamp_launch_grp_quant(p, X, q_hi, scales, reinterpret_cast<float*>(at(ws, p->ws_T[0])), st) == hipSuccess ? STAMP_OK
                                                                                                                     : STAMP_ERR_DEVICE;
  if (stamp_rag_quantizes(p, X))
    return stamp_launch_actquant_rag(p, X, q_hi, q_lo, scales, st, dir) == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
  float* const tb[3] = {reinterpret_cast<float*>(at(ws, p->ws_T[0])), reinterpret_cast<float*>(at(ws, p->ws_T[1])),
                        reinterpret_cast<float*>(at(ws, p->ws_T[2]))};
  float* T = nullptr;
  if (stamp_gen_forward(p, X, tb, &T, st) != hipSuccess) return STAMP_ERR_DEVICE;
  const hipError_t e = p->gen.group ? stamp_launch_quant_rows_grouped(p, T, q_hi, scales, st)
                                    : stamp_launch_quant_rows_f32(p, T, q_hi, q_lo, scales, st, dir);
  return e == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
}

// stamp_linear_forward: the quantizer writes the FP6 operands itself (no packed codes, no conversion pass) on the default route:
// FP6 engine, fused inverse (or none), 8-bit rows through the kernel for few rows.  Its stores are 8 bytes of 24-byte
// fragments where packed codes are 4-byte words of whole lines; it pays while the conversion's launch counts, and where a
// workgroup stores a few neighbouring rows, not one after another (1-D blocks of 8 and 16 tokens, blocks of a grid by lanes; not 1-D
// blocks of 32, 4096 -> 11008: 102.8, 103.3).  Layers, microseconds, conversion pass against direct: 2048 tokens 4096 -> 11008, 3 levels, first token left out 96.2,
// 91.1; 3 x 777 tokens 38.3, 35.1; with 256 outputs, blocks of 8: 65536 tokens x 512 50, 46, x 1024 72, 65, 32768 x 4096 135, 132,
// 262144 x 256 110, 112, 65536 x 256 with 8192 8-bit rows 73, 81.
// Lines fitted to 1210 such pairs (256 .. 262144 rows, depth 32 .. 11008).
bool direct_pays(const stamp_plan* p) {
  const StampGeom& g = p->geom;
  const int64_t rows = (int64_t)g.B * g.s, hi = (int64_t)g.B * g.khi;
  // rows by lanes, four to a workgroup, two where d > 8192: always, however many of them are 8-bit rows (packed, direct, 256 outputs:
  // 262144 x 256 188, 75, 65536 x 1024 83, 50, 4096 x 8192 fp32 96, 75, 256 x 32 19.3, 16.0; a quarter at 8 bits, 16384 x 1024 46.0, 34.6; all,
  // 4096 x 256 18.3, 12.7, x 1024 25.9, 20.8; 408 plans from 64 rows on, none the other way); one to a workgroup, whose pieces of 16 bytes
  // meet in no line, while the output is small (2048 x 24576 156, 152, but 4096 x 24576 with 256 8-bit rows 229, 233, 2048 x 32768 fp32
  // 271, 274)
  if (g.ident && !p->rag.on) return g.d <= 16384 || rows * g.d <= (3 << 24);
  // 1-D blocks of 8 and 16 tokens by stamp_lanes1d, blocks of a grid by stamp_lanes2d (32 x 4096 x 512 92, 80): whole fragments leave in 16 and 8 bytes, at any size as fast as they can be made;
  // only many 8-bit rows cost (packed, direct: 32768 x 4096 136, 112, x 8192 310, 233, 16 x 5000 x 4096 375, 288, 262144 x 256 106, 83;
  // 128 sequences of 512 with 64 8-bit rows each, x 256 71.5, 75.5, 64 of them 51.8, 49.1, 256 with 32 each 73.6, 66.4)
  if (g.is2d || stamp_lanes1d_fits(p, p->rag.on ? p->rag.r : g.r)) return rows + 16 * hi <= 140000 || 16 * hi <= rows;
  return rows + 16 * hi <= 140000 && rows * g.d <= (1 << 27);
}
bool direct_route(const stamp_plan* p, const void* X, const void* Y) {
  const StampGeom& g = p->geom;
  if (!p->direct_ok || p->engine != STAMP_GEMM_FP6 || p->gen.group || p->dbg[STAMP_CHOICE_OPERANDS] == 1) return false;
  if (p->dbg[STAMP_CHOICE_OPERANDS] == 0 && !direct_pays(p)) return false;
  if (p->rag.on ? p->rag.r > 4 : (!g.ident && (g.is2d ? !stamp_lanes2d_fits(p) : g.r > 4 && p->ws_parts_hi == 0))) return false;
  if (p->gen.kind != kGenNone || g.ident) return !p->rag.on || (rag_route(p, Y) && stamp_rag_quantizes(p, X) && p->hi6[0]);
  if (!p->fused_ok || p->unfused) return false;
  if (own_top(p)) return p->hi6[1];
  return p->hi6[0] && (g.L > 0 || g.khi == g.k);
}

// Written by the quantizer itself the 8-bit rows' operand lies over the packed codes.
inline HiPlace direct_place(const stamp_plan* p, int own) {
  StampHiTiles ht = stamp_hi_tiles(p, own);
  const size_t room = p->ws_scales - p->ws_qhi;
  if (ht.on && stamp_hi_tiles_bytes(p) > room) ht.on = 0;
  return {ht, p->ws_qhi, hi_place_bytes(p, ht, own), room};
}
// Blocks in parts of 8 tokens: place and form are the layout's (place_parts).
inline HiPlace parts_place(const stamp_plan* p) {
  const size_t off = p->ws_parts_hi;
  return {p->parts_tiles, off, hi_place_bytes(p, p->parts_tiles, 0), (off >= p->ws_base ? p->ws_total : off >= p->ws_ythi ? p->ws_a6 : p->ws_scales) - off};
}

// stamp_linear_forward, plans with top levels whose bottom kernel leaves packed codes: their conversion shares the launch of
// the top levels, which do not need it, and the 8-bit rows' quantizer writes their operand (the layer's one conversion launch
// less: 2048 tokens 4096 -> 11008, blocks of 32, 102.5 us, now 99.4).  Measured 2 to 12 us less from 512 to 131072 tokens and
// depths of 64 to 4096; with 8192 8-bit rows, whose operand leaves in small pieces, no less at depth 256 and 5 more at 64.
bool convert_beside_top(const stamp_plan* p) {
  const StampGeom& g = p->geom;
  return p->direct_ok && p->engine == STAMP_GEMM_FP6 && p->dbg[STAMP_CHOICE_OPERANDS] != 1 && p->gen.kind == kGenNone && !g.ident && p->fused_ok && !p->unfused && g.L > 0 &&
         p->hi6[0] && (int64_t)g.B * g.k <= 4096;
}

// what stamp_linear_forward does for these tensors
struct ForwardRoute {
  bool direct, beside, parts;
  int own;
  HiPlace hi;
};
ForwardRoute forward_route(const stamp_plan* p, const void* X, const void* Y) {
  ForwardRoute r = {};
  r.own = own_top(p);
  r.direct = direct_route(p, X, Y);
  r.beside = !r.direct && convert_beside_top(p);
  r.parts = r.direct && p->ws_parts_hi != 0;
  // (beside: written when the packed codes have been converted, over them)
  r.hi = r.parts ? parts_place(p) : r.direct || r.beside ? direct_place(p, r.own) : converted_place(p, r.own);
  return r;
}

}  // namespace

extern "C" {

const char* stamp_status_string(stamp_status_t s) {
  switch (s) {
    case STAMP_OK: return "ok";
    case STAMP_ERR_NULL: return "null pointer";
    case STAMP_ERR_SHAPE: return "inconsistent shape or parameter";
    case STAMP_ERR_UNSUPPORTED: return "setting not implemented by this library";
    case STAMP_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case STAMP_ERR_ALLOC: return "device allocation failed";
    case STAMP_ERR_DEVICE: return "HIP runtime error";
  }
  return "unknown status";
}

stamp_status_t stamp_plan_create(const stamp_plan_desc_t* desc, const void* W_dev, const float* bias_dev,
                                 void* hip_stream, stamp_plan_t** out) {
  if (desc == nullptr || out == nullptr) return STAMP_ERR_NULL;
  *out = nullptr;
  StampGeom g;
  int fused_ok = 0;
  StampGen gen;
  stamp_status_t vs = validate(desc, &g, &fused_ok, &gen);
  if (vs != STAMP_OK) return vs;
  if (W_dev == nullptr) return STAMP_ERR_NULL;

  stamp_plan* p = new (std::nothrow) stamp_plan;
  if (p == nullptr) return STAMP_ERR_ALLOC;
  init_plan(p, desc, g, fused_ok, gen);

  // physical row of every STaMP slot
  p->row_of_coeff = static_cast<int32_t*>(malloc(sizeof(int32_t) * (size_t)g.s));
  if (p->row_of_coeff == nullptr) { delete p; return STAMP_ERR_ALLOC; }
  if (g.ident)
    for (int q = 0; q < g.s; ++q) p->row_of_coeff[q] = q;
  else
    for (int q = 0; q < g.k; ++q) p->row_of_coeff[q] = q * g.R;
  for (int j = 0; j < g.k && !g.ident; ++j)
    for (int e = 1; e < g.R; ++e) {
      const int slot = g.is2d ? stamp_slot_of_block_e_2d(j / g.G, j % g.G, e, g.G) : stamp_slot_of_block_e_1d(j, e, g.k);
      p->row_of_coeff[slot] = j * g.R + e;
    }

  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  uint32_t* colmax = nullptr;
  // per-block scales: the weights have a layout of their own (stamp_gen_plan_tables); the GEMM's epilogue reads (and drops) sw
  const bool per_column = gen.group == 0;
  bool ok = hipMalloc(reinterpret_cast<void**>(&p->sw_dev), sizeof(float) * p->Npad) == hipSuccess &&
            hipMalloc(reinterpret_cast<void**>(&p->colsum_dev), sizeof(float) * p->Npad) == hipSuccess &&
            hipMalloc(reinterpret_cast<void**>(&colmax), sizeof(uint32_t) * g.N) == hipSuccess;
  if (per_column)
    ok = ok && hipMalloc(reinterpret_cast<void**>(&p->qW_dev), (size_t)p->Npad * p->Kpad) == hipSuccess &&
         hipMalloc(reinterpret_cast<void**>(&p->qW6_dev), stamp_b6_bytes(p)) == hipSuccess;
  if (ok && bias_dev != nullptr) ok = hipMalloc(reinterpret_cast<void**>(&p->bias_dev), sizeof(float) * p->Npad) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    if (colmax) (void)hipFree(colmax);
    stamp_plan_destroy(p);
    return STAMP_ERR_ALLOC;
  }
  // weights given in bf16 are widened once (exactly) into a temporary that the plan-time kernels read
  const float* Wf = static_cast<const float*>(W_dev);
  float* wtmp = nullptr;
  if (desc->w_dtype == STAMP_BF16) {
    const size_t nw = (size_t)g.d * g.N;
    if (hipMalloc(reinterpret_cast<void**>(&wtmp), nw * sizeof(float)) != hipSuccess) {
      (void)hipGetLastError();
      (void)hipFree(colmax);
      stamp_plan_destroy(p);
      return STAMP_ERR_ALLOC;
    }
    Wf = wtmp;
  }
  bool dev_ok = true;
  if (wtmp != nullptr) dev_ok = stamp_launch_bf16_to_f32(W_dev, wtmp, (size_t)g.d * g.N, st) == hipSuccess;
  if (dev_ok && bias_dev != nullptr) {
    dev_ok = hipMemsetAsync(p->bias_dev, 0, sizeof(float) * p->Npad, st) == hipSuccess &&
             hipMemcpyAsync(p->bias_dev, bias_dev, sizeof(float) * g.N, hipMemcpyDeviceToDevice, st) == hipSuccess;
  }
  if (dev_ok && per_column)
    dev_ok = stamp_launch_weight_quant(p, Wf, st, colmax) == hipSuccess && stamp_launch_weight_quant6(p, Wf, colmax, st) == hipSuccess;
  if (dev_ok && !per_column)
    dev_ok = hipMemsetAsync(p->sw_dev, 0, sizeof(float) * p->Npad, st) == hipSuccess &&
             hipMemsetAsync(p->colsum_dev, 0, sizeof(float) * p->Npad, st) == hipSuccess;
  if (dev_ok && gen.kind != kGenNone) dev_ok = stamp_gen_plan_tables(p, Wf, st) == hipSuccess;
  // the scratch buffers must outlive the kernels just enqueued: hipFree waits for the device
  (void)hipFree(colmax);
  if (wtmp != nullptr) (void)hipFree(wtmp);
  if (!dev_ok) {
    stamp_plan_destroy(p);
    return STAMP_ERR_DEVICE;
  }
  *out = p;
  return STAMP_OK;
}

stamp_status_t stamp_plan_destroy(stamp_plan_t* p) {
  if (p == nullptr) return STAMP_ERR_NULL;
  if (p->qW_dev) (void)hipFree(p->qW_dev);
  if (p->qW6_dev) (void)hipFree(p->qW6_dev);
  if (p->sw_dev) (void)hipFree(p->sw_dev);
  if (p->colsum_dev) (void)hipFree(p->colsum_dev);
  if (p->bias_dev) (void)hipFree(p->bias_dev);
  stamp_gen_plan_free(p);
  free(p->row_of_coeff);
  delete p;
  return STAMP_OK;
}

size_t stamp_plan_workspace_bytes(const stamp_plan_t* p) { return p ? p->ws_total : 0; }

int32_t stamp_plan_hi_rows(const stamp_plan_t* p) { return p ? p->geom.k : 0; }

stamp_status_t stamp_plan_set_unfused(stamp_plan_t* p, int32_t unfused) {
  if (p == nullptr) return STAMP_ERR_NULL;
  if (p->gen.kind != kGenNone) return STAMP_OK;  // the general path has one implementation
  p->unfused = unfused ? 1 : 0;
  layout_workspace(p);
  return STAMP_OK;
}

stamp_status_t stamp_plan_set_gemm_engine(stamp_plan_t* p, int32_t engine) {
  if (p == nullptr) return STAMP_ERR_NULL;
  if (engine != STAMP_GEMM_INT8 && engine != STAMP_GEMM_FP6) return STAMP_ERR_UNSUPPORTED;
  p->engine = engine;
  return STAMP_OK;
}

stamp_status_t stamp_debug_set_choice(stamp_plan_t* p, int32_t choice, int32_t value) {
  if (p == nullptr) return STAMP_ERR_NULL;
  if (choice < 0 || choice >= STAMP_CHOICE_COUNT || value < 0 || value > 2) return STAMP_ERR_SHAPE;
  if (p->gen.group) return STAMP_OK;
  p->dbg[choice] = value;
  layout_workspace(p);
  return STAMP_OK;
}

int32_t stamp_debug_routes(const stamp_plan_t* p) {
  if (p == nullptr) return 0;
  const StampGeom& g = p->geom;
  const void* const aligned = reinterpret_cast<const void*>((uintptr_t)256);
  const bool own = own_top(p), rag = rag_route(p, aligned);
  int32_t r = 0;
  if (p->gen.kind != kGenNone) r |= STAMP_ROUTE_GENERAL;
  if (p->grp_quant) r |= STAMP_ROUTE_GROUP_QUANT;
  if (p->grp) r |= STAMP_ROUTE_GROUP_BLOCKS;
  if (rag) r |= STAMP_ROUTE_ANY_LENGTH_BLOCKS;
  if (p->gen.group) return r;
  const ForwardRoute fr = forward_route(p, aligned, aligned);
  if (fr.direct) r |= STAMP_ROUTE_DIRECT;
  if (fr.parts) r |= STAMP_ROUTE_PARTS;
  if (fr.beside) r |= STAMP_ROUTE_BESIDE_TOP;
  if ((own ? g.khi : g.k) > 0) {
    if (p->hi6[own]) r |= STAMP_ROUTE_HI_FP6;
    else if (!own && stamp_hi_top_fused(p)) r |= STAMP_ROUTE_HI_TOP_FUSED;
    else if ((own ? p->hi_ksplit_own : p->hi_ksplit) > 1) r |= STAMP_ROUTE_HI_SPLIT;
  }
  if (fr.hi.ht.on) r |= STAMP_ROUTE_HI_IN_TILES;
  else if ((r & STAMP_ROUTE_HI_FP6) && stamp_hi6_rows_per_workgroup(p, own) == 32) r |= STAMP_ROUTE_HI_ROWS_32;
  else if ((r & STAMP_ROUTE_HI_FP6) && stamp_hi6_two_strips(p, own)) r |= STAMP_ROUTE_HI_TWO_STRIPS;
  if (converted_place(p, 0).ht.on) r |= STAMP_ROUTE_Q_HI_IN_TILES;
  const int M = rag ? (g.B * p->rag.nb) << p->rag.r : g.B * g.s;
  if (p->engine == STAMP_GEMM_FP6 && stamp_gemm6_half_tiles(M, p->Npad)) r |= STAMP_ROUTE_TILES_128;
  const int mode = rag ? 2 : p->gen.kind != kGenNone ? 1 : g.ident ? 3 : p->fused_ok && !p->unfused ? 2 : 1;
  if (p->engine == STAMP_GEMM_FP6 && !(r & STAMP_ROUTE_TILES_128) && stamp_gemm6_pairs(M, p->Npad, p->Kpad, mode)) r |= STAMP_ROUTE_TILES_PAIR;
  return r;
}

stamp_status_t stamp_debug_layout(const stamp_plan_desc_t* desc, int32_t relaid, size_t* out) {
  if (desc == nullptr || out == nullptr) return STAMP_ERR_NULL;
  StampGeom g;
  int fused_ok = 0;
  StampGen gen;
  const stamp_status_t vs = validate(desc, &g, &fused_ok, &gen);
  if (vs != STAMP_OK) return vs;
  stamp_plan p;
  init_plan(&p, desc, g, fused_ok, gen);
  if (relaid) {
    (void)stamp_plan_set_gemm_engine(&p, STAMP_GEMM_INT8);
    (void)stamp_plan_set_unfused(&p, 0);
    (void)stamp_plan_set_gemm_engine(&p, STAMP_GEMM_FP6);
  }
  const void* const aligned = reinterpret_cast<const void*>((uintptr_t)256);
  const HiPlace hi = forward_route(&p, aligned, aligned).hi;
  out[0] = p.ws_total;
  out[1] = (size_t)stamp_debug_routes(&p);
  out[2] = hi.off;
  out[3] = hi.bytes;
  out[4] = hi.room;
  return STAMP_OK;
}

stamp_status_t stamp_plan_row_of_coeff(const stamp_plan_t* p, int32_t* host_out) {
  if (p == nullptr || host_out == nullptr) return STAMP_ERR_NULL;
  memcpy(host_out, p->row_of_coeff, sizeof(int32_t) * (size_t)p->geom.s);
  return STAMP_OK;
}

stamp_status_t stamp_quantize_act(const stamp_plan_t* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales,
                                  void* ws, size_t ws_bytes, void* hip_stream) {
  if (p == nullptr || X == nullptr || q_hi == nullptr || scales == nullptr) return STAMP_ERR_NULL;
  if (q_lo == nullptr && !p->gen.group) return STAMP_ERR_NULL;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  if (p->gen.kind != kGenNone) {
    if (!ws_ok(p, ws, ws_bytes, p->ws_total)) return STAMP_ERR_WORKSPACE;
    return gen_quantize(p, X, q_hi, q_lo, scales, ws, st);
  }
  if (!ws_ok(p, ws, ws_bytes, p->ws_qhi)) return STAMP_ERR_WORKSPACE;  // needs the block sums and row maxima only
  hipError_t e = stamp_launch_actquant(p, X, q_hi, q_lo, scales, reinterpret_cast<float*>(at(ws, p->ws_abot)),
                                       reinterpret_cast<uint32_t*>(at(ws, p->ws_rowmax)),
                                       reinterpret_cast<uint32_t*>(at(ws, p->ws_gpart)), st);
  return e == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
}

stamp_status_t stamp_linear_forward_q(const stamp_plan_t* p, const int8_t* q_hi, const uint8_t* q_lo,
                                      const float* scales, void* Y, void* ws, size_t ws_bytes, void* hip_stream) {
  if (p == nullptr || q_hi == nullptr || scales == nullptr || Y == nullptr) return STAMP_ERR_NULL;
  if (q_lo == nullptr && !p->gen.group) return STAMP_ERR_NULL;
  if (!ws_ok(p, ws, ws_bytes, p->ws_total)) return STAMP_ERR_WORKSPACE;
  return forward_q(p, q_hi, q_lo, scales, Y, ws, reinterpret_cast<hipStream_t>(hip_stream), false);
}

stamp_status_t stamp_linear_forward(const stamp_plan_t* p, const void* X, void* Y, void* ws, size_t ws_bytes,
                                    void* hip_stream) {
  if (p == nullptr || X == nullptr || Y == nullptr) return STAMP_ERR_NULL;
  if (!ws_ok(p, ws, ws_bytes, p->ws_total)) return STAMP_ERR_WORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  int8_t* q_hi = reinterpret_cast<int8_t*>(at(ws, p->ws_qhi));
  uint8_t* q_lo = at(ws, p->ws_qlo);
  float* scales = reinterpret_cast<float*>(at(ws, p->ws_scales));
  const ForwardRoute route = forward_route(p, X, Y);
  StampDirect dir = {};
  if (route.direct || route.beside) {
    dir.a6 = at(ws, p->rag.on ? p->ws_ba6 : p->ws_a6);
    dir.hi = hi_operand(p, route.hi, route.own, ws);
    dir.lo_packed = route.beside;
    dir.parts = route.parts;
  }
  const StampDirect* const dp = route.direct || route.beside ? &dir : nullptr;
  if (p->gen.kind != kGenNone) {
    if (p->gen.group) {
      q_hi = reinterpret_cast<int8_t*>(at(ws, p->ws_codes8));
      scales = reinterpret_cast<float*>(at(ws, p->ws_scalesg));
    }
    const stamp_status_t qs = gen_quantize(p, X, q_hi, q_lo, scales, ws, st, dp);
    return qs != STAMP_OK ? qs : forward_q(p, q_hi, q_lo, scales, Y, ws, st, true, dp);
  }
  hipError_t e = stamp_launch_actquant(p, X, q_hi, q_lo, scales, reinterpret_cast<float*>(at(ws, p->ws_abot)),
                                       reinterpret_cast<uint32_t*>(at(ws, p->ws_rowmax)),
                                       reinterpret_cast<uint32_t*>(at(ws, p->ws_gpart)), st, 3, dp);
  if (e != hipSuccess) return STAMP_ERR_DEVICE;
  return forward_q(p, q_hi, q_lo, scales, Y, ws, st, true, dp);
}

stamp_status_t stamp_linear_forward_static(const stamp_plan_t* p, const void* X, void* Y, void* hip_stream) {
  if (p == nullptr || X == nullptr || Y == nullptr) return STAMP_ERR_NULL;
  if (p->ws_base > STAMP_STATIC_SCRATCH_BYTES) return STAMP_ERR_WORKSPACE;  // the plan needs more than the static array holds
  void* ws = nullptr;
  const stamp_status_t ss = static_scratch(&ws);
  if (ss != STAMP_OK) return ss;
  return stamp_linear_forward(p, X, Y, ws, STAMP_STATIC_SCRATCH_BYTES + kHi6Tail, hip_stream);
}

stamp_status_t stamp_inverse(const stamp_plan_t* p, const float* Yt, int32_t n_cols, void* Y, void* ws, size_t ws_bytes,
                             void* hip_stream) {
  if (p == nullptr || Yt == nullptr || Y == nullptr) return STAMP_ERR_NULL;
  if (n_cols < 1) return STAMP_ERR_SHAPE;
  if (p->gen.kind != kGenNone) {
    // two [batch, seq_len, n_cols] fp32 buffers for the levels; Yt itself is only read
    const size_t one = align256((size_t)p->geom.B * p->geom.s * (size_t)n_cols * sizeof(float));
    if (!ws_ok(p, ws, ws_bytes, 2 * one)) return STAMP_ERR_WORKSPACE;
    hipStream_t stg = reinterpret_cast<hipStream_t>(hip_stream);
    float* const yt[3] = {const_cast<float*>(Yt), reinterpret_cast<float*>(ws), reinterpret_cast<float*>(at(ws, one))};
    const float* gbias = (n_cols == p->geom.N) ? p->bias_dev : nullptr;
    return stamp_gen_inverse(p, yt, n_cols, gbias, Y, stg) == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
  }
  if (p->geom.ident) return STAMP_ERR_UNSUPPORTED;  // nothing to invert
  const size_t need = (size_t)p->geom.B * p->geom.k * (size_t)n_cols * sizeof(float);
  if (!ws_ok(p, ws, ws_bytes, need)) return STAMP_ERR_WORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  float* P = reinterpret_cast<float*>(ws);
  if (stamp_launch_inverse_top(p, Yt, 1, n_cols, P, n_cols, st) != hipSuccess) return STAMP_ERR_DEVICE;
  const float* bias = (n_cols == p->geom.N) ? p->bias_dev : nullptr;
  if (stamp_launch_inverse_bottom(p, Yt, 1, P, n_cols, n_cols, bias, Y, st) != hipSuccess) return STAMP_ERR_DEVICE;
  return STAMP_OK;
}

stamp_status_t stamp_debug_gemm_acc(const stamp_plan_t* p, const int8_t* q_hi, const uint8_t* q_lo, int32_t* acc,
                                    void* hip_stream) {
  if (p == nullptr || q_hi == nullptr || q_lo == nullptr || acc == nullptr) return STAMP_ERR_NULL;
  if (p->gen.group) return STAMP_ERR_UNSUPPORTED;  // per-block scales: there is no single integer sum per output
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  // accumulator mode never reads the activation scales
  if (p->geom.k > 0 && stamp_launch_gemm_hi(p, q_hi, nullptr, 0, acc, st) != hipSuccess) return STAMP_ERR_DEVICE;
  if (p->engine == STAMP_GEMM_FP6) {
    // parity aid, not a timed path: the converted operand lives in a temporary of its own
    uint8_t* a6 = nullptr;
    if (hipMalloc(reinterpret_cast<void**>(&a6), stamp_a6_bytes(p)) != hipSuccess) { (void)hipGetLastError(); return STAMP_ERR_ALLOC; }
    const bool ok = stamp_launch_repack6(p, q_lo, a6, st) == hipSuccess &&
                    stamp_launch_gemm_lo6(p, a6, nullptr, 0, acc, nullptr, st) == hipSuccess;
    (void)hipFree(a6);  // waits for the kernels above
    return ok ? STAMP_OK : STAMP_ERR_DEVICE;
  }
  if (stamp_launch_gemm_lo(p, q_lo, nullptr, 0, acc, nullptr, st) != hipSuccess) return STAMP_ERR_DEVICE;
  return STAMP_OK;
}

stamp_status_t stamp_debug_run_stage(const stamp_plan_t* p, int32_t stage, const void* X, int8_t* q_hi, uint8_t* q_lo,
                                     float* scales, void* Y, void* ws, size_t ws_bytes, void* hip_stream) {
  if (p == nullptr || X == nullptr || q_hi == nullptr || q_lo == nullptr || scales == nullptr || Y == nullptr)
    return STAMP_ERR_NULL;
  if (stage < 0 || stage > 6) return STAMP_ERR_SHAPE;
  if (p->gen.kind != kGenNone) return STAMP_ERR_UNSUPPORTED;  // the general path has no separately launchable stages
  if (stage == 6 && p->engine != STAMP_GEMM_FP6) return STAMP_ERR_UNSUPPORTED;
  if (stage == 5 && p->fused_ok && !p->unfused) return STAMP_ERR_UNSUPPORTED;
  if (!ws_ok(p, ws, ws_bytes, p->ws_total)) return STAMP_ERR_WORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  float* abot = reinterpret_cast<float*>(at(ws, p->ws_abot));
  uint32_t* rowmax = reinterpret_cast<uint32_t*>(at(ws, p->ws_rowmax));
  uint32_t* gpart = reinterpret_cast<uint32_t*>(at(ws, p->ws_gpart));
  float* ythi = reinterpret_cast<float*>(at(ws, p->ws_ythi));
  float* P = reinterpret_cast<float*>(at(ws, p->ws_P));
  float* ytlo = reinterpret_cast<float*>(at(ws, p->ws_ytlo));
  const bool fused = p->fused_ok && !p->unfused;
  hipError_t e = hipSuccess;
  if (p->geom.ident) {
    // stages of a plan without a transform: 0 quantization, 2 the 8-bit rows' GEMM, 3 their output pass,
    // 6 FP6 conversion, 4 the 4-bit rows' GEMM; 1 and 5 do not exist
    switch (stage) {
      case 0: e = stamp_launch_actquant(p, X, q_hi, q_lo, scales, abot, rowmax, gpart, st, 1); break;
      case 2:
        if (p->geom.k > 0 && p->hi6[0]) {
          e = convert_rows(p, q_hi, nullptr, nullptr, 0, ws, st);
          if (e == hipSuccess) e = stamp_launch_hi6(p, at(ws, p->ws_hi6), scales, 1, Y, 0, 0, nullptr, 1.0f, st);
        } else if (p->geom.k > 0) {
          e = stamp_launch_gemm_hi(p, q_hi, scales, 1, ythi, st);
        }
        break;
      case 3: if (!p->hi6[0]) e = stamp_launch_hi_rows_out(p, ythi, Y, st, p->hi_ksplit); break;
      case 4:
        if (p->engine == STAMP_GEMM_FP6) e = stamp_launch_gemm_lo6(p, at(ws, p->ws_a6), scales, 3, Y, nullptr, st);
        else e = stamp_launch_gemm_lo(p, q_lo, scales, 3, Y, nullptr, st);
        break;
      case 6: e = stamp_launch_repack6(p, q_lo, at(ws, p->ws_a6), st); break;
      default: return STAMP_ERR_UNSUPPORTED;
    }
    return e == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
  }
  switch (stage) {
    case 0: e = stamp_launch_actquant(p, X, q_hi, q_lo, scales, abot, rowmax, gpart, st, 1); break;
    case 1: e = stamp_launch_actquant(p, X, q_hi, q_lo, scales, abot, rowmax, gpart, st, 2); break;
    case 2:
      if (p->hi6[own_top(p)]) e = convert_rows(p, q_hi, nullptr, nullptr, own_top(p), ws, st);
      if (e != hipSuccess) break;
      if (own_top(p)) e = launch_block_sums_own(p, q_hi, scales, ythi, P, at(ws, p->ws_hi6), st);
      else if (p->hi6[0]) e = stamp_launch_hi6(p, at(ws, p->ws_hi6), scales, 0, P, p->Npad, 0, nullptr, 1.0f, st);
      else if (stamp_hi_top_fused(p)) e = stamp_launch_gemm_hi(p, q_hi, scales, 2, P, st, p->Npad);
      else
        e = stamp_hi_rows_are_block_sums(p) ? stamp_launch_gemm_hi(p, q_hi, scales, 1, P, st, p->Npad)
                                            : stamp_launch_gemm_hi(p, q_hi, scales, 1, ythi, st);
      break;
    case 3:  // nothing to launch when the plan has no top levels, or when the 8-bit rows' GEMM has run them
      if (!own_top(p) && !p->hi6[0] && !stamp_hi_rows_are_block_sums(p) && !stamp_hi_top_fused(p))
        e = stamp_launch_inverse_top(p, ythi, 0, p->geom.N, P, p->Npad, st, p->hi_ksplit);
      break;
    case 4:
      if (p->engine == STAMP_GEMM_FP6)
        e = stamp_launch_gemm_lo6(p, at(ws, p->ws_a6), scales, fused ? 2 : 1, fused ? Y : (void*)ytlo, fused ? P : nullptr, st,
                                  own_top(p));
      else
        e = stamp_launch_gemm_lo(p, q_lo, scales, fused ? 2 : 1, fused ? Y : (void*)ytlo, fused ? P : nullptr, st);
      break;
    case 6: e = stamp_launch_repack6(p, q_lo, at(ws, p->ws_a6), st); break;
    case 5: e = stamp_launch_inverse_bottom(p, ytlo, 0, P, p->Npad, p->geom.N, p->bias_dev, Y, st); break;
  }
  return e == hipSuccess ? STAMP_OK : STAMP_ERR_DEVICE;
}

stamp_status_t stamp_debug_weight_codes(const stamp_plan_t* p, int8_t* qW_host, float* sw_host) {
  if (p == nullptr || qW_host == nullptr || sw_host == nullptr) return STAMP_ERR_NULL;
  const int d = p->geom.d, N = p->geom.N;
  if (p->gen.group) {
    // per-block scales: codes [d_in, d_out], scales [d_in / 64][d_out]
    const int Npad = ((N + 127) / 128) * 128, G = d / 64;
    int8_t* tq = static_cast<int8_t*>(malloc((size_t)Npad * d));
    float* ts = static_cast<float*>(malloc(sizeof(float) * (size_t)G * Npad));
    bool ok = tq != nullptr && ts != nullptr && hipDeviceSynchronize() == hipSuccess &&
              hipMemcpy(tq, p->qWg_dev, (size_t)Npad * d, hipMemcpyDeviceToHost) == hipSuccess &&
              hipMemcpy(ts, p->swg_dev, sizeof(float) * (size_t)G * Npad, hipMemcpyDeviceToHost) == hipSuccess;
    if (ok) {
      for (int n = 0; n < N; ++n)
        for (int c = 0; c < d; ++c) qW_host[(size_t)c * N + n] = tq[(size_t)n * d + c];
      for (int gi = 0; gi < G; ++gi)
        for (int n = 0; n < N; ++n) sw_host[(size_t)gi * N + n] = ts[(size_t)gi * Npad + n];
    }
    free(tq);
    free(ts);
    return ok ? STAMP_OK : STAMP_ERR_DEVICE;
  }
  int8_t* tmp = static_cast<int8_t*>(malloc((size_t)p->Npad * p->Kpad));
  if (tmp == nullptr) return STAMP_ERR_ALLOC;
  if (hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(tmp, p->qW_dev, (size_t)p->Npad * p->Kpad, hipMemcpyDeviceToHost) != hipSuccess ||
      hipMemcpy(sw_host, p->sw_dev, sizeof(float) * N, hipMemcpyDeviceToHost) != hipSuccess) {
    free(tmp);
    return STAMP_ERR_DEVICE;
  }
  for (int n = 0; n < N; ++n)
    for (int c = 0; c < d; ++c) {
      const int g16 = c >> 4, cc = c & 15, half = cc >> 3, c8 = cc & 7;
      const int pos = half * 8 + (c8 & 1) * 4 + (c8 >> 1);
      qW_host[(size_t)c * N + n] = (int8_t)(tmp[stamp_w_offset(n, g16 * 16 + pos, p->Kpad)] / 16);
    }
  free(tmp);
  return STAMP_OK;
}

}  // extern "C"

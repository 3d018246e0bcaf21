// api.cpp - status strings, version, argument checks, launch plans and workspace queries.
// Pure host code: nothing here touches the GPU, so these paths are testable without one.
#include <algorithm>

#include "slim_host.h"

namespace {
constexpr int64_t kMaxDim = int64_t(1) << 31;
constexpr int64_t kMaxLargeRed = int64_t(1) << 23;     // large M: longest reduction
constexpr int64_t kMaxTiledElems = int64_t(1) << 30;   // large M: M r and rows r (fp16, 32-bit byte offsets)
constexpr size_t kCounterSlots = SLIM_COUNTER_SLOTS;
constexpr int64_t kDecodeAdSlice = SLIM_DECODE_AD_SLICE;

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
size_t round256(size_t x) { return (x + 255) & ~size_t(255); }
}  // namespace

extern "C" const char* slim_status_string(int status) {
  switch (status) {
    case SLIM_OK: return "SLIM_OK";
    case SLIM_EINVAL: return "SLIM_EINVAL: null pointer or argument out of range";
    case SLIM_ESHAPE: return "SLIM_ESHAPE: size breaks a divisibility or range rule";
    case SLIM_EDTYPE: return "SLIM_EDTYPE: unsupported dtype";
    case SLIM_EALIGN: return "SLIM_EALIGN: device array not 16-byte aligned";
    case SLIM_ENONFINITE: return "SLIM_ENONFINITE: weight holds NaN or Inf";
    case SLIM_ERANGE: return "SLIM_ERANGE: group scale overflows fp16";
    case SLIM_EWORKSPACE: return "SLIM_EWORKSPACE: workspace missing or too small";
    case SLIM_EDEVICE: return "SLIM_EDEVICE: HIP runtime or launch failure";
    case SLIM_EUNSUPPORTED: return "SLIM_EUNSUPPORTED: valid but not supported by this library";
    default: return "unknown slim status";
  }
}

extern "C" int slim_abi_version(void) { return SLIM_ABI_VERSION; }

int slim_check_pack(const float* W, int64_t N, int64_t K, const void* codes, const void* meta,
                    const void* scales, const void* mask) {
  if (!W || !codes || !meta || !scales) return SLIM_EINVAL;
  if (N < 16 || K < 128 || N >= kMaxDim || K >= kMaxDim) return SLIM_ESHAPE;
  if (N % 16 || K % 128) return SLIM_ESHAPE;   // whole 16-row blocks and 128-wide chunks
  if (!slim_aligned16(W) || !slim_aligned16(codes) || !slim_aligned16(meta) || !slim_aligned16(scales) ||
      (mask && !slim_aligned16(mask)))
    return SLIM_EALIGN;
  return SLIM_OK;
}

int slim_check_pack_bwd(const void* codes, const void* meta, const void* scales, int64_t N, int64_t K,
                        const void* codesT, const void* metaT, const void* scalesT, const void* mask_rc) {
  if (!codes || !meta || !scales || !codesT || !metaT || !scalesT) return SLIM_EINVAL;
  if (N < 128 || K < 128 || N >= kMaxDim || K >= kMaxDim) return SLIM_ESHAPE;
  if (N % 128 || K % 128) return SLIM_ESHAPE;   // the transposed pack chunks N by 128
  if (!slim_aligned16(codes) || !slim_aligned16(meta) || !slim_aligned16(scales) || !slim_aligned16(codesT) ||
      !slim_aligned16(metaT) || !slim_aligned16(scalesT) || (mask_rc && !slim_aligned16(mask_rc)))
    return SLIM_EALIGN;
  return SLIM_OK;
}

namespace {

// Slices of the adapter's first product in units of 128 ranks x 64 or 128 rows (at of them): as many as give
// about one block per CU, a power of two up to eight (the last unit of a tile sums four at a time) of at
// least 512 positions.
int64_t adapter_slices(int64_t at, int64_t red) {
  int64_t s = 8;
  while (s > 1 && (at * s > 256 || red < 512 * s)) s /= 2;
  return s;
}

// The middle path, where 512-row tiles are too few for the chip: 128 x 64 tiles, two blocks per CU, or
// 256 x 128, one, over S slices of the reduction, whichever the cost below favours. Returns false where the
// 512-row tiles are the better choice. `most`: bytes the partials and the fp16 activations may take.
bool mid_plan(bool bwd, int64_t M, int64_t rows, int64_t red, int64_t r, int64_t most, SlimPlan* q) {
  const int64_t nch = red / 128, big = cdiv(rows, 256) * cdiv(M, 128);
  // With about as many 256 x 128 tiles as CUs the 512-row tiles win (half the LDS and direct-load bytes per
  // weight row; with an adapter also no fp32 partials through memory): limits from both plans' times on 750 sizes of
  // 512 to 28672 rows, reductions of 512 to 14336 and M 33 to 8192; past them the middle path lost, below them no
  // call lost more than 2 %. Without an adapter one whole round is still better in the forward (4096 x 4096, M 2048:
  // 55 us against 58; 8192 x 8192, M 1024: 94 against 96), less of one in the backward, which scales every operand
  // fragment (7296 rows, reduction 13824, M 663: 147 against 162), unless M is larger than the rows: then each
  // block's output is the larger part, for short reductions most of all (1024 x 2048, M 8192: 58 against 47; 1024 x
  // 640, M 7963: 40 % over). With an adapter: forward 11008 x 4096, M 512 (172 tiles) 67 against 76, 3328 x 1280, M
  // 2246 (234) 53 against 48; longer reductions pay for the partials longer (28672 x 8192, M 200 (224) 116 against
  // 124) unless those are many (2048 x 9216, M 3500 (224) 157 against 151). Backward 5120 x 13824, M 333 (162) 93
  // against 102, 2944 rows, reduction 3584, M 2004 (192) 90 against 82.
  int64_t limit;
  if (r == 0) {
    if (M <= rows) limit = bwd ? 224 : 256;
    else if (!bwd && red > 4096) limit = 256;
    else limit = nch > (bwd ? 9 : 6) ? (bwd ? 200 : 190) : 140;
  } else if (bwd) {
    limit = 164;
  } else {
    limit = nch <= 4 ? 128 : (red >= 8192 && M <= rows ? 224 : 180);
  }
  if (big > limit) return false;
  if (r > 0 && cdiv(M, 64) * cdiv(r, 128) > (int64_t)kCounterSlots) return false;
  double best = 0;
  int cols = 0, slices = 1;
  int64_t chunks = nch;
  for (int tc = 64; tc <= 128; tc += 64) {
    const int64_t R = cdiv(rows, 2 * tc), C = cdiv(M, tc);
    for (int64_t s = 1; s <= 8 && (s == 1 || nch >= 4 * s); ++s) {
      const int64_t per = cdiv(nch, s), split = cdiv(nch, per), blocks = R * C * split;
      if (s > 1 && split * R * C * 2 * tc * tc * 4 + 2 * M * red > most) break;
      // microseconds per chunk: a lone 128 x 64 block on a CU 0.40, two 0.75, a 256 x 128 block 1.15; the
      // adapter's chain beside them takes at least about 7 (its units are not counted among the blocks here)
      double t = per * (tc == 64 ? (blocks <= 256 ? 0.40 : 0.75 * cdiv(blocks, 512)) : 1.15 * cdiv(blocks, 256));
      if (r > 0 && t < 7) t = 7;
      // partials written and read at about 4 TB/s
      if (split > 1 || r > 0) t += split * M * rows * 8 / 4e6;
      if (best == 0 || t < best) {
        best = t;
        cols = tc;
        slices = (int)split;
        chunks = per;
      }
    }
  }
  if (r > 0) {
    const int64_t at = cdiv(M, cols) * cdiv(r, 128), ad_slice = cdiv(cdiv(red, adapter_slices(at, red)), 64) * 64;
    // where the adapter's units and one round of 256 x 128 tiles are more blocks than CUs (by more than a few, where
    // the weights are the larger operand), they take two rounds (backward 4096 x 4096, r 384, M 1280: 93 us against
    // 85; forward 2432 x 3968, r 224, M 2250: 81 against 76), and the shortest reductions do not pay for the backward's
    // finish (16640 x 640, r 64, M 231: 34.8 against 33.8)
    const bool two = cols == 128 && slices == 1 && big + at * cdiv(red, ad_slice) > (M > rows ? 256 : 272);
    if (bwd ? two || (cols == 128 && nch <= 5 && big > 128) : two && red <= 8192 && 2 * M > rows && big > 150) return false;
    q->ad_tiles_m = (int)cdiv(M, cols);
    q->ad_tiles_j = (int)cdiv(r, 128);
    q->ad_slice = ad_slice;
    q->ad_split = (int)cdiv(red, ad_slice);
  }
  q->mid = true;
  q->sp_cols_tile = cols;
  q->sp_rows_tile = 2 * cols;
  q->sp_row_tiles = cdiv(rows, 2 * cols);
  q->sp_col_tiles = cdiv(M, cols);
  q->sp_split = slices;
  q->sp_chunks_per_split = chunks;
  return true;
}

// One plan. `rows512` (M > 32): 512-row tiles and the kernels of k_adapter_gemm; otherwise the middle path or its
// first-product units where they are the faster ones, `most` as above.
int plan_kernels(bool bwd, int64_t M, int64_t N, int64_t K, int64_t r, bool rows512, int64_t most, SlimPlan* p) {
  if (M < 1 || N < 16 || K < 128 || M >= kMaxDim || N >= kMaxDim || K >= kMaxDim) return SLIM_ESHAPE;
  if (N % 16 || K % 128 || r < 0 || r % 16 || r >= kMaxDim) return SLIM_ESHAPE;
  if (bwd && N % 128) return SLIM_ESHAPE;
  const int64_t rows = bwd ? K : N, red = bwd ? N : K;
  const int64_t nchunks = red / 128;
  SlimPlan q;
  size_t ad_counters = 0, tpart_bytes = 0, ypart_bytes = 0;
  if (M <= 32) {
    // small M: one launch of split-reduction sparse units plus adapter first-product units,
    // then the adapter's second product
    q.decode = true;
    q.dec_fm = M <= 16 ? 1 : 2;
    const int64_t mc = 16 * q.dec_fm;
    q.sp_rows_tile = 64;
    q.sp_cols_tile = (int)mc;
    q.sp_row_tiles = cdiv(rows, 64);
    q.sp_col_tiles = 1;
    // a sparse unit covers 4 * G quantisation groups of the reduction; two groups per lane group
    // when that still gives every CU a unit
    q.dec_g = (q.dec_fm == 1 && q.sp_row_tiles * cdiv(nchunks, 8) >= 256) ? 2 : 1;
    q.sp_chunks_per_split = 4 * q.dec_g;
    q.sp_split = (int)cdiv(nchunks, q.sp_chunks_per_split);
    // sparse blocks run several row tiles of one slice when there are more units than the target
    // block count (the backward's staged activations carry one 128-row group's scales: at most
    // the two row tiles of a group, starting at an even tile)
    const int64_t units = q.sp_row_tiles * q.sp_split;
    q.dec_units = (int)std::min<int64_t>(bwd ? 2 : SLIM_DECODE_MAX_UNITS, cdiv(units, SLIM_DECODE_BLOCKS));
    q.sp_blocks = cdiv(q.sp_row_tiles, q.dec_units) * q.sp_split;
    if (r > 0) {
      // adapter units: 16 ranks x 4 waves x ad_sub slices of SLIM_DECODE_AD_SLICE positions, at
      // most about SLIM_DECODE_AD_SPLITS splits (a wave takes several slices of a long reduction)
      q.ad_jblocks = cdiv(r, 16);
      const int64_t slices = cdiv(red, 4 * kDecodeAdSlice);
      q.ad_sub = (int)cdiv(slices, SLIM_DECODE_AD_SPLITS);
      q.ad_slice = 4 * kDecodeAdSlice * q.ad_sub;
      q.ad_split = (int)cdiv(slices, q.ad_sub);
      if (q.ad_split > 1) {
        ad_counters = (size_t)q.ad_jblocks;
        // per split and 16-row fragment: 256 fp32 partials and 16 row maxima
        tpart_bytes = (size_t)q.ad_jblocks * q.ad_split * q.dec_fm * 272 * 4;
      }
    }
    if (q.sp_split > 1 || r > 0) ypart_bytes = (size_t)q.sp_row_tiles * q.sp_split * 4 * q.dec_fm * 256 * 4;
    q.lds_bytes = 0;
  } else {
    // large M: dense adapter GEMM (128 x 128 tiles) then 512 x 96 or 512 x 128 sparse tiles. Their
    // per-lane buffer offsets are 32-bit: an activation offset spans up to 128 rows of the
    // reduction, and T and the adapter's second factor are addressed from their start.
    if (red > kMaxLargeRed || cdiv(M, 32) * 32 * r >= kMaxTiledElems || cdiv(rows, 32) * 32 * r >= kMaxTiledElems)
      return SLIM_EUNSUPPORTED;
    q.decode = false;
    if (!rows512 && mid_plan(bwd, M, rows, red, r, most, &q)) {
      if (q.sp_split > 1 || r > 0)
        ypart_bytes = (size_t)q.sp_split * (size_t)(q.sp_row_tiles * q.sp_rows_tile) * (size_t)(q.sp_col_tiles * q.sp_cols_tile) * 4;
      if (q.ad_split > 1) {
        ad_counters = (size_t)q.ad_tiles_m * q.ad_tiles_j;
        tpart_bytes = ad_counters * q.ad_split * 128 * q.sp_cols_tile * 4;
      }
    }
    if (!q.mid) {
      q.sp_rows_tile = 512;
      q.sp_row_tiles = cdiv(rows, 512);
      // 512 x 128 tiles spend less dequantisation per MFMA (a tile takes about 1.12x the time of a
      // 512 x 96 one for 4/3 the work); 512 x 96 tiles are more and can fill the last round of
      // blocks (one per CU) better. Take the one with fewer rounds, weighted.
      const int64_t r96 = cdiv(q.sp_row_tiles * cdiv(M, 96), 256), r128 = cdiv(q.sp_row_tiles * cdiv(M, 128), 256);
      q.sp_cols_tile = 112 * r128 <= 100 * r96 ? 128 : 96;
      q.sp_col_tiles = cdiv(M, q.sp_cols_tile);
      q.sp_split = 1;
      q.sp_chunks_per_split = nchunks;
      // 256 x 256 adapter tiles (half the operand bytes per flop) with a 128 KiB ring, one block per
      // CU, when they fill the 256 CUs with reduction slices of at least 2048: the long reductions
      // at large M (the 70B dX product took 320 -> 253 us with its split sum; the 13B layers, whose
      // slices would be shorter or whose blocks too few, were slower); 256 rows of the reduction
      // stay within 32-bit byte offsets
      const int64_t wtiles = cdiv(M, 256) * (r / 256);
      const int64_t wsplit = wtiles > 0 ? std::max<int64_t>(1, std::min<int64_t>(256 / wtiles, red / 1024)) : 0;
      if (r > 0 && r % 256 == 0 && red < (int64_t(1) << 22) && wtiles * wsplit >= 256 && red / wsplit >= 2048) {
        q.ad_wide = true;
        q.ad_tiles_m = (int)cdiv(M, 256);
        q.ad_tiles_j = (int)(r / 256);
        const int64_t slice = cdiv(cdiv(red, wsplit), 32) * 32;
        q.ad_split = (int)cdiv(red, slice);
        q.ad_slice = slice;
        if (q.ad_split > 1) tpart_bytes = (size_t)q.ad_split * (size_t)cdiv(M, 32) * 32 * (size_t)r * 4;
      } else if (r > 0 && !rows512 && cdiv(M, 128) * cdiv(r, 128) <= 64) {
        // few tiles of T: the middle path's first-product units, which sum their slices in the launch (7B
        // prefill 11008 x 4096, M 2048, r 384 (48 tiles): 20.0 against 19.4 us and a 5.3 us launch that sums;
        // 28672 x 8192, M 512 (16): 20.8 against 17.6 + 6.0). With more tiles two 128 x 128 blocks per CU are
        // as fast or faster (4096 x 11008, M 3000, r 400 (96): 68 against 50 + 6; 13B layers at M 4096 equal).
        q.ad_tn = true;
        q.ad_tiles_m = (int)cdiv(M, 128);
        q.ad_tiles_j = (int)cdiv(r, 128);
        const int64_t tiles = (int64_t)q.ad_tiles_m * q.ad_tiles_j;
        q.ad_slice = cdiv(cdiv(red, adapter_slices(tiles, red)), 64) * 64;
        q.ad_split = (int)cdiv(red, q.ad_slice);
        if (q.ad_split > 1) {
          ad_counters = (size_t)tiles;
          tpart_bytes = (size_t)tiles * q.ad_split * 128 * 128 * 4;
        }
      } else if (r > 0) {
        q.ad_tiles_m = (int)cdiv(M, 128);
        q.ad_tiles_j = (int)cdiv(r, 128);
        const int64_t tiles = (int64_t)q.ad_tiles_m * q.ad_tiles_j;
        // two blocks per CU (the GEMM's LDS ring takes 64 KB): at most 512 blocks, so one round
        const int64_t split = std::max<int64_t>(1, std::min<int64_t>(512 / tiles, red / 512));
        const int64_t slice = cdiv(cdiv(red, split), 64) * 64;
        q.ad_split = (int)cdiv(red, slice);
        q.ad_slice = slice;
        // split partials: fp32, one T-sized tiled array per split (summed by the next kernel)
        if (q.ad_split > 1) tpart_bytes = (size_t)q.ad_split * (size_t)cdiv(M, 32) * 32 * (size_t)r * 4;
      }
    }
  }
  // workspace: [counters][adapter intermediate fp16 M x r][adapter partials][sparse partials]
  // [fp16 activations (large M)]
  q.n_counters = ad_counters;
  q.off_counters = 0;
  if (q.n_counters > kCounterSlots) return SLIM_EUNSUPPORTED;
  // the counter region has a fixed size so that it stays at zero across calls with other sizes
  size_t off = kCounterSlots * 4;
  // T (fp16, from row-scaled activations): row-major [M, r] at small M; at large M in 32 x 16 tiles
  // ([ceil(M/32)][r/16][32][16], see adapter_gemm.hip), which the tile kernel's epilogue reads 1 KB
  // at a time
  q.off_t = off;
  off = round256(off + (size_t)(q.decode ? M : cdiv(M, 32) * 32) * (size_t)r * 2);
  q.off_tpart = off;
  off = round256(off + tpart_bytes);
  q.off_ypart = off;
  off = round256(off + ypart_bytes);
  // large M: the row-scaled fp16 copy of the activations for the tile kernel's direct-to-LDS loads, and (backward:
  // the forward's factor comes tiled from slim_pack_adapter) the adapter's second factor P
  // [rows, r] re-laid in 32 x 16 tiles
  q.off_x16 = off;
  if (!q.decode) off = round256(off + (size_t)M * (size_t)red * 2);
  // 2^-e per activation row: large M, the rows of the fp16 copy are scaled by 2^e; small M, the
  // rows of T are
  q.off_rowinv = off;
  off = round256(off + (size_t)M * 4);
  q.off_pb = off;
  if (!q.decode && bwd) off = round256(off + (size_t)cdiv(rows, 32) * 32 * (size_t)r * 2);
  q.total = off;
  q.query = off;
  *p = q;
  return SLIM_OK;
}

}  // namespace

// The faster plan where the workspace holds it, the 512-row one where it does not: the faster plan's size falls
// and rises with M (4096 x 4096, r 384: 46.0 MB at M 1280, 29.5 MB at M 2048), so a workspace made for a program's
// most rows may be short for it with fewer. The query is the larger of the two sizes, so that it also covers every
// smaller M that the 512-row plans' sizes cover.
int slim_make_plan(bool bwd, int64_t M, int64_t N, int64_t K, int64_t r, size_t ws_bytes, SlimPlan* p) {
  int st = plan_kernels(bwd, M, N, K, r, true, 0, p);
  if (st != SLIM_OK || p->decode) return st;
  // Sizes that fit the no-allocation entry point's scratch on either plan keep fitting (it sums in the order of the
  // calls with a workspace): there the partials leave room for the rest. Past it on both the scratch says nothing.
  constexpr size_t scratch = SLIM_NOALLOC_SCRATCH_BYTES;
  SlimPlan q;
  st = plan_kernels(bwd, M, N, K, r, false, (int64_t)scratch - (8 << 20), &q);
  if (st != SLIM_OK) return st;
  if ((q.mid || q.ad_tn) && q.total > scratch) {
    if (p->total <= scratch) return SLIM_OK;
    st = plan_kernels(bwd, M, N, K, r, false, INT64_MAX, &q);
    if (st != SLIM_OK) return st;
  }
  q.query = p->query = std::max(p->total, q.total);
  if (q.total <= ws_bytes) *p = q;
  return SLIM_OK;
}

int slim_check_linear(bool bwd, const void* X, int xdtype, int64_t M, int64_t N, int64_t K, const void* codes,
                      const void* meta, const void* scales, const void* L, const void* R, int64_t r, const void* Y,
                      const void* ws, size_t ws_bytes, SlimPlan* plan) {
  if (!X || !codes || !meta || !scales || !Y) return SLIM_EINVAL;
  if (r < 0) return SLIM_EINVAL;
  if (r == 0 ? (L != nullptr || R != nullptr) : (!L || !R)) return SLIM_EINVAL;
  if (xdtype != SLIM_F16 && xdtype != SLIM_BF16) return SLIM_EDTYPE;
  int st = slim_make_plan(bwd, M, N, K, r, ws_bytes, plan);
  if (st != SLIM_OK) return st;
  if (!slim_aligned16(X) || !slim_aligned16(codes) || !slim_aligned16(meta) || !slim_aligned16(scales) ||
      !slim_aligned16(Y) || (L && !slim_aligned16(L)) || (R && !slim_aligned16(R)))
    return SLIM_EALIGN;
  if (!ws || ws_bytes < plan->total) return SLIM_EWORKSPACE;
  if (!slim_aligned16(ws)) return SLIM_EALIGN;
  plan->scaled = !plan->decode && (bwd || xdtype == SLIM_BF16 || r > 0);
  return SLIM_OK;
}

extern "C" int slim_linear_workspace(int64_t M, int64_t N, int64_t K, int64_t r, size_t* bytes) {
  if (!bytes) return SLIM_EINVAL;
  SlimPlan p;
  int st = slim_make_plan(false, M, N, K, r, SIZE_MAX, &p);
  if (st == SLIM_OK) *bytes = p.query;
  return st;
}

extern "C" int slim_bwd_dx_workspace(int64_t M, int64_t N, int64_t K, int64_t r, size_t* bytes) {
  if (!bytes) return SLIM_EINVAL;
  SlimPlan p;
  int st = slim_make_plan(true, M, N, K, r, SIZE_MAX, &p);
  if (st == SLIM_OK) *bytes = p.query;
  return st;
}

int slim_make_plan_qa(int64_t M, int64_t N, int64_t K, int64_t r, size_t ws_bytes, SlimPlan* p) {
  if (r < 32 || r % 32) return SLIM_ESHAPE;   // 4-bit factor rows are whole 16-byte runs
  // the expansions follow the layer's own workspace (whose end is a multiple of 256)
  size_t q16 = 0, p16 = 0;
  if (M > 32 && N > 0 && K > 0 && N < kMaxDim && K < kMaxDim && r < kMaxDim) {
    q16 = round256((size_t)r * (size_t)K * 2);
    p16 = round256((size_t)cdiv(N, 32) * 32 * (size_t)r * 2);
  }
  int st = slim_make_plan(false, M, N, K, r, ws_bytes > q16 + p16 ? ws_bytes - q16 - p16 : 0, p);
  if (st != SLIM_OK) return st;
  p->off_q16 = p->total;
  p->off_p16 = p->total + q16;
  p->total += q16 + p16;
  p->query += q16 + p16;
  return SLIM_OK;
}

int slim_check_linear_qa(const void* X, int xdtype, int64_t M, int64_t N, int64_t K, const void* codes,
                         const void* meta, const void* scales, const void* Lq, const void* Ls, const void* Rq,
                         const void* Rs, int64_t r, const void* Y, const void* ws, size_t ws_bytes, SlimPlan* plan) {
  if (!X || !codes || !meta || !scales || !Y || !Lq || !Ls || !Rq || !Rs) return SLIM_EINVAL;
  if (xdtype != SLIM_F16 && xdtype != SLIM_BF16) return SLIM_EDTYPE;
  int st = slim_make_plan_qa(M, N, K, r, ws_bytes, plan);
  if (st != SLIM_OK) return st;
  if (!slim_aligned16(X) || !slim_aligned16(codes) || !slim_aligned16(meta) || !slim_aligned16(scales) ||
      !slim_aligned16(Y) || !slim_aligned16(Lq) || !slim_aligned16(Ls) || !slim_aligned16(Rq) || !slim_aligned16(Rs))
    return SLIM_EALIGN;
  if (!ws || ws_bytes < plan->total) return SLIM_EWORKSPACE;
  if (!slim_aligned16(ws)) return SLIM_EALIGN;
  plan->scaled = !plan->decode;
  return SLIM_OK;
}

extern "C" int slim_linear_qa_workspace(int64_t M, int64_t N, int64_t K, int64_t r, size_t* bytes) {
  if (!bytes) return SLIM_EINVAL;
  SlimPlan p;
  int st = slim_make_plan_qa(M, N, K, r, SIZE_MAX, &p);
  if (st == SLIM_OK) *bytes = p.query;
  return st;
}

// pack.hip - one-time packing kernels: forward 2:4 + int4 group-128 pack, and the SLoPe
// double-pruned backward pack (2:4 along N of the packed forward weight).
#include "slim_device.h"
#include "slim_host.h"
#include "slim_timing.h"

namespace {

constexpr int kPackThreads = 256;

// |x / s| rounded to the nearest integer, ties to even, at most 7: exactly the clamped rint of the quotient,
// without a division. r is 1 / s to an ulp, so the first guess is off by at most one, and only next to a
// half-way point. t - q s is then exact in fp32 (q s has 15 bits; for q >= 1 the difference, below s, is a
// multiple of t's last place, at least 2^-25 s), so it can be compared with s / 2 = hs; on an odd q a tie moves
// on to the even neighbour, which the bit pattern one below hs makes part of the same comparison.
SLIM_DEV uint32_t round_mag(float t, float s, float r, uint32_t hs) {
  const float q = rintf(fminf(t * r, 7.0f));
  const float d = fmaf(-q, s, t);
  const int qi = (int)q;
  const int step = fabsf(d) > __uint_as_float(hs - (uint32_t)(qi & 1)) ? ((int)__float_as_uint(d) >> 31) | 1 : 0;
  return (uint32_t)min(qi + step, 7);
}

// One thread per 16 positions of a row (four 4-groups, one code word and one index half-word); eight threads
// cover one 128-wide quantisation group, whose absmax takes three exchanges and whose division by 7 and
// reciprocal are made once for eight codes. With `alpha` (one float64 in device memory, SLiM-Quant's
// per-tensor parameter) every group takes it in place of its own absmax. Bound by the reading of W (11008 x
// 4096: 74 us with a thread per 4-group and two float64 divisions in each, 38 now).
__global__ void __launch_bounds__(kPackThreads)
k_pack(const u32x4_t* __restrict__ W, int64_t total16, int64_t nch, uint32_t* __restrict__ codes,
       uint16_t* __restrict__ meta, uint16_t* __restrict__ scales, u32x4_t* __restrict__ mask,
       int* __restrict__ status, const double* __restrict__ alpha) {
  const int64_t t = (int64_t)blockIdx.x * kPackThreads + threadIdx.x;
  if (t >= total16) return;                  // total16 is a multiple of 8: whole groups stay together
  u32x4_t v[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = W[4 * t + c];
  // magnitudes order as their bit patterns, and a non-finite one is at least infinity's
  uint32_t am = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int p = 0; p < 4; ++p) am = max(am, v[c][p] & 0x7FFFFFFFu);
  int bad = am >= 0x7F800000u ? 1 : 0;
#pragma unroll
  for (int off = 4; off >= 1; off >>= 1) am = max(am, (uint32_t)__shfl_xor((int)am, off, 64));
  float gmax = __uint_as_float(am);
  if (alpha) {
    const double ad = *alpha;
    if (!(ad >= 0.0)) bad |= 2;
    gmax = (float)ad;
  }
  // s16 = fp16_RNE(fp32 absmax / 7), IEEE division (alpha rounded to fp32 in its place)
  const _Float16 s16 = (_Float16)__fdiv_rn(gmax, 7.0f);
  const float sf = (float)s16;
  if (!__builtin_isfinite(sf)) bad |= 2;
  if (bad) atomicOr(status, bad);
  const bool pos = sf > 0.f;
  const float r = __builtin_amdgcn_rcpf(sf);
  const uint32_t hs = __float_as_uint(0.5f * sf);

  uint32_t cw = 0, mw = 0, mk[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    float w[4], a[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      w[p] = __uint_as_float(v[c][p]);
      a[p] = fabsf(w[p]);
    }
    // top two by (|w| desc, position asc): p < q comes first exactly when a[p] >= a[q]; kept are those that
    // come before at least two of the other three
    const bool c01 = a[0] >= a[1], c02 = a[0] >= a[2], c03 = a[0] >= a[3], c12 = a[1] >= a[2], c13 = a[1] >= a[3],
               c23 = a[2] >= a[3];
    auto two = [](bool x, bool y, bool z) { return (x & y) | (z & (x | y)); };
    const bool k0 = two(c01, c02, c03), k1 = two(!c01, c12, c13), k2 = two(!c02, !c12, c23),
               k3 = two(!c03, !c13, !c23);
    const uint32_t i0 = k0 ? 0u : (k1 ? 1u : 2u), i1 = k3 ? 3u : (k2 ? 2u : 1u);
    const float x0 = k0 ? w[0] : (k1 ? w[1] : w[2]), x1 = k3 ? w[3] : (k2 ? w[2] : w[1]);
    auto code = [&](float x) -> uint32_t {
      const int m = pos ? (int)round_mag(fabsf(x), sf, r, hs) : 0;
      return (uint32_t)(8 + (__float_as_uint(x) >> 31 ? -m : m));
    };
    cw |= (code(x0) << (4 * c)) | (code(x1) << (16 + 4 * c));
    mw |= (i0 | (i1 << 2)) << (4 * c);
    mk[c] = (k0 ? 1u : 0u) | (k1 ? 1u << 8 : 0u) | (k2 ? 1u << 16 : 0u) | (k3 ? 1u << 24 : 0u);
  }
  // W holds fewer than 2^32 groups of 128 (2 TiB): a 32-bit division
  const uint32_t g = (uint32_t)(t >> 3), row = g / (uint32_t)nch;
  const int64_t slot = packed_slot(row, g - row * (uint32_t)nch, nch);
  const int word = (int)(t & 7);
  codes[8 * slot + word] = cw;
  meta[8 * slot + word] = (uint16_t)mw;
  if (word == 0) scales[slot] = __builtin_bit_cast(uint16_t, s16);
  if (mask) mask[t] = u32x4_t{mk[0], mk[1], mk[2], mk[3]};
}

// Backward pack. Block = 256 threads, tile = 128 rows (n) x 128 columns (k): whole slots of both packs, so
// every load and store moves whole sectors. Phase 1 expands the tile into LDS, one byte per entry: its code
// (8 where pruned) in bits 0..3, 3 - n % 4 in bits 4..5, the forward-kept bit in bit 6; a thread makes 16
// columns of a row at a time, 16-byte LDS writes. Phase 2 gives each thread four columns (one LDS word per
// row) and one 16-row block, prunes each aligned 4-row group to its top two (|Wc| desc, forward-kept desc,
// row asc) and emits one codesT word and one metaT half-word per column. A key orders a group's entries in
// one integer comparison: |code - 8| s16 is exact in fp32 with ten low bits zero (3-bit x 11-bit
// significands), and the LDS byte fits below; the top two are a max / min network, and carry their codes.
// LDS rows are 128 bytes with one row of padding per 16, and the words of a row XOR-swizzled by
// 8 (n / 32 % 4), so the eight row blocks that a wave reads at once fall in distinct banks. Bound by
// instruction issue and the latency of the three phases (11008 x 4096: 54 us with 64 x 64 tiles, byte
// writes and fp32 ranking, 23 now; 34 MB).
constexpr int kBT = 128;
// Largest forward scale the backward accepts: its large-M path multiplies gradients scaled below
// 2^(kActExp + 1) = 32 by s16 in fp16, which stays below 65504 for s16 < 2048.
constexpr float kBwdScaleLimit = 2048.0f;
static_assert(kActExp == 4, "kBwdScaleLimit assumes row-scaled activations below 32");

// LDS word of columns 4 quad .. + 3 of row n
SLIM_DEV int pb_word(int n, int quad) { return (n + (n >> 4)) * (kBT / 4) + (quad ^ (8 * ((n >> 5) & 3))); }

template <bool MASK>
__global__ void __launch_bounds__(256)
k_pack_bwd(const uint32_t* __restrict__ codes, const uint16_t* __restrict__ meta,
           const uint16_t* __restrict__ scales, int64_t N, int64_t K, uint32_t* __restrict__ codesT,
           uint16_t* __restrict__ metaT, uint16_t* __restrict__ scalesT, uint8_t* __restrict__ mask_rc,
           int* __restrict__ status) {
  __shared__ __attribute__((aligned(16))) uint32_t e_s[(kBT + kBT / 16) * (kBT / 4)];
  __shared__ __attribute__((aligned(16))) float sc_s[kBT];     // |scale| of each row for this column tile
  const int tid = threadIdx.x;
  const int64_t kc = blockIdx.x, nc = blockIdx.y, n0 = nc * kBT, k0 = kc * kBT;   // N and K are multiples of 128

  // phase 1: thread -> (row tid / 8 + 32 j, word tid % 8)
  uint32_t cws[4], mws[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t slot = packed_slot(n0 + (tid >> 3) + 32 * j, kc, K / 128);
    cws[j] = codes[8 * slot + (tid & 7)];
    mws[j] = meta[8 * slot + (tid & 7)];
  }
  if (tid < kBT) {
    const uint16_t sb = scales[packed_slot(n0 + tid, kc, K / 128)];
    const float sc = h_bits_to_f(sb);
    sc_s[tid] = fabsf(sc);
    // the backward's fp16 product of a row-scaled gradient (below 32) and s16 must stay finite
    if (!(sc < kBwdScaleLimit)) atomicOr(status, 2);
    scalesT[kc * N + n0 + tid] = sb;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = (tid >> 3) + 32 * j;
    u32x4_t e;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t s0 = ((mws[j] >> (4 * c)) & 3u) * 8u, s1 = ((mws[j] >> (4 * c + 2)) & 3u) * 8u;
      const uint32_t u0 = (cws[j] >> (4 * c)) & 0xFu, u1 = (cws[j] >> (16 + 4 * c)) & 0xFu;
      uint32_t x = 0x08080808u;
      x = (x & ~(0xFFu << s0)) | ((u0 | 0x40u) << s0);
      x = (x & ~(0xFFu << s1)) | ((u1 | 0x40u) << s1);
      e[c] = x | 0x10101010u * (uint32_t)(3 - (row & 3));
    }
    *reinterpret_cast<u32x4_t*>(&e_s[pb_word(row, 4 * (tid & 7))]) = e;
  }
  __syncthreads();

  // phase 2: thread -> (16-row block tid % 8, columns 4 (tid / 8) .. + 3)
  const int rb = tid & 7, quad = tid >> 3;
  uint32_t cw[4] = {0, 0, 0, 0}, mw[4] = {0, 0, 0, 0}, sel[4] = {0, 0, 0, 0};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    uint32_t w[4], key[4][4];
    const f4_t sc = *reinterpret_cast<const f4_t*>(&sc_s[16 * rb + 4 * c]);
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = e_s[pb_word(16 * rb + 4 * c + i, quad)];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // |code - 8| of four columns: below 8 the two's complement of the low three bits (8 for code 0)
      const uint32_t neg = (~w[i] & 0x08080808u) >> 3;
      const uint32_t m = ((w[i] & 0x07070707u) ^ ((neg << 3) - neg)) + neg;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        key[b][i] = __float_as_uint((float)((m >> (8 * b)) & 0xFFu) * sc[i]) | ((w[i] >> (8 * b)) & 0xFFu);
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint32_t h0 = max(key[b][0], key[b][1]), l0 = min(key[b][0], key[b][1]);
      const uint32_t h1 = max(key[b][2], key[b][3]), l1 = min(key[b][2], key[b][3]);
      const uint32_t first = max(h0, h1), second = max(min(h0, h1), max(l0, l1));
      // in row order: the larger 3 - n % 4 is the earlier row
      const uint32_t lo = max(first & 0x3Fu, second & 0x3Fu), hi = min(first & 0x3Fu, second & 0x3Fu);
      cw[b] |= ((lo & 0xFu) << (4 * c)) | ((hi & 0xFu) << (16 + 4 * c));
      mw[b] |= ((lo >> 4) | ((hi >> 4) << 2)) << (4 * c);     // each 3 - position: complemented below
      if constexpr (MASK) {
        sel[b] |= ((first >> 6) & 1u) << (4 * c + 3 - ((first >> 4) & 3u));
        sel[b] |= ((second >> 6) & 1u) << (4 * c + 3 - ((second >> 4) & 3u));
      }
    }
  }
  // transposed pack: row k, reduction n
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int64_t slotT = packed_slot(k0 + 4 * quad + b, nc, N / 128);
    codesT[8 * slotT + rb] = cw[b];
    metaT[8 * slotT + rb] = (uint16_t)~mw[b];
  }
  if constexpr (MASK) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i)
      e_s[pb_word(16 * rb + i, quad)] = ((sel[0] >> i) & 1u) | (((sel[1] >> i) & 1u) << 8) | (((sel[2] >> i) & 1u) << 16) |
                                        (((sel[3] >> i) & 1u) << 24);
    __syncthreads();
    // rows of the tile: thread -> (row tid / 8 + 32 j, 16 bytes at column 16 (tid % 8))
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = (tid >> 3) + 32 * j;
      *reinterpret_cast<u32x4_t*>(mask_rc + (n0 + row) * K + k0 + 16 * (tid & 7)) =
          *reinterpret_cast<const u32x4_t*>(&e_s[pb_word(row, 4 * (tid & 7))]);
    }
  }
}

// fp16 transpose out[c][r] = in[r][c] of a row-major [R x C] matrix, through a 64 x 64 LDS tile.
__global__ void __launch_bounds__(256)
k_transpose16(const uint16_t* __restrict__ in, int64_t R, int64_t C, uint16_t* __restrict__ out) {
  __shared__ uint16_t t[64][66];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int rr = ty + 4 * i;
    if (r0 + rr < R && c0 + tx < C) t[rr][tx] = in[(r0 + rr) * C + c0 + tx];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int cc = ty + 4 * i;
    if (c0 + cc < C && r0 + tx < R) out[(c0 + cc) * R + r0 + tx] = t[tx][cc];
  }
}

// R [r, N] row-major -> R^T in 32 x 16 tiles: element (n, j) at ((n / 32) (r / 16) + j / 16) 512 +
// (n % 32) 16 + j % 16, rows n >= N of the last tile zero. One thread per output element, in
// output order (a one-time pack: the strided reads do not matter).
__global__ void __launch_bounds__(256) k_tile_rt(const uint16_t* __restrict__ R, int64_t r, int64_t N,
                                                 uint16_t* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t total = (N + 31) / 32 * 32 * r;
  if (i >= total) return;
  const int64_t tile = i >> 9, within = i & 511;
  const int64_t tn = tile / (r >> 4), tj = tile - tn * (r >> 4);
  const int64_t n = 32 * tn + (within >> 4), j = 16 * tj + (within & 15);
  out[i] = n < N ? R[j * N + n] : (uint16_t)0;
}

// 4-bit AbsMax pack of one adapter factor laid out as [rows, len] (row-major view of a transposed
// source: element (row, col) is src[col * ld + row]), groups of 128 along len (the last group of a
// row may be shorter). Sixteen consecutive threads share one (row, group): thread i of them codes
// the 8 elements at col = 128 g + 8 i into one 32-bit word (element 2c in nibble c, 2c + 1 in
// nibble c + 4), the group's absmax comes from a 16-lane shuffle, and thread 0 writes the scale.
__global__ void __launch_bounds__(256)
k_pack_adapter_q(const uint16_t* __restrict__ src, int64_t ld, int64_t rows, int64_t len, uint32_t* __restrict__ codes,
                 uint16_t* __restrict__ scales, int* __restrict__ status) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t ng = (len + 127) / 128;
  const int64_t pair = t / 16;
  const int i = (int)(t % 16);
  const int64_t row = pair / ng, g = pair % ng;
  const int64_t col0 = 128 * g + 8 * i;
  const bool valid = row < rows && col0 < len;
  float v[8];
  float amax = 0.f;
  int bad = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    v[e] = valid ? h_bits_to_f(src[(col0 + e) * ld + row]) : 0.f;
    if (!__builtin_isfinite(v[e])) bad = 1;
    amax = fmaxf(amax, fabsf(v[e]));
  }
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 16));
  if (valid && bad) atomicOr(status, 1);
  // s16 = fp16_RNE(fp32 absmax / 7), IEEE division; codes against the stored s16 in double precision
  const _Float16 s16 = (_Float16)__fdiv_rn(amax, 7.0f);
  const double sd = (double)(float)s16;
  uint32_t word = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    double q = sd > 0.0 ? rint((double)v[e] / sd) : 0.0;
    q = q < -7.0 ? -7.0 : (q > 7.0 ? 7.0 : q);
    const uint32_t u = (uint32_t)((int)q + 8);
    word |= u << (4 * (e >> 1) + 16 * (e & 1));
  }
  if (!valid) return;
  codes[row * (len / 8) + col0 / 8] = word;
  if (i == 0) scales[row * ng + g] = __builtin_bit_cast(uint16_t, s16);
}

}  // namespace

extern "C" int slim_pack_adapter_q(const uint16_t* L, const uint16_t* R, int64_t K, int64_t N, int64_t r, uint8_t* Lq,
                                   uint16_t* Ls, uint8_t* Rq, uint16_t* Rs, void* stream) {
  if (!L || !R || !Lq || !Ls || !Rq || !Rs) return SLIM_EINVAL;
  if (K < 128 || N < 1 || r < 32 || r % 32 || K % 128 || K >= (int64_t(1) << 31) || N >= (int64_t(1) << 31) ||
      r >= 65536)
    return SLIM_ESHAPE;
  if (!slim_aligned16(L) || !slim_aligned16(R) || !slim_aligned16(Lq) || !slim_aligned16(Ls) || !slim_aligned16(Rq) ||
      !slim_aligned16(Rs))
    return SLIM_EALIGN;
  hipStream_t s = (hipStream_t)stream;
  int* d_status = nullptr;
  if (hipMalloc(&d_status, sizeof(int)) != hipSuccess) return SLIM_EDEVICE;
  int h_status = 0;
  int rc = SLIM_OK;
  do {
    if (hipMemsetAsync(d_status, 0, sizeof(int), s) != hipSuccess) { rc = SLIM_EDEVICE; break; }
    // L^T [r, K]: element (j, k) = L[k * r + j]; R^T [N, r]: element (n, j) = R[j * N + n]
    const int64_t tl = r * ((K + 127) / 128) * 16, tr = N * ((r + 127) / 128) * 16;
    {
      SlimKernelTimer timer("pack_adapter_q", s);
      SLIM_LAUNCH(timer, k_pack_adapter_q, dim3((unsigned)((tl + 255) / 256)), dim3(256), s, L, r, r, K,
                  reinterpret_cast<uint32_t*>(Lq), Ls, d_status);
    }
    {
      SlimKernelTimer timer("pack_adapter_q", s);
      SLIM_LAUNCH(timer, k_pack_adapter_q, dim3((unsigned)((tr + 255) / 256)), dim3(256), s, R, N, N, r,
                  reinterpret_cast<uint32_t*>(Rq), Rs, d_status);
    }
    if (hipGetLastError() != hipSuccess) { rc = SLIM_EDEVICE; break; }
    if (hipMemcpyAsync(&h_status, d_status, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) { rc = SLIM_EDEVICE; break; }
    if (h_status & 1) rc = SLIM_ENONFINITE;
  } while (0);
  (void)hipFree(d_status);
  return rc;
}

extern "C" int slim_pack_adapter(const uint16_t* L, const uint16_t* R, int64_t K, int64_t N, int64_t r, uint16_t* Lt,
                                 uint16_t* Rt, void* stream) {
  if (!L || !R || !Lt || !Rt) return SLIM_EINVAL;
  if (K < 1 || N < 1 || r < 16 || r % 16 || K >= (int64_t(1) << 31) || N >= (int64_t(1) << 31) || r >= 65536)
    return SLIM_ESHAPE;
  if (!slim_aligned16(L) || !slim_aligned16(R) || !slim_aligned16(Lt) || !slim_aligned16(Rt)) return SLIM_EALIGN;
  hipStream_t s = (hipStream_t)stream;
  {
    SlimKernelTimer timer("pack_adapter", s);
    SLIM_LAUNCH(timer, k_transpose16, dim3((unsigned)((r + 63) / 64), (unsigned)((K + 63) / 64)), dim3(256), s, L, K, r,
                Lt);
  }
  {
    SlimKernelTimer timer("pack_adapter", s);
    const int64_t total = (N + 31) / 32 * 32 * r;
    SLIM_LAUNCH(timer, k_tile_rt, dim3((unsigned)((total + 255) / 256)), dim3(256), s, R, r, N, Rt);
  }
  return hipGetLastError() == hipSuccess ? SLIM_OK : SLIM_EDEVICE;
}

namespace {

int pack_forward(const float* W, int64_t N, int64_t K, uint8_t* codes, uint8_t* meta, uint16_t* scales,
                 uint8_t* mask, const double* alpha, void* stream) {
  int st = slim_check_pack(W, N, K, codes, meta, scales, mask);
  if (st != SLIM_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  int* d_status = nullptr;
  if (hipMalloc(&d_status, sizeof(int)) != hipSuccess) return SLIM_EDEVICE;
  int h_status = 0;
  int rc = SLIM_OK;
  const int64_t total16 = N * (K / 16);
  const int64_t blocks = (total16 + kPackThreads - 1) / kPackThreads;
  do {
    if (hipMemsetAsync(d_status, 0, sizeof(int), s) != hipSuccess) { rc = SLIM_EDEVICE; break; }
    {
      SlimKernelTimer timer("pack", s);
      SLIM_LAUNCH(timer, k_pack, dim3((unsigned)blocks), dim3(kPackThreads), s,
                  reinterpret_cast<const u32x4_t*>(W), total16, K / 128, reinterpret_cast<uint32_t*>(codes),
                  reinterpret_cast<uint16_t*>(meta), scales, reinterpret_cast<u32x4_t*>(mask), d_status, alpha);
    }
    if (hipGetLastError() != hipSuccess) { rc = SLIM_EDEVICE; break; }
    if (hipMemcpyAsync(&h_status, d_status, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) { rc = SLIM_EDEVICE; break; }
    if (h_status & 1) rc = SLIM_ENONFINITE;
    else if (h_status & 2) rc = SLIM_ERANGE;
  } while (0);
  (void)hipFree(d_status);
  return rc;
}

}  // namespace

extern "C" int slim_pack(const float* W, int64_t N, int64_t K, uint8_t* codes, uint8_t* meta,
                         uint16_t* scales, uint8_t* mask, void* stream) {
  return pack_forward(W, N, K, codes, meta, scales, mask, nullptr, stream);
}

extern "C" int slim_pack_alpha(const float* W, int64_t N, int64_t K, const double* alpha, uint8_t* codes,
                               uint8_t* meta, uint16_t* scales, uint8_t* mask, void* stream) {
  if (!alpha) return SLIM_EINVAL;
  if ((uintptr_t)alpha & 7u) return SLIM_EALIGN;
  return pack_forward(W, N, K, codes, meta, scales, mask, alpha, stream);
}

extern "C" int slim_pack_bwd(const uint8_t* codes, const uint8_t* meta, const uint16_t* scales, int64_t N,
                             int64_t K, uint8_t* codesT, uint8_t* metaT, uint16_t* scalesT, uint8_t* mask_rc,
                             void* stream) {
  int st = slim_check_pack_bwd(codes, meta, scales, N, K, codesT, metaT, scalesT, mask_rc);
  if (st != SLIM_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  int* d_status = nullptr;
  if (hipMalloc(&d_status, sizeof(int)) != hipSuccess) return SLIM_EDEVICE;
  int h_status = 0;
  int rc = SLIM_OK;
  do {
    if (hipMemsetAsync(d_status, 0, sizeof(int), s) != hipSuccess) { rc = SLIM_EDEVICE; break; }
    {
      dim3 grid((unsigned)(K / kBT), (unsigned)(N / kBT));
      SlimKernelTimer timer("pack_bwd", s);
      auto kernel = mask_rc ? k_pack_bwd<true> : k_pack_bwd<false>;
      SLIM_LAUNCH(timer, kernel, grid, dim3(256), s, reinterpret_cast<const uint32_t*>(codes),
                  reinterpret_cast<const uint16_t*>(meta), scales, N, K, reinterpret_cast<uint32_t*>(codesT),
                  reinterpret_cast<uint16_t*>(metaT), scalesT, mask_rc, d_status);
    }
    if (hipGetLastError() != hipSuccess) { rc = SLIM_EDEVICE; break; }
    if (hipMemcpyAsync(&h_status, d_status, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) { rc = SLIM_EDEVICE; break; }
    if (h_status & 2) rc = SLIM_ERANGE;
  } while (0);
  (void)hipFree(d_status);
  return rc;
}

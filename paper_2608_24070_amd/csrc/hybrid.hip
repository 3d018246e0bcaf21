// hybrid.hip - PATCH's hybrid dense / 2:4 tile layer (PATCH chapter, "Efficient deployment of
// PATCH"; appendix "STOICC Integration"): a weight whose 128 x 128 tiles are either dense fp16 or
// 2:4-sparse fp16, multiplied in one GEMM, Y = X Wp^T.
//
//   k_hybrid_pack    one thread per 16 positions of a row: the tile's payload, dense (fp16 values)
//                    or compressed (the two largest of each group of four as fp16, lower position
//                    first, and one index half-word per 16 positions), at the offset the host
//                    computed from the tile map
//   k_hybrid_gemm    128 x 128 output tiles of Y^T (rows n, columns m); a chunk of 128 along K is
//                    one weight tile, dense (v_mfma_f32_32x32x16_f16) or sparse
//                    (v_smfmac_f32_32x32x32_f16, half the MFMA issue for the same K); both write
//                    the same 32 x 32 accumulator layout, so a tile row may mix them freely
//   k_hybrid_few     up to 64 rows: 16 or 32 rows of Y^T per block, K shared by its waves
//   k_hybrid_reduce  the split partials of the GEMM, summed in a fixed order
#include <new>

#include "slim_device.h"
#include "slim_host.h"
#include "slim_timing.h"

namespace {

constexpr int kHT = 128;                        // weight tile edge
constexpr int kHDense = kHT * kHT * 2;          // bytes of a dense tile
constexpr int kHSparse = kHT * kHT + kHT * kHT / 8;
constexpr uint64_t kHSparseBit = 1ull << 63;
constexpr int kHThreads = 256;
constexpr int kHRing = 3;
constexpr int kHMaxChunks = 256;               // K <= 32768

// ------------------------------------------------------------------------------------- pack
__global__ void __launch_bounds__(kHThreads)
k_hybrid_pack(const float* __restrict__ W, int64_t N, int64_t K, const uint64_t* __restrict__ info,
              uint8_t* __restrict__ payload, int* __restrict__ status) {
  const int64_t t = (int64_t)blockIdx.x * kHThreads + threadIdx.x;
  const int64_t per_row = K / 16;
  if (t >= N * per_row) return;
  const int64_t n = t / per_row, j = t % per_row;
  const int64_t tk = (16 * j) / kHT, tkn = K / kHT;
  const uint64_t ti = info[(n / kHT) * tkn + tk];
  const uint64_t off = ti & ~kHSparseBit;
  const int r = (int)(n % kHT), kk = (int)((16 * j) % kHT);
  const float4* src = reinterpret_cast<const float4*>(W + n * K + 16 * j);
  float w[16];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 v = src[q];
    w[4 * q] = v.x;
    w[4 * q + 1] = v.y;
    w[4 * q + 2] = v.z;
    w[4 * q + 3] = v.w;
  }
  int bad = 0;
#pragma unroll
  for (int p = 0; p < 16; ++p)
    if (!__builtin_isfinite(w[p])) bad = 1;
  if (bad) atomicOr(status, 1);
  if (!(ti & kHSparseBit)) {
    h8_t lo, hi;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      lo[p] = (_Float16)w[p];
      hi[p] = (_Float16)w[8 + p];
    }
    u32x4_t* dst = reinterpret_cast<u32x4_t*>(payload + off + (uint64_t)r * 256 + 2 * kk);
    dst[0] = __builtin_bit_cast(u32x4_t, lo);
    dst[1] = __builtin_bit_cast(u32x4_t, hi);
    return;
  }
  h8_t vals;
  uint32_t half = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    float a[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) a[p] = fabsf(w[4 * c + p]);
    int i0 = -1, i1 = -1;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      int rank = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (q != p && (a[q] > a[p] || (a[q] == a[p] && q < p))) ++rank;
      if (rank < 2) {
        if (i0 < 0) i0 = p;
        else i1 = p;
      }
    }
    vals[2 * c] = (_Float16)w[4 * c + i0];
    vals[2 * c + 1] = (_Float16)w[4 * c + i1];
    half |= (uint32_t)(i0 | (i1 << 2)) << (4 * c);
  }
  // the tile's half (positions 0..63 or 64..127): 128 rows x 64 bytes of values, then 128 rows x
  // 8 bytes of index words
  const uint64_t hb = off + (uint64_t)(kHSparse / 2) * (uint64_t)(kk >> 6);
  const int kh = kk & 63;
  *reinterpret_cast<u32x4_t*>(payload + hb + (uint64_t)r * 64 + kh) = __builtin_bit_cast(u32x4_t, vals);
  *reinterpret_cast<uint16_t*>(payload + hb + 8192 + (uint64_t)r * 8 + 2 * (kh / 16)) = (uint16_t)half;
}

// ------------------------------------------------------------------------------------- GEMM
// A block computes 256 rows (two weight-tile rows) x 128 columns with 8 waves of 64 x 64; each
// 128-row half has its own tile kind per chunk. Ring stages hold 64 positions of K (half a weight
// tile) of both tile rows and of the 128 activation rows, 48 KiB per stage, three stages, two
// ahead: everything reaches LDS by direct loads (buffer_load ... lds, 16 bytes per lane), so no
// register holds data in flight. Waves 0-3 load tile row 0's weights and waves 4-7 tile row 1's:
// 4 loads per wave for a dense half-tile, 2 for a 2:4 one (+1 in the group's first wave, the
// index words); every wave loads 2 of the activations. The wait before stage s lets the loads of
// stage s + 1 be in flight, a count known from its kinds (a switch over the three possible
// immediates). LDS layouts (16-byte slots XOR-swizzled so that a wave's reads of one slot over
// consecutive rows hit distinct banks), per tile row at 16384 tr:
//   dense weights  row r (0..127): 128 bytes, slot s at s ^ (r % 8)
//   2:4 weights    values: row r 64 bytes, slot s at s ^ ((r / 4) % 2); index words at 8192 + 8 r
//   activations    (at 32768) row m (0..127): 128 bytes, slot s at s ^ (m % 8)
constexpr int kHStageK = 64;
constexpr int kHRows = 256;                   // output rows per block
constexpr int kHGemmThreads = 512;
struct HybridStage {
  uint8_t a[32768];
  uint8_t x[16384];
};

struct HybridArgs {
  const uint16_t* X;
  const uint64_t* info;
  const uint8_t* payload;
  float* out;          // Y [M, N] (one split) or partials [split][M][N]
  int64_t M, N, K;
  int64_t payload_bytes;
  int chunks_per_split;
  int chunks_per_sum;  // chunks that one accumulator sums before they are added to the others'
};

// One block per CU: 144 KiB of ring. CARRY: a split's sum is made of several (chunks_per_sum).
template <bool CARRY>
__global__ void __launch_bounds__(kHGemmThreads, 1)
k_hybrid_gemm(HybridArgs g) {
  // one variable per stage, selected by compile-time indices
  __shared__ __attribute__((aligned(16))) HybridStage st0, st1, st2;
  // the block's tile-info words (two tile rows), read once before any direct load: afterwards an
  // info word comes from LDS into scalar registers, where the loads' offsets must be
  __shared__ uint64_t infos[2][kHMaxChunks];
  auto ring = [&](auto zc) -> HybridStage& {
    constexpr int z = decltype(zc)::value;
    if constexpr (z == 0) return st0;
    else if constexpr (z == 1) return st1;
    else return st2;
  };
  // the wave index in a scalar register: load counts and waits are wave-uniform branches
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave >> 1, wm = wave & 1;       // rows 64 wn .. + 63 of the block, columns 64 wm ..
  const int tr = wn >> 1;                        // the wave's tile row (for compute)
  const int lt = wave >> 2, lw = wave & 3;       // the tile row this wave loads, and its rank there
  const int l32 = lane & 31, h = lane >> 5;
  const int64_t n0 = (int64_t)blockIdx.x * kHRows, m0 = (int64_t)blockIdx.y * kHT;
  const int64_t chunks = g.K / kHT;
  const int64_t c_begin = (int64_t)blockIdx.z * g.chunks_per_split;
  const int64_t c_end = c_begin + g.chunks_per_split < chunks ? c_begin + g.chunks_per_split : chunks;
  const int64_t s_begin = 2 * c_begin, s_end = 2 * c_end;
  const int64_t tn0 = n0 / kHT;
  // a last block of a 128-row remainder (N % 256 == 128) loads and computes tile row 0 twice; the
  // second copy's rows lie past N and are never stored
  const int64_t tn1 = tn0 + 1 < g.N / kHT ? tn0 + 1 : tn0;
  for (int64_t c = c_begin + tid; c < c_end; c += kHGemmThreads) {
    infos[0][c - c_begin] = g.info[tn0 * chunks + c];
    infos[1][c - c_begin] = g.info[tn1 * chunks + c];
  }
  __syncthreads();

  const rsrc_t rw = make_rsrc(g.payload, g.payload_bytes);
  const int64_t xrows = g.M - m0 < kHT ? g.M - m0 : kHT;
  const rsrc_t rx = make_rsrc(g.X + m0 * g.K, xrows * g.K * 2);     // rows past M read as zero
  // per-lane source offsets of the wave's loads
  uint32_t ad[4], as[2], xo[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int p = 4 * lw + i, row = 8 * p + (lane >> 3), phys = lane & 7;
    ad[i] = (uint32_t)row * 256u + 16u * (uint32_t)(phys ^ (row & 7));
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int p = 2 * lw + i, row = 16 * p + (lane >> 2), phys = lane & 3;
    as[i] = (uint32_t)row * 64u + 16u * (uint32_t)(phys ^ ((row >> 2) & 1));
    const int px = 2 * wave + i, rx_row = 8 * px + (lane >> 3), pxs = lane & 7;
    xo[i] = (uint32_t)rx_row * (uint32_t)g.K * 2u + 16u * (uint32_t)(pxs ^ (rx_row & 7));
  }
  const uint32_t ami = 8192u + 16u * (uint32_t)lane;     // the half's index words, 16 bytes per lane

  auto kind_of = [&](int t, int64_t s) -> uint64_t {
    const uint64_t v = infos[t][(s >> 1) - c_begin];
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
  };
  auto clamp_s = [&](int64_t s) -> int64_t { return s < s_end ? s : s_end - 1; };   // past the end: a dead slot
  // loads this wave issues for stage s
  auto loads_of = [&](int64_t s) -> int {
    return 2 + ((kind_of(lt, clamp_s(s)) & kHSparseBit) ? (lw == 0 ? 3 : 2) : 4);
  };
  auto issue = [&](int64_t s, auto zc) {
    const int64_t sc = clamp_s(s);
    const uint64_t ti = kind_of(lt, sc);
    const uint32_t toff = (uint32_t)(ti & ~kHSparseBit), half = (uint32_t)(sc & 1);
    HybridStage& S = ring(zc);
    uint8_t* A = &S.a[16384 * lt];
    if (!(ti & kHSparseBit)) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr_t)&A[(4 * lw + i) * 1024], 16, ad[i] + 128u * half, toff,
                                                 0, 0);
    } else {
      const uint32_t soff = toff + (uint32_t)(kHSparse / 2) * half;
#pragma unroll
      for (int i = 0; i < 2; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr_t)&A[(2 * lw + i) * 1024], 16, as[i], soff, 0, 0);
      if (lw == 0) __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr_t)&A[8192], 16, ami, soff, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)&S.x[(2 * wave + i) * 1024], 16, xo[i],
                                               (uint32_t)(sc * kHStageK * 2), 0, 0);
  };

  // the sum of chunks_per_sum chunks, and that of the sums before it
  f16_t acc[2][2], tot[CARRY ? 2 : 1][CARRY ? 2 : 1];
#pragma unroll
  for (int fn = 0; fn < 2; ++fn)
#pragma unroll
    for (int fm = 0; fm < 2; ++fm)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[fn][fm][e] = 0.f;
        if (CARRY) tot[fn][fm][e] = 0.f;
      }
  [[maybe_unused]] auto carry = [&]() {
#pragma unroll
    for (int fn = 0; fn < 2; ++fn)
#pragma unroll
      for (int fm = 0; fm < 2; ++fm) {
        tot[fn][fm] += acc[fn][fm];
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[fn][fm][e] = 0.f;
      }
  };

  // The compute phase reads LDS with ds_read instructions written out, and waits for them itself:
  // the compiler cannot tell which ring slot a direct load writes, so for reads it can see it would
  // wait for every direct load in flight, the next stage's included. Each wait names the registers
  // it completes, so no instruction using them is scheduled before it.
  auto rd16 = [](uint32_t addr) -> u32x4_t {
    u32x4_t v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr));
    return v;
  };
  auto rd_u16 = [](uint32_t addr) -> uint32_t {
    uint32_t v;
    asm volatile("ds_read_u16 %0, %1" : "=v"(v) : "v"(addr));
    return v;
  };
  struct DenseOps {
    u32x4_t a[2], b[2];
  };
  struct SparseOps {
    u32x4_t a[2], b[4];
    uint32_t i[2];
  };
  auto wait_dense = [](DenseOps& o) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(o.a[0]), "+v"(o.a[1]), "+v"(o.b[0]), "+v"(o.b[1]));
  };
  auto wait_sparse = [](SparseOps& o) {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(o.a[0]), "+v"(o.a[1]), "+v"(o.b[0]), "+v"(o.b[1]), "+v"(o.b[2]), "+v"(o.b[3]), "+v"(o.i[0]),
                   "+v"(o.i[1]));
  };
  // per-lane LDS byte offsets inside a stage (rows of this lane's fragments) of the first read; read t's 16-byte slot
  // is the first one's with 2 t (dense, activations of a 2:4 step 4 t and 4 t + 2) in its upper bits
  uint32_t ra_d[2], ra_s[2], ri_s[2], rx_[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int r = 64 * (wn & 1) + 32 * f + l32, m = 64 * wm + 32 * f + l32;   // r: row within the tile row
    ra_d[f] = 16384u * (uint32_t)tr + (uint32_t)r * 128u + 16u * (uint32_t)(h ^ (r & 7));
    ra_s[f] = 16384u * (uint32_t)tr + (uint32_t)r * 64u + 16u * (uint32_t)(h ^ ((r >> 2) & 1));
    ri_s[f] = 16384u * (uint32_t)tr + 8192u + (uint32_t)r * 8u + 2u * (uint32_t)h;
    rx_[f] = 32768u + (uint32_t)m * 128u + 16u * (uint32_t)(h ^ (m & 7));
  }

  auto compute = [&](auto zc, bool sparse) {
    const uint32_t base = (uint32_t)(uintptr_t)(lds_ptr_t)&ring(zc).a[0];   // the stage (a, then x)
    // opaque in place, so that no stage's addresses are kept across the loop: they would take the second
    // accumulators' registers
    if constexpr (CARRY)
      asm volatile("" : "+v"(ra_d[0]), "+v"(ra_d[1]), "+v"(ra_s[0]), "+v"(ra_s[1]), "+v"(ri_s[0]), "+v"(ri_s[1]),
                        "+v"(rx_[0]), "+v"(rx_[1]));
    if (!sparse) {
      auto read = [&](int t, DenseOps& o) {
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          o.a[f] = rd16((ra_d[f] ^ (32u * t)) + base);
          o.b[f] = rd16((rx_[f] ^ (32u * t)) + base);
        }
      };
      DenseOps o[2];
      read(0, o[0]);
      wait_dense(o[0]);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (t < 3) read(t + 1, o[(t + 1) & 1]);
        const DenseOps& c = o[t & 1];
#pragma unroll
        for (int fn = 0; fn < 2; ++fn)
#pragma unroll
          for (int fm = 0; fm < 2; ++fm)
            acc[fn][fm] = mfma32(__builtin_bit_cast(h8_t, c.a[fn]), __builtin_bit_cast(h8_t, c.b[fm]), acc[fn][fm]);
        if (t < 3) wait_dense(o[(t + 1) & 1]);
      }
    } else {
      auto read = [&](int t, SparseOps& o) {
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          // lane group h holds the 16 positions 32 t + 16 h .. + 15 of its row
          o.a[f] = rd16((ra_s[f] ^ (32u * t)) + base);
          o.i[f] = rd_u16(ri_s[f] + 4u * t + base);
          o.b[2 * f] = rd16((rx_[f] ^ (64u * t)) + base);
          o.b[2 * f + 1] = rd16((rx_[f] ^ (64u * t + 32u)) + base);
        }
      };
      SparseOps o[2];
      read(0, o[0]);
      wait_sparse(o[0]);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        if (t < 1) read(t + 1, o[1]);
        const SparseOps& c = o[t & 1];
#pragma unroll
        for (int fn = 0; fn < 2; ++fn)
#pragma unroll
          for (int fm = 0; fm < 2; ++fm)
            acc[fn][fm] = smfmac32(__builtin_bit_cast(h8_t, c.a[fn]),
                                   cat16(__builtin_bit_cast(h8_t, c.b[2 * fm]), __builtin_bit_cast(h8_t, c.b[2 * fm + 1])),
                                   acc[fn][fm], (int)c.i[fn], 0);
        if (t < 1) wait_sparse(o[1]);
      }
    }
  };

  // stage s in slot z: the wave's loads of stage s have landed once only those of s + 1 are
  // outstanding; the barrier then makes every wave's loads visible and ends every read of the slot
  // that stage s + 2 refills
  auto wait_ahead = [&](int n) {
    switch (n) {
      case 4: __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_wait(4)); break;
      case 5: __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_wait(5)); break;
      default: __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_wait(6)); break;
    }
  };
  [[maybe_unused]] int left = 2 * g.chunks_per_sum;      // stages until the next carry
  auto step = [&](int64_t s, auto zc) {
    constexpr int z = decltype(zc)::value;
    const int ahead = loads_of(s + 1);
    __builtin_amdgcn_sched_barrier(0);
    wait_ahead(ahead);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    issue(s + 2, std::integral_constant<int, (z + 2) % kHRing>{});
    compute(zc, (kind_of(tr, s) & kHSparseBit) != 0);
    if constexpr (CARRY)
      if (--left == 0) {
        carry();
        left = 2 * g.chunks_per_sum;
      }
  };

  if (s_begin < s_end) {
    issue(s_begin, std::integral_constant<int, 0>{});
    issue(s_begin + 1, std::integral_constant<int, 1>{});
    for (int64_t s = s_begin; s < s_end; s += kHRing) {
      step(s, std::integral_constant<int, 0>{});
      if (s + 1 < s_end) step(s + 1, std::integral_constant<int, 1>{});
      if (s + 2 < s_end) step(s + 2, std::integral_constant<int, 2>{});
    }
    // no direct load may still be writing LDS when the workgroup ends
    __builtin_amdgcn_s_waitcnt(0);
  }

  if constexpr (CARRY) carry();

  // D[i][j] of a 32x32 fragment: lane j + 32 ((i / 4) % 2), element 4 (i / 8) + i % 4
  float* out = g.out + (int64_t)blockIdx.z * g.M * g.N;
#pragma unroll
  for (int fm = 0; fm < 2; ++fm) {
    const int64_t m = m0 + 64 * wm + 32 * fm + l32;
    if (m >= g.M) continue;
#pragma unroll
    for (int fn = 0; fn < 2; ++fn)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t nn = n0 + 64 * wn + 32 * fn + 8 * q + 4 * h;
        if (nn >= g.N) continue;
        const f16_t& v = CARRY ? tot[CARRY ? fn : 0][CARRY ? fm : 0] : acc[fn][fm];
        *reinterpret_cast<f4_t*>(out + m * g.N + nn) = f4_t{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
      }
  }
}

// ------------------------------------------------------------------------------------- few rows
// Bound by the reading of the weights. A block takes 16 RF rows of one tile row and 16 MF rows of X with W waves
// that share K chunk by chunk (wave w takes chunks w, w + W, ...), and adds their sums through LDS in a fixed order:
// no partials in memory and no second launch. A wave loads its weights and its activations (from the L2) itself,
// two chunks in flight, X and dense weights as whole rows of a chunk (256 bytes); it turns them through its own
// LDS, without a barrier, into the MFMA's operand layout, which loaded directly is 64-byte pieces of 16 rows
// and reads every 128-byte line twice (16 x 11008 x 4096: 20.3 us; 13.7 now, 62 MB at 4.5 TB/s; 25.0 in
// 128-column tiles and partials). Dense chunks run four v_mfma_f32_16x16x32_f16, 2:4 ones two
// v_smfmac_f32_16x16x64_f16 per fragment, on the same X registers: lane (i, g = lane / 16) holds positions
// 8 g .. + 7 of each 32 of row i. 2:4 values (64-byte rows) and index words lie as the lanes take them.
template <int RF, int MF, int W>
__global__ void __launch_bounds__(64 * W)
k_hybrid_few(HybridArgs g) {
  // two buffers of 4 KiB per wave, 16 rows of 256 bytes each; the sums at the end
  static_assert(RF * MF <= 8, "a wave's sums fit its two buffers");
  __shared__ u32x4_t stage[W][2][256];
  f4_t* part = reinterpret_cast<f4_t*>(&stage[0][0][0]);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  const int64_t n0 = (int64_t)blockIdx.x * 16 * RF, m0 = (int64_t)blockIdx.y * 16 * MF;
  const int chunks = (int)(g.K / kHT);
  const uint64_t* info = g.info + (n0 / kHT) * chunks;
  const int rt = (int)(n0 % kHT), r0 = rt + li;
  const rsrc_t rw = make_rsrc(g.payload, g.payload_bytes), rx = make_rsrc(g.X + m0 * g.K, (g.M - m0) * g.K * 2);
  // whole rows of 256 bytes: load i of a fragment takes row 4 i + lg, 16-byte slot li (X rows past M read as
  // zero); the wave's LDS keeps slot s of row r at s ^ r, so neither the writes nor the reads below, lane (li, lg)
  // taking slot 4 t + lg of row li, conflict
  uint32_t xo[MF][4];
#pragma unroll
  for (int m = 0; m < MF; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) xo[m][i] = (uint32_t)(16 * m + 4 * i + lg) * (uint32_t)g.K * 2u + 16u * (uint32_t)li;
  const uint32_t od = (uint32_t)(rt + lg) * 256u + 16u * (uint32_t)li, os = (uint32_t)r0 * 64u + 16u * (uint32_t)lg,
                 oi = 8192u + (uint32_t)r0 * 8u + 2u * (uint32_t)lg;
  uint32_t wr[4], rd[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    wr[i] = (uint32_t)(16 * (4 * i + lg) + (li ^ (4 * i + lg)));
    rd[i] = (uint32_t)(16 * li + ((4 * i + lg) ^ li));
  }
  u32x4_t (*mine)[256] = stage[wave];
  struct Set {
    u32x4_t w[RF][4], x[MF][4];
    uint32_t i[RF][2];
    bool sparse;
  };
  auto load16 = [](const rsrc_t& r, uint32_t off, uint32_t base) {
    return __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, off, base, 0));
  };
  auto load = [&](Set& S, int c) {
    const uint64_t ti = info[c];
    const uint32_t toff = (uint32_t)(ti & ~kHSparseBit);
    S.sparse = (ti & kHSparseBit) != 0;
    if (S.sparse) {
#pragma unroll
      for (int f = 0; f < RF; ++f)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          S.w[f][t] = load16(rw, os + 1024u * f, toff + (uint32_t)(kHSparse / 2) * t);
          S.i[f][t] = __builtin_amdgcn_raw_buffer_load_b16(rw, oi + 128u * f, toff + (uint32_t)(kHSparse / 2) * t, 0);
        }
    } else {
#pragma unroll
      for (int f = 0; f < RF; ++f)
#pragma unroll
        for (int t = 0; t < 4; ++t) S.w[f][t] = load16(rw, od + 4096u * f + 1024u * t, toff);
    }
#pragma unroll
    for (int m = 0; m < MF; ++m)
#pragma unroll
      for (int t = 0; t < 4; ++t) S.x[m][t] = load16(rx, xo[m][t], (uint32_t)c * 256u);
  };
  // the sum of two chunks, and that of the pairs before them: one sum of all chunks would be a chain of up to 28
  // chunks' roundings (32 x 11008 x 14336 is 3.3e-7 from 64 bits with it, 2.1e-7 on k_hybrid_gemm's splits)
  f4_t acc[RF][MF], tot[RF][MF];
#pragma unroll
  for (int f = 0; f < RF; ++f)
#pragma unroll
    for (int m = 0; m < MF; ++m) acc[f][m] = tot[f][m] = f4_t{0.f, 0.f, 0.f, 0.f};
  auto carry = [&]() {
#pragma unroll
    for (int f = 0; f < RF; ++f)
#pragma unroll
      for (int m = 0; m < MF; ++m) {
        tot[f][m] += acc[f][m];
        acc[f][m] = f4_t{0.f, 0.f, 0.f, 0.f};
      }
  };
  auto h8 = [](u32x4_t v) { return __builtin_bit_cast(h8_t, v); };
  auto compute = [&](Set& S) {
    auto turn = [&](u32x4_t (&v)[4], u32x4_t* buf) {
#pragma unroll
      for (int i = 0; i < 4; ++i) buf[wr[i]] = v[i];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = buf[rd[i]];
    };
#pragma unroll
    for (int m = 0; m < MF; ++m) turn(S.x[m], mine[m & 1]);
    if (!S.sparse)
#pragma unroll
      for (int f = 0; f < RF; ++f) turn(S.w[f], mine[(MF + f) & 1]);
    if (S.sparse) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int f = 0; f < RF; ++f)
#pragma unroll
          for (int m = 0; m < MF; ++m)
            acc[f][m] = smfmac16(h8(S.w[f][t]), cat16(h8(S.x[m][2 * t]), h8(S.x[m][2 * t + 1])), acc[f][m], (int)S.i[f][t], 0);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int f = 0; f < RF; ++f)
#pragma unroll
          for (int m = 0; m < MF; ++m) acc[f][m] = mfma16(h8(S.w[f][t]), h8(S.x[m][t]), acc[f][m]);
    }
  };
  Set A, B;
  int c = wave;
  if (c < chunks) {
    load(A, c);
    while (true) {
      if (c + W < chunks) load(B, c + W);
      compute(A);
      if (c + W >= chunks) break;
      if (c + 2 * W < chunks) load(A, c + 2 * W);
      compute(B);
      carry();
      if (c + 2 * W >= chunks) break;
      c += 2 * W;
    }
  }
  __syncthreads();
#pragma unroll
  for (int f = 0; f < RF; ++f)
#pragma unroll
    for (int m = 0; m < MF; ++m) part[(wave * RF * MF + f * MF + m) * 64 + lane] = tot[f][m] + acc[f][m];
  __syncthreads();
  // D[i][j] of a 16 x 16 fragment: lane j + 16 (i / 4), element i % 4
  for (int t = tid; t < 64 * RF * MF; t += 64 * W) {
    const int fr = t >> 6;
    f4_t q[4];
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const f4_t v = part[(w * RF * MF + fr) * 64 + lane];
      q[w % 4] = w < 4 ? v : q[w % 4] + v;
    }
    const f4_t o = (q[0] + q[1]) + (q[2] + q[3]);
    const int64_t m = m0 + 16 * (fr % MF) + li, nn = n0 + 16 * (fr / MF) + 4 * lg;
    if (m < g.M) *reinterpret_cast<f4_t*>(g.out + m * g.N + nn) = o;
  }
}

// Sums of the split partials, in an order fixed by the split count: 64 outputs (of four values) per block, the
// splits over four groups of threads with four loads in flight each, the groups' sums added through LDS. One
// thread per output walking all splits waited for every load in turn (112 splits: 28 us).
__global__ void __launch_bounds__(kHThreads)
k_hybrid_reduce(const float* __restrict__ part, int splits, int64_t count4, float* __restrict__ Y) {
  __shared__ f4_t sums[3][64];
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  const f4_t* p = reinterpret_cast<const f4_t*>(part) + (i < count4 ? i : count4 - 1);
  f4_t s = f4_t{0.f, 0.f, 0.f, 0.f};
  int z = grp;
  for (; z + 12 < splits; z += 16) {
    const f4_t v0 = p[z * count4], v1 = p[(z + 4) * count4], v2 = p[(z + 8) * count4], v3 = p[(z + 12) * count4];
    s += (v0 + v1) + (v2 + v3);
  }
  for (; z < splits; z += 4) s += p[z * count4];
  if (grp > 0) sums[grp - 1][lane] = s;
  __syncthreads();
  if (grp == 0 && i < count4) reinterpret_cast<f4_t*>(Y)[i] = (s + sums[0][lane]) + (sums[1][lane] + sums[2][lane]);
}

// Rows served by k_hybrid_few. Its weights are read once whatever M is, and X once per row block, so it is the
// faster one while X is small beside them; a wave's chunks are a serial chain of about 1 us each.
//   M <= 16: always (16 x 11008 x 4096: 13.7 us against 20.8, 16 x 1024 x 1024 3.0 against 7.8, 14336 x 14336 59
//     against 72; 512 x 14336 level at 12; the sums' chains are no longer than in the GEMM's splits)
//   M <= 32: unless few row blocks each have a long chain (32 x 512 x 14336: 18.7 against 13.9; 4096 x 11008
//     17.5 against 22.4, 11008 x 14336 52 against 59, 14336 x 14336 74 against 80)
//   M <= 64: in two halves, up to 4096 x 4096 (64 rows: 10.1 against 17.4, 2048 x 4096 7.6 against 12.4)
bool hybrid_few(int64_t M, int64_t N, int64_t K) {
  if (M <= 16) return true;
  if (M <= 32) return N > 2048 || K <= 8192;
  return M <= 64 && N <= 4096 && K <= 4096;
}

struct HybridPlan {
  bool few;
  int64_t tiles, splits, chunks_per_split, chunks_per_sum;
  size_t ws;
};

// Splits of K: the count of least estimated time. A block takes t0 = 4.5 us and 2 us per chunk (fitted at 64
// rows of 4096 x 4096 in 1 to 32 splits, 65 to 13 us a launch; with 256 blocks at work a chunk's 45 KB each
// make 5.8 TB/s), blocks run 256 at a time with the last split's shorter ones last, and the partials cost
// the reduction's launch, 3 us, and their writing and reading at 7 TB/s.
// Fewer splits sum more of K each. One accumulator for all of it rounds worse than the most splits that are
// considered, s0 (no more than two rounds of blocks): 64 x 14336 x 14336 in four splits instead of ten was 3.3e-7 from
// 64 bits instead of 2.2e-7. So a split adds up sums of chunks_per_sum chunks, as many as leave the rounding no larger
// than s0's added one after another: a sum makes up to eight roundings per chunk, each about 1.6 times (in variance,
// measured) as heavy as an addition, of which the reduction's order leaves at most about s / 16 + 8 in a chain. That
// costs 2 to 6 % of the call (64 x 14336 x 14336: 79 -> 84 us, 93 in ten splits; 383 x 2688 x 640, five chunks in all,
// 16.6 -> 18.3).
HybridPlan hybrid_plan(int64_t M, int64_t N, int64_t K) {
  HybridPlan p{};
  p.few = hybrid_few(M, N, K);
  if (p.few) {
    p.splits = 1;
    return p;
  }
  const int64_t chunks = K / kHT;
  p.tiles = ((N + kHRows - 1) / kHRows) * ((M + kHT - 1) / kHT);
  int64_t most = p.tiles < 256 ? (512 + p.tiles - 1) / p.tiles : 1;     // no more than two rounds of blocks
  if (most > chunks) most = chunks;
  double best = 0;
  const uint32_t nch = (uint32_t)chunks;               // at most 256
  const uint32_t cps0 = (nch + (uint32_t)most - 1) / (uint32_t)most, s0 = (nch + cps0 - 1) / cps0;
  for (uint32_t s = 1; s <= (uint32_t)most; ++s) {
    const uint32_t cps = (nch + s - 1) / s;
    if (cps * (s - 1) >= nch) continue;                 // fewer splits of as many chunks
    const double full = 4.5 + 2.0 * cps, last = 4.5 + 2.0 * (nch - (s - 1) * cps);
    const int64_t nfull = p.tiles * (s - 1), busy = nfull % 256, idle = 256 - busy;
    // whole rounds, then the busy blocks' end or the last split's, in as many rounds as the idle CUs need
    double t = full * (double)(nfull / 256);
    const double ends = last * (double)((p.tiles + idle - 1) / idle), both = (busy ? full : 0) + last * (double)((p.tiles + 255) / 256);
    t += busy && ends < full ? full : (ends < both ? ends : both);
    if (s > 1) t += 3.0 + (double)s * (double)M * (double)N * (8 / 7e6);
    if (best == 0 || t < best) {
      best = t;
      p.splits = s;
      p.chunks_per_split = cps;
      uint32_t sum = cps;
      while (sum > cps0 && 13 * sum + (cps + sum - 1) / sum - 1 + s / 16 + 8 > 13 * cps0 + s0) --sum;
      p.chunks_per_sum = sum;
    }
  }
  p.ws = p.splits > 1 ? (size_t)p.splits * M * N * sizeof(float) : 0;
  return p;
}

}  // namespace

extern "C" int slim_hybrid_layout(const uint8_t* kinds, int64_t N, int64_t K, uint64_t* tile_info,
                                  size_t* payload_bytes) {
  if (!kinds || !payload_bytes) return SLIM_EINVAL;
  if (N < kHT || K < kHT || N % kHT || K % kHT) return SLIM_ESHAPE;
  const int64_t tiles = (N / kHT) * (K / kHT);
  uint64_t off = 0;
  for (int64_t t = 0; t < tiles; ++t) {
    if (kinds[t] > 1) return SLIM_EINVAL;
    if (tile_info) tile_info[t] = off | (kinds[t] ? kHSparseBit : 0);
    off += kinds[t] ? kHSparse : kHDense;
  }
  *payload_bytes = (size_t)off;
  return SLIM_OK;
}

extern "C" int slim_pack_hybrid(const float* W, int64_t N, int64_t K, const uint8_t* kinds, uint64_t* tile_info,
                                uint8_t* payload, size_t payload_bytes, void* stream) {
  if (!W || !kinds || !tile_info || !payload) return SLIM_EINVAL;
  size_t need = 0;
  int st = slim_hybrid_layout(kinds, N, K, nullptr, &need);
  if (st != SLIM_OK) return st;
  if (payload_bytes < need) return SLIM_EWORKSPACE;
  if (!slim_aligned16(W) || !slim_aligned16(payload) || !slim_aligned16(tile_info)) return SLIM_EALIGN;
  const int64_t tiles = (N / kHT) * (K / kHT);
  uint64_t* h_info = new (std::nothrow) uint64_t[tiles];
  if (!h_info) return SLIM_EDEVICE;
  slim_hybrid_layout(kinds, N, K, h_info, &need);
  hipStream_t s = (hipStream_t)stream;
  int* d_status = nullptr;
  int rc = SLIM_OK, h_status = 0;
  if (hipMalloc(&d_status, sizeof(int)) != hipSuccess) {
    delete[] h_info;
    return SLIM_EDEVICE;
  }
  do {
    if (hipMemcpyAsync(tile_info, h_info, tiles * sizeof(uint64_t), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemsetAsync(d_status, 0, sizeof(int), s) != hipSuccess) {
      rc = SLIM_EDEVICE;
      break;
    }
    const int64_t threads = N * (K / 16);
    {
      SlimKernelTimer timer("hybrid_pack", s);
      SLIM_LAUNCH(timer, k_hybrid_pack, dim3((unsigned)((threads + kHThreads - 1) / kHThreads)), dim3(kHThreads), s, W,
                  N, K, (const uint64_t*)tile_info, payload, d_status);
    }
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(&h_status, d_status, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) {
      rc = SLIM_EDEVICE;
      break;
    }
    if (h_status & 1) rc = SLIM_ENONFINITE;
  } while (0);
  (void)hipFree(d_status);
  delete[] h_info;
  return rc;
}

extern "C" int slim_linear_hybrid_workspace(int64_t M, int64_t N, int64_t K, size_t* bytes) {
  if (!bytes) return SLIM_EINVAL;
  if (M < 1 || N < kHT || K < kHT || N % kHT || K % kHT) return SLIM_ESHAPE;
  *bytes = hybrid_plan(M, N, K).ws;
  return SLIM_OK;
}

extern "C" int slim_linear_hybrid(const void* X, int64_t M, int64_t N, int64_t K, const uint64_t* tile_info,
                                  const uint8_t* payload, size_t payload_bytes, float* Y, void* ws, size_t ws_bytes,
                                  void* stream) {
  if (!X || !tile_info || !payload || !Y) return SLIM_EINVAL;
  if (M < 1 || N < kHT || K < kHT || N % kHT || K % kHT) return SLIM_ESHAPE;
  // 32-bit buffer offsets: the payload and 128 activation rows stay below 4 GiB
  if (payload_bytes >= ((size_t)1 << 32) || (size_t)kHT * K * 2 >= ((size_t)1 << 32) || K / kHT > kHMaxChunks)
    return SLIM_EUNSUPPORTED;
  if (M * K >= ((int64_t)1 << 40) || M * N >= ((int64_t)1 << 40) || (M + kHT) / kHT >= 65536) return SLIM_EUNSUPPORTED;
  if (!slim_aligned16(X) || !slim_aligned16(payload) || !slim_aligned16(Y) || ((uintptr_t)tile_info & 7u))
    return SLIM_EALIGN;
  const HybridPlan p = hybrid_plan(M, N, K);
  if (p.splits > 1 && (!ws || ws_bytes < p.ws)) return SLIM_EWORKSPACE;
  if (p.splits > 1 && !slim_aligned16(ws)) return SLIM_EALIGN;
  hipStream_t s = (hipStream_t)stream;
  if (p.few) {
    const HybridArgs a{static_cast<const uint16_t*>(X), tile_info, payload, Y, M, N, K, (int64_t)payload_bytes, 0, 0};
    SlimKernelTimer timer("hybrid_few", s);
    const int64_t cols = (M + 31) / 32;
    auto go = [&](auto kernel, int rows, int waves) {
      SLIM_LAUNCH(timer, kernel, dim3((unsigned)(N / rows), (unsigned)cols), dim3((unsigned)(64 * waves)), s, a);
    };
    // where there are at most 256 row blocks of 16, a block has a CU to itself and takes more waves; M <= 16: from
    // 12288 rows on, 32-row blocks still give every CU work and read X half as often (16 x 14336 x 14336: 59 us, 69
    // with 16; 16 x 11008 x 4096: 15.6, 13.7 with 16); M > 16: they do wherever there are more than 256 of 16
    // (32 x 4224 x 14336: 25.1 us, 35 with 16 rows and four waves; 32 x 8192 x 14336 32.5 against 39, 32 x 11008 x
    // 4096 19.8 against 20.8; 64 x 4096 x 4096 10.1 against 12.2)
    if (M <= 16) {
      if (N <= 4096) go(k_hybrid_few<1, 1, 16>, 16, 16);
      else if (N >= 12288) go(k_hybrid_few<2, 1, 8>, 32, 8);
      else go(k_hybrid_few<1, 1, 8>, 16, 8);
    } else {
      if (N * cols <= 4096) go(k_hybrid_few<1, 2, 8>, 16, 8);
      else go(k_hybrid_few<2, 2, 8>, 32, 8);
    }
    return hipGetLastError() == hipSuccess ? SLIM_OK : SLIM_EDEVICE;
  }
  HybridArgs a{static_cast<const uint16_t*>(X), tile_info, payload, p.splits > 1 ? static_cast<float*>(ws) : Y,
               M, N, K, (int64_t)payload_bytes, (int)p.chunks_per_split, (int)p.chunks_per_sum};
  {
    SlimKernelTimer timer("hybrid_gemm", s);
    auto kernel = p.chunks_per_split > p.chunks_per_sum ? k_hybrid_gemm<true> : k_hybrid_gemm<false>;
    SLIM_LAUNCH(timer, kernel, dim3((unsigned)((N + kHRows - 1) / kHRows), (unsigned)((M + kHT - 1) / kHT),
                                    (unsigned)p.splits),
                dim3(kHGemmThreads), s, a);
  }
  if (p.splits > 1) {
    const int64_t count4 = M * N / 4;
    SlimKernelTimer timer("hybrid_reduce", s);
    SLIM_LAUNCH(timer, k_hybrid_reduce, dim3((unsigned)((count4 + 63) / 64)), dim3(kHThreads), s,
                (const float*)static_cast<float*>(ws), (int)p.splits, count4, Y);
  }
  return hipGetLastError() == hipSuccess ? SLIM_OK : SLIM_EDEVICE;
}

// mid_gemm.hip - the compressed layer and its input gradient for a middle number of activation rows,
// where 512-row tiles would leave most of the chip idle:
//
//   out[m, row] = sum_red act[m, red] A[row, red] + sum_j tm[m, j] P[row, j],  tm[m, j] = sum_red act[m, red] Q[j, red]
//
// with the operands of sparse_gemm.hip (forward rows = N, red = K, Q = L^T, P = R^T; backward rows = K,
// red = N, Q = R, P = L), the activations already row-scaled to fp16 (k_rowprep) where the plan scales
// them. Measured against the 512-row tiles, which ran on 22 and 40 blocks there: a batch of 64 on 11008 x
// 4096, r 384, 68.7 -> 20.4 us; 333 rows on 5120 x 5120, r 512, 85.0 -> 37.7 us.
//
//  * k_mid: TR x TC tiles of out^T over one slice of the reduction, stored as fp32 partials (or, with
//    neither a split nor an adapter, as the output), and in the same launch the adapter's first
//    product in extra blocks. The two products share only the activations, so the adapter's chain
//    (its product, the sum of its reduction slices, the rounding to fp16) runs beside the sparse one.
//  * k_adapter_tn: the first product alone, for the 512-row tile path.
//  * k_mid_finish: the partials summed in slice order, the adapter's second product added on the
//    matrix cores, the row scaling undone.
#include <type_traits>

#include "slim_device.h"
#include "slim_launch.h"
#include "slim_timing.h"

namespace {

constexpr int kNS = 3;     // stages of the LDS rings

// ============================================================ sparse tiles
// A wave owns 32 rows and all TC columns of the tile (TC / 32 fragments of the 32x32x32 sparse MFMA), a
// block TR / 32 waves. Per 128-wide chunk of the reduction the block's packed words and its
// activation tile [TC x 128] go to LDS by direct loads into a ring of three stages, two chunks ahead;
// activation rows are 256 B with the 16-byte column index XOR-swizzled by the row, as in the
// 512-row tile kernel.
template <bool BWD, int TC, int TR> struct MidShape {
  static constexpr int kWaves = TR / 32;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kGroups = TR / 128;            // 128-row groups
  static constexpr int kFm = TC / 32;                 // column fragments of a wave
  static constexpr int kActRows = TC / kWaves;        // activation rows a wave brings in, four per load
  static constexpr int kActLoads = kActRows / 4;
  static constexpr int kPerChunk = kActLoads + 2;     // direct loads of a wave per chunk: its codes, its share of
                                                      // the index words or scales, activations
  static_assert(kActRows % 4 == 0 && kPerChunk == 6, "whole direct loads of four rows; two loads in each of three steps");
  // LDS: activations [kNS][TC][256 B], then words [kNS][group]: codes [4 fragments][64 lanes][16 B], index
  // words [128 rows][16 B], and in the forward 1 KiB that starts with the scales [128 rows][2 B]; in the
  // backward then the scale rows, a ring of four of 1 KiB each per group (they are read a step at a time,
  // after the chunk's other words)
  static constexpr uint32_t kX = TC * 256, kWGroup = 4096 + 2048 + (BWD ? 0 : 1024), kW = kGroups * kWGroup;
  static constexpr uint32_t kWBase = kNS * kX, kSBase = kNS * (kX + kW), kS = kGroups * 1024;
  static constexpr uint32_t kBytes = kSBase + (BWD ? 4 * kS : 0);
};

template <bool BWD, int TC, int TR>
SLIM_DEV void mid_sparse_tile(const SlimMidArgs& a, uint32_t b, uint8_t* lds) {
  using Sh = MidShape<BWD, TC, TR>;
  constexpr int kFm = Sh::kFm;
  const int tid = threadIdx.x, lane = tid & 63, ha = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, fr = wave & 3;      // the wave's 128-row group and its fragment there
  // XCD-aware order: block b runs on XCD b % 8, which takes a contiguous run of an order that walks
  // slices, then row tiles, then column tiles, so the column tiles that read one piece of the weight
  // share an L2 (32-bit indices: a 64-bit division costs hundreds of instructions)
  const uint32_t RC = (uint32_t)(a.row_tiles * a.col_tiles), C = (uint32_t)a.col_tiles, T = RC * (uint32_t)a.split;
  const uint32_t Q = (T + 7) / 8;
  const uint32_t pos = (b % 8) * Q + b / 8;
  if (pos >= T) return;
  const int s = (int)(pos / RC);
  const uint32_t rem = pos - (uint32_t)s * RC, rt = rem / C, ct = rem - rt * C;
  const int64_t row0 = (int64_t)rt * TR, m0 = (int64_t)ct * TC;
  const int64_t nch = a.red / 128;
  const int64_t cbeg = (int64_t)s * a.chunks;
  const int n = (int)(cbeg + a.chunks < nch ? a.chunks : nch - cbeg);

  // Addresses as in the 512-row tile kernel: buffer resources from the first 16-row block of the
  // wave's 128-row group; rows past the matrix or past M read as zero and are never stored.
  const int64_t grow0 = row0 + 128 * grp;
  const int64_t wblk = (grow0 < a.rows ? grow0 : a.rows - 16) / 16;
  const int64_t nblk = a.rows / 16 - wblk;
  const rsrc_t rc = make_rsrc(a.codes + wblk * nch * 128, nblk * nch * 512);
  const uint32_t d0 = (uint32_t)(grow0 - 16 * wblk), snch = 16u * (uint32_t)nch;
  auto rel_slot = [&](uint32_t d) { return (d >> 4) * snch + (d & 15u); };
  const uint32_t co = rel_slot(d0 + 32u * fr + (uint32_t)l32) * 32u + 16u * ha;         // the wave's codes
  // besides, waves 0 and 1 of a group bring in half of its index words each (64 rows, 16 B a row), waves 2
  // and 3 its scales (the same bytes, so that every wave issues the same loads; forward: 8 rows per lane,
  // backward: the group's scale row of the chunk, s16[n, g]; lanes past 15 read nothing)
  const bool mrole = fr < 2;
  const rsrc_t re = mrole ? make_rsrc(a.meta + wblk * nch * 64, nblk * nch * 256)
                          : (BWD ? make_rsrc(a.scales + (16 * wblk / 128) * a.red, a.red * 2)
                                 : make_rsrc(a.scales + wblk * nch * 16, nblk * nch * 32));
  const uint32_t eo = mrole ? rel_slot(d0 + 64u * fr + (uint32_t)lane) * 16u
                            : (lane > 15 ? 0x80000000u : (BWD ? 16u * (uint32_t)lane : rel_slot(d0 + 8u * (uint32_t)lane) * 2u));
  const int estep = mrole || BWD ? 256 : 32;
  const uint32_t edst = 4096u + (mrole ? 1024u * fr : 2048u), sdst = Sh::kSBase + 1024u * (uint32_t)grp;
  const int lrow = lane >> 4, lslot = lane & 15;
  const int64_t brows = a.M - m0 < TC ? a.M - m0 : TC;
  const rsrc_t rx = make_rsrc(a.act16 + m0 * a.red, brows * a.red * 2);
  uint32_t xo[Sh::kActLoads];
#pragma unroll
  for (int i = 0; i < Sh::kActLoads; ++i) {
    const uint32_t row = (uint32_t)(Sh::kActRows * wave + 4 * i + lrow);
    xo[i] = row * (uint32_t)a.red * 2u + 16u * ((uint32_t)lslot ^ (row & 15u));
  }

  // load i of chunk c's kPerChunk
  auto dma = [&](int c, auto zc, int i) {
    constexpr uint32_t z = decltype(zc)::value;
    const int cc = (int)cbeg + (c < n ? c : n - 1);     // past the end: a dead slot
    uint8_t* W = lds + Sh::kWBase + z * Sh::kW + (uint32_t)grp * Sh::kWGroup;
    uint8_t* X = lds + z * Sh::kX + (uint32_t)(Sh::kActRows * wave) * 256u;
    if (i == 0) __builtin_amdgcn_raw_ptr_buffer_load_lds(rc, (lds_ptr_t)(W + 1024 * fr), 16, co, 512 * cc, 0, 0);
    else if (i == 1)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(re, (lds_ptr_t)(!BWD || mrole ? W + edst : lds + sdst + (uint32_t)(c & 3) * Sh::kS), 16,
                                               eo, estep * cc, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(X + 1024 * (i - 2)), 16, xo[i - 2], 256 * cc, 0, 0);
  };
  auto dma_all = [&](int c, auto zc) {
#pragma unroll
    for (int i = 0; i < Sh::kPerChunk; ++i) dma(c, zc, i);
  };

  // LDS reads are written out with explicit waits that name the registers they complete. (Left to the
  // compiler, every fragment was read right before its MFMA, so that each step waited out the LDS
  // latency, and a read waited for the direct loads in flight.)
  auto rd16 = [](uint32_t addr, auto oc) -> u32x4_t {
    u32x4_t v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(decltype(oc)::value));
    return v;
  };
  auto rd8 = [](uint32_t addr, auto oc) -> u32x2_t {
    u32x2_t v;
    asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(decltype(oc)::value));
    return v;
  };
  auto rd2 = [](uint32_t addr, auto oc) -> uint32_t {
    uint32_t v;
    asm volatile("ds_read_u16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(decltype(oc)::value));
    return v;
  };
  // B fragment fm of step st: row 32 fm + L % 32 at 16-byte slots (2 st + L / 32) ^ (row % 16) and that + 8.
  // Stages past the 16-bit offset of a DS instruction have addresses of their own, 64 KiB on.
  constexpr bool kFar = (kNS - 1) * Sh::kX + (kFm - 1) * 8192 > 65535;
  const uint32_t lb = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
  uint32_t bo[4][2], bf[kFar ? 4 : 1][2];
#pragma unroll
  for (int st = 0; st < 4; ++st)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bo[st][h] = lb + 256u * (uint32_t)l32 + 16u * (uint32_t)((2 * st + ha + 8 * h) ^ (lane & 15));
      if (kFar) bf[st][h] = bo[st][h] + 65536u;
    }
  const uint32_t wo = lb + Sh::kWBase + (uint32_t)grp * Sh::kWGroup;
  const uint32_t cwo = wo + 1024u * (uint32_t)fr + 16u * (uint32_t)lane;
  const uint32_t mwo = wo + 4096u + 16u * (uint32_t)(32 * fr + l32) + 8u * (uint32_t)ha;
  const uint32_t swo = BWD ? lb + Sh::kSBase + 1024u * (uint32_t)grp + 16u * (uint32_t)ha
                           : wo + 6144u + 2u * (uint32_t)(32 * fr + l32);
  struct Frags {
    u32x4_t b[kFm][2];
  };
  struct Scl {       // backward: the scales of a step's positions
    u32x4_t lo, hi;
  };
  auto read_b = [&](auto zc, auto stc, Frags& F) {
    constexpr uint32_t z = decltype(zc)::value;
    constexpr int st = decltype(stc)::value;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      constexpr bool far = z * Sh::kX + (kFm - 1) * 8192 > 65535;
      static_assert(!far || z * Sh::kX >= 65536, "a stage lies on one side of the 64 KiB line");
      const uint32_t adr = far ? bf[kFar ? st : 0][h] : bo[st][h];
      constexpr uint32_t base = far ? z * Sh::kX - 65536 : z * Sh::kX;
      F.b[0][h] = rd16(adr, std::integral_constant<uint32_t, base>{});
      F.b[1][h] = rd16(adr, std::integral_constant<uint32_t, base + 8192>{});
      if constexpr (kFm == 4) {
        F.b[2][h] = rd16(adr, std::integral_constant<uint32_t, base + 16384>{});
        F.b[3][h] = rd16(adr, std::integral_constant<uint32_t, base + 24576>{});
      }
    }
  };
  auto read_s = [&](int c, auto stc, Scl& S) {
    constexpr uint32_t st = decltype(stc)::value;
    const uint32_t adr = swo + (uint32_t)(c & 3) * Sh::kS;
    S.lo = rd16(adr, std::integral_constant<uint32_t, 32 * st>{});
    S.hi = rd16(adr, std::integral_constant<uint32_t, 32 * st + 128>{});
  };
  auto landed = [](Frags& F) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(F.b[0][0]), "+v"(F.b[0][1]), "+v"(F.b[1][0]), "+v"(F.b[1][1]));
    if constexpr (kFm == 4) asm volatile("" : "+v"(F.b[2][0]), "+v"(F.b[2][1]), "+v"(F.b[3][0]), "+v"(F.b[3][1]));
  };
  struct Words {
    u32x4_t cw;
    u32x2_t mw;
    uint32_t sw;
  };
  auto read_words = [&](auto zc, Words& t) {
    constexpr uint32_t z = decltype(zc)::value;
    t.cw = rd16(cwo, std::integral_constant<uint32_t, z * Sh::kW>{});
    t.mw = rd8(mwo, std::integral_constant<uint32_t, z * Sh::kW>{});
    if constexpr (!BWD) t.sw = rd2(swo, std::integral_constant<uint32_t, z * Sh::kW>{});
  };
  const NibbleConsts nk = nibble_consts_reg();
  auto dequant = [&](const Words& t, int st) {
    return BWD ? dequant_word_int(t.cw[st], nk) : dequant_word(t.cw[st], splat_h2(t.sw), nk);
  };

  f16_t acc[kFm];
#pragma unroll
  for (int fm = 0; fm < kFm; ++fm)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[fm][v] = 0.f;
  // A phase is kPS of a chunk's four steps. While it runs, the next phase's fragments are read into the other
  // register set, so a read has a whole phase to land (with reads one step ahead each step took an LDS round
  // trip, about 250 cycles against 64 to 128 of MFMA issue).
  // (as much of a chunk as the registers hold: four steps of two fragments, two of four, one in the backward)
  constexpr int kPS = kFm == 2 ? 4 : (BWD ? 1 : 2), kNP = 4 / kPS;
  Frags F[2][kPS];
  Scl sq[2];
  h8_t aq[2];
  Words tw[2];
  if (BWD) tw[0].sw = tw[1].sw = 0;
  auto mma = [&](Frags& G, const Scl& S, h8_t av, uint32_t idx, auto abid, int fm) {
    h8_t lo = __builtin_bit_cast(h8_t, G.b[fm][0]), hi = __builtin_bit_cast(h8_t, G.b[fm][1]);
    if (BWD) {
      lo = mul_h8(lo, __builtin_bit_cast(h8_t, S.lo));
      hi = mul_h8(hi, __builtin_bit_cast(h8_t, S.hi));
    }
    acc[fm] = smfmac32(av, cat16(lo, hi), acc[fm], (int)idx, decltype(abid)::value);
  };

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  // Chunk c (stage z, word set p, first fragment set f). Its last phase opens with the chunk's one barrier:
  // every wave holds the rest of chunk c in registers, so chunk c + 3's loads may refill its stage, and chunk
  // c + 1 has landed once only chunk c + 2's loads are outstanding. From there the next chunk's words and
  // first fragments are read, and chunk c + 3's loads go out one after an MFMA each (in one burst they fill the
  // address unit's queue, about 16 cycles per load and CU, and every wave stops at it).
  auto chunk = [&](int c, auto zc, auto pc, auto fc) {
    constexpr int z = decltype(zc)::value, p = decltype(pc)::value;
    using zn = std::integral_constant<int, (z + 1) % 3>;
    Words& cur = tw[p];
    Words& nxt = tw[p ^ 1];
    auto step = [&](auto stc) {
      constexpr int st = decltype(stc)::value, ph = st / kPS, i = st % kPS, fs = (decltype(fc)::value + ph) & 1;
      constexpr bool last = ph == kNP - 1;
      using abid = std::integral_constant<int, st & 1>;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (last && i == 0) {
        __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_wait(Sh::kPerChunk));
        asm volatile("s_barrier" ::: "memory");
        read_words(zn{}, nxt);
      }
      if constexpr (BWD) read_s(st < 3 ? c : c + 1, std::integral_constant<int, (st + 1) & 3>{}, sq[(st + 1) & 1]);
      if constexpr (last) read_b(zn{}, std::integral_constant<int, i>{}, F[fs ^ 1][i]);
      else read_b(zc, std::integral_constant<int, st + kPS>{}, F[fs ^ 1][i]);
      __builtin_amdgcn_sched_barrier(0);
      auto load = [&](int j) {      // chunk c + 3's load j
        __builtin_amdgcn_sched_barrier(0);
        dma(c + 3, zc, j);
        __builtin_amdgcn_sched_barrier(0);
      };
      Frags& G = F[fs][i];
      mma(G, sq[st & 1], aq[st & 1], cur.mw[st >> 1], abid{}, 0);
      if constexpr (last && kPS == 4 && st < 3) load(2 * st);
      if constexpr (last && kPS == 2) load(3 * i);
      if constexpr (kPS == 1 && last) {
        load(0);
        load(1);
      }
      if constexpr (st == 3) {
        // the words were read before the phase's fragments, of which the later reads may be outstanding
        if constexpr (BWD) asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(nxt.cw), "+v"(nxt.mw) : "i"(kPS == 1 ? 10 : 12));
        else asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(nxt.cw), "+v"(nxt.mw), "+v"(nxt.sw) : "i"(12));
      }
      aq[(st + 1) & 1] = dequant(st < 3 ? cur : nxt, (st + 1) & 3);
#pragma unroll
      for (int fm = 1; fm < kFm; ++fm) {
        mma(G, sq[st & 1], aq[st & 1], cur.mw[st >> 1], abid{}, fm);
        if constexpr (kPS == 1 && last) {
          if (fm < 3) {
            load(2 * fm);
            load(2 * fm + 1);
          }
        }
        if constexpr (last && kPS == 4 && st < 3) load(2 * st + 1);
        if constexpr (last && kPS == 2) {
          if (fm < 3) load(3 * i + fm);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (i == kPS - 1) {
#pragma unroll
        for (int j = 0; j < kPS; ++j) landed(F[fs ^ 1][j]);
      }
      // the next step's scales were read before this step's fragments
      if constexpr (BWD) asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(sq[(st + 1) & 1].lo), "+v"(sq[(st + 1) & 1].hi) : "i"(2 * kFm));
    };
    step(I0{});
    step(I1{});
    step(I2{});
    step(I3{});
  };
  dma_all(0, I0{});
  dma_all(1, I1{});
  dma_all(2, I2{});
  // chunk 0 has landed once only the later chunks' loads are outstanding
  __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_wait(2 * Sh::kPerChunk));
  asm volatile("s_barrier" ::: "memory");
  read_words(I0{}, tw[0]);
  if constexpr (BWD) read_s(0, I0{}, sq[0]);
  read_b(I0{}, I0{}, F[0][0]);
  if constexpr (kPS > 1) read_b(I0{}, I1{}, F[0][kPS > 1 ? 1 : 0]);
  if constexpr (kPS == 4) {
    read_b(I0{}, I2{}, F[0][kPS - 2]);
    read_b(I0{}, I3{}, F[0][kPS - 1]);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(tw[0].cw), "+v"(tw[0].mw), "+v"(tw[0].sw));
#pragma unroll
  for (int j = 0; j < kPS; ++j) landed(F[0][j]);
  if constexpr (BWD) asm volatile("" : "+v"(sq[0].lo), "+v"(sq[0].hi));
  aq[0] = dequant(tw[0], 0);
  using Q0 = std::integral_constant<int, 0>;
  using Q1 = std::integral_constant<int, kNP & 1>;     // one phase per chunk: the fragment sets alternate
  int c0 = 0;
  for (; c0 + 6 <= n; c0 += 6) {
    chunk(c0, I0{}, I0{}, Q0{});
    chunk(c0 + 1, I1{}, I1{}, Q1{});
    chunk(c0 + 2, I2{}, I0{}, Q0{});
    chunk(c0 + 3, I0{}, I1{}, Q1{});
    chunk(c0 + 4, I1{}, I0{}, Q0{});
    chunk(c0 + 5, I2{}, I1{}, Q1{});
  }
  if (c0 < n) chunk(c0, I0{}, I0{}, Q0{});
  if (c0 + 1 < n) chunk(c0 + 1, I1{}, I1{}, Q1{});
  if (c0 + 2 < n) chunk(c0 + 2, I2{}, I0{}, Q0{});
  if (c0 + 3 < n) chunk(c0 + 3, I0{}, I1{}, Q1{});
  if (c0 + 4 < n) chunk(c0 + 4, I1{}, I0{}, Q0{});
  // the ring's last loads (repeats of the final chunk) must land before the block's LDS is released
  __builtin_amdgcn_s_waitcnt(0);

  const int64_t wrow = row0 + 32 * wave;
  if (wrow >= a.rows) return;
  if (a.part) {
    // fragment-wise partials [slice][row fragment][column fragment][4 q][64 lanes][4]: 1 KB stores
    float* dst = a.part + (((int64_t)s * a.row_frags + wrow / 32) * a.col_frags + m0 / 32) * 1024;
#pragma unroll
    for (int fm = 0; fm < kFm; ++fm) {
      if (m0 + 32 * fm >= a.M) break;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f4_t o = {acc[fm][4 * q], acc[fm][4 * q + 1], acc[fm][4 * q + 2], acc[fm][4 * q + 3]};
        *reinterpret_cast<f4_t*>(dst + fm * 1024 + q * 256 + 4 * lane) = o;
      }
    }
    return;
  }
  // D[i][j] of a 32x32 fragment: lane j + 32 ((i / 4) % 2), element 4 (i / 8) + i % 4
#pragma unroll
  for (int fm = 0; fm < kFm; ++fm) {
    const int64_t m = m0 + 32 * fm + l32;
    if (m >= a.M) continue;
    const float inv = a.rowinv ? a.rowinv[m] : 1.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t rr = wrow + 8 * q + 4 * ha;
      if (rr < a.rows) {
        const f4_t o = {acc[fm][4 * q], acc[fm][4 * q + 1], acc[fm][4 * q + 2], acc[fm][4 * q + 3]};
        *reinterpret_cast<f4_t*>(a.out + m * a.rows + rr) = o * inv;
      }
    }
  }
}

// ============================================================ adapter first product
// tm^T[j, m] for 128 ranks x TC columns over one slice of the reduction, on 32x32x16 MFMA; wave w owns ranks
// 32 (w % 4) .. + 31 and columns 64 (w / 4) .. + 63 (two fragments). Both operands are contiguous along the
// reduction; per 64 positions their rows (128 B in LDS, the 16-byte column index XOR-swizzled by the
// row) go to LDS by direct loads into the block's three stages, two ahead. (Operand loads straight
// into registers, 64 KB in flight per block, took 2.3 us per 512 positions: a lone block's loads are
// paced by latency, and a ring keeps them coming.) The last unit of a tile to finish sums the slices in
// slice order and writes the fp16 tile, so that the sum costs no launch of its own.
constexpr int kMidAdJ = 128;     // ranks of a unit
constexpr int kMidAdK = 64;      // reduction positions per stage
template <int TC> struct MidAdShape {
  static constexpr int kWaves = TC / 16;
  static constexpr int kQLoads = 16 / kWaves, kXLoads = TC / 8 / kWaves;   // direct loads of a wave per stage
  static constexpr uint32_t kXBase = kMidAdJ * kMidAdK * 2;                // the activation rows follow the ranks'
  static constexpr int kBytes = (kMidAdJ + TC) * kMidAdK * 2;
};

template <int TC>
SLIM_DEV void mid_adapter_unit(const SlimMidArgs& a, uint32_t u, uint8_t* lds) {
  using Sh = MidAdShape<TC>;
  constexpr int kPer = Sh::kQLoads + Sh::kXLoads;
  const int lane = threadIdx.x & 63, ha = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wj = wave & 3, wm = wave >> 2;
  auto stage = [&](auto zc) -> uint8_t* { return lds + decltype(zc)::value * Sh::kBytes; };
  const uint32_t SA = (uint32_t)a.ad_split;
  const uint32_t tile = u / SA, sa = u - tile * SA;
  const uint32_t jt = (uint32_t)((a.r + kMidAdJ - 1) / kMidAdJ), mt = tile / jt;
  const int64_t j0 = (int64_t)(tile - mt * jt) * kMidAdJ, m0 = (int64_t)mt * TC;
  const int kbeg = (int)(sa * a.ad_slice), kend = (int)(kbeg + a.ad_slice < a.red ? kbeg + a.ad_slice : a.red);
  const int n = (kend - kbeg) / kMidAdK;
  // rows past r or M lie beyond the resources and read as zero
  const rsrc_t rq = make_rsrc(a.ad_q + j0 * a.red, (a.r - j0 < kMidAdJ ? a.r - j0 : kMidAdJ) * a.red * 2);
  const rsrc_t rx = make_rsrc(a.act16 + m0 * a.red, (a.M - m0 < TC ? a.M - m0 : TC) * a.red * 2);
  // LDS keeps two 128-byte rows per 256-byte line: column slot c (16 B, 0..7) of row r sits at line r / 2,
  // position (8 (r % 2) + c) ^ ((r / 2) % 8), so the 16 consecutive rows that one pass of a fragment read
  // touches fall in 16 distinct positions (one row per 128 bytes with c ^ (r % 8) puts rows r and r + 8 in
  // the same banks). A load covers 8 rows, four lines: lane L writes position L % 16 of line L / 16. Odd
  // loads' lines start at 4 (mod 8), which flips bit 2 of the position, 64 bytes of the source column.
  const uint32_t lq = (uint32_t)((lane & 15) ^ (lane >> 4));
  const uint32_t lo = ((2u * (uint32_t)(lane >> 4) + (lq >> 3)) * (uint32_t)a.red + 8u * (lq & 7)) * 2u;
  const uint32_t rstep = 16u * (uint32_t)a.red;   // 8 rows
  // load i of stage t's kPer
  auto dma = [&](int t, auto zc, int i) {
    const int ko = 2 * (kbeg + (t < n ? t : n - 1) * kMidAdK);     // past the end: a dead slot
    uint8_t* S = stage(zc);
    if (i < Sh::kQLoads) {
      const uint32_t p = (uint32_t)(Sh::kQLoads * wave + i);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rq, (lds_ptr_t)(S + 1024u * p), 16, (lo ^ (64u * (p & 1))) + p * rstep, ko, 0, 0);
    } else {
      const uint32_t p = (uint32_t)(Sh::kXLoads * wave + i - Sh::kQLoads);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(S + Sh::kXBase + 1024u * p), 16, (lo ^ (64u * (p & 1))) + p * rstep, ko, 0, 0);
    }
  };
  auto dma_all = [&](int t, auto zc) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) dma(t, zc, i);
  };
  f16_t acc[2];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[f][v] = 0.f;
  // fragments of step st of a stage: rows L % 32, column slot 2 st + L / 32. The reads are written
  // out with explicit waits (the compiler would make them wait for every direct load in flight).
  struct Frags {
    u32x4_t q, x[2];
  };
  const uint32_t lb = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
  const uint32_t ro = (uint32_t)(l32 >> 1) * 256u, rq8 = 8u * (uint32_t)(l32 & 1), rx7 = (uint32_t)(l32 >> 1) & 7u;
  const uint32_t qo = lb + (uint32_t)wj * 4096u + ro, xo = lb + Sh::kXBase + (uint32_t)wm * 8192u + ro;
  auto read = [&](auto zc, int st, Frags& F) {
    const uint32_t so = 16u * ((rq8 + (uint32_t)(2 * st + ha)) ^ rx7), zo = decltype(zc)::value * (uint32_t)Sh::kBytes;
    const uint32_t aq = qo + so + zo, ax = xo + so + zo;
    asm volatile("ds_read_b128 %0, %1" : "=v"(F.q) : "v"(aq));
    asm volatile("ds_read_b128 %0, %1" : "=v"(F.x[0]) : "v"(ax));
    asm volatile("ds_read_b128 %0, %1 offset:4096" : "=v"(F.x[1]) : "v"(ax));
  };
  auto landed = [](Frags& F) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(F.q), "+v"(F.x[0]), "+v"(F.x[1])); };
  // Stage t in slot z, its fragments in registers (set f): each step reads a step of the next stage into the
  // other set beside its own MFMAs and a share of stage t + 3's direct loads (with reads, loads and MFMAs of a
  // stage one after the other, a stage took their sum, 1400 cycles; with reads one step ahead, four LDS round
  // trips). The barrier opens the stage: stage t + 1 has landed once only stage t + 2's loads are
  // outstanding, and every wave holds stage t in registers, whose slot stage t + 3's loads refill.
  Frags F[2][4];
  auto step = [&](int t, auto zc, auto fc) {
    constexpr int z = decltype(zc)::value, f0 = decltype(fc)::value;
    using zn = std::integral_constant<int, (z + 1) % kNS>;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_wait(kPer));
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      __builtin_amdgcn_sched_barrier(0);
      read(zn{}, st, F[f0 ^ 1][st]);
      __builtin_amdgcn_sched_barrier(0);
      const Frags& G = F[f0][st];
      if (t < n) {
#pragma unroll
        for (int f = 0; f < 2; ++f) acc[f] = mfma32(__builtin_bit_cast(h8_t, G.q), __builtin_bit_cast(h8_t, G.x[f]), acc[f]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = kPer * st / 4; i < kPer * (st + 1) / 4; ++i) dma(t + kNS, zc, i);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int st = 0; st < 4; ++st) landed(F[f0 ^ 1][st]);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  dma_all(0, I0{});
  dma_all(1, I1{});
  dma_all(2, I2{});
  __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_wait(2 * kPer));
  asm volatile("s_barrier" ::: "memory");
#pragma unroll
  for (int st = 0; st < 4; ++st) read(I0{}, st, F[0][st]);
#pragma unroll
  for (int st = 0; st < 4; ++st) landed(F[0][st]);
  // whole groups of six stages; past the last one a stage repeats it and its MFMAs are skipped
  for (int t = 0; t < n; t += 6) {
    step(t, I0{}, I0{});
    step(t + 1, I1{}, I1{});
    step(t + 2, I2{}, I0{});
    step(t + 3, I0{}, I1{});
    step(t + 4, I1{}, I0{});
    step(t + 5, I2{}, I1{});
  }
  // the ring's last loads (repeats of the final stage) must land before the block's LDS is released
  __builtin_amdgcn_s_waitcnt(0);
  f4_t sum[8];
#pragma unroll
  for (int f = 0; f < 8; ++f) sum[f] = f4_t{acc[f >> 2][4 * (f & 3)], acc[f >> 2][4 * (f & 3) + 1], acc[f >> 2][4 * (f & 3) + 2], acc[f >> 2][4 * (f & 3) + 3]};
  if (SA > 1) {
    // the hand-off between blocks: device-scope stores, completion, the counter, device-scope loads
    __shared__ uint32_t last;
    constexpr uint32_t kTileF = kMidAdJ * TC;     // floats of a tile's partial
    const rsrc_t pr = make_rsrc(a.tpart + (int64_t)tile * SA * kTileF, (int64_t)SA * kTileF * 4);
    auto off = [&](uint32_t ss, int f) { return (ss * kTileF + (uint32_t)((8 * wave + f) * 256 + 4 * lane)) * 4u; };
#pragma unroll
    for (int f = 0; f < 8; ++f) st_dev4(pr, off(sa, f), sum[f]);
    drain_stores();
    __syncthreads();
    if (threadIdx.x == 0) last = counter_arrive(&a.tcounters[tile]);
    __syncthreads();
    if (last != SA - 1) return;
#pragma unroll
    for (int f = 0; f < 8; ++f) sum[f] = f4_t{0.f, 0.f, 0.f, 0.f};
    for (uint32_t q0 = 0; q0 < SA; q0 += 4) {
      f4_t pv[4][8];
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j)
#pragma unroll
        for (int f = 0; f < 8; ++f) pv[j][f] = ld_dev4(pr, off(q0 + j < SA ? q0 + j : SA - 1, f));
      __builtin_amdgcn_sched_barrier(0);   // every load out before the first sum
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j)
        if (q0 + j < SA)
#pragma unroll
          for (int f = 0; f < 8; ++f) sum[f] = sum[f] + pv[j][f];
    }
    if (threadIdx.x == 0) counter_reset(&a.tcounters[tile]);
  }
  // D[j][m] of a 32x32 fragment: lane m + 32 ((j / 4) % 2), element 4 (j / 8) + j % 4: four consecutive
  // ranks of a row are 8 bytes of the tiled fp16 output
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int64_t m = m0 + 64 * wm + 32 * f + l32;
    if (m >= a.M) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t jj = j0 + 32 * wj + 8 * q + 4 * ha;
      if (jj >= a.r) continue;
      const f4_t v = sum[4 * f + q];
      const h2_t lo2 = {(_Float16)v[0], (_Float16)v[1]}, hi2 = {(_Float16)v[2], (_Float16)v[3]};
      *reinterpret_cast<u32x2_t*>(a.tm + ((m >> 5) * (a.r >> 4) + (jj >> 4)) * 512 + (m & 31) * 16 + (jj & 15)) =
          u32x2_t{bits_of(lo2), bits_of(hi2)};
    }
  }
}

// The first product alone, for the 512-row tile path.
__global__ void __launch_bounds__(512, 2) k_adapter_tn(SlimMidArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kNS * MidAdShape<128>::kBytes];
  mid_adapter_unit<128>(a, blockIdx.x, lds);
}

// Blocks [0, ad_blocks) run adapter units (dispatched first: their reduction is the longer chain), the
// rest sparse tiles.
template <bool BWD, int TC, int TR>
__global__ void __launch_bounds__((MidShape<BWD, TC, TR>::kThreads), 2) k_mid(SlimMidArgs a) {
  using Sh = MidShape<BWD, TC, TR>;
  static_assert(MidAdShape<TC>::kWaves == Sh::kWaves, "one block shape for both kinds");
  constexpr uint32_t kAd = kNS * MidAdShape<TC>::kBytes;
  __shared__ __attribute__((aligned(16))) uint8_t lds[Sh::kBytes > kAd ? Sh::kBytes : kAd];
  if (blockIdx.x < (uint32_t)a.ad_blocks) {
    if (blockIdx.x < (uint32_t)a.ad_units) mid_adapter_unit<TC>(a, blockIdx.x, lds);
    return;
  }
  mid_sparse_tile<BWD, TC, TR>(a, blockIdx.x - (uint32_t)a.ad_blocks, lds);
}

// ============================================================ finish
// One block per 64 rows x 64 columns; its four waves take a quarter of the rank each, so that the loads
// of the second product are one or two rounds of memory latency (a wave per 32 x 32 walking the whole
// rank took twice as long), and hand their quarters over in LDS. Wave w ends up with fragment
// (row w % 2, column w / 2): its split partials, which sit in the accumulator layout, summed in slice
// order, then the four quarters in wave order. tm and the forward's factor come in 32 x 16 tiles
// (1 KiB per fragment step), the backward's factor row-major.
template <bool TILED>
__global__ void __launch_bounds__(256, 3) k_mid_finish(SlimMidArgs a) {
  __shared__ f4_t hand[12][4][64];
  const int lane = threadIdx.x & 63, ha = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t rfs = (a.rows + 31) / 32, cfs = (a.M + 31) / 32;
  const uint32_t rb = (uint32_t)((rfs + 1) / 2), cb = blockIdx.x / rb;
  const int64_t rf0 = 2 * (int64_t)(blockIdx.x - cb * rb), cf0 = 2 * (int64_t)cb;
  const int64_t rf = rf0 + (wave & 1), cf = cf0 + (wave >> 1);
  const bool live = rf < rfs && cf < cfs;
  // the partials of the wave's fragment (a fragment past the edge reads the block's first)
  const float* src = a.part + ((live ? rf : rf0) * a.col_frags + (live ? cf : cf0)) * 1024 + 4 * lane;
  const int64_t sstep = a.row_frags * a.col_frags * 1024;
  f4_t pv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) pv[q] = *reinterpret_cast<const f4_t*>(src + 256 * q);
  const int nj = (int)(a.r / 16), nq = (nj + 3) / 4;
  f16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  if (nj > 0) {
    const rsrc_t rp = make_rsrc(a.ad_p, TILED ? rfs * 32 * a.r * 2 : a.rows * a.r * 2);
    const rsrc_t rt = make_rsrc(a.tm, cfs * 32 * a.r * 2);
    const uint32_t lo16 = 32u * (uint32_t)l32 + 16u * (uint32_t)ha;
    const uint32_t po = TILED ? (uint32_t)(rf0 * nj) * 1024u + lo16
                              : (uint32_t)(rf0 * 32 + l32) * (uint32_t)(a.r * 2) + 16u * (uint32_t)ha;
    const uint32_t pstep = TILED ? (uint32_t)nj * 1024u : (uint32_t)(a.r * 64);
    const uint32_t to = (uint32_t)(cf0 * nj) * 1024u + lo16, tstep = (uint32_t)nj * 1024u;
    constexpr int kU = 4;
    const int t0 = wave * nq, t1 = t0 + nq < nj ? t0 + nq : nj;
    for (int tb = t0; tb < t1; tb += kU) {
      u32x4_t p[kU][2], t[kU][2];
#pragma unroll
      for (int i = 0; i < kU; ++i) {
        const int tt = tb + i < t1 ? tb + i : t1 - 1;
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          p[i][f] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rp, po + f * pstep, tt * (TILED ? 1024 : 32), 0));
          t[i][f] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rt, to + f * tstep, tt * 1024, 0));
        }
      }
      __builtin_amdgcn_sched_barrier(0);   // every load out before the first MFMA
#pragma unroll
      for (int i = 0; i < kU; ++i)
        if (tb + i < t1)
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
              acc[x][y] = mfma32(__builtin_bit_cast(h8_t, p[i][x]), __builtin_bit_cast(h8_t, t[i][y]), acc[x][y]);
    }
  }
  for (int s = 1; s < a.split; ++s) {
    f4_t nv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) nv[q] = *reinterpret_cast<const f4_t*>(src + s * sstep + 256 * q);
#pragma unroll
    for (int q = 0; q < 4; ++q) pv[q] = pv[q] + nv[q];
  }
  if (nj > 0) {
    // fragment d = row d % 2, column d / 2 goes to wave d; slot 3 d + (source s < d ? s : s - 1)
    auto slot = [&](int d, int sw) { return 3 * d + (sw < d ? sw : sw - 1); };
    f4_t own[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f16_t& v = acc[d & 1][d >> 1];
        const f4_t o = {v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        if (d == wave) own[q] = o;
        else hand[slot(d, wave)][q][lane] = o;
      }
    }
    __syncthreads();
#pragma unroll
    for (int sw = 0; sw < 4; ++sw)
#pragma unroll
      for (int q = 0; q < 4; ++q) pv[q] = pv[q] + (sw == wave ? own[q] : hand[sw == wave ? 0 : slot(wave, sw)][q][lane]);
  }
  const int64_t m = 32 * cf + l32;
  if (!live || m >= a.M) return;
  const float inv = a.rowinv ? a.rowinv[m] : 1.0f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t rr = 32 * rf + 8 * q + 4 * ha;
    if (rr < a.rows) *reinterpret_cast<f4_t*>(a.out + m * a.rows + rr) = pv[q] * inv;
  }
}

template <bool BWD, int TC, int TR>
void launch_mid(const SlimMidArgs& a, const char* name, hipStream_t s) {
  SlimKernelTimer timer(name, s);
  const int64_t T = a.row_tiles * a.col_tiles * a.split;
  const dim3 grid((unsigned)(a.ad_blocks + 8 * ((T + 7) / 8)));
  SLIM_LAUNCH(timer, (k_mid<BWD, TC, TR>), grid, dim3(MidShape<BWD, TC, TR>::kThreads), s, a);
}

}  // namespace

int slim_launch_adapter_tn(const SlimMidArgs& a, hipStream_t s) {
  SlimKernelTimer timer("adapter_gemm", s);
  SLIM_LAUNCH(timer, k_adapter_tn, dim3((unsigned)a.ad_units), dim3(512), s, a);
  return hipGetLastError() == hipSuccess ? SLIM_OK : SLIM_EDEVICE;
}

int slim_launch_mid(const SlimMidArgs& a, bool bwd, hipStream_t s) {
  if (a.tile_cols == 128) {
    if (bwd) launch_mid<true, 128, 256>(a, "mid_bwd", s);
    else launch_mid<false, 128, 256>(a, "mid_fwd", s);
  } else {
    if (bwd) launch_mid<true, 64, 128>(a, "mid_bwd", s);
    else launch_mid<false, 64, 128>(a, "mid_fwd", s);
  }
  if (hipGetLastError() != hipSuccess) return SLIM_EDEVICE;
  if (a.part) {
    SlimKernelTimer timer(bwd ? "mid_finish_bwd" : "mid_finish_fwd", s);
    const int64_t rb = (a.rows + 63) / 64, cb = (a.M + 63) / 64;
    const dim3 grid((unsigned)(rb * cb));
    if (a.p_tiled) SLIM_LAUNCH(timer, k_mid_finish<true>, grid, dim3(256), s, a);
    else SLIM_LAUNCH(timer, k_mid_finish<false>, grid, dim3(256), s, a);
    if (hipGetLastError() != hipSuccess) return SLIM_EDEVICE;
  }
  return SLIM_OK;
}

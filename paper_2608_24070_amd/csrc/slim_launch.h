// slim_launch.h - launchers shared between the libslim translation units.
#pragma once

#include <hip/hip_runtime.h>

#include "slim_host.h"

// tm = A Q^T: A [M, Kd] fp16 activations (the row-scaled copy), Q [r, Kd] fp16 row-major; fp16
// result at ws + p.off_t in 32 x 16 tiles (adapter_gemm.hip).
int slim_launch_adapter_gemm(const uint16_t* A, int64_t M, int64_t Kd, const uint16_t* Q, int64_t r, const SlimPlan& p,
                             char* ws, hipStream_t s);

// One layer call on the middle path (mid_gemm.hip).
struct SlimMidArgs {
  const uint32_t* codes;   // packed operand: [rows, red]
  const uint32_t* meta;
  const uint16_t* scales;
  const uint16_t* act16;   // [M, red] fp16 activations (row-scaled when rowinv is set)
  const float* rowinv;     // 2^-e per activation row, or null
  float* out;              // [M, rows]
  float* part;             // sparse partials, fragment-wise (see k_mid), or null: tiles store to out
  int64_t M, rows, red, r;
  int tile_cols;           // 64 (128 x 64 tiles) or 128 (256 x 128)
  int64_t row_tiles, col_tiles;
  int64_t row_frags, col_frags;   // 32-wide fragments the partials' layout counts
  int split;               // reduction slices of the sparse product
  int64_t chunks;          // 128-wide chunks per slice
  const uint16_t* ad_q;    // adapter first factor, row-major [r, red]
  const uint16_t* ad_p;    // adapter second factor [rows, r]: 32 x 16 tiles or row-major
  int p_tiled;
  uint16_t* tm;            // fp16 adapter intermediate in 32 x 16 tiles
  float* tpart;            // its fp32 slice partials
  uint32_t* tcounters;     // one per 128-rank tile of it
  int ad_split;
  int64_t ad_slice;        // reduction positions per slice
  int64_t ad_units, ad_blocks;
};
int slim_launch_mid(const SlimMidArgs& a, bool bwd, hipStream_t s);
// tm alone (128 x 128 tiles of it, ad_units of them times ad_split).
int slim_launch_adapter_tn(const SlimMidArgs& a, hipStream_t s);

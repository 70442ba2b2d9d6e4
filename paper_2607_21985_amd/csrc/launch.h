// Kernel arguments of the decode launches, shared by the per-column kernels
// (spdp.hip) and the all-columns form (wide.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

// One product of a launch: the matrix's device arrays, the call's input and
// output, and the matrix's split.
struct MatArgs {
  const uint32_t* tile_offset;
  const uint32_t* col_info;
  const uint64_t* bitmap;
  const uint16_t* values;  // fp16 values, or one-byte codes (the kernel's Q form)
  const float* scales;     // Q form: one scale per row
  const uint16_t* x;
  uint16_t* y;
  // [segments][batch][n_stripes * tile_m]: {fp32 bits, phase} pairs
  unsigned long long* partials;
  // the tag of this call's partials, never 0 (the workspace starts zeroed).
  // A handle's own workspace has one phase per stripe (phase_step 1,
  // epoch_done NULL): the tag is phase[r], and the stripe's first reducer
  // advances it. The library's static workspace, shared by every handle, has
  // one device-wide epoch (phase_step 0): the tag is *phase + 1 (0 skipped);
  // each stripe's first reducer counts itself in *epoch_done, and the last
  // stripe's stores the tag as the new epoch and clears the count.
  uint32_t* phase;
  uint32_t* epoch_done;
  int phase_step;
  int rows, cols;
  int tile_m, tk_log2, n_colblocks, n_stripes;
  int code;       // threshold code: active iff code < (x & 0x7fff) <= 0x7c00
  int wave_cols;  // columns per wave (multiple of 16, <= kMaxWaveCols)
  int segments;   // workgroups per row stripe
  int n_wg;       // segments * n_stripes
  uint32_t zero_col;  // column index whose bitmap lies in the zeroed tail padding
  // nonzero: each wave requests its first batch before the workgroup list is
  // built (a property of the product and the batch, never of the launch, so
  // that grouping does not change the summation order)
  int early_first;
  // with the batch's shared column set (the kernel's BMASK form): a column
  // is active iff the fp32 running sum of |x[b, k]| over the tokens exceeds
  // batch_thr = fp32(batch * t), every token's activation kept there
  float batch_thr;
  // consecutive K ranges (of kWaves x wave_cols columns) per workgroup
  int passes;
  // the all-columns form (wide.hip): the word records, the chunks' value
  // offsets, the stripe's chunks and the chunks of one segment
  const unsigned char* rec;
  const uint32_t* chunk_off;
  int chunks;
  int seg_chunks;
};

// A launch runs up to kMaxGroup independent products (same tile height and
// batch): grid row y serves product y, its workgroup x being stripe
// x / segments, segment x % segments (segments ascending within a stripe);
// workgroups past the product's n_wg exit at once.
constexpr int kMaxGroup = 8;
struct LaunchArgs {
  MatArgs m[kMaxGroup];
  int batch;
  int slot;  // all-columns form: LDS bytes of a chunk's values, the most of the launch's products
};


// Launches the all-columns form (wide.hip) for `batch` tokens: the grid's
// workgroups are those of the per-column kernels.
hipError_t launch_wide(const LaunchArgs& args, int count, bool bmask, dim3 grid, hipStream_t stream);

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
  union {
    const float* scales;   // Q form: one scale per row
    // fp16 values: NULL, or the product's gate, a word that a launch of the
    // all-columns form has written before (wide.hip): not 0 where that launch
    // has done the product, which this one then leaves out
    const uint32_t* gate;
  };
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
};

// A launch runs up to kMaxGroup independent products (same tile height and
// batch): grid row y serves product y, its workgroup x being stripe
// x / segments, segment x % segments (segments ascending within a stripe);
// workgroups past the product's n_wg exit at once.
constexpr int kMaxGroup = 8;
struct LaunchArgs {
  MatArgs m[kMaxGroup];
  int batch;
};

// One product of an all-columns launch (wide.hip). Where a field's name is
// one of MatArgs, it means the same; segments and n_wg are this form's own.
struct WideArgs {
  const unsigned char* rec;   // word records, [stripe][chunk]
  const uint32_t* chunk_off;  // the chunks' value offsets
  const uint16_t* values;
  const uint16_t* x;
  uint16_t* y;
  unsigned long long* partials;
  uint32_t* phase;
  uint32_t* epoch_done;
  // NULL: every column takes part whatever the activations. Else the form
  // runs only if at least gate_min columns of a sample of the activations are
  // active for some token; the word tells the per-column launch that follows
  uint32_t* gate;
  int gate_min;
  int phase_step;
  int rows, cols;
  int n_stripes;
  int code;
  int segments;
  int n_wg;
  float batch_thr;
  int chunks;      // chunks of a stripe
  int seg_chunks;  // chunks of a segment
};

struct WideLaunch {
  WideArgs m[kMaxGroup];
  int batch;
  int slot;  // LDS bytes of a chunk's values, the most of the launch's products
};

// Launches the all-columns form for `batch` tokens.
hipError_t launch_wide(const WideLaunch& args, int count, bool bmask, dim3 grid, hipStream_t stream);

// Prefill product on the Tiled-CBC arrays (Sec. 4.3): Y = X W_sp^T for N
// tokens with static pruning only (no activation test), on gfx950's matrix
// cores. The weights stay in the decode format -- the same handle serves
// both phases -- and are expanded tile by tile into a dense operand in LDS
// (the paper's layout-alignment stage), then multiplied with
// v_mfma_f32_32x32x16_f16 (fp16 operands, fp32 accumulation).
//
// Expansion: lane i of bitmap word v of a column takes row 64 v + i; its
// value sits at the word's masked popcount below bit i plus the popcounts of
// the column's earlier words (HAD-SMBD, Sec. 4.2.1), or is 0 where the bit is
// clear.
//
// The forms (choose_spmm picks one):
//   * spmm_rows_kernel, for few tokens (tile_k >= 16, any width): every wave
//     expands 64 rows straight into MFMA operands (expand.h), no tile in LDS;
//   * spmm_ws_kernel and spmm_ws256_kernel, 256 x 16 GTiles and a width that
//     is a multiple of 8: warp-specialized, the GTile expanded once into a
//     dense tile in LDS (row-major, 16 fp16 per row, rows padded to 40 bytes
//     so that the MFMA operand reads of 32 consecutive rows spread over the
//     banks) for 128 or 256 tokens (described at the kernels);
//   * spmm_kernel, the plain form: four waves, a 256-row stripe x 128 tokens,
//     k-steps of 16 columns; each wave expands four columns of the tile and
//     multiplies it with its 32 tokens, operands fetched one step ahead into
//     registers. For handles without word records.
// The first three split K when their grid is small.

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "expand.h"
#include "internal.h"

namespace {

using namespace spdp_dev;

constexpr int kTM = 256;                       // rows of a stripe (four bitmap words per column)
constexpr int kKStep = 16;                     // columns per k-step (the MFMA's k)
constexpr int kWaves = 4;
constexpr int kTokPerWave = 32;
constexpr int kBN = kWaves * kTokPerWave;      // tokens per workgroup
constexpr int kRowBytes = 40;                  // a dense-tile row: 16 fp16 + 8 bytes of padding
constexpr int kTileBytes = kTM * kRowBytes;
constexpr int kBlocks = kTM / 32;              // 32-row MFMA blocks of a stripe

struct SpmmArgs {
  const uint32_t* tile_offset;
  const uint32_t* col_info;
  const uint64_t* bitmap;
  const uint16_t* values;
  const uint16_t* x;  // [n_tokens][cols]
  uint16_t* y;        // [n_tokens][rows]
  long long n_tokens;
  int rows, cols;
  int tk_log2;        // tile_k = 1 << tk_log2 >= 16
  int n_colblocks;
  int steps;          // k-steps over the padded width: n_colblocks * tile_k / 16
  int x_vec;          // cols % 8 == 0: X rows are read 16 bytes at a time
  int y_vec;          // rows % 4 == 0: Y rows are written 8 bytes at a time
};

__device__ __forceinline__ uint32_t mbcnt64(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// The plain form. What one wave fetches for one k-step: its four columns'
// values (one per lane and bitmap word, 0 where the bit is clear) and its B
// operand.
struct StepData {
  uint2 v[4];  // [word]: the four columns' fp16 bits, two per dword
  half8 b;
};

__global__ __launch_bounds__(256) void spmm_kernel(SpmmArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char tile[2][kTileBytes];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = blockIdx.x;  // stripe
  const long long n_wave = (long long)blockIdx.y * kBN + (long long)wave * kTokPerWave;
  const int tk = 1 << a.tk_log2;
  const int khalf = (lane >> 5) * 8;
  // this lane's token for the B operand (tokens past the end re-read the
  // last one; their outputs are not written)
  const long long tok = n_wave + (lane & 31) < a.n_tokens ? n_wave + (lane & 31) : a.n_tokens - 1;
  const uint16_t* const xrow = a.x + tok * (long long)a.cols;
  const const_ptr<uint32_t> ci_s = (const_ptr<uint32_t>)a.col_info;
  const const_ptr<uint32_t> to_s = (const_ptr<uint32_t>)a.tile_offset;
  const const_ptr<uint64_t> bm_s = (const_ptr<uint64_t>)a.bitmap;

  auto fetch = [&](int s, StepData& d) __attribute__((always_inline)) {
    const int k0 = s * kKStep;
    const int c = k0 >> a.tk_log2;
    const int g = r * a.n_colblocks + c;
    const uint32_t col0 = (uint32_t)g * (uint32_t)tk + (uint32_t)(k0 - (c << a.tk_log2)) + 4u * (uint32_t)wave;
    const uint32_t to = to_s[g];
    uint32_t h[4][4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const uint32_t ci = ci_s[col0 + jj];
      uint32_t base = to + (ci >> 16);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const uint64_t word = bm_s[(size_t)(col0 + jj) * 4 + v];
        h[v][jj] = 0;
        if ((word >> lane) & 1) h[v][jj] = a.values[base + mbcnt64(word)];
        base += (uint32_t)__builtin_popcountll(word);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) d.v[v] = make_uint2(h[v][0] | (h[v][1] << 16), h[v][2] | (h[v][3] << 16));
    // B operand: X[tok][k0 + khalf .. + 8], zero past the last column
    const int kb = k0 + khalf;
    if (a.x_vec) {
      if (kb < a.cols) {
        d.b = *reinterpret_cast<const half8*>(xrow + kb);
      } else {
        d.b = half8{0, 0, 0, 0, 0, 0, 0, 0};
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint16_t hx = kb + e < a.cols ? xrow[kb + e] : (uint16_t)0;
        d.b[e] = __builtin_bit_cast(_Float16, hx);
      }
    }
  };

  float16v acc[kBlocks];
#pragma unroll
  for (int i = 0; i < kBlocks; ++i) acc[i] = float16v{};

  StepData cur, nxt;
  fetch(0, cur);
  for (int s = 0; s < a.steps; ++s) {
    unsigned char* t = tile[s & 1];
    // 1. this wave's four columns into rows 64v + lane of the dense tile
#pragma unroll
    for (int v = 0; v < 4; ++v) *reinterpret_cast<uint2*>(t + (64 * v + lane) * kRowBytes + 8 * wave) = cur.v[v];
    __syncthreads();
    if (s + 1 < a.steps) fetch(s + 1, nxt);
    // 2. the stripe's eight 32-row blocks times this wave's 32 tokens
    const half8 b = cur.b;
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) {
      const unsigned char* p = t + (32 * i + (lane & 31)) * kRowBytes + 2 * khalf;
      const uint2 lo = *reinterpret_cast<const uint2*>(p);
      const uint2 hi = *reinterpret_cast<const uint2*>(p + 8);
      const half8 av = __builtin_bit_cast(half8, make_uint4(lo.x, lo.y, hi.x, hi.y));
      acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, b, acc[i], 0, 0, 0);
    }
    cur = nxt;
  }

  // 3. accumulator register e of block i holds row 32 i + 8 (e / 4) +
  // 4 (lane / 32) + e % 4 and token lane % 32: four consecutive rows per
  // group of four registers, rounded once to fp16
  const long long n = n_wave + (lane & 31);
  if (n >= a.n_tokens) return;
  uint16_t* const yrow = a.y + n * (long long)a.rows;
#pragma unroll
  for (int i = 0; i < kBlocks; ++i) {
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
      const int m = r * kTM + 32 * i + 8 * grp + 4 * (lane >> 5);
      uint16_t h[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = __half_as_ushort(__float2half_rn(acc[i][4 * grp + e]));
      if (a.y_vec && m + 3 < a.rows) {
        *reinterpret_cast<uint2*>(yrow + m) = make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (m + e < a.rows) yrow[m + e] = h[e];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Helpers of the pipelined form below.

constexpr int kValBytes = kTM * kKStep * 2;    // a dense GTile's worth of values
constexpr int kXBytes = kBN * kKStep * 2;      // 128 tokens x 16 columns

// Global -> LDS DMA of 4 bytes per lane (lane l's bytes land at lds + 4 l),
// as dma16 of expand.h.
__device__ __forceinline__ void dma4(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_nop 4\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "{m0}"(lds) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// ---------------------------------------------------------------------------
// Warp-specialized form, for 256 x 16 GTiles and a width that is a
// multiple of 8 (every Llama shape): each k-step is one GTile, and what a
// step reads from memory -- the GTile's padded values (one contiguous run)
// and the 128 x 16 block of X -- is copied into a ring of LDS slots by
// global->LDS DMA several steps ahead. Sixteen waves: waves 0-7 multiply, waves
// 8-15 expand. A wave issues in order and waits while the matrix core is
// busy with its previous MFMA, so a wave that did both would serialize
// them; with the roles in different waves every SIMD holds two multiplying
// and two expanding waves, and the expansion of step s + 1 runs while the
// MFMAs of step s do. One barrier per step (one GTile).
//   * multiplying wave m: rows 64 (m & 3) .., tokens 64 (m >> 2) .. of the
//     256 x 128 output tile (four 32 x 32 blocks, A and B each read once);
//     it also issues the step's DMA: one 16-byte load of values (8 x 64
//     lanes x 16 bytes cover a dense GTile) and one of X (m < 4: 32 tokens
//     each) or of bitmap words / ColInfo (m >= 4: these only warm L2 for
//     the expanding waves' scalar loads and land in a scratch area). The
//     TileOffsets come from the LDS table: no scalar memory load, so the
//     LDS waits of these waves never wait for one;
//   * expanding wave d: columns 2d, 2d + 1 of the GTile (eight bitmap
//     words, scalar loads two steps ahead, so the loads of step s + 2 are in
//     flight while step s + 1 is expanded), values from the slot.
// A slot is refilled in the step after its X rows were read: step s
// requests step s + kWsRing - 1 into the slot of step s - 1.
//
// Split-K (blockIdx.z of k_splits): a workgroup walks GTiles [z sps, (z + 1)
// sps) of its stripe and, with more than one split, stores its fp32 sums to
// part[z][token][row]; spmm_reduce_kernel adds the splits in order.

constexpr int kWsWaves = 16;
constexpr int kWsRing = 8;
constexpr int kWsDma = 2;      // loads per step of a multiplying wave
constexpr int kToCap = 1800;   // TileOffsets of one stripe's split held in LDS
constexpr int kGBytes = kValBytes + kXBytes;  // one GTile's values and X block in a ring slot

// wait until at most kWsDma x `later` loads are in flight (later < N + 1)
template <int N>
__device__ __forceinline__ void wait_steps(int later) {
  if constexpr (N > 0) {
    if (later >= N) {
      wait_vmcnt<kWsDma * N>();
      return;
    }
    wait_steps<N - 1>(later);
  } else {
    wait_vmcnt<0>();
  }
}

struct WsArgs {
  SpmmArgs s;
  float* part;  // [k_splits][n_tokens][rows] fp32 when k_splits > 1
  int k_splits;
  int sps;      // GTiles per split
};

// A wave's 64 rows x 32 NJ tokens from row m0 and token n0: the tokens are the
// MFMA's rows, so register e of block (i, j) holds row 32 i + lane % 32 and
// token 32 j + 8 (e / 4) + 4 (lane / 32) + e % 4, and a store writes 32
// consecutive rows of two tokens (with the rows as the MFMA's rows a store
// wrote four rows of 32 tokens each, elements one by one where the row count
// is no multiple of 4: 5003x3080 at 333 / 1000 tokens
// 69 / 101 -> 49 / 71 us; whole multiples of 4 within 2 %).
template <int NJ>
__device__ __forceinline__ void store_block(const WsArgs& wa, const float16v (&acc)[2][NJ], int m0, long long n0, int lane) {
  const SpmmArgs& a = wa.s;
  float* const part = wa.k_splits > 1 ? wa.part + (size_t)blockIdx.z * (size_t)a.n_tokens * (size_t)a.rows : nullptr;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = m0 + 32 * i + (lane & 31);
    if (m >= a.rows) continue;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const long long n = n0 + 32 * j + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (n >= a.n_tokens) continue;
        if (part)
          part[n * (long long)a.rows + m] = acc[i][j][e];
        else
          a.y[n * (long long)a.rows + m] = __half_as_ushort(__float2half_rn(acc[i][j][e]));
      }
  }
}

__global__ __launch_bounds__(kWsWaves * 64) void spmm_ws_kernel(WsArgs wa) {
  const SpmmArgs& a = wa.s;
  __shared__ __attribute__((aligned(1024))) unsigned char ring[kWsRing][kGBytes];
  __shared__ __attribute__((aligned(16))) unsigned char tile[2][kTileBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char warm[1024];
  __shared__ uint32_t toff[kToCap];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool mma = wave < 8;
  const int mw = wave & 7;  // index within the role
  const int r = blockIdx.x;
  const long long nb0 = (long long)blockIdx.y * kBN;
  const int khalf = (lane >> 5) * 8;
  const int c0 = (int)blockIdx.z * wa.sps;                 // first GTile of this split
  const int steps = min(wa.sps, a.n_colblocks - c0);       // >= 1 (the host makes every split non-empty)
  const uint32_t g0 = (uint32_t)r * (uint32_t)a.n_colblocks;
  for (int i = threadIdx.x; i <= steps; i += kWsWaves * 64) toff[i] = a.tile_offset[g0 + (uint32_t)(c0 + i)];

  // multiplying waves: the second DMA of a GTile, as (source, lane offset
  // at GTile 0, bytes per GTile, LDS offset): X into the slot, or bitmap
  // words / ColInfo into the warm-up area
  const bool x_dma = mw < 4;
  const void* d_src;
  uint32_t d_off, d_step, d_lds;
  {
    const long long left = a.n_tokens - nb0;
    const int xt = 32 * mw + (lane >> 1);
    if (x_dma) {
      d_src = a.x + nb0 * (long long)a.cols;
      d_off = (uint32_t)((xt < left ? xt : left - 1) * (long long)a.cols * 2) + 16u * (uint32_t)(lane & 1);
      d_step = 2u * kKStep;
      d_lds = (uint32_t)(kValBytes + 1024 * mw);
    } else if (mw < 6) {
      d_src = a.bitmap;
      d_off = g0 * 512u + 256u * (uint32_t)(mw - 4) + 4u * (uint32_t)lane;
      d_step = 512u;
      d_lds = lds_addr(warm) + 256u * (uint32_t)(mw - 4);
    } else {
      d_src = a.col_info;
      d_off = g0 * 64u + 4u * (uint32_t)(lane & 15);
      d_step = 64u;
      d_lds = lds_addr(warm) + 512u + 256u * (uint32_t)(mw - 6);
    }
  }
  const uint32_t q16 = 16u * (uint32_t)(mw * 64 + lane);
  __syncthreads();

  // requests step s (GTile c0 + s) into its slot
  auto issue = [&](int s) __attribute__((always_inline)) {
    const uint32_t c = (uint32_t)(c0 + s);
    const uint32_t slot = lds_addr(ring[s & (kWsRing - 1)]);
    // the GTile's values: lanes past the end re-read its last 16 bytes
    const uint32_t t0 = toff[s], t1 = toff[s + 1];
    const int span = 2 * (int)(t1 - t0) - 16;
    const uint32_t voff = 2u * t0 + min(q16, (uint32_t)max(span, 0));
    asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(a.values),
                 "{m0}"((uint32_t)__builtin_amdgcn_readfirstlane((int)(slot + 1024u * (uint32_t)mw)))
                 : "memory");
    if (x_dma) {
      // columns past the width (the last GTile of a width that is not a
      // multiple of 16): any valid 16 bytes, the B operand is cleared
      uint32_t off = d_off + c * d_step;
      if (c * kKStep + 8u * (uint32_t)(lane & 1) >= (uint32_t)a.cols) off = d_off - 16u * (uint32_t)(lane & 1);
      dma16(d_src, off, (uint32_t)__builtin_amdgcn_readfirstlane((int)(slot + d_lds)));
    } else {
      dma4(d_src, d_off + c * d_step, d_lds);
    }
  };

  // expanding waves: the two columns' words and ColInfo, by scalar loads
  struct Meta {
    uint64_t w[8];  // column 2d: words 0-3, column 2d + 1: words 4-7
    uint32_t ci[2];
  };
  const const_ptr<uint64_t> bm_s = (const_ptr<uint64_t>)a.bitmap;
  const const_ptr<uint32_t> ci_s = (const_ptr<uint32_t>)a.col_info;
  auto load_meta = [&](int s, Meta& m) __attribute__((always_inline)) {
    const uint32_t col0 = (g0 + (uint32_t)(c0 + s)) * (uint32_t)kKStep + 2u * (uint32_t)mw;
#pragma unroll
    for (int i = 0; i < 8; ++i) m.w[i] = bm_s[(size_t)col0 * 4 + i];
    m.ci[0] = ci_s[col0];
    m.ci[1] = ci_s[col0 + 1];
  };
  // column 2 d + jj, word v -> row 64 v + lane: the value at the word's
  // masked popcount below the lane plus the column's earlier words' counts
  auto decode = [&](int s, const Meta& m) __attribute__((always_inline)) {
    const uint32_t vb = lds_addr(ring[s & (kWsRing - 1)]);
    unsigned char* t = tile[s & 1];
    uint32_t hv[2][4];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      uint32_t sb = vb + 2u * (m.ci[jj] >> 16);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        hv[jj][v] = *(const __attribute__((address_space(3))) uint16_t*)(uintptr_t)(sb + 2u * mbcnt64(m.w[4 * jj + v]));
        if (v < 3) {
          const uint32_t pop = (uint32_t)__builtin_popcountll(m.w[4 * jj + v]);
          asm("s_lshl1_add_u32 %0, %1, %0" : "+s"(sb) : "s"(pop) : "scc");
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
      *reinterpret_cast<uint32_t*>(t + (64 * v + lane) * kRowBytes + 4 * mw) =
          select_word(hv[0][v], m.w[v]) | (select_word(hv[1][v], m.w[4 + v]) << 16);
  };

  const int rq = mw & 3, th = mw >> 2;
  float16v acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = float16v{};
  const half8 none = half8{0, 0, 0, 0, 0, 0, 0, 0};

  // one step. Multiplying waves: MFMAs of step s, request of step
  // s + kWsRing - 1, wait for step s + 2. Expanding waves: scalar loads of
  // step s + 2 into `next`, expansion of step s + 1 from `cur`. Barrier.
  // STEADY: every one of these happens, kWsRing - 3 later steps are in
  // flight, and every column is inside the width.
  auto step = [&](int s, Meta& cur, Meta& next, auto steady) __attribute__((always_inline)) {
    constexpr bool kSteady = decltype(steady)::value;
    if (mma) {
      const unsigned char* slot = ring[s & (kWsRing - 1)];
      const unsigned char* t = tile[s & 1];
      half8 b[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        b[j] = *reinterpret_cast<const half8*>(slot + kValBytes + (64 * th + 32 * j + (lane & 31)) * 32 + 2 * khalf);
        if constexpr (!kSteady)
          if ((c0 + s) * kKStep + khalf >= a.cols) b[j] = none;
      }
      half8 av[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const unsigned char* p = t + (64 * rq + 32 * i + (lane & 31)) * kRowBytes + 2 * khalf;
        const uint2 lo = *reinterpret_cast<const uint2*>(p);
        const uint2 hi = *reinterpret_cast<const uint2*>(p + 8);
        av[i] = __builtin_bit_cast(half8, make_uint4(lo.x, lo.y, hi.x, hi.y));
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b[j], av[i], acc[i][j], 0, 0, 0);
      if (kSteady || s + kWsRing - 1 < steps) issue(s + kWsRing - 1);
      if constexpr (kSteady)
        wait_vmcnt<kWsDma * (kWsRing - 3)>();
      else if (s + 2 < steps)
        wait_steps<kWsRing - 3>(min(kWsRing - 3, steps - 1 - (s + 2)));
    } else {
      if (kSteady || s + 2 < steps) load_meta(s + 2, next);
      if (kSteady || s + 1 < steps) decode(s + 1, cur);
    }
    __syncthreads();
  };

  // prologue: steps 0 .. kWsRing - 2 requested; step 0 expanded; step 1 landed
  Meta ma, mb;
  if (mma) {
    for (int s = 0; s < kWsRing - 1 && s < steps; ++s) issue(s);
    wait_steps<kWsRing - 2>(min(kWsRing - 2, steps - 1));
  } else {
    load_meta(0, ma);
    if (steps > 1) load_meta(1, mb);
  }
  __syncthreads();
  if (mma) {
    if (steps > 1) wait_steps<kWsRing - 3>(min(kWsRing - 3, steps - 2));
  } else {
    decode(0, ma);
  }
  __syncthreads();

  // step s expands s + 1 from the set loaded two steps before: step 0 uses
  // mb (step 1) and loads step 2 into ma, step 1 the other way round
  int s = 0;
  const int steady_end = steps - kWsRing;
  for (; s + 1 < steady_end; s += 2) {
    step(s, mb, ma, std::integral_constant<bool, true>{});
    step(s + 1, ma, mb, std::integral_constant<bool, true>{});
  }
  for (; s < steps; s += 2) {
    step(s, mb, ma, std::integral_constant<bool, false>{});
    if (s + 1 < steps) step(s + 1, ma, mb, std::integral_constant<bool, false>{});
  }

  if (!mma) return;
  store_block<2>(wa, acc, r * kTM + 64 * rq, nb0 + 64 * th, lane);
}

// ---------------------------------------------------------------------------
// 256-token form of the warp-specialized kernel: the expansion of a GTile
// is an instruction stream of fixed length whatever the token count, so a
// workgroup of 256 tokens pays it once for twice the MFMA work. Twelve
// waves (three per SIMD: two multiplying, one expanding):
//   * multiplying wave m (0-7): rows 64 (m & 3) .., tokens 128 (m >> 2) ..
//     of the 256 x 256 output tile (2 x 4 blocks of 32 x 32, 128
//     accumulators); per step one 16-byte DMA of values (8 x 64 lanes x 16
//     bytes: a dense GTile) and one of X (tokens 32 m .. 32 m + 31);
//   * expanding wave d (8-11): columns 4d .. 4d + 3 (sixteen bitmap words,
//     scalar loads two steps ahead); it also warms L2 for its own scalar
//     loads (a DMA of the words it will load, into a scratch area, never
//     waited for).
// The two roles run separate loops with the same number of barriers, so
// neither role's registers are held across the other's code.

constexpr int kW256Waves = 12;
constexpr int kW256Ring = 8;
constexpr int kBN256 = 256;
constexpr int kX256Bytes = kBN256 * kKStep * 2;
constexpr int kG256Bytes = kValBytes + kX256Bytes;

__global__ __launch_bounds__(kW256Waves * 64) void spmm_ws256_kernel(WsArgs wa) {
  const SpmmArgs& a = wa.s;
  __shared__ __attribute__((aligned(1024))) unsigned char ring[kW256Ring][kG256Bytes];
  __shared__ __attribute__((aligned(16))) unsigned char tile[2][kTileBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char warm[1024];
  __shared__ uint32_t toff[kToCap];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = blockIdx.x;
  const long long nb0 = (long long)blockIdx.y * kBN256;
  const int c0 = (int)blockIdx.z * wa.sps;
  const int steps = min(wa.sps, a.n_colblocks - c0);
  const uint32_t g0 = (uint32_t)r * (uint32_t)a.n_colblocks;
  for (int i = threadIdx.x; i <= steps; i += kW256Waves * 64) toff[i] = a.tile_offset[g0 + (uint32_t)(c0 + i)];
  __syncthreads();
  constexpr int R = kW256Ring;
  const int steady_end = steps - R;

  if (wave < 8) {
    // ---- multiplying waves
    const int mw = wave;
    const int khalf = (lane >> 5) * 8;
    const int rq = mw & 3, th = mw >> 2;
    const long long left = a.n_tokens - nb0;
    const int xt = 32 * mw + (lane >> 1);
    const uint16_t* const xsrc = a.x + nb0 * (long long)a.cols;
    const uint32_t x_off = (uint32_t)((xt < left ? xt : left - 1) * (long long)a.cols * 2) + 16u * (uint32_t)(lane & 1);
    const uint32_t q16 = 16u * (uint32_t)(mw * 64 + lane);
    auto issue = [&](int s) __attribute__((always_inline)) {
      const uint32_t c = (uint32_t)(c0 + s);
      const uint32_t slot = lds_addr(ring[s & (R - 1)]);
      const uint32_t t0 = toff[s], t1 = toff[s + 1];
      const int span = 2 * (int)(t1 - t0) - 16;
      const uint32_t voff = 2u * t0 + min(q16, (uint32_t)max(span, 0));
      asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(a.values),
                   "{m0}"((uint32_t)__builtin_amdgcn_readfirstlane((int)(slot + 1024u * (uint32_t)mw)))
                   : "memory");
      uint32_t off = x_off + c * (2u * kKStep);
      if (c * kKStep + 8u * (uint32_t)(lane & 1) >= (uint32_t)a.cols) off = x_off - 16u * (uint32_t)(lane & 1);
      dma16(xsrc, off, (uint32_t)__builtin_amdgcn_readfirstlane((int)(slot + kValBytes + 1024u * (uint32_t)mw)));
    };
    float16v acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = float16v{};
    const half8 none = half8{0, 0, 0, 0, 0, 0, 0, 0};
    auto step = [&](int s, auto steady) __attribute__((always_inline)) {
      constexpr bool kSteady = decltype(steady)::value;
      const unsigned char* slot = ring[s & (R - 1)];
      const unsigned char* t = tile[s & 1];
      half8 av[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const unsigned char* p = t + (64 * rq + 32 * i + (lane & 31)) * kRowBytes + 2 * khalf;
        const uint2 lo = *reinterpret_cast<const uint2*>(p);
        const uint2 hi = *reinterpret_cast<const uint2*>(p + 8);
        av[i] = __builtin_bit_cast(half8, make_uint4(lo.x, lo.y, hi.x, hi.y));
      }
      const bool zero_b = !kSteady && (c0 + s) * kKStep + khalf >= a.cols;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        half8 b = *reinterpret_cast<const half8*>(slot + kValBytes + (128 * th + 32 * j + (lane & 31)) * 32 + 2 * khalf);
        if (zero_b) b = none;
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b, av[i], acc[i][j], 0, 0, 0);
      }
      if (kSteady || s + R - 1 < steps) issue(s + R - 1);
      if constexpr (kSteady)
        wait_vmcnt<kWsDma * (R - 3)>();
      else if (s + 2 < steps)
        wait_steps<R - 3>(min(R - 3, steps - 1 - (s + 2)));
      __syncthreads();
    };
    for (int s = 0; s < R - 1 && s < steps; ++s) issue(s);
    wait_steps<R - 2>(min(R - 2, steps - 1));
    __syncthreads();
    if (steps > 1) wait_steps<R - 3>(min(R - 3, steps - 2));
    __syncthreads();
    int s = 0;
    for (; s < steady_end; ++s) step(s, std::integral_constant<bool, true>{});
    for (; s < steps; ++s) step(s, std::integral_constant<bool, false>{});

    store_block<4>(wa, acc, r * kTM + 64 * rq, nb0 + 128 * th, lane);
  } else {
    // ---- expanding waves
    const int d = wave - 8;
    struct Meta {
      uint64_t w[16];  // column 4d + jj: words 4 jj .. 4 jj + 3
      uint32_t ci[4];
    };
    const const_ptr<uint64_t> bm_s = (const_ptr<uint64_t>)a.bitmap;
    const const_ptr<uint32_t> ci_s = (const_ptr<uint32_t>)a.col_info;
    auto load_meta = [&](int s, Meta& m) __attribute__((always_inline)) {
      const uint32_t col0 = (g0 + (uint32_t)(c0 + s)) * (uint32_t)kKStep + 4u * (uint32_t)d;
#pragma unroll
      for (int i = 0; i < 16; ++i) m.w[i] = bm_s[(size_t)col0 * 4 + i];
#pragma unroll
      for (int i = 0; i < 4; ++i) m.ci[i] = ci_s[col0 + i];
    };
    // the words (128 bytes: two lanes of 64) and ColInfo (16 bytes) of step
    // s into L2, landing in a scratch area nobody reads
    auto warm_up = [&](int s) __attribute__((always_inline)) {
      const uint32_t col0 = (g0 + (uint32_t)(c0 + s)) * (uint32_t)kKStep + 4u * (uint32_t)d;
      dma4(a.bitmap, col0 * 32u + 4u * (uint32_t)(lane & 31), lds_addr(warm) + 256u * (uint32_t)d);
      dma4(a.col_info, col0 * 4u + 4u * (uint32_t)(lane & 3), lds_addr(warm) + 256u * (uint32_t)d);
    };
    auto decode = [&](int s, const Meta& m) __attribute__((always_inline)) {
      const uint32_t vb = lds_addr(ring[s & (R - 1)]);
      unsigned char* t = tile[s & 1];
      uint32_t hv[4][4];  // [column][word]
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        uint32_t sb = vb + 2u * (m.ci[jj] >> 16);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          hv[jj][v] = *(const __attribute__((address_space(3))) uint16_t*)(uintptr_t)(sb + 2u * mbcnt64(m.w[4 * jj + v]));
          if (v < 3) {
            const uint32_t pop = (uint32_t)__builtin_popcountll(m.w[4 * jj + v]);
            asm("s_lshl1_add_u32 %0, %1, %0" : "+s"(sb) : "s"(pop) : "scc");
          }
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        uint32_t sel[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) sel[jj] = select_word(hv[jj][v], m.w[4 * jj + v]);
        *reinterpret_cast<uint2*>(t + (64 * v + lane) * kRowBytes + 8 * d) =
            make_uint2(sel[0] | (sel[1] << 16), sel[2] | (sel[3] << 16));
      }
    };
    auto step = [&](int s, Meta& cur, Meta& next, auto steady) __attribute__((always_inline)) {
      constexpr bool kSteady = decltype(steady)::value;
      if (kSteady || s + 4 < steps) warm_up(s + 4);
      if (kSteady || s + 2 < steps) load_meta(s + 2, next);
      if (kSteady || s + 1 < steps) decode(s + 1, cur);
      __syncthreads();
    };
    Meta ma, mb;
    for (int s = 0; s < 4 && s < steps; ++s) warm_up(s);
    load_meta(0, ma);
    if (steps > 1) load_meta(1, mb);
    __syncthreads();
    decode(0, ma);
    __syncthreads();
    int s = 0;
    for (; s + 1 < steady_end; s += 2) {
      step(s, mb, ma, std::integral_constant<bool, true>{});
      step(s + 1, ma, mb, std::integral_constant<bool, true>{});
    }
    for (; s < steps; s += 2) {
      step(s, mb, ma, std::integral_constant<bool, false>{});
      if (s + 1 < steps) step(s + 1, ma, mb, std::integral_constant<bool, false>{});
    }
  }
}

// ---------------------------------------------------------------------------
// Row form, for few tokens: nothing is expanded into LDS. A workgroup of
// eight waves owns a stripe and 32 TB tokens; wave w expands bitmap word
// w mod 4 (64 rows) of the groups 2 (w / 4), 2 (w / 4) + 1 of every chunk (64
// columns) straight into MFMA operands (expand.h) and multiplies them with
// all the tokens; the chunk's two halves are added once, at the end. One
// barrier per chunk; values and X arrive by DMA one chunk ahead.

template <int TB>
struct RowCfg {
  static constexpr int kTokens = 32 * TB;
  static constexpr int kXBytes = kTokens * kChunkCols * 2;
  static constexpr int kRedBytes = 8 * TB * 16 * 64 * 4;  // half of every wave's accumulators
  static int lds(int slot) { return std::max(2 * (slot + kXBytes) + 1024, kRedBytes); }
};

struct RowArgs {
  const unsigned char* rec;   // word records, [stripe][chunk][group][word]
  const uint32_t* chunk_off;  // byte offset of each chunk's values, [stripe][chunk], one more at the end
  const uint16_t* values;
  const uint16_t* x;  // [n_tokens][cols]
  uint16_t* y;        // [n_tokens][rows]
  float* part;        // [splits][n_tokens][rows] fp32 with more than one split
  long long n_tokens;
  int rows, cols;
  int chunks;         // chunks of a stripe
  int cps;            // chunks per split
  int slot;           // LDS bytes of a chunk's values (a multiple of 1024)
};

// The sums of the chunks [c0, c0 + n) of a stripe, element e of token block j
// to emit(j, e, sum) (rows below a.rows only, unless ALL). XV: X rows are
// 16-byte aligned (else they are read by elements).
template <int TB, bool XV, bool ALL, class Emit>
__device__ __forceinline__ void rows_range(const RowArgs& a, unsigned char* lds, int c0, int n, Emit emit) {
  using C = RowCfg<TB>;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int word = wave & 3, half = wave >> 2;
  const int r = blockIdx.x;
  const long long nb0 = (long long)blockIdx.y * C::kTokens;
  const int last_tok = (int)min(a.n_tokens - nb0, (long long)C::kTokens) - 1;
  const uint32_t chunk0 = (uint32_t)r * (uint32_t)a.chunks + (uint32_t)c0;
  const uint32_t l0 = lds_addr(lds);
  const uint32_t slot = (uint32_t)a.slot;
  const uint32_t x0 = l0 + 2 * slot;
  const const_ptr<uint32_t> co = (const_ptr<uint32_t>)a.chunk_off + chunk0;
  const unsigned char* const rec0 = a.rec + (size_t)chunk0 * kChunkRecBytes;
  const uint16_t* const xb = a.x + nb0 * (long long)a.cols;

  // requests the values [t0, t1) and the X block of chunk s, and the records
  // of chunk s + 1 into L2 (landing where nobody reads). X: 128 bytes per
  // token, its 16-byte piece p at position p ^ (token mod 8); wave w brings
  // the tokens 8 w .. 8 w + 7 (TB = 1: the first four waves)
  const int piece = (lane & 7) ^ (lane >> 3);
  auto issue = [&](int s, uint32_t t0, uint32_t t1) __attribute__((always_inline)) {
    const uint32_t last = t1 > t0 ? t1 - t0 - 16u : 0u;
    const uint32_t vl = l0 + (uint32_t)(s & 1) * slot;
    for (uint32_t q0 = 1024u * (uint32_t)wave; q0 <= last; q0 += 8192u)
      dma16(a.values, t0 + min(q0 + 16u * (uint32_t)lane, last),
            (uint32_t)__builtin_amdgcn_readfirstlane((int)(vl + q0)));
    if (TB == 2 || wave < 4) {
      const uint32_t to = x0 + (uint32_t)((s & 1) * C::kXBytes + 1024 * wave);
      const uint32_t t = (uint32_t)min(8 * wave + (lane >> 3), last_tok);
      const int k = (c0 + s) * kChunkCols + 8 * piece;
      if constexpr (XV) {
        // pieces past the width are cleared (0 x a neighbour's infinity must
        // not reach the sums)
        if (k < a.cols)
          dma16(xb, (t * (uint32_t)a.cols + (uint32_t)k) * 2u, (uint32_t)__builtin_amdgcn_readfirstlane((int)to));
        else
          *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(to + 16u * (uint32_t)lane) = u32x4{0, 0, 0, 0};
      } else {
        uint32_t h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = k + e < a.cols ? xb[(size_t)t * a.cols + k + e] : 0u;
        *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(to + 16u * (uint32_t)lane) =
            u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
      }
    }
    const int wr = wave - 5;
    if (wr >= 0)
      dma16(rec0, (uint32_t)(s + 1) * kChunkRecBytes + min(1024u * (uint32_t)wr + 16u * (uint32_t)lane, (uint32_t)kChunkRecBytes - 16u),
            (uint32_t)__builtin_amdgcn_readfirstlane((int)(x0 + 2 * C::kXBytes)));
  };

  float16v acc[2][TB];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = float16v{};
  const_ptr<unsigned char> prec = (const_ptr<unsigned char>)rec0 + (size_t)((8 * half + word) * kRecBytes);
  WordRec m;
  auto fetch = [&](uint32_t step) __attribute__((always_inline)) {
    asm volatile("" : "+s"(prec));
    load_rec(prec, m);
    prec += step;
  };
  const uint32_t xlane = x0 + 128u * (uint32_t)(lane & 31);
  const uint32_t xpos = 16u * (uint32_t)(((lane >> 5) | (4 * half)) ^ (lane & 7));

  uint32_t t0 = co[0], t1 = co[1];
  issue(0, t0, t1);
  fetch(4 * kRecBytes);
  t0 = t1;
  t1 = co[min(2, n)];
  for (int s = 0; s < n; ++s) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (s + 1 < n) issue(s + 1, t0, t1);
    uint32_t base2 = (l0 + (uint32_t)(s & 1) * slot) >> 1;
    asm volatile("" : "+v"(base2));
    const uint32_t xm = xlane + (uint32_t)((s & 1) * C::kXBytes);
    uint32_t t_next = 0;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      uint32_t v[kGroupCols];
      half8 x[TB];
#pragma unroll
      for (int c = 0; c < kGroupCols; ++c) v[c] = gather_column(m, c, base2);
#pragma unroll
      for (int j = 0; j < TB; ++j)
        x[j] = *(const __attribute__((address_space(3))) half8*)(uintptr_t)(xm + (xpos ^ (32u * g)) + 4096u * (uint32_t)j);
      __builtin_amdgcn_sched_barrier(0);
      Operands o;
#pragma unroll
      for (int j = 0; j < 4; ++j) select_pairs(m, v, j, o);
      __builtin_amdgcn_sched_barrier(0);
      fetch(g == 0 ? 12 * kRecBytes : 4 * kRecBytes);
      if (g == 1) t_next = co[min(s + 3, n)];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[j], o.rows(i), acc[i][j], 0, 0, 0);
    }
    t0 = t1;
    t1 = t_next;
  }

  // the two halves' sums: wave (word, 0) takes rows 0-31 of the word, wave
  // (word, 1) rows 32-63, each the sum half 0 + half 1. Register e holds row
  // lane mod 32 and token 32 j + 8 (e / 4) + 4 (lane / 32) + e mod 4: a store
  // writes 32 consecutive rows of two tokens.
  __syncthreads();
  float* const red = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int j = 0; j < TB; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e)
      red[((wave * TB + j) * 16 + e) * 64 + lane] = half == 0 ? acc[1][j][e] : acc[0][j][e];
  __syncthreads();
  if (!ALL && r * kTM + 64 * word + 32 * half + (lane & 31) >= a.rows) return;
#pragma unroll
  for (int j = 0; j < TB; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float other = red[(((wave ^ 4) * TB + j) * 16 + e) * 64 + lane];
      emit(j, e, half == 0 ? acc[0][j][e] + other : other + acc[1][j][e]);
    }
}

// FOLD: one workgroup walks all the ranges of cps chunks and adds their sums
// in order in its registers; else grid.z workgroups write them to `part` for
// spmm_reduce_kernel. The same sums in the same order, so the same bits, with
// no workspace but on a smaller grid: for calls whose workspace cannot be had
// (4096x4090 at 64 tokens 25.8 us split, 111 folded, 11008x4096 with 32-wide
// tiles 30.6 and 96; the plain form takes 629 and 890).
template <int TB, bool XV, bool FOLD>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu((FOLD ? 4 : 6) - (TB == 1 ? 0 : 2)))) void spmm_rows_kernel(RowArgs a) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long nb0 = (long long)blockIdx.y * RowCfg<TB>::kTokens;
  const int last_tok = (int)min(a.n_tokens - nb0, (long long)RowCfg<TB>::kTokens) - 1;
  const int row = (int)blockIdx.x * kTM + 64 * (wave & 3) + 32 * (wave >> 2) + (lane & 31);
  const bool split = gridDim.z > 1;
  float* const part = a.part + (size_t)blockIdx.z * (size_t)a.n_tokens * (size_t)a.rows;
  auto store = [&](int j, int e, float sum) __attribute__((always_inline)) {
    const int t = 32 * j + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
    if (t > last_tok) return;
    const size_t at = (size_t)(nb0 + t) * (size_t)a.rows + (size_t)row;
    if (split)
      part[at] = sum;
    else
      a.y[at] = __half_as_ushort(__float2half_rn(sum));
  };
  if constexpr (FOLD) {
    float total[TB][16];
    rows_range<TB, XV, true>(a, lds, 0, min(a.cps, a.chunks), [&](int j, int e, float sum) __attribute__((always_inline)) {
      total[j][e] = sum;
    });
    for (int c0 = a.cps; c0 < a.chunks; c0 += a.cps) {
      __syncthreads();  // the range before has been read out of the LDS
      rows_range<TB, XV, true>(a, lds, c0, min(a.cps, a.chunks - c0),
                               [&](int j, int e, float sum) __attribute__((always_inline)) { total[j][e] += sum; });
    }
    if (row < a.rows)
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) store(j, e, total[j][e]);
  } else {
    const int c0 = (int)blockIdx.z * a.cps;
    rows_range<TB, XV, false>(a, lds, c0, min(a.cps, a.chunks - c0), store);  // at least one chunk
  }
}

// Y = fp16(sum over the splits of part[z]), the splits added in order
// (z = 0, 1, ...), so the result does not depend on timing. Four outputs
// per lane when the element count is a multiple of 4.
__global__ __launch_bounds__(256) void spmm_reduce_kernel(const float* __restrict__ part, int k_splits, long long count,
                                                          uint16_t* __restrict__ y) {
  const long long stride = (long long)gridDim.x * 256;
  if ((count & 3) == 0) {
    const long long n4 = count >> 2;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n4; i += stride) {
      float4 s = reinterpret_cast<const float4*>(part)[i];
      for (int z = 1; z < k_splits; ++z) {
        const float4 p = reinterpret_cast<const float4*>(part + (size_t)z * (size_t)count)[i];
        s.x += p.x;
        s.y += p.y;
        s.z += p.z;
        s.w += p.w;
      }
      const uint32_t lo = __half_as_ushort(__float2half_rn(s.x)) | ((uint32_t)__half_as_ushort(__float2half_rn(s.y)) << 16);
      const uint32_t hi = __half_as_ushort(__float2half_rn(s.z)) | ((uint32_t)__half_as_ushort(__float2half_rn(s.w)) << 16);
      reinterpret_cast<uint2*>(y)[i] = make_uint2(lo, hi);
    }
  } else {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < count; i += stride) {
      float s = part[i];
      for (int z = 1; z < k_splits; ++z) s += part[(size_t)z * (size_t)count + i];
      y[i] = __half_as_ushort(__float2half_rn(s));
    }
  }
}

int hip_fail(hipError_t e, const char* what) {
  return spdp::fail(SPDP_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

// How a prefill product is run: the kernel, its token tiles, and the splits
// of `per` GTiles (the row form: chunks) each.
enum { kFormPlain = 1, kFormWs128, kFormWs256, kFormRows32, kFormRows64 };
struct SpmmPlan {
  int form;
  long long tiles;
  int splits, per;
  int keep;  // the splits that the warp-specialized rule would take
};

// us to write and add `splits` partial products (a second launch, 4 bytes
// written and read per value at the rate of a large copy)
float split_us(int splits, long long n_tokens, long long rows) {
  return splits > 1 ? 3.0f + (float)splits * (float)n_tokens * (float)rows * 8.0f / 4.0e6f : 0.0f;
}

// The splits of the row form are bounded by the grid, and so that its
// partials stay within those of 128 tokens at that many splits and within
// 40 MB (a larger bound gave no shape less time, and the first call
// allocates it: 11008x4096 at 512 tokens 62 MB -> 45 MB, the
// warp-specialized form's own).
int row_max_splits(const spdp_matrix* h) { return (int)std::min<long long>(16, std::max<long long>(1, 512 / h->n_stripes)); }
long long row_part_tokens(const spdp_matrix* h) {
  return std::min<long long>(128ll * row_max_splits(h), 10000000ll / h->rows);
}

// The row form's least time over its splits (us; fills the plan): with m
// workgroups per CU a chunk takes 1.2 / 1.6 / 1.9 us at 32 tokens (one, two,
// three resident), 1.33 / 1.75 at 64 (one, two); 2 and 3 us per workgroup.
float row_us(const spdp_matrix* h, long long n_tokens, int cus, int tb, int forced, SpmmPlan* plan) {
  const long long tiles = (n_tokens + 32 * tb - 1) / (32 * tb);
  const int most = forced > 0 ? std::min(forced, h->chunks)
                              : std::max(1, (int)std::min<long long>(row_max_splits(h), row_part_tokens(h) / n_tokens));
  float least = -1.0f;
  for (int k = forced > 0 ? most : 1; k <= std::min(most, h->chunks); ++k) {
    const int per = (h->chunks + k - 1) / k;
    const int splits = (h->chunks + per - 1) / per;
    const long long m = (h->n_stripes * tiles * splits + cus - 1) / cus;
    constexpr float kLast32[3] = {0.0f, 1.2f, 1.6f};
    const float chunk = tb == 1 ? 1.9f * (float)(m / 3) + kLast32[m % 3] : 1.75f * (float)(m / 2) + (m % 2 ? 1.33f : 0.0f);
    const float us = (float)per * chunk + (tb == 1 ? 2.0f : 3.0f) * (float)m + split_us(splits, n_tokens, h->rows);
    if (least < 0.0f || us < least) {
      least = us;
      plan->form = tb == 1 ? kFormRows32 : kFormRows64;
      plan->tiles = tiles;
      plan->splits = splits;
      plan->per = per;
    }
  }
  return least;
}

// The warp-specialized forms: 256-token workgroups above 128 tokens when
// their grid, split, covers at least half the CUs (the expansion of a GTile
// is paid once per workgroup; below that the 128-token form's larger grid
// wins); split K when the (stripe, token tile) grid leaves CUs idle, so that
// a split's TileOffsets fit the LDS table, and with at least 8 GTiles per
// split (40 for the 256-token form). A workgroup of either form holds its
// CU, so the split never asks for more workgroups than there are CUs: a
// second round for a few of them doubles the time. Measured (us; 256-token
// workgroups only when two of them per CU were left unsplit and the split
// rounded up -> this rule): 11008x4096 at 256 / 512 tokens 108 / 148 -> 57 /
// 95, 8192x8192 at 512 149 -> 105, 28672x8192 at 512 334 -> 294, 4096x4096
// at 1024 90 -> 77. Returns the time of the model: 0.5 us per GTile at 128
// tokens, 0.55 at 256, and 2 us (4 at 128 tokens) per round.
float ws_us(const spdp_matrix* h, long long n_tokens, int cus, int form, int forced, SpmmPlan* plan) {
  const int ncb = (int)h->n_colblocks;
  const long long tiles256 = (n_tokens + kBN256 - 1) / kBN256, tiles128 = (n_tokens + kBN - 1) / kBN;
  const long long wgs256 = h->n_stripes * tiles256;
  long long k256 = wgs256 < cus ? std::max<long long>(1, std::min<long long>(8, cus / wgs256)) : 1;
  k256 = std::min<long long>(k256, std::max(1, ncb / 40));
  const bool wide = form == kFormWs256 || (form != kFormWs128 && n_tokens > kBN && 2 * wgs256 * k256 >= cus);
  const long long tiles = wide ? tiles256 : tiles128;
  const long long wgs = h->n_stripes * tiles;
  long long k = wide ? k256 : wgs < cus ? std::max<long long>(1, std::min<long long>(8, cus / wgs)) : 1;
  if (!wide) k = std::min<long long>(k, std::max(1, ncb / 8));
  if (forced > 0) k = forced;
  k = std::max<long long>(k, (ncb + kToCap - 2) / (kToCap - 1));
  k = std::min<long long>(k, ncb);
  const int per = (int)((ncb + k - 1) / k);
  plan->form = wide ? kFormWs256 : kFormWs128;
  plan->tiles = tiles;
  plan->per = per;
  plan->splits = (ncb + per - 1) / per;  // every split non-empty
  const float rounds = (float)((wgs * plan->splits + cus - 1) / cus);
  return rounds * ((float)per * (wide ? 0.55f : 0.5f) + (wide ? 2.0f : 4.0f)) + split_us(plan->splits, n_tokens, h->rows);
}

// The forms that stage X by DMA address a token tile with 32-bit offsets: one
// whose tile of X takes more than 4 GiB is left out (rows32 never does: a
// handle has fewer than 2^26 columns).
bool x_tile_fits(const spdp_matrix* h, long long n_tokens, int tile_tokens) {
  return std::min<long long>(n_tokens, tile_tokens) * h->cols * 2 <= 1ll << 32;
}

// The form with the least modelled time. The row form needs the word
// records, the warp-specialized ones 256 x 16 GTiles and a width that is a
// multiple of 8; the plain one takes what is left. Measured, the
// warp-specialized forms -> the row form, us: 4096x4096 at 16 / 64 / 128
// tokens 25.1 / 25.8 / 29.4 -> 14.7 / 19.4 / 23.8 (at 333 44.7 -> 43.6, at 512
// they tie), 4096x11008 at 64 / 256 53 / 66 -> 29 / 57, 11008x4096 at 32 / 64
// 36.8 / 36.9 -> 25.6 / 31.1 (at 128 41.7 -> 44.5), 28672x8192 at 32 / 64 / 128
// 138 / 134 / 139 -> 67 / 77 / 134 (at 256 173 -> 244). SPDP_SPMM_FORM (a
// testing aid) forces a form: 1 plain, 2 and 3 the warp-specialized ones of
// 128 and 256 tokens, 4 and 5 the row form of 32 and 64; SPDP_SPMM_SPLITS the
// splits. False: more splits than a grid holds.
bool choose_spmm(const spdp_matrix* h, long long n_tokens, int cus, bool x_vec, SpmmPlan* plan) {
  int form = 0, forced = 0;
  if (const char* env = std::getenv("SPDP_SPMM_FORM")) form = std::atoi(env);
  if (const char* env = std::getenv("SPDP_SPMM_SPLITS")) forced = std::max(1, std::atoi(env));
  const bool ws = h->tile_k == kKStep && x_vec && form != kFormPlain;
  const bool rows = h->d_rec != nullptr && form != kFormPlain && (n_tokens + 31) / 32 <= 65535;
  plan->form = kFormPlain;
  plan->tiles = (n_tokens + kBN - 1) / kBN;
  plan->splits = 1;
  plan->per = 0;
  plan->keep = 1;
  float least = -1.0f;
  if (ws) {
    SpmmPlan p = *plan;
    const float us = ws_us(h, n_tokens, cus, form, forced, &p);
    p.keep = p.splits;
    const bool fits = x_tile_fits(h, n_tokens, p.form == kFormWs256 ? kBN256 : kBN);
    if (fits && form != kFormRows32 && form != kFormRows64) {
      least = us;
      *plan = p;
    } else {
      plan->keep = p.splits;
    }
  }
  if (rows && !(ws && (form == kFormWs128 || form == kFormWs256)))
    for (int tb = 1; tb <= 2; ++tb) {
      if ((form == kFormRows32 && tb != 1) || (form == kFormRows64 && tb != 2)) continue;
      if (!x_tile_fits(h, n_tokens, 32 * tb)) continue;
      SpmmPlan p = *plan;
      const float us = row_us(h, n_tokens, cus, tb, forced, &p);
      if (least < 0.0f || us < least) {
        least = us;
        *plan = p;
      }
    }
  return plan->splits <= 65535;
}

// The rows of partials (fp32, one per output row) that any call of up to
// n_tokens tokens takes: splits are not monotone in the token count (2048x8192:
// 16 at 128 tokens, 4 at 511, 8 at 385), so the most over all counts, by
// blocks of 32 tokens. Within one the warp-specialized rule's splits are
// constant and the row form's do not rise (a split's cost rises with the
// tokens); above `last` neither splits, but for the splits that a
// TileOffset table forces on every count, which the last block has.
long long spmm_cover(const spdp_matrix* h, long long n_tokens, int cus) {
  int forced = 0;
  if (const char* env = std::getenv("SPDP_SPMM_SPLITS")) forced = std::max(1, std::atoi(env));
  const long long last = std::max<long long>(row_part_tokens(h), (long long)kBN256 * cus / h->n_stripes);
  const long long end = (n_tokens - 1) / 32 * 32;
  long long most = 0;
  SpmmPlan p;
  for (long long lo = 0; lo <= end; lo = lo < end && lo > last ? end : lo + 32) {
    int splits = 1;
    for (int tb = 1; tb <= 2 && h->d_rec != nullptr; ++tb) {
      row_us(h, lo + 1, cus, tb, forced, &p);
      splits = std::max(splits, p.splits);
    }
    if (h->tile_k == kKStep && h->cols % 8 == 0) {
      ws_us(h, lo + 1, cus, 0, forced, &p);
      splits = std::max(splits, p.splits);
    }
    if (splits > 1) most = std::max(most, splits * std::min(lo + 32, n_tokens));
  }
  return most;
}

// The split-K partial sums of the prefill product: grown on demand, the
// old buffer kept until the handle is freed (a captured graph may still
// name it); no allocation while the stream is being captured. A growth also
// covers every call of fewer tokens; where there is no memory for that, only
// this call (`own` rows of partials per token).
int ensure_spmm_part(spdp_matrix* h, int own, long long n_tokens, int cus, hipStream_t stream) {
  const size_t row_bytes = (size_t)h->rows * sizeof(float);
  const size_t own_bytes = (size_t)own * (size_t)n_tokens * row_bytes;
  const bool fits = own_bytes <= h->spmm_part_bytes;
  if (fits && n_tokens <= h->spmm_covered) return SPDP_OK;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  hipError_t e = hipStreamIsCapturing(stream, &cs);
  if (e != hipSuccess) return hip_fail(e, "hipStreamIsCapturing");
  if (cs != hipStreamCaptureStatusNone) {
    if (fits) return SPDP_OK;
    return spdp::fail(SPDP_ERR_INVALID_ARG,
                      "the prefill split-K workspace is too small for this token count and the stream is "
                      "capturing; call spdp_spmm once with this token count before the capture");
  }
  size_t bytes = std::max(own_bytes, (size_t)spmm_cover(h, n_tokens, cus) * row_bytes);
  if (bytes > h->spmm_part_bytes) {
    void* p = nullptr;
    e = hipMalloc(&p, bytes);
    if (e == hipErrorOutOfMemory && own_bytes < bytes) {
      (void)hipGetLastError();
      bytes = own_bytes;
      e = fits ? hipSuccess : hipMalloc(&p, bytes);
    }
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return e == hipErrorOutOfMemory ? spdp::fail(SPDP_ERR_OOM, "hipMalloc of the prefill workspace failed")
                                      : hip_fail(e, "hipMalloc");
    }
    if (p) {
      if (h->d_spmm_part) h->retired.push_back(h->d_spmm_part);
      h->d_spmm_part = p;
      h->spmm_part_bytes = bytes;
    }
  }
  h->spmm_covered = std::max<long long>(h->spmm_covered, n_tokens);
  return SPDP_OK;
}

template <int TB, bool XV, bool FOLD>
hipError_t launch_rows_form(const RowArgs& a, dim3 grid, hipStream_t st) {
  const int lds = RowCfg<TB>::lds(a.slot);
  const auto kernel = spmm_rows_kernel<TB, XV, FOLD>;
  if (lds > 64 * 1024) {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, grid, dim3(512), lds, st, a);
  return hipGetLastError();
}
template <int TB, bool XV>
hipError_t launch_rows_fold(const RowArgs& a, bool fold, dim3 grid, hipStream_t st) {
  return fold ? launch_rows_form<TB, XV, true>(a, grid, st) : launch_rows_form<TB, XV, false>(a, grid, st);
}
hipError_t launch_rows(const RowArgs& a, int tb, bool xv, bool fold, dim3 grid, hipStream_t st) {
  if (tb == 1) return xv ? launch_rows_fold<1, true>(a, fold, grid, st) : launch_rows_fold<1, false>(a, fold, grid, st);
  return xv ? launch_rows_fold<2, true>(a, fold, grid, st) : launch_rows_fold<2, false>(a, fold, grid, st);
}

}  // namespace

extern "C" int spdp_spmm(spdp_handle_t h, const uint16_t* X, int64_t n_tokens, uint16_t* Y, void* stream) {
  using spdp::fail;
  spdp::clear_error();
  if (!h) return fail(SPDP_ERR_INVALID_ARG, "handle is NULL");
  if (h->device < 0) return fail(SPDP_ERR_INVALID_ARG, "handle has no device copy");
  if (!X || !Y) return fail(SPDP_ERR_INVALID_ARG, "X or Y is NULL");
  if (n_tokens < 1) return fail(SPDP_ERR_INVALID_ARG, "n_tokens must be at least 1");
  if ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Y)) & 15)
    return fail(SPDP_ERR_INVALID_ARG, "X and Y must be 16-byte aligned");
  {
    const uintptr_t x0 = reinterpret_cast<uintptr_t>(X), x1 = x0 + (uintptr_t)n_tokens * h->cols * 2;
    const uintptr_t y0 = reinterpret_cast<uintptr_t>(Y), y1 = y0 + (uintptr_t)n_tokens * h->rows * 2;
    if (x0 < y1 && y0 < x1) return fail(SPDP_ERR_INVALID_ARG, "X and Y overlap");
  }
  if (h->value_bits < 16) return fail(SPDP_ERR_UNSUPPORTED, "the prefill product takes fp16 Values, not codes");
  if (h->tile_m != kTM || h->tile_k < kKStep)
    return fail(SPDP_ERR_UNSUPPORTED, "the prefill product needs tile_m = 256 and tile_k >= 16");
  if ((n_tokens + kBN - 1) / kBN > 65535 || h->n_stripes > 0x7FFFFFFF)
    return fail(SPDP_ERR_UNSUPPORTED, "more than 65535 x 128 tokens");
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev != h->device) return fail(SPDP_ERR_INVALID_ARG, "current device differs from the handle's");
  SpmmArgs a;
  std::memset(&a, 0, sizeof(a));
  a.tile_offset = static_cast<const uint32_t*>(h->d_tile_offset);
  a.col_info = static_cast<const uint32_t*>(h->d_col_info);
  a.bitmap = static_cast<const uint64_t*>(h->d_bitmap);
  a.values = static_cast<const uint16_t*>(h->d_values);
  a.x = X;
  a.y = Y;
  a.n_tokens = n_tokens;
  a.rows = (int)h->rows;
  a.cols = (int)h->cols;
  a.tk_log2 = __builtin_ctz((unsigned)h->tile_k);
  a.n_colblocks = (int)h->n_colblocks;
  a.steps = (int)(h->n_colblocks * h->tile_k / kKStep);
  a.x_vec = h->cols % 8 == 0;
  a.y_vec = h->rows % 4 == 0;
  auto st = static_cast<hipStream_t>(stream);
  const int cus = h->cus;
  SpmmPlan plan;
  if (!choose_spmm(h, n_tokens, cus, a.x_vec != 0, &plan))
    return fail(SPDP_ERR_UNSUPPORTED, "the width needs more than 65535 splits");
  float* part = nullptr;
  bool fold = false;
  if (plan.splits > 1 || plan.keep > 1) {
    const int st_ok = ensure_spmm_part(h, plan.splits > 1 ? plan.splits : plan.keep, n_tokens, cus, st);
    if (st_ok != SPDP_OK && plan.splits > 1) {
      // No workspace (the stream is capturing, or no memory). The row form
      // then folds its ranges in the kernel, where the warp-specialized rule
      // asks for no more than there is: where it takes one split (or does
      // not apply), or its splits fit.
      const bool rows = plan.form == kFormRows32 || plan.form == kFormRows64;
      const bool fits = plan.keep == 1 || (size_t)plan.keep * (size_t)n_tokens * (size_t)h->rows * sizeof(float) <= h->spmm_part_bytes;
      if (!rows || !fits) return st_ok;
      fold = true;
    }
    if (st_ok != SPDP_OK) spdp::clear_error();  // the call goes on without it
    if (plan.splits > 1 && !fold) part = static_cast<float*>(h->d_spmm_part);
  }
  const dim3 grid((unsigned)h->n_stripes, (unsigned)plan.tiles, fold ? 1u : (unsigned)plan.splits);
  if (plan.form == kFormRows32 || plan.form == kFormRows64) {
    RowArgs ra;
    std::memset(&ra, 0, sizeof(ra));
    ra.rec = static_cast<const unsigned char*>(h->d_rec);
    ra.chunk_off = static_cast<const uint32_t*>(h->d_chunk_off);
    ra.values = a.values;
    ra.x = X;
    ra.y = Y;
    ra.part = part;
    ra.n_tokens = n_tokens;
    ra.rows = a.rows;
    ra.cols = a.cols;
    ra.chunks = h->chunks;
    ra.cps = plan.per;
    ra.slot = h->chunk_bytes;
    e = launch_rows(ra, plan.form == kFormRows32 ? 1 : 2, a.x_vec != 0, fold, grid, st);
  } else if (plan.form == kFormPlain) {
    hipLaunchKernelGGL(spmm_kernel, grid, dim3(kWaves * 64), 0, st, a);
    e = hipGetLastError();
  } else {
    WsArgs wa;
    wa.s = a;
    wa.k_splits = plan.splits;
    wa.sps = plan.per;
    wa.part = part;
    if (plan.form == kFormWs256)
      hipLaunchKernelGGL(spmm_ws256_kernel, grid, dim3(kW256Waves * 64), 0, st, wa);
    else
      hipLaunchKernelGGL(spmm_ws_kernel, grid, dim3(kWsWaves * 64), 0, st, wa);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return hip_fail(e, "kernel launch");
  if (part) {
    const long long count = n_tokens * h->rows;
    const long long per = (count & 3) == 0 ? count / 4 : count;
    const unsigned blocks = (unsigned)std::min<long long>(8192, (per + 255) / 256);
    hipLaunchKernelGGL(spmm_reduce_kernel, dim3(blocks), dim3(256), 0, st, part, plan.splits, count, Y);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "kernel launch");
  return SPDP_OK;
}

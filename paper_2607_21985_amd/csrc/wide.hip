// Decode in which every column takes part (the all-columns form): for batches
// whose tokens' active columns, taken together, are most columns, and for
// products where leaving columns out gains less than finding out which
// (choose_route in spdp.hip). A column that no token has active is then
// multiplied by zeros instead of being skipped, and the values stream as
// contiguous runs, with no list of columns, into the expansion of expand.h
// and 32x32x16 MFMAs.
//
// A gated launch finds out for itself: each workgroup first counts, over four
// chunks of the activations, the columns that some token has active, and
// leaves if they are too few; a word tells the per-column launch behind it.
//
// The grid is the per-column kernels' in shape (workgroup x is stripe
// x / segments, segment x mod segments, of product blockIdx.y; the segments
// are this form's own, wide_seg_chunks), and so is the split-K exchange. Eight
// waves: wave w expands bitmap word w mod 4 (64 rows) of the groups 2 (w / 4),
// 2 (w / 4) + 1 of every chunk (64 columns) and multiplies them with all
// tokens; the two halves of the chunk are added once, at the end.
//
// A chunk's values arrive by global->LDS DMA one chunk ahead (two slots; three
// slots leave room for two workgroups per CU instead of three at 50 % weight
// sparsity and were 2-12 % slower), its activations four chunks ahead as they
// are; one chunk ahead they are masked in LDS (inactive entries, and columns
// past the width, to 0).
//
// What bounds it: the waves' waiting, and after it vector issue. A chunk costs
// a wave 200 VALU instructions (32 column words: 3 for the address, 1.5 for
// the select and pack, 0.25 for the operand swap each; the rest requests and
// masks the next chunk). Counters over the 13B layer at 8 tokens and the 70B
// layer at 32 (70 % weight sparsity, gates included): 6.2 and 6.6 VALU
// instructions per word, 25 and 26 cycles of the 63 and 65 (of 2.4 GHz) that a
// word takes a SIMD; the waves issue in 23 and 30 % of their cycles and wait in
// 53 and 50 % (in the loop: for a record's scalar loads and the gather's LDS
// reads, which share a counter, and at the chunk's barrier). So what helps is waves: three
// workgroups per CU (six waves per SIMD, hence 80 registers). At 32 tokens
// the partials add 36 MB written and as many read to 166 MB of input.
// 28672x8192 at 70 % weight sparsity and 8 / 32 tokens takes 66 / 85 us, 30 us
// of it VALU issue, 42 its bytes at the rate of a large copy; the per-column
// kernels (four words x the tokens' accumulators per wave, two to five waves
// per SIMD) 72 / 154.

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <new>
#include <string>
#include <vector>

#include "expand.h"
#include "internal.h"
#include "launch.h"

namespace {

using namespace spdp_dev;

constexpr int kWideWaves = 8;
constexpr int kWideThreads = 64 * kWideWaves;
constexpr int kXAhead = 4;   // raw activation slots
constexpr int kPieceBytes = 1024 * kWideWaves;  // values one load of every wave brings

template <int NT>
struct WideCfg {
  static constexpr int kXBytes = NT * kChunkCols * 2;
  static constexpr int kRegs = NT / 2;  // accumulator registers that hold tokens below NT
  static constexpr int kRaw = 0;        // offsets behind the value ring
  static constexpr int kMasked = kXAhead * kXBytes;
  static constexpr int kWarm = kMasked + 2 * kXBytes;
  static constexpr int kAct = kWarm + 1024;
  static constexpr int kEnd = kAct + 8 * kXAhead;
  static constexpr int kRed = std::max(kWideWaves * kRegs * 256, kWideWaves * 4 * 64 * 4);
  static int lds(int slot) { return std::max(2 * slot + kEnd, kRed); }
};

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <class T>
using lds_ptr = __attribute__((address_space(3))) T*;
template <class T>
__device__ __forceinline__ lds_ptr<T> at(uint32_t a) {
  return (lds_ptr<T>)(uintptr_t)a;
}

// waits until at most N loads are in flight, then the workgroup's barrier
template <int N>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// NT: tokens rounded up to 8, 16 or 32 (the MFMA multiplies 32; rows past NT
// repeat others and are dropped). NP: loads of values per wave and
// chunk; 0 for launches with a width that is no multiple of 8 (rows of X that
// are not 16-byte aligned are read by elements, and every wait is for all
// loads).
template <int NT, bool BMASK, int NP>
__global__ __launch_bounds__(kWideThreads) __attribute__((amdgpu_waves_per_eu(6))) void wide_kernel(WideLaunch) {
  using C = WideCfg<NT>;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int word = wave & 3;
  const int half = wave >> 2;

  const const_ptr<WideLaunch> L = (const_ptr<WideLaunch>)__builtin_amdgcn_kernarg_segment_ptr();
  const const_ptr<WideArgs> A = &L->m[blockIdx.y];
  const uint32_t local = blockIdx.x;
  const uint32_t n_seg0 = (uint32_t)A->segments;
  if (local >= (uint32_t)A->n_wg) return;  // the whole workgroup: no barrier has been reached
  const int r = (int)(local / n_seg0);
  const int seg = (int)(local - (uint32_t)r * n_seg0);
  const int c0 = seg * A->seg_chunks;
  const int n = min(A->seg_chunks, A->chunks - c0);  // >= 1
  const int cols = A->cols;
  const int batch = L->batch;
  const uint32_t chunk0 = (uint32_t)r * (uint32_t)A->chunks + (uint32_t)c0;
  // the stripe's tag: written by the previous call (the kernel boundary makes
  // the write visible), read by every workgroup before it publishes
  uint32_t phase = *((const_ptr<uint32_t>)A->phase + r * A->phase_step);
  if (A->phase_step == 0) phase = phase + 1u == 0u ? 1u : phase + 1u;

  const uint32_t l0 = lds_addr(lds);
  const uint32_t slot = (uint32_t)L->slot;
  const uint32_t x0 = l0 + 2 * slot;

  // Loads. Every chunk, a wave requests NP kilobytes of values (one chunk
  // ahead) and one more kilobyte: wave w < NT / 8 eight tokens' activations
  // (four chunks ahead), the others records, into L2 (they land where nobody
  // reads).
  const unsigned char* const values = (const unsigned char*)A->values;
  const const_ptr<uint32_t> co = (const_ptr<uint32_t>)A->chunk_off + chunk0;
  const bool x_wave = NP > 0 && wave < NT / 8;
  const unsigned char* const extra =
      x_wave ? (const unsigned char*)(A->x + (size_t)c0 * kChunkCols) : A->rec + (size_t)chunk0 * kChunkRecBytes;
  // position p of token t: piece p ^ (t mod 8)
  const int piece = (lane & 7) ^ (lane >> 3);
  const uint32_t row_off = (uint32_t)min(8 * wave + (lane >> 3), batch - 1) * (uint32_t)cols * 2u + 16u * (uint32_t)piece;
  uint32_t extra_off =
      x_wave ? row_off
             : (uint32_t)min(1024 * min(max(wave - (NP > 0 ? NT / 8 : 0), 0), 2) + 16 * lane, kChunkRecBytes - 16);
  const int pieces = NP > 0 ? NP : (int)((slot + kPieceBytes - 1) / kPieceBytes);
  // values [t0, t1) of a chunk into the slot at `to`
  auto issue_values = [&](uint32_t t0, uint32_t t1, uint32_t to) __attribute__((always_inline)) {
    const uint32_t last = t1 > t0 ? t1 - t0 - 16u : 0u;
#pragma unroll
    for (int i = 0; i < (NP > 0 ? NP : 4); ++i) {
      if (NP == 0 && i >= pieces) break;
      // where a slot ends before this wave's kilobyte, the load repeats the
      // slot's last one
      const uint32_t q = min((uint32_t)(i * kPieceBytes + 1024 * wave), slot - 1024u);
      dma16(values, t0 + min(q + 16u * (uint32_t)lane, last), (uint32_t)__builtin_amdgcn_readfirstlane((int)(to + q)));
    }
  };
  // the wave's other load for chunk s
  auto issue_extra = [&](int s) __attribute__((always_inline)) {
    uint32_t to = x0 + C::kWarm, off = extra_off;
    if (x_wave) {
      to = x0 + (uint32_t)((s & (kXAhead - 1)) * C::kXBytes + 1024 * wave);
      off -= 16u * (uint32_t)pieces_back(c0 + s, piece, cols);
    }
    dma16(extra, off, (uint32_t)__builtin_amdgcn_readfirstlane((int)to));
    extra_off += x_wave ? 2u * kChunkCols : (uint32_t)kChunkRecBytes;
  };
  // unaligned rows: the activations of chunk c by elements, to raw slot s
  auto copy_x = [&](int s, int c) __attribute__((always_inline)) {
    if (threadIdx.x >= NT * 8) return;
    const int t = min((int)(threadIdx.x >> 3), batch - 1);
    const int k = c * kChunkCols + 8 * piece;
    const uint16_t* const x = A->x + (size_t)t * cols;
    uint32_t h[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = x[min(k + e, cols - 1)];
    *at<u32x4>(x0 + (uint32_t)((s & (kXAhead - 1)) * C::kXBytes) + 16u * threadIdx.x) =
        u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
  };
  // BMASK: the active columns of chunk s, one wave: lane = column, the fp32
  // running sum of |x| over the tokens in ascending order (NaN makes it NaN,
  // never active)
  const float batch_thr = BMASK ? A->batch_thr : 0.0f;
  auto score = [&](int s) __attribute__((always_inline)) {
    const uint32_t raw = x0 + (uint32_t)((s & (kXAhead - 1)) * C::kXBytes) + 2u * (uint32_t)(lane & 7);
    float sum = 0.0f;
#pragma unroll 1
    for (int t0 = 0; t0 < batch; t0 += 4)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = t0 + i;
        if (t >= batch) break;
        const uint16_t h = *at<uint16_t>(raw + 128u * t + 16u * (uint32_t)((lane >> 3) ^ (t & 7)));
        sum += __half2float(__ushort_as_half((unsigned short)(h & 0x7FFFu)));
      }
    const uint64_t act = __builtin_amdgcn_ballot_w64(sum > batch_thr);
    if (lane == 0) *at<uint64_t>(x0 + C::kAct + 8u * (uint32_t)(s & (kXAhead - 1))) = act;
  };
  // masks the activations of chunk s: thread i takes columns 4 (i mod 16) ..
  // + 3 of token i / 16
  // active: magnitude bits in (code, 0x7C00], one unsigned compare per half
  // for code in [-1, 0x7C00]
  const uint32_t lo2 = (uint32_t)(A->code + 1) * 0x10001u;
  auto mask = [&](int s) __attribute__((always_inline)) {
    const uint32_t i = threadIdx.x;
    if (i >= NT * 16) return;
    const int mq = i & 15;
    const uint32_t mpos = x0 + 128u * (i >> 4) + 16u * (((i & 15) >> 1) ^ ((i >> 4) & 7)) + 8u * (i & 1);
    u32x2 v = *at<u32x2>(mpos + (uint32_t)((s & (kXAhead - 1)) * C::kXBytes));
    if constexpr (BMASK) {
      const uint64_t act = *at<uint64_t>(x0 + C::kAct + 8u * (uint32_t)(s & (kXAhead - 1)));
      const uint32_t b = (uint32_t)(act >> (4 * mq));
#pragma unroll
      for (int j = 0; j < 2; ++j)
        v[j] &= ((b >> (2 * j)) & 1u) * 0xFFFFu | ((b >> (2 * j + 1)) & 1u) * 0xFFFF0000u;
    } else {
      const uint32_t span2 = 0x7C017C01u - lo2;  // no borrow: code + 1 <= 0x7C01
      const u16x2 one = {1, 1}, zero = {0, 0};
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const u16x2 over = __builtin_bit_cast(u16x2, v[j] & 0x7FFF7FFFu) - __builtin_bit_cast(u16x2, lo2);
        const u16x2 on =
            __builtin_elementwise_min(__builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, span2), over), one);
        v[j] &= __builtin_bit_cast(uint32_t, (u16x2)(zero - on));
      }
    }
    if ((c0 + s + 1) * kChunkCols > cols) {
      const int left = cols - (c0 + s) * kChunkCols - 4 * mq;
      v[0] &= left >= 2 ? 0xFFFFFFFFu : left == 1 ? 0xFFFFu : 0u;
      v[1] &= left >= 4 ? 0xFFFFFFFFu : left == 3 ? 0xFFFFu : 0u;
    }
    *at<u32x2>(mpos + (uint32_t)(C::kMasked + (s & 1) * C::kXBytes)) = v;
  };

  float16v acc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) acc[i] = float16v{};
  // the wave's records, two of every chunk (those requested past the stripe's
  // end are not used; the array has the slack)
  const_ptr<unsigned char> prec =
      (const_ptr<unsigned char>)A->rec + ((size_t)chunk0 * kChunkRecBytes + (size_t)((8 * half + word) * kRecBytes));
  WordRec m;
  auto fetch = [&](uint32_t step) __attribute__((always_inline)) {
    asm volatile("" : "+s"(prec));
    load_rec(prec, m);
    prec += step;
  };

  if constexpr (!BMASK) {
    // A gated product: every workgroup counts the columns of the sample that
    // are active for some token (wave w: chunk w mod 4, half the tokens) and
    // leaves if they are too few; all of the product's see the same sample.
    uint32_t* const gate = A->gate;
    if (gate) {
#pragma unroll
      for (int j = 0; j < kSampleChunks; ++j) {
        const int c = sample_chunk(j, A->chunks);
        if (NP == 0)
          copy_x(j, c);
        else if (x_wave)
          dma16(A->x, row_off + (uint32_t)(c * kChunkCols * 2) - 16u * (uint32_t)pieces_back(c, piece, cols),
                (uint32_t)__builtin_amdgcn_readfirstlane((int)(x0 + (uint32_t)(j * C::kXBytes + 1024 * wave))));
      }
      wait_barrier<0>();
      const int c = sample_chunk(word, A->chunks);
      const uint32_t raw = x0 + (uint32_t)(word * C::kXBytes) + 2u * (uint32_t)(lane & 7);
      const uint32_t lo = (uint32_t)(A->code + 1);
      bool on = false;
#pragma unroll
      for (int i = 0; i < NT / 2; ++i) {  // rows past the batch repeat its last token
        const int t = half * (NT / 2) + i;
        const uint32_t h = *at<uint16_t>(raw + 128u * t + 16u * (uint32_t)((lane >> 3) ^ (t & 7))) & 0x7FFFu;
        on = on || (h >= lo && h <= 0x7C00u);
      }
      const uint64_t act = __builtin_amdgcn_ballot_w64(on && c * kChunkCols + lane < cols);
      if (lane == 0) *at<uint64_t>(x0 + C::kMasked + 8u * (uint32_t)wave) = act;
      wait_barrier<0>();
      int active = 0;
#pragma unroll
      for (int j = 0; j < kSampleChunks; ++j)
        active += __builtin_popcountll(*at<uint64_t>(x0 + C::kMasked + 8u * j) |
                                       *at<uint64_t>(x0 + C::kMasked + 8u * (j + 4)));
      const bool all = __builtin_amdgcn_readfirstlane(active) >= A->gate_min;
      if (local == 0 && threadIdx.x == 0) *gate = all ? 1u : 0u;
      if (!all) return;
    }
  }

  // prologue: a chunk of values, four of activations
  uint32_t t0 = co[0], t1 = co[1];
  issue_values(t0, t1, l0);
  t0 = t1;  // the next chunk's values are [t0, t1)
  t1 = co[min(2, n)];
#pragma unroll
  for (int s = 0; s < kXAhead; ++s)
    if (s < n) {
      if (NP == 0) copy_x(s, c0 + s);
      issue_extra(s);
    }
  fetch(4 * kRecBytes);
  wait_barrier<0>();
  if constexpr (BMASK) {
    if (wave == 0) score(0);
    if (wave == 1 && n > 1) score(1);
    wait_barrier<0>();
  }
  mask(0);

  const uint32_t xlane = x0 + C::kMasked + (uint32_t)(lane & 31 & (NT - 1)) * 128u;
  // groups 2 half, 2 half + 1: pieces 4 half + (0, 1), 4 half + 2 + (0, 1)
  const uint32_t xpos = 16u * (uint32_t)(((lane >> 5) | (4 * half)) ^ (lane & 7));

  for (int s = 0; s < n; ++s) {
    // chunk s's values, and every load before them, have landed when only the
    // last one of the step before is in flight (its wave's other load, if
    // chunk s - 1 + kXAhead exists)
    if (NP > 0 && s > 0 && s - 1 + kXAhead < n)
      wait_barrier<1>();
    else
      wait_barrier<0>();
    // the next chunk replaces the one whose readers the barrier has seen out
    if (s + 1 < n) issue_values(t0, t1, l0 + (uint32_t)((s + 1) & 1) * slot);
    if (s + kXAhead < n) {
      if (NP == 0) copy_x(s + kXAhead, c0 + s + kXAhead);
      issue_extra(s + kXAhead);
    }

    uint32_t base2 = (l0 + (uint32_t)(s & 1) * slot) >> 1;
    asm volatile("" : "+v"(base2));
    const uint32_t xm = xlane + (uint32_t)((s & 1) * C::kXBytes);
    // one group after the other, one record at a time (registers: vector for
    // six waves per SIMD, scalar for no spills): with six waves the others
    // cover a record's latency
    uint32_t v[kGroupCols];
    Operands o;
    half8 x;
    auto gather = [&](uint32_t pos) __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < kGroupCols; ++c) v[c] = gather_column(m, c, base2);
      x = *at<half8>(xm + pos);
      __builtin_amdgcn_sched_barrier(0);
    };
    gather(xpos);
#pragma unroll
    for (int j = 0; j < 4; ++j) select_pairs(m, v, j, o);
    __builtin_amdgcn_sched_barrier(0);
    fetch(12 * kRecBytes);
    __builtin_amdgcn_sched_barrier(0);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x, o.rows(0), acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x, o.rows(1), acc[1], 0, 0, 0);
    gather(xpos ^ 32u);
#pragma unroll
    for (int j = 0; j < 4; ++j) select_pairs(m, v, j, o);
    __builtin_amdgcn_sched_barrier(0);
    fetch(4 * kRecBytes);
    const uint32_t t_next = co[min(s + 3, n)];
    __builtin_amdgcn_sched_barrier(0);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x, o.rows(0), acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x, o.rows(1), acc[1], 0, 0, 0);

    if constexpr (BMASK)
      if (wave == (s & 7) && s + 2 < n) score(s + 2);
    if (s + 1 < n) mask(s + 1);

    t0 = t1;
    t1 = t_next;
  }

  // The two halves' sums: wave (word, 0) takes rows 0-31 of the word, wave
  // (word, 1) rows 32-63, each the sum half 0 + half 1. Register e holds row
  // lane mod 32 and token 8 (e / 4) + 4 (lane / 32) + e mod 4.
  wait_barrier<0>();
  float* const red = reinterpret_cast<float*>(lds);
  {
    float* const mine = red + (size_t)wave * C::kRegs * 64;
#pragma unroll
    for (int e = 0; e < C::kRegs; ++e) mine[e * 64 + lane] = half == 0 ? acc[1][e] : acc[0][e];
  }
  __syncthreads();
  float sum[C::kRegs];
  {
    const float* const other = red + (size_t)(wave ^ 4) * C::kRegs * 64;
#pragma unroll
    for (int e = 0; e < C::kRegs; ++e)
      sum[e] = half == 0 ? acc[0][e] + other[e * 64 + lane] : other[e * 64 + lane] + acc[1][e];
  }

  const_ptr<WideLaunch> kl = (const_ptr<WideLaunch>)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(kl));
  const const_ptr<WideArgs> ka = &kl->m[blockIdx.y];
  const int nb = kl->batch;
  const int n_seg = ka->segments;
  const int rows = ka->rows;
  const int mpad = ka->n_stripes * 256;
  const int row = r * 256 + 64 * word + 32 * half + (lane & 31);
  const int tok0 = 4 * (lane >> 5);
  if (n_seg == 1) {  // nothing to gather
    if (row < rows)
#pragma unroll
      for (int e = 0; e < C::kRegs; ++e) {
        const int t = 8 * (e >> 2) + tok0 + (e & 3);
        if (t < nb) ka->y[(size_t)t * rows + row] = __half_as_ushort(__float2half_rn(0.0f + sum[e]));
      }
    return;
  }
  {
    unsigned long long* const dst = ka->partials + (size_t)seg * nb * mpad + row;
    const unsigned long long tag = (unsigned long long)phase << 32;
#pragma unroll
    for (int e = 0; e < C::kRegs; ++e) {
      const int t = 8 * (e >> 2) + tok0 + (e & 3);
      if (t < nb)
        __hip_atomic_store(dst + (size_t)t * mpad, tag | __float_as_uint(sum[e]), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
  }

  // The gather of the per-column kernels, with eight waves: the stripe's last
  // n_red segments take the units (64-row block, four tokens), wave g the
  // segments g, g + 8, ..., each requested again until it carries this call's
  // tag; the waves' sums are added in order. Lower segments were dispatched
  // before, so the wait ends; a bound on the rounds still makes every wave
  // exit (the rows then read NaN).
  constexpr int kTok = 4;
  constexpr int kJ = 2;  // segments in flight per wave
  constexpr int kMaxRounds = 1 << 22;
  const int n_units = 4 * ((nb + kTok - 1) / kTok);
  const int n_red = min(n_seg, n_units);
  const int jr = seg - (n_seg - n_red);
  if (jr < 0) return;
  for (int u = jr; u < n_units; u += n_red) {
    const int m = r * 256 + 64 * (u & 3) + lane;
    const int b0 = (u >> 2) * kTok;
    const bool live = m < rows;
    const unsigned long long* const src = ka->partials + (live ? m : 0);
    float sums[kTok];
#pragma unroll
    for (int b = 0; b < kTok; ++b) sums[b] = 0.0f;
    if (live) {
      bool lost = false;
      auto part = [&](int sg, int b) {
        return __hip_atomic_load(src + ((size_t)sg * nb + b0 + b) * mpad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      for (int sg0 = wave; sg0 < n_seg; sg0 += kWideWaves * kJ) {
        unsigned long long v[kJ][kTok];
#pragma unroll
        for (int jj = 0; jj < kJ; ++jj)
#pragma unroll
          for (int b = 0; b < kTok; ++b)
            if (b0 + b < nb) v[jj][b] = part(min(sg0 + kWideWaves * jj, n_seg - 1), b);
        for (int round = 0;; ++round) {
          bool ready = true;
#pragma unroll
          for (int jj = 0; jj < kJ; ++jj)
#pragma unroll
            for (int b = 0; b < kTok; ++b)
              if (b0 + b < nb && sg0 + kWideWaves * jj < n_seg && (uint32_t)(v[jj][b] >> 32) != phase) {
                ready = false;
                v[jj][b] = part(sg0 + kWideWaves * jj, b);
              }
          if (ready) break;
          if (round >= kMaxRounds) {
            lost = true;
            break;
          }
        }
#pragma unroll
        for (int jj = 0; jj < kJ; ++jj)
#pragma unroll
          for (int b = 0; b < kTok; ++b)
            if (b0 + b < nb && sg0 + kWideWaves * jj < n_seg) sums[b] += __uint_as_float((uint32_t)v[jj][b]);
      }
      if (lost)
#pragma unroll
        for (int b = 0; b < kTok; ++b) sums[b] = __builtin_nanf("");
    }
    __syncthreads();  // the exchange above, or the unit before, has been read
#pragma unroll
    for (int b = 0; b < kTok; ++b) red[(wave * kTok + b) * 64 + lane] = sums[b];
    __syncthreads();
    // wave w < 4 adds token w of the unit
    if (live && wave < kTok && b0 + wave < nb) {
      float t = red[wave * 64 + lane];
#pragma unroll
      for (int g = 1; g < kWideWaves; ++g) t += red[(g * kTok + wave) * 64 + lane];
      ka->y[(size_t)(b0 + wave) * rows + m] = __half_as_ushort(__float2half_rn(t));
    }
  }
  // Reducer 0 has gathered row 0 of the stripe, which always exists, from
  // every segment, so every workgroup of the stripe has read the tag: the
  // next call's tag (or the device-wide epoch, see MatArgs).
  if (jr == 0 && threadIdx.x == 0) {
    uint32_t* const done = ka->epoch_done;
    if (done == nullptr) {
      ka->phase[r] = phase + 1u == 0u ? 1u : phase + 1u;
    } else if (__hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
               (uint32_t)ka->n_stripes - 1u) {
      __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(ka->phase, phase, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// The word records of a matrix with 256-row tiles and tile_k >= 16: thread
// (record, column) writes the column's word and offset. Columns past the
// padded width (the last chunk's missing groups) get empty words; padding
// columns past the last chunk have no record.
__global__ __launch_bounds__(256) void build_records_kernel(const uint32_t* tile_offset, const uint32_t* col_info,
                                                            const uint64_t* bitmap, const uint32_t* chunk_off,
                                                            int n_stripes, int n_colblocks, int tk_log2, int chunks,
                                                            unsigned char* rec) {
  using namespace spdp_dev;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;  // [stripe][column]
  const long long width = (long long)chunks * kChunkCols;
  if (i >= (long long)n_stripes * width) return;
  const int r = (int)(i / width);
  const int k = (int)(i - (long long)r * width);
  const int c = k >> tk_log2;
  const bool in = c < n_colblocks;
  const size_t g = (size_t)r * n_colblocks + (in ? c : n_colblocks - 1);
  const size_t col = (g << tk_log2) + (k & ((1 << tk_log2) - 1));
  const uint32_t first = chunk_off[(size_t)r * chunks + k / kChunkCols];
  uint32_t off = in ? 2u * (tile_offset[g] + (col_info[col] >> 16)) - first : 0u;
  const size_t rec0 = ((size_t)r * chunks * kChunkGroups + k / kGroupCols) * 4;
  const int j = k % kGroupCols;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint64_t word = in ? bitmap[col * 4 + w] : 0ull;
    unsigned char* const p = rec + (rec0 + w) * kRecBytes;
    reinterpret_cast<uint64_t*>(p)[j] = word;
    reinterpret_cast<uint16_t*>(p + 8 * kGroupCols)[j] = (uint16_t)off;
    off += 2u * (uint32_t)__builtin_popcountll(word);
  }
}

// *flag |= 1 if one of n fp16 values (n a multiple of 8, 16-byte aligned) is
// infinite or NaN.
__global__ __launch_bounds__(256) void flag_nonfinite_kernel(const uint4* v, long long n8, uint32_t* flag) {
  bool bad = false;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n8; i += (long long)gridDim.x * 256) {
    const uint4 q = v[i];
    for (uint32_t w : {q.x, q.y, q.z, q.w})
      bad = bad || (w & 0x7C00u) == 0x7C00u || (w & 0x7C000000u) == 0x7C000000u;
  }
  if (bad) atomicOr(flag, 1u);
}

template <int NT, bool BMASK, int NP>
hipError_t launch(const WideLaunch& args, dim3 grid, hipStream_t stream) {
  const int lds = WideCfg<NT>::lds(args.slot);
  const auto kernel = wide_kernel<NT, BMASK, NP>;
  if (lds > 64 * 1024) {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, grid, dim3(kWideThreads), lds, stream, args);
  return hipGetLastError();
}

template <int NT, bool BMASK>
hipError_t launch_loads(const WideLaunch& args, bool aligned, dim3 grid, hipStream_t stream) {
  if (!aligned) return launch<NT, BMASK, 0>(args, grid, stream);
  switch ((args.slot + kPieceBytes - 1) / kPieceBytes) {
    case 1: return launch<NT, BMASK, 1>(args, grid, stream);
    case 2: return launch<NT, BMASK, 2>(args, grid, stream);
    case 3: return launch<NT, BMASK, 3>(args, grid, stream);
    default: return launch<NT, BMASK, 4>(args, grid, stream);  // up to a dense chunk: 32 KB
  }
}

}  // namespace

hipError_t launch_wide(const WideLaunch& args, int count, bool bmask, dim3 grid, hipStream_t stream) {
  bool aligned = true;
  for (int i = 0; i < count; ++i) aligned = aligned && args.m[i].cols % 8 == 0;
  if (args.batch <= 8)
    return bmask ? launch_loads<8, true>(args, aligned, grid, stream) : launch_loads<8, false>(args, aligned, grid, stream);
  if (args.batch <= 16)
    return bmask ? launch_loads<16, true>(args, aligned, grid, stream)
                 : launch_loads<16, false>(args, aligned, grid, stream);
  return bmask ? launch_loads<32, true>(args, aligned, grid, stream)
               : launch_loads<32, false>(args, aligned, grid, stream);
}

namespace {

int hip_fail(hipError_t e, const char* what) {
  return spdp::fail(SPDP_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

}  // namespace

namespace spdp {

namespace {

int lay_out_records(spdp_matrix* m) {
  using namespace spdp_dev;
  const int64_t per_tile = m->tile_k / kGroupCols;
  const int64_t chunks = chunk_count(m->cols);
  std::vector<uint32_t> off((size_t)(m->n_stripes * chunks + 1));
  uint32_t widest = 0;
  for (int64_t r = 0; r < m->n_stripes; ++r)
    for (int64_t c = 0; c < chunks; ++c) {
      const int64_t q = c * kChunkGroups;
      const size_t g = (size_t)(r * m->n_colblocks + q / per_tile);
      const uint32_t v = m->tile_offset[g] + (m->col_info[g * m->tile_k + (q % per_tile) * kGroupCols] >> 16);
      off[(size_t)(r * chunks + c)] = 2u * v;
    }
  off.back() = 2u * m->tile_offset.back();
  for (size_t i = 0; i + 1 < off.size(); ++i) widest = std::max(widest, off[i + 1] - off[i]);
  // and slack for the records that the loops request past the end
  const size_t bytes = (size_t)(m->n_stripes * chunks + 3) * kChunkRecBytes;
  // the offsets, then the flag of the values' check, which later is the gate
  const size_t off_bytes = off.size() * sizeof(uint32_t);
  hipError_t e = hipMalloc(&m->d_chunk_off, off_bytes + 256);
  if (e == hipSuccess) e = hipMalloc(&m->d_rec, bytes);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    if (m->d_chunk_off) (void)hipFree(m->d_chunk_off);
    m->d_chunk_off = m->d_rec = nullptr;
    return SPDP_OK;
  }
  if (e != hipSuccess) return hip_fail(e, "hipMalloc");
  off.push_back(0u);
  e = hipMemcpy(m->d_chunk_off, off.data(), off.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpy");
  uint32_t* const flag = static_cast<uint32_t*>(m->d_chunk_off) + (off.size() - 1);
  const int64_t cols = m->n_stripes * chunks * kChunkCols;
  hipLaunchKernelGGL(build_records_kernel, dim3((unsigned)((cols + 255) / 256)), dim3(256), 0, nullptr,
                     static_cast<const uint32_t*>(m->d_tile_offset), static_cast<const uint32_t*>(m->d_col_info),
                     static_cast<const uint64_t*>(m->d_bitmap), static_cast<const uint32_t*>(m->d_chunk_off),
                     (int)m->n_stripes, (int)m->n_colblocks, __builtin_ctz((unsigned)m->tile_k), (int)chunks,
                     static_cast<unsigned char*>(m->d_rec));
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "kernel launch");
  const long long n8 = (long long)m->tile_offset.back() / 8;  // columns are padded to 8 values
  if (n8 > 0) {
    hipLaunchKernelGGL(flag_nonfinite_kernel, dim3((unsigned)std::min<long long>(2048, (n8 + 255) / 256)), dim3(256), 0,
                       nullptr, static_cast<const uint4*>(m->d_values), n8, flag);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "kernel launch");
  }
  uint32_t bad = 0;
  e = hipMemcpy(&bad, flag, sizeof(bad), hipMemcpyDeviceToHost);  // waits for both kernels
  if (e != hipSuccess) return hip_fail(e, "hipMemcpy");
  m->finite = bad == 0;
  m->d_gate = flag;
  m->chunks = (int)chunks;
  m->chunk_bytes = std::max(1024, (int)((widest + 1023) / 1024 * 1024));
  return SPDP_OK;
}

}  // namespace

int build_records(spdp_matrix* m) {
  if (m->tile_m != 256 || m->tile_k < spdp_dev::kGroupCols || m->value_bits != 16) return SPDP_OK;
  try {
    return lay_out_records(m);
  } catch (const std::bad_alloc&) {  // no host memory for the offsets: no records
    if (m->d_chunk_off) (void)hipFree(m->d_chunk_off);
    if (m->d_rec) (void)hipFree(m->d_rec);
    m->d_chunk_off = m->d_rec = nullptr;
    return SPDP_OK;
  }
}

}  // namespace spdp

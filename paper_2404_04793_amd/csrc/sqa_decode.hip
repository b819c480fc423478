// Decode step over per-layer compact KV caches: Algorithm 1 steps 14-21 with the
// append of Eq. 2-3.  One launch covers every (layer, sequence, KV head) unit of
// the call.  A unit's tokens are cut into chunks of `chunk` slots; a workgroup
// of 4 waves owns one chunk:
//   0. read len / ring head / the eviction decision carried over from the
//      previous step (H2O: which heavy slot, if any, the ring leaver replaces);
//   1. stream the chunk's K and V rows once with non-temporal 16-byte loads (8-byte ones for V in section 1X, bf16)
//      (1 KiB per wave load), online softmax in fp32;
//   2. combine the 4 waves.  Unit with one chunk: write out[g][D].  Split unit:
//      write the partial (acc, m, l) and the logits to scratch, bump the unit's
//      arrival counter; the workgroup that arrives last merges the partials in
//      chunk order (fixed order: results do not depend on who arrives last);
//   3. H2O: score_acc += softmax probabilities (summed over the g query heads),
//      one read and one write of the score per token, and in the same pass the
//      NEXT step's eviction decision (arg-min over the updated heavy scores
//      against the next ring leaver), stored in evict_hint;
//   4. only now touch the cache: move the surviving ring token into the evicted
//      heavy slot, write the new token's rows, pos, lens, ring_head.
// During 1 the two slots that 4 will rewrite are read through a remap (new
// token from k_new/v_new, moved token from its old ring slot), so the cache is
// read-only until every workgroup of the unit has finished reading.  HBM
// traffic per unit is the kept rows of K and V once plus 8 bytes of score per
// token under H2O (split units add 8 bytes of logit scratch per token and
// head).  The only atomic is the arrival counter; it decides who merges, never
// what is computed: results are bit-identical from run to run.
// Short units (at most kWpuMaxSlots slots, when the call has enough of them)
// are not shared by the 4 waves: each wave of the workgroup owns a unit of its
// own and runs steps 0-4 alone, without a barrier.  A 4-wave pass over 64 rows
// leaves most lanes idle on such a unit and ends in a merge that costs as much
// as the streaming; one wave walks it 16 rows at a time with nothing to merge.
// Calls of at most one work item per CU have workgroups of 8 waves instead of 4
// (decode_wide_kernel, the same body): there is nothing else on the CU to hide a
// workgroup's round trips, so it asks for more rows at a time, all waves take part
// in step 3 with the scores and positions requested at the start, the decision costs
// one barrier, and the rows of step 4 are written by one wave meanwhile.
#include "sqa_common.h"
#include <algorithm>
#include <cstring>
#include <type_traits>

namespace sqa {

constexpr int kDecThreads = 256;
constexpr int kDecWaves = kDecThreads / SQA_WAVE;
constexpr int kUnroll = 4;                  // rows per lane group in flight per loop trip

struct DecodeArgs {
  const void* q;
  const void* k_new;
  const void* v_new;
  void* out;
  const sqa_layer_cache* layers;   // DEVICE table
  int32_t* status;
  int32_t* cnt;                    // scratch: arrival counter per unit (zero between launches)
  float* part;                     // scratch: per-chunk partial (acc[D], m, l) of split units
  float* logit;                    // scratch: logits of split units (H2O)
  const int32_t* new_pos_seq;      // DEVICE [B] or NULL: per-sequence position, < 0 = sequence sits this step out
  const int32_t* budget_seq;       // DEVICE [n_layers][B] or NULL: per-sequence budgets
  int B, Hq, Hkv, n_layers;
  int new_pos, policy, n_sink;
  int ae;                          // 1 = attend over all len+1 tokens first, evict afterwards
  float scale_log2;                // log2(e) / sqrt(D)
  uint8_t order[SQA_MAX_LAYERS];       // layers in descending budget (long units start first)
  uint32_t blk_end[SQA_MAX_LAYERS];    // work items up to and including ordered layer i
  int lds_chunk;                       // row length of the LDS logit buffer
  // Per-layer launch plan.  All fields are 32-bit on purpose: with a 16-bit
  // table next to a 32-bit one, hipcc 7.2 folded the two uniform indices into
  // one scalar load whose base address was only 2-byte aligned, and scalar
  // loads drop the low address bits of the base (the wrong entry was read).
  struct Layer {
    uint32_t nsplit;      // chunks per unit, with the tile count and the flag described below the struct
    uint32_t chunk;       // slots per chunk
    uint32_t unit_off;    // first unit number of the layer within the call
    uint32_t part_off;    // first partial record
    uint32_t logit_off;   // first logit (floats)
  } lay[SQA_MAX_LAYERS];
  int lds_chunk_w;                     // row length of a wave's LDS logit buffer in one-wave-per-unit layers
  int wide_tail;                       // an unsplit unit's tail keeps all four waves if it has more tokens than this (0: never)
  int lds_probs_w;                     // bytes of a wave's own LDS region for those probabilities in one-wave-per-unit layers
  int tbl_off;                         // blocked allocation: where in the dynamic LDS the unit's block numbers are staged (bytes)
};
// Layer::nsplit: bits 0-15 the number of work items per unit, bits 16-29 how many of a unit's leading 32-token
// tiles keep their H2O probabilities in LDS (matrix-core variant), bit 31 one wave per unit
constexpr uint32_t kWpuBit = 0x80000000u;
constexpr int kLdsTilesShift = 16;
constexpr uint32_t kLdsTilesMask = 0x3fffu;

// Data that one workgroup hands to another inside a launch (partial results,
// logits) moves through agent-scope relaxed atomics: such stores are written
// through and such loads read the coherent copy, so the hand-over needs no
// cache write-back or invalidate (each XCD of the chip has an L2 of its own;
// a device-scope fence would flush it, which costs far more than the data).
__device__ __forceinline__ void st_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_agent(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_agent(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// element i of an array whose base is the same in all lanes: a global access (the pointers come from a table in
// memory, where the compiler can only take them for generic ones) with a 32-bit offset, one register instead of two
typedef __attribute__((address_space(1))) char g_char_t;
typedef __attribute__((address_space(1))) float g_float_t;
typedef __attribute__((address_space(1))) int32_t g_int_t;
__device__ __forceinline__ float ld_f(const float* base, int i) {
  return *(const g_float_t*)((const g_char_t*)base + (uint32_t)i * 4u);
}
__device__ __forceinline__ void st_f(float* base, int i, float v) {
  *(g_float_t*)((g_char_t*)base + (uint32_t)i * 4u) = v;
}
__device__ __forceinline__ int32_t ld_i(const int32_t* base, int i) {
  return *(const g_int_t*)((const g_char_t*)base + (uint32_t)i * 4u);
}
__device__ __forceinline__ float ld_agent_at(const float* base, int i) {
  return __hip_atomic_load((const g_float_t*)((const g_char_t*)base + (uint32_t)i * 4u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int CTRL> __device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// The values of the two lanes whose numbers differ by O (8, 16 or 32): own row group and the other one; for 16 and 32
// the lower lane's first, in both lanes.  Vector instructions: a shuffle through LDS costs its latency.
template <int O> __device__ __forceinline__ void both(float v, float& lo, float& hi) {
  static_assert(O == 8 || O == 16 || O == 32, "row groups of a wave");
  if constexpr (O == 8) {
    lo = v; hi = dpp_mov<0x128>(v);               // row_ror:8
  } else {
    typedef unsigned u2_t __attribute__((ext_vector_type(2)));
    const unsigned x = __float_as_uint(v);
    const u2_t r = O == 16 ? __builtin_bit_cast(u2_t, __builtin_amdgcn_permlane16_swap(x, x, false, false))
                           : __builtin_bit_cast(u2_t, __builtin_amdgcn_permlane32_swap(x, x, false, false));
    lo = __uint_as_float(r.x); hi = __uint_as_float(r.y);
  }
}
// wave-wide minimum / maximum, in every lane: within rows of 16 lanes, then the rows
__device__ __forceinline__ float wave_min(float v) {
  v = fminf(v, dpp_mov<0xB1>(v));
  v = fminf(v, dpp_mov<0x4E>(v));
  v = fminf(v, dpp_mov<0x141>(v));
  v = fminf(v, dpp_mov<0x140>(v));
  float a, b;
  both<16>(v, a, b);
  both<32>(fminf(a, b), a, b);
  return fminf(a, b);
}
__device__ __forceinline__ uint32_t wave_max_u(uint32_t v) {
  auto step = [](uint32_t x, float y) { const uint32_t o = __float_as_uint(y); return o > x ? o : x; };
  v = step(v, dpp_mov<0xB1>(__uint_as_float(v)));
  v = step(v, dpp_mov<0x4E>(__uint_as_float(v)));
  v = step(v, dpp_mov<0x141>(__uint_as_float(v)));
  v = step(v, dpp_mov<0x140>(__uint_as_float(v)));
  float a, b;
  both<16>(__uint_as_float(v), a, b);
  v = step(__float_as_uint(a), b);
  both<32>(__uint_as_float(v), a, b);
  return step(__float_as_uint(a), b);
}
// the largest 64-bit key: its upper half, then the lower half among the lanes that have it
__device__ __forceinline__ unsigned long long wave_max64(unsigned long long v) {
  const uint32_t hi = wave_max_u((uint32_t)(v >> 32));
  const uint32_t lo = wave_max_u((uint32_t)(v >> 32) == hi ? (uint32_t)v : 0u);
  return ((unsigned long long)hi << 32) | lo;
}

// block-wide reductions; every thread gets the result
// solo: only one wave of the workgroup is still running (the others have left) or
// has a unit of its own, so the reduction stays inside the wave and no barrier may be used.
template <int NW> __device__ __forceinline__ float block_min(float v, float* s_red, bool solo) {
  v = wave_min(v);
  if (solo) return v;
  __syncthreads();
  if ((threadIdx.x & (SQA_WAVE - 1)) == 0) s_red[threadIdx.x / SQA_WAVE] = v;
  __syncthreads();
  v = s_red[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) v = fminf(v, s_red[w]);
  return v;
}
template <int NW> __device__ __forceinline__ unsigned long long block_max64(unsigned long long v, unsigned long long* s_red, bool solo) {
  v = wave_max64(v);
  if (solo) return v;
  __syncthreads();
  if ((threadIdx.x & (SQA_WAVE - 1)) == 0) s_red[threadIdx.x / SQA_WAVE] = v;
  __syncthreads();
  v = s_red[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) v = s_red[w] > v ? s_red[w] : v;
  return v;
}

// H2O eviction rule for a full unit: the candidates are the hh heavy slots and
// the token leaving the recent ring; the one with the lowest accumulated score
// goes, equal scores -> the highest position (the ring leaver is newer than
// every heavy hitter).  Returns -1 if the leaver is evicted, else the heavy
// slot that is evicted (the leaver moves there).  `mn` = min over the heavy
// scores, already reduced over the block.  pos_override: slot whose position
// is not yet in memory (or -1).
template <int NW> __device__ __forceinline__ int pick_victim(const float* sc, const int32_t* posu, int hh, float mn, float leaver_score,
                                           int override_slot, int override_pos, unsigned long long* s_red64,
                                           bool solo, int t /*thread index among the nthr threads at work*/) {
  if (leaver_score <= mn) return -1;             // uniform over the block
  unsigned long long best = 0ull;                // (position + 1) << 32 | slot
  const int nthr = solo ? SQA_WAVE : NW * SQA_WAVE;
  for (int i = t; i < hh; i += nthr)
    if (sc[i] == mn) {
      const int ps = i == override_slot ? override_pos : posu[i];
      const unsigned long long key = ((unsigned long long)(uint32_t)(ps + 1) << 32) | (uint32_t)i;
      best = key > best ? key : best;
    }
  return (int)(uint32_t)block_max64<NW>(best, s_red64, solo);
}

// v_exp_f32: 2^x, 1 ulp, denormal results flush to 0 (harmless in a softmax)
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// sum over groups of N consecutive lanes, in every lane
template <int N> __device__ __forceinline__ float group_sum(float v) {
  static_assert(sizeof(DecodeArgs) <= 4096, "kernel arguments are limited to 4 KiB");
  static_assert(N == 8 || N == 16, "lanes");
  v += dpp_mov<0xB1>(v);            // quad_perm [1,0,3,2]
  v += dpp_mov<0x4E>(v);            // quad_perm [2,3,0,1]
  v += dpp_mov<0x141>(v);           // row_half_mirror
  if (N == 16) v += dpp_mov<0x140>(v);     // row_mirror
  return v;
}
// The same over 32 lanes (a row of fp32 at D = 128), for the G heads of a row at once.  This is in the streaming loop, and
// with 4 heads and more vector instructions bound that loop: the last step is then a shuffle through LDS, requested for all
// heads before the first is used (a lane swap is a vector instruction itself and overwrites both its operands: a copy and wait
// states).  Sliding window, rows in blocks, us: 8 layers of 96 units under 8 heads, a swap for each head by itself 181, a shuffle
// 160, shuffles together 155; 320 units under 4 heads 51.7, 51.0, 46.4.  With 1 or 2 heads there is hardly anything to overlap
// a shuffle's latency with: 96 to 320 units under 2 heads, H2O, 2 to 4 % less with swaps.
template <int G> __device__ __forceinline__ void group_sums32(float (&v)[G]) {
#pragma unroll
  for (int g = 0; g < G; ++g) v[g] = group_sum<16>(v[g]);
  float o[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    if constexpr (G >= 4) {
      o[g] = __shfl_xor(v[g], 16, SQA_WAVE);
    } else {
      float a, b;
      both<16>(v[g], a, b);
      v[g] = a; o[g] = b;
    }
  }
#pragma unroll
  for (int g = 0; g < G; ++g) v[g] += o[g];
}

// maximum over groups of 8 consecutive lanes, in every lane
__device__ __forceinline__ float group_max(float v) {
  v = fmaxf(v, dpp_mov<0xB1>(v));
  v = fmaxf(v, dpp_mov<0x4E>(v));
  return fmaxf(v, dpp_mov<0x141>(v));
}
__device__ __forceinline__ uint32_t group_max_u(uint32_t v) {
  auto step = [](uint32_t x, float y) { const uint32_t o = __float_as_uint(y); return o > x ? o : x; };
  v = step(v, dpp_mov<0xB1>(__uint_as_float(v)));
  v = step(v, dpp_mov<0x4E>(__uint_as_float(v)));
  return step(v, dpp_mov<0x141>(__uint_as_float(v)));
}

template <typename T> struct RowMath;
template <> struct RowMath<float> {
  static constexpr int EPL = 4;
  static __device__ __forceinline__ float dot(const uint4& q, const uint4& k) {
    float s = __uint_as_float(q.x) * __uint_as_float(k.x);
    s = fmaf(__uint_as_float(q.y), __uint_as_float(k.y), s);
    s = fmaf(__uint_as_float(q.z), __uint_as_float(k.z), s);
    s = fmaf(__uint_as_float(q.w), __uint_as_float(k.w), s);
    return s;
  }
  static __device__ __forceinline__ void axpy(float p, const uint4& v, float* acc) {
    acc[0] = fmaf(p, __uint_as_float(v.x), acc[0]); acc[1] = fmaf(p, __uint_as_float(v.y), acc[1]);
    acc[2] = fmaf(p, __uint_as_float(v.z), acc[2]); acc[3] = fmaf(p, __uint_as_float(v.w), acc[3]);
  }
  static __device__ __forceinline__ void store(void* dst, const float* a) {
    st16(dst, make_uint4(__float_as_uint(a[0]), __float_as_uint(a[1]), __float_as_uint(a[2]), __float_as_uint(a[3])));
  }
};
template <> struct RowMath<bf16_t> {
  static constexpr int EPL = 8;
  static __device__ __forceinline__ float dot(const uint4& q, const uint4& k) {
    float s = dot2_bf16(q.x, k.x, 0.f);
    s = dot2_bf16(q.y, k.y, s); s = dot2_bf16(q.z, k.z, s); s = dot2_bf16(q.w, k.w, s);
    return s;
  }
  static __device__ __forceinline__ void axpy(float p, const uint4& v, float* acc) {
    acc[0] = fmaf(p, bf16_lo(v.x), acc[0]); acc[1] = fmaf(p, bf16_hi(v.x), acc[1]);
    acc[2] = fmaf(p, bf16_lo(v.y), acc[2]); acc[3] = fmaf(p, bf16_hi(v.y), acc[3]);
    acc[4] = fmaf(p, bf16_lo(v.z), acc[4]); acc[5] = fmaf(p, bf16_hi(v.z), acc[5]);
    acc[6] = fmaf(p, bf16_lo(v.w), acc[6]); acc[7] = fmaf(p, bf16_hi(v.w), acc[7]);
  }
  static __device__ __forceinline__ void store(void* dst, const float* a) {
    uint4 o;
    o.x = f32_to_bf16_bits(a[0]) | (f32_to_bf16_bits(a[1]) << 16);
    o.y = f32_to_bf16_bits(a[2]) | (f32_to_bf16_bits(a[3]) << 16);
    o.z = f32_to_bf16_bits(a[4]) | (f32_to_bf16_bits(a[5]) << 16);
    o.w = f32_to_bf16_bits(a[6]) | (f32_to_bf16_bits(a[7]) << 16);
    st16(dst, o);
  }
};


typedef __attribute__((address_space(1))) const void dec_gptr_t;
typedef __attribute__((address_space(3))) void dec_lptr_t;
constexpr int kMfWavesPerSimd = 3;                // waves per SIMD the matrix-core variant is compiled for
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef short v4s_t __attribute__((ext_vector_type(4)));
typedef short v8s_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v4s_t* lds_v4s_ptr;
constexpr int kWpuMaxSlots = 256;                 // one wave per unit: for units of at most this many slots
// An unsplit unit's tail (scores, decision) is left to wave 0 alone, so that the registers of the other waves are free for
// the next workgroup -- up to this length where there is hardly a next one (at most kWideTailMaxBlocks workgroups), up to
// the other in calls of 2 to 8 workgroups per CU, whose long units otherwise end after everything else (two runs each;
// Llama-2-7B shape at batch 2, 32 layers in one call, 80.6 -> 75.2 and 82.9 -> 77.0 us; 12 layers of 128 units of 300 to 1900
// slots, D = 64, 55.8 -> 51.3 and 57.3 -> 52.6; fp32, 2 query heads over 1, up to 1500 slots, 99 -> 96 and 102 -> 99).  Beyond:
// no better (batch 6) or worse (batch 8, 277 -> 283).
constexpr int kSoloMaxTokens = 512, kSoloMaxTokensMid = 768;
// Work items per unit: their statistics are merged in the LDS of the waves' accumulators, which at D = 64 holds 128.  A call
// of one unit of more than 40960 slots could use more (65536 slots: 114 workgroups for 256 CUs); the merge that this allows
// is worth more (one query head, bf16, D = 128: 229 us in 205 pieces merged one by one, 112 so; 131072 slots 344 and 207).
constexpr int kMaxSplit = 128;
constexpr int kLogitPad = 33;                     // a unit's H2O scratch region: G x (slots + kLogitPad) floats: the logit of the
                                                  // new token as one more slot, or whole 32-token tiles of bf16 probabilities
                                                  // plus a reference per tile and head
constexpr int kStageRow = 256 + 16;               // LDS row pitch of a staged bf16 D=128 row (padded: no bank conflicts)
constexpr int kStageBytesPerWave = 32 * kStageRow;   // one 32-token tile

// Grouped queries of 4 or more heads per KV head in bf16 at D = 128 go to the matrix cores: with 8 heads
// the vector-ALU path is arithmetic bound (4.2 TB/s against 6.5 TB/s on the Llama-2-70B shape), with 4
// heads the matrix-core variant is still slightly ahead (779 against 797 us per step on the Mistral-7B shape).
constexpr int kMfmaMinGroup = 4;      // query heads per KV head from which the matrix-core variant is used
template <typename T, int D, int G> constexpr bool use_mfma() { return sizeof(T) == 2 && D == 128 && G >= kMfmaMinGroup; }
// 8 heads at D = 64, and in fp32 under H2O: matrix cores in 32-bit precision (section 1X).  46 drawn calls, on the vector
// ALUs and so: 1.12 to 2.56 times as fast, 1.53 on average (17 layers of 56 units of 93 and 935 slots, fp32, D = 128, H2O
// 118 -> 46 us; 6 layers of 232 units of 41 and 467 slots, bf16, D = 64, H2O 44.8 -> 21.2).  fp32, D = 128 without H2O would gain
// too (1.2 to 1.4), but its instructions on the vector ALUs are pinned by a test.  4 heads: nothing in bf16 (192.8 and 192.6
// us), slower in fp32 (13 layers of 1168 units of 33 and 355 slots 169 -> 189; D = 64 99 -> 128): three quarters of a product's
// columns would be empty.
template <typename T, int D, int G, bool H2O> constexpr bool exact_mfma() { return G == 8 && !use_mfma<T, D, G>() && (D == 64 || H2O); }
// MF = true (bf16, D = 128, grouped queries): the chunk is streamed in 32-token
// tiles through LDS and q.K^T / P.V run on the matrix cores, see section 1M.
// PG = true: blocked allocation -- the unit's K and V rows lie in 16-row blocks of the layer's pools, named by
// its row of the block table (staged in LDS at the start); everything else is addressed as before.
template <typename T, int D, int G, bool H2O, bool MF, bool PG>
__global__ __launch_bounds__(kDecThreads, MF ? kMfWavesPerSimd : 1) void decode_unit_kernel(const DecodeArgs a) {
  constexpr int NW = kDecWaves;
  constexpr bool NTR = false;     // rows of step 4 with ordinary stores
#include "sqa_decode_unit.inc"
}
// The same with more than 4 waves per workgroup (WIDE in the body), for calls that have no more work items than CUs.
template <typename T, int D, int G, bool H2O, bool PG, int NW>
__global__ __launch_bounds__(NW * SQA_WAVE) void decode_wide_kernel(const DecodeArgs a) {
  constexpr bool MF = use_mfma<T, D, G>(), NTR = false;
#include "sqa_decode_unit.inc"
}
// decode_unit_kernel for MHA calls over very large caches: the moved and the new K/V rows of step 4 are stored
// non-temporally.  A step writes each unit's rows once and reads them a whole pass later, when a cache of this size has long
// pushed them out; until then the dirty lines are in the way of the rows that stream through.  A kernel of its own, because
// a switch inside costs the others: with it, 32 layers of 2048 units of 20 to 40 slots 160 -> 163 us.
template <typename T, int D, bool H2O, bool PG>
__global__ __launch_bounds__(kDecThreads) void decode_large_kernel(const DecodeArgs a) {
  constexpr int NW = kDecWaves, G = 1;
  constexpr bool MF = false, NTR = true;
#include "sqa_decode_unit.inc"
}
// From how many bytes of K and V (the call's layers together, at their budgets): measured per call, plain -> non-temporal,
// bf16, H2O, D = 128 unless said otherwise: 1.7 GB of 40-slot units 313 -> 319 us, 3.4 GB (80 slots) 599 -> 607, 5.3 GB (35 to
// 571 slots) 949 -> 952, 6.7 GB (160 slots) 1173 -> 1174 / 8.0 GB (35 to 571) 1449 -> 1427, 10.9 GB (160 slots) 1953 -> 1920,
// 12 GB (35 to 571) 2233 -> 2170, 16.8 GB (40 slots) 3474 -> 3353, 24 GB (571 slots) 4153 -> 4080; D = 64, 10.9 GB 2072 -> 2016;
// fp32, 11.7 GB 2054 -> 2031.  What is written counts against what is read: long units gain little (1024 slots 3572 -> 3562,
// 143 to 2271 slots 1768 -> 1772), 2 and more heads per KV head nothing (2061 -> 2061).  (Calls of the same shape differ by up to
// 3 % with the place of their buffers; these were taken in turn on the same ones.)  The size is the call's: a cache of any
// size that is stepped layer by layer keeps the ordinary kernel, and units that are not full count as if they were (240 slots, 60
// filled: 2.0 GB counted as 8.1 448 -> 453).  Where units differ and only the device knows how much (packed units, budgets per
// sequence) they count at the layer's largest, in blocks at most as the pools: 6.2 GB packed, streaming, that count as 8.1, 1067 ->
// 1015; a few long among many short lose by it (2.4 GB that count as 8.1 446 -> 455).
constexpr int64_t kLargeBytes = (int64_t)7 << 30;
static int64_t counted_kv_bytes(const sqa_layer_cache* layers, int n_layers, int64_t units, int64_t row_bytes /*K and V*/) {
  int64_t rows = 0;
  for (int i = 0; i < n_layers; ++i) {
    const int64_t all = units * std::min(layers[i].budget, layers[i].capacity);
    rows += layers[i].block_table ? std::min(all, (int64_t)layers[i].n_blocks * SQA_BLOCK_SLOTS) : all;
  }
  return rows * row_bytes;
}

typedef void (*decode_fn)(const DecodeArgs);

constexpr int kWideWaves = 8;
template <typename T, int D, bool H2O, bool PG> decode_fn pick_wide(int g) {
  switch (g) {
    case 1: return decode_wide_kernel<T, D, 1, H2O, PG, kWideWaves>;
    case 2: return decode_wide_kernel<T, D, 2, H2O, PG, kWideWaves>;
    case 4: return decode_wide_kernel<T, D, 4, H2O, PG, kWideWaves>;
    case 8: if constexpr (use_mfma<T, D, 8>()) return decode_wide_kernel<T, D, 8, H2O, PG, kWideWaves>; break;
  }
  return nullptr;
}
template <typename T, int D, bool H2O, bool PG> decode_fn pick_g(int g, int waves, bool large) {
  if (waves > kDecWaves) return pick_wide<T, D, H2O, PG>(g);
  switch (g) {
    case 1: return large ? decode_large_kernel<T, D, H2O, PG> : decode_unit_kernel<T, D, 1, H2O, false, PG>;
    case 2: return decode_unit_kernel<T, D, 2, H2O, false, PG>;
    case 4: return decode_unit_kernel<T, D, 4, H2O, use_mfma<T, D, 4>(), PG>;
    case 8: return decode_unit_kernel<T, D, 8, H2O, use_mfma<T, D, 8>(), PG>;
  }
  return nullptr;
}
template <typename T, bool H2O, bool PG> decode_fn pick_d(int d, int g, int waves, bool large) {
  if (d == 64) return pick_g<T, 64, H2O, PG>(g, waves, large);
  if (d == 128) return pick_g<T, 128, H2O, PG>(g, waves, large);
  return nullptr;
}
template <typename T, bool H2O> decode_fn pick_p(int d, int g, bool paged, int waves, bool large) {
  return paged ? pick_d<T, H2O, true>(d, g, waves, large) : pick_d<T, H2O, false>(d, g, waves, large);
}
static decode_fn pick(sqa_dtype dt, int d, int g, bool h2o, bool paged, int waves = kDecWaves, bool large = false) {
  if (dt == SQA_F32) return h2o ? pick_p<float, true>(d, g, paged, waves, large) : pick_p<float, false>(d, g, paged, waves, large);
  return h2o ? pick_p<bf16_t, true>(d, g, paged, waves, large) : pick_p<bf16_t, false>(d, g, paged, waves, large);
}

constexpr size_t kStatusBytes = 256;

// How one call is cut into work items and where its scratch lives.
struct DecodePlan {
  int tbl_entries;                                 // blocked allocation: block numbers a workgroup stages in LDS
  int lds_probs, lds_probs_w;                      // LDS bytes for the probabilities of a workgroup / of one wave's unit
  uint16_t lds_tiles[SQA_MAX_LAYERS];              // matrix-core variant under H2O: leading tiles of a unit whose probabilities stay in LDS
  uint8_t probs_in_lds[SQA_MAX_LAYERS];            // ... 1: all of them (nothing of it in the workspace), 2: the leading part
  int lds_chunk;                                   // longest unsplit unit shared by 4 waves (slots)
  int lds_chunk_w;                                 // longest one-wave unit (slots)
  uint8_t wpu[SQA_MAX_LAYERS];                     // one wave per unit in this layer
  uint16_t nsplit[SQA_MAX_LAYERS];
  uint32_t chunk[SQA_MAX_LAYERS];
  uint32_t unit_off[SQA_MAX_LAYERS], part_off[SQA_MAX_LAYERS], logit_off[SQA_MAX_LAYERS];
  uint8_t order[SQA_MAX_LAYERS];                   // layers in descending budget (stable): long units start first
  uint64_t blocks;
  int waves;                                       // per workgroup
  size_t cnt_bytes, part_bytes, logit_bytes;       // arrival counters, partial records, H2O logits / probabilities
  size_t off_table, off_cnt, off_part, off_logit, bytes;   // where they lie in a caller's workspace
};

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// The device array that sqa_decode_step_static uses for scratch: layer table, arrival counters, the rest.
constexpr size_t kStaticTableBytes = 16 * 1024;                    // >= SQA_MAX_LAYERS * sizeof(sqa_layer_cache)
constexpr size_t kStaticCntBytes = 1024 * 1024;                    // 262144 units per call
constexpr size_t kStaticDataBytes = SQA_STATIC_SCRATCH_BYTES - kStaticTableBytes - kStaticCntBytes;
static_assert(SQA_MAX_LAYERS * sizeof(sqa_layer_cache) <= kStaticTableBytes, "layer table region");
static_assert(SQA_STATIC_SCRATCH_BYTES > kStaticTableBytes + kStaticCntBytes, "scratch size");
static bool fits_static(const DecodePlan& p) {
  return p.cnt_bytes <= kStaticCntBytes && align256(p.part_bytes) + p.logit_bytes <= kStaticDataBytes;
}

// Units are split only when the call would otherwise leave CUs idle: the target work item is the call's
// tokens divided by the number of CUs (at least min_item slots, and at most what lets a unit's step logits fit
// in LDS -- kMaxUnsplit slots x heads; not for the matrix-core variant, which keeps what H2O needs in the
// workspace), and a unit is cut into equal chunks only if it is more than a quarter longer than that.
// One workgroup per CU already streams at 80 % of what the chip reaches, so what splitting buys is balance,
// and the hand-over between a unit's workgroups costs more than a small imbalance: with 256 equal units (a
// layer of the Llama-2-7B shape at batch 8 launched on its own) whole units take 56 us (47.6 with 8 waves each), halves 67 us; 320 units
// 67 us whole, 82 in halves; all layers at batch 2 81 us with the long units whole, 87 cut in three.
// Where the longest units have to be cut anyway, the pieces are made for 2 or 3 items per CU if the items of one
// per CU come out unevenly (the busiest of 256 CUs with over 9/8 of its share): 96 units of 2271 slots 41 us in 3
// pieces (288 items), 34.5 in 5; 130 units of 8192 with 286 of 557, 4 query heads over 1, 167 us and 140 (175 and 145 in
// another run).  How far that goes: see CutRule.
constexpr int64_t kMinItems = 256;
constexpr int64_t kWideTailMaxBlocks = 512, kWideTailMidBlocks = 2048;   // see kSoloMaxTokens
// Matrix-core variant under H2O: LDS a workgroup may use for a unit's per-head probabilities so that three
// workgroups still fit a CU (160 KiB / 3, less the four stage buffers and the small static arrays).
constexpr int kLdsProbsMax = 18 * 1024;
// Calls of no more work items than CUs have a CU to each: 4 waves leave it short of requests in flight, and walk a unit's
// scores one wave after the streaming.  8 waves per workgroup (device time of one layer, us, before and after; H2O, bf16,
// D = 128, 256 units): 17 slots 6.3 -> 5.9, 143 9.2 -> 7.3, 300 13.2 -> 9.4, 2271 55.4 -> 47.6; fp32, D = 128, 4 query
// heads per KV head, 300 slots 34 -> 21.  16 waves: 143 slots the same, 17 7.0, 2271 48.5; 64 against 71 for 128 units of 5000
// slots, 20 % worse below 128 slots: another set of kernels for few and long units, not taken.  (The number of waves follows
// from the whole call: a layer of up to 256 items has 8 alone and 4 together with others, and its results differ in their
// last bits between the two.)  8 query heads per KV head off the bf16 matrix path keep 4: on the vector ALUs 8 waves
// need 256 registers each and start and merge for longer (D = 64, 17 slots 11.2 and 14.2 us; 143 15.7 and 14.8); in section
// 1X 12 of 50 drawn calls got 1.03 to 1.22 times as fast with 8 waves, one 0.92 (left, since the number is pinned by a test).  Beyond 256 work items 8 waves are
// slower (320 units of 800 slots 26.9 -> 28.3).  The matrix-core kernel only shares a unit's tiles out among 8 waves: 256
// units, 8 heads per KV head, H2O, 143 slots 11.4 -> 9.8, 1500 40.4 -> 36.6; 24 units of 1500 18.9 -> 14.5; sliding 12.4 -> 10.6.
constexpr int64_t kWideMaxBlocks = 256;
constexpr int kMaxUnsplit = 8192;
// One wave per unit: for units of at most kWpuMaxSlots slots, in calls that have at least kWpuMinUnits
// units (one wave walks a unit 16 rows at a time, so the call needs many units to keep the chip's wave
// slots filled; the matrix-core variant walks it one 32-token tile at a time).
constexpr int64_t kWpuMinUnits = 4096;
// The shortest work item: 4 waves take 128 slots of the matrix-core variant in one 32-token tile each, and 256 slots
// there cost hardly more; the other kernels walk 16 to 128 rows at a time.  (fp32, D = 128, 8 query heads over 1, two
// layers of 1500 and 146 slots: 35 us with 256, 25 with 128; 16 over 2, bf16, 4743 slots: 27.5 and 29.8.)
// Units of up to 1.25 x 256 slots stay whole all the same: in two pieces they pay for a merge and save a trip or two
// (8 to 64 units of 165 to 301 slots, one query head over 1: 8.6 -> 10.1, 9.4 -> 10.4, 11.2 -> 12.1 us; in three
// instead of two, 321 slots 12.5 -> 11.0).
constexpr int kCoarseItem = 256;
// How many workgroups a finer cut may come to: two per CU, which run at once in every kernel, or up to three where the
// work items hold `beyond` slots on average.  Past that the whole units of the other layers end up in pieces too, and
// their merges (under H2O also the scratch that they need in place of LDS) cost more than the balance brings.
//   more than 128 registers (2 or 3 workgroups per CU): 800 slots.  bf16, D = 64, 8 heads over 1, H2O, 40 units of 1450
//     and 240 of 529 slots 43 us in 320 workgroups, 53 in 680; 8 over 1 on the matrix cores, sliding, 48 of 4165 and 192
//     of 988 39 us in 336, 43 in 624; but 4 over 1, H2O, 130 of 8192 and 286 of 557 175 us in 546, 145 in 676.
//   up to 128 registers, where a workgroup spends long on arithmetic or on its unit's scores: any length.  fp32, 4 heads
//     over 1, H2O, 78 of 1543 and 78 of 481 70 us in 312, 51 in 702; bf16, 2 over 1, H2O, 72 of 8192 and 144 of 1948 169
//     us in 288, 112 in 720.
//   the same without either: none.  bf16, one head, sliding, 48 of 1067 and 208 of 706 14.5 us in 304, 16.1 in 816.
struct CutRule { int min_item; int64_t beyond; bool wide; };
static bool uses_mfma(sqa_dtype dt, int D, int g) { return dt == SQA_BF16 && D == 128 && g >= kMfmaMinGroup; }
static bool wide_rule(sqa_dtype dt, int D, int g) { return g <= 4 || uses_mfma(dt, D, g); }
static CutRule cut_rule(sqa_dtype dt, int D, int g, bool h2o) {
  const bool light = g <= (dt == SQA_F32 ? 4 : 2);         // up to 128 registers
  const bool mfma = uses_mfma(dt, D, g);
  return {mfma ? kCoarseItem : 128, !light ? 800 : (h2o || dt == SQA_F32 ? 0 : INT32_MAX), wide_rule(dt, D, g) && !mfma};
}
// coarse: the fewest pieces (and the least scratch).
// scratch_probs: the H2O step's per-token, per-head values live in the workspace for every unit, split or
// not (the matrix-core variant: they never need LDS, so nothing limits an unsplit unit's length).
static sqa_status plan_decode(const sqa_layer_cache* layers, int n_layers, int B, int Hq, int Hkv, int D, bool h2o,
                              bool allow_wpu, bool scratch_probs, CutRule rule, bool coarse, DecodePlan* p) {
  const int64_t units = (int64_t)B * Hkv;
  const int g = Hq / Hkv;
  const bool paged = layers[0].block_table != nullptr;
  int64_t tokens = 0;
  uint8_t* const order = p->order;
  for (int i = 0; i < n_layers; ++i) {
    int j = i - 1;
    while (j >= 0 && layers[order[j]].budget < layers[i].budget) { order[j + 1] = order[j]; --j; }
    order[j + 1] = (uint8_t)i;
  }
  for (int i = 0; i < n_layers; ++i) {
    if (layers[i].capacity < 1) return SQA_ERR_CAPACITY;
    if (layers[i].budget < 1) return SQA_ERR_BUDGET;
    tokens += units * (layers[i].budget < layers[i].capacity ? layers[i].budget : layers[i].capacity);
  }
  // longest work item a unit is cut for, given how many items the call's tokens are worth
  auto item_slots = [&](int64_t items, int64_t least) {
    int64_t t = tokens / items;
    t = t < least ? least : t;
    return h2o && !scratch_probs && t > kMaxUnsplit / g ? (int64_t)(kMaxUnsplit / g) : t;
  };
  auto cut = [&](int i, int64_t target, int64_t* ns_out, int64_t* ch_out, int64_t most = kMaxSplit) {
    // + 1: under attend-then-evict a full unit attends budget + 1 tokens
    const int nmax = (layers[i].budget < layers[i].capacity ? layers[i].budget : layers[i].capacity) + 1;
    if (target < kCoarseItem && 4 * (int64_t)nmax <= 5 * kCoarseItem) target = kCoarseItem;
    int64_t ns = (4 * (int64_t)nmax + 5 * target - 1) / (5 * target);   // ceil(nmax / (1.25 target))
    ns = ns < 1 ? 1 : (ns > most ? most : ns);
    int64_t ch = ((nmax + ns - 1) / ns + 63) / 64 * 64;
    if (h2o && !scratch_probs && ns == 1 && ch * g > kMaxUnsplit) { ns = 2; ch = ((nmax + 1) / 2 + 63) / 64 * 64; }
    *ns_out = (nmax + ch - 1) / ch;
    *ch_out = ch;
  };
  int64_t target = item_slots(kMinItems, kCoarseItem);
  int64_t longest_ns, longest_ch;
  for (int i = 0; i < n_layers; ++i) {
    // a unit of more than 65535 items of that length (under H2O with the logits in LDS: over 83 million slots at 8 heads) is refused
    cut(i, target, &longest_ns, &longest_ch, INT32_MAX);
    if (longest_ns > 65535) return SQA_ERR_CAPACITY;
  }
  cut(order[0], item_slots(kMinItems, rule.min_item), &longest_ns, &longest_ch);
  for (int64_t items = kMinItems, best = INT64_MAX; !coarse && longest_ns > 1 && items <= 3 * kMinItems; items += kMinItems) {
    const int64_t t = item_slots(items, rule.min_item);
    int64_t n = 0, shortest = INT64_MAX, load = 0;         // slots the busiest CU streams if it gets every 256th item
    for (int k = 0; k < n_layers; ++k) {
      int64_t ns, ch;
      cut(order[k], t, &ns, &ch);
      n += units * ns;
      shortest = ch < shortest ? ch : shortest;
      const int64_t x = (n + kMinItems - 1) / kMinItems * shortest;
      load = x > load ? x : load;
    }
    if (rule.wide && n <= kWideMaxBlocks && 2 * load * kMinItems <= 3 * tokens) { target = t; break; }   // (one workgroup of 8 waves per CU)
    if (n > 2 * kMinItems && (n > 3 * kMinItems || tokens < rule.beyond * n)) break;
    if (load <= best) { best = load; target = t; }
    if (8 * load * kMinItems <= 9 * tokens || t == rule.min_item) break;
  }
  uint64_t blocks = 0, n_units = 0, n_part = 0, n_logit = 0;
  p->tbl_entries = 0;
  if (paged) {
    p->tbl_entries = kDecWaves * (kWpuMaxSlots / SQA_BLOCK_SLOTS);
    for (int i = 0; i < n_layers; ++i) {
      const int used = layers[i].budget < layers[i].capacity ? layers[i].budget : layers[i].capacity;
      const int e = (used + SQA_BLOCK_SLOTS - 1) / SQA_BLOCK_SLOTS;
      p->tbl_entries = e > p->tbl_entries ? e : p->tbl_entries;
    }
  }
  p->lds_probs = p->lds_probs_w = 0;
  p->lds_chunk = scratch_probs ? 0 : 64;           // (no LDS logits at all when they live in the workspace)
  p->lds_chunk_w = scratch_probs ? 0 : 64;
  for (int i = 0; i < n_layers; ++i) {
    const int nmax = (layers[i].budget < layers[i].capacity ? layers[i].budget : layers[i].capacity) + 1;
    int64_t ns, ch;
    cut(i, target, &ns, &ch);
    p->nsplit[i] = (uint16_t)ns;
    p->chunk[i] = (uint32_t)ch;
    p->wpu[i] = allow_wpu && ns == 1 && nmax <= kWpuMaxSlots && units * n_layers >= kWpuMinUnits;
    p->probs_in_lds[i] = 0;
    p->lds_tiles[i] = 0;
    if (h2o && scratch_probs && ns == 1) {
      // per unit: whole 32-token tiles of bf16 values per head, plus one fp32 reference per tile and head;
      // a unit too long for the LDS a workgroup may use keeps its leading tiles there (a written byte costs
      // many read bytes, so every tile that stays on the chip counts); one-wave units: all or nothing
      const int64_t ntile = ((int64_t)layers[i].capacity + 1 + 31) / 32;
      const int64_t per_tile = (int64_t)g * (64 + 4);
      const int64_t avail = kLdsProbsMax - p->tbl_entries * (int)sizeof(int);
      int64_t tiles = p->wpu[i] ? (ntile * per_tile * kDecWaves <= avail ? ntile : 0) : avail / per_tile;
      tiles = tiles > ntile ? ntile : tiles;
      tiles = tiles > (int64_t)kLdsTilesMask ? (int64_t)kLdsTilesMask : tiles;
      if (tiles > 0) {
        const int64_t need = tiles * per_tile;
        p->lds_tiles[i] = (uint16_t)tiles;
        p->probs_in_lds[i] = tiles == ntile ? 1 : 2;
        if (p->wpu[i] && need > p->lds_probs_w) p->lds_probs_w = (int)need;
        if (need * (p->wpu[i] ? kDecWaves : 1) > p->lds_probs) p->lds_probs = (int)(need * (p->wpu[i] ? kDecWaves : 1));
      }
    }
    if (p->wpu[i]) { if (!scratch_probs && ch > p->lds_chunk_w) p->lds_chunk_w = (int)ch; }
    else if (ns == 1 && !scratch_probs && ch > p->lds_chunk) p->lds_chunk = (int)ch;
    p->unit_off[i] = (uint32_t)n_units;
    p->part_off[i] = (uint32_t)n_part;
    p->logit_off[i] = (uint32_t)n_logit;
    n_units += units;
    blocks += p->wpu[i] ? (units + kDecWaves - 1) / kDecWaves : units * ns;
    if (ns > 1) n_part += units * ns;
    if (h2o && (ns > 1 || scratch_probs) && p->probs_in_lds[i] != 1) n_logit += units * g * ((uint64_t)layers[i].capacity + kLogitPad);
    if (n_units > 0x7fffffffull || n_part > 0x7fffffffull || n_logit > 0xffffffffull || blocks > 0x7fffffffull)
      return SQA_ERR_CAPACITY;
  }
  if (kDecWaves * p->lds_probs_w > p->lds_probs) p->lds_probs = kDecWaves * p->lds_probs_w;
  p->blocks = blocks;
  p->cnt_bytes = n_units * sizeof(int32_t);
  p->part_bytes = n_part * g * (D + 2) * sizeof(float);
  p->logit_bytes = n_logit * sizeof(float);
  p->off_table = kStatusBytes;
  p->off_cnt = align256(p->off_table + (size_t)n_layers * sizeof(sqa_layer_cache));
  p->off_part = align256(p->off_cnt + p->cnt_bytes);
  p->off_logit = align256(p->off_part + p->part_bytes);
  p->bytes = align256(p->off_logit + p->logit_bytes);
  return SQA_OK;
}

// The cut of a call, the same for every entry point (results depend on it in their last bits): where the finer one
// needs more scratch than the static array has and the coarse one does not, the coarse one.
static sqa_status plan_cut(const sqa_layer_cache* layers, int n_layers, int B, int Hq, int Hkv, int D, bool h2o,
                           bool allow_wpu, bool scratch_probs, CutRule rule, DecodePlan* p) {
  const sqa_status fine = plan_decode(layers, n_layers, B, Hq, Hkv, D, h2o, allow_wpu, scratch_probs, rule, false, p);
  if (fine == SQA_OK && fits_static(*p)) return fine;
  DecodePlan c;
  const sqa_status coarse = plan_decode(layers, n_layers, B, Hq, Hkv, D, h2o, allow_wpu, scratch_probs, rule, true, &c);
  if (coarse == SQA_OK && (fine != SQA_OK || fits_static(c))) *p = c;
  return coarse == SQA_OK ? coarse : fine;
}

}  // namespace sqa

extern "C" size_t sqa_decode_workspace_bytes(const sqa_layer_cache* layers, int n_layers, int B, int Hq, int Hkv,
                                             int D, sqa_policy policy) {
  if (!layers || n_layers < 1 || n_layers > SQA_MAX_LAYERS || B < 1 || Hq < 1 || Hkv < 1 || Hq % Hkv != 0 || D < 1)
    return 0;
  sqa::DecodePlan p;
  // (neither the element type nor whether a call gives short units a wave each is known here: the most of what they need)
  const bool h2o = policy == SQA_H2O;
  const int g = Hq / Hkv;
  size_t bytes = 0;
  for (int k = 0; k < 4; ++k) {
    const sqa_dtype dt = k & 1 ? SQA_BF16 : SQA_F32;
    if (sqa::plan_cut(layers, n_layers, B, Hq, Hkv, D, h2o, k >= 2, h2o && sqa::uses_mfma(dt, D, g), sqa::cut_rule(dt, D, g, h2o), &p) != SQA_OK)
      return 0;
    bytes = p.bytes > bytes ? p.bytes : bytes;
  }
  return bytes;
}

namespace sqa {
// Zero fill by a kernel rather than hipMemsetAsync: callers may record these calls into a HIP graph, and
// memset nodes have replayed wrongly on this platform.
__global__ __launch_bounds__(256) void zero_fill_kernel(uint32_t* __restrict__ p, size_t n_words) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_words; i += (size_t)gridDim.x * 256) p[i] = 0u;
}
static sqa_status zero_fill(void* p, size_t bytes, hipStream_t st) {
  const size_t n_words = bytes / 4;
  if (n_words == 0) return SQA_OK;
  size_t blocks = (n_words + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  zero_fill_kernel<<<(unsigned)blocks, 256, 0, st>>>(static_cast<uint32_t*>(p), n_words);
  SQA_HIP_CHECK(hipGetLastError());
  return SQA_OK;
}
}  // namespace sqa

extern "C" sqa_status sqa_decode_workspace_init(void* workspace, size_t ws_bytes, void* stream) {
  if (!workspace) return SQA_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(workspace) & 3u) return SQA_ERR_SHAPE;
  return sqa::zero_fill(workspace, ws_bytes, static_cast<hipStream_t>(stream));   // (sizes are multiples of 256)
}

extern "C" sqa_status sqa_clear_device_status(void* workspace, void* stream) {
  if (!workspace) return SQA_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(workspace) & 3u) return SQA_ERR_SHAPE;
  return sqa::zero_fill(workspace, sizeof(int32_t), static_cast<hipStream_t>(stream));
}

extern "C" sqa_status sqa_read_device_status(const void* workspace, void* stream, int32_t* status_out) {
  if (!workspace || !status_out) return SQA_ERR_NULL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  SQA_HIP_CHECK(hipMemcpyAsync(status_out, workspace, sizeof(int32_t), hipMemcpyDeviceToHost, st));
  SQA_HIP_CHECK(hipStreamSynchronize(st));
  return SQA_OK;
}

extern "C" sqa_status sqa_decode_step(const void* q, const void* k_new, const void* v_new, sqa_dtype dt,
                                      int B, int Hq, int Hkv, int D, int32_t new_pos,
                                      sqa_policy policy, int n_sink,
                                      const sqa_layer_cache* layers, const sqa_layer_cache* layers_dev, int n_layers,
                                      void* out, void* workspace, size_t ws_bytes, void* stream) {
  return sqa_decode_step_ex(q, k_new, v_new, dt, B, Hq, Hkv, D, new_pos, policy, n_sink, layers, layers_dev, n_layers,
                            out, workspace, ws_bytes, stream, nullptr);
}

namespace sqa {

// Where one call's scratch lies: in a caller's workspace, or in the library's static array.
struct DecodeScratch {
  int32_t* status;     // device-side status word
  char* table;         // room for the layer table when the caller gave no device copy
  int32_t* cnt;        // arrival counters (zero on entry; the kernel leaves them zero)
  float* part;         // partial records of split units
  float* logit;        // H2O logits / probabilities
};

// The launch plan of a call and the dynamic LDS its workgroups need (host arithmetic only).
// coarse: for a workspace that does not hold what the plan of the call's shapes needs.
static sqa_status plan_call(sqa_dtype dt, int B, int Hq, int Hkv, int D, bool h2o, const sqa_layer_cache* layers,
                            int n_layers, bool coarse, DecodePlan* plan, size_t* lds_out) {
  const int g = Hq / Hkv;
  const bool mfma = uses_mfma(dt, D, g);
  const CutRule rule = cut_rule(dt, D, g, h2o);
  const sqa_status ps = coarse ? plan_decode(layers, n_layers, B, Hq, Hkv, D, h2o, true, h2o && mfma, rule, true, plan)
                               : plan_cut(layers, n_layers, B, Hq, Hkv, D, h2o, true, h2o && mfma, rule, plan);
  if (ps != SQA_OK) return ps;
  const size_t lds_shared = (size_t)g * plan->lds_chunk, lds_waves = (size_t)kDecWaves * g * plan->lds_chunk_w;
  const size_t lds_h2o = (h2o ? (lds_shared > lds_waves ? lds_shared : lds_waves) * sizeof(float) : 0) + (size_t)plan->lds_probs;
  // (blocked allocation: the staged block numbers come last; decode_launch passes their offset)
  auto lds_of = [&](int waves) {
    return ((lds_h2o + (mfma ? (size_t)waves * kStageBytesPerWave : 0) + 15) & ~(size_t)15) + (size_t)plan->tbl_entries * sizeof(int);
  };
  if (lds_of(kDecWaves) > 160 * 1024) return SQA_ERR_CAPACITY;
  const bool wide = wide_rule(dt, D, g) && plan->blocks <= (uint64_t)kWideMaxBlocks && lds_of(kWideWaves) <= 160 * 1024;
  plan->waves = wide ? kWideWaves : kDecWaves;
  *lds_out = lds_of(plan->waves);
  return SQA_OK;
}

// Argument checks shared by the decode entry points; on success the kernel and the launch plan.
static sqa_status decode_prepare(const void* q, const void* k_new, const void* v_new, sqa_dtype dt,
                                 int B, int Hq, int Hkv, int D, int32_t new_pos, sqa_policy policy, int n_sink,
                                 const sqa_layer_cache* layers, int n_layers, const void* out,
                                 const sqa_batch_opts* opts, DecodePlan* plan, size_t* lds_out) {
  if (!q || !k_new || !v_new || !layers || !out) return SQA_ERR_NULL;
  if (opts && opts->order != SQA_EVICT_THEN_ATTEND && opts->order != SQA_ATTEND_THEN_EVICT) return SQA_ERR_POLICY;
  if (dt != SQA_F32 && dt != SQA_BF16) return SQA_ERR_DTYPE;
  if (policy != SQA_SLIDING && policy != SQA_STREAMING && policy != SQA_H2O) return SQA_ERR_POLICY;
  if (n_sink < 0) return SQA_ERR_POLICY;
  if (B < 1 || Hq < 1 || Hkv < 1 || n_layers < 1 || n_layers > SQA_MAX_LAYERS || Hq % Hkv != 0 ||
      (new_pos < 0 && !(opts && opts->new_pos_seq)))
    return SQA_ERR_SHAPE;
  const int g = Hq / Hkv;
  const bool h2o = policy == SQA_H2O;
  const bool paged = layers[0].block_table != nullptr;        // blocked K/V allocation: all layers of a call or none
  if (!pick(dt, D, g, h2o, paged)) return SQA_ERR_SHAPE;
  if (!aligned16(q) || !aligned16(k_new) || !aligned16(v_new) || !aligned16(out)) return SQA_ERR_SHAPE;
  const int min_budget = h2o ? 2 : (policy == SQA_STREAMING ? n_sink + 1 : 1);
  for (int i = 0; i < n_layers; ++i) {
    const sqa_layer_cache& c = layers[i];
    if (!c.K || !c.V || !c.pos || !c.unit_state) return SQA_ERR_NULL;
    if (h2o && !c.score_acc) return SQA_ERR_NULL;
    if (!aligned16(c.K) || !aligned16(c.V) || !aligned16(c.unit_state)) return SQA_ERR_SHAPE;
    if (c.budget < min_budget) return SQA_ERR_BUDGET;
    if (c.capacity < 1) return SQA_ERR_CAPACITY;
    if ((c.block_table != nullptr) != paged) return SQA_ERR_SHAPE;
    if (paged && (c.unit_offset || c.n_blocks < 1 || c.blocks_per_unit > SQA_MAX_BLOCKS_PER_UNIT ||
                  (int64_t)c.blocks_per_unit * SQA_BLOCK_SLOTS < (c.budget < c.capacity ? c.budget : c.capacity)))
      return SQA_ERR_SHAPE;
  }
  return plan_call(dt, B, Hq, Hkv, D, h2o, layers, n_layers, false, plan, lds_out);
}

static sqa_status decode_launch(sqa_dtype dt, const DecodePlan& plan, size_t lds, const DecodeScratch& sc,
                                const void* q, const void* k_new, const void* v_new,
                                int B, int Hq, int Hkv, int D, int32_t new_pos, sqa_policy policy, int n_sink,
                                const sqa_layer_cache* layers, const sqa_layer_cache* layers_dev, int n_layers,
                                void* out, hipStream_t st, const sqa_batch_opts* opts) {
  const int64_t kv_bytes = counted_kv_bytes(layers, n_layers, (int64_t)B * Hkv, 2 * D * (dt == SQA_F32 ? 4 : 2));
  const decode_fn fn = pick(dt, D, Hq / Hkv, policy == SQA_H2O, layers[0].block_table != nullptr, plan.waves, kv_bytes >= kLargeBytes);
  if (lds > 64 * 1024) SQA_HIP_CHECK(allow_dynamic_lds(reinterpret_cast<const void*>(fn), lds));
  DecodeArgs a;
  a.q = q; a.k_new = k_new; a.v_new = v_new; a.out = out;
  a.status = sc.status;
  a.cnt = sc.cnt;
  a.part = sc.part;
  a.logit = sc.logit;
  a.B = B; a.Hq = Hq; a.Hkv = Hkv; a.n_layers = n_layers;
  a.new_pos = new_pos; a.policy = (int)policy; a.n_sink = n_sink;
  a.new_pos_seq = opts ? opts->new_pos_seq : nullptr;
  a.budget_seq = opts ? opts->budget_seq : nullptr;
  a.ae = (opts && opts->order == SQA_ATTEND_THEN_EVICT) ? 1 : 0;
  a.lds_chunk = plan.lds_chunk;
  a.lds_chunk_w = plan.lds_chunk_w;
  a.scale_log2 = (float)(1.4426950408889634 / sqrt((double)D));
  memcpy(a.order, plan.order, (size_t)n_layers);
  uint64_t run = 0;
  for (int i = 0; i < n_layers; ++i) {
    const int l = a.order[i];
    run += plan.wpu[l] ? ((uint64_t)B * Hkv + kDecWaves - 1) / kDecWaves : (uint64_t)B * Hkv * plan.nsplit[l];
    a.blk_end[i] = (uint32_t)run;
    a.lay[i].nsplit = plan.nsplit[i] | (plan.wpu[i] ? kWpuBit : 0u) | ((uint32_t)plan.lds_tiles[i] << kLdsTilesShift);
    a.lay[i].chunk = plan.chunk[i];
    a.lay[i].unit_off = plan.unit_off[i];
    a.lay[i].part_off = plan.part_off[i];
    a.lay[i].logit_off = plan.logit_off[i];
  }
  a.wide_tail = plan.blocks <= (uint64_t)kWideTailMaxBlocks ? kSoloMaxTokens : (plan.blocks <= (uint64_t)kWideTailMidBlocks ? kSoloMaxTokensMid : 0);
  a.lds_probs_w = plan.lds_probs_w;
  a.tbl_off = (int)(lds - (size_t)plan.tbl_entries * sizeof(int));
  if (layers_dev) {
    a.layers = layers_dev;
  } else {
    SQA_HIP_CHECK(hipMemcpyAsync(sc.table, layers, (size_t)n_layers * sizeof(sqa_layer_cache), hipMemcpyHostToDevice, st));
    a.layers = reinterpret_cast<const sqa_layer_cache*>(sc.table);
  }
  fn<<<(unsigned)plan.blocks, plan.waves * SQA_WAVE, lds, st>>>(a);
  SQA_HIP_CHECK(hipGetLastError());
  return SQA_OK;
}

}  // namespace sqa

namespace sqa {
// The plan of a call from its shapes alone.
static sqa_status plan_shapes(const sqa_layer_cache* layers, int n_layers, int B, int Hq, int Hkv, int D, sqa_dtype dt,
                              sqa_policy policy, DecodePlan* plan, size_t* lds) {
  if (!layers) return SQA_ERR_NULL;
  if (dt != SQA_F32 && dt != SQA_BF16) return SQA_ERR_DTYPE;
  if (policy != SQA_SLIDING && policy != SQA_STREAMING && policy != SQA_H2O) return SQA_ERR_POLICY;
  if (B < 1 || Hq < 1 || Hkv < 1 || n_layers < 1 || n_layers > SQA_MAX_LAYERS || Hq % Hkv != 0) return SQA_ERR_SHAPE;
  const bool h2o = policy == SQA_H2O;
  if (!pick(dt, D, Hq / Hkv, h2o, layers[0].block_table != nullptr)) return SQA_ERR_SHAPE;
  return plan_call(dt, B, Hq, Hkv, D, h2o, layers, n_layers, false, plan, lds);
}
}  // namespace sqa

extern "C" int32_t sqa_decode_plan_waves(const sqa_layer_cache* layers, int n_layers, int B, int Hq, int Hkv, int D,
                                         sqa_dtype dt, sqa_policy policy) {
  sqa::DecodePlan plan;
  size_t lds = 0;
  return sqa::plan_shapes(layers, n_layers, B, Hq, Hkv, D, dt, policy, &plan, &lds) == SQA_OK ? plan.waves : 0;
}

extern "C" sqa_status sqa_decode_plan(const sqa_layer_cache* layers, int n_layers, int B, int Hq, int Hkv, int D,
                                      sqa_dtype dt, sqa_policy policy, sqa_decode_plan_info* info,
                                      sqa_decode_layer_plan* per_layer) {
  using namespace sqa;
  if (!info) return SQA_ERR_NULL;
  DecodePlan plan;
  size_t lds = 0;
  const sqa_status ps = plan_shapes(layers, n_layers, B, Hq, Hkv, D, dt, policy, &plan, &lds);
  if (ps != SQA_OK) return ps;
  info->workgroups = (int64_t)plan.blocks;
  info->workspace_bytes = (int64_t)plan.bytes;
  info->lds_bytes = (int32_t)lds;
  info->matrix_cores = uses_mfma(dt, D, Hq / Hkv) ? 1 : 0;
  info->wide_tail = plan.blocks <= (uint64_t)kWideTailMaxBlocks ? 1 : 0;
  info->table_entries = plan.tbl_entries;
  if (per_layer)
    for (int i = 0; i < n_layers; ++i) {
      per_layer[i].workgroups_per_unit = plan.wpu[i] ? 0 : plan.nsplit[i];
      per_layer[i].slots_per_workgroup = (int32_t)plan.chunk[i];
      per_layer[i].wave_per_unit = plan.wpu[i];
      per_layer[i].probs_in_lds = plan.probs_in_lds[i];
    }
  return SQA_OK;
}

extern "C" sqa_status sqa_decode_step_ex(const void* q, const void* k_new, const void* v_new, sqa_dtype dt,
                                         int B, int Hq, int Hkv, int D, int32_t new_pos,
                                         sqa_policy policy, int n_sink,
                                         const sqa_layer_cache* layers, const sqa_layer_cache* layers_dev, int n_layers,
                                         void* out, void* workspace, size_t ws_bytes, void* stream,
                                         const sqa_batch_opts* opts) {
  using namespace sqa;
  if (!workspace) return SQA_ERR_NULL;
  DecodePlan plan;
  size_t lds = 0;
  const sqa_status ps = decode_prepare(q, k_new, v_new, dt, B, Hq, Hkv, D, new_pos, policy, n_sink, layers, n_layers, out,
                                       opts, &plan, &lds);
  if (ps != SQA_OK) return ps;
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return SQA_ERR_SHAPE;
  if (ws_bytes < plan.bytes) {                     // less than sqa_decode_workspace_bytes: fewer pieces need less
    const sqa_status cs = plan_call(dt, B, Hq, Hkv, D, policy == SQA_H2O, layers, n_layers, true, &plan, &lds);
    if (cs != SQA_OK) return cs;
    if (ws_bytes < plan.bytes) return SQA_ERR_CAPACITY;
  }
  char* ws = static_cast<char*>(workspace);
  DecodeScratch sc;
  sc.status = reinterpret_cast<int32_t*>(ws);
  sc.table = ws + plan.off_table;
  sc.cnt = reinterpret_cast<int32_t*>(ws + plan.off_cnt);
  sc.part = reinterpret_cast<float*>(ws + plan.off_part);
  sc.logit = reinterpret_cast<float*>(ws + plan.off_logit);
  return decode_launch(dt, plan, lds, sc, q, k_new, v_new, B, Hq, Hkv, D, new_pos, policy, n_sink, layers, layers_dev,
                       n_layers, out, static_cast<hipStream_t>(stream), opts);
}

// ---- the same step for callers that cannot allocate -------------------------------------------------
// The scratch a decode step needs lives in a file-scope device array instead of a caller's workspace.
// Fixed layout (so that a region only ever holds one kind of data, whatever the shapes of successive
// calls): layer table | arrival counters | partial records and H2O logits / probabilities.
// The counters are the only words that must be zero when a kernel starts.  Their region holds nothing
// else, is cleared once per device at set-up, and every launch returns the counters it used to zero
// (the workgroup that merges a split unit resets the unit's counter), so each call finds them zero
// although the array keeps the previous call's contents everywhere else.
static __device__ __align__(256) unsigned char scratch[SQA_STATIC_SCRATCH_BYTES];

namespace sqa {
constexpr int kMaxDevices = 64;
// Device address of `scratch` on each device (every GPU holds its own copy of the array at its own
// address; in host code the array's name is only a handle for this lookup, never an address).
static sqa_status static_scratch_base(hipStream_t st, char** base_out) {
  static std::mutex mu;
  static char* base[kMaxDevices] = {};
  int dev = -1;
  SQA_HIP_CHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return SQA_ERR_CAPACITY;
  std::lock_guard<std::mutex> lock(mu);
  if (!base[dev]) {
    char* p = nullptr;
    SQA_HIP_CHECK(hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch)));
    if (!p || (reinterpret_cast<uintptr_t>(p) & 255u)) return SQA_ERR_HIP;
    // once per device: the counter region starts at zero (fill kernel, then wait, so that the set-up
    // is complete whatever stream later calls use)
    const sqa_status zs = zero_fill(p + kStaticTableBytes, kStaticCntBytes, st);
    if (zs != SQA_OK) return zs;
    SQA_HIP_CHECK(hipStreamSynchronize(st));
    base[dev] = p;
  }
  *base_out = base[dev];
  return SQA_OK;
}
}  // namespace sqa

extern "C" sqa_status sqa_decode_step_static(const void* q, const void* k_new, const void* v_new, sqa_dtype dt,
                                             int B, int Hq, int Hkv, int D, int32_t new_pos,
                                             sqa_policy policy, int n_sink,
                                             const sqa_layer_cache* layers, const sqa_layer_cache* layers_dev,
                                             int n_layers, void* out, int32_t* status, void* stream,
                                             const sqa_batch_opts* opts) {
  using namespace sqa;
  if (!status) return SQA_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(status) & 3u) return SQA_ERR_SHAPE;
  DecodePlan plan;
  size_t lds = 0;
  const sqa_status ps = decode_prepare(q, k_new, v_new, dt, B, Hq, Hkv, D, new_pos, policy, n_sink, layers, n_layers, out,
                                       opts, &plan, &lds);
  if (ps != SQA_OK) return ps;
  // beyond the array's fixed size: refused, nothing is enqueued (use sqa_decode_step with a workspace)
  if (!fits_static(plan)) return SQA_ERR_CAPACITY;
  const size_t part_bytes = align256(plan.part_bytes);
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* base = nullptr;
  const sqa_status bs = static_scratch_base(st, &base);
  if (bs != SQA_OK) return bs;
  DecodeScratch sc;
  sc.status = status;
  sc.table = base;
  sc.cnt = reinterpret_cast<int32_t*>(base + kStaticTableBytes);
  sc.part = reinterpret_cast<float*>(base + kStaticTableBytes + kStaticCntBytes);
  sc.logit = reinterpret_cast<float*>(base + kStaticTableBytes + kStaticCntBytes + part_bytes);
  return decode_launch(dt, plan, lds, sc, q, k_new, v_new, B, Hq, Hkv, D, new_pos, policy, n_sink, layers, layers_dev,
                       n_layers, out, st, opts);
}

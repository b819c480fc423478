// H2O's accumulated attention over the prompt (Sec. 5.1 "Heavy-Hitter"): column
// sums of the causal softmax(Q K^T / sqrt(D)), added over the g query heads that
// share a KV head.  This is the producer of sqa_prefill_compress's attn_scores.
//
// The causal logits are computed on the matrix cores; the P x P probabilities never
// reach HBM and every sum has a fixed order (LDS atomics have one writer per key and stripe).  Two ways:
//   one pass (score_stripes): a workgroup keeps the exponentials of a stripe of query
//           rows in registers until their sums are known; what most calls use;
//   two passes, for prompts of more than 4096 tokens, where they are the cheaper way
//           (many short prompts, bf16 at D = 64 with many heads: see StripeCut), and (the
//           second alone) normalisers that the caller has:
//   pass 1  row statistics of every query row: a reference m_i and the sum of
//           exp2(s - m_i), stored as m_i and 1 / l_i;
//   pass 2  per key, sum of exp2(s - m_i) / l_i over its KV head's query rows.
//   The contraction of a 16x16 block of logits over 16 bytes of each row:
//   bf16  v_mfma_f32_16x16x32_bf16: A row / B column = lane%16, contraction slots
//         of a lane = 8*(lane/16)+e;
//   fp32  four v_mfma_f32_16x16x4_f32 (fp32 multiply-adds, 256 flop per cycle and
//         CU: twice what the vector ALUs do without packed instructions), one slot
//         per lane group;
//   C column = lane%16, rows 4*(lane/16)+i in both.  For both operands a lane of
//   group j takes the 16-byte pieces NP*j .. NP*j + NP-1 of its row (NP = row bytes
//   / 64), so a lane's fragments are contiguous bytes.
//   pass 1  S^T = K.Q^T: a wave keeps NB blocks of 16 query rows as B operands
//           in registers (block b of wave w = rows 16 (w + 4 b) of the
//           workgroup's 64 NB rows, so the diagonal's work is spread evenly);
//           64-key tiles of K go from global memory straight into LDS (direct
//           loads, no register staging; 16-byte pieces XOR-swizzled by the row;
//           two buffers) and are shared by the 4 waves.  Every fragment read
//           from LDS feeds NB products.  A lane sees 4 keys of one query per
//           product and keeps a running (reference, sum) of its own; the 4
//           lanes of a query merge once at the end.
//   pass 2  S = Q.K^T: a wave keeps NB blocks of 16 keys as B operands; 64-row
//           tiles of Q and their m_i, 1/l_i are staged in LDS the same way; a lane
//           sees 4 query rows of one key per product and adds exp2(s - m_i) / l_i
//           into a per-lane column sum over all row tiles and all g heads.
// What bounds the two passes.  bf16, D = 128: per 16x16 block a lane issues 4 products (64
// cycles of the matrix pipeline) and at least 4 x (multiply-add, exp2, add); on this
// chip vector instructions hide only partly behind matrix instructions of the same
// SIMD (measured: 16 products + 16 such triples take 201 ns with 4 waves per SIMD,
// 119 and 109 ns on their own), and the clock falls while it runs, so every vector
// instruction beside them counts: 0.335 ms for both passes of 8 x 32 heads x 2048
// tokens, 820 TFLOP/s (0.353 with 24 more address instructions per tile and, in pass
// 2, no tile fetched ahead).  bf16, D = 64: the vector instructions (4 x 32 heads x
// 1024 tokens 432 -> 58 us from fp32 multiply-adds on the vector ALUs).  fp32: the
// products, 512 or 1024 cycles per block (64 heads over 8, D = 128, 1289 tokens
// 2325 -> 326 us, 84 of 157 TFLOP/s; 16 over 8, D = 64, prompts up to 777 183 -> 62).
// NB = 2 in bf16 (with 1, LDS reads: 447 against 355 us), 1 in fp32 (finer grid,
// the same rate).  Blocks of 32x32 with the exponentials issued between the products
// reach 150 ns per 16 + 16 on their own, but need 2 waves per SIMD and came out at
// 397-419 us here.
#include "sqa_common.h"
#include <type_traits>

namespace sqa {

constexpr int kScThreads = 256;

// Which (tile, head) a workgroup of a 1-D launch works on.  Consecutive workgroups go to the 8 XCDs of the
// chip in turn, each with an L2 of its own; all tiles of a head re-read that head's K (or Q) rows, so a head
// (with the `per` query heads that share its K rows) is given to one XCD (group mod 8) and an XCD walks its
// groups one after the other, the tile with the most work first: the rows are then fetched into one L2 once
// instead of into all eight.  Measured at the 7B shape: 0.45 -> 0.30 ms and 0.54 -> 0.35 ms per layer.
__device__ __forceinline__ bool xcd_tile_head(int tiles, int heads, int per, bool heavy_is_last, int& tile, int& head) {
  const int n = blockIdx.x, xcd = n & 7, slot = n >> 3;
  const int group = (slot / (tiles * per)) * 8 + xcd, rem = slot % (tiles * per);
  head = group * per + rem / tiles;
  const int t = rem % tiles;
  tile = heavy_is_last ? tiles - 1 - t : t;
  return head < heads;
}

typedef __bf16 sc_bf16x8_t __attribute__((ext_vector_type(8)));
typedef float sc_f32x4_t __attribute__((ext_vector_type(4)));
constexpr int kMT = 64;                 // rows of a staged tile
constexpr float kRefFar = 65536.f;      // a row's reference moves when 4 exponentials against it add up to this
constexpr float kLog2e = 1.4426950408889634f;

// Direct global -> LDS copies, `lds` + 16 (or 4) bytes x lane <- *g of each lane.  Written as instructions rather
// than with the builtin because the compiler, which cannot see that the two buffers of a tile loop are different
// ones, otherwise waits for the NEXT tile's copy (vmcnt 0) before the first read of the present one, and nothing
// is fetched ahead.  Whoever reads what was copied waits for it: s_waitcnt vmcnt(0), then the workgroup barrier.
typedef __attribute__((address_space(3))) const char sc_lds_t;
__device__ __forceinline__ uint32_t lds_offset(const char* p) { return (uint32_t)(uintptr_t)(sc_lds_t*)p; }
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // (m0 is named as clobbered although the compiler never allocates it: nothing else here uses it)
__device__ __forceinline__ void copy16_to_lds(const void* g, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(g), "s"(lds) : "m0", "memory");
}
__device__ __forceinline__ void copy16_to_lds(const void* base /*uniform*/, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(off), "s"(base), "s"(lds) : "m0", "memory");
}
__device__ __forceinline__ void copy4_to_lds(const void* g, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" :: "v"(g), "s"(lds) : "m0", "memory");
}
#pragma clang diagnostic pop

// Rows of D elements in 16-byte pieces, as they are staged in LDS (RB bytes per row, no padding).  Piece c of
// row R lies at piece at(R, c): a fragment read takes one piece of each of 16 rows, and with this order those
// 16 pieces lie in 16 different 16-byte columns of the 64 banks, whatever c (two 128-byte rows share a line of
// the banks, a 512-byte row fills two).
template <typename T, int D> struct Rows {
  static constexpr int RB = D * (int)sizeof(T);
  static constexpr int PPR = RB / 16;             // pieces per row: 8, 16 or 32
  static constexpr int NP = PPR / 4;              // pieces of a row that one lane holds
  static constexpr int TILE = kMT * RB;
  static constexpr int RPI = 1024 / RB;           // rows per 1 KB wave instruction
  static __device__ __forceinline__ int at(int row, int piece) {
    return PPR == 8 ? piece ^ ((row >> 1) & 7) : piece ^ (row & 15);
  }
  // Copies 64-row tiles (rows row0.., clamped to P-1) straight into LDS: each wave instruction fills 1 KB in lane
  // order, so a lane fetches the piece that belongs at its position (the permutation stays inside a row: the access
  // is still coalesced).  A lane's place is worked out once; a tile costs scalar additions only, except the last.
  struct Copier {
    uint32_t off[2];                              // row and piece of this lane in a wave's even / odd instructions
    __device__ __forceinline__ Copier() {
      const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int r = wave * RPI + lane / PPR;
        off[k] = r * RB + at(r + 4 * k * RPI, lane % PPR) * 16;    // (at() has period 8 RPI in the row, or a divisor of it)
      }
    }
    __device__ __forceinline__ void operator()(const T* __restrict__ src, int row0, int P, char* lds) const {
      const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
      const char* base = reinterpret_cast<const char*>(src) + (int64_t)row0 * RB;
      const uint32_t dst = lds_offset(lds) + wave * 1024;
      if (row0 + kMT <= P) {
#pragma unroll
        for (int i = 0; i < kMT / RPI / 4; ++i) copy16_to_lds(base + 4 * i * RPI * RB, off[i & 1], dst + 4096 * i);
      } else {                                    // rows beyond the end: the last one again
#pragma unroll
        for (int i = 0; i < kMT / RPI / 4; ++i) {
          const int past = max(row0 + 4 * i * RPI + (int)(off[i & 1] / RB) - (P - 1), 0);
          copy16_to_lds(base + 4 * i * RPI * RB + off[i & 1] - (int64_t)past * RB, dst + 4096 * i);
        }
      }
    }
  };
  // The same for a workgroup of NW waves and ROWS rows (rows beyond `last`: that one again).
  template <int ROWS, int NW> static __device__ __forceinline__ void stage(const T* __restrict__ src, int row0, int last, char* lds) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t dst = lds_offset(lds);
#pragma unroll
    for (int i = wave; i < ROWS / RPI; i += NW) {
      const int r = i * RPI + lane / PPR;
      copy16_to_lds(reinterpret_cast<const char*>(src) + (int64_t)min(row0 + r, last) * RB + at(r, lane % PPR) * 16, dst + 1024 * i);
    }
  }
  // the fragments of row `row` (global memory) for a lane of contraction group j
  static __device__ __forceinline__ void row_fragments(const T* __restrict__ src, int row, int j, uint4 (&fr)[NP]) {
#pragma unroll
    for (int i = 0; i < NP; ++i) fr[i] = ld16(reinterpret_cast<const char*>(src) + (int64_t)row * RB + (NP * j + i) * 16);
  }
  // Has the fragments arrive here (the compiler does not see the copies above in its count of outstanding loads, so
  // a fragment first used inside a tile loop would have it wait there, trip after trip, for the copy of the next tile).
  static __device__ __forceinline__ void arrive(uint4 (&fr)[NP]) {
#pragma unroll
    for (int i = 0; i < NP; ++i) asm volatile("" : "+v"(fr[i].x), "+v"(fr[i].y), "+v"(fr[i].z), "+v"(fr[i].w));
  }
  // the A fragments of rows 16 sub .. 16 sub + 15 of a staged tile
  static __device__ __forceinline__ void tile_fragments(const char* lds, int sub, uint4 (&fr)[NP]) {
    const int lane = threadIdx.x & 63, row = 16 * sub + (lane & 15);
#pragma unroll
    for (int i = 0; i < NP; ++i) fr[i] = *reinterpret_cast<const uint4*>(lds + row * RB + at(row, NP * (lane >> 4) + i) * 16);
  }
  static __device__ __forceinline__ sc_f32x4_t block_product(const uint4 (&a)[NP], const uint4 (&b)[NP]) {
    sc_f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      if constexpr (sizeof(T) == 2) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(sc_bf16x8_t, a[i]), __builtin_bit_cast(sc_bf16x8_t, b[i]), c, 0, 0, 0);
      } else {
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i].x), __uint_as_float(b[i].x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i].y), __uint_as_float(b[i].y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i].z), __uint_as_float(b[i].z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i].w), __uint_as_float(b[i].w), c, 0, 0, 0);
      }
    }
    return c;
  }
  // the same for NB blocks side by side: a product does not wait for the one before it
  template <int NB> static __device__ __forceinline__ void block_products(const uint4 (&a)[NP], const uint4 (&b)[NB][NP], sc_f32x4_t (&c)[NB]) {
#pragma unroll
    for (int bb = 0; bb < NB; ++bb) c[bb] = sc_f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int bb = 0; bb < NB; ++bb)
          c[bb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(sc_bf16x8_t, a[i]), __builtin_bit_cast(sc_bf16x8_t, b[bb][i]), c[bb], 0, 0, 0);
      } else {
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) c[bb] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i].x), __uint_as_float(b[bb][i].x), c[bb], 0, 0, 0);
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) c[bb] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i].y), __uint_as_float(b[bb][i].y), c[bb], 0, 0, 0);
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) c[bb] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i].z), __uint_as_float(b[bb][i].z), c[bb], 0, 0, 0);
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) c[bb] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i].w), __uint_as_float(b[bb][i].w), c[bb], 0, 0, 0);
      }
    }
  }
};

// bf16 at D = 128 keeps one value per row, c_i = m_i + log2(l_i), instead of the pair: the second pass is bound by
// its vector instructions and LDS reads there (0.190 against 0.201 ms per pass at the 7B shape), and the rounding of
// c_i (2e-7 of a score) is far below that of the inputs.
template <typename T, int D> constexpr bool kMerged = sizeof(T) == 2 && D == 128;

struct ScoreArgs {
  const void* Q;
  const void* K;
  int B, Hq, Hkv, P;
  float scale_log2;
  const int32_t* prompt_len;    // [B] or NULL: queries beyond a sequence's own prompt are padding
  float* ref;                   // [B*Hq][P] m_i in the exp2 domain (pass 2 with given normalisers: ln of them, read only)
  float* inv;                   // [B*Hq][P] 1 / l_i
  float* out;                   // pass 2: [B*Hkv][P] scores, or [B*Hq][P] one partial sum per query head
  int chunks;                   // one pass: workgroups (and partial sums) per query head
};

template <int I, typename F> __device__ __forceinline__ void for_down(F& f) {      // f(I), f(I - 1), ... f(0) with constants
  f(std::integral_constant<int, I>{});
  if constexpr (I > 0) for_down<I - 1>(f);
}

template <typename T, int D, int NB>
__device__ __forceinline__ void score_rowstats(const ScoreArgs& a, char* s_tiles /*2 tiles*/) {
  using R = Rows<T, D>;
  constexpr int OWN = kMT * NB;                     // query rows of a workgroup
  const int P = a.P, Hq = a.Hq, Hkv = a.Hkv;
  const float scale_log2 = a.scale_log2;
  int tile_x, bh;
  if (!xcd_tile_head((P + OWN - 1) / OWN, a.B * Hq, Hq / Hkv, true, tile_x, bh)) return;   // (query tile t reads key tiles 0..t: the last is the longest)
  const int b = bh / Hq, h = bh % Hq, kvh = h / (Hq / Hkv);
  const int Pq = a.prompt_len ? max(0, min(a.prompt_len[b], P)) : P;
  if (tile_x * OWN >= Pq) return;                   // nobody asks for the statistics of padding rows
  const T* Qh = static_cast<const T*>(a.Q) + (int64_t)bh * P * D;
  const T* Kh = static_cast<const T*>(a.K) + ((int64_t)b * Hkv + kvh) * P * D;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n16 = lane & 15, j4 = lane >> 4;
  const int r0 = tile_x * OWN + 16 * wave;          // first row of own block 0; block bb starts at r0 + 64 bb
  uint4 qfr[NB][R::NP];
  float m_run[NB], l_run[NB];
#pragma unroll
  for (int bb = 0; bb < NB; ++bb) {
    R::row_fragments(Qh, min(r0 + 64 * bb + n16, P - 1), j4, qfr[bb]);
    m_run[bb] = -INFINITY; l_run[bb] = 0.f;
  }
  const typename R::Copier tile_to_lds;
  tile_to_lds(Kh, 0, P, s_tiles);
#pragma unroll
  for (int bb = 0; bb < NB; ++bb) R::arrive(qfr[bb]);
  const int n_tiles = (min((tile_x + 1) * OWN, Pq) - 1) / kMT + 1;   // key tiles 0 .. the one holding the last row
  for (int kt = 0; kt < n_tiles; ++kt) {
    char* buf = s_tiles + (kt & 1) * R::TILE;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's part of tile kt has landed
    __syncthreads();                                // tile kt visible; everyone is past tile kt-1
    if (kt + 1 < n_tiles) tile_to_lds(Kh, (kt + 1) * kMT, P, s_tiles + ((kt + 1) & 1) * R::TILE);
    if ((kt + 1) * kMT - 1 <= r0 && (kt + 1) * kMT <= P) {
      // Every key of the tile is visible to every row of this wave (wave-uniform test, block 0 has the
      // lowest rows; true for all tiles but those on the diagonal): no mask.  The exponentials are taken
      // against the row's current reference without looking for the maximum first; only when a partial
      // sum shows that a logit lies far above the reference (or there is no reference yet: the sum is then
      // infinite) does the wave redo the 16 keys with the reference moved.  After the first tiles that is
      // rare, and the common case costs one comparison per block instead of a maximum per element.
#pragma unroll
      for (int sub = 0; sub < 4; ++sub) {
        uint4 afr[R::NP];
        R::tile_fragments(buf, sub, afr);
        sc_f32x4_t s4[NB];
        float part[NB];
        bool far = false;
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) {
          s4[bb] = R::block_product(afr, qfr[bb]);
          const float e0 = __builtin_amdgcn_exp2f(fmaf(s4[bb][0], scale_log2, -m_run[bb]));
          const float e1 = __builtin_amdgcn_exp2f(fmaf(s4[bb][1], scale_log2, -m_run[bb]));
          const float e2 = __builtin_amdgcn_exp2f(fmaf(s4[bb][2], scale_log2, -m_run[bb]));
          const float e3 = __builtin_amdgcn_exp2f(fmaf(s4[bb][3], scale_log2, -m_run[bb]));
          part[bb] = (e0 + e1) + (e2 + e3);
          far |= !(part[bb] < kRefFar);
        }
        if (__builtin_amdgcn_ballot_w64(far)) {
#pragma unroll
          for (int bb = 0; bb < NB; ++bb) {
            const float top = fmaxf(fmaxf(s4[bb][0], s4[bb][1]), fmaxf(s4[bb][2], s4[bb][3])) * scale_log2;
            const float mx = fmaxf(m_run[bb], top);
            const float ms = mx == -INFINITY ? 0.f : mx;       // (nothing but logits of -inf so far)
            l_run[bb] *= __builtin_amdgcn_exp2f(m_run[bb] - ms);
            m_run[bb] = mx;
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) sum += __builtin_amdgcn_exp2f(fmaf(s4[bb][e], scale_log2, -ms));
            part[bb] = sum;
          }
        }
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) l_run[bb] += part[bb];
      }
      continue;
    }
#pragma unroll
    for (int sub = 0; sub < 4; ++sub) {
      const int c0 = kt * kMT + 16 * sub;
      if (c0 > r0 + 64 * (NB - 1) + 15 || c0 >= P) continue;   // wave-uniform: beyond all rows of this wave
      uint4 afr[R::NP];
      R::tile_fragments(buf, sub, afr);
#pragma unroll
      for (int bb = 0; bb < NB; ++bb) {
        const int rb = r0 + 64 * bb, my_row = rb + n16;
        if (c0 > rb + 15) continue;                 // wave-uniform: all keys beyond all rows of the block
        const sc_f32x4_t s4 = R::block_product(afr, qfr[bb]);
        float v[4], mx = m_run[bb];
        if (c0 + 15 <= rb && c0 + 16 <= P) {        // wave-uniform: the whole block is visible, only its neighbours are not
#pragma unroll
          for (int e = 0; e < 4; ++e) { v[e] = s4[e] * scale_log2; mx = fmaxf(mx, v[e]); }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int key = c0 + 4 * j4 + e;
            v[e] = (key <= my_row && key < P) ? s4[e] * scale_log2 : -INFINITY;
            mx = fmaxf(mx, v[e]);
          }
        }
        const float ms = mx == -INFINITY ? 0.f : mx;
        float sum = l_run[bb] * __builtin_amdgcn_exp2f(m_run[bb] - ms);
#pragma unroll
        for (int e = 0; e < 4; ++e) sum += __builtin_amdgcn_exp2f(v[e] - ms);
        l_run[bb] = sum; m_run[bb] = mx;
      }
    }
  }
  // the 4 lanes of a query row (contraction groups) merge their statistics
#pragma unroll
  for (int bb = 0; bb < NB; ++bb) {
    float m = m_run[bb], l = l_run[bb];
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) {
      const float mo = __shfl_xor(m, o, 64), lo = __shfl_xor(l, o, 64);
      const float mx = fmaxf(m, mo);
      const float ms = mx == -INFINITY ? 0.f : mx;
      l = l * __builtin_amdgcn_exp2f(m - ms) + lo * __builtin_amdgcn_exp2f(mo - ms);
      m = mx;
    }
    const int my_row = r0 + 64 * bb + n16;
    if (j4 == 0 && my_row < P) {
      if constexpr (kMerged<T, D>) {
        a.ref[(int64_t)bh * P + my_row] = m + __builtin_amdgcn_logf(l);
      } else {
        a.ref[(int64_t)bh * P + my_row] = m;
        a.inv[(int64_t)bh * P + my_row] = 1.f / l;
      }
    }
  }
}

// LSE: the caller's normalisers (natural logarithms) take the place of pass 1.
// SPLIT: a workgroup per (64 NB keys, query head) instead of per (64 NB keys, KV head); out holds one partial
// sum per query head, which sum_heads_kernel adds up.
template <typename T, int D, int NB, bool LSE, bool SPLIT>
__device__ __forceinline__ void score_colsum(const ScoreArgs& a, char* s_tiles /*2 x (tile, 64 m_i, 64 1/l_i)*/) {
  using R = Rows<T, D>;
  constexpr int BUF = R::TILE + 2 * kMT * (int)sizeof(float);
  constexpr int OWN = kMT * NB;                     // keys of a workgroup
  constexpr bool PAIR = !LSE && !kMerged<T, D>;     // a row's statistics are two values
  const int P = a.P, Hq = a.Hq, Hkv = a.Hkv, g = Hq / Hkv;
  const float scale_log2 = a.scale_log2;
  int tile_x, head;
  if (!xcd_tile_head((P + OWN - 1) / OWN, SPLIT ? a.B * Hq : a.B * Hkv, SPLIT ? g : 1, false, tile_x, head)) return;  // (key tile t is read by query tiles t..last: the first is the longest)
  const int bk = SPLIT ? head / g : head, b = bk / Hkv;            // (query heads of a KV head are consecutive)
  const int64_t bh0 = SPLIT ? head : (int64_t)bk * g;              // first query head of this workgroup
  const T* Kh = static_cast<const T*>(a.K) + (int64_t)bk * P * D;
  const T* Qall = static_cast<const T*>(a.Q);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n16 = lane & 15, j4 = lane >> 4;
  const int Pq = a.prompt_len ? max(0, min(a.prompt_len[b], P)) : P;   // queries beyond the sequence's own prompt are padding
  const int k0 = tile_x * OWN + 16 * wave;          // first key of own block 0; block bb starts at k0 + 64 bb
  uint4 kfr[NB][R::NP];
  float colsum[NB];
#pragma unroll
  for (int bb = 0; bb < NB; ++bb) {
    R::row_fragments(Kh, min(k0 + 64 * bb + n16, P - 1), j4, kfr[bb]);
    colsum[bb] = 0.f;
  }
  const int first = tile_x * NB, n_rt = (Pq + kMT - 1) / kMT;      // row tiles first .. n_rt - 1 see these keys
  const int per_head = max(n_rt - first, 0);
  const int total = (SPLIT ? 1 : g) * per_head;     // (head, row tile) pairs, head-major
  int req_h = 0, req_rt = first, req_n = 0;         // the next (head, row tile) to request, requests so far
  const typename R::Copier tile_to_lds;
  auto request = [&]() {
    const int64_t bh = bh0 + req_h;
    char* dst = s_tiles + (req_n++ & 1) * BUF;
    tile_to_lds(Qall + bh * P * D, req_rt * kMT, P, dst);
    if (wave < (PAIR ? 2 : 1)) {                     // the statistics of the tile's rows, 4 bytes per lane
      const float* src = wave == 0 ? a.ref : a.inv;
      copy4_to_lds(src + bh * P + min(req_rt * kMT + lane, P - 1), lds_offset(dst) + R::TILE + wave * kMT * 4);
    }
    if (++req_rt == n_rt) { req_rt = first; ++req_h; }
  };
  if (total > 0) request();
#pragma unroll
  for (int bb = 0; bb < NB; ++bb) R::arrive(kfr[bb]);
  int rt = first - 1;
  for (int it = 0; it < total; ++it) {
    char* buf = s_tiles + (it & 1) * BUF;
    const float* st_lds = reinterpret_cast<const float*>(buf + R::TILE);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's part of tile `it` has landed
    __syncthreads();                                // tile `it` visible; everyone is past tile it-1
    if (it + 1 < total) request();
    if (++rt == n_rt) rt = first;
    float tsum[NB];                                 // this tile's share first: short chains of additions round less
#pragma unroll                                        // (not where the additions are what bounds the pass)
    for (int bb = 0; bb < NB; ++bb) tsum[bb] = kMerged<T, D> ? colsum[bb] : 0.f;
    auto add_tile = [&](auto whole_tag) {
      constexpr bool whole = decltype(whole_tag)::value;
#pragma unroll
      for (int sub = 0; sub < 4; ++sub) {
        const int i0 = rt * kMT + 16 * sub;
        if (!whole && (i0 + 15 < k0 || i0 >= Pq)) continue;   // wave-uniform: all rows above all of this wave's keys, or padding
        uint4 afr[R::NP];
        R::tile_fragments(buf, sub, afr);
        // rows 4 j4 .. 4 j4 + 3 of the 16
        const float4 m4 = *reinterpret_cast<const float4*>(&st_lds[16 * sub + 4 * j4]);
        float4 i4 = make_float4(1.f, 1.f, 1.f, 1.f);
        if constexpr (PAIR) i4 = *reinterpret_cast<const float4*>(&st_lds[kMT + 16 * sub + 4 * j4]);
        const float mul = LSE ? kLog2e : 1.f;
        const float mrow[4] = {m4.x * mul, m4.y * mul, m4.z * mul, m4.w * mul}, irow[4] = {i4.x, i4.y, i4.z, i4.w};
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) {
          const int kb = k0 + 64 * bb, my_key = kb + n16;
          if (!whole && i0 + 15 < kb) continue;     // wave-uniform: all rows above all keys of the block
          const sc_f32x4_t s4 = R::block_product(afr, kfr[bb]);
          if (whole || (i0 >= kb + 15 && i0 + 16 <= Pq)) {    // wave-uniform: every row of the block sees every key of it
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float p = __builtin_amdgcn_exp2f(fmaf(s4[e], scale_log2, -mrow[e]));
              tsum[bb] = PAIR ? fmaf(p, irow[e], tsum[bb]) : tsum[bb] + p;
            }
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int row = i0 + 4 * j4 + e;
              const float p = __builtin_amdgcn_exp2f(fmaf(s4[e], scale_log2, -mrow[e])) * (PAIR ? irow[e] : 1.f);
              tsum[bb] += (row >= my_key && row < Pq) ? p : 0.f;
            }
          }
        }
      }
    };
    // every row of the tile sees every key of this wave and is a real query (wave-uniform; all tiles but those
    // on the diagonal and the last): no mask
    if (rt * kMT >= k0 + 64 * (NB - 1) + 15 && (rt + 1) * kMT <= Pq) add_tile(std::true_type{});
    else add_tile(std::false_type{});
#pragma unroll
    for (int bb = 0; bb < NB; ++bb) colsum[bb] = kMerged<T, D> ? tsum[bb] : colsum[bb] + tsum[bb];
  }
#pragma unroll
  for (int bb = 0; bb < NB; ++bb) {
    float c = colsum[bb];
    c += __shfl_xor(c, 16, 64);
    c += __shfl_xor(c, 32, 64);
    const int my_key = k0 + 64 * bb + n16;
    if (j4 == 0 && my_key < P) a.out[(int64_t)head * P + my_key] = c;
  }
}

// ---- both passes in one -------------------------------------------------------------------------------------
// A workgroup takes stripes of 16 NB query rows.  The keys a stripe sees are dealt to the waves in blocks of 16, the
// last block first (block nkb-1 to wave 0, nkb-2 to wave 1, ...: the waves differ by at most one block and the masked
// blocks on the diagonal lie in slot 0).  A wave computes S^T = K.Q^T block by block and KEEPS exp2(s - m) of its last
// SLOTS blocks in registers (m: a reference per lane and row that moves only when a sum shows it is far too low), so
// that after the waves have put their row sums together the column sums cost one multiply-add per element instead of
// the products and exponentials once more.  Keys further back than NW x SLOTS blocks are taken twice, as in two passes.
// A workgroup adds its stripes' column sums up in LDS and writes one partial row; sum_heads_kernel adds those.
// What bounds it: vector and matrix instructions of two waves per SIMD (the registers allow no more), which on this
// chip share their time rather than overlap (bf16, D = 128: 606 cycles per block of 16 keys and 64 rows with another
// wave's beside it, 256 of them products, 292 exponentials and sums; products 26 %, vector instructions 59 % of the time
// at 256 heads of 2048 tokens, 8 waves), hence the fewest possible of both.  In fp32 the products (2 x 1024 cycles per block at
// D = 128).  bf16 key blocks come through a ring in LDS, one ahead and across stripes (loaded into registers one ahead:
// 381 us at 256 heads of 2048 tokens, 8 waves; 247 with no loads at all; 290 through the ring).  Two passes -> one, us:
//   bf16, D = 128   256 heads of 2048 tokens  330 -> 290;  of 1024  115 -> 82;  of 512  43 -> 28;  64 of 1024  47 -> 26
//   bf16, D = 64    256 of 1024  94 -> 65;  16 of 2048  54 -> 23;  fp32, D = 64  ragged up to 777, 64 heads  63 -> 30
//   fp32, D = 128   64 of 1289  322 -> 148;  256 of 512  249 -> 98
// Rows of fp32 are half as many per stripe, so that registers hold twice the keys.
template <typename T, int D> struct Stripe;                        // NB row blocks, SLOTS key blocks kept per wave, RING key blocks in LDS
template <> struct Stripe<bf16_t, 128> { static constexpr int NB = 4, SLOTS = 8, RING = 2; };
template <> struct Stripe<bf16_t, 64> { static constexpr int NB = 4, SLOTS = 8, RING = 2; };
template <> struct Stripe<float, 64> { static constexpr int NB = 2, SLOTS = 16, RING = 0; };
template <> struct Stripe<float, 128> { static constexpr int NB = 2, SLOTS = 14, RING = 0; };
constexpr float kNoRef = 3.402823466e+38f;                         // minus the reference of a lane that has none yet

template <int CTRL> __device__ __forceinline__ float sc_dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

template <typename T, int D, int NB, int SLOTS, int RING, int NW>
__device__ __forceinline__ void score_stripes(const ScoreArgs& a, char* lds) {
  using R = Rows<T, D>;
  constexpr int OWN = 16 * NB, QB = OWN * R::RB;
  static_assert(NB == 2 || NB == 4, "rows of a stripe");
  static_assert(NB <= NW, "the blocks on the diagonal lie in slot 0");
  const int P = a.P, Hq = a.Hq, Hkv = a.Hkv, nch = a.chunks;
  const float scale_log2 = a.scale_log2;
  int chunk, bh;
  if (!xcd_tile_head(nch, a.B * Hq, Hq / Hkv, false, chunk, bh)) return;
  const int b = bh / Hq, kvh = (bh % Hq) / (Hq / Hkv);
  const int Pq = a.prompt_len ? max(0, min(a.prompt_len[b], P)) : P;
  const T* Qh = static_cast<const T*>(a.Q) + (int64_t)bh * P * D;
  const char* Kh = reinterpret_cast<const char*>(static_cast<const T*>(a.K) + ((int64_t)b * Hkv + kvh) * P * D);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n16 = lane & 15, j4 = lane >> 4;
  constexpr int KB = 16 * R::RB;                                   // bytes of a key block
  char* const s_ring = lds + QB + wave * RING * KB;                // this wave's key blocks on their way
  float2* const s_st = reinterpret_cast<float2*>(lds + QB + NW * RING * KB);       // [NW][OWN] (reference, sum) of a wave's keys
  float* const s_col = reinterpret_cast<float*>(lds + QB + NW * RING * KB + NW * OWN * 8);     // [P rounded up to 16]
  for (int i = tid; i < P + 15; i += 64 * NW) s_col[i] = 0.f;

  // the workgroup's stripes, longest first, dealt to a head's workgroups back and forth
  const int n_str = (Pq + OWN - 1) / OWN;
  auto stripe_at = [&](int k) { return n_str - 1 - (k * nch + ((k & 1) ? nch - 1 - chunk : chunk)); };
  int st = stripe_at(0);
  if (st >= 0) R::template stage<OWN, NW>(Qh, st * OWN, Pq - 1, lds);
  // A wave's key blocks of stripe `of`: from..to in steps of NW (to < 0: none)
  auto last_block = [&](int of) { return (min((of + 1) * OWN, Pq) + 15) / 16 - 1 - wave; };
  // The ring is filled in the order in which the blocks are used, across stripes (at the end: the last one again, so
  // that the number of copies in flight stays the same).  What happens per block is kept to a handful of scalar
  // instructions: with two waves per SIMD they are not hidden.
  constexpr int COPIES = KB / 1024;                                // instructions per block
  struct { const char* at; int kb, to, last, k, buf; bool again; } rq = {Kh + NW * KB, NW, -1, -1, -1, 0, false};
  const uint32_t roff = (lane / R::PPR) * R::RB + R::at(lane / R::PPR, lane % R::PPR) * 16;
  auto next_run = [&]() {                                          // the blocks that were not kept once more, or the next stripe's
    if (!rq.again && rq.last % NW + NW * SLOTS <= rq.last) {
      rq.again = true;
      rq.to = rq.last - NW * SLOTS;
    } else {
      do {
        const int of = stripe_at(rq.k + 1);
        if (of < 0) { rq.kb -= NW; rq.at -= NW * KB; return; }
        ++rq.k;
        rq.last = last_block(of);
      } while (rq.last < 0);
      rq.again = false;
      rq.to = rq.last;
    }
    rq.kb = rq.last % NW;
    rq.at = Kh + (int64_t)rq.kb * KB;
  };
  auto request = [&]() {
    const uint32_t dst = lds_offset(s_ring) + rq.buf;
    if (16 * rq.kb + 16 <= P) {
#pragma unroll
      for (int i = 0; i < COPIES; ++i) copy16_to_lds(rq.at + 1024 * i, roff ^ (16 * R::at(i * R::RPI, 0)), dst + 1024 * i);
    } else {                                                       // rows beyond the end: the last one again
#pragma unroll
      for (int i = 0; i < COPIES; ++i) {
        const int r = i * R::RPI + lane / R::PPR;
        copy16_to_lds(rq.at, (uint32_t)(min(r, P - 1 - 16 * rq.kb) * R::RB + R::at(r, lane % R::PPR) * 16), dst + 1024 * i);
      }
    }
    rq.buf = rq.buf + KB == RING * KB ? 0 : rq.buf + KB;
    rq.kb += NW;
    rq.at += NW * KB;
    if (rq.kb > rq.to) next_run();
  };
  int use = 0;                                                     // ring position of the next block to be used
  if constexpr (RING > 0) {
    if (st >= 0) {
      next_run();
#pragma unroll
      for (int i = 0; i < RING - 1; ++i) request();
    }
  }
  for (int k = 0; st >= 0; ++k) {
    const int i0 = st * OWN;
    const int next = stripe_at(k + 1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");               // this wave's part of the stripe's Q has landed
    __syncthreads();                                               // ... everyone's; and the column sums of the last stripe are in
    uint4 kf[R::NP];
    auto load_k = [&](int kb) {                                    // (without a ring: the next block, one ahead)
      if constexpr (RING == 0) {
        const uint32_t off = (uint32_t)min(n16, P - 1 - 16 * kb) * R::RB + 16 * j4;
        const char* base = Kh + (int64_t)kb * KB;
#pragma unroll
        for (int i = 0; i < R::NP; ++i) kf[i] = ld16(base + (off + 64 * i));
      }
    };
    auto arrive_k = [&]() {                                        // (with one: the next block in order)
      if constexpr (RING > 0) {
        request();
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"((RING - 1) * COPIES) : "memory");
        const char* at = s_ring + use;
#pragma unroll
        for (int i = 0; i < R::NP; ++i) kf[i] = *reinterpret_cast<const uint4*>(at + n16 * R::RB + R::at(n16, 4 * i + j4) * 16);
        use = use + KB == RING * KB ? 0 : use + KB;
      }
    };
    const int kb_last = last_block(st), kb_first = kb_last < 0 ? -1 : kb_last % NW;    // this wave's blocks: kb_first, + NW, ... kb_last
    int kb = kb_first;
    if (kb >= 0) load_k(kb);
    uint4 qf[NB][R::NP];
#pragma unroll
    for (int bb = 0; bb < NB; ++bb)
#pragma unroll
      for (int i = 0; i < R::NP; ++i) {
        const int row = 16 * bb + n16;
        qf[bb][i] = *reinterpret_cast<const uint4*>(lds + row * R::RB + R::at(row, 4 * i + j4) * 16);
      }
    float nm[NB], l[NB];                                           // minus the reference, the sum against it
#pragma unroll
    for (int bb = 0; bb < NB; ++bb) { nm[bb] = kNoRef; l[bb] = 0.f; }
    sc_f32x4_t E[SLOTS][NB];
    auto exps = [&](sc_f32x4_t (&s4)[NB], sc_f32x4_t (&e4)[NB], auto kept_tag) {
      constexpr int S = decltype(kept_tag)::value;                 // E[S ..] hold values against the present reference
      float part[NB];
      bool far = false;
      auto one = [&](int bb) {
#pragma unroll
        for (int e = 0; e < 4; ++e) e4[bb][e] = __builtin_amdgcn_exp2f(fmaf(s4[bb][e], scale_log2, nm[bb]));
        part[bb] = (e4[bb][0] + e4[bb][1]) + (e4[bb][2] + e4[bb][3]);
      };
#pragma unroll
      for (int bb = 0; bb < NB; ++bb) { one(bb); far |= !(part[bb] < kRefFar); }
      if (__builtin_amdgcn_ballot_w64(far)) {
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) {
          const float top = fmaxf(fmaxf(s4[bb][0], s4[bb][1]), fmaxf(s4[bb][2], s4[bb][3])) * scale_log2;
          const float mx = fmaxf(-nm[bb], top), alpha = __builtin_amdgcn_exp2f(-nm[bb] - mx);
          l[bb] *= alpha;
#pragma unroll
          for (int s = S; s < SLOTS; ++s) E[s][bb] *= alpha;
          nm[bb] = -mx;
          one(bb);
        }
      }
#pragma unroll
      for (int bb = 0; bb < NB; ++bb) l[bb] += part[bb];
    };
    // blocks further back than what is kept: sums only
    for (; kb >= 0 && kb + NW * SLOTS <= kb_last; kb += NW) {
      sc_f32x4_t s4[NB], e4[NB];
      arrive_k();
      R::template block_products<NB>(kf, qf, s4);
      load_k(kb + NW);
      exps(s4, e4, std::integral_constant<int, SLOTS>{});
    }
    auto slot = [&](auto tag) {
      constexpr int S = decltype(tag)::value;
      if (kb_last - NW * S < 0) return;                            // (wave-uniform)
      sc_f32x4_t s4[NB];
      arrive_k();
      R::template block_products<NB>(kf, qf, s4);
      if constexpr (S > 0) {
        load_k(kb_last - NW * (S - 1));
      } else if (16 * kb_last + 15 > i0) {                         // on the diagonal
#pragma unroll
        for (int bb = 0; bb < NB; ++bb)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            s4[bb][e] = 16 * kb_last + 4 * j4 + e <= min(i0 + 16 * bb + n16, Pq - 1) ? s4[bb][e] : -INFINITY;
      }
      exps(s4, E[S], std::integral_constant<int, S + 1>{});
    };
    for_down<SLOTS - 1>(slot);
    // ---- the rows' sums: the 4 lanes of a row, then the waves
    auto merge = [](float& m, float& s, float mo, float so) {
      const float mx = fmaxf(m, mo);
      s = s * __builtin_amdgcn_exp2f(m - mx) + so * __builtin_amdgcn_exp2f(mo - mx);
      m = mx;
    };
    float m, s;
    {
      float m2[2], l2[2];
      const bool up = lane & 32, up2 = lane & 16;
      if constexpr (NB == 4) {                                     // lane j4 ends up with row block j4
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          m2[x] = up ? -nm[2 + x] : -nm[x]; l2[x] = up ? l[2 + x] : l[x];
          const float mo = __shfl_xor(up ? -nm[x] : -nm[2 + x], 32, 64), lo = __shfl_xor(up ? l[x] : l[2 + x], 32, 64);
          merge(m2[x], l2[x], mo, lo);
        }
        m = up2 ? m2[1] : m2[0]; s = up2 ? l2[1] : l2[0];
        const float mo = __shfl_xor(up2 ? m2[0] : m2[1], 16, 64), lo = __shfl_xor(up2 ? l2[0] : l2[1], 16, 64);
        merge(m, s, mo, lo);
      } else {                                                     // lanes 0 and 1, 2 and 3 with row blocks 0, 1
        m = up ? -nm[1] : -nm[0]; s = up ? l[1] : l[0];
        const float mo = __shfl_xor(up ? -nm[0] : -nm[1], 32, 64), lo = __shfl_xor(up ? l[0] : l[1], 32, 64);
        merge(m, s, mo, lo);
        merge(m, s, __shfl_xor(m, 16, 64), __shfl_xor(s, 16, 64));
      }
      (void)m2; (void)l2; (void)up2;
    }
    const int my_row = NB == 4 ? lane : 16 * (lane >> 5) + n16;
    s_st[wave * OWN + my_row] = make_float2(m, s);
    __syncthreads();
    if (next >= 0) R::template stage<OWN, NW>(Qh, next * OWN, Pq - 1, lds);          // (all waves have their fragments)
    float2 w[NW];
#pragma unroll
    for (int x = 0; x < NW; ++x) w[x] = s_st[x * OWN + my_row];
    m = w[0].x;
#pragma unroll
    for (int x = 1; x < NW; ++x) m = fmaxf(m, w[x].x);
    s = 0.f;
#pragma unroll
    for (int x = 0; x < NW; ++x) s += w[x].y * __builtin_amdgcn_exp2f(w[x].x - m);
    const float inv = i0 + my_row < Pq ? 1.f / s : 0.f;            // (rows of padding count nothing)
    float M[NB], I[NB], f[NB];
#pragma unroll
    for (int bb = 0; bb < NB; ++bb) {
      M[bb] = __shfl(m, 64 / NB * bb + n16, 64);
      I[bb] = __shfl(inv, 64 / NB * bb + n16, 64);
      f[bb] = __builtin_amdgcn_exp2f(-nm[bb] - M[bb]) * I[bb];
    }

    // ---- the column sums
    auto add = [&](const float (&c)[4], int at) {                  // c[e]: this lane's share of key 16 at + 4 j4 + e
      const bool b0 = lane & 1, b1 = lane & 2;
      const float a0 = (b0 ? c[1] : c[0]) + sc_dpp<0xB1>(b0 ? c[0] : c[1]);
      const float a1 = (b0 ? c[3] : c[2]) + sc_dpp<0xB1>(b0 ? c[2] : c[3]);
      float v = (b1 ? a1 : a0) + sc_dpp<0x4E>(b1 ? a0 : a1);      // ... of key 16 at + 4 j4 + n16 % 4
      v += sc_dpp<0x128>(v);                                       // row_ror:8, row_ror:4
      v += sc_dpp<0x124>(v);
      // (in a stripe a key belongs to one wave, and stripes follow each other: the order of the additions is fixed)
      if (n16 < 4) __hip_atomic_fetch_add(&s_col[16 * at + 4 * j4 + n16], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto column = [&](auto tag) {
      constexpr int S = decltype(tag)::value;
      const int at = kb_last - NW * S;
      if (at < 0) return;
      float c[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        c[e] = 0.f;
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) {
          const float p = E[S][bb][e] * f[bb];
          if (S == 0) c[e] += 16 * at + 4 * j4 + e <= min(i0 + 16 * bb + n16, Pq - 1) ? p : 0.f;
          else c[e] = bb == 0 ? p : fmaf(E[S][bb][e], f[bb], c[e]);
        }
      }
      add(c, at);
    };
    for_down<SLOTS - 1>(column);
    if (kb_first >= 0 && kb_first + NW * SLOTS <= kb_last) {       // the blocks that were not kept, once more
      load_k(kb_first);
      for (int at = kb_first; at + NW * SLOTS <= kb_last; at += NW) {
        sc_f32x4_t s4[NB];
        arrive_k();
        R::template block_products<NB>(kf, qf, s4);
        load_k(at + NW);
        float c[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int bb = 0; bb < NB; ++bb)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            c[e] = fmaf(__builtin_amdgcn_exp2f(fmaf(s4[bb][e], scale_log2, -M[bb])), I[bb], c[e]);
        add(c, at);
      }
    }
    st = next;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                 // (copies that nobody waited for)
  __syncthreads();
  float* out = a.out + ((int64_t)bh * nch + chunk) * P;
  const int me = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));    // (= lane, not kept in a register all along)
  for (int i = 64 * wave + me; i < P; i += 64 * NW) out[i] = s_col[i];
}
template <typename T, int D, int NW>
__global__ __launch_bounds__(64 * NW, 2) void score_stripes_kernel(const ScoreArgs a) {
  extern __shared__ char s_tiles[];
  score_stripes<T, D, Stripe<T, D>::NB, Stripe<T, D>::SLOTS, Stripe<T, D>::RING, NW>(a, s_tiles);
}

// The two passes of the headline configuration under names of their own, and all others.
__global__ __launch_bounds__(kScThreads) void score_rowstats_mfma_kernel(const ScoreArgs a) {
  extern __shared__ char s_tiles[];
  score_rowstats<bf16_t, 128, 2>(a, s_tiles);
}
__global__ __launch_bounds__(kScThreads) void score_colsum_mfma_kernel(const ScoreArgs a) {
  extern __shared__ char s_tiles[];
  score_colsum<bf16_t, 128, 2, false, false>(a, s_tiles);
}
template <typename T, int D, int NB>
__global__ __launch_bounds__(kScThreads) void score_rowstats_kernel(const ScoreArgs a) {
  extern __shared__ char s_tiles[];
  score_rowstats<T, D, NB>(a, s_tiles);
}
template <typename T, int D, int NB, bool LSE, bool SPLIT>
__global__ __launch_bounds__(kScThreads) void score_colsum_kernel(const ScoreArgs a) {
  extern __shared__ char s_tiles[];
  score_colsum<T, D, NB, LSE, SPLIT>(a, s_tiles);
}
// scores[bk][j] = the sum of the g partial rows of a KV head (one per query head, or per workgroup of one), in order
__global__ __launch_bounds__(256) void sum_heads_kernel(const float* __restrict__ part, int g, int P, int64_t n /*B*Hkv*P*/,
                                                        float* __restrict__ scores) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t bk = i / P, j = i % P;
  double t = 0.0;                                 // (up to some hundred terms: fp32 would round more than the terms are off)
  int h = 0;
  for (; h + 8 <= g; h += 8) {
    float v[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) v[x] = part[(bk * g + h + x) * P + j];
#pragma unroll
    for (int x = 0; x < 8; ++x) t += v[x];
  }
  for (; h < g; ++h) t += part[(bk * g + h) * P + j];
  scores[i] = (float)t;
}

// the caller's normalisers, where they lie in memory that the call writes
__global__ __launch_bounds__(256) void copy_lse_kernel(const float* __restrict__ lse, int64_t n, float* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) out[i] = lse[i];
}

typedef void (*score_fn)(const ScoreArgs);
template <typename T, int D, int NB> score_fn pick_rowstats() {
  if constexpr (sizeof(T) == 2 && D == 128 && NB == 2) return score_rowstats_mfma_kernel;
  else return score_rowstats_kernel<T, D, NB>;
}
template <typename T, int D, int NB> score_fn pick_colsum(bool lse, bool split) {
  if (lse) return split ? score_colsum_kernel<T, D, NB, true, true> : score_colsum_kernel<T, D, NB, true, false>;
  if (split) return score_colsum_kernel<T, D, NB, false, true>;
  if constexpr (sizeof(T) == 2 && D == 128 && NB == 2) return score_colsum_mfma_kernel;
  else return score_colsum_kernel<T, D, NB, false, false>;
}

template <typename T, int D, int NB>
static sqa_status launch_scores(ScoreArgs a, bool lse, float* part /*NULL: not split by query head*/, float* scores, hipStream_t st) {
  using R = Rows<T, D>;
  const int tiles = (a.P + kMT * NB - 1) / (kMT * NB), g = a.Hq / a.Hkv;
  const size_t lds1 = 2 * (size_t)R::TILE, lds2 = 2 * ((size_t)R::TILE + 2 * kMT * sizeof(float));
  auto grid = [&](int heads, int per) { return (unsigned)(((heads / per + 7) / 8) * 8 * per * tiles); };
  if (!lse) {
    const score_fn fn = pick_rowstats<T, D, NB>();
    if (lds1 > 48 * 1024) SQA_HIP_CHECK(allow_dynamic_lds(reinterpret_cast<const void*>(fn), lds1));
    fn<<<grid(a.B * a.Hq, g), kScThreads, lds1, st>>>(a);
  }
  const bool split = part != nullptr;
  const score_fn fn = pick_colsum<T, D, NB>(lse, split);
  if (lds2 > 48 * 1024) SQA_HIP_CHECK(allow_dynamic_lds(reinterpret_cast<const void*>(fn), lds2));
  a.out = split ? part : scores;
  fn<<<split ? grid(a.B * a.Hq, g) : grid(a.B * a.Hkv, 1), kScThreads, lds2, st>>>(a);
  if (split) {
    const int64_t n = (int64_t)a.B * a.Hkv * a.P;
    sum_heads_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(part, g, a.P, n, scores);
  }
  SQA_HIP_CHECK(hipGetLastError());
  return SQA_OK;
}


template <typename T, int D, int NW>
static sqa_status launch_stripes(ScoreArgs a, float* part, float* scores, hipStream_t st) {
  using R = Rows<T, D>;
  constexpr int OWN = 16 * Stripe<T, D>::NB;
  const int g = a.Hq / a.Hkv, heads = a.B * a.Hq;
  const size_t lds = (size_t)OWN * R::RB + (size_t)NW * (16 * R::RB * Stripe<T, D>::RING + OWN * 8) + (size_t)(a.P + 15) * sizeof(float);
  if (lds > 48 * 1024) SQA_HIP_CHECK(allow_dynamic_lds(reinterpret_cast<const void*>(score_stripes_kernel<T, D, NW>), lds));
  const bool direct = g * a.chunks == 1;
  a.out = direct ? scores : part;
  score_stripes_kernel<T, D, NW><<<(unsigned)(((heads / g + 7) / 8) * 8 * g * a.chunks), 64 * NW, lds, st>>>(a);
  if (!direct) {
    const int64_t n = (int64_t)a.B * a.Hkv * a.P;
    sum_heads_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(part, g * a.chunks, a.P, n, scores);
  }
  SQA_HIP_CHECK(hipGetLastError());
  return SQA_OK;
}
// How a call goes: in one pass, with 4 waves per workgroup (two workgroups per CU) or 8 (one, which keeps twice the keys of a
// stripe) and so many workgroups per query head, or in two passes.  Both ways are estimated (us), the cheaper one is taken.
// All workgroups of a KV head run on one XCD, so what counts is the fullest XCD: (KV heads / 8, rounded up) x g x chunks
// workgroups on 32 CUs.  (Counted over the whole chip, 44 heads of 3817 tokens, bf16, D = 128, got 11 workgroups each: 66 on an
// XCD, three rounds, 275 us; 5 each take 214.)
// The constants are fitted to 3700 shapes of one length, each measured in two passes and in up to 14 cuts (1 to 4096 heads,
// 33 to 4096 tokens, 1 to 8 query heads per KV head): what is chosen takes 1.1 % longer than the fastest of a shape's ways on
// average, over 10 % longer in one of 60.  Measured, us:
//   bf16, D = 128   16 heads of 2048 tokens  4 waves 43, 8 waves 26.5;  64 of 777  21.3 and 22.4;  256 of 2048  304 and 290
//   fp32, D = 128   16 of 2048  117 and 86;  256 of 512  98 and 112
//   two passes and one   bf16, D = 64: 640 heads of 96 tokens 12.2 and 14.7, 400 of 2154 (8 per KV head) 392 and 457;
//                        D = 128: 736 of 71 15.4 and 18.2;  fp32, D = 64: 640 of 41 12.1 and 13.2
struct StripeCut { int waves, chunks; double us; };
constexpr int kStripeMaxP = 4096;
constexpr int kXcds = 8, kXcdCus = 32;
struct StripeFit {
  double stripe, block, again;                   // of a workgroup of 4 waves: per stripe, per key block of a wave, and that much more per block that is not kept
  double alone;                                  // 4 waves: as the only workgroup of a CU it takes this share of the time
  double start;                                  // a workgroup's start: nothing is on its way yet
  double whole, spread;                          // several rounds: how much of a last, partial round counts; of the longest workgroup beyond the average
  double base;                                   // the launches
  double far, l2;                                // keys read at a time, in units of an XCD's 4 MB of L2: beyond l2 each costs this much more
  double stripe8, block8;                        // 8 waves: the first two times these
};
constexpr StripeFit kStripeFit[2][2] = {         // [bf16, fp32][D = 64, 128]
    {{1.88, 0.498, 0.75, 0.842, 2.84, 0.669, 0.926, 2.679, 0.101, 0.529, 1.318, 0.983},
     {2.221, 0.611, 0.959, 0.82, 3.3, 0.725, 0.481, 2.047, 0.142, 1.168, 1.202, 0.893}},
    {{1.411, 1.042, 1.227, 0.688, 3.11, 0.607, 0.564, 2.554, 0.129, 0.518, 1.11, 1.039},
     {1.897, 1.897, 1.193, 0.617, 3.141, 0.784, 0.637, 2.395, 0.057, 0.531, 0.786, 1.032}}};
struct TwoPassFit {
  double alone1, alone2;                         // per 64-row tile of the longest workgroup of each pass
  double each1, each2;                           // per tile and workgroup of the fullest XCD's CUs
  double start, wg, base;                        // per pass, per workgroup of a CU, the launches
  double power;                                  // the two add up as powers (latency and throughput overlap)
  double split;                                  // column sums per query head: the kernel that adds them
  double whole;                                  // how much of a partly filled CU counts
};
constexpr TwoPassFit kTwoPassFit[2][2] = {
    {{0.845, 0.435, 0.502, 0.178, 3.312, 0.466, 0, 1.23, 1.939, 0.467},
     {0.739, 0.95, 0.104, 0.812, 3.327, 1.547, 0, 1.6, 2.813, 0.076}},
    {{1.609, 0.786, 0.024, 2.302, 2.933, 0.628, 0, 1.767, 1.355, 0.65},
     {3.048, 1.421, 1.854, 2.794, 0, 1.122, 3.515, 1.759, 3.068, 0.701}}};

// Pass 2 per query head where the KV heads alone give the chip too few workgroups (8 per CU), unless the call is
// so small that the additional launch is what one sees.  64 query heads over 8, one sequence, 1024 tokens, bf16,
// D = 64: 129 -> 42 us for both passes; the same at 4096 tokens, D = 128: 650 -> 362; 32 over 8, 69 tokens: 14 -> 17.
static bool split_heads(sqa_dtype dt, int B, int Hq, int Hkv, int P) {
  const int own = dt == SQA_F32 ? kMT : 2 * kMT;
  return Hq != Hkv && P > 128 && (int64_t)((P + own - 1) / own) * B * Hkv < 2048;
}

static StripeCut stripe_cut(sqa_dtype dt, int D, int B, int Hq, int Hkv, int P, bool ragged, int64_t most_chunks) {
  const bool f32 = dt == SQA_F32;
  const StripeFit& f = kStripeFit[f32][D == 128];
  const int own = f32 ? 32 : 64, slots = f32 ? (D == 64 ? 16 : 14) : 8, g = Hq / Hkv;
  const int n_str = (P + own - 1) / own;
  const int64_t xcd_heads = ((int64_t)B * Hkv + kXcds - 1) / kXcds * g;
  StripeCut best = {4, 1, 1e30};
  for (int waves = 4; waves <= 8; waves += 4) {
    const int64_t resident = waves == 4 ? 2 * kXcdCus : kXcdCus;
    const double stripe = waves == 4 ? f.stripe : f.stripe * f.stripe8, block = waves == 4 ? f.block : f.block * f.block8;
    auto stripe_us = [&](int st) {
      const int rows = (st + 1) * own < P ? (st + 1) * own : P, blocks = (rows + 16 * waves - 1) >> (waves == 4 ? 6 : 7);
      return stripe + block * (blocks + (blocks > slots ? f.again * (blocks - slots) : 0.0));
    };
    double all = 0.0;
    for (int st = 0; st < n_str; ++st) all += stripe_us(st);
    int64_t before = 0;
    // (sequences of different length, which the host does not see: more and shorter workgroups even out long ones; 64 heads
    // of 2766 tokens and 64 of 1383, bf16, D = 128: 261 us in one round, 183 in three; 5 x 32 heads of 613 to 306 23 and 38)
    const int least = ragged ? (P > 2048 ? 6 : (P > 1024 ? 4 : 2)) : 1;      // in half rounds
    for (const int halves : {1, 2, 3, 4, 6, 8, 12}) {
      if (halves < least) continue;
      int64_t n = resident * halves / (2 * xcd_heads);
      n = n < n_str ? n : n_str;
      n = n < most_chunks ? n : most_chunks;
      n = n < 1 ? 1 : n;
      if (n == before) continue;
      before = n;
      // the longest workgroup: the first of a head, its last, or the last that has a stripe more than others
      double longest = n == 1 ? f.start + all : 0.0;
      const int m = (int)n, rem = n_str % m;
      for (const int c : {0, m - 1, rem ? m - rem : 0}) {
        if (m == 1) break;
        double us = f.start;
        for (int top = n_str - 1, odd = 0; top >= 0; top -= m, odd ^= 1) {
          const int st = top - (odd ? m - 1 - c : c);
          if (st >= 0) us += stripe_us(st);
        }
        longest = us > longest ? us : longest;
      }
      const int64_t wgs = xcd_heads * n, at_once = wgs < resident ? wgs : resident;
      double us = longest;
      if (wgs > resident) {
        const double average = f.start + all / (double)n;
        const double rounds = f.whole * (double)((wgs + resident - 1) / resident) + (1.0 - f.whole) * (double)wgs / (double)resident;
        const double queued = rounds * average + f.spread * (longest - average);
        us = queued > us ? queued : us;
      } else if (waves == 4 && 2 * wgs <= resident) {
        us *= f.alone;
      }
      const double keys = (double)((at_once + n * g - 1) / (n * g)) * P * D * (f32 ? 4 : 2) / (4 << 20);
      us = f.base + us * (1.0 + f.far * (keys > f.l2 ? keys - f.l2 : 0.0));
      if (us < best.us) best = {waves, (int)n, us};
    }
  }
  return best;
}
// Are two passes estimated below `limit` us?
static bool two_passes_below(double limit, sqa_dtype dt, int D, int B, int Hq, int Hkv, int P, bool split) {
  const bool f32 = dt == SQA_F32;
  const TwoPassFit& f = kTwoPassFit[f32][D == 128];
  const int nb = f32 ? 1 : 2, own = kMT * nb, g = Hq / Hkv, tiles = (P + own - 1) / own, n64 = (P + kMT - 1) / kMT;
  double rows = 0.0, cols = 0.0;                 // 64-row tiles of an average workgroup of each pass
  for (int t = 0; t < tiles; ++t) {
    rows += (((t + 1) * own < P ? (t + 1) * own : P) + kMT - 1) / kMT;
    cols += n64 - t * nb;
  }
  const double xcd_kv = (double)(((int64_t)B * Hkv + kXcds - 1) / kXcds);
  const int heads_each = split ? 1 : g;          // query heads that a workgroup of pass 2 adds up
  const double per_cu[2] = {xcd_kv * g * tiles / kXcdCus, xcd_kv * (g / heads_each) * tiles / kXcdCus};
  const double latency[2] = {f.start + f.alone1 * n64, f.start + f.alone2 * n64 * heads_each};
  const double each[2] = {f.wg + f.each1 * rows / tiles, f.wg + f.each2 * cols / tiles * heads_each};
  double work[2], least = f.base + (split ? f.split : 0.0);
  limit -= least;
  least = 0.0;
  for (int i = 0; i < 2; ++i) {
    work[i] = each[i] * (f.whole * ceil(per_cu[i]) + (1.0 - f.whole) * per_cu[i]);
    least += latency[i] > work[i] ? latency[i] : work[i];
  }
  if (least >= limit) return false;              // (the power sum lies between the larger term and the sum: most calls end here)
  double us = 0.0;
  for (int i = 0; i < 2; ++i) us += pow(pow(latency[i], f.power) + pow(work[i], f.power), 1.0 / f.power);
  return us < limit;
}
// The way of a call whose workspace holds `most_chunks` floats per query row.  Two passes have to be clearly ahead where
// the sequences' lengths differ: the estimates know the longest only.
static bool two_passes(sqa_dtype dt, int D, int B, int Hq, int Hkv, int P, bool ragged, int64_t most_chunks, const StripeCut& cut) {
  return two_passes_below((ragged ? 0.93 : 1.0) * cut.us, dt, D, B, Hq, Hkv, P, most_chunks >= 3 && split_heads(dt, B, Hq, Hkv, P));
}

}  // namespace sqa

// In one pass: a partial row of column sums per workgroup of a query head.  In two, per query row: reference, 1/sum, and
// (pass 2 split by query head) a partial column sum.  A workspace of two floats per row is enough too: fewer workgroups,
// or two passes where those are faster then (8 heads of 4096 tokens, bf16, D = 128, two floats per row: 544 us in one pass,
// 114 in two; 48 with the whole workspace.  16 of 2048, fp32, D = 64: 353, 155 and 54).
extern "C" size_t sqa_prefill_scores_workspace_bytes(int B, int Hq, int Hkv, int P, int D) {
  if (B < 1 || Hq < 1 || P < 1) return 0;
  if (Hkv < 1 || Hq % Hkv != 0) Hkv = Hq;
  // (neither the element type nor whether the sequences differ in length is known here: the most of what they need)
  const int64_t rows = (int64_t)B * Hq * P;
  int floats = 3;
  for (const int d : {64, 128}) {
    if (P > sqa::kStripeMaxP || (D != d && (D == 64 || D == 128))) continue;
    for (const sqa_dtype dt : {SQA_F32, SQA_BF16})
      for (const bool ragged : {false, true}) {
        const sqa::StripeCut cut = sqa::stripe_cut(dt, d, B, Hq, Hkv, P, ragged, INT32_MAX);
        if (cut.chunks > floats && !sqa::two_passes(dt, d, B, Hq, Hkv, P, ragged, INT32_MAX, cut)) floats = cut.chunks;
      }
  }
  return (size_t)rows * floats * sizeof(float);
}

extern "C" sqa_status sqa_prefill_scores(const void* Q, const void* K, sqa_dtype dt,
                                         int B, int Hq, int Hkv, int P, int D,
                                         float* scores_out, void* workspace, size_t ws_bytes, void* stream) {
  return sqa_prefill_scores_ex(Q, K, dt, B, Hq, Hkv, P, D, scores_out, workspace, ws_bytes, stream, nullptr);
}

namespace sqa {
static sqa_status prefill_scores_impl(const void* Q, const void* K, const float* row_lse, sqa_dtype dt,
                                      int B, int Hq, int Hkv, int P, int D,
                                      float* scores_out, void* workspace, size_t ws_bytes, void* stream,
                                      const sqa_batch_opts* opts) {
  if (!Q || !K || !scores_out || !workspace) return SQA_ERR_NULL;
  if (dt != SQA_F32 && dt != SQA_BF16) return SQA_ERR_DTYPE;
  if (B < 1 || Hq < 1 || Hkv < 1 || P < 1 || Hq % Hkv != 0 || (D != 64 && D != 128)) return SQA_ERR_SHAPE;
  if (((int64_t)B * Hq + 8) * ((P + 63) / 64) > INT32_MAX) return SQA_ERR_SHAPE;   // workgroups of one launch
  if (!aligned16(Q) || !aligned16(K) || (reinterpret_cast<uintptr_t>(workspace) & 7u)) return SQA_ERR_SHAPE;
  if (row_lse && (reinterpret_cast<uintptr_t>(row_lse) & 3u)) return SQA_ERR_SHAPE;
  const size_t rows = (size_t)B * Hq * P;
  if (ws_bytes < rows * 2 * sizeof(float)) return SQA_ERR_CAPACITY;
  const bool lse = row_lse != nullptr;
  float* ws = static_cast<float*>(workspace);
  ScoreArgs a;
  a.Q = Q; a.K = K; a.B = B; a.Hq = Hq; a.Hkv = Hkv; a.P = P;
  a.scale_log2 = (float)(1.4426950408889634 / sqrt((double)D));
  a.prompt_len = opts ? opts->prompt_len : nullptr;
  a.ref = lse ? const_cast<float*>(row_lse) : ws;          // (read only when given)
  a.inv = ws + rows;
  a.out = nullptr;
  float* part = lse ? ws : (ws_bytes >= rows * 3 * sizeof(float) ? ws + 2 * rows : nullptr);
  // The normalisers are read while the sums are written.  A caller may give them in memory that it hands over for the
  // scores (they are copied into the workspace first) or in the workspace itself (the partial sums then keep off them).
  bool copy_lse = false;
  if (lse) {
    auto shares = [&](const float* p, size_t n) { return row_lse < p + n && p < row_lse + rows; };
    copy_lse = shares(scores_out, (size_t)B * Hkv * P);
    if (copy_lse) { a.ref = ws; part = ws + rows; }
    else if (shares(ws, rows)) part = shares(ws + rows, rows) ? nullptr : ws + rows;
  }
  a.chunks = 0;
  const int64_t chunks = (int64_t)(ws_bytes / (rows * sizeof(float)));
  StripeCut cut = {4, 0, 0.0};
  if (!lse && P <= kStripeMaxP) cut = stripe_cut(dt, D, B, Hq, Hkv, P, a.prompt_len != nullptr, chunks);
  if (cut.chunks > 0 && !two_passes(dt, D, B, Hq, Hkv, P, a.prompt_len != nullptr, chunks, cut)) {
    a.chunks = cut.chunks;
    auto launch = [&](auto type, auto dim) {
      using T = decltype(type);
      constexpr int D_ = decltype(dim)::value;
      hipStream_t st = static_cast<hipStream_t>(stream);
      return cut.waves == 4 ? launch_stripes<T, D_, 4>(a, ws, scores_out, st) : launch_stripes<T, D_, 8>(a, ws, scores_out, st);
    };
    using D64 = std::integral_constant<int, 64>;
    using D128 = std::integral_constant<int, 128>;
    if (dt == SQA_F32) return D == 64 ? launch(float{}, D64{}) : launch(float{}, D128{});
    return D == 64 ? launch(bf16_t{}, D64{}) : launch(bf16_t{}, D128{});
  }
  if (!split_heads(dt, B, Hq, Hkv, P)) part = nullptr;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (copy_lse) copy_lse_kernel<<<(unsigned)(rows / 256 + 1 < 4096 ? rows / 256 + 1 : 4096), 256, 0, st>>>(row_lse, (int64_t)rows, ws);
  if (dt == SQA_F32) {
    if (D == 64) return launch_scores<float, 64, 1>(a, lse, part, scores_out, st);
    return launch_scores<float, 128, 1>(a, lse, part, scores_out, st);
  }
  if (D == 64) return launch_scores<bf16_t, 64, 2>(a, lse, part, scores_out, st);
  return launch_scores<bf16_t, 128, 2>(a, lse, part, scores_out, st);
}
}  // namespace sqa

extern "C" sqa_status sqa_prefill_scores_ex(const void* Q, const void* K, sqa_dtype dt,
                                            int B, int Hq, int Hkv, int P, int D,
                                            float* scores_out, void* workspace, size_t ws_bytes, void* stream,
                                            const sqa_batch_opts* opts) {
  return sqa::prefill_scores_impl(Q, K, nullptr, dt, B, Hq, Hkv, P, D, scores_out, workspace, ws_bytes, stream, opts);
}

extern "C" sqa_status sqa_prefill_scores_lse(const void* Q, const void* K, const float* row_lse, sqa_dtype dt,
                                             int B, int Hq, int Hkv, int P, int D,
                                             float* scores_out, void* workspace, size_t ws_bytes, void* stream,
                                             const sqa_batch_opts* opts) {
  if (!row_lse) return SQA_ERR_NULL;
  return sqa::prefill_scores_impl(Q, K, row_lse, dt, B, Hq, Hkv, P, D, scores_out, workspace, ws_bytes, stream, opts);
}

// Layer-importance probe: Algorithm 1 steps 1-4 with the cosine-similarity
// equation of Sec. 3.  A pure streaming reduction (each hidden-state element is
// read once), so the only roofline is HBM bandwidth.
//
// Mapping: grid = (blocks per layer, layers); a workgroup has 4 waves; a wave
// owns whole token rows (row = wave id, stepping by the number of waves of the
// layer; several sequences: see imp_share) and its 64 lanes read the row in 16-byte pieces, 1 KiB per wave load.
// The three dot products accumulate in fp32 per lane, are summed over the wave,
// and lane 0 adds the row's cosine to a per-wave fp64 sum.  Partial sums go to
// the workspace and a second tiny kernel adds them in a fixed order: no atomics,
// results are bit-identical from run to run.  Rows of up to 1 KiB go several to a
// wave (importance_short_rows_kernel).
//
// The same kernel also runs fused into the producer of the "after" tensor: the
// residual connection h_out = h_in + attn_out.  Then it reads h_in and attn_out,
// writes h_out rounded to the storage type, and takes the cosine against those
// stored values in the same pass, so the probe itself moves no extra byte.
#include "sqa_common.h"
#include <type_traits>

namespace sqa {

constexpr int kImpThreads = 256;
constexpr int kImpWaves = kImpThreads / SQA_WAVE;
constexpr int kImpMaxBlocks = 1024;   // partial sums per layer
constexpr int kImpMaxPieces = 2 * kImpMaxBlocks;      // the same of several sequences (the workspace holds kImpMaxBlocks for each)
// A workgroup that has at most 3 turns takes them all and needs no second kernel, as long as what it does alone is short: 16-byte
// pieces of a row times further turns.  One layer, us on the device (replayed graphs), two kernels and one: 5 rows of
// 4096 bf16 (512) 3.9 and 3.0, 12 of 2048 (512) 3.6 and 3.4 / 12 of 4096 (1024) 3.9 and 6.2, 12 of 8192 fp32 (4096) 8.6 and
// 17.5, 12 of 16384 (8192) 13.5 and 32.1; back to back from the host, which two launches hold up for 6.8, up to 512 4.0 to 4.8.
constexpr int kImpOnePieces = 512;

template <typename T> struct Dots;
template <> struct Dots<float> {
  static __device__ __forceinline__ void acc(const uint4& a, const uint4& b, float& ab, float& aa, float& bb) {
    const float a0 = __uint_as_float(a.x), a1 = __uint_as_float(a.y), a2 = __uint_as_float(a.z), a3 = __uint_as_float(a.w);
    const float b0 = __uint_as_float(b.x), b1 = __uint_as_float(b.y), b2 = __uint_as_float(b.z), b3 = __uint_as_float(b.w);
    ab = fmaf(a0, b0, ab); ab = fmaf(a1, b1, ab); ab = fmaf(a2, b2, ab); ab = fmaf(a3, b3, ab);
    aa = fmaf(a0, a0, aa); aa = fmaf(a1, a1, aa); aa = fmaf(a2, a2, aa); aa = fmaf(a3, a3, aa);
    bb = fmaf(b0, b0, bb); bb = fmaf(b1, b1, bb); bb = fmaf(b2, b2, bb); bb = fmaf(b3, b3, bb);
  }
};
template <> struct Dots<bf16_t> {
  static __device__ __forceinline__ void acc(const uint4& a, const uint4& b, float& ab, float& aa, float& bb) {
    ab = dot2_bf16(a.x, b.x, ab); ab = dot2_bf16(a.y, b.y, ab); ab = dot2_bf16(a.z, b.z, ab); ab = dot2_bf16(a.w, b.w, ab);
    aa = dot2_bf16(a.x, a.x, aa); aa = dot2_bf16(a.y, a.y, aa); aa = dot2_bf16(a.z, a.z, aa); aa = dot2_bf16(a.w, a.w, aa);
    bb = dot2_bf16(b.x, b.x, bb); bb = dot2_bf16(b.y, b.y, bb); bb = dot2_bf16(b.z, b.z, bb); bb = dot2_bf16(b.w, b.w, bb);
  }
};

// a + r element by element: fp32 add, rounded to the storage type
template <typename T> struct Residual;
template <> struct Residual<float> {
  static __device__ __forceinline__ uint4 add(const uint4& a, const uint4& r) {
    return make_uint4(__float_as_uint(__uint_as_float(a.x) + __uint_as_float(r.x)),
                      __float_as_uint(__uint_as_float(a.y) + __uint_as_float(r.y)),
                      __float_as_uint(__uint_as_float(a.z) + __uint_as_float(r.z)),
                      __float_as_uint(__uint_as_float(a.w) + __uint_as_float(r.w)));
  }
};
template <> struct Residual<bf16_t> {
  static __device__ __forceinline__ uint32_t add2(uint32_t a, uint32_t r) {
    return f32_to_bf16_bits(bf16_lo(a) + bf16_lo(r)) | (f32_to_bf16_bits(bf16_hi(a) + bf16_hi(r)) << 16);
  }
  static __device__ __forceinline__ uint4 add(const uint4& a, const uint4& r) {
    return make_uint4(add2(a.x, r.x), add2(a.y, r.y), add2(a.z, r.z), add2(a.w, r.w));
  }
};

struct ImpArgs {
  const void* h_in;
  const void* other;             // h_out, or attn_out where h_out is written
  void* h_out_w;                 // may be h_in or other
  int64_t n_tokens;
  int hidden;
  const int32_t* seq_start;      // [n_seq + 1] or NULL
  int n_seq;
  int piece;                     // see imp_share
  double* partial;               // [layers][gridDim.x]
  float* cos_out;                // [layers][n_seq]
};
enum { kImpAll = -2, kImpWhole = -1 };   // ImpArgs::piece: a layer's rows in turns; a sequence per workgroup; else log2 of a piece's rows

template <int CTRL> __device__ __forceinline__ float imp_dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// sum over groups of W lanes, in every lane, by vector instructions
template <int W> __device__ __forceinline__ float lanes_sum(float v) {
  static_assert(W == 32 || W == 64, "lanes of a row");
  typedef unsigned u2_t __attribute__((ext_vector_type(2)));
  v += imp_dpp<0xB1>(v);              // quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror, row_mirror
  v += imp_dpp<0x4E>(v);
  v += imp_dpp<0x141>(v);
  v += imp_dpp<0x140>(v);
  u2_t r = __builtin_bit_cast(u2_t, __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  v = __uint_as_float(r.x) + __uint_as_float(r.y);
  if constexpr (W == 64) {
    r = __builtin_bit_cast(u2_t, __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false));
    v = __uint_as_float(r.x) + __uint_as_float(r.y);
  }
  return v;
}

// rows [lo, hi) of a sequence: all of the layer's unless the tokens are segmented
__device__ __forceinline__ void imp_rows(const ImpArgs& a, int seq, int64_t& lo, int64_t& hi) {
  lo = 0;
  hi = a.n_tokens;
  if (a.seq_start) {
    lo = a.seq_start[seq];
    hi = a.seq_start[seq + 1];
    lo = lo < 0 ? 0 : lo;
    hi = hi > a.n_tokens ? a.n_tokens : hi;
  }
}

// Which rows a workgroup takes.  One sequence: all of them, in turns with the layer's other workgroups.  Several, together no
// more than one workgroup is given: a workgroup each.  Otherwise the layer's rows are cut into pieces of 2^piece, and again
// where a sequence ends, so that the work is shared out evenly whatever the lengths: the part of sequence s in piece j belongs
// to workgroup j + s, which grows by at least one from each part to the next.  Every wave finds the s of its workgroup from
// the sequences' starts, 64 at a time (one round for up to 63 sequences).  us per call on the device, one layer, rows of 4096
// bf16, with 1024 workgroups for each sequence / with as many as twice the average length needs / so: 4096 rows and 32 of one
// row 23.2 / 34.0 / 15.4; 4000 and 1000 of one 326 / 1660 / 18.6; 8192 and 100 of 20 60 / 79 / 32; 16 of 1000 45.4 / 44.4 / 45.6,
// 1000 of 10 361 / 29 / 31; 11 layers, 9 of 1000 rows of 256 56.2 / 20.0 / 20.4.  (Where a workgroup per sequence was enough by the
// average length, the second kernel comes on top: 64 of 30 rows of 256 14.8 / 3.6 / 6.1.)
struct ImpShare {
  int64_t row, hi, step;          // of a wave with `rows` rows at a time
  int seq;
};
template <bool SEQS /*there may be several*/> __device__ __forceinline__ ImpShare imp_share(const ImpArgs& a, int wave, int rows) {
  ImpShare r;
  int64_t lo;
  r.seq = 0;
  r.step = (int64_t)kImpWaves * rows;
  int64_t first = 0;
  if (!SEQS || a.piece == kImpAll) {
    first = blockIdx.x * r.step;
    r.step *= gridDim.x;
    imp_rows(a, 0, lo, r.hi);
  } else if (a.piece == kImpWhole) {
    r.seq = blockIdx.x;
    imp_rows(a, r.seq, lo, r.hi);
  } else {
    const int w = blockIdx.x, lane = threadIdx.x & (SQA_WAVE - 1);
    int base = 0, n = a.n_seq, at = 0;
    auto count = [&](int every) {                 // samples of base, base + every, .. below base + n that are at w or before
      at = a.seq_start[base + min(lane * every, n)];
      return __popcll(__ballot(lane * every < n && (max(at, 0) >> a.piece) + base + lane * every <= w));
    };
    while (n >= SQA_WAVE) {
      const int every = (n + SQA_WAVE - 1) / SQA_WAVE, skip = max(count(every) - 1, 0) * every;
      base += skip;
      n = min(every, n - skip);
    }
    const int s = max(count(1) - 1, 0);           // (before the first sequence: its part of that piece is empty)
    r.seq = base + s;
    lo = max(__builtin_amdgcn_readlane(at, s), 0);
    r.hi = min((int64_t)__builtin_amdgcn_readlane(at, s + 1), a.n_tokens);
    const int64_t from = (int64_t)(w - r.seq) << a.piece;
    lo = max(lo, from);
    r.hi = min(r.hi, from + ((int64_t)1 << a.piece));
  }
  r.row = lo + first + wave * rows;
  return r;
}

// the cosine of a (layer, sequence) from the sum over its rows
__device__ __forceinline__ void imp_store(const ImpArgs& a, int64_t item, int64_t rows, double sum) {
  a.cos_out[item] = rows > 0 ? (float)(sum / (double)rows) : 0.f;
}

// a workgroup's sum, or (if it had all rows of the sequence) the result
__device__ __forceinline__ void imp_put(const ImpArgs& a, int seq, const double* waves) {
  double s = 0.0;
  for (int w = 0; w < kImpWaves; ++w) s += waves[w];
  if (a.piece == kImpWhole) {
    int64_t lo, hi;
    imp_rows(a, seq, lo, hi);
    imp_store(a, (int64_t)blockIdx.y * a.n_seq + seq, hi - lo, s);
  } else {
    a.partial[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
  }
}

// FUSE = false: h_out is read.  FUSE = true: `other` is attn_out and h_out is written (NT: non-temporally).
template <typename T, bool FUSE, bool NT>
__global__ __launch_bounds__(kImpThreads) void importance_partial_kernel(const ImpArgs args) {
  constexpr int E = elem<T>::per16;
  const int lane = threadIdx.x & (SQA_WAVE - 1);
  const int wave = threadIdx.x / SQA_WAVE;
  const int layer = blockIdx.y;
  const int chunks = args.hidden / E;            // 16-byte pieces per row
  const int64_t row_bytes = args.hidden * (int64_t)sizeof(T), layer_bytes = args.n_tokens * row_bytes;
  const char* A = static_cast<const char*>(args.h_in) + layer * layer_bytes;
  const char* Bp = static_cast<const char*>(args.other) + layer * layer_bytes;
  char* Wp = FUSE ? static_cast<char*>(args.h_out_w) + layer * layer_bytes : nullptr;
  const ImpShare mine = imp_share<!FUSE>(args, wave, 1);
  auto put = [](char* p, const uint4& v) { if constexpr (NT) st16_nt(p, v); else st16(p, v); };
  double wave_cos = 0.0;
  for (int64_t row = mine.row; row < mine.hi; row += mine.step) {
    const char* a = A + row * row_bytes;
    const char* b = Bp + row * row_bytes;
    char* w = FUSE ? Wp + row * row_bytes : nullptr;
    float ab = 0.f, aa = 0.f, bb = 0.f;
    int c = lane;
    for (; c + 3 * SQA_WAVE < chunks; c += 4 * SQA_WAVE) {      // 8 loads in flight per lane
      const uint4 a0 = ld16_nt(a + (int64_t)c * 16);
      uint4 b0 = ld16_nt(b + (int64_t)c * 16);
      const uint4 a1 = ld16_nt(a + (int64_t)(c + SQA_WAVE) * 16);
      uint4 b1 = ld16_nt(b + (int64_t)(c + SQA_WAVE) * 16);
      const uint4 a2 = ld16_nt(a + (int64_t)(c + 2 * SQA_WAVE) * 16);
      uint4 b2 = ld16_nt(b + (int64_t)(c + 2 * SQA_WAVE) * 16);
      const uint4 a3 = ld16_nt(a + (int64_t)(c + 3 * SQA_WAVE) * 16);
      uint4 b3 = ld16_nt(b + (int64_t)(c + 3 * SQA_WAVE) * 16);
      if (FUSE) {
        b0 = Residual<T>::add(a0, b0); b1 = Residual<T>::add(a1, b1);
        b2 = Residual<T>::add(a2, b2); b3 = Residual<T>::add(a3, b3);
        put(w + (int64_t)c * 16, b0); put(w + (int64_t)(c + SQA_WAVE) * 16, b1);
        put(w + (int64_t)(c + 2 * SQA_WAVE) * 16, b2); put(w + (int64_t)(c + 3 * SQA_WAVE) * 16, b3);
      }
      Dots<T>::acc(a0, b0, ab, aa, bb); Dots<T>::acc(a1, b1, ab, aa, bb);
      Dots<T>::acc(a2, b2, ab, aa, bb); Dots<T>::acc(a3, b3, ab, aa, bb);
    }
    for (; c + SQA_WAVE < chunks; c += 2 * SQA_WAVE) {
      const uint4 a0 = ld16_nt(a + (int64_t)c * 16);
      uint4 b0 = ld16_nt(b + (int64_t)c * 16);
      const uint4 a1 = ld16_nt(a + (int64_t)(c + SQA_WAVE) * 16);
      uint4 b1 = ld16_nt(b + (int64_t)(c + SQA_WAVE) * 16);
      if (FUSE) {
        b0 = Residual<T>::add(a0, b0); b1 = Residual<T>::add(a1, b1);
        put(w + (int64_t)c * 16, b0); put(w + (int64_t)(c + SQA_WAVE) * 16, b1);
      }
      Dots<T>::acc(a0, b0, ab, aa, bb); Dots<T>::acc(a1, b1, ab, aa, bb);
    }
    for (; c < chunks; c += SQA_WAVE) {
      const uint4 a0 = ld16_nt(a + (int64_t)c * 16);
      uint4 b0 = ld16_nt(b + (int64_t)c * 16);
      if (FUSE) { b0 = Residual<T>::add(a0, b0); put(w + (int64_t)c * 16, b0); }
      Dots<T>::acc(a0, b0, ab, aa, bb);
    }
    ab = wave_sum(ab); aa = wave_sum(aa); bb = wave_sum(bb);
    const double na = fmax(sqrt((double)aa), 1e-8), nb = fmax(sqrt((double)bb), 1e-8);
    wave_cos += (double)ab / (na * nb);
  }
  __shared__ double s_part[kImpWaves];
  if (lane == 0) s_part[wave] = wave_cos;
  __syncthreads();
  if (threadIdx.x == 0) imp_put(args, mine.seq, s_part);
}

// Rows of up to 1 KiB: W lanes share a row and hold one 16-byte piece of it, a wave takes 64 / W rows side by side and 4 such
// groups at a time.  A lane keeps a row's sums until W rows per group have come; then their cosines are worked out together (one
// row at a time, each cost a wave some 300 double-precision instructions, half of the lanes had nothing to load at 512 bytes,
// and there was one load in flight).  Residual add, 19 layers of 2159 rows of 256 bf16 29.0 -> 17.0 us; 9 sequences, 11 layers
// of 9000 rows of 256 56.8 -> 21.4.  Longer rows are better off one to a wave (2048 rows of 4096 bf16 13.2, 15.4 so: the sums
// over the lanes at the end come on top).
template <typename T, bool FUSE, bool NT, int W>
__global__ __launch_bounds__(kImpThreads) void importance_short_rows_kernel(const ImpArgs args) {
  constexpr int E = elem<T>::per16, SIDE = SQA_WAVE / W, ROWS = 4 * SIDE;
  const int lane = threadIdx.x & (SQA_WAVE - 1), side = lane / W, lw = lane % W;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / SQA_WAVE);
  const int chunks = args.hidden / E;            // at most W
  const int64_t row_bytes = (int64_t)chunks * 16, layer_bytes = args.n_tokens * row_bytes;
  const char* A = static_cast<const char*>(args.h_in) + blockIdx.y * layer_bytes;
  const char* B = static_cast<const char*>(args.other) + blockIdx.y * layer_bytes;
  char* O = FUSE ? static_cast<char*>(args.h_out_w) + blockIdx.y * layer_bytes : nullptr;
  const ImpShare mine = imp_share<!FUSE>(args, wave, ROWS);
  double cosines = 0.0;
  float k_ab = 0.f, k_aa = 0.f, k_bb = 0.f;      // the sums of the row that this lane keeps
  int kept = 0;                                  // rows kept per lane group
  auto flush = [&]() {                           // (a lane without a row has zeros: it adds 0)
    const double na = fmax(sqrt((double)k_aa), 1e-8), nb = fmax(sqrt((double)k_bb), 1e-8);
    cosines += (double)k_ab / (na * nb);
    k_ab = k_aa = k_bb = 0.f;
    kept = 0;
  };
  for (int64_t row0 = mine.row; row0 < mine.hi; row0 += mine.step) {
    const int there = (int)min(mine.hi - row0, (int64_t)ROWS);      // rows of this turn
    uint4 x[4], y[4];
    uint32_t off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {                // (beyond the last row or piece: that one again, counted as zeros)
      off[i] = (uint32_t)min(i * SIDE + side, there - 1) * (uint32_t)row_bytes + min(lw, chunks - 1) * 16u;
      x[i] = ld16_nt(A + row0 * row_bytes + off[i]);
      y[i] = ld16_nt(B + row0 * row_bytes + off[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool own = i * SIDE + side < there && lw < chunks;
      if (FUSE) {
        y[i] = Residual<T>::add(x[i], y[i]);
        char* o = O + row0 * row_bytes + off[i];
        if (own) { if constexpr (NT) st16_nt(o, y[i]); else st16(o, y[i]); }
      }
      if (!own) x[i] = y[i] = make_uint4(0, 0, 0, 0);
      float ab = 0.f, aa = 0.f, bb = 0.f;
      Dots<T>::acc(x[i], y[i], ab, aa, bb);
      ab = lanes_sum<W>(ab); aa = lanes_sum<W>(aa); bb = lanes_sum<W>(bb);
      if (lw == kept) { k_ab = ab; k_aa = aa; k_bb = bb; }
      if (++kept == W) flush();
    }
  }
  if (kept > 0) flush();
  __shared__ double s_part[kImpWaves];
  cosines = wave_sum(cosines);
  if (lane == 0) s_part[wave] = cosines;
  __syncthreads();
  if (threadIdx.x == 0) imp_put(args, mine.seq, s_part);
}

// one workgroup per (sequence, layer).  All of its partial sums are requested
// at once and added in a fixed order (one wave that took 16 turns for 1024 of them: 5.8 us; 16384 rows of 4096 bf16
// in one layer, both kernels: 45.9 -> 42.3 us, inside the residual add 71.5 -> 68.0).  64 threads for up to 256.
// (The last workgroup to arrive adding them instead was slower: its round trips -- stores acknowledged, arrivals counted, sums
// fetched -- take longer than a launch: 2048 rows of 4096 13.4 -> 17.2, 300 8.8 -> 11.0.)
template <bool SEQS /*pieces of several sequences, see imp_share*/>
__global__ __launch_bounds__(kImpThreads) void importance_final_kernel(const ImpArgs a, int per_layer /*partial sums*/) {
  const int seq = SEQS ? blockIdx.x : 0, layer = blockIdx.y;
  const int lane = threadIdx.x & (SQA_WAVE - 1);
  int64_t lo = 0, hi = 0;
  int first = 0, n = per_layer;
  if constexpr (SEQS) {
    imp_rows(a, seq, lo, hi);
    first = min((int)(lo >> a.piece) + seq, per_layer - 1);
    n = hi > lo ? (int)(((hi - 1) >> a.piece) - (lo >> a.piece)) + 1 : 0;
  }
  constexpr int N = SEQS ? 8 : 4;                 // >= n / threads
  double v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int at = threadIdx.x + i * blockDim.x;
    v[i] = 0.0;
    if (SEQS && i >= N / 2 && n <= (int)blockDim.x * (N / 2)) continue;
    v[i] = a.partial[(int64_t)layer * per_layer + first + max(min(at, n - 1), 0)];
    v[i] = at < n ? v[i] : 0.0;
  }
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < N; ++i) s += v[i];
  s = wave_sum(s);
  if (blockDim.x > SQA_WAVE) {
    __shared__ double s_wave[kImpWaves];
    if (lane == 0) s_wave[threadIdx.x / SQA_WAVE] = s;
    __syncthreads();
    s = 0.0;
    for (int w = 0; w < kImpWaves; ++w) s += s_wave[w];
  }
  if (threadIdx.x == 0) {
    if (!SEQS) imp_rows(a, 0, lo, hi);
    imp_store(a, (int64_t)layer * a.n_seq + seq, hi - lo, s);
  }
}

static int imp_blocks(int64_t n_tokens) {
  int64_t b = (n_tokens + kImpWaves - 1) / kImpWaves;
  return (int)(b < kImpMaxBlocks ? b : kImpMaxBlocks);
}

}  // namespace sqa

extern "C" size_t sqa_layer_importance_workspace_bytes(int n_layers, int64_t n_tokens, int hidden) {
  (void)hidden;
  if (n_layers < 1 || n_tokens < 1) return 0;
  return (size_t)n_layers * sqa::imp_blocks(n_tokens) * sizeof(double);
}

namespace sqa {
static sqa_status launch_importance(const void* h_in, const void* other, void* h_out_w, sqa_dtype dt,
                                    int n_layers, int64_t n_tokens, int hidden, const int32_t* seq_start, int n_seq,
                                    float* cos_out, void* workspace, size_t ws_bytes, void* stream) {
  const bool fuse = h_out_w != nullptr;
  if (!h_in || !other || !cos_out || !workspace) return SQA_ERR_NULL;
  if (dt != SQA_F32 && dt != SQA_BF16) return SQA_ERR_DTYPE;
  if (n_layers < 1 || n_layers > 65535 || n_tokens < 1 || hidden < 8 || hidden % 8 != 0) return SQA_ERR_SHAPE;
  if (n_seq < 1 || n_seq > 65535 || (int64_t)n_layers * n_seq > INT32_MAX) return SQA_ERR_SHAPE;
  if (!aligned16(h_in) || !aligned16(other) || !aligned16(h_out_w) || (reinterpret_cast<uintptr_t>(workspace) & 7u))
    return SQA_ERR_SHAPE;
  if (ws_bytes < (size_t)n_seq * sqa_layer_importance_workspace_bytes(n_layers, n_tokens, hidden)) return SQA_ERR_CAPACITY;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int pieces = hidden / (dt == SQA_F32 ? 4 : 8);
  const int rows = pieces <= 32 ? 8 : (pieces <= 64 ? 4 : 1);      // of a wave at a time
  int nblk = imp_blocks((n_tokens + rows - 1) / rows);
  // (one workgroup, or one per sequence, needs no second kernel: 23 layers of 20 rows of 256 bf16 9.2 -> 6.0 us)
  int piece = nblk <= 3 && (nblk - 1) * pieces <= kImpOnePieces ? kImpWhole : kImpAll;
  if (piece == kImpWhole) {
    nblk = n_seq;
  } else if (n_seq > 1) {
    for (piece = 0; (1 << piece) < kImpWaves * rows || (n_tokens - 1) >> piece >= kImpMaxPieces - 1; ++piece) {}
    nblk = (int)((n_tokens - 1) >> piece) + n_seq;
  }
  ImpArgs a;
  a.h_in = h_in; a.other = other; a.h_out_w = h_out_w;
  a.n_tokens = n_tokens; a.hidden = hidden; a.seq_start = seq_start;
  a.n_seq = n_seq; a.piece = piece;
  a.partial = static_cast<double*>(workspace);
  a.cos_out = cos_out;
  const dim3 grid(nblk, n_layers);
  // h_out is stored non-temporally where it is larger than the 256 MB Infinity Cache: nothing of it would be found
  // there again (16 layers of 4096 x 4096 bf16, 537 MB: 304 us, 285 so); below that plain stores are absorbed by the
  // cache and found by the next kernel (16384 x 4096, 134 MB: 68 us, 74 so.  From inputs that lie in memory 79 and 75, but
  // with a norm of h_out after it 132 and 151).
  const bool nt = fuse && (int64_t)n_layers * n_tokens * hidden * (dt == SQA_F32 ? 4 : 2) >= ((int64_t)256 << 20);
  auto launch = [&](auto type, auto fused, auto streamed) {
    using T = decltype(type);
    constexpr bool F = decltype(fused)::value, N = decltype(streamed)::value;
    if (rows == 8) importance_short_rows_kernel<T, F, N, 32><<<grid, kImpThreads, 0, st>>>(a);
    else if (rows == 4) importance_short_rows_kernel<T, F, N, 64><<<grid, kImpThreads, 0, st>>>(a);
    else importance_partial_kernel<T, F, N><<<grid, kImpThreads, 0, st>>>(a);
  };
  auto pick = [&](auto type) {
    if (nt) launch(type, std::true_type{}, std::true_type{});
    else if (fuse) launch(type, std::true_type{}, std::false_type{});
    else launch(type, std::false_type{}, std::false_type{});
  };
  if (dt == SQA_F32) pick(float{}); else pick(bf16_t{});
  SQA_HIP_CHECK(hipGetLastError());
  static_assert(kImpMaxPieces <= 8 * kImpThreads, "partial sums per thread of the final kernel");
  if (piece != kImpWhole) {
    const int most = nblk - (n_seq - 1);          // partial sums of a sequence
    const dim3 items(n_seq, n_layers);
    const int threads = most <= 4 * SQA_WAVE ? SQA_WAVE : kImpThreads;
    if (piece == kImpAll) importance_final_kernel<false><<<items, threads, 0, st>>>(a, nblk);
    else importance_final_kernel<true><<<items, threads, 0, st>>>(a, nblk);
  }
  SQA_HIP_CHECK(hipGetLastError());
  return SQA_OK;
}
}  // namespace sqa

extern "C" sqa_status sqa_layer_importance(const void* h_in, const void* h_out, sqa_dtype dt,
                                           int n_layers, int64_t n_tokens, int hidden,
                                           float* cos_out, void* workspace, size_t ws_bytes, void* stream) {
  return sqa::launch_importance(h_in, h_out, nullptr, dt, n_layers, n_tokens, hidden, nullptr, 1, cos_out, workspace,
                                ws_bytes, stream);
}

extern "C" sqa_status sqa_layer_importance_seq(const void* h_in, const void* h_out, sqa_dtype dt,
                                               int n_layers, int64_t n_tokens, int hidden,
                                               const int32_t* seq_start, int n_seq,
                                               float* cos_out, void* workspace, size_t ws_bytes, void* stream) {
  if (!seq_start) return SQA_ERR_NULL;
  return sqa::launch_importance(h_in, h_out, nullptr, dt, n_layers, n_tokens, hidden, seq_start, n_seq, cos_out,
                                workspace, ws_bytes, stream);
}

extern "C" sqa_status sqa_residual_add_importance(const void* h_in, const void* attn_out, void* h_out, sqa_dtype dt,
                                                  int n_layers, int64_t n_tokens, int hidden,
                                                  float* cos_out, void* workspace, size_t ws_bytes, void* stream) {
  if (!h_out) return SQA_ERR_NULL;
  return sqa::launch_importance(h_in, attn_out, h_out, dt, n_layers, n_tokens, hidden, nullptr, 1, cos_out, workspace,
                                ws_bytes, stream);
}

// prefix_prefill_attn for the shapes the work-list kernels (prefill_attn.hip) do not cover: fp32, head_dim 64, group sizes
// that are no power of two, blocks of fewer than 16 tokens.
#include "attn_lanes.h"

namespace symph {

struct RowsParams {
  const void* k_layer;
  const void* v_layer;
  int64_t block_stride;
  int32_t n_blocks, block_size, bs_shift, n_kv_heads, n_q_heads;  // bs_shift: log2(block_size) or -1
  const void* q;
  const void* k_new;
  const void* v_new;
  void* out;
  const int32_t* cu_new_lens;
  const int32_t* prefix_lens;
  const int32_t* table;
  int32_t table_stride, n_sessions, total_new_tokens;
  float scale;
  uint32_t group_bytes;  // bytes between blocks where 16 consecutive keys lie in one block (a power of two >= 16 of tokens)
                         // and a block fits 32 bits; else 0
};

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(__bf16 x) { return (float)x; }
__device__ __forceinline__ void from_f32(float* p, float x) { *p = x; }
__device__ __forceinline__ void from_f32(__bf16* p, float x) { *p = (__bf16)x; }

// ---- one wave per (token, query head), lanes over keys, fp32 throughout.  q_s: 2 * D floats in LDS of the wave's own (q, the
// result).  CH output columns at a time (the scores are worked out again for each: where registers matter more than time).
template <typename T, int D, int CH>
__device__ __forceinline__ void row_by_lanes(const RowsParams& p, int32_t s, int32_t tok, int32_t h, float* q_s) {
  const int lane = threadIdx.x & 63;
  const int32_t cu_s = p.cu_new_lens[s];
  const int32_t i = tok - cu_s;
  const int32_t P = p.prefix_lens[s];
  const int32_t G = p.n_q_heads / p.n_kv_heads;
  const int32_t g = h / G;
  const int32_t n_keys = P + i + 1;

  const T* q = (const T*)p.q + ((int64_t)tok * p.n_q_heads + h) * D;
  for (int c = lane; c < D; c += 64) q_s[c] = to_f32(q[c]);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  T* out = (T*)p.out + ((int64_t)tok * p.n_q_heads + h) * D;

  for (int c0 = 0; c0 < D; c0 += CH) {
    float m = -INFINITY, l = 0.f;
    float acc[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[c] = 0.f;

    for (int32_t j = lane; j < n_keys; j += 64) {
      const T* kp = nullptr;  // a block id outside the cache names a row of zeros (score 0, value 0), as in the other kernels
      const T* vp = nullptr;
      if (j < P) {
        const int32_t jb = j / p.block_size;
        const int32_t b = jb < p.table_stride ? p.table[(int64_t)s * p.table_stride + jb] : -1;
        if (b >= 0 && b < p.n_blocks) {
          const int64_t e = (int64_t)b * p.block_stride + ((int64_t)(j - jb * p.block_size) * p.n_kv_heads + g) * D;
          kp = (const T*)p.k_layer + e;
          vp = (const T*)p.v_layer + e;
        }
      } else {
        const int64_t e = ((int64_t)(cu_s + j - P) * p.n_kv_heads + g) * D;
        kp = (const T*)p.k_new + e;
        vp = (const T*)p.v_new + e;
      }
      float dot = 0.f;
      if (kp) {
#pragma unroll 8
        for (int c = 0; c < D; ++c) dot = fmaf(q_s[c], to_f32(kp[c]), dot);
      }
      const float x = p.scale * dot;
      const float m_new = fmaxf(m, x);
      const float alpha = expf(m - m_new);  // m = -inf on the first key: alpha = 0
      const float w = expf(x - m_new);
      l = l * alpha + w;
      if (vp) {
#pragma unroll
        for (int c = 0; c < CH; ++c) acc[c] = fmaf(w, to_f32(vp[c0 + c]), acc[c] * alpha);
      } else {
#pragma unroll
        for (int c = 0; c < CH; ++c) acc[c] *= alpha;
      }
      m = m_new;
    }

    // merge the 64 per-lane partial softmaxes
    float M = m;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) M = fmaxf(M, __shfl_xor(M, o));
    const float f = (m == -INFINITY) ? 0.f : expf(m - M);
    float lt = l * f;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) lt += __shfl_xor(lt, o);
    const float inv = lt > 0.f ? 1.0f / lt : 0.f;  // (every row sees at least itself, so the sum is positive)
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      float a = acc[c] * f;
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) a += __shfl_xor(a, o);
      if (lane == 0) q_s[D + c0 + c] = a * inv;  // (a store by lane c each would keep CH lane masks in scalar registers)
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int c = lane; c < D; c += 64) from_f32(out + c, q_s[D + c]);
}

// Addresses that the tiled kernel below cannot load 16 bytes wide from.
template <typename T, int D>
__global__ __launch_bounds__(64) void attn_row_kernel(const RowsParams p) {
  __shared__ float q_s[2 * D];
  const int64_t row = blockIdx.x;  // (token, head)
  const int32_t tok = (int32_t)(row / p.n_q_heads);
  int32_t lo = 0, hi = p.n_sessions;  // session with cu[s] <= tok < cu[s+1]
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (p.cu_new_lens[mid] <= tok)
      lo = mid;
    else
      hi = mid;
  }
  row_by_lanes<T, D, D>(p, lo, tok, (int32_t)(row % p.n_q_heads), q_s);
}

// ---- the tiled kernel: one workgroup per (session, kv-head, tile of R query rows).  The rows of a kv-head, token by
// token and the G heads of a token beside each other (any G), are cut into tiles of R = 32 (bf16) or 16 (fp32); the W
// waves of a workgroup take the tile's key blocks of R keys in turn, each with a softmax of its own, and are combined
// through LDS at the end.  No scheduling kernel, no workspace, one launch: these shapes are small models and odd group
// sizes, whose calls are short, so what counts is how few trips to memory stand one behind the other.
//
// What is held in 32 bits: probabilities too.  The bf16 kernel splits them into three bf16 values whose sum is the 32-bit
// value (8 bits of the 24 each, taken from the top: two instructions a part and one for two values of an operand; with
// conversions that round it was three, and the first call below took 18.3 instead of 17.3 us) and multiplies V with all three,
// which leaves the rounding of the output and the 32-bit sums as the only ones; the fp32 kernel uses the fp32 matrix instruction
// throughout.  (Two values, 2^-17, were 6 to 13 % faster on full chips and rounded ten times as many outputs to the other
// neighbour of the 64-bit result: 1.7e-3 of them for 1.1e-4 to 1.7e-4.)
//
// Measured against one wave per row (attn_row_kernel above, 32-bit arithmetic on the vector unit, lanes over keys): six
// sessions of 300 to 2000 tokens, 64-wide heads, 380 -> 17.7 us; one fp32 session of 256 tokens, 24.7 -> 8.7; 16 new tokens of
// three fp32 sessions of 8192, eight heads on two kv-heads, 385 -> 109 with 64-wide heads and 798 -> 185 with 128-wide ones;
// 100 new tokens of eight sessions of 2000 with 64-wide heads, 1921 -> 51.  The error against 64 bits is the same in bf16 and
// lower in fp32 (2.9e-7 for 4.7e-7 at 128 x 8000 keys).  A small call is a chain load -> product -> softmax -> product, and a
// full chip counts instructions of the vector unit: about 1000 of its clocks per 32-key block, 500 of the matrix
// cores'.  Tried and not kept: two key blocks per turn (as fast at best, fp32 slower), the next block's first product in front
// of this one's exponentials (17 -> 23 us), twelve or six waves a tile (17 -> 21), block ids asked for without a branch (the
// compiler waits for them at once: 17 -> 23).
//
// K goes from memory straight into operand registers: a row's D values are the operand's contraction index, and any order
// of it will do as long as Q has the same.  V is needed transposed: in bf16 through LDS (a tile of the wave's own, rows
// 64 bytes apart in banks so that the transposing read has no conflicts), in fp32 not at all (its operand has one value
// per lane).  The next block's rows are asked for before the present one is used, the block ids one block earlier.
static __device__ __attribute__((aligned(256))) const unsigned kAbsentRow[128] = {};  // a head's row of zeros

template <typename T>
struct RowsTile;
template <>
struct RowsTile<__bf16> {
  static constexpr int R = 32;
};
template <>
struct RowsTile<float> {
  static constexpr int R = 16;
};

// Last index i of [0, n) with holds(i), for a predicate that holds up to some index and not after it (holds(0) is taken for
// granted): 64 lanes at once, one trip to memory for up to 64 sessions, two for 4096.
template <typename F>
__device__ __forceinline__ int wave_last(int n, F holds) {
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) >> 6;
    const int i = lo + lane * step;
    const int k = __popcll(__ballot(lane == 0 || (i < hi && holds(i)))) - 1;
    lo += k * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

// The W waves' results of a tile of R rows through LDS: out = sum_w f_w O_w / sum_w f_w l_w with f_w = e^(m_w - max_w m_w)
// (base 2 or e, as the caller's references are); wave_m has been written.  put(f, mine) writes the lane's part of the wave's
// columns, scaled.  A row with a result that is not finite (an infinity or a NaN among the inputs, which the matrix product
// spreads over rows that must not see its key) is worked out again by itself.  Its q is read again for that, so it is not
// written before: out may be q.
template <typename T, int D, int R, int W, typename Put, typename Exp>
__device__ __forceinline__ void combine_rows(const RowsParams& p, char* lds, const float (*wave_m)[R], float (*wave_l)[R],
                                             float l_row, unsigned& bad_rows, Put put, Exp exp_of, int s, int cu_s, int kvh,
                                             int G, unsigned row0, int n_rows) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int kStride = D + 4;  // floats between rows (the padding spreads them over the banks)
  float* const all = reinterpret_cast<float*>(lds);
  const int n = lane & (R - 1);
  float M = -INFINITY;
#pragma unroll
  for (int w = 0; w < W; ++w) M = fmaxf(M, wave_m[w][n]);
  const float mine_m = wave_m[wave][n];
  const float f = mine_m == -INFINITY ? 0.f : exp_of(mine_m - M);
  if (lane < R) wave_l[wave][n] = mine_m == -INFINITY ? 0.f : l_row * f;
  put(f, all + wave * R * kStride);
  __syncthreads();
  // a thread adds up four columns of a row at a time
  constexpr int kQuads = R * D / 4, kTurns = (kQuads + 64 * W - 1) / (64 * W);
  typedef T vec __attribute__((ext_vector_type(4)));
  vec x[kTurns];
#pragma unroll
  for (int t = 0; t < kTurns; ++t) {
    const int i = tid + t * 64 * W, r = i / (D / 4), c0 = 4 * (i % (D / 4));
    if (kQuads % (64 * W) != 0 && i >= kQuads) break;
    float L = 0.f;
    f32x4 sum{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < W; ++w) {
      L += wave_l[w][r];
      sum += *reinterpret_cast<const f32x4*>(all + (w * R + r) * kStride + c0);
    }
    const float inv = 1.0f / L;
    bool bad = false;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      bad = bad || !(fabsf(sum[v] * inv) < INFINITY);
      x[t][v] = (T)(sum[v] * inv);
    }
    // (a sum that is NaN comes from a score that is: every value of the row is NaN, worked out either way)
    if (bad && L == L && r < n_rows) atomicOr(&bad_rows, 1u << r);
  }
  __syncthreads();
  const unsigned again = __builtin_amdgcn_readfirstlane(bad_rows);
#pragma unroll
  for (int t = 0; t < kTurns; ++t) {
    const int i = tid + t * 64 * W, r = i / (D / 4), c0 = 4 * (i % (D / 4));
    if (i < kQuads && r < n_rows && !((again >> r) & 1)) {
      const unsigned row = row0 + r, tok = row / (unsigned)G;
      T* const op = (T*)p.out + ((int64_t)(cu_s + (int)tok) * p.n_q_heads + kvh * G + (int)(row - tok * G)) * D;
      *reinterpret_cast<vec*>(op + c0) = x[t];
    }
  }
  int turn = 0;
  for (unsigned left = again; left; left &= left - 1) {
    if (turn++ % W != wave) continue;
    const unsigned row = row0 + __builtin_ctz(left), tok = row / (unsigned)G;
    row_by_lanes<T, D, 64>(p, s, cu_s + (int)tok, kvh * G + (int)(row - tok * G), all + wave * 2 * D);
  }
}

// The part of a float that a bf16 value holds without rounding, and two such parts as neighbours of an operand
__device__ __forceinline__ float leading_bits(float x) {
  return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, x) & 0xFFFF0000u);
}
__device__ __forceinline__ void put_upper_halves(bf16x8& v, int at, float x, float y) {
  u32x4 words = __builtin_bit_cast(u32x4, v);
  words[at >> 1] = __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, y), __builtin_bit_cast(unsigned, x), 0x07060302u);
  v = __builtin_bit_cast(bf16x8, words);
}

template <typename T, int D, int W, bool EARLY>
__global__ __launch_bounds__(64 * W, 2) void attn_rows_kernel(const RowsParams p) {
  constexpr bool kBf16 = sizeof(T) == 2;
  constexpr int R = RowsTile<T>::R;
  constexpr int kVRow = D * 2 + 64;                                  // bytes between V rows in LDS (bf16)
  constexpr int kVBytes = kBf16 ? W * 32 * kVRow : 0;
  constexpr int kCombBytes = W * R * (D + 4) * 4;
  __shared__ __attribute__((aligned(16))) char lds[kVBytes > kCombBytes ? kVBytes : kCombBytes];
  __shared__ float wave_m[W][R], wave_l[W][R];
  __shared__ unsigned bad_rows;

  const int Hkv = p.n_kv_heads;
  const int G = p.n_q_heads / Hkv;
  const int kvh = blockIdx.x % Hkv;
  const int slot = blockIdx.x / Hkv;
  // Session s has the tile slots from floor(cu[s] * G / R) + s on: at least as many as it has tiles, without a list
  auto first_slot = [&](int s, int cu) { return (int)((int64_t)cu * G / R) + s; };
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & (R - 1);   // query row of this lane; also its row of the K operand
  const int kg = lane / R;        // its share of the contraction index: half (bf16) or quarter (fp32) of the wave
  auto block_of = [&](int key) { return p.bs_shift >= 0 ? key >> p.bs_shift : key / p.block_size; };
  // EARLY: a single fp32 session.  Its row of the table needs no lengths to be found: the block ids of the wave's first two key
  // blocks are asked for beside them, one trip to memory less in front of the first K rows.  (Whether the keys exist is seen
  // later; an index past the row's end reads its last entry.)  One session of 256 tokens 9.26 -> 8.70 us, of 1000 with 128-wide
  // heads 31.6 -> 31.3; bf16, whose first block waits for two ids per lane group, 7.60 -> 7.71: not there.  An instantiation of
  // its own: as a branch in every call it made three sessions of 256 tokens 9.35 -> 9.60.
  int early_id[2];
  if constexpr (EARLY) {
#pragma unroll
    for (int i = 0; i < 2; ++i) early_id[i] = p.table[(unsigned)min(block_of((wave + i * W) * R + n), p.table_stride - 1)];
  }
  int s, cu_s, cu_next, P;
  if (!EARLY && p.n_sessions > 1 && p.n_sessions <= 64) {
    // a session per lane: one trip to memory for all there is to know of it
    const int i = min(lane, p.n_sessions - 1);
    const int cu_i = p.cu_new_lens[i], next_i = p.cu_new_lens[i + 1], P_i = p.prefix_lens[i];
    s = __popcll(__ballot(lane < p.n_sessions && (lane == 0 || first_slot(lane, cu_i) <= slot))) - 1;
    cu_s = __builtin_amdgcn_readlane(cu_i, s);
    cu_next = __builtin_amdgcn_readlane(next_i, s);
    P = __builtin_amdgcn_readlane(P_i, s);
  } else {
    s = EARLY ? 0 : wave_last(p.n_sessions, [&](int i) { return first_slot(i, p.cu_new_lens[i]) <= slot; });
    cu_s = p.cu_new_lens[s];
    cu_next = p.cu_new_lens[s + 1];
    P = p.prefix_lens[s];
  }
  const int N = max(min(cu_next, p.total_new_tokens) - cu_s, 0);  // (rows past total_new_tokens do not exist)
  // (rows of a kv-head fit 31 bits: the host has checked all heads' rows)
  const int64_t row0_64 = (int64_t)(slot - first_slot(s, cu_s)) * R;
  if (row0_64 >= (int64_t)N * G) return;
  const unsigned row0 = (unsigned)row0_64, rows = (unsigned)N * (unsigned)G;
  const int n_rows = (int)min((unsigned)R, rows - row0);

  const unsigned my_row = row0 + min(n, n_rows - 1);
  const int tok = (int)(my_row / (unsigned)G);
  const int limit = P + tok;      // last key this row may see
  const int total_keys = P + N;
  const int n_blocks_k = (P + (int)((row0 + n_rows - 1) / (unsigned)G) + R) / R;  // key blocks up to the last row's limit
  const T* const qp =
      (const T*)p.q + ((int64_t)(cu_s + tok) * p.n_q_heads + kvh * G + (int)(my_row - (unsigned)tok * G)) * D;
  if (tid == 0) bad_rows = 0;

  // ---- rows of K and V: block ids are read one per lane (lane i: key i of the block) and passed between lanes
  const int32_t* const table_row = p.table + (int64_t)s * p.table_stride;
  auto fetch_id = [&](int blk) {
    const int key = blk * R + n;
    const int j = block_of(key);
    return blk < n_blocks_k && key < P && j < p.table_stride ? table_row[j] : -1;
  };
  auto first_id = [&](int i) {  // of the wave's block i (0 or 1)
    const int blk = wave + i * W, key = blk * R + n;
    if constexpr (!EARLY) return fetch_id(blk);
    return blk < n_blocks_k && key < P && block_of(key) < p.table_stride ? early_id[i] : -1;
  };
  auto row_of = [&](const void* pool, const void* fresh, int key, int id) {
    if (key < P) {
      if (id < 0 || id >= p.n_blocks) return (const T*)kAbsentRow;
      return (const T*)pool + (int64_t)id * p.block_stride +
             ((int64_t)(key - block_of(key) * p.block_size) * Hkv + kvh) * D;
    }
    return key < total_keys ? (const T*)fresh + ((int64_t)(cu_s + key - P) * Hkv + kvh) * D : (const T*)kAbsentRow;
  };

  // A block of keys that lies in the prefix, its 16-key groups in blocks of the cache each (block sizes that are powers of
  // two >= 16): a group's rows start at a scalar address and a lane adds a constant.  (The general form, row_of per lane, is
  // half of the vector instructions of an iteration.)
  const bool grouped = p.group_bytes != 0;
  auto group_id = [&](int id, int g) { return __builtin_amdgcn_readlane(id, 16 * g); };
  auto in_cache = [&](int id) { return (unsigned)id < (unsigned)p.n_blocks; };
  const unsigned row_bytes = (unsigned)(Hkv * D * (int)sizeof(T));  // between the rows of consecutive keys
  // Place of `key`, a multiple of 16, in the pool of this kv-head.  (A block fits 32 bits here: two multiplications.  A wave
  // that has its SIMD to itself issues an instruction every five to six clocks, address work included.)
  auto group_off = [&](int key, int id) {
    return (uint64_t)(unsigned)id * p.group_bytes + (unsigned)(key & (p.block_size - 1)) * row_bytes;
  };
  // 16 bytes of global memory (a pointer that the compiler cannot place is loaded from by an instruction that counts among the
  // LDS reads too); at a scalar base and a lane's 32-bit offset, kept apart for the compiler, which otherwise adds them per lane
  // (fp32 with 64 columns is 1 to 3 % faster when it does, 128 columns 9 % slower)
  auto load_vec = [](const void* at) { return *(const u32x4 __attribute__((address_space(1)))*)(uintptr_t)at; };
  auto load16 = [&](const char* base, unsigned lane_off) {
    if constexpr (kBf16 || D == 128) asm("" : "+s"(base), "+v"(lane_off));
    return load_vec(base + lane_off);
  };
  const char* const k_head = (const char*)((const T*)p.k_layer + kvh * D);
  const char* const v_head = (const char*)((const T*)p.v_layer + kvh * D);

  if constexpr (kBf16) {
    constexpr int NS = D / 16;            // contraction steps of the first product
    constexpr int NT = D / 32;            // 32-column tiles of the output
    constexpr int LPR = D / 8, RPI = 64 / LPR, NV = 32 / RPI;  // lanes per V row, rows per load, loads
    char* const v_lds = lds + wave * 32 * kVRow;
    bf16x8 q[NS];
#pragma unroll
    for (int st = 0; st < NS; ++st) q[st] = *reinterpret_cast<const bf16x8*>(qp + 16 * st + 8 * kg);
    const int krow = key_of_row(n);
    const int vlane_row = lane / LPR, vlane_col = (lane % LPR) * 16;
    bf16x8 kr[NS];
    u32x4 vr[NV];
    const unsigned k_off = (krow & 15) * row_bytes + 16 * kg;
    unsigned v_off_mem[NV / 2];
#pragma unroll
    for (int i = 0; i < NV / 2; ++i) v_off_mem[i] = (unsigned)(i * RPI + vlane_row) * row_bytes + vlane_col;
    auto load_block = [&](int blk, int id) {
      const int id0 = group_id(id, 0), id1 = group_id(id, 1);
      if (grouped && (blk + 1) * 32 <= P && in_cache(id0) && in_cache(id1)) {
        const uint64_t off0 = group_off(blk * 32, id0), off1 = group_off(blk * 32 + 16, id1);
        const char* const k_row = k_head + (krow < 16 ? off0 : off1) + k_off;
#pragma unroll
        for (int st = 0; st < NS; ++st) kr[st] = __builtin_bit_cast(bf16x8, load_vec(k_row + 32 * st));
        const char* const v0 = v_head + off0;
        const char* const v1 = v_head + off1;
#pragma unroll
        for (int i = 0; i < NV; ++i) vr[i] = load16(i < NV / 2 ? v0 : v1, v_off_mem[i % (NV / 2)]);
        return;
      }
      const T* const k_row = row_of(p.k_layer, p.k_new, blk * 32 + krow, __shfl(id, krow)) + 8 * kg;
#pragma unroll
      for (int st = 0; st < NS; ++st) kr[st] = __builtin_bit_cast(bf16x8, load_vec(k_row + 16 * st));
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int r = i * RPI + vlane_row;
        const T* const v_row = row_of(p.v_layer, p.v_new, blk * 32 + r, __shfl(id, r));
        vr[i] = load_vec(reinterpret_cast<const char*>(v_row) + vlane_col);
      }
    };
    const int i16 = lane & 15;
    const int v_off = (8 * kg + (i16 >> 2)) * kVRow + 32 * ((lane >> 4) & 1) + 8 * (i16 & 3);
    const float cs = p.scale * 1.4426950408889634f;
    f32x16 o[NT];
#pragma unroll
    for (int dt = 0; dt < NT; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
    float m = -INFINITY, l = 0.f;  // in log2 units
    int id_next = first_id(0);
    if (wave < n_blocks_k) load_block(wave, id_next);
    id_next = first_id(1);
    for (int blk = wave; blk < n_blocks_k; blk += W) {
      f32x16 x;
#pragma unroll
      for (int e = 0; e < 16; ++e) x[e] = 0.f;
#pragma unroll
      for (int st = 0; st < NS; ++st) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kr[st], q[st], x, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < NV; ++i)
        *reinterpret_cast<u32x4*>(v_lds + (i * RPI + vlane_row) * kVRow + vlane_col) = vr[i];
      if (blk + W < n_blocks_k) load_block(blk + W, id_next);
      id_next = fetch_id(blk + 2 * W);
      if (blk * 32 + 31 > P) {
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (blk * 32 + 16 * (e >> 3) + 8 * kg + (e & 7) > limit) x[e] = -INFINITY;
      }
      float mx = x[0];
#pragma unroll
      for (int e = 1; e < 16; ++e) mx = fmaxf(mx, x[e]);
      const float m_new = fmaxf(m, max_across_halves(mx) * cs);
      if (__any(m_new > m)) {
        const float a = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - m_new);
        m = m_new;
        l *= a;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt)
#pragma unroll
          for (int e = 0; e < 16; ++e) o[dt][e] *= a;
      }
      const float ref = m == -INFINITY ? 0.f : m;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // (here, so that V operands can be read beside the exponentials)
      __builtin_amdgcn_wave_barrier();
      // the probabilities, 8 bits each: w = hi + mid + lo, each part the leading bits of what the ones before leave (no
      // rounding: one instruction takes the upper halves of two floats)
      bf16x8 hi[2], mid[2], lo[2];
      float sum = 0.f;
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        float w[2], rest[2], last[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          w[k] = __builtin_amdgcn_exp2f(fmaf(x[e + k], cs, -ref));
          sum += w[k];
          rest[k] = w[k] - leading_bits(w[k]);
          last[k] = rest[k] - leading_bits(rest[k]);
        }
        put_upper_halves(hi[e >> 3], e & 7, w[0], w[1]);
        put_upper_halves(mid[e >> 3], e & 7, rest[0], rest[1]);
        put_upper_halves(lo[e >> 3], e & 7, last[0], last[1]);
      }
      l += sum;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int dt = 0; dt < NT; ++dt) {
          const char* vp = v_lds + v_off + 16 * u * kVRow + 64 * dt;
          const s16x4 a0 = lds_read_tr16(reinterpret_cast<const __bf16*>(vp));
          const s16x4 a1 = lds_read_tr16(reinterpret_cast<const __bf16*>(vp + 4 * kVRow));
          const bf16x8 v = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, hi[u], o[dt], 0, 0, 0);
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, mid[u], o[dt], 0, 0, 0);
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, lo[u], o[dt], 0, 0, 0);
        }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      __builtin_amdgcn_wave_barrier();  // the tile has been read before the next one is written
    }
    const float l_row = sum_across_halves(l);
    if (kg == 0) wave_m[wave][n] = m;
    __syncthreads();  // (also: no wave reads its V tile any more, the buffer is free)
    combine_rows<T, D, R, W>(p, lds, wave_m, wave_l, l_row, bad_rows, [&](float f, float* mine) {
#pragma unroll
      for (int dt = 0; dt < NT; ++dt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *reinterpret_cast<f32x4*>(mine + n * (D + 4) + 32 * dt + 4 * kg + 8 * i) =
              f32x4{o[dt][4 * i] * f, o[dt][4 * i + 1] * f, o[dt][4 * i + 2] * f, o[dt][4 * i + 3] * f};
    }, [](float x) { return __builtin_amdgcn_exp2f(x); }, s, cu_s, kvh, G, row0, n_rows);
  } else {
    constexpr int NS = D / 16;  // 16-byte loads of a row per lane
    constexpr int NH = D / 64;  // groups of 64 output columns
    f32x4 q[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) q[j] = *reinterpret_cast<const f32x4*>(qp + 16 * j + 4 * kg);
    f32x4 kr[NS], vr[4][NH];
    const unsigned k_off = n * row_bytes + 16 * kg, v_off_mem = 4 * kg * row_bytes + 16 * n;
    auto load_block = [&](int blk, int id) {
      const int id0 = group_id(id, 0);
      if (grouped && (blk + 1) * 16 <= P && in_cache(id0)) {
        const uint64_t off = group_off(blk * 16, id0);
#pragma unroll
        for (int j = 0; j < NS; ++j) kr[j] = __builtin_bit_cast(f32x4, load16(k_head + off + 64 * j, k_off));
        const char* const v_rows = v_head + off;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int h = 0; h < NH; ++h)
            vr[e][h] = __builtin_bit_cast(f32x4, load16(v_rows + e * row_bytes + 256 * h, v_off_mem));
        return;
      }
      const T* const k_row = row_of(p.k_layer, p.k_new, blk * 16 + n, id) + 4 * kg;
#pragma unroll
      for (int j = 0; j < NS; ++j) kr[j] = __builtin_bit_cast(f32x4, load_vec(k_row + 16 * j));
#pragma unroll
      for (int e = 0; e < 4; ++e) {  // key 4 * kg + e: values 64 * h + 4 * n .. + 3 of its row
        const T* const v_row = row_of(p.v_layer, p.v_new, blk * 16 + 4 * kg + e, __shfl(id, 4 * kg + e)) + 4 * n;
#pragma unroll
        for (int h = 0; h < NH; ++h) vr[e][h] = __builtin_bit_cast(f32x4, load_vec(v_row + 64 * h));
      }
    };
    // o[h][c][e]: column 64 * h + 16 * kg + 4 * e + c of row n.  A sum over thousands of keys in one chain loses bits (6.0e-7
    // from 64 bits at 8192 keys, a lane's shorter chain in the kernel above 4.6e-7): kRun blocks are added up by themselves
    // (o_run, l_run) before they join the rest.
    constexpr int kRun = 8;
    f32x4 o[NH][4], o_run[NH][4];
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int c = 0; c < 4; ++c) o[h][c] = o_run[h][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f, l_run = 0.f;
    auto join_run = [&]() {
      l += l_run;
      l_run = 0.f;
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          o[h][c] += o_run[h][c];
          o_run[h][c] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    int run = 0;
    // With 64 columns both ids before the first K rows: one that is still under way when the loop begins makes the compiler
    // wait in every turn for all that is under way (six sessions of 300 to 2000 tokens 33.0 -> 30.9 us, three of 8192 116.8 ->
    // 109.4, three of 256 9.31 -> 8.98).  With 128 columns that is slower (three of 8192 184.9 -> 187.0, one of 256 to 4000 the
    // same), and where the ids are early nothing is under way.
    constexpr bool kBothIds = D == 64 && !EARLY;
    int id_next = first_id(0);
    const int id_second = kBothIds ? first_id(1) : -1;
    if (wave < n_blocks_k) load_block(wave, id_next);
    id_next = kBothIds ? id_second : first_id(1);
    for (int blk = wave; blk < n_blocks_k; blk += W) {
      f32x4 sc[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) sc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < NS; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[j][e], q[j][e], sc[e], 0, 0, 0);
      f32x4 v[4][NH];
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int h = 0; h < NH; ++h) v[e][h] = vr[e][h];
      if (blk + W < n_blocks_k) load_block(blk + W, id_next);
      id_next = fetch_id(blk + 2 * W);
      float x[4];  // key 4 * kg + e
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[e] = p.scale * ((sc[0][e] + sc[1][e]) + (sc[2][e] + sc[3][e]));
        if (blk * 16 + 4 * kg + e > limit) x[e] = -INFINITY;
      }
      float mx = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m, mx);
      if (__any(m_new > m)) {
        const float a = m == -INFINITY ? 0.f : expf(m - m_new);
        m = m_new;
        l *= a;
        l_run *= a;
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            o[h][c] *= a;
            o_run[h][c] *= a;
          }
      }
      const float ref = m == -INFINITY ? 0.f : m;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float w = expf(x[e] - ref);
        l_run += w;
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
          for (int c = 0; c < 4; ++c)
            o_run[h][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e][h][c], w, o_run[h][c], 0, 0, 0);
      }
      if (++run == kRun) {
        join_run();
        run = 0;
      }
    }
    join_run();
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (kg == 0) wave_m[wave][n] = m;
    __syncthreads();
    combine_rows<T, D, R, W>(p, lds, wave_m, wave_l, l, bad_rows, [&](float f, float* mine) {
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          *reinterpret_cast<f32x4*>(mine + n * (D + 4) + 64 * h + 16 * kg + 4 * e) =
              f32x4{o[h][0][e] * f, o[h][1][e] * f, o[h][2][e] * f, o[h][3][e] * f};
    }, [](float x) { return expf(x); }, s, cu_s, kvh, G, row0, n_rows);
  }
}

// ------------------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------------------
constexpr int64_t kComputeUnits = 256;

template <typename T, int D>
static int32_t launch_rows(const AttnArgs& a, hipStream_t stream) {
  RowsParams p;
  p.k_layer = a.k_layer;
  p.v_layer = a.v_layer;
  p.block_stride = a.block_stride;
  p.n_blocks = a.n_blocks;
  p.block_size = a.block_size;
  p.bs_shift = (a.block_size & (a.block_size - 1)) == 0 ? __builtin_ctz((unsigned)a.block_size) : -1;
  p.n_kv_heads = a.n_kv_heads;
  p.n_q_heads = a.n_q_heads;
  p.q = a.q;
  p.k_new = a.k_new;
  p.v_new = a.v_new;
  p.out = a.out;
  p.cu_new_lens = a.cu_new_lens;
  p.prefix_lens = a.prefix_lens;
  p.table = a.table;
  p.table_stride = a.table_stride;
  p.n_sessions = a.n_sessions;
  p.total_new_tokens = a.total_new_tokens;
  p.scale = a.scale;
  const int64_t block_bytes = a.block_stride * (int64_t)sizeof(T);
  p.group_bytes = p.bs_shift >= 4 && block_bytes <= 0x7FFFFFFFLL ? (uint32_t)block_bytes : 0;
  const int64_t rows = (int64_t)a.total_new_tokens * a.n_q_heads;
  if (rows > 0x7FFFFFFFLL) return SYMPH_EUNSUPPORTED;
  const uintptr_t address_bits = (uintptr_t)a.k_layer | (uintptr_t)a.v_layer | (uintptr_t)a.q | (uintptr_t)a.k_new |
                                 (uintptr_t)a.v_new | (uintptr_t)a.out | (uintptr_t)(a.block_stride * (int64_t)sizeof(T));
  const int64_t slots = (rows / a.n_kv_heads) / RowsTile<T>::R + a.n_sessions;  // see first_slot in the kernel
  const int64_t groups = slots * a.n_kv_heads;
  // The tiled kernel loads 16 bytes at a time.  (A row of a head is a multiple of that, so the bases and the block stride
  // decide.)
  // Eight waves a tile give the shortest chain of key blocks to a call that does not fill the chip.  With more tiles than
  // compute units, four waves each (two or three workgroups then share a compute unit) leave a last round less empty.  Eight
  // / four waves, sessions of 1000 to 2000 tokens, bf16 with 64-wide heads: 16.5 / 20.3 us at 192 tiles, 28.4 / 24.5 at 304,
  // 39.5 / 33.8 at 552; with 128-wide heads 30.1 / 30.1, 52 / 46, 71 / 58; fp32 with 64-wide heads 33.5 / 49, 58.3 / 58.9 at
  // 344, 83 / 74 at 608; with 128-wide heads 52.5 / 62, 92.6 / 94, 135 / 138; 150 to 300 tokens: 8.8 / 8.7, 12.1 / 9.1, 17.1 /
  // 11.4 and 15.3 / 16.7, 27.6 / 23.1, 39.6 / 34.4.
  if ((address_bits & 15) == 0 && groups <= 0x7FFFFFFFLL) {
    constexpr bool kFp32 = sizeof(T) == 4;
    if (groups > kComputeUnits)
      hipLaunchKernelGGL((attn_rows_kernel<T, D, 4, false>), dim3((unsigned)groups), dim3(256), 0, stream, p);
    else if (kFp32 && a.n_sessions == 1 && a.max_prefix_len > 0)  // (a prefix: there is a table, one that may be read)
      hipLaunchKernelGGL((attn_rows_kernel<T, D, 8, kFp32>), dim3((unsigned)groups), dim3(512), 0, stream, p);
    else
      hipLaunchKernelGGL((attn_rows_kernel<T, D, 8, false>), dim3((unsigned)groups), dim3(512), 0, stream, p);
  } else
    hipLaunchKernelGGL((attn_row_kernel<T, D>), dim3((unsigned)rows), dim3(64), 0, stream, p);
  return hipGetLastError() == hipSuccess ? SYMPH_OK : SYMPH_ELAUNCH;
}

int32_t launch_rows_attn(const AttnArgs& a, hipStream_t stream) {
  if (a.dtype == SYMPH_BF16) {
    if (a.head_dim == 64) return launch_rows<__bf16, 64>(a, stream);
    if (a.head_dim == 128) return launch_rows<__bf16, 128>(a, stream);
  } else {
    if (a.head_dim == 64) return launch_rows<float, 64>(a, stream);
    if (a.head_dim == 128) return launch_rows<float, 128>(a, stream);
  }
  return SYMPH_EUNSUPPORTED;
}

}  // namespace symph

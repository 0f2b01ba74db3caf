// prefix_prefill_attn: the new turn's GQA queries against [paged cached prefix ; causal new tokens]
// (Symphony Sec. 2.1: A_h = softmax(Q_h K_h^T * scale), y = concat_h A_h V_h; a token sees all prior tokens).
//
// bf16 path (head_dim 128), one workgroup of 4 waves per (session, kv-head, tile of query tokens):
//   * the G query heads that share a kv-head are stacked into the tile (128 query rows = G heads x 128/G tokens),
//     so every K,V tile staged in LDS is reused by all of them;
//   * scores are computed TRANSPOSED, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16: the MFMA result layout then puts
//     one query per lane, so the online-softmax state (reference, running sum) is per-lane scalars, and the bf16
//     probabilities a lane holds are exactly the B operand of O^T += V^T P^T;
//   * the row order in which K rows are fed to the MFMA is permuted so that the 8 probabilities a lane needs for
//     one 16-key step of the second product are 8 consecutive keys; the matching V^T operand comes from the
//     transposing LDS read (ds_read_b64_tr_b16), V stays row-major in LDS;
//   * K,V tiles of 64 keys go from the paged pool (block-table indirection per 16-token block) or from the
//     contiguous new-turn K,V straight into LDS (global_load_lds_dwordx4), double-buffered, one tile ahead;
//   * the softmax reference is stale on purpose (refreshed only when a row sum shows that it has to be), so no
//     per-tile maximum and no per-tile rescaling of the accumulators.
// Every other shape (fp32, head_dim 64, other group sizes, smaller blocks): rows_attn.hip.
#include "attn_lanes.h"

#include <type_traits>

namespace symph {

// ------------------------------------------------------------------------------------------------------------
// bf16 MFMA path, head_dim 128
// ------------------------------------------------------------------------------------------------------------
// Work decomposition.  A "unit" is (session, tile of BMT = 128/G query tokens); its cost is the number of 64-key
// tiles it has to visit.  A scheduling kernel (one workgroup) turns the ragged batch into a list of work items:
// units longer than a chunk length C are split along the key axis into near-equal chunks (C is chosen so that the
// batch gives about `target` workgroup-sized pieces), and the items are ordered longest first, so that the
// hardware's in-order workgroup dispatch is a longest-processing-time list schedule.  Every item is executed for
// every kv-head by one workgroup: global index g -> (item g / H_kv, kv-head g % H_kv), which with 8 kv-heads also
// pins each kv-head to one XCD (workgroups are dealt round-robin to the 8 XCDs), so the query tiles of a session
// that re-read the same K,V share that XCD's L2.  Chunks of a split unit write unnormalised partial results
// (running max, running sum, accumulators) to the workspace and the last of them to arrive combines them.  Batches of few
// units are cut without that kernel (direct mode, below).
struct WorkItem {   // 96 bytes
  int32_t s, t0, tile_begin, tile_end;
  int32_t pslot;                  // < 0: whole unit, the workgroup writes the output rows itself
  int32_t cu_s, n_new, n_prefix;  // of session s, so that a workgroup starts without looking them up
  int32_t merge, pslot0, n_chunks;  // chunk of a split unit: the unit's counter, its first slot, its number of chunks
  int32_t first_ids[8];           // block ids of the eight 16-key groups of tiles tile_begin and tile_begin + 1: the
                                  // workgroup's first K,V loads wait for this item only, not for a table read as well
  int32_t pad[5];
};
struct MergeItem {  // 16 bytes, one per unit of a direct call or of the decode kernel
  int32_t row0, n_unit, pslot0, n_chunks;  // its first row of q / out and its tokens; the slot of its first piece (decode:
                                           // 2 * range + 0 / 1); n_chunks 0: nothing to combine
};
// Header of the workspace (ints): counts and flags written by the scheduler (by the attention kernel itself where none
// runs).
constexpr int kHdrItems = 0, kHdrChunk = 1, kHdrSplitUnits = 2, kHdrPslots = 3, kHdrPlan = 4, kHdrDecTiles = 5,
              kHdrFlags = kAttnHdrFlags;
constexpr int kPlanList = 0, kPlanDirect = 1, kPlanDecode = 2;  // what the call ran (kHdrPlan)
static_assert(kHdrFlags < kAttnHdrInts, "the header holds the counts and flags");
constexpr int kPartialFloats = 256 * 66;  // per workgroup: 64 accumulators + running max + running sum per thread
// A piece of a short turn (decode kernel): only the session's own rows, r = head * N + token (at most 32), packed:
// rows x 128 accumulators, then the rows' softmax references, then their sums.  Whole 128-byte lines are written and
// nothing else: a slot in the layout above would be 528 lines with 32 of their 128 bytes dirty, and writing such lines
// back cost the decode step 13 % of its time.
constexpr int kDecPartialFloats = 32 * 130;

struct SchedParams {
  const int32_t* cu_new_lens;
  const int32_t* prefix_lens;
  int32_t n_sessions, bmt, n_kv_heads, target, target_slots, c_min, coarse_ok;
  int32_t items_bound, merges_bound, pslots_bound;
  int32_t* hdr;
  WorkItem* items;
  int32_t* merge_cnt;   // [merges_bound][n_kv_heads]: chunks of a split unit that have written their partial result
  const int32_t* table; // block table (may be null) and what is needed to find the ids of an item's first tiles
  int32_t table_stride, log_bs;
};

constexpr int kBN = 64;  // keys per tile
constexpr int kSchedThreads = 256, kSchedWaves = kSchedThreads / 64;
constexpr int kSchedBuckets = 64;      // one per lane of a wave: the bucket offsets are a single wave-level scan
constexpr int kSchedMaxSessions = 4096;  // sessions whose lengths and unit offsets fit the scheduler's LDS tables

__device__ __forceinline__ int unit_tiles(int P, int N, int t0, int bmt) {
  return (P + min(N, t0 + bmt) + kBN - 1) / kBN;
}

// Inclusive scan over the 64 lanes of a wave with data-parallel moves: shifts by 1, 2, 4, 8 inside each row of 16
// lanes (a lane without a source adds 0), then the last lane of rows 0 and 2 added to rows 1 and 3, then lane 31 to
// rows 2 and 3.  (A shuffle per step goes through the LDS crossbar and takes ten times as long.)
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_from(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xF, true);
}
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += dpp_from<0x111, 0xF>(v);  // row_shr:1
  v += dpp_from<0x112, 0xF>(v);  // row_shr:2
  v += dpp_from<0x114, 0xF>(v);  // row_shr:4
  v += dpp_from<0x118, 0xF>(v);  // row_shr:8
  v += dpp_from<0x142, 0xA>(v);  // row_bcast:15
  v += dpp_from<0x143, 0xC>(v);  // row_bcast:31
  return v;
}

// Maximum over the 64 lanes of a wave of values >= 0 (the same moves as the scan; a lane without a source sees 0);
// lane 63 holds the result.
__device__ __forceinline__ int wave_inclusive_max(int v) {
  v = max(v, dpp_from<0x111, 0xF>(v));
  v = max(v, dpp_from<0x112, 0xF>(v));
  v = max(v, dpp_from<0x114, 0xF>(v));
  v = max(v, dpp_from<0x118, 0xF>(v));
  v = max(v, dpp_from<0x142, 0xA>(v));
  v = max(v, dpp_from<0x143, 0xC>(v));
  return v;
}

// Inclusive scan of two ints per thread across the scheduler's block; the block totals come back through tot_a, tot_b.
__device__ __forceinline__ void block_inclusive_scan2(int& a, int& b, int (*wave_sums)[2], int& tot_a, int& tot_b) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  a = wave_inclusive_scan(a);
  b = wave_inclusive_scan(b);
  __syncthreads();
  if (lane == 63) {
    wave_sums[w][0] = a;
    wave_sums[w][1] = b;
  }
  __syncthreads();
  const int up_to_a = wave_inclusive_scan(lane < kSchedWaves ? wave_sums[lane][0] : 0);
  const int up_to_b = wave_inclusive_scan(lane < kSchedWaves ? wave_sums[lane][1] : 0);
  tot_a = __builtin_amdgcn_readlane(up_to_a, kSchedWaves - 1);
  tot_b = __builtin_amdgcn_readlane(up_to_b, kSchedWaves - 1);
  if (w > 0) {
    a += __builtin_amdgcn_readlane(up_to_a, w - 1);
    b += __builtin_amdgcn_readlane(up_to_b, w - 1);
  }
}

// One workgroup turns the ragged batch into the ordered work list.  All passes run over the flat list of units
// (session, query tile), one unit per thread per step, so a batch of one long session is as parallel as a batch of many
// short ones.  Which units are split, and which partial-result slots and counters their chunks get, follows from
// prefix sums in unit order: the same for every run, and a unit for whose chunks the workspace has no room is simply
// left whole (flag bit 0), never dropped.
// It is a chain that one compute unit walks, 20 000 clocks for 512 units.  What a batch does not need is left out: the
// divisions, block-wide sums and counters of cuts where no unit is cut, the barrier behind the cut's length, which every wave
// works out for itself, half of the steps of the search for a unit's session: 16 500.  Calls: 16 x 78 new tokens over 99,
// 20.7 -> 19.6 us; 70 x 20..60 over 100..300, 37.0 -> 35.4; 256 x 4..30 over 16..64, 39.5 -> 38.7; long calls the same.  512
// threads are as fast, 1024 slower; two 16-byte loads for a unit's eight block ids change nothing.
__global__ __launch_bounds__(kSchedThreads) void attn_schedule_kernel(const SchedParams p) {
  __shared__ int unit_off[kSchedMaxSessions + 1];
  __shared__ int len_new[kSchedMaxSessions], len_prefix[kSchedMaxSessions], cu_of[kSchedMaxSessions];
  __shared__ int wave_sums[kSchedWaves][2];
  __shared__ unsigned long long total_tiles_s;
  __shared__ int max_nt_s, inv_min_nt_s;  // longest unit, and 0x7FFFFFFF - shortest unit (tiles; units with tiles only)
  __shared__ int hist[kSchedBuckets];
  __shared__ int n_items_s, n_split_s, n_pslot_s, flags_s;
  const int tid = threadIdx.x;
  const int S = p.n_sessions;
  if (tid == 0) {
    total_tiles_s = 0ull;
    max_nt_s = 0;
    inv_min_nt_s = 0;
    n_items_s = 0;
    n_split_s = 0;
    n_pslot_s = 0;
    flags_s = 0;
  }
  if (tid < kSchedBuckets) hist[tid] = 0;
  // unit offsets: exclusive prefix sum of ceil(N_s / bmt)
  int U = 0;
  for (int base = 0; base < S; base += kSchedThreads) {
    const int s = base + tid;
    // the lengths are read from memory once and kept in LDS for the passes below
    const int cu_s = s < S ? p.cu_new_lens[s] : 0;
    const int N = s < S ? p.cu_new_lens[s + 1] - cu_s : 0;
    const int P = s < S ? p.prefix_lens[s] : 0;
    if (s < S) {
      len_new[s] = N;
      len_prefix[s] = P;
      cu_of[s] = cu_s;
    }
    int nq = N > 0 ? (N + p.bmt - 1) / p.bmt : 0, zero = 0, tot_q, tot_z;
    block_inclusive_scan2(nq, zero, wave_sums, tot_q, tot_z);
    if (s < S) unit_off[s] = U + nq - (N > 0 ? (N + p.bmt - 1) / p.bmt : 0);
    U += tot_q;
  }
  if (tid == 0) {
    unit_off[S] = U;
  }
  if (U == 0) {  // no session has new tokens
    if (tid < kAttnHdrInts) p.hdr[tid] = 0;
    return;
  }
  __syncthreads();
  // unit u -> tiles it has to visit (0: it is past the list), with its session and lengths
  struct Unit {
    int s, t0, P, N, nt;
  };
  auto unit = [&](int u) {
    Unit r{0, 0, 0, 0, 0};
    if (u >= U) return r;
    int lo = 0, hi = S;  // last s with unit_off[s] <= u, a quarter of the range at a time; unit_off[hi] > u
    while (hi - lo > 1) {
      const int q = (hi - lo + 3) >> 2;
      const int at1 = unit_off[min(lo + q, hi)], at2 = unit_off[min(lo + 2 * q, hi)], at3 = unit_off[min(lo + 3 * q, hi)];
      lo += q * ((at1 <= u) + (at2 <= u) + (at3 <= u));
      hi = min(hi, lo + q);
    }
    r.s = lo;
    r.t0 = (u - unit_off[lo]) * p.bmt;
    r.P = len_prefix[lo];
    r.N = len_new[lo];
    r.nt = unit_tiles(r.P, r.N, r.t0, p.bmt);
    return r;
  };
  // A thread's units (u = tid, tid + 256, ...) and the way they are cut are worked out once and kept in registers
  // between the passes while there are at most kSchedCached of them per thread; longer lists recompute them.
  constexpr int kSchedCached = 4;
  const int n_rounds = (U + kSchedThreads - 1) / kSchedThreads;
  const bool cached = n_rounds <= kSchedCached;
  Unit uc[kSchedCached];
  // Block ids of a unit's first two key tiles: what its first (for most units: only) work item carries.  Their loads
  // start here and return while the passes below run.
  int ids0[kSchedCached][8];
  const bool has_table = p.table && p.table_stride > 0;
  auto first_ids_of = [&](int s, int first_tile, int (&ids)[8]) {
    const int32_t* table_row = p.table + (int64_t)s * p.table_stride;
#pragma unroll
    for (int i = 0; i < 8; ++i)  // (index clamped to the row: an entry past the session's keys is never used)
      ids[i] = has_table ? table_row[min((first_tile * kBN + 16 * i) >> p.log_bs, p.table_stride - 1)] : -1;
  };
  // pass 1: total number of (unit, key tile) pairs
  unsigned long long mine = 0;
  int longest = 0, inv_shortest = 0;
  auto note = [&](int nt) {
    mine += (unsigned long long)nt;
    if (nt > 0) {
      longest = max(longest, nt);
      inv_shortest = max(inv_shortest, 0x7FFFFFFF - nt);
    }
  };
  if (cached) {
#pragma unroll
    for (int r = 0; r < kSchedCached; ++r) {
      uc[r] = unit(r * kSchedThreads + tid);
      note(uc[r].nt);
      if (r < n_rounds && uc[r].nt > 0) first_ids_of(uc[r].s, 0, ids0[r]);
    }
  } else {
    for (int u = tid; u < U; u += kSchedThreads) note(unit(u).nt);
  }
  // (summed inside each wave first: atomics of all threads on the one LDS word run one after the other, and took
  // longer than every other step of this kernel)
  {
    // three scans of 20-bit pieces: none can overflow an int over 64 lanes (a thread's count is below 2^60)
    const int s0 = wave_inclusive_scan((int)(mine & 0xFFFFFull));
    const int s1 = wave_inclusive_scan((int)((mine >> 20) & 0xFFFFFull));
    const int s2 = wave_inclusive_scan((int)(mine >> 40));
    const unsigned long long wave_total =
        ((unsigned long long)(unsigned)s2 << 40) + ((unsigned long long)(unsigned)s1 << 20) + (unsigned)s0;
    longest = wave_inclusive_max(longest);
    inv_shortest = wave_inclusive_max(inv_shortest);
    if ((tid & 63) == 63 && wave_total) {
      atomicAdd(&total_tiles_s, wave_total);
      atomicMax(&max_nt_s, longest);
      atomicMax(&inv_min_nt_s, inv_shortest);
    }
  }
  __syncthreads();
  const long long max_nt = max_nt_s;
  int C;
  {  // (every wave works it out)
    // With at least two workgroup-sized units per slot, longest-first dispatch balances well without splitting
    // anything but the longest units; with fewer, every unit is cut so that there are about two pieces per slot.
    const long long wg_units = (long long)U * p.n_kv_heads;
    const int target = (p.coarse_ok && wg_units >= 2ll * p.target_slots) ? p.target_slots : p.target;
    // C = ceil(total tiles * kv-heads / target): a single-precision estimate, then exact steps in integers
    const unsigned long long tot = total_tiles_s * (unsigned long long)p.n_kv_heads;
    long long c = (long long)((float)tot * (1.0f / (float)target));
    if (c > 0x3FFFFFFF) c = 0x3FFFFFFF;
    while (c < 0x3FFFFFFF && (unsigned long long)c * (unsigned long long)target < tot) ++c;
    while (c > 0 && (unsigned long long)(c - 1) * (unsigned long long)target >= tot) --c;
    // Units of (nearly) one length, and too few of them for the coarse rule: a single long session, or a batch of
    // equal ones.  Equal pieces are dispatched in whole rounds, so what counts is rounds x (piece + fixed cost), and
    // one round of longer pieces can beat two rounds of shorter ones.  Only cuts that are not finer than the one
    // above are tried (the workspace bounds are derived from it): lane k - 1 tries k pieces.  (One lane that tried them
    // all took 17 us for its 128 divisions.)
    const long long min_nt = 0x7FFFFFFF - inv_min_nt_s;
    if (target == p.target && max_nt > 0 && min_nt * 51 >= max_nt * 50 && c > 0) {
      constexpr unsigned kFixedTiles = 6;  // a work item's fixed cost (~11 us) in key tiles (~1.9 us)
      const unsigned k = (tid & 63) + 1;
      const unsigned ck = ((unsigned)max_nt + k - 1) / k;
      // (units past 2^25 in number make every cost so large that their order no longer matters)
      const unsigned pieces = (unsigned)(wg_units < (1 << 25) ? wg_units : (1 << 25)) * k;
      const unsigned rounds = (pieces + p.target_slots - 1) / (unsigned)p.target_slots;
      unsigned long long best = (long long)ck < c && k > 1 ? ~0ull : (unsigned long long)rounds * (ck + kFixedTiles);
      unsigned best_k = k;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {  // smallest cost; of equal costs the finer cut: more pieces in flight
        const unsigned long long other = __shfl_xor(best, o);
        const unsigned other_k = __shfl_xor(best_k, o);
        if (other < best || (other == best && other_k > best_k)) {
          best = other;
          best_k = other_k;
        }
      }
      const long long best_c = ((unsigned)max_nt + best_k - 1) / best_k;
      if (best_c >= c) c = best_c;
    }
    if (c < p.c_min) c = p.c_min;
    C = (int)c;
  }
  // bucket of a chunk length: longer chunks get smaller bucket numbers (they are dispatched first).  Any monotone
  // function of the length will do, as long as both passes below use the same one.
  const float buckets_per_tile = (float)kSchedBuckets / (float)C;
  auto bucket_of = [&](int len) {
    const int b = (int)((float)(C - len) * buckets_per_tile);
    return b < 0 ? 0 : (b >= kSchedBuckets ? kSchedBuckets - 1 : b);
  };
  // How a unit is cut: chunks of `len` tiles, n_real of them, in slots pslot0 .. and with counter `merge` when it is
  // split (n_real > 1).  The running totals of chunks and of split units (carry_c, carry_m) go through the rounds in
  // unit order; a unit whose chunks would pass the end of the slots or of the counters stays whole, and so does every
  // split candidate after it.  (Every thread of the block calls this the same number of times: it holds barriers.)
  struct Cut {
    int len, n_real, pslot0, merge;
  };
  auto cut_of = [&](const Unit& un, int& carry_c, int& carry_m) {
    Cut c;
    const int nt = un.nt;
    if (max_nt <= C) {  // no unit of the batch is cut
      c.len = nt;
      c.n_real = nt > 0 ? 1 : 0;
      c.pslot0 = c.merge = -1;
      return c;
    }
    const int nc = nt > 0 ? (nt + C - 1) / C : 0;
    c.len = nc > 0 ? (nt + nc - 1) / nc : 0;
    c.n_real = c.len > 0 ? (nt + c.len - 1) / c.len : 0;
    const bool want = c.n_real > 1;
    int ic = want ? c.n_real : 0, im = want ? 1 : 0, tot_c, tot_m;
    block_inclusive_scan2(ic, im, wave_sums, tot_c, tot_m);
    const bool fits = carry_c + ic <= p.pslots_bound && carry_m + im <= p.merges_bound;
    c.pslot0 = carry_c + ic - c.n_real;
    c.merge = carry_m + im - 1;
    if (want && !fits) {
      c.len = nt;
      c.n_real = 1;
      atomicOr(&flags_s, 1);
    }
    // slots and counters in use = the largest prefix sums that fitted (one LDS atomic per wave, not per unit: atomics
    // of many lanes on one word run one after the other)
    const int end_c = wave_inclusive_max(want && fits ? carry_c + ic : 0);
    const int end_m = wave_inclusive_max(want && fits ? carry_m + im : 0);
    if ((threadIdx.x & 63) == 63 && end_c) {
      atomicMax(&n_pslot_s, end_c);
      atomicMax(&n_split_s, end_m);
    }
    if (c.n_real <= 1) {
      c.pslot0 = -1;
      c.merge = -1;
    }
    carry_c += tot_c;
    carry_m += tot_m;
    return c;
  };
  // pass 2: histogram of chunk lengths
  auto count = [&](const Unit& un, const Cut& c) {
    if (c.n_real == 0) return;
    if (c.n_real == 1) {
      atomicAdd(&hist[bucket_of(c.len)], 1);
      return;
    }
    const int n_full = un.nt / c.len, rem = un.nt - n_full * c.len;  // n_full chunks of len tiles, one of rem
    if (n_full) atomicAdd(&hist[bucket_of(c.len)], n_full);
    if (rem) atomicAdd(&hist[bucket_of(rem)], 1);
  };
  Cut cc[kSchedCached];
  {
    int carry_c = 0, carry_m = 0;
    if (cached) {
#pragma unroll
      for (int r = 0; r < kSchedCached; ++r)
        if (r < n_rounds) {
          cc[r] = cut_of(uc[r], carry_c, carry_m);
          count(uc[r], cc[r]);
        }
    } else {
      for (int base = 0; base < U; base += kSchedThreads) {
        const Unit un = unit(base + tid);
        count(un, cut_of(un, carry_c, carry_m));
      }
    }
  }
  __syncthreads();
  if (tid < kSchedBuckets) {  // wave 0: exclusive prefix sum, hist[b] becomes the first list position of bucket b
    const int h = hist[tid];
    const int incl = wave_inclusive_scan(h);
    hist[tid] = incl - h;
    if (tid == kSchedBuckets - 1) n_items_s = incl;
  }
  __syncthreads();
  for (int i = tid; i < n_split_s * p.n_kv_heads; i += kSchedThreads) p.merge_cnt[i] = 0;
  // pass 3: emit items
  auto emit = [&](const Unit& un, const Cut& c, const int (*ids_first)[8]) {  // ids_first: of chunk 0, or null
    if (c.n_real == 0) return;
    const int cu_s = cu_of[un.s];
    // four chunks at a time: their table reads are issued together, before the first item is written (one wait for
    // memory per group instead of one per chunk)
    for (int ch0 = 0; ch0 < c.n_real; ch0 += 4) {
      int ids[4][8];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int ch = ch0 + k;
        if (ch >= c.n_real) break;
        if (ch == 0 && ids_first) {
#pragma unroll
          for (int i = 0; i < 8; ++i) ids[k][i] = (*ids_first)[i];
        } else {
          first_ids_of(un.s, ch * c.len, ids[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int ch = ch0 + k;
        if (ch >= c.n_real) break;
        const int tb = ch * c.len, te = min(un.nt, tb + c.len);
        const int pos = atomicAdd(&hist[bucket_of(te - tb)], 1);
        if (pos < p.items_bound) {
          WorkItem w{un.s, un.t0, tb, te, c.n_real > 1 ? c.pslot0 + ch : -1, cu_s, un.N, un.P,
                     c.merge, c.pslot0, c.n_real, {-1, -1, -1, -1, -1, -1, -1, -1}, {0, 0, 0, 0, 0}};
#pragma unroll
          for (int i = 0; i < 8; ++i) w.first_ids[i] = ids[k][i];
          p.items[pos] = w;
        } else {
          atomicOr(&flags_s, 2);  // more units than total_new_tokens and n_sessions allow: the lengths on the device
                                  // disagree with the host's bounds, and this piece of work is not done
        }
      }
    }
  };
  if (cached) {
#pragma unroll
    for (int r = 0; r < kSchedCached; ++r)
      if (r < n_rounds) emit(uc[r], cc[r], &ids0[r]);
  } else {
    int carry_c = 0, carry_m = 0;
    for (int base = 0; base < U; base += kSchedThreads) {
      const Unit un = unit(base + tid);
      emit(un, cut_of(un, carry_c, carry_m), nullptr);
    }
  }
  __syncthreads();
  if (tid == 0) {
    p.hdr[kHdrItems] = min(n_items_s, p.items_bound);
    p.hdr[kHdrChunk] = C;
    p.hdr[kHdrSplitUnits] = n_split_s;
    p.hdr[kHdrPslots] = n_pslot_s;
    p.hdr[kHdrPlan] = kPlanList;
    p.hdr[kHdrDecTiles] = 0;
    p.hdr[kHdrFlags] = flags_s;
  }
}

struct MfmaParams {
  const __bf16* k_layer;
  const __bf16* v_layer;
  int64_t block_stride;
  uint32_t block_bytes;  // block_stride in bytes (the MFMA path requires it to fit 32 bits)
  uint32_t row_bytes;    // one token row of K (or V): n_kv_heads * 128 * 2
  int32_t n_blocks, log_bs, n_kv_heads, n_q_heads;
  const __bf16* q;
  const __bf16* k_new;
  const __bf16* v_new;
  __bf16* out;
  const int32_t* cu_new_lens;
  const int32_t* prefix_lens;
  const int32_t* table;
  int32_t table_stride, n_sessions;
  float scale_log2e;
  int32_t* hdr;
  const WorkItem* items;
  int32_t* merge_cnt;   // [split unit][kv-head]: chunks that have written their partial result
  float* partials;
  // direct mode of attn_mfma_kernel: shortest piece (tiles), workgroups the pieces are cut for, one record per unit
  int32_t direct_c_min, direct_slots, units_bound;
  MergeItem* unit_recs;
  // attn_decode_kernel: new tokens per unit, the rows of q / out, its ranges, one record per
  // unit, and the pieces of units that several ranges share
  int32_t dec_m, total_new_tokens, dec_ranges, dec_records;
  MergeItem* dec_merges;    // [dec_records]
  float* dec_partials;      // [2 * key ranges][n_kv_heads][dec_slot_floats], for units of up to dec_stated tokens
  float* dec_long_partials; // the same for longer units
  int32_t dec_stated, dec_slot_floats, dec_long_slot_floats;  // room for the packed piece of a unit (whole lines)
};


constexpr int kD = 128;  // head_dim
// Source of absent key rows (one head's 256 bytes)
static __device__ __attribute__((aligned(256))) const unsigned kZeroRow[64] = {};
// A row sum above this (one probability of 2^40 or more, or an overflow) makes the softmax reference stale.
constexpr float kRefreshSum = 1.0995116e12f;  // 2^40

// Write one query row's 128 outputs: this lane holds d = 32*dt + 4*g2 + 8*i + j at acc[dt][4*i + j].
__device__ __forceinline__ void store_out_row(__bf16* op, const f32x16 (&acc)[4], float inv, int g2) {
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bf16x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = (__bf16)(acc[dt][4 * i + j] * inv);
      *reinterpret_cast<bf16x4*>(op + 32 * dt + 4 * g2 + 8 * i) = v;
    }
}

// A slot of partial results, written and read at device scope (sc1: the access goes to the point where the XCDs' L2
// caches agree), 8 or 16 bytes per lane.  Offsets in bytes from the slot's start.
struct PartialSlot {
  static constexpr int kDeviceScope = 16;  // the sc1 bit of the cache-policy operand
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ explicit PartialSlot(float* slot)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(slot, 0, kPartialFloats * 4, 0x00027000)) {}
  __device__ __forceinline__ void store4(int off, f32x4 v) const {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rsrc, off, 0, kDeviceScope);
  }
  __device__ __forceinline__ void store2(int off, f32x2 v) const {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rsrc, off, 0, kDeviceScope);
  }
  __device__ __forceinline__ f32x4 load4(int off) const {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, kDeviceScope));
  }
  __device__ __forceinline__ f32x2 load2(int off) const {
    return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, off, 0, kDeviceScope));
  }
};

// The 32 output rows of a wave through a buffer of its own in LDS: every store instruction then writes whole 128-byte
// lines (the G heads of a token are neighbours in memory: a wave's rows, in (token, head) order, are 32 / G runs of
// G x 256 bytes), where the direct form writes 8 bytes per lane, i.e. sixteen separate pieces per line for the L2 to put
// together.  row_of_lane: this lane's row in (token, head) order; valid_bits: bit m set = row m is written.
constexpr int kOutRowBytes = 256 + 16;
__device__ __forceinline__ void store_out_rows_staged(char* stage, __bf16* first_row, int64_t token_stride_elems,
                                                      int rows_per_token, int row_of_lane, unsigned valid_bits,
                                                      const f32x16 (&acc)[4], float inv, int g2, int lane) {
  char* wr = stage + row_of_lane * kOutRowBytes + 8 * g2;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bf16x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = (__bf16)(acc[dt][4 * i + j] * inv);
      *reinterpret_cast<bf16x4*>(wr + 64 * dt + 16 * i) = v;
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const int m = 4 * it + (lane >> 4);
    const int tok = m / rows_per_token, hd = m - tok * rows_per_token;
    if ((valid_bits >> m) & 1u) {
      const u32x4_t v = *reinterpret_cast<const u32x4_t*>(stage + m * kOutRowBytes + 16 * (lane & 15));
      *reinterpret_cast<u32x4_t*>(reinterpret_cast<char*>(first_row + tok * token_stride_elems + (int64_t)hd * kD) + 16 * (lane & 15)) = v;
    }
  }
}


// LDS tile layout shared by K and V (64 key rows x 256 bytes): rows are stored in groups of four; a group is the
// 1 KiB that one wave writes with one direct global->LDS load (lane l lands at group base + 16*l), groups are
// kGroupBytes apart (16 bytes of padding), and inside row r of a group the 16-byte chunk c sits at position
// c ^ ((r & 3) << 2).  With this, the 16 rows that a quarter-wave reads with ds_read_b128 (K fragments) and the
// 4 rows x 32 bytes that 16 lanes read with ds_read_b64_tr_b16 (V fragments) each cover all banks once.
constexpr int kGroupBytes = 1024 + 16;
constexpr int kTileBytes = 16 * kGroupBytes;  // 16640

#define SYMPH_GLDS16(src, dst)                                                                       \
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src),             \
                                   (__attribute__((address_space(3))) void*)(dst), 16, 0, 0)

// The same with the non-temporal cache policy (bit 1 of the last operand): for rows that are read once
#define SYMPH_GLDS16_NT(src, dst)                                                                    \
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src),             \
                                   (__attribute__((address_space(3))) void*)(dst), 16, 0, 2)

// ---- direct mode: a batch of at most 64 units, where a scheduling kernel in front and a last piece that combines all
// others behind would take longer than the attention.  Every wave reads the sessions' lengths (lane s those of session s),
// lists the units (lane u has unit u, in session order), chooses the cut (64 lanes price 64 cuts of the longest unit, from
// whole to 63 pieces) and picks its workgroup's piece: no LDS, no barrier, one trip to memory for the lengths and one for
// the first block ids.
// What a cut into W workgroups of at most C tiles costs, in microseconds, fitted to 280 timings of 27 batches (1 to 48
// sessions of 500 to 32 768 tokens, 8 to 1000 new ones, 2 to 8 kv-heads; the cut it chooses is on average 0.5 % slower
// than the best one tried): a tile takes 1.1 while every workgroup has its CU to itself and up to 1.65 when two share it,
// a further round of workgroups 14 beside its tiles and a piece that has to be combined 0.018 (its 66 KB written and
// read back with the merge kernel the timings were taken with).  Today's merge kernel is faster, but a price of 0.012 serves
// one of twelve calls (45 new tokens over 3001 17.0 us for 17.5), costs three (6 x 20 over 2000 22.9 for 21.8, 3 x 20 .. 40
// over 8000 37.7 for 35.5, 160 over 3001 26.6 for 26.0), and every cut that moves makes probabilities be rounded against other
// references, which moves outputs by 2.8e-3.  Against the work list: 45 new tokens over 3001, 29.7 -> 17.5 us (47 before the
// scheduling kernel was reworked); 17 over 16 000, 53 -> 24; 8 x 64 .. 128 over 1500 .. 3000, 75 -> 55; 512 over 32 768 in
// groups of eight heads, 504 -> 502.
constexpr int kDirectUnits = 64;
constexpr float kTileAlone = 1.1f, kTilePaired = 1.65f, kRoundFixed = 14.f, kPieceMerge = 0.018f;

__device__ __forceinline__ bool direct_item(const MfmaParams& p, int bmt, int piece, WorkItem& it) {
  const int lane = threadIdx.x & 63;
  int cu = 0, N = 0, P = 0;
  if (lane < p.n_sessions) {
    cu = p.cu_new_lens[lane];  // (rows past total_new_tokens do not exist; such lengths are flagged below)
    N = max(min(p.cu_new_lens[lane + 1], p.total_new_tokens) - cu, 0);
    P = max(p.prefix_lens[lane], 0);
  }
  const int nq = (N + bmt - 1) / bmt;
  const int q_end = wave_inclusive_scan(nq);
  const int n_units = min(__builtin_amdgcn_readlane(q_end, 63), kDirectUnits);
  // lane u: the session of unit u is the first one whose units end past u
  int lo = 0;
  if (p.n_sessions <= 8) {  // (a step by a lane's value costs a quarter of a shuffle: 2.6 us for the piece of a single session's
    for (int i = 0; i < p.n_sessions; ++i) lo += __builtin_amdgcn_readlane(q_end, i) <= lane;  // call, 2.0 with what follows)
  } else {
#pragma unroll
    for (int step = 32; step > 0; step >>= 1)
      if (__shfl(q_end, lo + step - 1) <= lane) lo += step;
  }
  const int s = min(lo, 63);
  const int t0 = (lane - (__shfl(q_end, s) - __shfl(nq, s))) * bmt;
  const int uN = __shfl(N, s), uP = __shfl(P, s), ucu = __shfl(cu, s);
  const int nt = lane < n_units ? unit_tiles(uP, uN, t0, bmt) : 0;
  const int total = __builtin_amdgcn_readlane(wave_inclusive_scan(nt), 63);
  const int max_nt = __builtin_amdgcn_readlane(wave_inclusive_max(nt), 63);
  // (no cut finer than c_lo: the slots for partial results are sized by it)
  const int64_t work = (int64_t)total * p.n_kv_heads;
  int c_lo = (int)((float)work / (float)p.direct_slots);  // ceil(work / slots): an estimate, then exact steps
  while ((int64_t)c_lo * p.direct_slots < work) ++c_lo;
  while (c_lo > 0 && (int64_t)(c_lo - 1) * p.direct_slots >= work) --c_lo;
  c_lo = max(c_lo, p.direct_c_min);
  // lanes 0 .. 31: 1, 1.25, .. 8.75 pieces of the longest unit; lanes 32 .. 63: 9, 10.75, .. 63.25
  const float cuts = lane < 32 ? 1.f + 0.25f * (float)lane : 9.f + 1.75f * (float)(lane - 32);
  int C = max((int)ceilf((float)max_nt / cuts), c_lo);
  {
    const float inv_c = 1.0f / (float)C;
    const float below = (float)(nt - 1);
    float pieces = 0.f, split = 0.f;
    for (int u = 0; u < n_units; ++u) {
      const float n = floorf(__builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, below), u)) * inv_c);
      pieces += n;
      split += n > 0.f ? n + 1.f : 0.f;
    }
    const float heads = (float)p.n_kv_heads, slots = (float)p.direct_slots;
    const float w = (pieces + (float)n_units) * heads;
    const float shared = fminf(fmaxf(2.f * w / slots - 1.f, 0.f), 1.f);
    const float tile = kTileAlone + (kTilePaired - kTileAlone) * __builtin_amdgcn_sqrtf(shared);
    const float cost = ceilf(w / slots) * fmaf((float)C, tile, kRoundFixed) + split * heads * kPieceMerge;
    // (positive floats compare as their bits do; of equal costs the last lane, which cuts finest)
    const int inv_cost = 0x7FFFFFFF - __builtin_bit_cast(int, cost);
    const int best = __builtin_amdgcn_readlane(wave_inclusive_max(inv_cost), 63);
    C = __builtin_amdgcn_readlane(C, 63 - __builtin_clzll(__ballot(inv_cost == best)));
  }
  const int nc = (nt + C - 1) / C;
  const int end = wave_inclusive_scan(nc);
  const int n_pieces = __builtin_amdgcn_readlane(end, 63);
  if (blockIdx.x == 0 && threadIdx.x < 64) {
    const bool dropped = p.cu_new_lens[p.n_sessions] > p.total_new_tokens;
    if (lane < kAttnHdrInts)
      p.hdr[lane] = lane == kHdrItems   ? n_pieces
                    : lane == kHdrChunk ? C
                    : lane == kHdrPlan  ? kPlanDirect
                                        : (lane == kHdrFlags && dropped ? 2 : 0);
    if (lane < p.units_bound)
      p.unit_recs[lane] = MergeItem{ucu + t0, min(bmt, uN - t0), end - nc, lane < n_units && nc > 1 ? nc : 0};
  }
  if (piece >= n_pieces) return false;
  const int u = __builtin_ctzll(__ballot(piece < end));
  auto of_unit = [&](int x) { return __builtin_amdgcn_readlane(x, u); };
  const int n = of_unit(nc), tiles = of_unit(nt), ch = piece - (of_unit(end) - n);
  it.s = of_unit(s);
  it.t0 = of_unit(t0);
  const unsigned each = (unsigned)tiles / (unsigned)n, rest = (unsigned)tiles - each * n;
  it.tile_begin = ch * each + ch * rest / (unsigned)n;  // ch * tiles / n: near-equal pieces
  it.tile_end = (ch + 1) * each + (ch + 1) * rest / (unsigned)n;
  it.pslot = n > 1 ? piece : -1;
  it.n_chunks = n;
  it.cu_s = of_unit(ucu);
  it.n_new = of_unit(uN);
  it.n_prefix = of_unit(uP);
  // block ids of the first two tiles: lane i < 8 reads that of group i
  int raw = -1;
  if (p.table && p.table_stride > 0)
    raw = p.table[(int64_t)it.s * p.table_stride +
                  min((it.tile_begin * kBN + 16 * (lane & 7)) >> p.log_bs, p.table_stride - 1)];
#pragma unroll
  for (int i = 0; i < 8; ++i) it.first_ids[i] = __builtin_amdgcn_readlane(raw, i);
  return true;
}

// One workgroup = one work item x one kv-head: 128 query rows (G heads x 128/G tokens) against the item's key tiles.
// Requires block_size >= 16 (a power of two): the 16 consecutive key rows of a staging group then lie in ONE block, so
// block ids are workgroup-uniform and a row address is scalar base + per-lane constant.
// LB = log2(block_size) when it is 4 (the common 16-token block), else 0 = runtime.
//
// Pipeline, iteration j (tiles are double-buffered in LDS, buffers are separate arrays so that the compiler can tell
// which loads an LDS read has to wait for):
//   start : direct global->LDS loads of K(j+2) and V(j+1) are issued (no registers, no LDS store instructions);
//   block : S(j+1) = K(j+1) Q^T on the matrix cores  ||  online softmax of S(j) on the vector ALU  -> P(j);
//   then  : O += V(j)^T P(j);   end: wait for the loads, one barrier.
// The first product of the NEXT tile is independent of the softmax of the current one, so one wave keeps the matrix
// pipe and the vector ALU busy at the same time instead of alternating between them.
// DIRECT: without a scheduling kernel.  Workgroup g works out piece g / H_kv by itself (direct_item) and the pieces of split
// units are combined by attn_merge_kernel.
template <int G, int LB, bool DIRECT>
__global__ __launch_bounds__(256, 2) void attn_mfma_kernel(const MfmaParams p) {
  constexpr int BMT = 128 / G;  // query tokens per tile
  __shared__ __attribute__((aligned(16))) char K0[kTileBytes];
  __shared__ __attribute__((aligned(16))) char K1[kTileBytes];
  __shared__ __attribute__((aligned(16))) char V0[kTileBytes];
  __shared__ __attribute__((aligned(16))) char V1[kTileBytes];

  const int Hkv = p.n_kv_heads;
  const int item_idx = blockIdx.x / Hkv;
  __shared__ int merges_here;  // set for the chunk of a split unit that arrives last
  const int kvh = blockIdx.x - item_idx * Hkv;
  WorkItem it;
  if constexpr (DIRECT) {
    if (!direct_item(p, BMT, item_idx, it)) return;
  } else {
    // The array covers the whole grid, so the item is read beside the count, not after it: one trip to memory less in
    // front of the first K,V loads.  (The empty statement makes the compiler issue both loads before the branch.)
    it = p.items[item_idx];
    const int n_items = p.hdr[kHdrItems];
    asm volatile("" ::"s"(it.s), "s"(it.pslot), "s"(it.n_chunks), "s"(it.first_ids[0]), "s"(it.first_ids[7]), "s"(n_items));
    if (item_idx >= n_items) return;
  }
  const int s = it.s;
  const int t0 = it.t0;
  const int cu_s = it.cu_s;
  const int N = it.n_new;
  const int P = it.n_prefix;
  const int lb = LB ? LB : p.log_bs;
  const int bs_mask = (1 << lb) - 1;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int n = lane & 31;  // query column of this lane inside the wave's 32 rows; also its A-operand row
  const int g2 = lane >> 5;

  // Query row of this lane.  The tile's 128 / G tokens are dealt to the waves in order, 32 / G tokens x G heads each
  // (head-major inside the wave), so that the tokens a tile does not have (a session's last tile, a short turn) leave
  // WHOLE waves without rows.  Such a wave only issues its share of the K,V loads and keeps the barriers: it skips the
  // matrix and vector work, which would be padding, and leaves those pipes to the workgroup that shares the CU (a
  // one-token turn fills 4 of the 128 rows: all in wave 0).
  constexpr int TW = BMT / 4;  // tokens per wave
  const int hh = n / TW;
  const int tt = wave * TW + (n - hh * TW);
  const bool q_valid = t0 + tt < N;
  const bool wave_works = t0 + wave * TW < N;
  const int tok = t0 + tt;
  const int head = kvh * G + hh;

  bf16x8 qreg[8];
  {
    const __bf16* qp = p.q + ((int64_t)(cu_s + (q_valid ? tok : 0)) * p.n_q_heads + head) * kD + 8 * g2;
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      qreg[st] = *reinterpret_cast<const bf16x8*>(qp + 16 * st);
      if (!q_valid) {
#pragma unroll
        for (int e = 0; e < 8; ++e) qreg[st][e] = (__bf16)0.0f;
      }
    }
  }

  const int total_keys = P + N;
  const int tile_begin = it.tile_begin, tile_end = it.tile_end;
  // tiles below fast_end lie entirely inside the paged prefix: every row comes from the pool
  const int fast_end = min(tile_end, P / kBN);

  // ---- global -> LDS: wave w writes row group 4*i + w (rows 16*i + 4*w .. +3 of the tile) with its i-th load;
  // lane l covers row 4*w + l/16 of the 16-row group and holds logical chunk (l % 16) ^ ((l/16) << 2) of it.
  const bool has_table = p.table != nullptr && p.table_stride > 0;
  const int32_t* table_row = p.table + (int64_t)s * p.table_stride;
  const int dma_row = 4 * wave + (lane >> 4);                          // row inside a 16-row group
  const int dma_chunk = (lane & 15) ^ (((lane >> 4) & 3) << 2);        // logical 16-byte chunk this lane fetches
  const unsigned row_bytes = p.row_bytes;
  const unsigned voff = (unsigned)dma_row * row_bytes + (unsigned)kvh * 256u + (unsigned)dma_chunk * 16u;
  const char* k_bytes = reinterpret_cast<const char*>(p.k_layer);
  const char* v_bytes = reinterpret_cast<const char*>(p.v_layer);

  // Block ids of the tile's four 16-row groups.  The table entries are fetched (vector loads, every lane the same
  // address) a whole iteration before they are needed and only then moved to scalar registers: asking for the value
  // right after issuing the load would also wait for the K,V loads issued just before it.
  int ids[4];   // scalar: ids of the tile whose K rows are loaded next
  int ids_raw;  // in flight: lane i < 4 holds the id of group i of the tile after that
  auto fetch_ids = [&](int tile) {
    const int jb = (tile * kBN + 16 * (lane & 3)) >> lb;
    ids_raw = has_table ? table_row[min(jb, p.table_stride - 1)] : -1;
  };
  auto take_ids = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) ids[i] = __builtin_amdgcn_readlane(ids_raw, i);
  };
  // Issue the loads of one tile of K or of V into an LDS buffer.  Rows that do not exist (past the session's keys, or
  // named by a block id outside the cache) are read from a row of zeros, so they are finite and add nothing.
  auto issue_tile = [&](const char* pool_bytes, const __bf16* new_rows, char* lds_buf, int tile) {
    // one comparison of the largest id (as unsigned: a negative id is huge)
    const unsigned id_max = max(max((unsigned)ids[0], (unsigned)ids[1]), max((unsigned)ids[2], (unsigned)ids[3]));
    const bool fast = tile < fast_end && id_max < (unsigned)p.n_blocks;
    if (__builtin_expect(fast, 1)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint64_t off = (uint64_t)(unsigned)ids[i] * p.block_bytes;
        if (LB != 4) off += (uint64_t)((tile * kBN + 16 * i) & bs_mask) * row_bytes;
        // Scalar base + 32-bit lane offset, kept apart for the compiler: with 64-bit per-lane addresses the issue of
        // such a load waits for the matrix instructions of the SIMD's other wave (microbenchmark: eight loads take
        // 290 clocks in this form whatever the other wave does, and 500-2100 in the other while it runs MFMAs).
        const char* base = pool_bytes + off;
        unsigned lane_off = voff;
        asm("" : "+s"(base), "+v"(lane_off));
        SYMPH_GLDS16(base + lane_off, lds_buf + (4 * i + wave) * kGroupBytes);
      }
      asm volatile("; end of the scalar-base loads");  // keeps the last one from being merged with the other path's
    } else {
      // rare path: its per-lane address pieces are derived here, from a lane id the optimiser cannot see through, so
      // that they do not occupy registers throughout the main loop
      int l = lane;
      asm volatile("" : "+v"(l));
      const int row = 4 * wave + (l >> 4);
      const unsigned in_row = (unsigned)kvh * 256u + (unsigned)((l & 15) ^ (((l >> 4) & 3) << 2)) * 16u;
      const char* const zeros = reinterpret_cast<const char*>(kZeroRow) + (l & 15) * 16;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int key = tile * kBN + 16 * i + row;
        const unsigned b = (unsigned)ids[i];
        const bool in_pool = key < P && (key >> lb) < p.table_stride && b < (unsigned)p.n_blocks;
        const bool in_new = key >= P && key < total_keys;
        const char* src = zeros;
        if (in_pool)
          src = pool_bytes + (uint64_t)b * p.block_bytes + (uint64_t)(key & bs_mask) * row_bytes + in_row;
        else if (in_new)
          src = reinterpret_cast<const char*>(new_rows) + (uint64_t)(cu_s + key - P) * row_bytes + in_row;
        SYMPH_GLDS16(src, lds_buf + (4 * i + wave) * kGroupBytes);
      }
    }
  };

  // ---- LDS reads.  K fragment (A operand of S^T = K Q^T): lane (n, g2) reads 16 bytes of key row
  // key_of_row(n) (+32 for the second block), logical chunk 2*st + g2.
  const int krow = key_of_row(n);
  const int k_lane = (krow >> 2) * kGroupBytes + (krow & 3) * 256 + g2 * 16;
  int k_off[4];  // byte offset for st >> 1 == q: chunk pair position q ^ (row & 3)
#pragma unroll
  for (int q = 0; q < 4; ++q) k_off[q] = k_lane + 64 * (q ^ (krow & 3));
  // V fragment (A operand of O^T += V^T P^T) via the transposing read: 16 lanes read 4 rows x 32 bytes and each gets
  // one column (4 consecutive keys of one d).  Lane group lane/16 = 2*g2 + dhalf, i16 = lane % 16:
  // row = 8*g2 + i16/4 (+ 32*kb + 16*u + 4*half), bytes 64*dt + 32*dhalf + 8*(i16 % 4) of the row.
  const int i16 = lane & 15;
  const int vrow = 8 * g2 + (i16 >> 2);
  const int v_lane = (vrow >> 2) * kGroupBytes + (vrow & 3) * 256 + 32 * ((lane >> 4) & 1) + 8 * (i16 & 3);
  int v_off[4];  // byte offset for d tile dt: chunk quad position dt ^ (row & 3)
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) v_off[dt] = v_lane + 64 * (dt ^ (vrow & 3));

  f32x16 o_acc[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o_acc[dt][e] = 0.f;
  float m_run = -INFINITY;  // running max of raw scores (before scale)
  float l_run = 0.f;        // this lane's share of the running sum
  const float cs = p.scale_log2e;
  const int q_limit = P + tok;  // last key this query may see
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

  // S^T of one tile (64 keys x 32 queries per wave) on the matrix cores
  auto qk = [&](const char* kbuf, f32x16 (&sc)[2]) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e) sc[kb][e] = 0.f;
    {
      // the two 32-key blocks alternate, so consecutive MFMAs never wait for each other's accumulator
#pragma unroll
      for (int st = 0; st < 8; ++st)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
          const bf16x8 a = *reinterpret_cast<const bf16x8*>(kbuf + k_off[st >> 1] + 32 * (st & 1) + kb * 8 * kGroupBytes);
          sc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[st], sc[kb], 0, 0, 0);
        }
    }
  };
  // causal mask: only tiles that reach past the first query's limit
  auto mask = [&](f32x16 (&sc)[2], int tile) {
    const int key0 = tile * kBN;
    if (key0 + kBN - 1 > P + t0) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int key = key0 + kb * 32 + 16 * (e >> 3) + 8 * g2 + (e & 7);
          if (key > q_limit) sc[kb][e] = -INFINITY;
        }
    }
  };
  // Online softmax on the vector ALU, one query per lane (lanes l and l^32 split its keys), with a STALE reference:
  // probabilities are 2^((s - m_ref) * scale') for a reference m_ref that is NOT the running maximum but the maximum
  // at the time it was last refreshed.  Numerator and denominator carry the same factor, so the result is the exact
  // softmax as long as nothing overflows, and bf16 / fp32 keep their relative precision at any magnitude.  The
  // reference is refreshed (below) only when a tile's row sum shows that some score exceeds it by more than
  // kRefreshLog2, which after the first tile practically never happens; the per-tile maximum, the rescale factor
  // and the rescaling of the accumulators thereby leave the loop.
  // reference := max(reference, maximum of this tile), in log2 units; returns the factor by which everything
  // accumulated so far has to be rescaled (0 for a first reference, 1 where nothing moved)
  auto raise_reference = [&](const f32x16 (&sc)[2], float& mb) {
    float mx = sc[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sc[kb][e]);
    mx = max_across_halves(mx);
    const float m_new = fmaxf(m_run, mx * cs);
    // a row that has seen no key yet (a work item may start past its causal limit) keeps m_run = -inf, which the
    // merge step reads as "no contribution"; its exponent arguments use 0 so that they stay finite
    const float a = (m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
    m_run = m_new;
    mb = (m_new == -INFINITY) ? 0.f : m_new;
    return a;
  };
  // ... then the bf16 probabilities, one 32-key half at a time: the first half follows the statistics directly (in
  // the block that is otherwise almost pure matrix work), the second half runs beside the next tile's first product,
  // so that both blocks of the pipeline carry a similar mix of matrix and vector work whatever block the other
  // workgroup of the CU happens to be in
  auto softmax_exp_half = [&](const f32x16& sc, float mb, bf16x8 (&pb)[2]) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      pb[e >> 3][e & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sc[e], cs, -mb));
    }
  };
  // row sum of the ROUNDED probabilities (the values the second product uses), two per instruction
  auto row_sum = [&](const bf16x8 (&pb)[2][2]) {
    float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const bf16x8 v = pb[kb][u];
        ps0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v[0], v[1]}, ones, ps0, false);
        ps1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v[2], v[3]}, ones, ps1, false);
        ps0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v[4], v[5]}, ones, ps0, false);
        ps1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v[6], v[7]}, ones, ps1, false);
      }
    return ps0 + ps1;
  };
  // Refresh of a stale reference (rare): rescale what has been accumulated, redo this tile's probabilities.
  auto refresh_reference = [&](const f32x16 (&sc)[2], float& mb, bf16x8 (&pb)[2][2], float& ps) {
    const float a = raise_reference(sc, mb);
    l_run *= a;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) o_acc[dt][e] *= a;
    softmax_exp_half(sc[0], mb, pb[0]);
    softmax_exp_half(sc[1], mb, pb[1]);
    ps = row_sum(pb);
  };
  auto wait_loads_and_sync = [&]() {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's global->LDS loads have landed
    __syncthreads();
  };

  // Pipeline.  K(t) lives in K[t' & 1], V(t) in V[t' & 1] with t' = t - tile_begin.  Iteration j issues the loads
  // of K(j+2) and V(j+1) and then runs two straight-line blocks in which the matrix pipe and the vector ALU work on
  // INDEPENDENT data, so that one wave keeps both busy:
  //   block A:  S(j+1) = K(j+1) Q^T   (matrix)   ||   exponentials of S(j) -> P(j), row sums     (vector)
  //   block B:  O += V(j)^T P(j)      (matrix)   ||   running max / rescale factor of S(j+1)      (vector)
  // A wave issues in order, so the instruction stream itself has to alternate between the two kinds; the
  // sched_group_barrier sequences ask the scheduler for that interleaving and for LDS reads that run several matrix
  // instructions ahead of their use (a read issued right before its MFMA exposes the full LDS latency every time).
  f32x16 s_even[2], s_odd[2];  // scores of the even and of the odd tiles (counted from tile_begin)
  int ids_v[4];  // ids of the tile whose V rows are loaded next
  {
    // the ids of the first two tiles came with the work item
#pragma unroll
    for (int i = 0; i < 4; ++i) ids[i] = it.first_ids[i];
    issue_tile(k_bytes, p.k_new, K0, tile_begin);
    issue_tile(v_bytes, p.v_new, V0, tile_begin);
    if (tile_begin + 1 < tile_end) {
#pragma unroll
      for (int i = 0; i < 4; ++i) ids[i] = it.first_ids[4 + i];
      issue_tile(k_bytes, p.k_new, K1, tile_begin + 1);
    }
  }
  // The first product needs K0 only: V0 and K1, issued after it, may still be on their way (loads return in order).
  if (tile_begin + 1 < tile_end)
    __builtin_amdgcn_s_waitcnt(0x0F70 | 8);  // vmcnt(8)
  else
    __builtin_amdgcn_s_waitcnt(0x0F70 | 4);  // vmcnt(4)
  __syncthreads();
  if (wave_works) qk(K0, s_even);
#pragma unroll
  for (int i = 0; i < 4; ++i) ids_v[i] = ids[i];  // ids of tile b+1
  fetch_ids(tile_begin + 2);                      // taken at the top of the first iteration
  float mb_cur = 0.f;  // reference of the exponentials, in log2 units
  bf16x8 pb[2][2];     // P(j); its first half is produced one block ahead of the second
  if (wave_works) {
    mask(s_even, tile_begin);
    raise_reference(s_even, mb_cur);   // first reference: the maximum of the first tile
    softmax_exp_half(s_even[0], mb_cur, pb[0]);
  }
  // Every wave has read all of K0 for the first product before any wave overwrites it (the first iteration loads
  // K(tile_begin + 2) into K0), and V0 and K1 have landed for all waves.  Later iterations end with the same pair.
  wait_loads_and_sync();

  auto iteration = [&](const int j, auto par_c) {
    constexpr int PAR = decltype(par_c)::value;
    char* const k_same = PAR ? K1 : K0;   // held K(j), free now: receives K(j+2)
    char* const k_other = PAR ? K0 : K1;  // holds K(j+1)
    char* const v_same = PAR ? V1 : V0;   // holds V(j)
    char* const v_other = PAR ? V0 : V1;  // held V(j-1), free now: receives V(j+1)
    f32x16 (&s_cur)[2] = PAR ? s_odd : s_even;   // S(j)
    f32x16 (&s_nxt)[2] = PAR ? s_even : s_odd;   // receives S(j+1)
    {
      int keep[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { keep[i] = ids[i]; ids[i] = ids_v[i]; }
      issue_tile(v_bytes, p.v_new, v_other, j + 1);   // ids of tile j+1
#pragma unroll
      for (int i = 0; i < 4; ++i) ids[i] = keep[i];
    }
    if (j + 2 < tile_end) issue_tile(k_bytes, p.k_new, k_same, j + 2);
    if (wave_works) {
    // ---- block A
    qk(k_other, s_nxt);                          // S(j+1)
    softmax_exp_half(s_cur[1], mb_cur, pb[1]);   // second half of P(j)
    float ps = row_sum(pb);
    __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);      // K fragments: six reads up front
#pragma unroll
    for (int g = 0; g < 16; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // one MFMA of S(j+1)
      if (g < 10) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);    // vector ALU: scale, convert, sum
      __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);    // one exponential
    }
    // keep the probabilities (and with them the exponentials) in this block: without a use here the compiler sinks
    // them past the branch below, next to the second product
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int u = 0; u < 2; ++u) asm volatile("" : "+v"(pb[kb][u]));
    asm volatile("" : "+v"(ps));
    // The reference is stale when some score exceeds it by more than 40 in log2 units (then the row sum is huge,
    // infinite or NaN), or when a row that had seen no key now has one.  Rare: redo this tile's probabilities from
    // its scores, which are still in registers, against a refreshed reference.
    if (__any(!(ps <= kRefreshSum) || (m_run == -INFINITY && ps > 0.f))) refresh_reference(s_cur, mb_cur, pb, ps);
    l_run += ps;
    mask(s_nxt, j + 1);
    // ---- block B
    // O += V(j)^T P(j)  ||  first half of P(j+1), in an explicit order: each of the 16 slots holds the two LDS reads
    // of the MFMA four slots ahead, one MFMA, and the scale / exponential (/ convert) of one score; nothing moves
    // between slots.
    bf16x8 pb_first[2];
    {
      auto v_frag = [&](int g) {  // operand of MFMA g = ((kb * 2 + u) * 4 + dt)
        const char* vp = v_same + v_off[g & 3] + (8 * (g >> 3) + 4 * ((g >> 2) & 1)) * kGroupBytes;
        const s16x4 lo = lds_read_tr16(reinterpret_cast<const __bf16*>(vp));
        const s16x4 hi = lds_read_tr16(reinterpret_cast<const __bf16*>(vp + kGroupBytes));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      };
      bf16x8 frag[16];
      float pe[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) frag[g] = v_frag(g);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int g = 0; g < 16; ++g) {
        if (g + 4 < 16) frag[g + 4] = v_frag(g + 4);
        o_acc[g & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[g], pb[g >> 3][(g >> 2) & 1], o_acc[g & 3], 0, 0, 0);
        pe[g] = __builtin_amdgcn_exp2f(fmaf(s_nxt[0][g], cs, -mb_cur));
        asm volatile("" : "+v"(pe[g]));  // evaluated in this slot (a value without side effects is otherwise placed
                                         // next to its use, after the last slot)
        if (g & 1) {
          pb_first[g >> 3][(g & 7) - 1] = (__bf16)pe[g - 1];
          pb_first[g >> 3][g & 7] = (__bf16)pe[g];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    pb[0][0] = pb_first[0];
    pb[0][1] = pb_first[1];
    asm volatile("" : "+v"(pb[0][0]), "+v"(pb[0][1]));   // computed here, not after the barrier
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) ids_v[i] = ids[i];      // the next V tile is j+2
    wait_loads_and_sync();
  };
  // Before each iteration the ids fetched an iteration ago become scalar and the fetch of the next ones starts (it
  // completes under the wait at the end of the iteration).
  auto step = [&](int j, auto par_c) {
    take_ids();         // ids of tile j+2
    fetch_ids(j + 3);   // index clamped to the table: harmless past the last tile
    iteration(j, par_c);
  };
  for (int j = tile_begin; j + 1 < tile_end; j += 2) {
    step(j, std::integral_constant<int, 0>{});
    if (j + 2 < tile_end) step(j + 1, std::integral_constant<int, 1>{});
  }
  // The last tile has no successor: the second half of its probabilities, then its second product, and nothing beside
  // them.  (As one more turn of the loop it computed a first product, exponentials and loads that nobody used.)
  if (wave_works) {
    const bool odd = (tile_end - 1 - tile_begin) & 1;
    if (odd) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) s_even[kb] = s_odd[kb];
    }
    const char* const v_last = odd ? V1 : V0;
    softmax_exp_half(s_even[1], mb_cur, pb[1]);
    float ps = row_sum(pb);
    if (__any(!(ps <= kRefreshSum) || (m_run == -INFINITY && ps > 0.f))) refresh_reference(s_even, mb_cur, pb, ps);
    l_run += ps;
#pragma unroll
    for (int g = 0; g < 16; ++g) {
      const char* vp = v_last + v_off[g & 3] + (8 * (g >> 3) + 4 * ((g >> 2) & 1)) * kGroupBytes;
      const s16x4 lo = lds_read_tr16(reinterpret_cast<const __bf16*>(vp));
      const s16x4 hi = lds_read_tr16(reinterpret_cast<const __bf16*>(vp + kGroupBytes));
      const bf16x8 v = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      o_acc[g & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pb[g >> 3][(g >> 2) & 1], o_acc[g & 3], 0, 0, 0);
    }
  }
  __syncthreads();  // the tile buffers are free

  // rows of this wave in (token, head) order, and which of them exist
  const int row_m = (n - hh * TW) * G + hh;
  const int n_tok_here = min(max(N - (t0 + wave * TW), 0), TW);           // tokens of this wave's TW that exist
  const unsigned valid_bits = n_tok_here * G >= 32 ? 0xFFFFFFFFu : ((1u << (n_tok_here * G)) - 1u);
  char* const out_stage = wave == 0 ? K0 : (wave == 1 ? K1 : (wave == 2 ? V0 : V1));
  __bf16* const out_first = p.out + ((int64_t)(cu_s + t0 + wave * TW) * p.n_q_heads + kvh * G) * kD;
  if (it.pslot < 0) {
    const float l_tot = sum_across_halves(l_run);
    if (wave_works)
      store_out_rows_staged(out_stage, out_first, (int64_t)p.n_q_heads * kD, G, row_m, valid_bits, o_acc, 1.0f / l_tot, g2,
                            lane);
  } else if constexpr (DIRECT) {
    // The piece's accumulators, 16 bytes per lane per store, for the merge kernel.  A wave without rows has none.
    float* const part = p.partials + ((int64_t)it.pslot * Hkv + kvh) * kPartialFloats;
    if (wave_works) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *reinterpret_cast<f32x4*>(part + ((dt * 4 + i) * 256 + tid) * 4) =
              f32x4{o_acc[dt][4 * i], o_acc[dt][4 * i + 1], o_acc[dt][4 * i + 2], o_acc[dt][4 * i + 3]};
      // (a piece whose every score is NaN has no reference either: with one, the merge does not take it for a piece that
      // saw no key, and its sum makes the row NaN)
      *reinterpret_cast<f32x2*>(part + 64 * 256 + tid * 2) = f32x2{l_run == l_run ? m_run : 0.f, l_run};
    }
  } else {
    // Register dump, 16 bytes per lane per store: fully coalesced.  The chunks of a unit may run on different XCDs,
    // whose L2 caches do not see each other's lines, so everything that passes between them is written and read at
    // device scope (each access goes to the point where the XCDs agree) instead of flushing and invalidating whole
    // caches around the hand-over: a release / acquire fence pair at device scope per chunk cost a quarter of the
    // kernel's time on a batch that is all split units.  A wave without rows has nothing to hand over.
    const int64_t chunk_floats = (int64_t)Hkv * kPartialFloats;
    float* const unit_parts = p.partials + ((int64_t)it.pslot0 * Hkv + kvh) * kPartialFloats;
    if (wave_works) {
      const PartialSlot part(unit_parts + (it.pslot - it.pslot0) * chunk_floats);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          part.store4(((dt * 4 + i) * 256 + tid) * 16,
                      f32x4{o_acc[dt][4 * i], o_acc[dt][4 * i + 1], o_acc[dt][4 * i + 2], o_acc[dt][4 * i + 3]});
      part.store2(64 * 256 * 4 + tid * 8, f32x2{m_run, l_run});
    }
    // The chunk that arrives last combines all of them (no further kernel).  Every wave waits until its stores have
    // been performed, then one thread counts the chunk in.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
    if (tid == 0)
      merges_here = __hip_atomic_fetch_add(p.merge_cnt + (int64_t)it.merge * Hkv + kvh, 1, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT) == it.n_chunks - 1;
    __syncthreads();
    if (!merges_here || !wave_works) return;
    // out = sum_c w_c O_c / sum_c w_c l_c with w_c = 2^(m_c - max_c m_c), m_c being chunk c's softmax reference in log2
    // units (-inf: the chunk saw no key of the row).  All chunks are read back in chunk order, this one's too, so the
    // result does not depend on which chunk came last.  Same thread -> (row, d) mapping as the dump above.  kAtOnce chunks
    // of one half of the accumulators are asked for at a time (more would not fit the registers beside the other half)
    // and the weights follow a running maximum: 2 * n / kAtOnce waits for memory for n chunks, not n + 1.
    constexpr int kAtOnce = 3;
    float l_all = 0.f;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int e = 0; e < 32; ++e) o_acc[2 * half + (e >> 4)][e & 15] = 0.f;
      float M = -INFINITY, L = 0.f;
      for (int ch = 0; ch < it.n_chunks; ch += kAtOnce) {
        f32x4 oc[kAtOnce][8];
        f32x2 ml[kAtOnce];
#pragma unroll
        for (int k = 0; k < kAtOnce; ++k) {  // (past the last chunk: it again, without weight)
          const PartialSlot src(unit_parts + min(ch + k, it.n_chunks - 1) * chunk_floats);
          ml[k] = src.load2(64 * 256 * 4 + tid * 8);
#pragma unroll
          for (int i = 0; i < 8; ++i) oc[k][i] = src.load4(((8 * half + i) * 256 + tid) * 16);
        }
        float m_new = M;
#pragma unroll
        for (int k = 0; k < kAtOnce; ++k) {
          if (ch + k >= it.n_chunks) ml[k][0] = -INFINITY;
          m_new = fmaxf(m_new, ml[k][0]);
        }
        const float a = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - m_new);
        M = m_new;
        L *= a;
#pragma unroll
        for (int e = 0; e < 32; ++e) o_acc[2 * half + (e >> 4)][e & 15] *= a;
#pragma unroll
        for (int k = 0; k < kAtOnce; ++k) {
          const float w = ml[k][0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[k][0] - M);
          L = fmaf(w, ml[k][1], L);
#pragma unroll
          for (int e = 0; e < 32; ++e)
            o_acc[2 * half + (e >> 4)][e & 15] = fmaf(w, oc[k][e >> 2][e & 3], o_acc[2 * half + (e >> 4)][e & 15]);
        }
      }
      l_all = L;
    }
    const float L = l_all;
    const float l_tot = sum_across_halves(L);
    store_out_rows_staged(out_stage, out_first, (int64_t)p.n_q_heads * kD, G, row_m, valid_bits, o_acc, 1.0f / l_tot, g2,
                          lane);
  }
}

// Combines the pieces of split units in direct mode: PARTS workgroups per (unit, kv-head), an equal part of the sixteen 16-byte
// vectors of a thread's slot for each.  Few units are cut into many pieces, and what counts is how few trips to memory a thread
// makes: sixteen workgroups of one vector, sixteen pieces at a time (45 new tokens over 3001, 12 pieces: 18.8 us with four
// workgroups and eight pieces at a time, 17.5; 17 over 16 000, 32 pieces: 27.1 and 23.8).  Many units have few pieces each, and
// every workgroup reads their references and sums again: four workgroups (8 x 100 over 3000: 63.7 us, 67.9 with sixteen).
template <int G, int PARTS>
__global__ __launch_bounds__(256) void attn_merge_kernel(const MfmaParams p) {
  constexpr int TW = 128 / G / 4;  // tokens per wave, as in attn_mfma_kernel
  constexpr int kVecs = 16 / PARTS;
  const int Hkv = p.n_kv_heads;
  const int u = blockIdx.x / (PARTS * Hkv);
  const MergeItem mg = p.unit_recs[u];
  if (mg.n_chunks == 0) return;
  const int part_of = blockIdx.x % PARTS, kvh = blockIdx.x / PARTS - u * Hkv;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = lane & 31, g2 = lane >> 5;
  const int hh = n / TW, tt = wave * TW + (n - hh * TW);
  if (wave * TW >= mg.n_unit) return;
  f32x4 o[kVecs];
#pragma unroll
  for (int i = 0; i < kVecs; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float M = -INFINITY, L = 0.f;
  constexpr int kAtOnce = PARTS == 16 ? 16 : 8;
  for (int ch = 0; ch < mg.n_chunks; ch += kAtOnce) {
    f32x4 oc[kAtOnce][kVecs];
    f32x2 ml[kAtOnce];
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k) {
      ml[k] = f32x2{-INFINITY, 0.f};
      if (ch + k < mg.n_chunks) {
        const float* part = p.partials + ((int64_t)(mg.pslot0 + ch + k) * Hkv + kvh) * kPartialFloats;
        ml[k] = *reinterpret_cast<const f32x2*>(part + 64 * 256 + tid * 2);
#pragma unroll
        for (int i = 0; i < kVecs; ++i)
          oc[k][i] = *reinterpret_cast<const f32x4*>(part + ((part_of * kVecs + i) * 256 + tid) * 4);
      }
    }
#pragma unroll
    for (int k0 = 0; k0 < kAtOnce; k0 += 8) {  // (sums go by eight pieces however many are in flight: one result)
      float m_new = M;
#pragma unroll
      for (int k = k0; k < k0 + 8; ++k) m_new = fmaxf(m_new, ml[k][0]);
      const float a = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - m_new);
      M = m_new;
      L *= a;
#pragma unroll
      for (int i = 0; i < kVecs; ++i) o[i] *= a;
#pragma unroll
      for (int k = k0; k < k0 + 8; ++k) {
        if (ml[k][0] == -INFINITY) continue;  // absent, or it saw no key of the row
        const float w = __builtin_amdgcn_exp2f(ml[k][0] - M);
        L = fmaf(w, ml[k][1], L);
#pragma unroll
        for (int i = 0; i < kVecs; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[i][e] = fmaf(w, oc[k][i][e], o[i][e]);
      }
    }
  }
  const float inv = 1.0f / sum_across_halves(L);
  if (tt >= mg.n_unit) return;
  // vector j of the slot is columns 32 * (j / 4) + 8 * (j % 4) + 4 * g2 .. + 3
  __bf16* const op = p.out + ((int64_t)(mg.row0 + tt) * p.n_q_heads + kvh * G + hh) * kD + 4 * g2;
#pragma unroll
  for (int i = 0; i < kVecs; ++i) {
    bf16x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (__bf16)(o[i][e] * inv);
    *reinterpret_cast<bf16x4*>(op + 8 * (part_of * kVecs + i)) = v;
  }
}

// ------------------------------------------------------------------------------------------------------------
// Short turns (decode-like rows): a session whose new rows fit one wave (n_new * G <= 32) reads its whole K,V for
// 32 query rows or fewer, so the work is moving K,V, not arithmetic.  A unit is (session, up to 32 / G of its new tokens):
// one per session, more only where the caller understated max_new_len.  The units' key ranges, laid end to end,
// are cut into equal ranges; a workgroup takes one range for a group of kv-heads, ONE WAVE PER KV-HEAD (eight waves
// for the usual eight heads, else single-wave workgroups).  A wave loads each 32-key tile of its head into an LDS
// buffer of its own (direct global->LDS loads) and uses it; the waves of a workgroup therefore read the eight 256-byte
// slices of the same 2 KiB token rows at the same time, kept together by a barrier per tile, and DRAM sees whole rows
// (a microbenchmark of this load stream: 7.0 TB/s as full rows, 6.7 as independent streams of slices, each pinned to
// an XCD, which is what one workgroup per kv-head gave).  A wave only alternates between "load a tile" and "use it",
// and using it is short, so what keeps HBM busy is the number of waves waiting for a tile: eight per CU, eight tiles
// (133 KiB) on their way nearly all the time.  (Double buffers per wave would halve the waves that fit, and a wave
// cannot keep a second, slower load in the background: loads return in order.)  Same fragment layouts, same
// transposed scores and same stale-reference softmax as attn_mfma_kernel; a wave owns all keys of its range, so its
// result needs no combining inside the workgroup.
// ------------------------------------------------------------------------------------------------------------
constexpr int kSub = 32;                    // keys per tile of this kernel
constexpr int kSubBytes = 8 * kGroupBytes;  // 8320
constexpr int kDecWaveBytes = 2 * kSubBytes;  // K and V of one tile, per wave
// Slots of a unit's pieces.  Units of the stated length have slots of their own: one stride for all, of 32 rows, spread a step's
// pieces over eight times the memory and made 96 sessions take 509 instead of 502 us.
struct DecSlots {
  float* head;        // slot 0 of this kv-head
  int32_t per_slot;   // floats between slots
  __device__ __forceinline__ DecSlots(const MfmaParams& p, int n_unit, int kvh) {
    const bool as_stated = n_unit <= p.dec_stated;
    const int32_t floats = as_stated ? p.dec_slot_floats : p.dec_long_slot_floats;
    head = (as_stated ? p.dec_partials : p.dec_long_partials) + kvh * floats;
    per_slot = p.n_kv_heads * floats;
  }
  __device__ __forceinline__ float* operator[](int slot) const { return head + (int64_t)slot * per_slot; }
};

template <int G, int LB, int HW>
__global__ __launch_bounds__(64 * HW, HW == 8 ? 1 : 2) void attn_decode_kernel(const MfmaParams p) {
  constexpr int BMTD = 32 / G;   // query tokens this kernel covers per session
  static_assert(kDecPartialFloats * 4 <= kDecWaveBytes, "a wave stages its piece in its own tile buffers");
  __shared__ __attribute__((aligned(16))) char lds[HW * kDecWaveBytes];

  // Even split: the units' key ranges, laid end to end, are cut into equal ranges of 32-key tiles, whatever the sessions'
  // lengths.  A range covers the end of one unit, whole units and the start of another: one segment each, processed one
  // after the other.  A unit that lies in one range is finished here; the pieces of one that spans several ranges go to
  // the merge kernel.
  const int Hkv = p.n_kv_heads;
  const int n_groups = Hkv / HW;                 // groups of HW kv-heads: one wave per head of the group
  const int wg = blockIdx.x / n_groups;          // the range
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kvh = (blockIdx.x - wg * n_groups) * HW + wave;
  const int lb = LB ? LB : p.log_bs;
  const int bs_mask = (1 << lb) - 1;

  // Every workgroup works its range out from the sessions' lengths by itself, 64 sessions at a time, one per lane.  (A
  // scheduling kernel in front, whose result every workgroup then read, was two more trips to memory, a launch and the gap
  // behind it: 6 us of a decode step.)
  const int m = p.dec_m;
  const int lane_s = tid & 63;
  auto span_of = [&](int s, int& cu_s, int& N, int& P) {  // rows past total_new_tokens do not exist (flagged below)
    cu_s = p.cu_new_lens[s];
    N = max(min(p.cu_new_lens[s + 1], p.total_new_tokens) - cu_s, 0);
    P = max(p.prefix_lens[s], 0);
  };
  auto tiles_to = [](int P, int end) { return (P + end + kSub - 1) / kSub; };  // of a unit whose last token is end - 1
  int my_cu, my_N, my_P, my_tiles, my_units;  // of session 64 * chunk + lane
  auto take_chunk = [&](int chunk) {
    my_cu = my_N = my_P = my_tiles = 0;
    if (64 * chunk + lane_s < p.n_sessions) span_of(64 * chunk + lane_s, my_cu, my_N, my_P);
    for (int t = 0; t < my_N; t += m) my_tiles += tiles_to(my_P, min(my_N, t + m));
    my_units = (my_N + m - 1) / m;
  };
  int total, n_units, per_wg, range_begin, range_end;
  auto take_range = [&]() {
    // A step with fewer tiles than ranges has pieces of one tile, each rounded against its own maximum.  (Two tiles to a
    // piece, the second rounded against the first one's maximum, made one session of 1777 tokens 14.2 instead of 15.7 us and
    // its error against 64 bits 2.16e-3 instead of 2.02e-3.)
    per_wg = (total + p.dec_ranges - 1) / p.dec_ranges;
    range_begin = wg * per_wg;
    range_end = min(total, range_begin + per_wg);
  };
  auto first_past = [&](int incl) { return __builtin_ctzll(__ballot(range_begin < incl) | (1ull << 63)); };
  // Above 64 sessions the waves add up the chunks of 64 in turn first, and the range's chunk is read once more.  (A thread
  // that walked n_sessions / threads sessions one after the other: 4096 sessions of up to 128 tokens, one kv-head 95 us, four
  // 187, eight 289; this way 62, 151 and 289.)
  static_assert(kSchedMaxSessions <= 64 * 64, "one lane per chunk");
  __shared__ int chunk_sums[64][2];
  int chunk = 0, incl, units;  // inclusive sums up to the lane's session
  if (p.n_sessions <= 64) {
    take_chunk(0);
    incl = wave_inclusive_scan(my_tiles);
    units = wave_inclusive_scan(my_units);
    total = __builtin_amdgcn_readlane(incl, 63);
    n_units = __builtin_amdgcn_readlane(units, 63);
    take_range();
  } else {
    const int n_chunks = (p.n_sessions + 63) >> 6;
#pragma unroll 4
    for (int c = wave; c < n_chunks; c += HW) {
      take_chunk(c);
      const int t = wave_inclusive_scan(my_tiles), u = wave_inclusive_scan(my_units);
      if (lane_s == 63) {
        chunk_sums[c][0] = t;
        chunk_sums[c][1] = u;
      }
    }
    __syncthreads();
    const int t = lane_s < n_chunks ? chunk_sums[lane_s][0] : 0, u = lane_s < n_chunks ? chunk_sums[lane_s][1] : 0;
    const int t_incl = wave_inclusive_scan(t), u_incl = wave_inclusive_scan(u);
    total = __builtin_amdgcn_readlane(t_incl, 63);
    n_units = __builtin_amdgcn_readlane(u_incl, 63);
    take_range();
    chunk = first_past(t_incl);
    take_chunk(chunk);
    incl = wave_inclusive_scan(my_tiles) + __builtin_amdgcn_readlane(t_incl, chunk) - __builtin_amdgcn_readlane(t, chunk);
    units = wave_inclusive_scan(my_units) + __builtin_amdgcn_readlane(u_incl, chunk) - __builtin_amdgcn_readlane(u, chunk);
  }
  // Where the range begins.  Units are numbered in session order.  The range that has a unit's first tile writes its record,
  // block 0 those of the numbers past the last unit.  (More units than records would be lengths that break the caller's
  // contract.)
  const int owner = first_past(incl);
  int s = 64 * chunk + owner;
  int N = __builtin_amdgcn_readlane(my_N, owner);
  int P = __builtin_amdgcn_readlane(my_P, owner);
  int cu = __builtin_amdgcn_readlane(my_cu, owner);
  int unit_begin = __builtin_amdgcn_readlane(incl, owner) - __builtin_amdgcn_readlane(my_tiles, owner);
  int unit = __builtin_amdgcn_readlane(units, owner) - __builtin_amdgcn_readlane(my_units, owner);
  int t0 = 0;
  while (t0 + m < N && unit_begin + tiles_to(P, t0 + m) <= range_begin) {
    unit_begin += tiles_to(P, t0 + m);
    t0 += m;
    ++unit;
  }
  if (blockIdx.x == 0) {
    const bool dropped = p.cu_new_lens[p.n_sessions] > p.total_new_tokens;
    if (tid < kAttnHdrInts)
      p.hdr[tid] = tid == kHdrDecTiles ? total : tid == kHdrPlan ? kPlanDecode : (tid == kHdrFlags && dropped ? 2 : 0);
    for (int i = n_units + tid; i < p.dec_records; i += 64 * HW) p.dec_merges[i] = MergeItem{0, 0, 0, 0};
  }
  if (range_begin >= range_end) return;
  for (int pos = range_begin; pos < range_end;) {
  const int cu_s = cu + t0;                                    // the unit's first row
  const int n_end = min(N, t0 + m);                            // its tokens: t0 .. n_end - 1
  const int n_unit = n_end - t0;
  const int unit_end = unit_begin + tiles_to(P, n_end);
  const int u_begin = pos - unit_begin;                        // this segment: tiles [u_begin, u_end) of the unit
  const int u_end = min(range_end, unit_end) - unit_begin;
  const bool whole = u_begin == 0 && u_end == unit_end - unit_begin;
  const bool at_range_start = pos == range_begin;
  pos = unit_begin + u_end;

  const int lane = tid & 63;
  const int n = lane & 31;
  const int g2 = lane >> 5;
  // a wave holds the 32 query rows of its kv-head: row n = head n / BMTD, token n % BMTD
  const int hh = n / BMTD;
  const int tt = n - hh * BMTD;
  const bool q_valid = tt < n_unit;
  const int head = kvh * G + hh;

  bf16x8 qreg[8];
  {
    const __bf16* qp = p.q + ((int64_t)(cu_s + (q_valid ? tt : 0)) * p.n_q_heads + head) * kD + 8 * g2;
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      qreg[st] = *reinterpret_cast<const bf16x8*>(qp + 16 * st);
      if (!q_valid) {
#pragma unroll
        for (int e = 0; e < 8; ++e) qreg[st][e] = (__bf16)0.0f;
      }
    }
  }

  const int total_keys = P + n_end;  // keys past the unit's last token are masked for all its rows
  const int fast_end = min(u_end, P / kSub);  // tiles below lie entirely inside the paged prefix

  const bool has_table = p.table != nullptr && p.table_stride > 0;
  const int32_t* table_row = p.table + (int64_t)s * p.table_stride;
  const unsigned row_bytes = p.row_bytes;
  // a wave loads all eight row groups of a tile: lane l fetches row l/16 of the group's four, logical 16-byte chunk
  // (l % 16) ^ ((l/16) << 2)
  const unsigned voff = (unsigned)(lane >> 4) * row_bytes + (unsigned)kvh * 256u +
                        (unsigned)((lane & 15) ^ (((lane >> 4) & 3) << 2)) * 16u;
  const char* k_bytes = reinterpret_cast<const char*>(p.k_layer);
  const char* v_bytes = reinterpret_cast<const char*>(p.v_layer);
  char* const my_lds = lds + wave * kDecWaveBytes;  // K, then V

  // Ids of the two 16-row blocks of tile u (index clamped to the table); uniform addresses in read-only memory, so
  // these are scalar loads that do not count among the vector loads the waits below wait for.
  struct Ids {
    int a, b;
  };
  auto fetch_ids = [&](int u) {
    typedef const int32_t __attribute__((address_space(4))) * ConstTable;
    ConstTable row = (ConstTable)(uintptr_t)table_row;
    Ids r{-1, -1};
    if (has_table) {
      r.a = row[min((u * kSub) >> lb, p.table_stride - 1)];
      r.b = row[min((u * kSub + 16) >> lb, p.table_stride - 1)];
    }
    return r;
  };
  // The K rows (which = 0) or the V rows (1) of tile u into this wave's buffer for them: eight loads
  auto issue_half = [&](const int which, int u, const Ids ids) {
    char* const buf = my_lds + which * kSubBytes;
    const char* const pool = which ? v_bytes : k_bytes;
    const bool fast = u < fast_end && max((unsigned)ids.a, (unsigned)ids.b) < (unsigned)p.n_blocks;
    if (fast) {
#pragma unroll
      for (int g = 0; g < 8; ++g) {
        uint64_t off = (uint64_t)(unsigned)(g < 4 ? ids.a : ids.b) * p.block_bytes + (uint64_t)(4 * (g & 3)) * row_bytes;
        if (LB != 4) off += (uint64_t)((u * kSub + 16 * (g >> 2)) & bs_mask) * row_bytes;
        const char* base = pool + off;  // scalar base + 32-bit lane offset, as in attn_mfma_kernel
        unsigned lane_off = voff;
        asm("" : "+s"(base), "+v"(lane_off));
        SYMPH_GLDS16_NT(base + lane_off, buf + g * kGroupBytes);  // every cached row is read once per kv-head
      }
      asm volatile("; end of the scalar-base loads");
    } else {
      const unsigned in_row = (unsigned)kvh * 256u + (unsigned)((lane & 15) ^ (((lane >> 4) & 3) << 2)) * 16u;
      const char* const zeros = reinterpret_cast<const char*>(kZeroRow) + (lane & 15) * 16;
      const char* const fresh = reinterpret_cast<const char*>(which ? p.v_new : p.k_new);
#pragma unroll
      for (int g = 0; g < 8; ++g) {
        const int key = u * kSub + 4 * g + (lane >> 4);
        const unsigned bid = (unsigned)(g < 4 ? ids.a : ids.b);
        const bool in_pool = key < P && (key >> lb) < p.table_stride && bid < (unsigned)p.n_blocks;
        const bool in_new = key >= P && key < total_keys;
        const char* src = zeros;
        if (in_pool)
          src = pool + (uint64_t)bid * p.block_bytes + (uint64_t)(key & bs_mask) * row_bytes + in_row;
        else if (in_new)
          src = fresh + (uint64_t)(cu_s - t0 + key - P) * row_bytes + in_row;
        SYMPH_GLDS16(src, buf + g * kGroupBytes);
      }
    }
  };

  // ---- LDS reads: the fragment layouts of attn_mfma_kernel, for one 32-key block
  const int krow = key_of_row(n);
  const int k_lane = (krow >> 2) * kGroupBytes + (krow & 3) * 256 + g2 * 16;
  int k_off[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) k_off[q] = k_lane + 64 * (q ^ (krow & 3));
  const int i16 = lane & 15;
  const int vrow = 8 * g2 + (i16 >> 2);
  const int v_lane = (vrow >> 2) * kGroupBytes + (vrow & 3) * 256 + 32 * ((lane >> 4) & 1) + 8 * (i16 & 3);
  int v_off[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) v_off[dt] = v_lane + 64 * (dt ^ (vrow & 3));

  f32x16 o_acc[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o_acc[dt][e] = 0.f;
  float m_run = -INFINITY;  // softmax reference in log2 units, -inf: no key seen yet
  float mb = 0.f;           // the same, finite
  float l_run = 0.f;
  const float cs = p.scale_log2e;
  const int q_limit = P + t0 + tt;
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

  auto exps = [&](const f32x16& sc, bf16x8 (&pb)[2]) {
#pragma unroll
    for (int e = 0; e < 16; ++e) pb[e >> 3][e & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sc[e], cs, -mb));
    float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const bf16x8 v = pb[u];
      ps0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v[0], v[1]}, ones, ps0, false);
      ps1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v[2], v[3]}, ones, ps1, false);
      ps0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v[4], v[5]}, ones, ps0, false);
      ps1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v[6], v[7]}, ones, ps1, false);
    }
    return ps0 + ps1;
  };
  // reference := max(reference, maximum of this tile); everything accumulated so far is rescaled
  auto raise_reference = [&](const f32x16& sc) {
    float mx = sc[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[e]);
    mx = max_across_halves(mx);
    const float m_new = fmaxf(m_run, mx * cs);
    const float a = (m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
    m_run = m_new;
    mb = (m_new == -INFINITY) ? 0.f : m_new;
    l_run *= a;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) o_acc[dt][e] *= a;
  };

  bf16x8 pb[2];  // the tile's probabilities, from scores_of_tile to values_of_tile
  auto scores_of_tile = [&](const int u, const bool first) {
    const char* const kb_cur = my_lds;
    // ---- S^T = K Q^T
    f32x16 sc;
#pragma unroll
    for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const bf16x8 frag = *reinterpret_cast<const bf16x8*>(kb_cur + k_off[g >> 1] + 32 * (g & 1));
      sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag, qreg[g], sc, 0, 0, 0);
    }
    // causal mask: only tiles that reach past the first query's limit
    if (u * kSub + kSub - 1 > P + t0) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int key = u * kSub + 16 * (e >> 3) + 8 * g2 + (e & 7);
        if (key > q_limit) sc[e] = -INFINITY;
      }
    }
    // ---- probabilities against the (stale) reference
    if (first) raise_reference(sc);
    float ps = exps(sc, pb);
    if (__any(!(ps <= kRefreshSum) || (m_run == -INFINITY && ps > 0.f))) {
      raise_reference(sc);
      ps = exps(sc, pb);
    }
    l_run += ps;
  };
  auto values_of_tile = [&]() {
    const char* const vb_cur = my_lds + kSubBytes;
    // ---- O^T += V^T P^T
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const char* vp = vb_cur + v_off[dt] + 4 * ks * kGroupBytes;
        const s16x4 lo = lds_read_tr16(reinterpret_cast<const __bf16*>(vp));
        const s16x4 hi = lds_read_tr16(reinterpret_cast<const __bf16*>(vp + kGroupBytes));
        const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        o_acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pb[ks], o_acc[dt], 0, 0, 0);
      }
  };

  // ---- the segment's tiles, one after the other; the buffers are the wave's own.  The K buffer is refilled with the
  // next tile's rows as soon as the scores are done, the V buffer as soon as the values are, so one of the two is
  // always on its way while the other is used.  Loads return in order: "all but the last eight" is exactly the older
  // of the two halves.  The waves of a workgroup read the slices of the SAME token rows, one kv-head each, and a
  // barrier per tile keeps them together: whole 2 KiB rows are fetched at about the same time (a stream of full rows
  // runs 5 % faster than the same bytes as eight independent streams of 256-byte slices).
  {
    bool first = true;
    int u = u_begin;
    Ids ids = fetch_ids(u);
    if (u < u_end) {
      issue_half(0, u, ids);
      issue_half(1, u, ids);
    }
    for (; u < u_end; ++u) {
      const bool more = u + 1 < u_end;
      const Ids ids_next = fetch_ids(u + 1);
      if (HW > 1) __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_s_waitcnt(0x0F70 | 8);  // vmcnt(8): K(u) has landed, V(u) may be on its way
      asm volatile("" ::: "memory");
      scores_of_tile(u, first);
      first = false;
      asm volatile("" ::: "memory");
      if (more) issue_half(0, u + 1, ids_next);
      if (more)
        __builtin_amdgcn_s_waitcnt(0x0F70 | 8);  // V(u) has landed, K(u+1) may be on its way
      else
        __builtin_amdgcn_s_waitcnt(0x0F70);
      asm volatile("" ::: "memory");
      values_of_tile();
      asm volatile("" ::: "memory");
      if (more) issue_half(1, u + 1, ids_next);
    }
  }

  const float l_row = sum_across_halves(l_run);
  if (whole) {
    if (kvh == 0 && lane == 0 && unit < p.dec_records) p.dec_merges[unit] = MergeItem{0, 0, 0, 0};
    if (q_valid)
      store_out_row(p.out + ((int64_t)(cu_s + tt) * p.n_q_heads + head) * kD, o_acc, 1.0f / l_row, g2);
  } else {
    // Two slots per range: 2 * wg for a segment that starts where the range starts (a unit continued from the range
    // before), 2 * wg + 1 for one that starts inside it.  The pieces of a unit are then its first one and, for every
    // further range it reaches into, that range's even slot.
    const int pslot = 2 * wg + (at_range_start ? 0 : 1);
    if (u_begin == 0 && kvh == 0 && lane == 0 && unit < p.dec_records)
      p.dec_merges[unit] = MergeItem{cu_s, n_unit, pslot, (unit_end - 1) / per_wg - wg + 1};
    // The piece goes through the wave's LDS buffers into the packed layout, so that every store instruction writes
    // whole lines (the wave's own reads of the buffers are done: it has used the last tile).
    const int rows = G * n_unit;
    const int n_floats = rows * 130;
    const int n_padded = (n_floats + 31) & ~31;
    float* const stage = reinterpret_cast<float*>(my_lds);
    if (q_valid) {
      const int r = hh * n_unit + tt;
      float* so = stage + r * 128 + 4 * g2;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) so[32 * dt + 8 * i + j] = o_acc[dt][4 * i + j];
      if (g2 == 0) {
        stage[rows * 128 + r] = l_row == l_row ? m_run : 0.f;  // (NaN scores only: not a piece that saw no key)
        stage[rows * 129 + r] = l_row;
      }
    }
    if (n_floats + lane < n_padded) stage[n_floats + lane] = 0.f;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    float* part = DecSlots(p, n_unit, kvh)[pslot];
    for (int idx = lane; idx < n_padded; idx += 64) part[idx] = stage[idx];
    __builtin_amdgcn_wave_barrier();
  }
  unit_begin = unit_end;
  ++unit;
  t0 += m;
  if (t0 >= N && pos < range_end) {  // the next session with new tokens (there is one: tiles are left)
    t0 = 0;
    do {
      ++s;
      span_of(s, cu, N, P);
    } while (N == 0);
  }
  }
}

// Combine the pieces of a unit that the decode kernel cut at the boundaries of its ranges:
// out = sum_c w_c O_c / sum_c w_c l_c with w_c = 2^(m_c - max_c m_c), m_c being the piece's softmax reference in log2
// units (-inf: the piece saw no key of the row).  The first piece is in slot pslot0, piece c >= 1 in the even slot of
// the c-th range after the one that wrote pslot0.
// A workgroup takes RW rows of a (record, kv-head) at a time: half-wave h has row h % RW of them and every (8 / RW)-th piece
// from h / RW on, eight in flight.  A merge is nothing but trips to memory, so few units get a workgroup per row, which asks
// for up to 64 pieces at once: one session of 1777 tokens in 56 pieces, 50 us by a thread that read one piece after the
// other, 8 us by four waves that asked for sixteen at once, 3.7 us this way.  Many units have few pieces each and get
// four rows per workgroup: fewer workgroups, no half-wave without a piece to read.
// Records are per unit, not per key range, so that the grid follows the batch: 8 instead of 2048 workgroups for one session
// (14.9 -> 14.4 us with the lengths added up inside a wave for up to 64 sessions, without a barrier).
template <int G, int RW>
__global__ __launch_bounds__(256) void attn_decode_merge_kernel(const MfmaParams p) {
  constexpr int kParts = 8 / RW;  // half-waves per row
  constexpr int kAtOnce = 8;
  __shared__ f32x4 part_o[8][32];
  __shared__ float part_m[8], part_l[8];
  const int Hkv = p.n_kv_heads;
  const int record = blockIdx.x / Hkv;
  const MergeItem mg = p.dec_merges[record];
  if (mg.n_chunks == 0) return;
  const int kvh = blockIdx.x - record * Hkv;
  const int range = mg.pslot0 >> 1;
  const int n_unit = mg.n_unit;
  const int rows = G * n_unit;
  const int half = threadIdx.x >> 5, c4 = threadIdx.x & 31;  // columns 4 * c4 .. + 3
  const DecSlots slots(p, n_unit, kvh);
  auto piece = [&](int c) { return slots[c == 0 ? mg.pslot0 : 2 * (range + c)]; };
  for (int r0 = RW * blockIdx.y; r0 < rows; r0 += RW * gridDim.y) {
    const int row = r0 + half % RW;
    f32x4 o{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;
    for (int c0 = half / RW; c0 < mg.n_chunks; c0 += kParts * kAtOnce) {
      f32x4 oc[kAtOnce];
      float mc[kAtOnce], lc[kAtOnce];
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) {
        const int c = c0 + kParts * k;
        mc[k] = -INFINITY;
        lc[k] = 0.f;
        if (c < mg.n_chunks && row < rows) {
          const float* const src = piece(c);
          oc[k] = *reinterpret_cast<const f32x4*>(src + row * 128 + 4 * c4);
          mc[k] = src[rows * 128 + row];
          lc[k] = src[rows * 129 + row];
        }
      }
      float m_new = m_run;
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) m_new = fmaxf(m_new, mc[k]);
      if (m_new == -INFINITY) continue;
      const float a = __builtin_amdgcn_exp2f(m_run - m_new);  // (0 for the first pieces)
      m_run = m_new;
      l_run *= a;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] *= a;
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) {
        if (mc[k] == -INFINITY) continue;  // absent, or it saw no key of the row
        const float w = __builtin_amdgcn_exp2f(mc[k] - m_new);
        l_run = fmaf(w, lc[k], l_run);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = fmaf(w, oc[k][e], o[e]);
      }
    }
    if (r0 > RW * (int)blockIdx.y) __syncthreads();  // the rows before have been read
    part_o[half][c4] = o;
    if (c4 == 0) {
      part_m[half] = m_run;
      part_l[half] = l_run;
    }
    __syncthreads();
    if (half < RW && row < rows) {  // the row's half-waves, in order
      float M = -INFINITY, L = 0.f;
#pragma unroll
      for (int k = 0; k < kParts; ++k) M = fmaxf(M, part_m[half + RW * k]);
      f32x4 sum{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < kParts; ++k) {
        const float mk = part_m[half + RW * k];
        const float f = mk == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mk - M);
        L = fmaf(f, part_l[half + RW * k], L);
        const f32x4 ok = part_o[half + RW * k][c4];
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] = fmaf(f, ok[e], sum[e]);
      }
      const float inv = 1.0f / L;
      const int hh = row / n_unit, tt = row - hh * n_unit;
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (__bf16)(sum[e] * inv);
      *reinterpret_cast<bf16x4*>(p.out + ((int64_t)(mg.row0 + tt) * p.n_q_heads + (kvh * G + hh)) * kD + 4 * c4) = v;
    }
  }
}

// ------------------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------------------
// Tuning values with the defaults filled in (a field of symph_attn_tuning that is 0 keeps its default).
struct AttnTuning {
  int32_t slots, c_min, coarse, decode, decode_wgs;
  int32_t direct = 1;  // (no field of symph_attn_tuning: 0 asks make_plan for the work list)
};
static AttnTuning resolve_tuning(const symph_attn_tuning* t) {
  AttnTuning r{512, 8, 1, 1, 512, 1};  // 512 slots: 256 compute units x 2 resident workgroups
  if (t) {
    if (t->slots > 0) r.slots = t->slots;
    if (t->c_min > 0) r.c_min = t->c_min;
    if (t->coarse != 0) r.coarse = t->coarse > 0;
    if (t->decode != 0) r.decode = t->decode > 0;
    if (t->decode_wgs > 0) r.decode_wgs = t->decode_wgs;
  }
  return r;
}

// A workgroup per row in the merge of a decode step up to this many rows (1 / 4 rows per workgroup: one session of 1777 tokens
// 12.3 / 13.7 us, of 16 000 in one kv-head 17.1 / 41.8, 8 of 2000 to 4000 26.1 / 27.0, 16 and 32 sessions the same, 64 70.8 /
// 69.7, 256 79.3 / 75.0); above it at most this many workgroups, as far as one per record and kv-head allows.
constexpr int64_t kMergeSingleRows = 1024, kMergeGroups = 4096;

// Direct calls: (unit, kv-head) pairs up to which a merge has sixteen workgroups each; above it four.  The pairs are the bound
// that the grid is made for, total_new_tokens / bmt + n_sessions units: two turns of 22 tokens in groups of four count
// as three units.  Four /
// sixteen, in us: 16 pairs 18.7 / 17.5, 24 20.0 / 19.4, 32 22.5 / 22.9 (one turn) and 19.2 / 18.1 (two), 48 26.0 / 26.7, 64
// 22.2 / 22.3 and 47.0 / 48.0, 96 25.4 / 26.3, 128 34.5 / 35.0, 192 47.9 / 50.8, 264 63.8 / 67.9.
constexpr unsigned kMergeFewPairs = 32;

struct MfmaPlan {
  int32_t bmt, target, target_slots, c_min, coarse, units_bound, items_bound, merges_bound, pslots_bound;
  // decode kernel: whether this call runs it (alone), its key ranges (two slots per kv-head each), the new tokens of a unit,
  // its units' records
  int32_t dec_mode, dec_wgs, dec_m, dec_records, dec_slot_floats, dec_long_slot_floats;
  int32_t direct;  // no scheduling kernel: pslots_bound pieces at most, one record per unit
  int64_t off_items, off_dec_merges, off_merge_cnt, off_partials, off_dec_partials, off_dec_long, total_bytes;
};

constexpr int kDirectCMin = 2;  // shortest piece of a direct call, in tiles

static inline int64_t align256(int64_t x) { return (x + 255) & ~(int64_t)255; }

static void lay_out(MfmaPlan& pl, int32_t n_kv_heads) {
  pl.items_bound = pl.units_bound + pl.pslots_bound;  // every unit once, plus one more item per chunk of a split unit
  pl.merges_bound = pl.pslots_bound / 2;              // a split unit has at least two chunks
  pl.off_items = align256(kAttnHdrInts * 4);
  pl.off_dec_merges = align256(pl.off_items + (pl.direct ? 0 : (int64_t)pl.items_bound * sizeof(WorkItem)));
  pl.off_merge_cnt = align256(pl.off_dec_merges + (int64_t)(pl.direct ? pl.units_bound : pl.dec_records) * sizeof(MergeItem));
  pl.off_partials = align256(pl.off_merge_cnt + (int64_t)pl.merges_bound * n_kv_heads * 4);
  pl.off_dec_partials = pl.off_partials + (int64_t)pl.pslots_bound * n_kv_heads * kPartialFloats * 4;
  pl.off_dec_long = pl.off_dec_partials + (int64_t)2 * pl.dec_wgs * n_kv_heads * pl.dec_slot_floats * 4;
  pl.total_bytes = pl.off_dec_long + (int64_t)2 * pl.dec_wgs * n_kv_heads * pl.dec_long_slot_floats * 4;
}

// Sizes that depend only on host-visible bounds and the tuning values, so that the workspace query and the launch
// agree.  budget_bytes > 0: the plan has to fit that many bytes; the decode kernel then gets fewer workgroups and the
// work list is cut into fewer pieces (fewer partial-result slots).  Returns false if not even the uncut list fits.
static bool make_plan(MfmaPlan& pl, int32_t n_sessions, int32_t n_q_heads, int32_t n_kv_heads,
                      int32_t total_new_tokens, int32_t max_new_len, int32_t max_prefix_len, const AttnTuning& tu,
                      int64_t budget_bytes) {
  const int G = n_q_heads / n_kv_heads;
  pl.bmt = 128 / G;
  pl.target_slots = tu.slots < n_kv_heads ? n_kv_heads : tu.slots;  // workgroups resident at once
  pl.target = 2 * pl.target_slots;                                  // most pieces the batch is ever cut into
  pl.c_min = tu.c_min;
  pl.coarse = tu.coarse;
  pl.units_bound = total_new_tokens / pl.bmt + n_sessions;
  // A batch in which no session has more new rows than one wave holds (decode steps) takes the decode kernel: one
  // equal share of the keys per workgroup, two partial-result slots per workgroup.  Mixed batches do not: their short
  // turns are memory-bound pieces that share the CUs with the compute-bound ones inside the main kernel, which
  // measured faster than two kernels one after the other.  A session longer than max_new_len is taken dec_m tokens at a time
  // and its prefix is streamed once for each of them; more tokens than n_sessions * max_new_len show that the bound is wrong,
  // and the batch is then no decode step.
  pl.dec_mode = tu.decode && max_new_len >= 1 && max_new_len <= 32 / G &&
                total_new_tokens <= (int64_t)n_sessions * max_new_len;
  // ranges of the decode kernel: one wave per (range, kv-head), as many waves as decode_wgs workgroups of four would have
  pl.dec_wgs = pl.dec_mode ? (4 * tu.decode_wgs / n_kv_heads < 1 ? 1 : 4 * tu.decode_wgs / n_kv_heads) : 0;
  pl.dec_m = pl.dec_records = pl.dec_slot_floats = pl.dec_long_slot_floats = 0;
  // Units of m tokens: at most one per token, or one per session and full m tokens; a piece has at most G rows of 130 values
  // per token of its unit, in a slot of whole lines.
  auto set_unit_tokens = [&](int32_t m) {
    const int64_t units = (int64_t)total_new_tokens / m + n_sessions;
    pl.dec_m = m;
    pl.dec_records = (int32_t)(units < total_new_tokens ? units : total_new_tokens);
    pl.dec_slot_floats = (G * max_new_len * 130 + 31) & ~31;
    pl.dec_long_slot_floats = m > max_new_len ? (G * m * 130 + 31) & ~31 : 0;
  };
  // Chunks of split units: a unit is split when it has more than C tiles, C >= total tiles * kv-heads / target, so
  // there are at most target / kv-heads split units and their chunks number at most twice that.
  pl.pslots_bound = 2 * (pl.target / n_kv_heads + 1);
  if (pl.dec_mode) {
    // No work list.  A unit has as many tokens as a wave has rows for, so that a session longer than stated (96 tokens over
    // 16 384, stated as 1) is streamed 12 times and not 96: 151 instead of 600 us; shorter ones are one unit either way.
    // Where the slots do not fit, units go down to the stated length, then the ranges are halved.
    pl.units_bound = pl.pslots_bound = pl.direct = 0;
    set_unit_tokens(32 / G);
    lay_out(pl, n_kv_heads);
    while (budget_bytes > 0 && pl.total_bytes > budget_bytes && (pl.dec_m > max_new_len || pl.dec_wgs > 1)) {
      if (pl.dec_m > max_new_len)
        set_unit_tokens(pl.dec_m / 2 > max_new_len ? pl.dec_m / 2 : max_new_len);
      else
        pl.dec_wgs /= 2;
      lay_out(pl, n_kv_heads);
    }
    return budget_bytes <= 0 || pl.total_bytes <= budget_bytes;
  }
  // Direct calls: few units, and few enough for the chip.  Cutting what fills it half already gains little, and a cut that
  // takes a second round of workgroups loses; a long turn's units grow with their place in it, so that the work list's
  // longest-first order is worth more than the scheduling kernel, unless a much longer prefix makes them alike.  Below half
  // of the slots the list is as fast only for such turns (groups of four on four kv-heads: 1500 new tokens over none, 32.9 us by
  // the list, 31.9 directly; 2 x 772 over 129, 30.5 and 30.3; but 3 x 600 over 15 000 on two, 164 and 128).  Above it short
  // turns over short prefixes are better listed (groups of four on eight: 16 x 78 over 99, 19.6 and 21.0; 20 x 70 over 300, 25.4
  // and 28.2), long prefixes cut directly (8 x 143 over 1724, 77 and 56; 512 over 32 768 in groups of eight, 504 and 502) up to
  // five sixths of the slots (6 x 343 over 5656 in groups of two, 144 and 147).  The lines were fitted to 175 batches of 1 to 60
  // sessions, 0 to 20 000 cached tokens and 1 to 2000 new ones with the list and direct calls of that time.  Both have become
  // faster since, direct calls more, and the lines were left where they were (a batch that changes sides is cut elsewhere, and
  // its outputs are others): 30 x 30 over 700 or 800 is listed and takes 44.7 and 47.4 us where a direct call takes 31.6 and
  // 34.8, 34 x 5 .. 20 over 500 in groups of eight 40 and 28.
  const int64_t wg_units = pl.units_bound * (int64_t)n_kv_heads;
  const bool short_turns = max_new_len * wg_units <= 160 * (int64_t)tu.slots;
  const bool direct_pays =
      2 * wg_units < tu.slots
          ? short_turns || max_prefix_len >= 8 * (int64_t)max_new_len
          : 6 * wg_units < 5 * (int64_t)tu.slots && max_prefix_len >= 768 &&
                max_prefix_len >= (short_turns ? 4 : 8) * (int64_t)max_new_len;
  pl.direct = tu.direct && tu.coarse && pl.units_bound <= kDirectUnits && direct_pays;
  if (pl.direct) {
    const int32_t listed = pl.pslots_bound;
    pl.pslots_bound = pl.target_slots / n_kv_heads + 1 + pl.units_bound;
    lay_out(pl, n_kv_heads);
    if (budget_bytes <= 0 || pl.total_bytes <= budget_bytes) return true;
    pl.direct = 0;
    pl.pslots_bound = listed;
  }
  lay_out(pl, n_kv_heads);
  if (budget_bytes <= 0 || pl.total_bytes <= budget_bytes) return true;
  // the work list gets as many partial-result slots as the room beside the uncut list holds
  const int64_t slot_bytes = (int64_t)n_kv_heads * kPartialFloats * 4;
  const int32_t wanted = pl.pslots_bound;
  pl.pslots_bound = 0;
  lay_out(pl, n_kv_heads);
  const int64_t per_slot = slot_bytes + (int64_t)sizeof(WorkItem) + 4 * n_kv_heads;
  const int64_t room = budget_bytes - pl.total_bytes - 4 * 256;  // (the arrays are aligned to 256 bytes)
  if (room < 0) return false;
  const int64_t fit = room / per_slot;
  pl.pslots_bound = (int32_t)(fit < wanted ? fit : wanted) & ~1;
  const int64_t pieces = (int64_t)(pl.pslots_bound / 2) * n_kv_heads;  // (the bound above, solved for the target)
  if (pieces < pl.target) pl.target = pieces < n_kv_heads ? n_kv_heads : (int32_t)pieces;
  if (pl.target_slots > pl.target) pl.target_slots = pl.target;
  lay_out(pl, n_kv_heads);
  return pl.total_bytes <= budget_bytes;
}

static bool mfma_path_ok(int32_t dtype, int32_t head_dim, int32_t n_q_heads, int32_t n_kv_heads, int32_t block_size) {
  if (dtype != SYMPH_BF16 || head_dim != 128) return false;
  const int G = n_q_heads / n_kv_heads;
  if (G != 1 && G != 2 && G != 4 && G != 8 && G != 16) return false;
  return block_size >= 16 && (block_size & (block_size - 1)) == 0;
}

int64_t prefill_attn_workspace_bytes(const symph_kv_cache* c, int32_t n_sessions, int32_t n_q_heads,
                                     int32_t total_new_tokens, int32_t max_new_len, int32_t max_prefix_len,
                                     const symph_attn_tuning* tuning) {
  if (n_q_heads % c->n_kv_heads != 0) return -1;
  if (!mfma_path_ok(c->dtype, c->head_dim, n_q_heads, c->n_kv_heads, c->block_size)) return 0;
  MfmaPlan pl, listed;
  AttnTuning tu = resolve_tuning(tuning);
  make_plan(pl, n_sessions, n_q_heads, c->n_kv_heads, total_new_tokens, max_new_len, max_prefix_len, tu, 0);
  // Never less than the work list needs, so that a workspace serves the same batch whichever kernels its tuning values or
  // its bounds choose (the other plans are smaller).
  tu.decode = tu.direct = 0;
  make_plan(listed, n_sessions, n_q_heads, c->n_kv_heads, total_new_tokens, max_new_len, max_prefix_len, tu, 0);
  return pl.total_bytes > listed.total_bytes ? pl.total_bytes : listed.total_bytes;
}

template <int G>
static int32_t launch_mfma(const AttnArgs& a, hipStream_t stream) {
  MfmaPlan pl;
  const AttnTuning tu = resolve_tuning(a.tuning);
  char* ws = (char*)a.workspace;
  // fit_workspace: the caller's buffer has a fixed size and the plan is made to fit it (a coarser cut of the work list)
  if (!make_plan(pl, a.n_sessions, a.n_q_heads, a.n_kv_heads, a.total_new_tokens, a.max_new_len, a.max_prefix_len, tu,
                 a.fit_workspace ? a.workspace_bytes : 0) ||
      !ws || a.workspace_bytes < pl.total_bytes)
    return SYMPH_EWORKSPACE;
  if (((uintptr_t)ws & 255) != 0) return SYMPH_EUNSUPPORTED;

  SchedParams sp;
  sp.cu_new_lens = a.cu_new_lens;
  sp.prefix_lens = a.prefix_lens;
  sp.n_sessions = a.n_sessions;
  sp.bmt = pl.bmt;
  sp.n_kv_heads = a.n_kv_heads;
  sp.target = pl.target;
  sp.target_slots = pl.target_slots;
  sp.coarse_ok = pl.coarse;
  sp.c_min = pl.c_min;
  sp.items_bound = pl.items_bound;
  sp.merges_bound = pl.merges_bound;
  sp.pslots_bound = pl.pslots_bound;
  sp.hdr = (int32_t*)ws;
  sp.items = (WorkItem*)(ws + pl.off_items);
  sp.merge_cnt = (int32_t*)(ws + pl.off_merge_cnt);
  sp.table = a.table;
  sp.table_stride = a.table_stride;
  sp.log_bs = __builtin_ctz((unsigned)a.block_size);

  MfmaParams p;
  p.k_layer = (const __bf16*)a.k_layer;
  p.v_layer = (const __bf16*)a.v_layer;
  p.block_stride = a.block_stride;
  p.block_bytes = (uint32_t)(a.block_stride * 2);
  p.row_bytes = (uint32_t)a.n_kv_heads * kD * 2u;
  p.n_blocks = a.n_blocks;
  p.log_bs = __builtin_ctz((unsigned)a.block_size);
  p.n_kv_heads = a.n_kv_heads;
  p.n_q_heads = a.n_q_heads;
  p.q = (const __bf16*)a.q;
  p.k_new = (const __bf16*)a.k_new;
  p.v_new = (const __bf16*)a.v_new;
  p.out = (__bf16*)a.out;
  p.cu_new_lens = a.cu_new_lens;
  p.prefix_lens = a.prefix_lens;
  p.table = a.table;
  p.table_stride = a.table_stride;
  p.n_sessions = a.n_sessions;
  p.scale_log2e = a.scale * 1.4426950408889634f;
  p.hdr = sp.hdr;
  p.items = sp.items;
  p.merge_cnt = sp.merge_cnt;
  p.dec_m = pl.dec_m;
  p.total_new_tokens = a.total_new_tokens;
  p.dec_ranges = pl.dec_wgs;
  p.dec_records = pl.dec_records;
  p.direct_c_min = a.tuning && a.tuning->c_min > 0 ? a.tuning->c_min : kDirectCMin;
  p.direct_slots = pl.target_slots;
  p.units_bound = pl.units_bound;
  p.dec_merges = p.unit_recs = (MergeItem*)(ws + pl.off_dec_merges);
  p.dec_partials = (float*)(ws + pl.off_dec_partials);
  p.dec_long_partials = (float*)(ws + pl.off_dec_long);
  p.dec_stated = a.max_new_len;
  p.dec_slot_floats = pl.dec_slot_floats;
  p.dec_long_slot_floats = pl.dec_long_slot_floats;
  p.partials = (float*)(ws + pl.off_partials);

  const int64_t g_main = (int64_t)pl.items_bound * a.n_kv_heads;
  const int dec_hw = a.n_kv_heads % 8 == 0 ? 8 : 1;   // kv-heads (= waves) per workgroup of the decode kernel
  const int64_t g_dec = (int64_t)pl.dec_wgs * (a.n_kv_heads / dec_hw);
  const int64_t g_merge = (int64_t)pl.dec_records * a.n_kv_heads;
  if (g_main > 0x7FFFFFFFLL || g_merge > 0x7FFFFFFFLL) return SYMPH_EUNSUPPORTED;
  // The scheduler keeps one table entry per session in LDS (and the decode kernel adds the sessions up in every
  // workgroup): larger batches run as consecutive slices of sessions (same stream, same workspace; the bounds of the
  // whole batch cover every slice).
  for (int32_t s0 = 0; s0 < a.n_sessions; s0 += kSchedMaxSessions) {
    const int32_t ns = a.n_sessions - s0 < kSchedMaxSessions ? a.n_sessions - s0 : kSchedMaxSessions;
    sp.cu_new_lens = a.cu_new_lens + s0;
    sp.prefix_lens = a.prefix_lens + s0;
    sp.n_sessions = ns;
    p.cu_new_lens = sp.cu_new_lens;
    p.prefix_lens = sp.prefix_lens;
    p.table = a.table ? a.table + (int64_t)s0 * a.table_stride : nullptr;
    sp.table = p.table;
    p.n_sessions = ns;
    if (pl.dec_mode) {
      if (dec_hw == 8) {
        if (a.block_size == 16)
          hipLaunchKernelGGL((attn_decode_kernel<G, 4, 8>), dim3((unsigned)g_dec), dim3(512), 0, stream, p);
        else
          hipLaunchKernelGGL((attn_decode_kernel<G, 0, 8>), dim3((unsigned)g_dec), dim3(512), 0, stream, p);
      } else {
        if (a.block_size == 16)
          hipLaunchKernelGGL((attn_decode_kernel<G, 4, 1>), dim3((unsigned)g_dec), dim3(64), 0, stream, p);
        else
          hipLaunchKernelGGL((attn_decode_kernel<G, 0, 1>), dim3((unsigned)g_dec), dim3(64), 0, stream, p);
      }
      // (rows that no workgroup starts with, those of units longer than stated among them, are taken in further turns)
      const int stated_rows = G * a.max_new_len;
      if (g_merge * stated_rows <= kMergeSingleRows) {
        hipLaunchKernelGGL((attn_decode_merge_kernel<G, 1>), dim3((unsigned)g_merge, (unsigned)stated_rows), dim3(256), 0,
                           stream, p);
      } else {
        const int64_t wanted = (stated_rows + 3) / 4, room = kMergeGroups / g_merge;
        const unsigned gy = (unsigned)(wanted < room ? wanted : (room < 1 ? 1 : room));
        hipLaunchKernelGGL((attn_decode_merge_kernel<G, 4>), dim3((unsigned)g_merge, gy), dim3(256), 0, stream, p);
      }
    } else if (pl.direct) {
      const unsigned g_pieces = (unsigned)(pl.pslots_bound * a.n_kv_heads);
      if (a.block_size == 16)
        hipLaunchKernelGGL((attn_mfma_kernel<G, 4, true>), dim3(g_pieces), dim3(256), 0, stream, p);
      else
        hipLaunchKernelGGL((attn_mfma_kernel<G, 0, true>), dim3(g_pieces), dim3(256), 0, stream, p);
      const unsigned pairs = (unsigned)(pl.units_bound * a.n_kv_heads);
      if (pairs <= kMergeFewPairs)
        hipLaunchKernelGGL((attn_merge_kernel<G, 16>), dim3(16 * pairs), dim3(256), 0, stream, p);
      else
        hipLaunchKernelGGL((attn_merge_kernel<G, 4>), dim3(4 * pairs), dim3(256), 0, stream, p);
    } else {
      hipLaunchKernelGGL(attn_schedule_kernel, dim3(1), dim3(kSchedThreads), 0, stream, sp);
      if (a.block_size == 16)
        hipLaunchKernelGGL((attn_mfma_kernel<G, 4, false>), dim3((unsigned)g_main), dim3(256), 0, stream, p);
      else
        hipLaunchKernelGGL((attn_mfma_kernel<G, 0, false>), dim3((unsigned)g_main), dim3(256), 0, stream, p);
    }
  }
  return hipGetLastError() == hipSuccess ? SYMPH_OK : SYMPH_ELAUNCH;
}

int32_t launch_prefill_attn(const AttnArgs& a, hipStream_t stream) {
  const int G = a.n_q_heads / a.n_kv_heads;
  const bool aligned16 = (((uintptr_t)a.k_layer | (uintptr_t)a.v_layer | (uintptr_t)a.q | (uintptr_t)a.k_new |
                           (uintptr_t)a.v_new | (uintptr_t)a.out | (uintptr_t)(a.block_stride * 2)) & 15) == 0;
  if (mfma_path_ok(a.dtype, a.head_dim, a.n_q_heads, a.n_kv_heads, a.block_size) &&
      a.block_stride * 2 <= 0xFFFFFFFFLL) {
    if (!aligned16) return SYMPH_EUNSUPPORTED;
    switch (G) {
      case 1: return launch_mfma<1>(a, stream);
      case 2: return launch_mfma<2>(a, stream);
      case 4: return launch_mfma<4>(a, stream);
      case 8: return launch_mfma<8>(a, stream);
      case 16: return launch_mfma<16>(a, stream);
      default: break;
    }
  }
  return launch_rows_attn(a, stream);
}

// ------------------------------------------------------------------------------------------------------------
// matrix-core reference: nothing but MFMAs on registers, four independent accumulators per wave
// ------------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 2) void mfma_reference_kernel(int iters, float* sink) {
  f32x16 acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  bf16x8 a, b;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    a[e] = (__bf16)(0.001f * (float)(threadIdx.x & 7));
    b[e] = (__bf16)0.5f;
  }
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[i], 0, 0, 0);
  }
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) t += acc[i][3];
  if (t == -1.0f) *sink = t;  // sums of non-negative products: never taken, keeps the accumulators alive
}

int32_t launch_mfma_reference(int32_t iters, int64_t* h_flops, void* d_sink, hipStream_t stream) {
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess) return SYMPH_ELAUNCH;
  if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu <= 0)
    return SYMPH_ELAUNCH;
  const int n_wg = 2 * n_cu;
  if (h_flops) *h_flops = (int64_t)n_wg * 4 * iters * 32 * (2LL * 32 * 32 * 16);
  hipLaunchKernelGGL(mfma_reference_kernel, dim3((unsigned)n_wg), dim3(256), 0, stream, (int)iters, (float*)d_sink);
  return hipGetLastError() == hipSuccess ? SYMPH_OK : SYMPH_ELAUNCH;
}

}  // namespace symph

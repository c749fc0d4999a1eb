// Capacity-limited top-k slotting (Sec. 3), Intra-GPU Rectification (Sec. 4.1), Fill-in
// Rectification (Sec. 4.2) and the Eq. 2 / Eq. 3 combine weights: logits -> tables.
//
// Structure.  The number of tokens an expert keeps in round r depends only on how many candidates
// it received in rounds 0..r (kept = min(candidates, C - filled)), never on WHICH ones were kept.
// So all k top-k rounds and the Fill-in round (the (k+1)-th round at unchanged capacity, Sec. 4.2)
// are planned from candidate counts alone and then resolved concurrently, one workgroup per
// (round, expert) list:
//   topk_rank          per token: ranked experts, score keys, best expert of its own group,
//                      candidate counts per (list, token block)
//   scan_candidates    exclusive scan of those counts over token blocks, per list
//   scatter_candidates stable split of the tokens into per-list arrays (ascending token index);
//                      lists whose kept set follows from the counts (nobody, everybody, the first m
//                      in token order) get their slots here and are not materialised
//   select_slot        per remaining list: kept count and first free slot from the counts,
//                      select the score threshold of the kept set (ties -> lower token
//                      index), then a prefix scan in token order hands out consecutive slots
//   ir_count / ir_scan / ir_weights
//                      per-expert Intra-GPU lists (stable, token order), dispatched-row layout and
//                      row tiles for the grouped GEMM, combine weights
// Plans that are a few dozen numbers (array bases, kept counts, row layout) are recomputed by every
// workgroup that needs them instead of being a launch of their own: a dependent launch costs about
// 6 us on this part, more than any of these kernels needs for a small batch.
// Small batches (one_is_cheaper: up to 1024 tokens, fewer with more experts and rounds) skip all of it: one workgroup
// builds every table (route_small_kernel), from the router's scores or ranks, or from logits - where those are more than
// kOneTile, topk_rank ranks them first.
// Every table is a deterministic function of the logits: integer atomics are only used for counts.
#include <algorithm>
#include <type_traits>

#include "rr_device.h"

namespace rr {

namespace {

constexpr int TS = kMaxE + 1;  // LDS row stride of a [token][expert] tile

// Experts x count blocks up to which ir_weights adds up the counts of the Intra-GPU lists itself, in workgroups of 128 tokens;
// past it in workgroups of 1024, which make an eighth of the blocks and add eight times as fast, up to kIrLargeSelfMax; then the scan
// launch, behind blocks of 128.  64 experts, the Intra-GPU kernels / the whole call, us: 100000 tokens 14.2 with the scan, 11.3 without;
// 131072 tokens (the line) 20.1 / 59 and 15.9 / 55; past it, 163840 tokens 20.3 / 65.3 and 16.5 / 65.4, 262144 tokens 21.1 / 76.1 and 18.9 / 77.5,
// 524288 tokens 24.4 / 117 and 27.1 / 122: the adding up, of all blocks in every workgroup, takes what the launch would.  (The lower line is not
// where both sides are equal: 8192 tokens, just under it, 20.7 / 33.7 and in workgroups of 1024 13.7 / 26.8; 4096 tokens 16.9 / 27.7.)
constexpr int kIrSelfMax = 4096, kIrLargeBlock = 1024, kIrLargeSelfMax = 8192;

struct DispatchArgs {
  int T, E, k, C, NR, NCAT, NB, Eg, Tg, ir, fr, arrival, BM, max_mtiles;
  int Cq, Gq, NL;  // capacity blocks: Gq per expert (1, or one per group with per-group quotas) of Cq slots
  int NBc, cb;     // candidate counts come per count block: cb of them per token block, NBc in all
  int ir_self;     // small batches: ir_weights sums the Intra-GPU block counts itself (no scan launch)
  int direct;      // small batches, one capacity block per expert: select_direct_kernel finds its candidates itself
  int Ts;          // row length of the per-round arrays (key, rank8)
};

// lanes of this wave whose (valid, e) equals the caller's; e < 64
__device__ inline unsigned long long same_expert_mask(bool valid, int e) {
  unsigned long long mask = __ballot(valid);
#pragma unroll
  for (int b = 0; b < 6; ++b) {
    bool bit = (e >> b) & 1;
    unsigned long long bb = __ballot(valid && bit);
    mask &= bit ? bb : ~bb;
  }
  return mask;
}

__device__ inline int lanes_below(unsigned long long mask) {
  int lane = lane_id();
  return __popcll(mask & ((1ull << lane) - 1ull));
}

// Inclusive sum over the lanes of the wave (data-parallel moves).
__device__ inline int wave_scan(int v) {
  auto step = [&](auto ctrl, auto row_mask) {
    v += __builtin_amdgcn_update_dpp(0, v, decltype(ctrl)::value, decltype(row_mask)::value, 0xf, false);
  };
  using std::integral_constant;
  step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});  // row_shr 1, 2, 4, 8
  step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
  step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
  step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
  step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});  // row_bcast 15 into rows 1 and 3
  step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});  // row_bcast 31 into rows 2 and 3
  return v;
}

__device__ inline int wave_sum(int v) { return __builtin_amdgcn_readlane(wave_scan(v), 63); }

// ------------------------------------------------------------------ topk_rank
// One token block per workgroup, two lanes per token: lanes l and l + 32 of a wave each rank half of token l's experts
// and merge, as in the router's epilogue.  What bounds it is the instructions of a token's insertions, so half the
// experts per lane, lists no longer than k + 1 and four waves per SIMD instead of two.  100000 tokens, 64 experts, k = 2:
// topk_rank_kernel 19.1 -> 13.5 us.
constexpr int TK_THREADS = 2 * kTokBlock;
__global__ __launch_bounds__(TK_THREADS) void topk_rank_kernel(const float *__restrict__ logits, DispatchArgs A,
                                                               int32_t *__restrict__ rank_expert,
                                                               int32_t *__restrict__ slot, u32 *__restrict__ key,
                                                               uint8_t *__restrict__ rank8,
                                                               float *__restrict__ ir_score,
                                                               int32_t *__restrict__ ir_cand,
                                                               int32_t *__restrict__ blk_cnt) {
  __shared__ float tile[kTokBlock * TS];
  __shared__ int cnt[kMaxRounds * kMaxE];
  const int tid = threadIdx.x, b = blockIdx.x;
  const int t0 = b * kTokBlock;
  const int ntok = min(kTokBlock, A.T - t0);
  const int E = A.E;
  const float *src = logits + (size_t)t0 * E;  // 16-byte aligned: t0 is a multiple of 128
  const int nvec = (ntok * E) >> 2;
  // row of an element: idx / E = the high word of idx * ceil(2^32 / E), exact for idx < 2^13 and 2 <= E <= 64
  const u32 inv = 0xffffffffu / (u32)E + 1u;
  auto put = [&](int idx, float v) {
    const int row = E == 1 ? idx : (int)__umulhi((u32)idx, inv);
    tile[row * TS + idx - row * E] = v;
  };
  for (int v = tid; v < nvec; v += TK_THREADS) {
    const float4 q = reinterpret_cast<const float4 *>(src)[v];
    put(4 * v, q.x);
    put(4 * v + 1, q.y);
    put(4 * v + 2, q.z);
    put(4 * v + 3, q.w);
  }
  for (int idx = 4 * nvec + tid; idx < ntok * E; idx += TK_THREADS) put(idx, src[idx]);
  for (int c = tid; c < A.NCAT; c += TK_THREADS) cnt[c] = 0;
  __syncthreads();
  const int lane = tid & 63, half = lane >> 5, tok = (tid >> 6) * 32 + (lane & 31);
  if (tok < ntok) {  // (both lanes of a token are here)
    const int i = t0 + tok;
    const float *row = tile + tok * TS;
    const int n = min(A.k + 1, E), mid = (E + 1) >> 1;
    auto rank = [&](auto tag) {
      constexpr int N = decltype(tag)::value;  // list length: at least k + 1 and NR
      rank_t top[N], o[N];
      top_keys_of_range<N>(row, half ? mid : 0, half ? E : mid, top);
#pragma unroll
      for (int q = 0; q < N; ++q) o[q] = rank_of_lane(top[q], 32);  // the other half's list, fetched whole before this one changes
#pragma unroll
      for (int q = 0; q < N; ++q) insert_key(top, o[q]);
      if (half) return;
#pragma unroll
      for (int q = 0; q < N; ++q) {
        const int e = rank_key_expert(top[q]);  // -1 past the number of experts
        if (q <= A.k) rank_expert[(size_t)i * (A.k + 1) + q] = (q < n) ? e : -1;
        if (q < A.NR) {
          key[(size_t)q * A.Ts + i] = rank_key_score(top[q]);
          if (rank8) rank8[(size_t)q * A.Ts + i] = (uint8_t)e;
          atomicAdd(&cnt[q * E + e], 1);
        }
      }
      if (!A.fr) slot[(size_t)i * (A.k + 1) + A.k] = -1;
    };
    if (A.k == 1) rank(std::integral_constant<int, 2>{});
    else if (A.k == 2) rank(std::integral_constant<int, 3>{});
    else rank(std::integral_constant<int, kMaxRank>{});
    if (half) {
      const int g = i / A.Tg;
      float best;
      int arg;
      best_in_group(row, g * A.Eg, (g + 1) * A.Eg, best, arg);
      ir_score[i] = best;
      ir_cand[i] = arg;
    }
  }
  __syncthreads();
  for (int c = tid; c < A.NCAT; c += TK_THREADS) blk_cnt[(size_t)c * A.NBc + b] = cnt[c];  // here cb == 1
}

// ------------------------------------------------------------------ scan over token blocks
// One workgroup per list: exclusive scan of a[list][0..NB) in place, total to tot[list].  A thread
// scans SC_PER consecutive entries in registers, so 8192 entries are one trip with two barriers.
constexpr int SC_THREADS = 1024, SC_PER = 8, SC_WAVES = SC_THREADS / kWave;
// zero: nullptr, or an array of which every workgroup clears nzero entries from blockIdx.x * nzero on.
__global__ __launch_bounds__(SC_THREADS) void scan_blocks_kernel(int32_t *__restrict__ a, int32_t *__restrict__ tot,
                                                                 int NB, int32_t *__restrict__ zero, int nzero) {
  __shared__ int wsum[SC_WAVES];
  if (zero)
    for (int q = threadIdx.x; q < nzero; q += SC_THREADS) zero[(size_t)blockIdx.x * nzero + q] = 0;
  int32_t *p = a + (size_t)blockIdx.x * NB;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const bool vec = (NB & 3) == 0;  // then every list starts 16-byte aligned
  int running = 0;
  for (int base = 0; base < NB; base += SC_THREADS * SC_PER) {
    const int idx = base + tid * SC_PER;
    int v[SC_PER];
    if (vec && idx + SC_PER <= NB) {
      const int4 q0 = *reinterpret_cast<const int4 *>(p + idx), q1 = *reinterpret_cast<const int4 *>(p + idx + 4);
      v[0] = q0.x; v[1] = q0.y; v[2] = q0.z; v[3] = q0.w; v[4] = q1.x; v[5] = q1.y; v[6] = q1.z; v[7] = q1.w;
    } else {
#pragma unroll
      for (int u = 0; u < SC_PER; ++u) v[u] = idx + u < NB ? p[idx + u] : 0;
    }
    int sum = 0;
#pragma unroll
    for (int u = 0; u < SC_PER; ++u) {  // v[u] becomes the exclusive prefix inside the thread
      const int t = v[u];
      v[u] = sum;
      sum += t;
    }
    const int incl = wave_scan(sum);
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int q = 0; q < SC_WAVES; ++q) {
      int s = wsum[q];
      if (q < w) before += s;
      total += s;
    }
    const int off0 = running + before + incl - sum;
    if (vec && idx + SC_PER <= NB) {
      *reinterpret_cast<int4 *>(p + idx) = make_int4(off0 + v[0], off0 + v[1], off0 + v[2], off0 + v[3]);
      *reinterpret_cast<int4 *>(p + idx + 4) = make_int4(off0 + v[4], off0 + v[5], off0 + v[6], off0 + v[7]);
    } else {
#pragma unroll
      for (int u = 0; u < SC_PER; ++u)
        if (idx + u < NB) p[idx + u] = off0 + v[u];
    }
    running += total;
    __syncthreads();
  }
  if (tid == 0) tot[blockIdx.x] = running;
}

// ------------------------------------------------------------------ scatter_candidates
// Besides splitting the tokens into per-list arrays this kernel settles every list whose outcome
// follows from the candidate counts alone: nobody kept (the capacity block is full), everybody kept,
// or the first m in token order (arrival order).  A candidate's position in its list is known here,
// so its slot is too: the token's slot entry is written with the rest of its row (whole cache
// lines) and the candidate never enters the arrays.  Only the lists that are selected by score
// (Sec. 3: the lowest scores are dropped; Sec. 4.2: Fill-in takes the highest) are materialised for
// select_slot.
__global__ __launch_bounds__(kTokBlock) void scatter_candidates_kernel(DispatchArgs A,
                                                                       const int32_t *__restrict__ rank_expert,
                                                                       const u32 *__restrict__ key,
                                                                       const int32_t *__restrict__ blk_off,
                                                                       const int32_t *__restrict__ cat_cnt,
                                                                       u32 *__restrict__ cand_key,
                                                                       int32_t *__restrict__ cand_tok,
                                                                       int32_t *__restrict__ slot,
                                                                       int32_t *__restrict__ slot_token) {
  constexpr int NW = kTokBlock / kWave;
  __shared__ int wcnt[kMaxRounds][NW][kMaxE];
  __shared__ int s_base[kMaxRounds * kMaxE];
  // per list of this block's capacity block: first candidate (position in the candidate array), kept
  // count (-1: selected by score, the list goes to select_slot) and first slot
  __shared__ int s_lo[kMaxRounds * kMaxE], s_keep[kMaxRounds * kMaxE], s_fill0[kMaxRounds * kMaxE];
  const int tid = threadIdx.x, b = xcd_block(blockIdx.x, A.NB), w = tid >> 6, lane = tid & 63;
  const int i = b * kTokBlock + tid;
  const bool valid = i < A.T;
  for (int c = tid; c < kMaxRounds * NW * kMaxE; c += kTokBlock) (&wcnt[0][0][0])[c] = 0;
  // the token's experts are fetched in the same round trip as the array counts below (loads do not
  // move across barriers by themselves)
  int e_r[kMaxRounds], rank_r[kMaxRounds], off_r[kMaxRounds];
  u32 key_r[kMaxRounds];
#pragma unroll
  for (int r = 0; r < kMaxRounds; ++r) {
    e_r[r] = 0;
    if (valid && r < A.NR) e_r[r] = rank_expert[(size_t)i * (A.k + 1) + r];
  }
  // every token is a candidate of exactly one array per round: round r's arrays tile [r T, (r+1) T)
  // in expert order (a dozen counts: recomputed by every workgroup rather than by a launch of its own)
  for (int r = w; r < A.NR; r += NW) {
    const int c = lane < A.E ? cat_cnt[r * A.E + lane] : 0;
    const int incl = wave_scan(c);
    if (lane < A.E) s_base[r * A.E + lane] = r * A.T + incl - c;
  }
  // the plan of the lists that this block's tokens can be candidates of: capacity block g of every
  // (round, expert); kept = min(candidates, free slots) round after round, as in select_slot
  {
    const int bpg = A.NB / A.Gq * A.cb, g = b / (A.NB / A.Gq);
    for (int c = tid; c < A.NCAT; c += kTokBlock) {
      const int r = c / A.E, j = c - r * A.E;
      int n = 0, m = 0, fill = 0, lo = 0;
      for (int rr = 0; rr <= r; ++rr) {
        const int cc = rr * A.E + j;
        fill += m;
        lo = g == 0 ? 0 : blk_off[(size_t)cc * A.NBc + g * bpg];
        const int hi = g == A.Gq - 1 ? cat_cnt[cc] : blk_off[(size_t)cc * A.NBc + (g + 1) * bpg];
        n = hi - lo;
        m = min(n, A.Cq - fill);
      }
      const bool by_score = !A.arrival || r == A.k;
      s_lo[c] = lo;
      s_keep[c] = (m == n || m == 0 || !by_score) ? m : -1;
      s_fill0[c] = g * A.Cq + fill;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kMaxRounds; ++r) {
    rank_r[r] = 0;
    off_r[r] = 0;
    key_r[r] = 0;
    if (r < A.NR) {
      const int e = e_r[r];
      // in flight across the barrier, and only what the list's plan needs: nothing for a list that keeps
      // nobody, the position for a list that keeps by position, the key as well for a score-selected one
      const int keep = s_keep[r * A.E + e];
      if (valid && keep != 0) off_r[r] = blk_off[(size_t)(r * A.E + e) * A.NBc + b * A.cb];
      if (valid && keep < 0) key_r[r] = key[(size_t)r * A.Ts + i];
      unsigned long long mask = same_expert_mask(valid, e);
      int below = lanes_below(mask);
      if (valid && below == 0) wcnt[r][w][e] = __popcll(mask);
      rank_r[r] = below;
    }
  }
  __syncthreads();
  if (!valid) return;
#pragma unroll
  for (int r = 0; r < kMaxRounds; ++r) {
    if (r < A.NR) {
      int e = e_r[r], cat = r * A.E + e;
      int at = off_r[r] + rank_r[r];  // position in the (round, expert) array
      for (int q = 0; q < w; ++q) at += wcnt[r][q][e];
      const int keep = s_keep[cat], idx = at - s_lo[cat];
      int sl = -1;  // "dropped" until select_slot says otherwise (it only touches the entries of the tokens it keeps)
      if (keep < 0) {
        cand_key[s_base[cat] + at] = key_r[r];
        cand_tok[s_base[cat] + at] = i;
      } else if (keep > 0 && idx < keep) {  // (keep == 0: the position was not even fetched)
        sl = s_fill0[cat] + idx;
        slot_token[(size_t)e * A.C + sl] = i;
      }
      slot[(size_t)i * (A.k + 1) + r] = sl;
    }
  }
}

// ------------------------------------------------------------------ select_slot
constexpr int SS_THREADS = 1024;
constexpr int SS_WAVES = SS_THREADS / kWave;
constexpr int SS_PER = kSelectRegMax / SS_THREADS;  // keys a thread keeps in registers (24)
constexpr int kHistCopies = 32;  // counters per histogram bin (see radix_select)
constexpr int kHistWords = 256 * (1 + kHistCopies);

// Smallest value of the wave, in a scalar (data-parallel moves: no LDS round trips).
__device__ inline u32 wave_min(u32 v) {
  auto step = [&](auto ctrl, auto row_mask) {
    v = min(v, (u32)__builtin_amdgcn_update_dpp((int)0xffffffff, (int)v, decltype(ctrl)::value, decltype(row_mask)::value, 0xf, false));
  };
  using std::integral_constant;
  step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});  // row_shr 1, 2, 4, 8: lane 15 of a row has the row's
  step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
  step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
  step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
  step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});  // row_bcast 15 into rows 1 and 3
  step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});  // row_bcast 31 into rows 2 and 3
  return (u32)__builtin_amdgcn_readlane((int)v, 63);
}

// m-th largest key among those that `each` enumerates (Sec. 3: the lowest scores are dropped), by 8-bit digits
// from the highest bit in which the keys differ at all.  Returns the threshold key; need_eq = how many of the keys
// equal to it are kept (the first ones in token order).  `each(f)` calls f(key, valid) for every key slot of the
// calling thread, the same number of times in every lane of a wave (invalid slots with valid = false);
// all threads of the workgroup call this together.
// For lists streamed from memory, and what value_select leaves over.  A digit pass is four barriers and an LDS histogram, 1.6 us; a few thousand scores differ in 24 or 25 bits, and
// two digits below their common prefix as a rule leave a bin of which every key is kept: the threshold is then
// the key below the bin, and the passes end (3001 tokens, 6 experts: four fixed passes 6.5 us, now 4.2; all of
// select_slot_kernel at 4096 tokens with per-group capacity 21.0 -> 17.5).
// Most lanes of a wave can hit the same histogram bin (scores tied or close), and LDS atomics of one instruction on
// one address are served one lane after the other: every bin has kHistCopies counters, lane l adds to copy
// l % kHistCopies (consecutive words, different banks), and the copies are added up before the bins are scanned.
// IN_RANGE: of the keys in [lo, hi] only, from the highest bit in which lo and hi differ; the caller knows how many keys
// of the list lie above hi.  Otherwise the digits start at the highest bit: where `each` reads memory (lists past the registers)
// finding the extremes is a pass of its own and saves none as a rule: 400 K tokens, 8 experts, top-2, lists of up to 190 K
// candidates, select_slot_kernel 464 us without it, 504 with it.
template <bool IN_RANGE, class Each>
__device__ inline u32 radix_select(int m, Each each, u32 *hist, u32 *s_pick, u32 &need_eq, u32 lo = 0, u32 hi = 0xffffffffu) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  u32 *copies = hist + 256;  // [256][kHistCopies]
  u32 prefix = 0, remaining = (u32)m;
  int left = 32;  // bits below the prefix
  if constexpr (IN_RANGE) {
    const u32 diff = lo ^ hi;
    left = diff ? 32 - __clz((int)diff) : 0;
    prefix = left < 32 ? lo >> left << left : 0u;
  }
  while (left > 0) {
    const int bits = min(left, 8), shift = left - bits;
#pragma unroll
    for (int q = 0; q < 256 * kHistCopies / SS_THREADS; ++q) copies[q * SS_THREADS + tid] = 0;
    __syncthreads();
    each([&](u32 kx, bool valid) {
      const u32 digit = (kx ^ prefix) >> shift;  // (the prefix has zeros there: past 8 bits only in keys of another prefix)
      if (valid && digit >> bits == 0 && (!IN_RANGE || kx - lo <= hi - lo)) atomicAdd(&copies[digit * kHistCopies + (lane & (kHistCopies - 1))], 1u);
    });
    __syncthreads();
    {  // thread t adds up a quarter of the copies of bin t / 4
      static_assert(SS_THREADS == 4 * 256 && kHistCopies % 4 == 0, "four threads per bin");
      const u32 *c = copies + (tid >> 2) * kHistCopies + (tid & 3) * (kHistCopies / 4);
      u32 sum = 0;
#pragma unroll
      for (int q = 0; q < kHistCopies / 4; ++q) sum += c[q];
      sum += __shfl_xor(sum, 1);
      sum += __shfl_xor(sum, 2);
      if ((tid & 3) == 0) hist[tid >> 2] = sum;
    }
    __syncthreads();
    if (w == 0) {
      // lane l owns bins 255-4l .. 252-4l, i.e. bins in descending order across lanes
      u32 c0 = hist[255 - 4 * lane], c1 = hist[254 - 4 * lane], c2 = hist[253 - 4 * lane], c3 = hist[252 - 4 * lane];
      const u32 sum = c0 + c1 + c2 + c3, incl = (u32)wave_scan((int)sum), excl = incl - sum;
      if (excl < remaining && remaining <= incl) {
        u32 rem = remaining - excl, in_bin = c0;
        int bkt = 255 - 4 * lane;
        if (rem > c0) { rem -= c0; --bkt; in_bin = c1;
          if (rem > c1) { rem -= c1; --bkt; in_bin = c2;
            if (rem > c2) { rem -= c2; --bkt; in_bin = c3; } } }
        s_pick[0] = (u32)bkt;
        s_pick[1] = rem;
        s_pick[2] = in_bin;
      }
    }
    __syncthreads();  // the picks are next written three barriers from here: no barrier needed after reading them
    prefix |= s_pick[0] << shift;
    remaining = s_pick[1];
    left = shift;
    if (s_pick[2] == remaining && max(prefix, lo) > 0) {  // the whole bin is kept
      need_eq = 0;
      return max(prefix, lo) - 1;  // (keys below lo can share the bin's digits)
    }
  }
  need_eq = remaining;
  return prefix;
}

// The same as radix_select for keys held in registers, by one histogram of the scores themselves: kValueBins bins of equal width
// (score - lowest, scaled, rounded and clamped to the bins, never decreases with the key).  Scores spread
// over such bins, where the leading digits of their keys - sign and exponent - are a handful of values: the bin
// with the m-th highest holds a few keys as a rule, which every wave ranks for itself.  Five barriers, where
// three digit passes are thirteen.  3001 tokens, 6 experts: select_direct_kernel 11.8 -> 9.6 us.
//   * The bins span the list's scores, or - lists of more than kShortList keys, and shorter ones that half of whose waves have their first
//     key in one bin - three times the range between the waves' usual extremes (of the lowest keys of two waves the higher one, of
//     eight such the lowest, and the mirror image): a few scores that lie far from all others then share the bins at the ends.
//     (Bins as wide as their distance would hold all other keys in one, by LDS atomics on one address.  Waves of short lists hold runs of
//     neighbouring tokens, whose scores can be alike: their extremes say little.)
//   * Where half of the waves' first keys share a bin all the same, scores are spread in no such way and the digits select.
//   * More keys in the bin than a wave has lanes: one score, many times (done), or the digits go on among its keys.
//   * Lists of up to kTinyList keys need no bins: 1024 tokens, 64 experts, top-2, lists of 32: the kernel 10.7 -> 9.7 us.  (Every wave goes
//     over the keys one by one, 64 of them 2.7 us: 1024 tokens, 16 experts, top-4, lists of 64: 10.5 us, 12.4 without bins.)
// Us of the selecting kernel, digits alone / bins from the lowest to the highest score, then digits over again / now, for scores
// that are normal, with one of 1e4, with every hundredth times 1e6, multiples of 1/4: 3001 tokens, 6 experts 13.5 / 10.8 / 10.8, 13.3 /
// 13.5 / 10.9, 13.1 / 14.3 / 11.8, 14.7 / 15.3 / 12.0; 16384 tokens, 2 experts 22.5 / 19.9 / 20.1, 22.2 / 29.0 / 20.3, 22.2 / 29.2 / 21.9, 24.5 /
// 26.6 / 22.9; 32768 tokens 22.7 / 20.7 / 19.3, 23.0 / 35.8 / 21.0, 22.8 / 35.4 / 22.7, 25.4 / 27.8 / 21.9.
constexpr int kValueBins = 4 * SS_THREADS, kTinyList = 32, kShortList = 4096;
static_assert(kValueBins + 2 * kWave + 1 <= kHistWords, "bins, the bin's keys, wave results, their number");
static_assert(SS_WAVES == 16, "a row of 16 lanes for each of the waves' results");
template <class Each>
__device__ inline u32 value_select(int n, int m, Each each, u32 *hist, u32 *s_pick, u32 &need_eq) {
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  u32 *const few = hist + kValueBins, *const wres = few + kWave, *const n_few = wres + kWave;
  // v of another lane of the row of 16
  auto row_step = [](auto ctrl, u32 v) { return (u32)__builtin_amdgcn_mov_dpp((int)v, decltype(ctrl)::value, 0xf, 0xf, false); };
  using std::integral_constant;
  const integral_constant<int, 0xb1> quad1; const integral_constant<int, 0x4e> quad2;    // lane ^ 1, ^ 2
  const integral_constant<int, 0x124> ror4; const integral_constant<int, 0x128> ror8;
  auto wave_results = [&](u32 lo, u32 nhi, u32 probe) {  // (one LDS access per wave, whatever the number of waves)
    lo = wave_min(lo);
    nhi = wave_min(nhi);
    if (lane == 0) {
      wres[w] = lo;
      wres[SS_WAVES + w] = nhi;
      wres[2 * SS_WAVES + w] = probe;
    }
  };
  auto row_min = [&](u32 v) {
    v = min(v, row_step(quad1, v));
    v = min(v, row_step(quad2, v));
    v = min(v, row_step(ror4, v));
    return min(v, row_step(ror8, v));
  };
  auto lane_value = [](u32 v, int l) { return (u32)__builtin_amdgcn_readlane((int)v, l); };
  u32 lo = 0xffffffffu, nhi = 0xffffffffu;  // smallest key, smallest complement
  auto extremes = [&](u32 kx, bool valid) {
    if (valid) {
      lo = min(lo, kx);
      nhi = min(nhi, ~kx);
    }
  };
  // the m-th highest of `count` keys, at most a wave's lanes, that `is_in` tells: every wave ranks them for itself
  auto ranked = [&](int count, auto is_in) {
    each([&](u32 kx, bool valid) {
      if (valid && is_in(kx)) few[atomicAdd(n_few, 1u)] = kx;
    });
    __syncthreads();
    const u32 mine = lane < count ? few[lane] : 0u;  // (a key is never 0)
    int above = 0, equal = 0;
    for (int q = 0; q < count; ++q) {
      const u32 other = lane_value(mine, q);
      above += other > mine;
      equal += other == mine;
    }
    const unsigned long long at = __ballot(lane < count && above < m && m <= above + equal);
    const int src = __ffsll((long long)at) - 1;
    need_eq = (u32)(m - __builtin_amdgcn_readlane(above, src));
    return lane_value(mine, src);
  };
  if (tid == 0) *n_few = 0;
  if (n <= kTinyList) {  // (uniform over the workgroup)
    __syncthreads();
    return ranked(n, [](u32) { return true; });
  }
  each(extremes);
  const unsigned long long have = __ballot(lo != 0xffffffffu);
  wave_results(lo, nhi, have ? lane_value(lo, __ffsll((long long)have) - 1) : 0u);  // (a key is never 0)
  reinterpret_cast<uint4 *>(hist)[tid] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  const u32 wave_v = wres[lane];  // lanes 0 .. 15: lowest keys of the waves, 16 .. 31: complements of the highest, 32 .. 47: a key
  const u32 all = row_min(wave_v);
  lo = lane_value(all, 0);
  nhi = lane_value(all, SS_WAVES);
  u32 hi = ~nhi;
  if (lo == hi) {  // all scores are equal
    need_eq = (u32)m;
    return lo;
  }
  const float lowest = key_score(lo), highest = key_score(hi);
  float low, scale;
  auto bin_of = [&](u32 kx) { return (int)__builtin_amdgcn_fmed3f((key_score(kx) - low) * scale, 0.0f, (float)(kValueBins - 1)); };
  // bins between two scores; false: no ordinary range, or half of the waves' keys share a bin and the bin may be crowded (uniform over
  // the workgroup)
  auto bins_over = [&](float from, float to) {
    const float width = to - from;
    low = from;
    scale = (float)kValueBins * __builtin_amdgcn_rcpf(width);
    if (!(width < INFINITY) || !(scale < INFINITY)) return false;
    if (n <= kWave) return true;
    const bool probe = (lane & 48) == 2 * SS_WAVES && wave_v != 0;
    const int bin = probe ? bin_of(wave_v) : -1 - lane, probes = __popcll(__ballot(probe));
    auto sharers = [&](int q) { return __popcll(__ballot(bin == __builtin_amdgcn_readlane(bin, 2 * SS_WAVES + q))); };
    return max(sharers(0), sharers(2)) < max(3, (probes + 1) / 2);
  };
  bool spread = n <= kShortList && bins_over(lowest, highest);
  if (!spread && lowest <= highest) {  // (both are numbers)
    u32 ends = max(wave_v, row_step(quad1, wave_v));  // (a wave without keys: all ones, and so its pair)
    ends = min(ends, row_step(quad2, ends));
    ends = min(ends, row_step(ror4, ends));
    ends = min(ends, row_step(ror8, ends));
    const float usual_low = key_score(lane_value(ends, 0)), usual_high = key_score(~lane_value(ends, SS_WAVES));
    const float apart = usual_high - usual_low, margin = apart > 0.0f ? apart : INFINITY;  // (else the list's own extremes)
    spread = bins_over(fmaxf(lowest, usual_low - margin), fminf(highest, usual_high + margin));
  }
  if (spread) {
    each([&](u32 kx, bool valid) {
      if (valid) atomicAdd(&hist[bin_of(kx)], 1u);
    });
    __syncthreads();
    // thread t owns four bins, t = 0 the highest
    const uint4 c = reinterpret_cast<const uint4 *>(hist)[SS_THREADS - 1 - tid];
    const int sum = (int)(c.x + c.y + c.z + c.w), incl = wave_scan(sum);
    if (lane == 63) wres[w] = (u32)incl;  // (the extremes were read before the last barrier)
    __syncthreads();
    const int waves = wave_scan(lane < SS_WAVES ? (int)wres[lane] : 0);
    const int excl = incl - sum + (w ? (int)lane_value((u32)waves, w - 1) : 0);
    if (excl < m && m <= excl + sum) {
      u32 rem = (u32)(m - excl), in_bin = c.w;
      int bin = 4 * (SS_THREADS - 1 - tid) + 3;
      if (rem > in_bin) { rem -= in_bin; --bin; in_bin = c.z;
        if (rem > in_bin) { rem -= in_bin; --bin; in_bin = c.y;
          if (rem > in_bin) { rem -= in_bin; --bin; in_bin = c.x; } } }
      s_pick[0] = (u32)bin;
      s_pick[1] = rem;
      s_pick[2] = in_bin;
    }
    __syncthreads();
    const int bin = (int)s_pick[0], in_bin = (int)s_pick[2];
    m = (int)s_pick[1];  // of the bin's keys
    if (in_bin <= kWave) return ranked(in_bin, [&](u32 kx) { return bin_of(kx) == bin; });
    lo = nhi = 0xffffffffu;  // the bin's extremes
    each([&](u32 kx, bool valid) { extremes(kx, valid && bin_of(kx) == bin); });
    wave_results(lo, nhi, 0);  // (the sums were read before the last barrier)
    __syncthreads();
    const u32 ext = row_min(wres[lane]);
    lo = lane_value(ext, 0);
    hi = ~lane_value(ext, SS_WAVES);
    if (lo == hi) {
      need_eq = (u32)m;
      return lo;
    }
  }
  __syncthreads();
  return radix_select<true>(m, each, hist, s_pick, need_eq, lo, hi);
}

// Shared memory of the selection kernels.
struct __attribute__((aligned(16))) SelectSmem {
  u32 hist[kHistWords];
  u32 pick[3];
  int wtot[SS_PER][SS_WAVES];  // counts per (trip, wave): kept for sure, and equal to the threshold << 16
  int wsum[8];
};

// Selection and slotting of a list of n <= SS_THREADS * NU candidates held in registers: candidate
// idx = u * SS_THREADS + tid is element u of thread tid (`load(idx, key, tok)` fetches it), so the
// candidates are met in token order.  The m < n highest keys are kept, equal keys in token order.  Kept candidates take slots
// fill0, fill0 + 1, ... in token order: one scan over the (trip, wave) totals of the kept flags.
// Only kept candidates are written (every slot entry starts as -1).
template <int NU, class Load>
__device__ inline void select_trips(const DispatchArgs &A, int n, int m, int r, int j, int fill0, Load load, SelectSmem &S,
                                    int32_t *__restrict__ slot, int32_t *__restrict__ slot_token) {
  static_assert(SS_THREADS * NU < 1 << 16, "two counts in a word");
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const unsigned long long below = (1ull << lane) - 1ull;
  const int nu = (n + SS_THREADS - 1) / SS_THREADS;
  u32 kreg[NU];
  int treg[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int idx = u * SS_THREADS + tid;
    kreg[u] = 0;
    treg[u] = 0;
    if (u < nu && idx < n) load(idx, kreg[u], treg[u]);
  }
  u32 need_eq = 0;
  const u32 thr = value_select(n, m, [&](auto f) {
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (u < nu) f(kreg[u], u * SS_THREADS + tid < n);
  }, S.hist, S.pick, need_eq);

  int pre[NU];  // lanes of this wave before this one: kept-for-sure | equal << 8
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    pre[u] = 0;
    if (u < nu) {
      const bool valid = u * SS_THREADS + tid < n;
      const bool gt = valid && kreg[u] > thr, eq = valid && kreg[u] == thr;
      const unsigned long long bgt = __ballot(gt), beq = __ballot(eq);
      pre[u] = __popcll(bgt & below) | (__popcll(beq & below) << 8) | (gt ? 1 << 16 : 0) | (eq ? 1 << 17 : 0);
      if (lane == 0) S.wtot[u][w] = __popcll(bgt) | __popcll(beq) << 16;
    }
  }
  __syncthreads();
  // exclusive scan of the nu * SS_WAVES totals in (trip, wave) order = token order
  constexpr int kScanWaves = (NU * SS_WAVES + kWave - 1) / kWave;
  static_assert(kScanWaves <= 8, "wsum");
  const int ne = nu * SS_WAVES;
  int mine = 0, incl = 0;
  if (tid < kScanWaves * kWave) {
    if (tid < ne) mine = (&S.wtot[0][0])[tid];
    incl = wave_scan(mine);
    if (kScanWaves > 1 && lane == 63) S.wsum[w] = incl;
  }
  if constexpr (kScanWaves > 1) __syncthreads();
  if (tid < ne) {
    int before = 0;
    if constexpr (kScanWaves > 1)
      for (int q = 0; q < w; ++q) before += S.wsum[q];
    (&S.wtot[0][0])[tid] = before + incl - mine;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    if (u < nu && u * SS_THREADS + tid < n) {
      const int base = S.wtot[u][w];
      const bool gt = (pre[u] >> 16) & 1, eq = (pre[u] >> 17) & 1;
      const int eqs = (int)((u32)base >> 16) + ((pre[u] >> 8) & 255);  // equal keys before this one
      if (gt || (eq && (u32)eqs < need_eq)) {
        const int sl = fill0 + (base & 0xffff) + (pre[u] & 255) + min(eqs, (int)need_eq);
        slot[(size_t)treg[u] * (A.k + 1) + r] = sl;
        slot_token[(size_t)j * A.C + sl] = treg[u];
      }
    }
  }
}
// (lists of up to 4096 candidates without the other twenty trips' tests)
template <class Load>
__device__ inline void select_in_registers(const DispatchArgs &A, int n, int m, int r, int j, int fill0, Load load, SelectSmem &S,
                                           int32_t *__restrict__ slot, int32_t *__restrict__ slot_token) {
  if (n <= 4 * SS_THREADS) select_trips<4>(A, n, m, r, j, fill0, load, S, slot, slot_token);
  else select_trips<SS_PER>(A, n, m, r, j, fill0, load, S, slot, slot_token);
}

// The same for a list of any length, streamed from memory by one workgroup: the threshold by digit
// passes over the keys, then a pass that hands out the slots.  The path for lists that fit neither the registers nor the
// split scheme below; exact for any input.  Bound by the latency of its loads and barriers, so 8192 candidates are in
// flight at a time: 326862 tokens, 8 experts Zipf(1.5), top-4: select_slot_kernel
// 381 -> 150 us (1024 at a time with two barriers each before).
__device__ inline void select_streaming(const DispatchArgs &A, int n, int m, int r, int j, int fill0,
                                        const u32 *__restrict__ keys, const int32_t *__restrict__ toks, SelectSmem &S,
                                        int32_t *__restrict__ slot, int32_t *__restrict__ slot_token) {
  constexpr int NU = 8;
  static_assert(NU * SS_WAVES == 2 * kWave, "two totals per lane");
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned long long below = (1ull << lane) - 1ull;
  u32 need_eq = 0;
  const u32 thr = radix_select<false>(m, [&](auto f) {
    for (int base = tid; base - tid < n; base += NU * SS_THREADS) {
      u32 kx[NU];
#pragma unroll
      for (int u = 0; u < NU; ++u) kx[u] = base + u * SS_THREADS < n ? keys[base + u * SS_THREADS] : 0u;
#pragma unroll
      for (int u = 0; u < NU; ++u) f(kx[u], base + u * SS_THREADS < n);
    }
  }, S.hist, S.pick, need_eq);
  int run_gt = 0, run_eq = 0;
  for (int base = tid; base - tid < n; base += NU * SS_THREADS) {
    u32 kreg[NU];
    int treg[NU], pre[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int idx = base + u * SS_THREADS;
      kreg[u] = idx < n ? keys[idx] : 0u;
      treg[u] = idx < n ? toks[idx] : 0;
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const bool valid = base + u * SS_THREADS < n, gt = valid && kreg[u] > thr, eq = valid && kreg[u] == thr;
      const unsigned long long bgt = __ballot(gt), beq = __ballot(eq);
      pre[u] = __popcll(bgt & below) | (__popcll(beq & below) << 8) | (gt ? 1 << 16 : 0) | (eq ? 1 << 17 : 0);
      if (lane == 0) S.wtot[u][w] = __popcll(bgt) | __popcll(beq) << 16;
    }
    __syncthreads();
    // every wave scans the totals in (trip, wave) order = token order, two per lane
    const int t0 = (&S.wtot[0][0])[2 * lane], t1 = (&S.wtot[0][0])[2 * lane + 1], incl = wave_scan(t0 + t1), excl = incl - t0 - t1;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int e = u * SS_WAVES + w;  // uniform
      const int before = __builtin_amdgcn_readlane(e & 1 ? excl + t0 : excl, e >> 1);
      const bool gt = (pre[u] >> 16) & 1, eq = (pre[u] >> 17) & 1;
      const int eqs = run_eq + (int)((u32)before >> 16) + ((pre[u] >> 8) & 255);  // equal keys before this one
      if (gt || (eq && (u32)eqs < need_eq)) {
        const int sl = fill0 + run_gt + (before & 0xffff) + (pre[u] & 255) + min(eqs, (int)need_eq);
        slot[(size_t)treg[u] * (A.k + 1) + r] = sl;
        slot_token[(size_t)j * A.C + sl] = treg[u];
      }
    }
    const int total = __builtin_amdgcn_readlane(incl, 63);
    run_gt += total & 0xffff;
    run_eq += (int)((u32)total >> 16);
    __syncthreads();
  }
}

// A selection list is the piece of a (round, expert) candidate array that competes for one capacity
// block: the whole array and the expert's whole queue by default; with per-group quotas (Sec. 3's
// capacity read per GPU) the candidates of group g - a contiguous piece, since candidates are in
// ascending token index and groups are token ranges that end on block boundaries - and the group's
// Cq slots.  The kept count of a round is min(candidates, free slots of the block), so every round
// (Fill-in, the (k+1)-th, included) is planned from the candidate counts alone; each workgroup derives
// its own list's numbers from them, and the workgroup of an expert's last round and first block also
// writes the expert's fill counts.
//
// Lists of up to SS_THREADS * SS_PER candidates are one workgroup's work (select_in_registers).  A
// longer list - a skewed router sends most tokens to a few experts - is cut into segments of
// kSegLen candidates, one workgroup each (the first workgroups of the grid are the segments after a
// list's first; each derives its (list, segment) from the candidate counts):
//   * nobody, everybody or the first m in token order kept: scatter_candidates has handed out the
//     slots already, the list's workgroups leave at once;
//   * the m highest scores kept: every segment workgroup takes the same sample of the list's keys
//     (runs of 64 consecutive candidates, spread evenly) and selects in it a key L that, with a
//     margin of several standard deviations, lies below the list's m-th highest key; it then copies its segment's candidates with key >= L,
//     in order, to a second pair of arrays and counts them.  The workgroup that finishes last
//     (a ticket from an atomic counter - nobody waits for anybody) adds up the counts: if they
//     number at least m and fit the registers, the kept set is among them and it finishes the
//     list with select_in_registers; otherwise (the sample misled, or the scores are tied en
//     masse) it streams the original list.  The result is exact either way.
constexpr int kRegMax = kSelectRegMax;           // candidates that fit the registers of one workgroup
constexpr int kMapLists = kSelectMapLists;       // lists up to which long lists are split (the map is kept in LDS)

// Exclusive scan of one value per thread over the workgroup (two barriers); total = sum over all threads.
__device__ inline int block_scan_exclusive(int v, int *s_wave, int &total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int incl = wave_scan(v);
  if (lane == 63) s_wave[w] = incl;
  __syncthreads();
  int before = 0;
  total = 0;
#pragma unroll
  for (int q = 0; q < SS_WAVES; ++q) {
    const int t = s_wave[q];
    if (q < w) before += t;
    total += t;
  }
  __syncthreads();
  return before + incl - v;
}

// kSegLen: 16384, or 4096 where that makes at most 256 further segments (kSelectShortMax candidates in all); the sample is as long.
// 100000 tokens, 64 experts Zipf(1.1), top-2 (longest list 73 K): 35.5 -> 29.4 us, with the histogram of scores and trips for 4096
// candidates 19.1.  (Lists that fit the registers are not cut, though with independent scores the few kept of 18 K would be found 3 us
// sooner - 32768 tokens, 32 experts Zipf(1.1), 512 kept of each: 18.3, not 21.5; digits alone 24.9 -: 10 K lists are 2.5 us
// slower cut, and where ties or the order of the tokens defeat the sample 24 K ones 31, not 20.)
template <int kSegLen>
__global__ __launch_bounds__(SS_THREADS) void select_slot_kernel(DispatchArgs A, const int32_t *__restrict__ cat_cnt,
                                                                 const int32_t *__restrict__ blk_off,
                                                                 const u32 *__restrict__ cand_key,
                                                                 const int32_t *__restrict__ cand_tok,
                                                                 u32 *__restrict__ comp_key,
                                                                 int32_t *__restrict__ comp_tok,
                                                                 int32_t *__restrict__ seg_cnt,
                                                                 int32_t *__restrict__ seg_more,
                                                                 int32_t *__restrict__ list_done,
                                                                 int32_t *__restrict__ slot,
                                                                 int32_t *__restrict__ slot_token,
                                                                 int32_t *__restrict__ grp_fill,
                                                                 int32_t *__restrict__ grp_off,
                                                                 int32_t *__restrict__ fill_topk,
                                                                 int32_t *__restrict__ fill_total) {
  constexpr int kSegPer = kSegLen / SS_THREADS;  // candidates per thread of a segment workgroup
  constexpr int kSampleLen = kSegLen;            // keys in the sample
  // candidates of the longest list: tokens of a batch, or what the launch takes for short segments
  constexpr int kMaxList = kSegLen == kSelectShortLen ? kSelectShortMax : kMaxTokens;
  static_assert(kMaxList / kSegLen + 1 <= kMapLists + 1, "the offsets of a list's segments take the map's place");
  __shared__ SelectSmem S;
  __shared__ int s_extra[kMapLists + 1];  // exclusive scan over the lists of their segments after the first
  __shared__ int s_wave[SS_WAVES];
  __shared__ int s_bcast;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int bpg = A.NB / A.Gq * A.cb;  // count blocks per group (exact with quotas; all of them otherwise)
  // candidates [lo, hi) of (round rr, expert jj) that belong to group gg
  auto piece = [&](int rr, int jj, int gg, int &lo, int &hi) {
    const int c = rr * A.E + jj;
    lo = gg == 0 ? 0 : blk_off[(size_t)c * A.NBc + gg * bpg];
    hi = gg == A.Gq - 1 ? cat_cnt[c] : blk_off[(size_t)c * A.NBc + (gg + 1) * bpg];
  };

  // ---- which (list, segment) is this workgroup.  The workgroups of the further segments come first
  // in the grid (those that turn out to have no segment leave at once): a split list is finished
  // by the last of its segments, so they should not queue behind the one-workgroup lists.
  const bool can_split = select_splits(A.T, A.NR, A.NL);  // otherwise the grid has one workgroup per list
  const int n_extra = (int)gridDim.x - A.NL;
  int lst = (int)blockIdx.x - n_extra, seg = 0, extra_base = 0;
  if (can_split) {
    int carry = 0;
    for (int l0 = 0; l0 < A.NL; l0 += SS_THREADS) {
      const int l = l0 + tid;
      int ex = 0;
      if (l < A.NL) {
        const int c = l / A.Gq, gg = l - c * A.Gq, rr = c / A.E;
        int lo, hi;
        piece(rr, c - rr * A.E, gg, lo, hi);
        ex = hi - lo > kRegMax ? (hi - lo + kSegLen - 1) / kSegLen - 1 : 0;
      }
      int total;
      const int excl = block_scan_exclusive(ex, s_wave, total);
      if (l < A.NL) s_extra[l] = carry + excl;
      carry += total;
    }
    if (tid == 0) s_extra[A.NL] = carry;
    __syncthreads();
    if ((int)blockIdx.x < n_extra) {
      const int x = blockIdx.x;
      if (x >= s_extra[A.NL]) return;  // no such segment
      int a = 0, b = A.NL - 1;  // the last list whose scan value is <= x (lists without extra segments repeat their successor's value)
      while (a < b) {
        const int mid = (a + b + 1) >> 1;
        if (s_extra[mid] <= x) a = mid; else b = mid - 1;
      }
      lst = a;
      seg = x - s_extra[lst] + 1;
    }
    extra_base = s_extra[lst];
  }

  // ---- the list: (round r, expert j, capacity block g); n candidates, m of them kept, in slots fill0 ..
  const int cat = lst / A.Gq, g = lst - cat * A.Gq, r = cat / A.E, j = cat - r * A.E;
  int n = 0, m = 0, fill = 0, lo = 0;
  const int before_j = lane < A.E ? cat_cnt[r * A.E + lane] : 0;  // (every load of the plan in one round trip)
  int lo_r[kMaxRounds], hi_r[kMaxRounds];
#pragma unroll
  for (int rr = 0; rr < kMaxRounds; ++rr) {
    lo_r[rr] = hi_r[rr] = 0;
    if (rr <= r) piece(rr, j, g, lo_r[rr], hi_r[rr]);
  }
#pragma unroll
  for (int rr = 0; rr < kMaxRounds; ++rr)
    if (rr <= r) {
      fill += m;
      lo = lo_r[rr];
      n = hi_r[rr] - lo;
      m = min(n, A.Cq - fill);
    }
  const int fill0 = g * A.Cq + fill;
  // round r's arrays tile [r T, (r+1) T) in expert order
  const int base = r * A.T + lo + __builtin_amdgcn_readlane(wave_scan(before_j) - before_j, j);
  const u32 *keys = cand_key + base;
  const int32_t *toks = cand_tok + base;
  if (seg == 0) {
    if (r == A.NR - 1 && g == 0 && w == 0) {
      // lane gg: occupied slots of block gg after the top-k rounds and after every round
      int topk = 0, total = 0;
      if (lane < A.Gq) {
        for (int rr = 0; rr < A.NR; ++rr) {
          int l, h;
          piece(rr, j, lane, l, h);
          total += min(h - l, A.Cq - total);
          if (rr == A.k - 1) topk = total;
        }
      }
      const int incl = wave_scan(total), sum_topk = wave_sum(topk);
      if (lane < A.Gq) {
        grp_fill[j * A.Gq + lane] = total;
        grp_off[j * A.Gq + lane] = incl - total;
      }
      if (lane == 63) fill_total[j] = incl;
      if (lane == 0) fill_topk[j] = sum_topk;
    }
    // the last round pads the rest of the capacity block (Sec. 3: zero padding)
    if (r == A.NR - 1)
      for (int sl = fill0 + m + tid; sl < (g + 1) * A.Cq; sl += SS_THREADS) slot_token[(size_t)j * A.C + sl] = -1;
  }
  if (m == 0) return;  // nobody kept: every slot entry already says so
  const bool by_score = !A.arrival || r == A.k;  // the Fill-in round always selects by score (Sec. 4.2)
  if (m == n || !by_score) return;  // everybody, or the first m in token order: settled by scatter_candidates
  if (n <= kRegMax) {
    select_in_registers(A, n, m, r, j, fill0, [&](int idx, u32 &kx, int &tok) { kx = keys[idx]; tok = toks[idx]; }, S, slot,
                        slot_token);
    return;
  }

  // ---- long list (if can_split it has a workgroup per segment), the m highest scores: sample, copy the candidates that may be
  // kept, last one finishes
  const int nseg = (n + kSegLen - 1) / kSegLen;
  // rank in the sample: the expected number of sampled keys among the list's m highest, plus five
  // standard deviations and a few; the candidates with key >= L then number about n / kSampleLen times that
  const float expect = (float)m * (float)kSampleLen / (float)n;
  const int qsel = (int)(expect + 5.0f * sqrtf(expect) + 16.0f);
  const bool split = can_split && qsel < kSampleLen && (long long)qsel * n / kSampleLen <= kRegMax * 7 / 8;
  if (!split) {
    if (seg == 0) select_streaming(A, n, m, r, j, fill0, keys, toks, S, slot, slot_token);
    return;
  }
  u32 L;
  {
    // the sample: kSampleLen / 64 runs of 64 consecutive candidates, spread evenly over the list (a wave
    // instruction then reads one run - two cache lines - where single candidates a stride apart would
    // touch 64 lines: 19 -> 5 us for a list of 900 K candidates)
    static_assert(kSegPer * SS_WAVES * kWave == kSampleLen, "one run per (trip, wave)");
    const int run = n / (kSampleLen / kWave);  // > 64: n > kRegMax >= 1.5 kSampleLen
    u32 sk[kSegPer];
#pragma unroll
    for (int u = 0; u < kSegPer; ++u) sk[u] = keys[(size_t)(u * SS_WAVES + w) * run + lane];
    u32 dummy;
    L = value_select(kSampleLen, qsel, [&](auto f) {
#pragma unroll
      for (int u = 0; u < kSegPer; ++u) f(sk[u], true);
    }, S.hist, S.pick, dummy);
  }
  {
    const unsigned long long below = (1ull << lane) - 1ull;
    const int i0 = seg * kSegLen, len = min(n - i0, kSegLen);
    u32 kreg[kSegPer];
    int pre[kSegPer];
#pragma unroll
    for (int u = 0; u < kSegPer; ++u) {
      const int idx = u * SS_THREADS + tid;
      kreg[u] = idx < len ? keys[i0 + idx] : 0u;
      const bool ge = idx < len && kreg[u] >= L;
      const unsigned long long bge = __ballot(ge);
      pre[u] = __popcll(bge & below) | (ge ? 1 << 16 : 0);
      if (lane == 0) S.wtot[u][w] = __popcll(bge);
    }
    __syncthreads();
    // exclusive scan of the kSegPer * SS_WAVES wave totals in (trip, wave) order = token order
    int mine = 0, incl = 0;
    if (tid < kSegPer * SS_WAVES) mine = (&S.wtot[0][0])[tid];
    if (tid < 4 * kWave) {  // kSegPer * SS_WAVES is at most 256 entries = 4 waves
      incl = wave_scan(mine);
      if (lane == 63) S.wsum[w] = incl;
    }
    __syncthreads();
    int count = 0;
    if (tid < kSegPer * SS_WAVES) {
      int before = 0;
      for (int q = 0; q < w; ++q) before += S.wsum[q];
      (&S.wtot[0][0])[tid] = before + incl - mine;
    }
    count = S.wsum[0] + S.wsum[1] + S.wsum[2] + S.wsum[3];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSegPer; ++u) {
      if ((pre[u] >> 16) & 1) {
        const int idx = u * SS_THREADS + tid, pos = base + i0 + S.wtot[u][w] + (pre[u] & 255);
        comp_key[pos] = kreg[u];
        comp_tok[pos] = toks[i0 + idx];
      }
    }
    // publish: count, then the ticket.  Every wave waits until its own copies have been written (a
    // store counts as done when the L2 has it), the barrier collects the waves, and ONE device-scope
    // fence (a write-back of the L2, which the other XCDs do not see into) goes before the ticket.
    // Whoever draws the last ticket fences once more before it reads the other segments' copies.
    int32_t *const my_cnt = seg == 0 ? seg_cnt + lst : seg_more + extra_base + seg - 1;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
      *my_cnt = count;
      __threadfence();
      s_bcast = atomicAdd(&list_done[lst], 1);
      if (s_bcast == nseg - 1) __threadfence();
    }
    __syncthreads();
    if (s_bcast != nseg - 1) return;
  }
  // ---- the last workgroup of the list: segments' counts -> offsets of their copies (s_extra is free now)
  __syncthreads();
  int total = 0;
  {
    int carry = 0;
    for (int q0 = 0; q0 < nseg; q0 += SS_THREADS) {  // (nseg fits s_extra)
      const int q = q0 + tid;
      const int c = q < nseg ? (q == 0 ? seg_cnt[lst] : seg_more[extra_base + q - 1]) : 0;
      int tot;
      const int excl = block_scan_exclusive(c, s_wave, tot);
      if (q < nseg) s_extra[q] = carry + excl;
      carry += tot;
    }
    total = carry;
    __syncthreads();
  }
  if (total < m || total > kRegMax) {
    select_streaming(A, n, m, r, j, fill0, keys, toks, S, slot, slot_token);
    return;
  }
  const int *s_off = s_extra;  // first copy of every segment
  select_in_registers(A, total, m, r, j, fill0, [&](int idx, u32 &kx, int &tok) {
    int a = 0, b = nseg - 1;  // segment whose copies hold position idx
    while (a < b) {
      const int mid = (a + b + 1) >> 1;
      if (s_off[mid] <= idx) a = mid; else b = mid - 1;
    }
    const int pos = base + a * kSegLen + (idx - s_off[a]);
    kx = comp_key[pos];
    tok = comp_tok[pos];
  }, S, slot, slot_token);
}

// ------------------------------------------------------------------ select_slot, small batches
// Up to kDirectMaxT tokens and one capacity block per expert: the workgroup of list (round r, expert j) finds
// its candidates itself - it reads the ranked experts of rounds 0 .. r of every token (one byte each) and the
// keys of round r - and counts expert j's candidates of the earlier rounds on the way (the kept count of a
// round is min(candidates, free slots)).  No candidate counts, no scan, no scatter: three launches fewer.
// A thread owns `per` neighbouring tokens (4, 8, 12 or 16), so thread order is token order: one scan over the threads
// hands out the slots.  What bounds it is what one CU reads for a list, then a chain of nine barriers around the LDS
// histogram: with the [T, k + 1] table of 32-bit ranks and the keys of all rounds side by side it read 24 bytes per token at k = 2,
// now 4 + (r + 1).  16384 tokens, 8 experts, top-2: reading 10.1 -> 5.6 us, kernel 29.1 -> 22.2, with the histogram of scores 18.0; 4000
// tokens, 16 experts: 18.9 -> 13.4 -> 11.2; 3001, 6 experts: 13.5 -> 10.8.
constexpr int kDirectPer = kDirectMaxT / SS_THREADS;
static_assert(kDirectPer == 16, "a thread's tokens are quadruples, at most four");

__global__ __launch_bounds__(SS_THREADS) void select_direct_kernel(DispatchArgs A,
                                                                   const uint8_t *__restrict__ rank8,
                                                                   const u32 *__restrict__ key,
                                                                   int32_t *__restrict__ slot,
                                                                   int32_t *__restrict__ slot_token,
                                                                   int32_t *__restrict__ grp_fill,
                                                                   int32_t *__restrict__ grp_off,
                                                                   int32_t *__restrict__ fill_topk,
                                                                   int32_t *__restrict__ fill_total) {
  __shared__ __attribute__((aligned(16))) u32 hist[kHistWords];
  __shared__ u32 s_pick[3];
  __shared__ u32 s_wave[SS_WAVES];
  __shared__ int s_cnt[kMaxRounds];
  const int r = blockIdx.x / A.E, j = blockIdx.x - r * A.E;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int per = ((A.T + SS_THREADS - 1) / SS_THREADS + 3) / 4 * 4;
  const int tok0 = tid * per;
  if (tid < kMaxRounds) s_cnt[tid] = 0;
  __syncthreads();
  // All loads first.  Quadruples of tokens past the batch read its last one (rows of Ts elements, a multiple of 16).
  uint4 kq[4];
  u32 eq8[kMaxRounds][4];
  const int last = (A.T - 1) & ~3;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (4 * q < per) kq[q] = *reinterpret_cast<const uint4 *>(key + (size_t)r * A.Ts + min(tok0 + 4 * q, last));
#pragma unroll
  for (int rr = 0; rr < kMaxRounds; ++rr)
    if (rr <= r)  // r is uniform over the workgroup
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (4 * q < per) eq8[rr][q] = *reinterpret_cast<const u32 *>(rank8 + (size_t)rr * A.Ts + min(tok0 + 4 * q, last));
  u32 kreg[kDirectPer];
  u32 member = 0;  // bit u: token tok0 + u is a candidate of this list
  u32 c01 = 0, c23 = 0, c4 = 0;  // candidates of expert j in rounds 0 .. r, 16 bits each
#pragma unroll
  for (int u = 0; u < kDirectPer; ++u) {
    kreg[u] = 0;
    if (u < per) {
      const uint4 kv = kq[u / 4];
      kreg[u] = u % 4 == 0 ? kv.x : (u % 4 == 1 ? kv.y : (u % 4 == 2 ? kv.z : kv.w));
      const bool in = tok0 + u < A.T;
#pragma unroll
      for (int rr = 0; rr < kMaxRounds; ++rr)
        if (rr <= r) {
          const bool hit = in && ((eq8[rr][u / 4] >> (u % 4 * 8)) & 255u) == (u32)j;
          const u32 one = hit ? (rr & 1 ? 1u << 16 : 1u) : 0u;
          if (rr < 2) c01 += one;
          else if (rr < 4) c23 += one;
          else c4 += one;
          if (rr == r && hit) member |= 1u << u;
        }
    }
  }
  c01 = (u32)wave_sum((int)c01);
  if (r >= 2) c23 = (u32)wave_sum((int)c23);
  if (r >= 4) c4 = (u32)wave_sum((int)c4);
  if (lane <= r) {  // lane rr adds the wave's count of round rr
    const u32 both = lane < 2 ? c01 : (lane < 4 ? c23 : c4);
    const int v = lane & 1 ? both >> 16 : both & 0xffffu;
    if (v) atomicAdd(&s_cnt[lane], v);
  }
  __syncthreads();
  int n = 0, m = 0, fill = 0, topk = 0;
  for (int rr = 0; rr <= r; ++rr) {
    fill += m;
    n = s_cnt[rr];
    m = min(n, A.Cq - fill);
    if (rr == A.k - 1) topk = fill + m;
  }
  const int fill0 = fill;
  if (r == A.NR - 1 && tid == 0) {  // the expert's last round also writes its fill counts
    grp_fill[j] = fill + m;
    grp_off[j] = 0;
    fill_total[j] = fill + m;
    fill_topk[j] = topk;
  }
  const bool by_score = !A.arrival || r == A.k;  // the Fill-in round always selects by score (Sec. 4.2)
  // mode 0: nobody kept; 1: everybody kept; 2: the first m in token order; 3: by score threshold
  const int mode = m == 0 ? 0 : (m == n ? 1 : (by_score ? 3 : 2));
  u32 thr = 0, need_eq = 0;
  if (mode == 3)
    thr = value_select(n, m, [&](auto f) {
#pragma unroll
      for (int u = 0; u < kDirectPer; ++u)
        if (u < per) f(kreg[u], (member >> u) & 1u);
    }, hist, s_pick, need_eq);
  if (mode == 2) need_eq = (u32)m;  // arrival order: every candidate "ties", the first m of them are kept

  u32 gt = 0, eq = 0;  // this thread's candidates kept for sure, equal to the threshold
  if (mode == 1) gt = member;
  if (mode == 2) eq = member;
  if (mode == 3)
#pragma unroll
    for (int u = 0; u < kDirectPer; ++u) {
      if (kreg[u] > thr) gt |= 1u << u;
      if (kreg[u] == thr) eq |= 1u << u;
    }
  gt &= member;
  eq &= member;
  // exclusive scan over the threads of both counts, 16 bits each (at most kDirectMaxT candidates)
  const u32 mine = (u32)__popc(gt) | (u32)__popc(eq) << 16;
  const u32 incl = (u32)wave_scan((int)mine);
  if (lane == 63) s_wave[w] = incl;
  __syncthreads();
  u32 before = incl - mine;
#pragma unroll
  for (int q = 0; q < SS_WAVES; ++q) before += q < w ? s_wave[q] : 0u;
#pragma unroll
  for (int u = 0; u < kDirectPer; ++u) {
    if ((member >> u) & 1u) {
      const u32 low = (1u << u) - 1u;
      const int tok = tok0 + u;
      const int gts = (int)(before & 0xffffu) + __popc(gt & low), eqs = (int)(before >> 16) + __popc(eq & low);
      const bool kept = ((gt >> u) & 1u) || (((eq >> u) & 1u) && (u32)eqs < need_eq);
      const int sl = fill0 + gts + min(eqs, (int)need_eq);
      slot[(size_t)tok * (A.k + 1) + r] = kept ? sl : -1;
      if (kept) slot_token[(size_t)j * A.C + sl] = tok;
    }
  }
  // the last round pads the rest of the queue (Sec. 3: zero padding)
  if (r == A.NR - 1)
    for (int sl = fill0 + m + tid; sl < A.Cq; sl += SS_THREADS) slot_token[(size_t)j * A.C + sl] = -1;
}

// ------------------------------------------------------------------ Intra-GPU lists
__device__ inline int drops_of_token(const int32_t *slot, int i, int k) {
  int n = 0;
  for (int r = 0; r < k; ++r) n += slot[(size_t)i * (k + 1) + r] < 0;
  return n;
}

// TB tokens per workgroup and count block: kTokBlock, or kIrLargeBlock where ir_weights can then add up the counts of every
// block itself but not those of the small blocks (ir_large).
template <int TB>
__global__ __launch_bounds__(TB) void ir_count_kernel(DispatchArgs A, const int32_t *__restrict__ slot,
                                                             const int32_t *__restrict__ ir_cand,
                                                             int32_t *__restrict__ ir_blk_cnt) {
  __shared__ int cnt[kMaxE];
  // neighbouring blocks write neighbouring words of the per-expert count rows: XCD-aware block order
  const int tid = threadIdx.x, b = xcd_block(blockIdx.x, gridDim.x);
  const int i = b * TB + tid;
  if (tid < kMaxE) cnt[tid] = 0;
  __syncthreads();
  if (i < A.T && drops_of_token(slot, i, A.k) > 0) atomicAdd(&cnt[ir_cand[i]], 1);
  __syncthreads();
  // (ir_weights adds them up itself: block by block; else expert by expert, for the scan)
  if (tid < A.E) ir_blk_cnt[A.ir_self ? (size_t)b * A.E + tid : (size_t)tid * gridDim.x + b] = cnt[tid];
}

// Dispatched-row layout: expert e owns rows [row_base[e], row_base[e+1]): its occupied capacity
// slots first, then its Intra-GPU rows.  One wave, lane e = expert e: the offsets of the experts'
// Intra-GPU lists go to s_off (LDS, every workgroup of ir_weights needs them); the wave that `writes`
// also stores them with row_base and cuts every expert's rows into tiles of BM rows (skipped when
// max_mtiles == 0: routing-only calls have no grouped GEMM).
// fill, nir: occupied slots and Intra-GPU rows of the lane's expert (0 past the last one).
__device__ inline void row_plan_wave(const DispatchArgs &A, bool writes, int fill, int nir, int *s_off, int *s_rbase,
                                     int32_t *__restrict__ ir_offset,
                                     int32_t *__restrict__ row_base, TileInfo *__restrict__ tiles,
                                     int32_t *__restrict__ tile_ctl) {
  const int e = threadIdx.x & 63;
  const bool on = e < A.E;
  const int rows = fill + nir;
  const int ntile = A.max_mtiles > 0 ? (rows + A.BM - 1) / A.BM : 0;
  const int s_ir = wave_scan(nir), s_rows = wave_scan(rows), s_tiles = wave_scan(ntile);  // inclusive, over experts
  if (on) {
    s_off[e] = s_ir - nir;
    s_rbase[e] = s_rows - rows;
  }
  if (!writes) return;
  if (on) {
    ir_offset[e] = s_ir - nir;
    row_base[e] = s_rows - rows;
    int t = s_tiles - ntile;
    for (int m0 = 0; m0 < rows && ntile > 0 && t < A.max_mtiles; m0 += A.BM, ++t)
      tiles[t] = TileInfo{e, m0, s_rows - rows, rows, fill, s_ir - nir, 0, 0};
  }
  if (e == A.E - 1) {
    ir_offset[A.E] = s_ir;
    row_base[A.E] = s_rows;
    tile_ctl[0] = min(s_tiles, A.max_mtiles);
  }
}

// Per-group quotas only: the occupied slots of an expert are not a prefix of its queue, so the
// token behind every dispatched row is written out once (rows skip the holes between blocks).
__global__ __launch_bounds__(256) void row_token_kernel(DispatchArgs A, const int32_t *__restrict__ slot_token,
                                                        const int32_t *__restrict__ grp_fill,
                                                        const int32_t *__restrict__ grp_off,
                                                        const int32_t *__restrict__ fill_total,
                                                        const int32_t *__restrict__ ir_offset,
                                                        const int32_t *__restrict__ ir_token,
                                                        const int32_t *__restrict__ row_base,
                                                        int32_t *__restrict__ row_token) {
  const int e = blockIdx.x, base = row_base[e];
  for (int s = threadIdx.x; s < A.C; s += 256) {
    const int g = s / A.Cq, p = s - g * A.Cq;
    if (p < grp_fill[e * A.Gq + g]) row_token[base + grp_off[e * A.Gq + g] + p] = slot_token[(size_t)e * A.C + s];
  }
  const int nir = ir_offset[e + 1] - ir_offset[e], first = base + fill_total[e];
  for (int t = threadIdx.x; t < nir; t += 256) row_token[first + t] = ir_token[ir_offset[e] + t];
}

// Every dispatched row belongs to one (token, assignment): the token marks each of its rows - with its own
// index if this is the token's only row (Eq. 2 / Eq. 3 then give it weight exactly 1 and the expert's
// output row IS the layer's output row: the down projection stores it there), else with -1.
// row_of_slot(e, slot): the dispatched row of a slot; ir_row: that of the token's Intra-GPU row.
template <class RowOfSlot>
__device__ inline void mark_rows(int i, int NR, const int (&slot_r)[kMaxRank], const int (&e_r)[kMaxRank], bool has_ir,
                                 int ir_row, RowOfSlot row_of_slot, int32_t *__restrict__ row_dest) {
  int nrows = has_ir ? 1 : 0;
#pragma unroll
  for (int r = 0; r < kMaxRank; ++r) nrows += (r < NR && slot_r[r] >= 0) ? 1 : 0;
  const int mark = nrows == 1 ? i : -1;
#pragma unroll
  for (int r = 0; r < kMaxRank; ++r)
    if (r < NR && slot_r[r] >= 0) row_dest[row_of_slot(e_r[r], slot_r[r])] = mark;
  if (has_ir) row_dest[ir_row] = mark;
}

// Eq. 2 / Eq. 3: softmax over the successfully routed experts, a placed Fill-in expert, and the
// Intra-GPU expert counted (k - |R_i|) times
__device__ inline void write_weights(int i, int k, int NR, const int (&slot_r)[kMaxRank], const u32 (&key_r)[kMaxRank],
                                     bool has_ir, int ndrop, float score_h, float *__restrict__ combine_w) {
  const float a_h = has_ir ? score_h : 0.0f;
  float a_r[kMaxRank];
  bool kept[kMaxRank];
  float mx = has_ir ? a_h : -INFINITY;
#pragma unroll
  for (int r = 0; r < kMaxRank; ++r) {
    kept[r] = false;
    a_r[r] = 0.0f;
    if (r < NR) {
      kept[r] = slot_r[r] >= 0;
      if (kept[r]) {
        a_r[r] = key_score(key_r[r]);
        mx = fmaxf(mx, a_r[r]);
      }
    }
  }
  float term[kMaxRank], t_ir = has_ir ? (float)ndrop * expf(a_h - mx) : 0.0f, Z = t_ir;
#pragma unroll
  for (int r = 0; r < kMaxRank; ++r) {
    term[r] = kept[r] ? expf(a_r[r] - mx) : 0.0f;
    Z += term[r];
  }
  const float inv = Z > 0.0f ? 1.0f / Z : 0.0f;
  float *cw = combine_w + (size_t)i * (k + 2);
#pragma unroll
  for (int r = 0; r < kMaxRank; ++r)
    if (r <= k) cw[r] = term[r] * inv;
  cw[k + 1] = t_ir * inv;
}

// Per token: Intra-GPU list position (Sec. 4.1) and the Eq. 2 / Eq. 3 weights.
template <int TB>
__global__ __launch_bounds__(TB) void ir_weights_kernel(DispatchArgs A, const int32_t *__restrict__ slot,
                                                               const u32 *__restrict__ key,
                                                               const float *__restrict__ ir_score,
                                                               const int32_t *__restrict__ ir_cand,
                                                               const int32_t *__restrict__ ir_blk_off,
                                                               const int32_t *__restrict__ ir_cnt,
                                                               const int32_t *__restrict__ fill_total,
                                                               int32_t *__restrict__ ir_offset,
                                                               int32_t *__restrict__ row_base,
                                                               TileInfo *__restrict__ tiles,
                                                               int32_t *__restrict__ tile_ctl,
                                                               int32_t *__restrict__ ir_expert,
                                                               int32_t *__restrict__ ir_row,
                                                               int32_t *__restrict__ ir_token,
                                                               float *__restrict__ combine_w,
                                                               const int32_t *__restrict__ rank_expert,
                                                               const int32_t *__restrict__ grp_off,
                                                               int32_t *__restrict__ row_dest) {
  constexpr int NW = TB / kWave;
  const int NB = gridDim.x;
  __shared__ int wcnt[NW][kMaxE];
  __shared__ int s_off[kMaxE], s_rbase[kMaxE];
  const int tid = threadIdx.x, b = xcd_block(blockIdx.x, NB), w = tid >> 6, lane = tid & 63;
  const int i = b * TB + tid;
  const bool valid = i < A.T;
  for (int c = tid; c < NW * kMaxE; c += TB) (&wcnt[0][0])[c] = 0;
  __shared__ int s_cnt[kMaxE], s_before[kMaxE];
  const bool self = A.ir_self && A.ir;
  __shared__ int s_fill[kMaxE];
  if (self && tid < kMaxE) s_cnt[tid] = s_before[tid] = 0;
  // everything this token needs from global memory is fetched here, in one round trip, ahead of the
  // barriers (loads do not move across them)
  int slot_r[kMaxRank], cand = 0, ndrop = 0;
  u32 key_r[kMaxRank];
  float score_h = 0.0f;
#pragma unroll
  for (int r = 0; r < kMaxRank; ++r) {
    slot_r[r] = -1;
    key_r[r] = 0;
    if (valid && r < A.NR) {
      slot_r[r] = slot[(size_t)i * (A.k + 1) + r];
      key_r[r] = key[(size_t)r * A.Ts + i];
    }
  }
  if (valid && A.ir) {
    cand = ir_cand[i];
    score_h = ir_score[i];
  }
  const int fill_e = lane < A.E ? fill_total[lane] : 0, nir_e = !self && A.ir && lane < A.E ? ir_cnt[lane] : 0;
  if (w == 0) s_fill[lane] = fill_e;
  int e_r[kMaxRank];  // only for row_dest: the experts behind the token's slots
#pragma unroll
  for (int r = 0; r < kMaxRank; ++r) {
    e_r[r] = 0;
    if (row_dest && valid && r < A.NR) e_r[r] = rank_expert[(size_t)i * (A.k + 1) + r];
  }
#pragma unroll
  for (int r = 0; r < kMaxRank; ++r)
    if (r < A.k) ndrop += slot_r[r] < 0;
  const bool has_ir = valid && A.ir && ndrop > 0;
  const int h = has_ir ? cand : 0;
  unsigned long long mask = same_expert_mask(has_ir, h);
  const int below = lanes_below(mask);
  __syncthreads();
  if (has_ir && below == 0) wcnt[w][h] = __popcll(mask);
  // ir_self: ir_blk_off holds the raw counts, block by block, and every workgroup adds up what it needs - the tokens of each
  // expert's list in earlier blocks and in all blocks - instead of a scan launch of its own in front of this kernel.  A
  // lane takes one expert of every so many blocks.  (One count per thread and turn, an integer division and
  // two LDS atomics each, and the experts' fill counts fetched behind the barrier: the kernel at 3001 tokens, 6 experts 6.0 us, now
  // 5.4; 2048 tokens, 8 experts 6.7, 5.5.)
  if (self) {
    const int shift = A.E > 1 ? 32 - __clz(A.E - 1) : 0, per = kWave >> shift;  // blocks that a wave reads at a time
    const int e = lane & ((1 << shift) - 1);
    int total = 0, before = 0;
#pragma unroll 4
    for (int bb = w * per + (lane >> shift); bb < NB; bb += NW * per) {
      const int v = e < A.E ? ir_blk_off[bb * A.E + e] : 0;
      total += v;
      before += bb < b ? v : 0;
    }
    for (int off = 1 << shift; off < kWave; off <<= 1) {
      total += __shfl_xor(total, off);
      before += __shfl_xor(before, off);
    }
    if (lane < A.E) {
      atomicAdd(&s_cnt[lane], total);
      atomicAdd(&s_before[lane], before);
    }
    __syncthreads();
  }
  // the row plan is a few dozen numbers: every workgroup recomputes the list offsets it needs, the
  // first one also writes the plan out for the kernels that follow
  if (w == 0)
    row_plan_wave(A, blockIdx.x == 0, fill_e, self ? (lane < A.E ? s_cnt[lane] : 0) : nir_e, s_off, s_rbase, ir_offset, row_base, tiles,
                  tile_ctl);
  __syncthreads();
  if (!valid) return;
  int my_ir_row = -1;
  if (has_ir) {
    int row = (A.ir_self ? s_before[h] : ir_blk_off[(size_t)h * NB + b]) + below;
    for (int q = 0; q < w; ++q) row += wcnt[q][h];
    ir_expert[i] = h;
    ir_row[i] = row;
    ir_token[s_off[h] + row] = i;
    my_ir_row = row;
  } else {
    ir_expert[i] = -1;
    ir_row[i] = -1;
  }
  if (row_dest)
    mark_rows(i, A.NR, slot_r, e_r, has_ir, has_ir ? s_rbase[h] + s_fill[h] + my_ir_row : 0,
              [&](int e, int s) {
                if (A.Gq == 1) return s_rbase[e] + s;
                const int g = s / A.Cq;
                return s_rbase[e] + grp_off[e * A.Gq + g] + (s - g * A.Cq);
              },
              row_dest);
  write_weights(i, A.k, A.NR, slot_r, key_r, has_ir, ndrop, score_h, combine_w);
}

// ------------------------------------------------------------------ small batches: all tables in one workgroup
// Up to kOneT tokens (one_is_cheaper) one workgroup of 1024 threads builds every table: a batch of
// a few hundred tokens is three or four dependent launches of 4 - 14 us otherwise, most of it latency.  Thread
// tid owns tokens u * 1024 + tid, so (u, wave) is token order.  Steps, a barrier between any two:
//   ranking (SRC: by the router already; or from logits; or from partial scores, which are summed here)
//   candidate counts per (round, expert, 64 tokens) by ballot matching; exclusive scans over the 64-token rows
//   stable split of the candidates into per-list arrays in LDS
//   one wave per list: kept count from the counts; threshold of the kept set by 4-ary search on the keys (as many
//     rounds as it takes to separate m of n keys; no histogram, no barrier); slots by ballots
//   Intra-GPU lists by the same matching and scan, row plan, weights
enum { ROUTE_RANKED = 0, ROUTE_LOGITS = 1, ROUTE_PARTS = 2 };
constexpr int OR_THREADS = 1024, OR_WAVES = OR_THREADS / kWave;
constexpr int kOneT = OR_THREADS, kOneSlots = 32768, kOneTile = 16384;  // kOneTile: T * E with the ranking done here
constexpr int kMaxParts = 16;            // parts of the router's K
constexpr int kMaxPartFloats = 65536;    // partial scores in all

// Who is kept: a wave per list searches for a threshold; or, for up to 128 tokens and more lists than two per wave, a thread per
// candidate counts the keys of its list that beat its own.  Us for the call, search / counting: 16 tokens, 96 lists
// 28.3 / 25.2; 64, 64 lists 37.4 / 35.0; 128, 64 lists 37.1 / 35.3; but 88 tokens, 12 lists 26.3 / 26.9 and 256, 16 lists (of up
// to 100 candidates) 27.0 / 29.8: one list per wave is searched in the time that the longest list takes to be counted.
__host__ __device__ inline bool counts_candidates(int T, int NL) { return T <= 128 && NL > 2 * OR_WAVES; }

struct OneLayout {  // dynamic LDS: the score tile, later the candidate arrays; slots; counts
  int tops, ctok, slot, wcnt, wir, plan, plan_topk, clist, kept, total;
};
__host__ __device__ inline OneLayout one_layout(int T, int E, int NR, int Gq, bool tile) {
  const int rows = (T + kWave - 1) / kWave, n = NR * T;
  // the tile, and behind it the ranked lists of tokens that several lanes rank
  const int cand = n * 4 + (n * 2 + 3) / 4 * 4, tops = (T * (E + 1) * 4 + 7) / 8 * 8;
  const int tile_bytes = tile ? tops + (T <= 512 ? T * kMaxRank * 8 : 0) : 0;
  OneLayout L;
  L.tops = tops;
  L.ctok = n * 4;
  L.slot = cand > tile_bytes ? cand : tile_bytes;
  L.wcnt = L.slot + (n * 2 + 3) / 4 * 4;
  L.wir = L.wcnt + (NR * rows * E * 2 + 3) / 4 * 4;
  L.plan = L.wir + (rows * E * 2 + 3) / 4 * 4;
  L.plan_topk = L.plan + NR * E * Gq * 4;
  L.clist = L.plan_topk + (Gq > 1 ? E * Gq * 4 : 0);
  const bool count = counts_candidates(T, NR * E * Gq);
  L.kept = L.clist + (count ? (n * 2 + 3) / 4 * 4 : 0);
  L.total = L.kept + (count ? (n + 31) / 32 * 4 : 0);
  return L;
}

// Lanes that rank a token together (a power of two; at least eight experts each).
__host__ __device__ inline int rank_lanes(int T, int E) {
  const int threads = T <= 128 ? 8 : (T <= 256 ? 4 : (T <= 512 ? 2 : 1)), share = E >> 3 < threads ? E >> 3 : threads;
  return share >= 8 ? 8 : (share >= 4 ? 4 : (share >= 2 ? 2 : 1));
}

template <int SRC>
__global__ __launch_bounds__(OR_THREADS) void route_small_kernel(
    DispatchArgs A, const float *__restrict__ part, int kparts, const float *__restrict__ bias, float *__restrict__ logits,
    int32_t *__restrict__ rank_expert, const u32 *__restrict__ key, const float *__restrict__ ir_score,
    const int32_t *__restrict__ ir_cand, int32_t *__restrict__ slot, int32_t *__restrict__ slot_token,
    int32_t *__restrict__ grp_fill, int32_t *__restrict__ grp_off, int32_t *__restrict__ fill_topk,
    int32_t *__restrict__ fill_total, int32_t *__restrict__ ir_offset, int32_t *__restrict__ row_base,
    TileInfo *__restrict__ tiles, int32_t *__restrict__ tile_ctl, int32_t *__restrict__ ir_expert,
    int32_t *__restrict__ ir_row, int32_t *__restrict__ ir_token, float *__restrict__ combine_w,
    int32_t *__restrict__ row_dest) {
  constexpr u32 NOSLOT = 0xffffu;  // handed-out slots lie below kMaxRounds * kOneT, counted from the first of the capacity block
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ int s_cnt[kMaxRounds * kMaxE], s_base[kMaxRounds * kMaxE];
  __shared__ int s_fill[kMaxE], s_ircnt[kMaxE], s_off[kMaxE], s_rbase[kMaxE];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int i = tid, row = w;  // this thread's token, its row of 64 tokens
  const unsigned long long below_mask = (1ull << lane) - 1ull;
  const int T = A.T, E = A.E, NR = A.NR, rows = (T + kWave - 1) / kWave;
  const OneLayout L = one_layout(T, E, NR, A.Gq, SRC != ROUTE_RANKED);
  float *const tile = reinterpret_cast<float *>(lds);
  rank_t *const tops = reinterpret_cast<rank_t *>(lds + L.tops);
  u32 *const ckey = reinterpret_cast<u32 *>(lds);                  // [NR][T] keys, lists of a round in expert order
  uint16_t *const ctok = reinterpret_cast<uint16_t *>(lds + L.ctok);  // [NR][T] tokens of the same
  uint16_t *const s_slot = reinterpret_cast<uint16_t *>(lds + L.slot);  // [NR][T] slot of the token, relative (see below)
  uint16_t *const wcnt = reinterpret_cast<uint16_t *>(lds + L.wcnt);  // [NR][rows][E] candidates, scanned over rows
  uint16_t *const wir = reinterpret_cast<uint16_t *>(lds + L.wir);    // [rows][E] the same for the Intra-GPU lists
  u32 *const plan = reinterpret_cast<u32 *>(lds + L.plan);            // [NL] kept count << 16 | slots of earlier rounds
  const bool count = counts_candidates(T, A.NL);
  uint16_t *const clist = reinterpret_cast<uint16_t *>(lds + L.clist);  // [NR][T] (count) list of the candidate
  u32 *const kept_bits = reinterpret_cast<u32 *>(lds + L.kept);         // (count) a bit per candidate
  u32 *const plan_topk = reinterpret_cast<u32 *>(lds + L.plan_topk);  // [E][Gq] (quotas) occupied after all rounds << 16 | after the top-k ones

  // ---- everything from global memory first: one round trip
  int e_r[kMaxRank], cand_h = 0;
  u32 key_r[kMaxRank];
  float score_h = 0.0f;
#pragma unroll
  for (int r = 0; r < kMaxRank; ++r) {
    e_r[r] = 0;
    key_r[r] = 0;
    if (SRC == ROUTE_RANKED && i < T && r < NR) {
      e_r[r] = rank_expert[(size_t)i * (A.k + 1) + r];
      key_r[r] = key[(size_t)r * A.Ts + i];
    }
  }
  if (SRC == ROUTE_RANKED && i < T && A.ir) {
    score_h = ir_score[i];
    cand_h = ir_cand[i];
  }
  for (int c = tid; c < (L.plan - L.wcnt) / 4; c += OR_THREADS) reinterpret_cast<u32 *>(lds + L.wcnt)[c] = 0;
  if constexpr (SRC != ROUTE_RANKED) {
    // (all loads of an element, or of several, in flight together: one CU's latency is what this kernel consists of)
    if constexpr (SRC == ROUTE_PARTS) {
      // The partial sums in order, then the bias; `elements` scores at a time, of up to `parts` parts each, about 32
      // loads in flight.  (One score at a time: 5.2 us of an 18 us kernel at 300 tokens x 16 experts; kernel 20.3 ->
      // 18.9 between events, 256 x 8 one part 15.8 -> 15.1 and the layer 28.5 -> 27.6.)
      auto sum_parts = [&](auto parts, auto elements) {
        constexpr int PN = decltype(parts)::value, EN = decltype(elements)::value;
        for (int i0 = tid; i0 < T * E; i0 += EN * OR_THREADS) {
          float p[EN][PN], b[EN];
#pragma unroll
          for (int u = 0; u < EN; ++u) {
            const int idx = min(i0 + u * OR_THREADS, T * E - 1);
            b[u] = bias ? bias[idx % E] : 0.0f;
#pragma unroll
            for (int q = 0; q < PN; ++q) p[u][q] = part[(size_t)(q < kparts ? q : 0) * T * E + idx];
          }
#pragma unroll
          for (int u = 0; u < EN; ++u) {
            const int idx = i0 + u * OR_THREADS, row = idx / E, e = idx - row * E;
            float v = p[u][0];
#pragma unroll
            for (int q = 1; q < PN; ++q) v += q < kparts ? p[u][q] : 0.0f;
            v += b[u];
            if (idx < T * E) {
              logits[idx] = v;
              tile[row * (E + 1) + e] = v;
            }
          }
        }
      };
      using std::integral_constant;
      if (kparts == 1) sum_parts(integral_constant<int, 1>{}, integral_constant<int, 8>{});
      else if (kparts <= 8) sum_parts(integral_constant<int, 8>{}, integral_constant<int, 4>{});
      else sum_parts(integral_constant<int, kMaxParts>{}, integral_constant<int, 2>{});
    } else {
      constexpr int AHEAD = 8;
      for (int i0 = tid; i0 < T * E; i0 += AHEAD * OR_THREADS) {
        float v[AHEAD];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) v[q] = logits[min(i0 + q * OR_THREADS, T * E - 1)];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) {
          const int idx = i0 + q * OR_THREADS, row = idx / E, e = idx - row * E;
          if (idx < T * E) tile[row * (E + 1) + e] = v[q];
        }
      }
    }
    __syncthreads();
    // Ranking.  With fewer tokens than threads several lanes share a token: each ranks a part of its row (at
    // least eight experts), the lists are merged by shuffles and handed to the token's thread through LDS.
    const int lpt = rank_lanes(T, E), per = (E + lpt - 1) / lpt;
    auto rank = [&](auto tag) {
      constexpr int N = decltype(tag)::value;  // list length: at least k + 1 and NR
      const int n = min(A.k + 1, E);
      rank_t top[N];
      auto rank_part = [&](const float *row, int e0, int e1) {
#pragma unroll
        for (int q = 0; q < N; ++q) top[q] = 0.0;
        for (int eb = e0; eb < e1; eb += 8) {
          float v[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] = row[min(eb + q, E - 1)];
#pragma unroll
          for (int q = 0; q < 8; ++q)
            if (eb + q < e1) insert_key(top, rank_key(v[q], eb + q));
        }
      };
      if (lpt > 1) {
        const int tok = tid / lpt, sub = tid & (lpt - 1);
        if (tok < T) {  // (T * lpt is a multiple of lpt: the lanes of a token are all here)
          rank_part(tile + tok * (E + 1), sub * per, min(E, (sub + 1) * per));
          for (int off = 1; off < lpt; off <<= 1) {
            rank_t o[N];
#pragma unroll
            for (int q = 0; q < N; ++q) o[q] = rank_of_lane(top[q], off);  // the other list, fetched whole before this one changes
#pragma unroll
            for (int q = 0; q < N; ++q) insert_key(top, o[q]);
          }
          if (sub == 0)
#pragma unroll
            for (int q = 0; q < N; ++q) tops[q * T + tok] = top[q];
        }
        __syncthreads();
        if (i < T)
#pragma unroll
          for (int q = 0; q < N; ++q) top[q] = tops[q * T + i];
      } else if (i < T) {
        rank_part(tile + i * (E + 1), 0, E);
      }
      if (i < T) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
          const int e = rank_key_expert(top[q]);  // -1 past the number of experts
          if (q <= A.k) rank_expert[(size_t)i * (A.k + 1) + q] = q < n ? e : -1;
          if (q < NR) {
            e_r[q] = e;
            key_r[q] = rank_key_score(top[q]);
          }
        }
        const int g = i / A.Tg;
        best_in_group(tile + i * (E + 1), g * A.Eg, (g + 1) * A.Eg, score_h, cand_h);
      }
    };
    if (A.k == 1) rank(std::integral_constant<int, 2>{});
    else if (A.k == 2) rank(std::integral_constant<int, 3>{});
    else rank(std::integral_constant<int, kMaxRank>{});
  }
  __syncthreads();  // counts are zero, the tile has been read
  // ---- candidates per (round, 64 tokens, expert)
  int below[kMaxRank];
#pragma unroll
  for (int r = 0; r < kMaxRank; ++r) {
    below[r] = 0;
    if (r < NR && row < rows) {
      const unsigned long long mask = same_expert_mask(i < T, e_r[r]);
      below[r] = __popcll(mask & below_mask);
      if (i < T && below[r] == 0) wcnt[(r * rows + row) * E + e_r[r]] = (uint16_t)__popcll(mask);
      if (i < T) s_slot[r * T + i] = (uint16_t)NOSLOT;
    }
  }
  __syncthreads();
  for (int c = tid; c < A.NCAT; c += OR_THREADS) {
    const int r = c / E, e = c - r * E;
    uint16_t *p = wcnt + r * rows * E + e;
    int sum = 0;
    for (int q = 0; q < rows; ++q) {
      const int v = p[q * E];
      p[q * E] = (uint16_t)sum;
      sum += v;
    }
    s_cnt[c] = sum;
  }
  __syncthreads();
  // first candidate of every list of round w, by wave w; meanwhile the last waves plan the rounds (kept =
  // min(candidates, free slots) round after round): one thread per (expert, capacity block)
  const int rpg = rows / A.Gq;  // 64-token rows per capacity block (quotas: groups end on 128 tokens)
  auto piece = [&](int rr, int j, int g, int &lo, int &hi) {
    lo = g == 0 ? 0 : wcnt[(rr * rows + g * rpg) * E + j];
    hi = g == A.Gq - 1 ? s_cnt[rr * E + j] : wcnt[(rr * rows + (g + 1) * rpg) * E + j];
  };
  if (w < NR) {
    const int c = lane < E ? s_cnt[w * E + lane] : 0;
    const int incl = wave_scan(c);
    if (lane < E) s_base[w * E + lane] = w * T + incl - c;
  } else {
    for (int c = OR_THREADS - 1 - tid; c < E * A.Gq; c += OR_THREADS - NR * kWave) {
      const int j = c / A.Gq, g = c - j * A.Gq;
      int fill = 0, topk = 0;
#pragma unroll
      for (int r = 0; r < kMaxRounds; ++r)
        if (r < NR) {
          int lo, hi;
          piece(r, j, g, lo, hi);
          const int m = min(hi - lo, A.Cq - fill);
          plan[(r * E + j) * A.Gq + g] = (u32)m << 16 | (u32)fill;
          fill += m;
          if (r == A.k - 1) topk = fill;
        }
      grp_fill[c] = fill;
      if (A.Gq == 1) {
        grp_off[j] = 0;
        s_fill[j] = fill;
        fill_total[j] = fill;
        fill_topk[j] = topk;
      } else {
        plan_topk[c] = (u32)fill << 16 | (u32)topk;
      }
    }
  }
  __syncthreads();
  if (A.Gq > 1) {  // quotas: one wave per expert adds up its blocks
    for (int j = w; j < E; j += OR_WAVES) {
      const u32 v = lane < A.Gq ? plan_topk[j * A.Gq + lane] : 0u;
      const int total = v >> 16;
      const int incl = wave_scan(total), sum_topk = wave_sum(v & 0xffffu);
      if (lane < A.Gq) grp_off[j * A.Gq + lane] = incl - total;
      if (lane == 63) {
        fill_total[j] = incl;
        s_fill[j] = incl;
      }
      if (lane == 0) fill_topk[j] = sum_topk;
    }
  }
  if (i < T) {
#pragma unroll
    for (int r = 0; r < kMaxRank; ++r)
      if (r < NR) {
        const int at = s_base[r * E + e_r[r]] + wcnt[(r * rows + row) * E + e_r[r]] + below[r];
        ckey[at] = key_r[r];
        ctok[at] = (uint16_t)i;
        if (count) clist[at] = (uint16_t)((r * E + e_r[r]) * A.Gq + (A.Gq == 1 ? 0 : i / A.Tg));
      }
  }
  if (count && tid < (NR * T + 31) / 32) kept_bits[tid] = 0;
  __syncthreads();
  // ---- the lists.  A slot is kept in LDS as its offset from the first slot of the list's capacity block.
  for (int c = tid; c < E * A.C; c += OR_THREADS) {  // zero padding (Sec. 3)
    const int j = c / A.C, sl = c - j * A.C, g = A.Gq == 1 ? 0 : sl / A.Cq;
    const u32 last = plan[((NR - 1) * E + j) * A.Gq + g];
    if (sl - g * A.Cq >= (int)((last >> 16) + (last & 0xffffu))) slot_token[c] = -1;
  }
  if (count) {
    // candidate at position `at`: its list's first position, length, plan
    struct Cand { int start, n, m, fill, r, j, g; };
    auto cand_of = [&](int at) {
      const int lst = clist[at], cat = A.Gq == 1 ? lst : lst / A.Gq, g = lst - cat * A.Gq;
      int r = 0;
#pragma unroll
      for (int q = 1; q < kMaxRounds; ++q) r += at >= q * T;
      int lo, hi;
      piece(r, cat - r * E, g, lo, hi);
      return Cand{s_base[cat] + lo, hi - lo, (int)(plan[lst] >> 16), (int)(plan[lst] & 0xffffu), r, cat - r * E, g};
    };
    for (int at = tid; at < NR * T; at += OR_THREADS) {
      const Cand c = cand_of(at);
      const int pos = at - c.start;
      bool kept = c.m == c.n;
      if (c.m > 0 && c.m < c.n) {
        if (A.arrival && c.r < A.k) {
          kept = pos < c.m;
        } else {
          const u32 mine = ckey[at];  // (a key is never 0)
          int better = 0;
#pragma unroll 8
          for (int q = 0; q < c.n; ++q) better += ckey[c.start + q] > (q < pos ? mine - 1 : mine);  // ties: the earlier token
          kept = better < c.m;
        }
      }
      if (kept) atomicOr(&kept_bits[at >> 5], 1u << (at & 31));
    }
    __syncthreads();
    for (int at = tid; at < NR * T; at += OR_THREADS) {
      if (!((kept_bits[at >> 5] >> (at & 31)) & 1u)) continue;
      const Cand c = cand_of(at);
      int sl = c.fill;  // and one for every kept candidate between the list's first and this one
      const int w0 = c.start >> 5, w1 = at >> 5;
      for (int q = w0; q <= w1; ++q) {
        u32 bits = kept_bits[q];
        if (q == w0) bits &= ~0u << (c.start & 31);
        if (q == w1) bits &= (1u << (at & 31)) - 1u;
        sl += __popc(bits);
      }
      const int tok = ctok[at];
      s_slot[c.r * T + tok] = (uint16_t)sl;
      slot_token[(size_t)c.j * A.C + c.g * A.Cq + sl] = tok;
    }
  } else for (int lst = w; lst < A.NL; lst += OR_WAVES) {
    const int cat = lst / A.Gq, g = lst - cat * A.Gq, r = cat / E, j = cat - r * E;
    int lo, hi;
    piece(r, j, g, lo, hi);
    const u32 pl = plan[lst];
    const int n = __builtin_amdgcn_readfirstlane(hi - lo), m = __builtin_amdgcn_readfirstlane((int)(pl >> 16));
    const int fill = pl & 0xffffu;
    if (m == 0) continue;
    const u32 *keys = ckey + s_base[cat] + lo;
    const uint16_t *toks = ctok + s_base[cat] + lo;
    int32_t *queue = slot_token + (size_t)j * A.C + g * A.Cq;
    const int trips = (n + kWave - 1) / kWave;
    const bool all = m == n, by_pos = m < n && A.arrival && r < A.k;
    auto place = [&](auto tag) {
      constexpr int NQ = decltype(tag)::value;  // at least `trips`: candidate q * 64 + lane is element q of the lane
      u32 kr[NQ], tr[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int idx = min(q * kWave + lane, n - 1);
        kr[q] = keys[idx];
        tr[q] = toks[idx];
      }
      // kept: keys above `thr`, and the first need_eq of those equal to it (by_pos: the first m)
      u32 thr = 0;
      int need_eq = by_pos ? m : 0;
      if (!all && !by_pos) {
        u32 a = 0xffffffffu, b = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {  // (copies of the last key past the end of the list)
          a = min(a, kr[q]);
          b = max(b, kr[q]);
          if (q * kWave + lane >= n) kr[q] = 0u;  // below every probe
        }
        a = wave_min(a);
        b = ~wave_min(~b) + 1;  // keys of finite scores stay below the largest u32
        // count(key >= a) >= m > count(key >= b) = cb; three probes a round, independent of each other
        int cb = 0;
        bool exact = false;
        while (b - a > 1) {
          const u32 h = (b - a) / 4, x1 = a + (h ? h : 1), x2 = a + (b - a) / 2, x3 = b - (h ? h : 1);
          int c1 = 0, c2 = 0, c3 = 0;
#pragma unroll
          for (int q = 0; q < NQ; ++q)
            if (q < trips) {
              c1 += __popcll(__ballot(kr[q] >= x1));
              c2 += __popcll(__ballot(kr[q] >= x2));
              c3 += __popcll(__ballot(kr[q] >= x3));
            }
          if (c1 == m || c2 == m || c3 == m) {
            thr = (c1 == m ? x1 : (c2 == m ? x2 : x3)) - 1;  // exactly the keys above it; nothing equal to it is taken
            exact = true;
            break;
          }
          if (c3 >= m) a = x3;
          else if (c2 >= m) { a = x2; b = x3; cb = c3; }
          else if (c1 >= m) { a = x1; b = x2; cb = c2; }
          else { b = x1; cb = c1; }
        }
        if (!exact) {
          thr = a;
          need_eq = m - cb;
        }
      }
      int run = 0, run_eq = 0;
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (q < trips) {
          const bool valid = q * kWave + lane < n;
          const bool gt = valid && (all || (!by_pos && kr[q] > thr)), eq = valid && !all && (by_pos || kr[q] == thr);
          const unsigned long long beq = __ballot(eq);
          const bool kept = gt || (eq && run_eq + (int)__popcll(beq & below_mask) < need_eq);
          const unsigned long long bk = __ballot(kept);
          if (kept) {
            const int sl = fill + run + __popcll(bk & below_mask);
            s_slot[r * T + tr[q]] = (uint16_t)sl;
            queue[sl] = tr[q];
          }
          run += __popcll(bk);
          run_eq += __popcll(beq);
        }
    };
    if (trips <= 1) place(std::integral_constant<int, 1>{});
    else if (trips <= 4) place(std::integral_constant<int, 4>{});
    else place(std::integral_constant<int, OR_WAVES>{});
  }
  __syncthreads();
  // ---- the tokens' slots; Intra-GPU candidates (Sec. 4.1)
  int slot_r[kMaxRank], ndrop = 0, ir_below = 0;
#pragma unroll
  for (int r = 0; r < kMaxRank; ++r) {
    slot_r[r] = -1;
    if (r < NR && i < T) {
      const u32 s = s_slot[r * T + i];
      if (s != NOSLOT) slot_r[r] = (A.Gq == 1 ? 0 : i / A.Tg * A.Cq) + (int)s;
      if (r < A.k) ndrop += s == NOSLOT;
      slot[(size_t)i * (A.k + 1) + r] = slot_r[r];
    }
  }
  if (i < T && !A.fr) slot[(size_t)i * (A.k + 1) + A.k] = -1;
  const bool has_ir = A.ir && ndrop > 0;
  if (row < rows) {
    const unsigned long long mask = same_expert_mask(has_ir, cand_h);
    ir_below = __popcll(mask & below_mask);
    if (has_ir && ir_below == 0) wir[row * E + cand_h] = (uint16_t)__popcll(mask);
  }
  __syncthreads();
  if (tid < E) {
    int sum = 0;
    for (int q = 0; q < rows; ++q) {
      const int v = wir[q * E + tid];
      wir[q * E + tid] = (uint16_t)sum;
      sum += v;
    }
    s_ircnt[tid] = sum;
  }
  __syncthreads();
  if (w == 0)
    row_plan_wave(A, true, lane < E ? s_fill[lane] : 0, lane < E && A.ir ? s_ircnt[lane] : 0, s_off, s_rbase, ir_offset, row_base,
                  tiles, tile_ctl);
  __syncthreads();
  if (i >= T) return;
  const int at = has_ir ? wir[row * E + cand_h] + ir_below : -1;
  ir_expert[i] = has_ir ? cand_h : -1;
  ir_row[i] = at;
  if (has_ir) ir_token[s_off[cand_h] + at] = i;
  if (row_dest)
    mark_rows(i, NR, slot_r, e_r, has_ir, has_ir ? s_rbase[cand_h] + s_fill[cand_h] + at : 0,
              [&](int e, int s) {
                const int g = s / A.Cq;
                return s_rbase[e] + (A.Gq == 1 ? 0 : grp_off[e * A.Gq + g]) + (s - g * A.Cq);
              },
              row_dest);
  write_weights(i, A.k, NR, slot_r, key_r, has_ir, ndrop, score_h, combine_w);
}

}  // namespace

static bool ir_large(const Dims &D) {
  return D.ir && D.E * D.NB > kIrSelfMax && D.E * ((D.T + kIrLargeBlock - 1) / kIrLargeBlock) <= kIrLargeSelfMax;
}
static DispatchArgs dispatch_args(const Dims &D) {
  return {D.T, D.E, D.k, D.C, D.NR, D.NCAT, D.NB, D.Eg, D.Tg, D.ir, D.fr, D.arrival, D.BM, D.max_mtiles,
          D.Cq, D.Gq, D.NL, D.NBc, D.cb, D.E * D.NB <= kIrSelfMax || ir_large(D) ? 1 : 0,
          select_direct(D) ? 1 : 0, D.Ts};
}

// One workgroup or the chain of launches?  One CU works through the lists (a wave each) and the candidates; the chain pays
// for its launches, one more with Intra-GPU lists and three more with several capacity blocks.  `saved`: us that one
// workgroup saves apart from those - more from logits that it ranks itself, less what the longest run of one lane's
// insertions takes.  The costs are a fit to 3100 batches of 8 to 1024 tokens, 1 to 64 experts, k 1 to 4, tables from logits
// and from ranks: with a line that the sizes of the LDS arrays alone set, one in five of them was up to 1.5 times as fast the
// other way; with this one the choice is 0.8 % off the better way on average.  Us, one workgroup / chain:
// 256 x 8, k 1: 12 / 22; 998 x 4, k 2: 22 / 29; 944 x 16, k 4: 30 / 22; 760 x 64, k 3, no Intra-GPU lists: 32 / 27; 1024 x 16, k 4: 47 / 32.
static bool one_is_cheaper(const Dims &D, float saved) {
  if (D.T > kOneT || (long long)D.E * D.C > kOneSlots) return false;
  return (float)D.NL * 0.01375f + (float)(D.T * D.NR) * 0.00212f <= saved + (D.ir ? 3.16f : 0.0f) + (D.Gq > 1 ? 8.93f : 0.0f);
}
bool route_in_one(const Dims &D, bool ranked) {
  float saved = 3.66f;
  if (!ranked && D.T * D.E <= kOneTile) {
    const int lanes = rank_lanes(D.T, D.E), list = D.k == 1 ? 2 : (D.k == 2 ? 3 : kMaxRank);
    saved += 2.95f - 0.04f * (float)((D.E + lanes - 1) / lanes * list);
  }
  return one_is_cheaper(D, saved);
}

// The forward call's router splits K over workgroups (of four waves) while they leave most CUs idle and the partial
// scores, which one workgroup reads, stay small: 16 tokens x 4096, 8 experts, router + tables 34 us with the router
// that ranks (one workgroup) and three table kernels, 26 us with it and one, 15 us with K split; 300 tokens x 2048,
// 16 experts 46, 31, 27 us.  Short rows gain less from the split, so that it ends at half as many scores for them.
// With the split one workgroup saves some 6 us more.
int router_parts(const Dims &D) {
  const int tiles = (D.T + 31) / 32, steps = (D.d + (D.dtype == RR_BF16 ? 63 : 31)) / (D.dtype == RR_BF16 ? 64 : 32);
  if (D.T > kOneT || D.T * D.E > (steps >= 32 ? 8192 : 4096) || !one_is_cheaper(D, 10.0f)) return 0;
  return std::max(1, std::min({kMaxParts, 256 / tiles, steps / 4, kMaxPartFloats / (D.T * D.E)}));
}
size_t router_parts_reserve(const Dims &D) { return std::min((size_t)kMaxPartFloats, (size_t)D.T * D.E * kMaxParts); }

static void launch_row_token(const Dims &D, const DispatchArgs &A, const rr_tables &tb, const Work &W, hipStream_t s) {
  if (D.quota && D.max_mtiles > 0)  // the forward pass addresses dispatched rows through row_token
    row_token_kernel<<<D.E, 256, 0, s>>>(A, tb.slot_token, W.grp_fill, W.grp_off, tb.fill_total, tb.ir_offset,
                                         tb.ir_token, W.row_base, W.row_token);
}

hipError_t launch_route_small(const Dims &D, const float *part, int kparts, const float *bias, float *logits,
                              const rr_tables &tb, const Work &W, bool ranked, int32_t *row_dest, hipStream_t s) {
  const DispatchArgs A = dispatch_args(D);
  const int src = ranked ? ROUTE_RANKED : (kparts ? ROUTE_PARTS : ROUTE_LOGITS);
  const OneLayout L = one_layout(D.T, D.E, D.NR, D.Gq, src != ROUTE_RANKED);
  prof_begin(K_ROUTE_SMALL, s);
  auto go = [&](auto kern) {
    kern<<<1, OR_THREADS, L.total, s>>>(A, part, kparts, bias, logits, tb.rank_expert, W.key, W.ir_score, W.ir_cand, tb.slot,
                                        tb.slot_token, W.grp_fill, W.grp_off, tb.fill_topk, tb.fill_total, tb.ir_offset,
                                        W.row_base, W.tiles, W.tile_ctl, tb.ir_expert, tb.ir_row, tb.ir_token,
                                        tb.combine_w, row_dest);
  };
  if (src == ROUTE_RANKED) go(route_small_kernel<ROUTE_RANKED>);
  else if (src == ROUTE_LOGITS) go(route_small_kernel<ROUTE_LOGITS>);
  else go(route_small_kernel<ROUTE_PARTS>);
  prof_end(K_ROUTE_SMALL, s);
  launch_row_token(D, A, tb, W, s);
  return hipGetLastError();
}

// route_small_kernel's dynamic LDS can exceed the default limit: raised once per device by the caller.
hipError_t dispatch_kernel_attributes() {
  hipError_t e = hipSuccess;
  auto set = [&e](auto kern) {
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 152 * 1024);
  };
  set(route_small_kernel<ROUTE_RANKED>);
  set(route_small_kernel<ROUTE_LOGITS>);
  set(route_small_kernel<ROUTE_PARTS>);
  return e;
}

hipError_t launch_dispatch(const Dims &D, const float *logits, const rr_tables &tb, const Work &W, bool ranked,
                           int32_t *row_dest, hipStream_t s) {
  const DispatchArgs A = dispatch_args(D);
  const bool in_one = route_in_one(D, ranked);
  if (in_one && !ranked && D.T * D.E <= kOneTile)
    return launch_route_small(D, nullptr, 0, nullptr, const_cast<float *>(logits), tb, W, false, row_dest, s);
  if (!ranked) {  // otherwise the router's epilogue has already written what topk_rank writes
    prof_begin(K_TOPK, s);
    topk_rank_kernel<<<D.NB, TK_THREADS, 0, s>>>(logits, A, tb.rank_expert, tb.slot, W.key, W.rank8, W.ir_score,
                                                W.ir_cand, W.blk_cnt);
    prof_end(K_TOPK, s);
  }
  if (in_one) return launch_route_small(D, nullptr, 0, nullptr, nullptr, tb, W, true, row_dest, s);
  if (A.direct) {
    prof_begin(K_SELECT_SLOT, s);
    select_direct_kernel<<<D.NCAT, SS_THREADS, 0, s>>>(A, W.rank8, W.key, tb.slot, tb.slot_token, W.grp_fill, W.grp_off,
                                                        tb.fill_topk, tb.fill_total);
    prof_end(K_SELECT_SLOT, s);
  } else {
    prof_begin(K_SCAN_CAND, s);
    // (also clears the tickets of the lists' segments: Gq lists per candidate array)
    scan_blocks_kernel<<<D.NCAT, SC_THREADS, 0, s>>>(W.blk_cnt, W.cat_cnt, D.NBc, W.list_done, D.Gq);
    prof_end(K_SCAN_CAND, s);
    prof_begin(K_SCATTER_CAND, s);
    scatter_candidates_kernel<<<D.NB, kTokBlock, 0, s>>>(A, tb.rank_expert, W.key, W.blk_cnt, W.cat_cnt, W.cand_key,
                                                         W.cand_tok, tb.slot, tb.slot_token);
    prof_end(K_SCATTER_CAND, s);
    prof_begin(K_SELECT_SLOT, s);
    // one workgroup per list, plus one for every further segment that a long list can have
    const bool splits = select_splits(D.T, D.NR, D.NL);
    auto select = [&](auto kern, int seg_len, int32_t *seg_more) {
      const int grid = D.NL + (splits ? (int)((long long)D.T * D.NR / seg_len) : 0);
      kern<<<grid, SS_THREADS, 0, s>>>(A, W.cat_cnt, W.blk_cnt, W.cand_key, W.cand_tok, W.comp_key, W.comp_tok, W.seg_cnt,
                                       seg_more, W.list_done, tb.slot, tb.slot_token, W.grp_fill, W.grp_off, tb.fill_topk,
                                       tb.fill_total);
    };
    // The counts of the further segments: one per kSelectShortLen candidates fits the Intra-GPU counts, which are written later.
    if (splits && (long long)D.T * D.NR <= kSelectShortMax) select(select_slot_kernel<kSelectShortLen>, kSelectShortLen, W.ir_blk_cnt);
    else select(select_slot_kernel<kSelectSegLen>, kSelectSegLen, W.seg_cnt + (splits ? D.NL : 0));
    prof_end(K_SELECT_SLOT, s);
  }
  auto intra_gpu = [&](auto count, auto weights, int block) {
    const int NB = (D.T + block - 1) / block;
    if (D.ir) {
      prof_begin(K_IR_COUNT, s);
      count<<<NB, block, 0, s>>>(A, tb.slot, W.ir_cand, W.ir_blk_cnt);
      prof_end(K_IR_COUNT, s);
      if (!A.ir_self) {
        prof_begin(K_IR_SCAN, s);
        scan_blocks_kernel<<<D.E, SC_THREADS, 0, s>>>(W.ir_blk_cnt, W.ir_cnt, NB, nullptr, 0);
        prof_end(K_IR_SCAN, s);
      }
    }
    prof_begin(K_IR_WEIGHTS, s);
    weights<<<NB, block, 0, s>>>(A, tb.slot, W.key, W.ir_score, W.ir_cand, W.ir_blk_cnt, W.ir_cnt, tb.fill_total, tb.ir_offset,
                                 W.row_base, W.tiles, W.tile_ctl, tb.ir_expert, tb.ir_row, tb.ir_token, tb.combine_w,
                                 tb.rank_expert, W.grp_off, row_dest);
  };
  if (ir_large(D)) intra_gpu(ir_count_kernel<kIrLargeBlock>, ir_weights_kernel<kIrLargeBlock>, kIrLargeBlock);
  else intra_gpu(ir_count_kernel<kTokBlock>, ir_weights_kernel<kTokBlock>, kTokBlock);
  prof_end(K_IR_WEIGHTS, s);
  launch_row_token(D, A, tb, W, s);
  return hipGetLastError();
}

}  // namespace rr

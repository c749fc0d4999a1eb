// Expert FFN as a grouped GEMM over the dispatched rows (Sec. 5.1: every expert is a LLaMA FFN):
//   up   : h[row, f] = silu(x[row] . W1_e[f]) * (x[row] . W3_e[f])      (SwiGLU)
//          h[row, f] = gelu(x[row] . W1_e[f])                            (GELU)
//   down : y[row, c] = h[row] . W2_e[c]
// Both are "A[rows,K] times B[N,K]^T" with K contiguous in both operands.  Rows of expert e are
// row_base[e] .. row_base[e+1]-1 and are cut into row tiles when the routing tables are built (TileInfo).
//
// Large bf16 layers: persistent kernel, one workgroup of 8 waves per CU, tiles of 256 x 256 staged rows
// dealt in an XCD-aware panel order (see "Tile order" in the kernel).
//   * v_mfma_f32_16x16x32_bf16, fp32 accumulate; 2 x 4 waves, wave tile 128 x 64; two waves per SIMD
//     so that one wave's LDS reads overlap the other's MFMAs.  (A loop of MFMAs alone on normally
//     distributed operands sustains 2030 TFLOP/s with this shape and 1330 with 32x32x16, 2470 and 1670
//     on zeros: the wide shape was the kernel's ceiling.)
//   * K advances in chunks of 64 through LDS rings - two 32 KB stages of A, three of B, 160 KB in all
//     - filled by buffer_load ... lds (16 bytes per lane straight into LDS, no staging registers);
//     the chunks of a workgroup's successive tiles form one stream.  A wave instruction fills 1 KB = 8
//     consecutive LDS rows (lane l -> row l/8, chunk position l%8), so the swizzle is applied on the
//     global side: the lane fetches the chunk that belongs at its position.  Rows past the end of
//     an operand read as zero (buffer range check): ragged tiles need no masks on the load side.
//   * LDS rows are 128 B; chunk c of row r sits at position c ^ ((r >> 1) & 7): conflict-free for
//     the 16 lanes x 16 B that the 64-bank LDS serves per cycle, for the DMA writes as well.
//   * The K loop is software-pipelined by hand (see k_loop): the compiler's own schedule waits for
//     every LDS read right before its first use.
//   * The up projection can read its A rows straight from x through the dispatch tables (GATHER):
//     the dispatch gather is then a per-lane row offset of the LDS DMA and costs no pass over HBM.
//   * The last round of tiles rarely fills the chip: where its tiles are at most half as many as the
//     workgroups they are cut by rows into up to eight parts (see "cut").  8 K tokens top-1, 2048 x 5632: down
//     projection 292 -> 249 us (384 tiles for 256 CUs); 4 K tokens 4096 x 11008, top-2: down 829 -> 695 (576 tiles).
//     The waves of a column take turns at the 16-row fragments, so that a short tile keeps all four SIMDs busy.
//   * While a tile's epilogue stores drain, the first K chunk of the workgroup's next tile is
//     already in flight (its tile id and table entries were fetched during the K loop).
// Layers with few rows or short rows, and all fp32 layers: gemm_tile_kernel, smaller tiles of several shapes
// (ffn_plan chooses the pair).
#include <algorithm>
#include <type_traits>

#include "rr_device.h"

namespace rr {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// Scheduling groups for the instruction scheduler (masks of sched_group_barrier: 0x008 MFMA,
// 0x100 LDS read, 0x020 global or buffer load).  They order the instructions of the surrounding
// scheduling region only; what the instructions compute is untouched.
// N times "one MFMA, then one LDS read":
template <int N>
__device__ __forceinline__ void sched_mfma_lds_read() {
  if constexpr (N > 0) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    sched_mfma_lds_read<N - 1>();
  }
}
// The step's R LDS reads and then its D LDS-DMA loads, each behind one of the step's first MFMAs.  The loads come last, as in
// the source: they write LDS, so the compiler moves no LDS read across them, and groups that ask for a load between two
// reads are not followed at all (the reads then run in one burst; 16384 tokens x 4096 x 11008: gate/up 4.66 -> 4.50 ms,
// down 2.34 -> 2.24, the MFMA pipe's share of the busy cycles 0.71 -> 0.77, the clock 1.75 -> 1.71 GHz).
template <int M, int R, int D>
__device__ __forceinline__ void sched_step() {
  if constexpr (M > 0 && R > 0) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    sched_step<M - 1, R - 1, D>();
  } else if constexpr (M > 0 && D > 0) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    sched_step<M - 1, 0, D - 1>();
  }
}

__device__ inline float silu(float g) { return g / (1.0f + __expf(-g)); }
// for results that are rounded to bf16 right away, in layers of whole K chunks, three at least (swiglu_divides): hardware
// reciprocal (1 ulp; 0 for arguments below -87.4, where the result is below 2e-36) instead of a division.  300 tokens, 2048 x
// 5632, 16 experts, 128 x 128 tiles: the layer 235 us, with the division 237.
__device__ inline float silu_fast(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
// two fp32 -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32), first value in the low half
__device__ inline u32 pack_bf16(float a, float b) {
  const f32x2_t f = {a, b};
  return __builtin_bit_cast(u32, __builtin_convertvector(f, bf16x2_t));
}
// g Phi(g).  (A single polynomial for erfc in 1 / (1 + 0.45 |g|) is 3 us less of a 6161 x 2728 up projection, 55 us, but
// 5 times the error for |g| < 1: 41 of 2^20 normal arguments of sigma 0.3 round to another bf16 than g Phi(g) does, here 3.)
__device__ inline float gelu_erf(float g) { return 0.5f * g * (1.0f + erff(g * 0.70710678118654752f)); }
constexpr int GB_BK = 64;             // bf16 elements per K chunk = 128 B per LDS row
constexpr int GB_ROW_BYTES = 128;
[[maybe_unused]] constexpr u32 BUF_FLAGS = 0x00020000; // raw buffer descriptor word 3 (32-bit data format)

struct GemmArgs {
  const void *A;        // [rows, K] dispatched rows; with GATHER: x [T, K]
  const void *B0;       // [E, N, K]
  const void *B1;       // [E, N, K] gated only
  void *Cout;           // [rows, N]
  int K, N;
  int NT;               // column tiles
  int sub;              // small-tile kernel: row tiles per row tile of the table
  const TileInfo *tiles;
  const int32_t *ctl;   // [0] number of row tiles
  // GATHER only
  const int32_t *slot_token, *ir_token;
  const int32_t *row_token;  // token of every dispatched row (per-group quotas), or NULL: rows are slots, then the Intra-GPU list
  int C;
  long long a_bytes;    // size of the A operand in bytes (buffer range of the gather)
  // DIRECT only (down projection): row_dest[row] = the token whose only processed row this is, else -1;
  // such a row is also stored as row row_dest[row] of Out, the layer's output (Eq. 2 with a single term)
  const int32_t *row_dest;
  void *Out;
};

// Two neighbouring 16x16 accumulators of a lane (four columns 4 * fg .. + 3 of column fragments j and j + 1, as bf16 pairs) ->
// eight columns in a row, eight_columns_at(fg) .. + 7 from fragment j on: lanes 16 apart exchange halves.  16384 tokens,
// 4096 x 11008, top-2: gate/up 4.47 -> 4.41 ms, down 2.25 -> 2.22; 8192 tokens, 2048 x 5632: down 272 -> 265 us.
__device__ __forceinline__ int eight_columns_at(int fg) { return (fg & 1) * 16 + (fg >> 1) * 8; }
__device__ __forceinline__ uint4 eight_columns(uint2 a, uint2 b) {
  const auto x = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false), y = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
  return make_uint4(x[0], y[0], x[1], y[1]);
}

// Epilogue of the persistent kernel, which multiplies with the operands swapped (B fragment first):
// the 16x16 accumulator then holds the transposed tile, i.e. a lane owns ONE output row (lane % 16 of
// the A fragment) and four consecutive columns, 4 * (lane / 16) .. + 3 of the B fragment; two accumulators make one
// 16-byte store per lane, 64 bytes of each of 16 rows.
// dest (DIRECT): per fragment row of this lane, the row of Ob that the same values are also stored to, or -1.
// The WAVES_M waves of a column take turns at the 16-row fragments of the tile.
template <int WM, int WN, int WAVES_M, bool GATED, int ACT, bool DIRECT = false>
__device__ inline void store_tile_t(f32x4 (&acc)[WM][WN], uint16_t *Cb, int rbase, int rows_e, int m0, int n0, int N,
                                    int wm, int wn, int lane, const int *dest = nullptr, uint16_t *Ob = nullptr) {
  constexpr int NJ = GATED ? WN / 2 : WN;  // output column fragments per wave
  const int fr = lane & 15, fg = lane >> 4;
  const int wrow0 = m0 + wm * 16, wcol0 = n0 + wn * NJ * 16;
  const bool cols_in = wcol0 + NJ * 16 <= N;  // N % 8 == 0: a group of eight columns is inside or outside as a whole
  const int ecol = eight_columns_at(fg);
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    const int row = wrow0 + i * WAVES_M * 16 + fr;
    if (row >= rows_e) continue;
    uint16_t *prow = Cb + (size_t)(rbase + row) * N + wcol0 + ecol;
    uint16_t *orow = nullptr;
    if (DIRECT && dest[i] >= 0) orow = Ob + (size_t)dest[i] * N + wcol0 + ecol;
#pragma unroll
    for (int j = 0; j < NJ; j += 2) {
      uint2 v[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          c[u] = acc[i][j + h][u];
          if (GATED) c[u] = (ACT == RR_ACT_SWIGLU ? silu(c[u]) : silu_fast(c[u])) * acc[i][j + h + NJ][u];
          if (ACT == RR_ACT_GELU) c[u] = gelu_erf(c[u]);
        }
        v[h] = make_uint2(pack_bf16(c[0], c[1]), pack_bf16(c[2], c[3]));
      }
      const uint4 val = eight_columns(v[0], v[1]);
      if (cols_in || wcol0 + j * 16 + ecol < N) {
        *reinterpret_cast<uint4 *>(prow + j * 16) = val;
        if (DIRECT && orow) *reinterpret_cast<uint4 *>(orow + j * 16) = val;
      }
    }
  }
}

__device__ inline int swz(int r) { return (r >> 1) & 7; }

// Barrier that publishes LDS-DMA data.  Before it signals, a wave's own buffer_load ... lds must
// have written LDS - all of them but the youngest YOUNGER, which belong to a later chunk (memory
// instructions complete in order) - and its own fragment reads of the stage that is about to be
// refilled must have returned (lgkmcnt 0).  Spelled out in assembly: the compiler's barrier waits
// for what its memory model takes for LDS traffic only, and when it does drain vmcnt it drains all.
template <int YOUNGER>
__device__ inline void dma_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(YOUNGER) : "memory");
}

// ------------------------------------------------------------------ bf16, persistent, LDS DMA
constexpr int PK_WAVES_M = 2, PK_WAVES_N = 4, PK_WM = 8, PK_WN = 4;  // waves, and 16-row fragments of a wave: 128 x 64
constexpr int PK_NW = PK_WAVES_M * PK_WAVES_N;
constexpr int PK_THREADS = PK_NW * 64;
constexpr int PK_BM = PK_WAVES_M * PK_WM * 16;     // 256
constexpr int PK_BROWS = PK_WAVES_N * PK_WN * 16;  // 256 staged B rows
constexpr int PK_A_STAGE = PK_BM * GB_ROW_BYTES, PK_B_STAGE = PK_BROWS * GB_ROW_BYTES;
[[maybe_unused]] constexpr int PK_MAX_CUT = 8;
constexpr int PK_A_STAGES = 2, PK_B_STAGES = 3;
constexpr int PK_B_BASE = PK_A_STAGES * PK_A_STAGE;
constexpr int PK_SMEM = PK_B_BASE + PK_B_STAGES * PK_B_STAGE;  // 160 KB: all of a CU's LDS
[[maybe_unused]] constexpr int PK_NI = (PK_BM + PK_BROWS) / 8 / PK_NW;  // 1 KB load instructions per wave per chunk
[[maybe_unused]] constexpr int PK_NIA = PK_BM / 8 / PK_NW;

template <bool GATED, int ACT, bool GATHER, bool DIRECT = false>
__global__ __launch_bounds__(PK_THREADS) void gemm_bf16_persistent_kernel(GemmArgs P) {
#if defined(__HIP_DEVICE_COMPILE__)  // buffer-resource and LDS-DMA builtins exist in the device pass only
  constexpr int WM = PK_WM, WN = PK_WN, NW = PK_NW, BM = PK_BM, NI = PK_NI, NIA = PK_NIA;
  constexpr int BN = GATED ? PK_BROWS / 2 : PK_BROWS;
  constexpr int NIB0 = BN / 8 / NW;
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "operand boundaries must fall between load instructions");
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int K = P.K, N = P.N, NT = P.NT, KT = (K + GB_BK - 1) / GB_BK;
  // Tile order.  Workgroups are dealt to the 8 XCDs round-robin (workgroup g runs on XCD g % 8) and
  // each XCD has its own L2.  The tiles are numbered panel by panel - panels of pm x pn neighbouring
  // tiles (4 row tiles x 8 column tiles for 32 workgroups per XCD), column panels first, ragged at the
  // right and bottom edges of the tile grid - and each run of pm * pn consecutive numbers goes to the
  // workgroups of one XCD: a chunk of an A row tile is then fetched into that L2 once for pn tiles
  // and a chunk of a B column tile once for pm, instead of once per tile, and consecutive rounds of
  // an XCD stay on the same rows of the same expert.
  const int MT = P.ctl[0], total = MT * NT;
  const int G = gridDim.x;
  const int nX = (G & 7) == 0 ? 8 : 1, S = G / nX;
  const int pn = (S & 7) == 0 ? 8 : 1, pm = S / pn;
  const int xcd = blockIdx.x % nX, slot = blockIdx.x / nX;
  const int PMf = MT / pm, PNf = NT / pn;  // full panel rows / columns
  // tile number k (panel order) -> linear index mt * NT + nt
  auto tile_at = [&](int k) {
    int qm = k / (pm * NT);
    if (qm > PMf) qm = PMf;
    const int r = k - qm * pm * NT, h = qm < PMf ? pm : MT - PMf * pm;
    int qn = r / (h * pn);
    if (qn > PNf) qn = PNf;
    const int r2 = r - qn * h * pn, wd = qn < PNf ? pn : NT - PNf * pn;
    const int dm = r2 / wd, dn = r2 - dm * wd;
    return (qm * pm + dm) * NT + qn * pn + dn;
  };
  // This workgroup's i-th tile is number (i * nX + xcd) * S + slot.  The tiles of the last, partial round are
  // spread over the XCDs and, where they are at most half as many as the workgroups, cut by rows into up to
  // PK_MAX_CUT parts that different workgroups take.
  const int rounds = total / G, left = total - rounds * G;
  const int cut = left > 0 ? min(G / left, PK_MAX_CUT) : 1;
  const int units = left * cut, per_xcd = (units + nX - 1) / nX;
  // tile of round i and, in the last round, which part of it; -1: none
  struct Unit { int L, part; };
  auto unit_at = [&](int i) {
    if (i < rounds) return Unit{tile_at((i * nX + xcd) * S + slot), -1};
    const int u = xcd * per_xcd + slot;
    if (i > rounds || slot >= per_xcd || u >= units) return Unit{-1, -1};
    return Unit{tile_at(rounds * G + u / cut), cut > 1 ? u % cut : -1};
  };
  int round = 0;
  Unit U = unit_at(0), U1 = unit_at(1), U2 = unit_at(2);  // this workgroup's current tile and the two after it
  if (U.L < 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps LDS-DMA addressing scalar
  const int wm = w / PK_WAVES_N, wn = w % PK_WAVES_N;
  const int fr = lane & 15, fg = lane >> 4;

  // fragment addressing (the same for every tile): lane reads row (lane & 15), chunk 4*ks + (lane >> 4)
  const int fsw = swz(fr);  // fragment rows start at multiples of 16, so the swizzle depends on fr only
  const int a_off = (wm * 16 + fr) * GB_ROW_BYTES;  // fragment i: + i * PK_WAVES_M * 16 rows
  // gated: the first half of a wave's column fragments are gate columns, the second the matching up columns
  const int b_off = (wn * (GATED ? WN / 2 : WN) * 16 + fr) * GB_ROW_BYTES;
  auto b_frag = [&](int j) { return (GATED && j >= WN / 2 ? BN + (j - WN / 2) * 16 : j * 16) * GB_ROW_BYTES; };

  // per-tile state.  A tile's table entry is fetched two tiles ahead and (GATHER) its token indices
  // one tile ahead, as plain vector loads issued right after a tile's first barrier: they complete
  // in the shadow of the K loop (whose next barrier is a whole K chunk of MFMAs away) and are only
  // touched after it, so no tile ever waits for a table lookup.
  struct Info { int e, m0, rbase, rows_e, fill_e, iroff_e, n0; };
  // Load addressing.  Instruction i of wave w fills stage rows [8 q, 8 q + 8), q = i * NW + w: lane l
  // fetches row 8 q + l / 8.  The swizzle of that row, ((8 q + l / 8) >> 1) & 7, does not depend on i
  // (8 NW is a multiple of 16), so a lane's offsets into one operand differ by a wave-uniform row
  // step from one instruction to the next: one register per operand (A gathered: one per
  // instruction), the step added when the load is issued.
  static_assert((8 * NW) % 16 == 0, "swizzle must not depend on the instruction index");
  constexpr int NVA = GATHER ? NIA : 1;
  // A tile keeps the base and range of its operands; the buffer descriptors are put together from
  // them when loads are issued, through readfirstlane: a descriptor that the register allocator has
  // parked in vector registers would otherwise be treated as divergent and every load wrapped in a
  // waterfall loop.
  struct Tile {
    int e, m0, rbase, rows_e, n0, live;
    int va[NVA], vb;
    unsigned long long pa, pb0, pb1;
    int na;
  };
  auto rsrc_of = [](unsigned long long base, int range) {
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)base);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(base >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char *>(((unsigned long long)hi << 32) | lo), 0,
                                             __builtin_amdgcn_readfirstlane(range), BUF_FLAGS);
  };
  const int lrow = w * 8 + (lane >> 3);            // stage row of this lane in instruction 0
  const int lcol = ((lane & 7) ^ swz(lrow)) * 16;  // byte position of its 16-byte chunk in the global row
  const unsigned rstep = NW * 8 * K * 2;           // bytes between the rows of consecutive instructions
  // this lane's piece of the last chunk lies past the end of the row (K no multiple of the chunk)
  const bool past = (KT - 1) * GB_BK * 2 + lcol >= K * 2;
  const char *Ab = static_cast<const char *>(P.A);
  auto raw_load = [&](int Lt, int4 &ra, int4 &rb) {
    const int4 *q = reinterpret_cast<const int4 *>(P.tiles + Lt / NT);
    ra = q[0];
    rb = q[1];
  };
  auto finalize = [&](const Unit &u, const int4 &ra, const int4 &rb) {
    Info f;
    f.e = __builtin_amdgcn_readfirstlane(ra.x);
    f.m0 = __builtin_amdgcn_readfirstlane(ra.y);
    f.rbase = __builtin_amdgcn_readfirstlane(ra.z);
    f.rows_e = __builtin_amdgcn_readfirstlane(ra.w);
    f.fill_e = __builtin_amdgcn_readfirstlane(rb.x);
    f.iroff_e = __builtin_amdgcn_readfirstlane(rb.y);
    f.n0 = (u.L % NT) * BN;
    if (u.part >= 0) {  // an equal share of the tile's rows, in whole fragments of both waves; past the last row: empty
      const int h = (min(BM, f.rows_e - f.m0) + cut * 32 - 1) / (cut * 32) * 32;
      f.m0 += u.part * h;
      f.rows_e = min(f.rows_e, f.m0 + h);
    }
    return f;
  };
  // the dispatch gather (Sec. 3: tokens travel to their experts): the tokens behind this lane's A
  // rows - occupied capacity slots first, then the expert's Intra-GPU rows; -1 = padding
  // Every lane always loads (rows past the expert's end read a valid dummy and are masked when the
  // offsets are built): the number of memory instructions per tile is then fixed, which the counted
  // waits of the K loop rely on.
  auto lookup_tokens = [&](const Info &f, int (&tok)[NIA]) {
#pragma unroll
    for (int i = 0; i < NIA; ++i) {
      const int lr = f.m0 + (i * NW + w) * 8 + (lane >> 3);  // row within the expert
      const int32_t *src = lr < f.fill_e ? P.slot_token + ((size_t)f.e * P.C + lr) : P.ir_token + (f.iroff_e + lr - f.fill_e);
      if (P.row_token) src = P.row_token + (f.rbase + lr);
      if (lr >= f.rows_e) src = P.slot_token;
      tok[i] = *src;
    }
  };
  auto make_tile = [&](const Info &f, const int (&tok)[NIA], Tile &t) {
    t.e = f.e; t.m0 = f.m0; t.rbase = f.rbase; t.rows_e = f.rows_e; t.n0 = f.n0;
    t.live = (min(BM, f.rows_e - f.m0) + PK_WAVES_M * 16 - 1) / (PK_WAVES_M * 16);
    const char *B0b = static_cast<const char *>(P.B0) + (size_t)f.e * N * K * 2;
    const char *B1b = GATED ? static_cast<const char *>(P.B1) + (size_t)f.e * N * K * 2 : B0b;
    if (GATHER) {
      t.pa = reinterpret_cast<unsigned long long>(Ab);
      t.na = (int)P.a_bytes;
    } else {
      t.pa = reinterpret_cast<unsigned long long>(Ab + (size_t)f.rbase * K * 2);
      t.na = (int)min((size_t)f.rows_e * K * 2, (size_t)0x7fffffff);
    }
    t.pb0 = reinterpret_cast<unsigned long long>(B0b);
    t.pb1 = reinterpret_cast<unsigned long long>(B1b);
    if (GATHER) {
#pragma unroll
      for (int i = 0; i < NVA; ++i) {
        const bool real = f.m0 + (i * NW + w) * 8 + (lane >> 3) < f.rows_e && tok[i] >= 0;
        t.va[i] = real ? tok[i] * K * 2 + lcol : 0x7ffffff0;  // padding: past the range, reads as zero
      }
    } else {
      t.va[0] = (f.m0 + lrow) * K * 2 + lcol;
    }
    t.vb = (f.n0 + lrow) * K * 2 + lcol;  // gate and up rows (GATED) sit at the same offsets of W1 and W3
  };
  // The stream of K chunks that the LDS rings are filled from: where the next chunk of A (NIA instructions
  // per wave) and of B (NIB) comes from.  It runs ahead of the multiplication into the next tile; past the
  // last tile its ranges are 0, so that every chunk issues the same number of loads.
  constexpr int NIB = NI - NIA;
  unsigned sva[NVA], svb;  // offsets of this lane
  int ska, skb, sna, snb;  // byte positions in K, ranges
  unsigned long long spa, spb0, spb1;
  auto stream_a = [&](const Tile &t, bool real) {
#pragma unroll
    for (int i = 0; i < NVA; ++i) sva[i] = t.va[i];
    spa = t.pa;
    sna = real ? t.na : 0;
    ska = 0;
  };
  auto stream_b = [&](const Tile &t, bool real) {
    svb = t.vb;
    spb0 = t.pb0;
    spb1 = t.pb1;
    snb = real ? N * K * 2 : 0;
    skb = 0;
  };
  auto issue_a = [&](int stage) {
    char *st = smem + stage * PK_A_STAGE + w * 1024;
    const __amdgpu_buffer_rsrc_t rsA = rsrc_of(spa, sna);
#pragma unroll
    for (int i = 0; i < NIA; ++i) {
      auto lp = (__attribute__((address_space(3))) void *)(st + i * NW * 1024);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, lp, 16, GATHER ? sva[i < NVA ? i : 0] : sva[0] + i * rstep, ska, 0, 0);
    }
    ska += GB_BK * 2;
  };
  auto issue_b = [&](int stage, int i0, int i1) {  // instructions i0 .. i1 - 1 of the chunk
    char *st = smem + PK_B_BASE + stage * PK_B_STAGE + w * 1024;
    const __amdgpu_buffer_rsrc_t rsB0 = rsrc_of(spb0, snb), rsB1 = rsrc_of(spb1, snb);
#pragma unroll
    for (int i = 0; i < NIB; ++i) {
      if (i < i0 || i >= i1) continue;
      // which weight matrix instruction i reads is known at compile time
      auto lp = (__attribute__((address_space(3))) void *)(st + i * NW * 1024);
      if (!GATED || i < NIB0)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB0, lp, 16, svb + i * rstep, skb, 0, 0);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB1, lp, 16, svb + (i - NIB0) * rstep, skb, 0, 0);
    }
    if (i1 == NIB) skb += GB_BK * 2;
  };
  auto next_b = [](int sb) { return sb == PK_B_STAGES - 1 ? 0 : sb + 1; };

  // LDS rings: A has two stages, B three (160 KB together).  The K chunks of a workgroup's tiles
  // form one stream (chunk KT of a tile is chunk 0 of its next tile).  While chunk c is multiplied,
  // A(c+1), B(c+1) and B(c+2) are in flight or landed: the weights, which stream from HBM, are
  // fetched two chunks ahead, the activations (mostly L2 hits: a row tile is shared by all column
  // tiles) one.  Each chunk issues A(c+1) and then B(c+2), so the barrier that publishes chunk c+1
  // waits for everything but the NIB youngest loads.  KT >= 3.
  f32x4 acc[WM][WN];
  Tile cur, nxt;
  Info info1{}, info2{};                              // table entries of this workgroup's next two tiles
  int4 ra2 = make_int4(0, 0, 0, 0), rb2 = ra2;        // raw table entry of the tile after next
  int tok1[NIA];        // token indices of the next tile's A rows
  int sa = 0, sb = 0;   // ring stages of the current chunk
  {
    int4 ra, rb;
    raw_load(U.L, ra, rb);
    const Info f0 = finalize(U, ra, rb);
    if (f0.m0 >= f0.rows_e) return;  // an empty part
    int tok0[NIA];
#pragma unroll
    for (int i = 0; i < NIA; ++i) tok0[i] = -1;
    if (GATHER) lookup_tokens(f0, tok0);
    make_tile(f0, tok0, cur);
    if (U1.L >= 0) {
      raw_load(U1.L, ra, rb);
      info1 = finalize(U1, ra, rb);
    }
    stream_a(cur, true);
    stream_b(cur, true);
    issue_a(sa);
    issue_b(sb, 0, NIB);
    issue_b(next_b(sb), 0, NIB);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NIB) : "memory");  // own A(0), B(0) have landed
  }
  while (true) {
    const bool have1 = U1.L >= 0 && info1.m0 < info1.rows_e;  // (only a workgroup's last tile can be an empty part)
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // Everybody's A(0), B(0) have landed: each wave saw its own arrive before it stored the previous
    // tile's results, so the barrier itself waits for no memory operation (the stores and B(1) may
    // still be on their way).
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // table lookups for the tiles to come, issued before this chunk's loads so that they are older
    // than anything a counted wait lets pass
    if (GATHER) lookup_tokens(info1, tok1);
    raw_load(U2.L >= 0 ? U2.L : U.L, ra2, rb2);
    int dest[WM];  // DIRECT: where the rows that this lane will store also go (this tile's, used in its epilogue)
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      dest[i] = -1;
      if (DIRECT) {
        const int row = cur.m0 + (i * PK_WAVES_M + wm) * 16 + fr;
        dest[i] = P.row_dest[cur.rbase + min(row, cur.rows_e - 1)];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    issue_a(sa ^ 1);
    issue_b(next_b(next_b(sb)), 0, NIB);

    // Ragged and cut row tiles: the two waves of a column take turns at the tile's 16-row fragments, and
    // the K loop comes in copies for 2, 4, 6 and 8 fragments per wave (branch-free, which keeps the counted
    // LDS waits exact), so a short tile costs MFMA time in proportion to its rows on all four SIMDs.
    auto k_loop = [&](auto live_tag) {
      // A chunk is four steps: k-step ks (of two), half hf of the wave's A rows.  A step multiplies half of the
      // A fragments with all B fragments of its k-step: 16 MFMAs in a full tile.
      constexpr int HM = decltype(live_tag)::value / 2, MF = HM * WN;
      bf16x8 af[2][HM], bfr[2][WN];
      auto load_a = [&](const char *sta, int ks, int hf) {
        const char *p = sta + a_off + (((4 * ks + fg) ^ fsw) << 4);
#pragma unroll
        for (int i = 0; i < HM; ++i)
          af[hf][i] = *reinterpret_cast<const bf16x8 *>(p + (hf * HM + i) * PK_WAVES_M * 16 * GB_ROW_BYTES);
      };
      auto load_b = [&](const char *stb, int ks) {
        const char *p = stb + b_off + (((4 * ks + fg) ^ fsw) << 4);
#pragma unroll
        for (int j = 0; j < WN; ++j) bfr[ks][j] = *reinterpret_cast<const bf16x8 *>(p + b_frag(j));
      };
      auto mfma_step = [&](int ks, int hf) {
#pragma unroll
        for (int i = 0; i < HM; ++i)
#pragma unroll
          for (int j = 0; j < WN; ++j)
            // B fragment first: the accumulator holds the transposed tile (see store_tile_t)
            acc[hf * HM + i][j] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[ks][j], af[hf][i], acc[hf * HM + i][j], 0, 0, 0);
      };
      // The chunk's LDS-DMA loads are spread over its steps, behind an MFMA each: A(kt+1) in the step
      // after the barrier, B(kt+2) in the two after it.  (All eight in one place - 64 per CU, 16 clocks of the
      // load unit each - kept the waves waiting at the issue: down projection at 8 K tokens x 5632 296 -> 275 us.
      // It takes straight-line code, hence the stream of chunks that runs past the tile's end.)
      // Software pipeline: the fragments that the NEXT step needs and this one does not hold are read
      // under the MFMAs of this one, one LDS read behind each of the first MFMAs.  (With all the reads in
      // front of the MFMAs the LDS pipe is asked for several KB per wave in one burst and is then idle
      // for the rest of the step; both waves of a SIMD doing so in turn leaves MFMA slots empty.)  The
      // last step of a chunk runs after the barrier; the global loads of the stream go behind its last
      // MFMAs.  The loop is rotated so that its body starts at the barrier (the compiler's wait
      // counting is exact only inside one basic block).
      // the first three steps of a chunk; the B loads of the stream ride in the first two of them
      auto steps = [&](const char *sta, const char *stb, auto dma_tag, int bstage) {
        constexpr bool DMA = decltype(dma_tag)::value;
        load_a(sta, 0, 1);
        if (DMA) issue_b(bstage, 0, NIB / 2);
        mfma_step(0, 0);
        sched_step<MF, HM, DMA ? NIB / 2 : 0>();
        __builtin_amdgcn_sched_barrier(0);
        load_a(sta, 1, 0);
        load_b(stb, 1);
        if (DMA) issue_b(bstage, NIB / 2, NIB);
        mfma_step(0, 1);
        sched_step<MF, HM + WN, DMA ? NIB - NIB / 2 : 0>();
        __builtin_amdgcn_sched_barrier(0);
        load_a(sta, 1, 1);
        mfma_step(1, 0);
        sched_step<MF, HM, 0>();
        __builtin_amdgcn_sched_barrier(0);
      };
      const char *sta = smem + sa * PK_A_STAGE, *stb = smem + PK_B_BASE + sb * PK_B_STAGE;
      load_a(sta, 0, 0);
      load_b(stb, 0);
      steps(sta, stb, std::false_type{}, 0);
      // The looked-up values are consumed here, unconditionally, rather than where they are first
      // needed: in straight-line code after the lookups the compiler's wait for them is a counted
      // one (the A(1) and B(2) loads behind them stay in flight), and nothing it tracks is pending
      // when the loop is entered or the tile ends - there it would drain every outstanding load
      // and store.  Without a next tile the values are unused.
      make_tile(info1, tok1, nxt);
      info2 = finalize(U2.L >= 0 ? U2 : U, ra2, rb2);
      if (DIRECT) {  // consumed here like the other lookups, so that no load is pending when the loop is entered
#pragma unroll
        for (int i = 0; i < WM; ++i) asm volatile("" : "+v"(dest[i]));
      }
      for (int kt = 1; kt < KT; ++kt) {
        // the stream moves on to the next tile: A one chunk, B two chunks before this tile ends
        if (kt == KT - 2) stream_b(nxt, have1);
        if (kt == KT - 1) stream_a(nxt, have1);
        if (K % GB_BK) {  // in the last chunk of a row, pieces past its end are sent out of range: they read as zero
          if (kt == KT - 3 && past) svb = 0x7ffffff0;
          if (kt == KT - 2 && past) {
#pragma unroll
            for (int i = 0; i < NVA; ++i) sva[i] = 0x7ffffff0;
          }
        }
        // A(kt) and B(kt) have landed - the B issued after A(kt) may still be on its way - and
        // nobody reads the stages of chunk kt-1 any more
        dma_barrier<NIB>();
        sa ^= 1;
        sb = next_b(sb);
        sta = smem + sa * PK_A_STAGE;
        stb = smem + PK_B_BASE + sb * PK_B_STAGE;
        load_a(sta, 0, 0);
        load_b(stb, 0);
        issue_a(sa ^ 1);
        mfma_step(1, 1);  // last step of chunk kt-1
        sched_step<MF, HM + WN, NIA>();
        __builtin_amdgcn_sched_barrier(0);
        steps(sta, stb, std::true_type{}, next_b(next_b(sb)));
      }
      mfma_step(1, 1);
    };
    const int live = cur.live;
    if (live > 6) k_loop(std::integral_constant<int, 8>{});
    else if (live > 4) k_loop(std::integral_constant<int, 6>{});
    else if (live > 2) k_loop(std::integral_constant<int, 4>{});
    else k_loop(std::integral_constant<int, 2>{});

    // own A(0), B(0) of the next tile have landed (they were issued one and two chunks ago), before
    // the stores below join the queue of outstanding memory operations
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NIB) : "memory");
    sa ^= 1;
    sb = next_b(sb);
    store_tile_t<WM, WN, PK_WAVES_M, GATED, ACT, DIRECT>(acc, static_cast<uint16_t *>(P.Cout), cur.rbase, cur.rows_e, cur.m0, cur.n0,
                                             N, wm, wn, lane, dest, static_cast<uint16_t *>(P.Out));
    if (!have1) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the stream's loads past the last tile still write this LDS
      break;
    }
    cur = nxt;
    U = U1;
    U1 = U2;
    U2 = unit_at(++round + 2);
    info1 = info2;
  }
#endif
}

// Four fp32 values, times kSplitScale, as sums of three bf16 values, each the nearest of what the ones before it leave (8
// mantissa bits and a sign: three of them hold all 24): plane[p] gets part p of the four.  bf16 counts down to 2^-133, so the
// parts of values below 2^-110 would lose bits: the scale lifts fp32's smallest step, 2^-149, to there, and the sum of
// products is brought back by kSplitUnscale (powers of two: nothing is rounded).  Values from 2^89 and sums from 2^50 on
// become infinities and are computed again (see the end of the K loop).  2048 tokens, 1024 x 2816, 8 experts: 510 us without the
// scale (tokens at 2^-122: an error of 8e-4), 503 with it as a 4-byte multiplication and 4-byte subtractions, 519 as 8-byte ones.
// Conversions and subtractions only: v_dot2c_f32_bf16 with (-1, 0) would subtract a packed value from its fp32 one without unpacking
// it (7 instructions for two values, not 11 and the 2 of the scale), but does not run beside MFMAs (22 cycles each, v_sub_f32 8).
constexpr float kSplitScale = 0x1p39f, kSplitUnscale = 0x1p-78f;
__device__ __forceinline__ void split3(const f32x4 &x, float scale, uint2 (&plane)[3]) {
#pragma clang fp contract(off)  // (the first subtraction as a fused one is 8 bytes long too)
  u32 w[3][2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    float a = x[2 * q] * scale, b = x[2 * q + 1] * scale;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      w[p][q] = pack_bf16(a, b);
      if (p < 2) {
        a -= __builtin_bit_cast(float, w[p][q] << 16);
        b -= __builtin_bit_cast(float, w[p][q] & 0xffff0000u);
      }
    }
  }
#pragma unroll
  for (int p = 0; p < 3; ++p) plane[p] = make_uint2(w[p][0], w[p][1]);
}

// ------------------------------------------------------------------ small tiles, bf16 and fp32, any K % 8 == 0
// Everything the 256 x 256 kernel is not made for: fp32 layers, row lengths that are no multiple of the
// K chunk or shorter than three of them, and batches whose experts get few rows.  One workgroup per tile,
// several workgroups per CU: one's epilogue, table lookups and barrier waits run under another's MFMAs.
//   * K advances in chunks of 128 bytes of every staged row through a ring of ST stages filled by
//     buffer_load ... lds with the same row layout and swizzle as above; a chunk is requested ST - 1 chunks
//     ahead, into the stage that the barrier at the top of the chunk has just freed, and every chunk
//     issues the same number of loads (past the end: out of range, which costs no traffic), so one
//     counted wait serves any K.  Pieces past the end of a row are sent out of range as well: they read as zero.
//   * bf16: v_mfma_f32_16x16x32_bf16.  fp32: v_mfma_f32_16x16x4_f32, fp32 products and accumulation; a
//     lane's 16-byte piece is its operand of four MFMAs - the K order inside a chunk is then a
//     permutation, the same for both operands.
//   * fp32 rows of five chunks and more that fill their tiles (TILE_SPLIT): every operand is split into three bf16 parts
//     that hold its 24 bits, and the six products down to 2^-18 of the leading one run on the bf16 pipe, accumulated in
//     fp32 (a split of Dekker's kind, as the router's; the three left out are up to 2^-24.2 of a product, so a lone product is
//     off by up to 0.94 ulp, where an fp32 MFMA rounds it to 0.5): 96 cycles of MFMAs per pair of fragments and chunk instead of 256.
//     The parts are made once per workgroup, on the way to LDS (a wave that splits its own fragments does it two to four
//     times over, and conversions run at half speed beside MFMAs: 285 us instead of 265 for the layer below).  Error
//     against 64 bits below that of the fp32 MFMAs, which round as often (1024 tokens, 1024 x 2816 SwiGLU 1.09e-6
//     of the output's norm, 1.29e-6; 4096 x 4096 1.80e-6, 2.09e-6; 64 x 128 GELU 1.8e-7, 2.6e-7).
//     Of 40 layers from 32 to 4096 wide none has a larger error; with tokens of one to four nonzero values 1.5 % at most, 2.5 % less on average.
//     3931 rows, 1024 x 2816 SwiGLU, 64 x 128 tiles: up 355 -> 284 us, down 187 - 208 -> 198 (530 tiles, two on a CU that holds four: too
//     little beside the barriers); 7900 rows, 2112 x 4224 GELU, 128 x 128: 1077 -> 745, 1075 -> 773.  Bound by the bf16 pipe (57 % of the cycles
//     at 2.03 GHz) and the splitting beside it.
// Measured, before (register-staged bf16 kernel, fp32 FMA kernel) -> now: 6161 rows, 1000 x 2728, bf16 GELU, down 118 -> 47 us
// (the up projection runs on 256 x 256 tiles: 163 -> 58); 3931 rows, 1024 x 2816, fp32 SwiGLU: up 612 -> 354 us (128 TFLOP/s; the fp32 MFMA pipe sustains 154),
// down 397 -> 184.  bf16 tiles of this size are bound by the operand bytes per flop (L2 -> LDS), fp32 ones by the MFMAs.
// WM x WN: 16-row fragments of a wave.
enum TileMath { TILE_BF16, TILE_F32, TILE_SPLIT };  // TILE_SPLIT: fp32 operands as three bf16 parts each
template <TileMath MATH_, int WAVES_M_, int WAVES_N_, int WM_, int WN_, int ST_, int OCC_>
struct TileShape {
  static constexpr TileMath MATH = MATH_;
  static constexpr bool BF16 = MATH == TILE_BF16;
  static constexpr int WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, WM = WM_, WN = WN_, ST = ST_, OCC = OCC_;
  static constexpr int NW = WAVES_M * WAVES_N, THREADS = NW * 64;
  static constexpr int BM = WAVES_M * WM * 16, BROWS = WAVES_N * WN * 16;
  static constexpr int STAGE = (BM + BROWS) * (MATH == TILE_SPLIT ? 3 * GB_ROW_BYTES / 2 : GB_ROW_BYTES), SMEM = ST * STAGE;
};

// ACT: RR_ACT_GELU, RR_ACT_SWIGLU (bf16: with the division), or -1
template <class S, bool GATED, int ACT, bool GATHER, bool DIRECT>
__global__ __launch_bounds__(S::THREADS, S::OCC) void gemm_tile_kernel(GemmArgs P) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int WM = S::WM, WN = S::WN, NW = S::NW, BM = S::BM, ST = S::ST;
  constexpr int BN = GATED ? S::BROWS / 2 : S::BROWS;
  constexpr int NIA = BM / 8 / NW, NIB = S::BROWS / 8 / NW, NI = NIA + NIB, NIB0 = BN / 8 / NW;
  constexpr int ES = S::BF16 ? 2 : 4, CE = GB_ROW_BYTES / ES, PE = 16 / ES;  // elements per chunk of a row, per piece
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "operand boundaries must fall between load instructions");
  static_assert((8 * NW) % 16 == 0, "swizzle must not depend on the instruction index");
  static_assert(!GATED || WN % 2 == 0, "a wave holds the gate and the up columns of its outputs");
  constexpr int kPanel = 8;  // row tiles that share a column tile of weights before the next column tile
  extern __shared__ __attribute__((aligned(16))) char smem[];

  // tile number: each XCD (workgroup g runs on XCD g % 8) takes a contiguous run; panels of kPanel row
  // tiles, column tiles inside a panel, row tiles inside a column: neighbours share weights
  // (the table's row tiles are P.sub times as high as this kernel's)
  const int MT = P.ctl[0] * P.sub, NT = P.NT, total = MT * NT;
  const unsigned g = blockIdx.y * gridDim.x + blockIdx.x;  // rows of whole XCD runs (tile_grid)
  const int per = (total + 7) >> 3, run = (int)(g >> 3), t = (int)(g & 7) * per + run;
  if (run >= per || t >= total) return;
  const int panel = t / (kPanel * NT), r = t - panel * kPanel * NT, h = min(kPanel, MT - panel * kPanel);
  const int nt = r / h, mt = panel * kPanel + r - nt * h;
  const TileInfo ti = P.tiles[mt / P.sub];
  const int m0 = ti.row0 + mt % P.sub * BM;
  if (m0 >= ti.rows) return;
  const int K = P.K, N = P.N, KT = (K + CE - 1) / CE;
  const int e = ti.expert, rbase = ti.rbase, rows_e = ti.rows, n0 = nt * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w / S::WAVES_N, wn = w % S::WAVES_N;
  const int fr = lane & 15, fg = lane >> 4;
  constexpr unsigned PAST = 0x7ffffff0u;  // past every operand's range: reads as zero

  // ---- operands: buffers that start at the tile's first row (GATHER: at x) and end with its last one
  const int lrow = w * 8 + (lane >> 3);            // stage row of this lane in instruction 0
  const int piece = S::MATH == TILE_SPLIT ? lane & 7 : (lane & 7) ^ swz(lrow);  // 16-byte piece of the row's chunk that belongs at its position
  const unsigned rowb = (unsigned)K * ES;
  const unsigned rstep = NW * 8 * rowb;            // between the rows of consecutive instructions
  auto rsrc = [](const char *base, size_t off, long long range) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base) + off, 0,
                                             __builtin_amdgcn_readfirstlane((int)range), BUF_FLAGS);
  };
  const size_t mat = (size_t)e * N * K * ES + (size_t)n0 * rowb;
  const long long brange = (long long)min(BN, N - n0) * rowb;
  const __amdgpu_buffer_rsrc_t rsB0 = rsrc(static_cast<const char *>(P.B0), mat, brange);
  const __amdgpu_buffer_rsrc_t rsB1 = GATED ? rsrc(static_cast<const char *>(P.B1), mat, brange) : rsB0;
  const __amdgpu_buffer_rsrc_t rsA =
      GATHER ? rsrc(static_cast<const char *>(P.A), 0, P.a_bytes)
             : rsrc(static_cast<const char *>(P.A), (size_t)(rbase + m0) * rowb, (long long)min(BM, rows_e - m0) * rowb);
  auto load16 = [](const __amdgpu_buffer_rsrc_t &rs, unsigned off, int koff) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, koff, 0));
  };
  auto token_of = [&](int lr) {  // row within the expert: capacity slots first, then its Intra-GPU rows
    const int32_t *src = lr < ti.fill ? P.slot_token + ((size_t)e * P.C + lr) : P.ir_token + (ti.ir_offset + lr - ti.fill);
    if (P.row_token) src = P.row_token + (rbase + lr);
    if (lr >= rows_e) src = P.slot_token;  // a valid dummy: the lookups of all instructions are in flight together
    return *src;
  };
  unsigned va[GATHER ? NIA : 1];
  if (GATHER) {
#pragma unroll
    for (int i = 0; i < NIA; ++i) va[i] = (unsigned)token_of(m0 + i * NW * 8 + lrow);
#pragma unroll
    for (int i = 0; i < NIA; ++i) va[i] = m0 + i * NW * 8 + lrow < rows_e ? va[i] * rowb + piece * 16 : PAST;
  } else {
    va[0] = lrow * rowb + piece * 16;
  }
  const unsigned vb = lrow * rowb + piece * 16;
  auto issue = [&](int kt, int stage) {
    char *st = smem + stage * S::STAGE + w * 1024;
    const bool past = kt * CE + piece * PE >= K;  // the last chunk of a ragged K, and chunks past the end
    const int koff = min(kt, KT - 1) * GB_ROW_BYTES;
#pragma unroll
    for (int i = 0; i < NIB; ++i) {
      auto lp = (__attribute__((address_space(3))) void *)(st + BM * GB_ROW_BYTES + i * NW * 1024);
      const unsigned v = vb + (GATED && i >= NIB0 ? i - NIB0 : i) * rstep;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(!GATED || i < NIB0 ? rsB0 : rsB1, lp, 16, past ? PAST : v, koff, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < NIA; ++i) {
      auto lp = (__attribute__((address_space(3))) void *)(st + i * NW * 1024);
      const unsigned v = GATHER ? va[GATHER ? i : 0] : va[0] + i * rstep;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, lp, 16, past ? PAST : v, koff, 0, 0);
    }
  };

  // ---- fragments: lane reads row (lane & 15), piece 4 ks + (lane >> 4) of k-step ks (two per chunk)
  int a_off[WM], b_off[WN];
  const int fsw = swz(fr);  // fragment rows start at multiples of 16, so the swizzle depends on fr only
#pragma unroll
  for (int i = 0; i < WM; ++i) a_off[i] = ((wm * WM + i) * 16 + fr) * GB_ROW_BYTES;
#pragma unroll
  for (int j = 0; j < WN; ++j) {
    constexpr int H = WN / 2;
    int row = (wn * WN + j) * 16 + fr;
    if (GATED) row = (j < H) ? (wn * H + j) * 16 + fr : BN + (wn * H + (j - H)) * 16 + fr;
    b_off[j] = (BM + row) * GB_ROW_BYTES;
  }
  using Frag = typename std::conditional<S::BF16, bf16x8, f32x4>::type;
  f32x4 acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  Frag af[2][WM], bfr[2][WN];
  auto load_frags = [&](const char *st, int ks) {
    const int pos = ((4 * ks + fg) ^ fsw) << 4;
#pragma unroll
    for (int i = 0; i < WM; ++i) af[ks][i] = *reinterpret_cast<const Frag *>(st + a_off[i] + pos);
#pragma unroll
    for (int j = 0; j < WN; ++j) bfr[ks][j] = *reinterpret_cast<const Frag *>(st + b_off[j] + pos);
  };
  // B fragment first: the accumulator holds the transposed tile, a lane owns row (lane & 15) of the A
  // fragment and four consecutive columns, 4 * (lane >> 4) .. + 3 of the B fragment
  auto mfma_step = [&](int ks) {
    if constexpr (S::BF16) {
#pragma unroll
      for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[ks][j], af[ks][i], acc[i][j], 0, 0, 0);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
          for (int j = 0; j < WN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bfr[ks][j][q], af[ks][i][q], acc[i][j], 0, 0, 0);
    }
  };

  if constexpr (S::MATH != TILE_SPLIT)
#pragma unroll
    for (int q = 0; q < ST - 1; ++q) issue(q, q);
  int dest[WM];
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    dest[i] = -1;
    if (DIRECT) dest[i] = P.row_dest[rbase + min(m0 + (wm * WM + i) * 16 + fr, rows_e - 1)];
  }
  int cur = 0, fill = ST - 1;
  if constexpr (S::MATH == TILE_SPLIT) {
    // Chunks go through registers: a lane holds four elements of NI rows, splits them and writes 8 bytes to each of the
    // three planes in LDS, 64 bytes per row and chunk; the next chunk is requested before this one is multiplied.
    f32x4 raw[NI];
    auto fetch = [&](int kt) {
      const bool past = kt * CE + piece * PE >= K;
      const int koff = min(kt, KT - 1) * GB_ROW_BYTES;
#pragma unroll
      for (int i = 0; i < NIB; ++i) {
        const unsigned v = vb + (GATED && i >= NIB0 ? i - NIB0 : i) * rstep;
        raw[NIA + i] = load16(!GATED || i < NIB0 ? rsB0 : rsB1, past ? PAST : v, koff);
      }
#pragma unroll
      for (int i = 0; i < NIA; ++i) {
        const unsigned v = GATHER ? va[GATHER ? i : 0] : va[0] + i * rstep;
        raw[i] = load16(rsA, past ? PAST : v, koff);
      }
    };
    // 16-byte piece c of a plane's row sits at c ^ ((row >> 2) & 3): the 16 rows of a fragment then fill all 64 banks
    constexpr int PLANE = (BM + S::BROWS) * GB_ROW_BYTES / 2;
    char *const wr = smem + lrow * 64 + (((piece >> 1) ^ ((lrow >> 2) & 3)) << 4) + (piece & 1) * 8;
    const int fpos = fr * 64 + ((fg ^ (fr >> 2)) << 4);
    float scale;  // in a register: a multiplication of 4 bytes instead of 8
    asm("s_mov_b32 %0, %1" : "=s"(scale) : "i"(__builtin_bit_cast(int, kSplitScale)));
    fetch(0);
    for (int kt = 0; kt < KT; ++kt) {
      if (kt > 0) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // everybody has read chunk kt - 1
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        uint2 q[3];
        split3(raw[i], scale, q);
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<uint2 *>(wr + p * PLANE + i * NW * 8 * 64) = q[p];
        // (128 x 128: all rows' parts at once do not fit the registers.  9048 tokens, 768 x 1344, 64 experts: 690 us, two rows at a time 662;
        // 64 x 128 has the room: 2048 tokens, 1024 x 2816, 8 experts 504, two rows at a time 514)
        if (WM == 4 && i % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
      fetch(kt + 1);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // chunk kt is written
      bf16x8 b3[WN][3];
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int p = 0; p < 3; ++p)
          b3[j][p] = *reinterpret_cast<const bf16x8 *>(smem + p * PLANE + (b_off[j] / GB_ROW_BYTES - fr) * 64 + fpos);
#pragma unroll
      for (int i = 0; i < WM; ++i) {
        bf16x8 a3[3];
#pragma unroll
        for (int p = 0; p < 3; ++p)
          a3[p] = *reinterpret_cast<const bf16x8 *>(smem + p * PLANE + (wm * WM + i) * 16 * 64 + fpos);
        // the products of parts down to 2^-18 of the leading one, smallest first
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
          for (int j = 0; j < WN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b3[j][PB[q]], a3[PA[q]], acc[i][j], 0, 0, 0);
      }
    }
    // An infinity, or a value that the scale or bf16's rounding makes one, leaves NaN behind its first part: a fragment of
    // which any element is not finite is computed again from fp32 operands.
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      const int arow = (wm * WM + i) * 16 + fr;  // of the tile
      unsigned ao = arow * rowb;
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        bool finite = true;
#pragma unroll
        for (int u = 0; u < 4; ++u) finite = finite && __builtin_isfinite(acc[i][j][u]);
        if (__all(finite)) {
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[i][j][u] *= kSplitUnscale;
          continue;
        }
        if (GATHER) ao = m0 + arow < rows_e ? (unsigned)token_of(m0 + arow) * rowb : PAST;
        const bool up = GATED && j >= WN / 2;
        const unsigned bo = (unsigned)(GATED ? (wn * (WN / 2) + j % (WN / 2)) * 16 + fr : (wn * WN + j) * 16 + fr) * rowb;
        f32x4 c = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int k = 0; k < K; k += 16) {
          const unsigned kb = (k + 4 * fg) * ES;
          const bool past = kb >= rowb;
          const f32x4 a = load16(rsA, past || ao == PAST ? PAST : ao + kb, 0), b = load16(up ? rsB1 : rsB0, past ? PAST : bo + kb, 0);
#pragma unroll
          for (int u = 0; u < 4; ++u) c = __builtin_amdgcn_mfma_f32_16x16x4f32(b[u], a[u], c, 0, 0, 0);
        }
        acc[i][j] = c;
      }
    }
  } else {
    for (int kt = 0; kt < KT; ++kt) {
      // own loads of chunk kt have landed (ST - 2 younger chunks may be on their way), own reads of chunk kt - 1 too
      dma_barrier<(ST - 2) * NI>();
      const char *st = smem + cur * S::STAGE;
      // software pipeline: the fragments of the next k-step are read under the MFMAs of this one
      load_frags(st, 0);
      if (kt > 0) mfma_step(1);  // last k-step of chunk kt - 1
      issue(kt + ST - 1, fill);
      __builtin_amdgcn_sched_barrier(0);
      load_frags(st, 1);
      mfma_step(0);
      if constexpr (S::BF16) sched_mfma_lds_read<(WM + WN < WM * WN ? WM + WN : WM * WN)>();
      __builtin_amdgcn_sched_barrier(0);
      cur = cur == ST - 1 ? 0 : cur + 1;
      fill = fill == ST - 1 ? 0 : fill + 1;
    }
    mfma_step(1);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // loads past the last chunk still write this LDS

  // ---- epilogue
  constexpr int NJ = GATED ? WN / 2 : WN;
  const int wrow0 = m0 + wm * WM * 16, wcol0 = n0 + wn * NJ * 16 + 4 * fg;
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    const int row = wrow0 + i * 16 + fr;
    if (row >= rows_e) continue;
    char *prow = static_cast<char *>(P.Cout) + (size_t)(rbase + row) * N * ES;
    char *orow = DIRECT && dest[i] >= 0 ? static_cast<char *>(P.Out) + (size_t)dest[i] * N * ES : nullptr;
    constexpr bool PAIRS = S::BF16 && NJ % 2 == 0;
    uint2 even = make_uint2(0, 0);  // PAIRS: the accumulator before this one
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int col = PAIRS ? wcol0 - 4 * fg + (j & ~1) * 16 + eight_columns_at(fg) : wcol0 + j * 16;
      float c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        c[u] = acc[i][j][u];
        if (GATED) c[u] = (!S::BF16 ? c[u] / (1.0f + expf(-c[u])) : (ACT == RR_ACT_SWIGLU ? silu(c[u]) : silu_fast(c[u]))) * acc[i][j + NJ][u];
        if (ACT == RR_ACT_GELU) c[u] = gelu_erf(c[u]);
      }
      uint2 val2 = make_uint2(0, 0);
      uint4 val4 = make_uint4(0, 0, 0, 0);
      if constexpr (S::BF16) val2 = make_uint2(pack_bf16(c[0], c[1]), pack_bf16(c[2], c[3]));
      if constexpr (PAIRS) {
        if (j % 2 == 0) {
          even = val2;
          continue;
        }
        val4 = eight_columns(even, val2);
      }
      if (col < N) {  // N % 8 == 0: a group of four or eight columns is inside or outside as a whole
        if constexpr (PAIRS) {
          *reinterpret_cast<uint4 *>(prow + (size_t)col * ES) = val4;
          if (DIRECT && orow) *reinterpret_cast<uint4 *>(orow + (size_t)col * ES) = val4;
        } else if constexpr (S::BF16) {
          *reinterpret_cast<uint2 *>(prow + (size_t)col * ES) = val2;
          if (DIRECT && orow) *reinterpret_cast<uint2 *>(orow + (size_t)col * ES) = val2;
        } else {
          const float4 val = make_float4(c[0], c[1], c[2], c[3]);
          *reinterpret_cast<float4 *>(prow + (size_t)col * ES) = val;
          if (DIRECT && orow) *reinterpret_cast<float4 *>(orow + (size_t)col * ES) = val;
        }
      }
    }
  }
#endif
}

// ------------------------------------------------------------------ rows or columns of 2^23 elements and more, bf16 and fp32
// The kernels above address a tile's rows with 32-bit byte offsets.  Past kLongRow elements this one takes over, with
// 64-bit addresses: 32 rows x 16 columns (gated: of both matrices) per workgroup, its waves split K, fragments come
// straight from global memory (a lane's 16 bytes are its operand, as above), the partial tiles are summed through
// LDS in a fixed order.  Bound by the latency of its loads; such layers are one or two tiles wide in the
// other dimension, so that splitting K is what fills the chip: 6 rows, 2 experts, 8 x 2^23 bf16: down 10.5 ms, up 5.5 (256 x 256
// tiles: 117 and 5.4); the layer of 2^23 x 24 in fp32 84 ms (64 x 64 tiles of FMAs: 1047).
constexpr int kLongRow = 1 << 23;
constexpr int LG_NW = 16, LG_THREADS = LG_NW * 64, LG_ROWS = 32, LG_COLS = 16;

template <bool BF16, bool GATED, int ACT, bool GATHER, bool DIRECT>
__global__ __launch_bounds__(LG_THREADS) void gemm_long_kernel(GemmArgs P) {
  constexpr int ES = BF16 ? 2 : 4, PE = 16 / ES, KM = 4 * PE, NB = GATED ? 2 : 1;
  using Frag = typename std::conditional<BF16, bf16x8, f32x4>::type;
  __shared__ float red[LG_NW][2 * NB * 4][64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 15, q = lane >> 4;
  const int N = P.N, NT = P.NT;
  const long long K = P.K, t = (long long)blockIdx.y * gridDim.x + blockIdx.x;
  if (t >= (long long)P.ctl[0] * NT) return;
  const TileInfo ti = P.tiles[t / NT];
  const int n0 = (int)(t % NT) * LG_COLS;
  const char *a[2], *b[NB];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int lr = min(ti.row0 + i * 16 + r, ti.rows - 1);  // rows past the last one repeat it and are not stored
    long long row = ti.rbase + lr;
    if (GATHER) row = P.row_token ? P.row_token[row] : (lr < ti.fill ? P.slot_token[(size_t)ti.expert * P.C + lr] : P.ir_token[ti.ir_offset + lr - ti.fill]);
    a[i] = static_cast<const char *>(P.A) + (size_t)row * K * ES;
  }
#pragma unroll
  for (int m = 0; m < NB; ++m)
    b[m] = static_cast<const char *>(m ? P.B1 : P.B0) + ((size_t)ti.expert * N + min(n0 + r, N - 1)) * K * ES;
  f32x4 acc[2][NB];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int m = 0; m < NB; ++m) acc[i][m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  auto fetch = [&](long long k, Frag (&fa)[2], Frag (&fb)[NB]) {
    const bool in = k + q * PE < K;  // K % 8 == 0: a lane's piece is inside or outside as a whole
    const size_t off = (size_t)(in ? k + q * PE : 0) * ES;
    const Frag zero = {};
#pragma unroll
    for (int i = 0; i < 2; ++i) fa[i] = in ? *reinterpret_cast<const Frag *>(a[i] + off) : zero;
#pragma unroll
    for (int m = 0; m < NB; ++m) fb[m] = in ? *reinterpret_cast<const Frag *>(b[m] + off) : zero;
  };
  Frag fa[2], fb[NB], na[2], nb[NB];
  const long long step = (long long)LG_NW * KM;
  fetch((long long)w * KM, fa, fb);
  for (long long k = (long long)w * KM; k < K; k += step) {
    fetch(k + step, na, nb);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int m = 0; m < NB; ++m) {
        // B fragment first, as in the other kernels: lane owns row (lane & 15), columns 4 * (lane >> 4) .. + 3
        if constexpr (BF16) {
          acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[m], fa[i], acc[i][m], 0, 0, 0);
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[m][u], fa[i][u], acc[i][m], 0, 0, 0);
        }
      }
#pragma unroll
    for (int i = 0; i < 2; ++i) fa[i] = na[i];
#pragma unroll
    for (int m = 0; m < NB; ++m) fb[m] = nb[m];
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int m = 0; m < NB; ++m)
#pragma unroll
      for (int u = 0; u < 4; ++u) red[w][(i * NB + m) * 4 + u][lane] = acc[i][m][u];
  __syncthreads();
  if (tid >= LG_ROWS * LG_COLS) return;
  const int i = w >> 2, u = w & 3;  // wave w < 8 finishes element u of row fragment i
  float c[NB];
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    c[m] = 0.0f;
#pragma unroll
    for (int s = 0; s < LG_NW; ++s) c[m] += red[s][(i * NB + m) * 4 + u][lane];
  }
  if (GATED) c[0] = (BF16 ? silu(c[0]) : c[0] / (1.0f + expf(-c[0]))) * c[NB - 1];
  if (ACT == RR_ACT_GELU) c[0] = gelu_erf(c[0]);
  const int row = ti.row0 + i * 16 + r, col = n0 + 4 * q + u;
  if (row >= ti.rows || col >= N) return;
  const int dest = DIRECT ? P.row_dest[ti.rbase + row] : -1;
  const size_t at = (size_t)(ti.rbase + row) * N + col, to = (size_t)max(dest, 0) * N + col;
  if constexpr (BF16) {
    const uint16_t v = (uint16_t)pack_bf16(c[0], 0.0f);
    static_cast<uint16_t *>(P.Cout)[at] = v;
    if (DIRECT && dest >= 0) static_cast<uint16_t *>(P.Out)[to] = v;
  } else {
    static_cast<float *>(P.Cout)[at] = c[0];
    if (DIRECT && dest >= 0) static_cast<float *>(P.Out)[to] = c[0];
  }
}

template <typename Kern>
hipError_t set_lds(Kern kern, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

int cu_count() {
  static const int n = [] {  // initialised once, thread-safe (C++11 static)
    int dev = 0, cus = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) cus = prop.multiProcessorCount;
    return cus > 0 ? cus : 256;
  }();
  return n;
}

// Whole K chunks, at least three (the rings); a ragged row needs one more, so that its last chunk is requested inside the K loop.
bool persistent_ok(int K) { return K % GB_BK == 0 ? K >= 3 * GB_BK : K > 3 * GB_BK; }

//                         BF16   waves  frags ring waves per SIMD
using TileS128 = TileShape<TILE_SPLIT, 2, 2, 4, 4, 1, 3>;  // fp32, 128 rows x 128 staged weight rows
using TileS64 = TileShape<TILE_SPLIT, 2, 2, 2, 4, 1, 4>;   // fp32, 64 x 128
using TileF64 = TileShape<TILE_F32, 2, 2, 2, 4, 2, 2>;     // fp32, 64 x 128
using TileF32 = TileShape<TILE_F32, 2, 2, 1, 4, 2, 2>;     // fp32, 32 x 128
using TileF32n = TileShape<TILE_F32, 2, 2, 1, 2, 3, 2>;    // fp32, 32 x 64
using TileB256 = TileShape<TILE_BF16, 4, 2, 4, 4, 3, 2>;     // bf16, 256 x 128, 8 waves
using TileB128 = TileShape<TILE_BF16, 2, 4, 4, 2, 4, 2>;     // bf16, 128 x 128, 8 waves
using TileB64 = TileShape<TILE_BF16, 2, 2, 2, 4, 3, 2>;      // bf16, 64 x 128
using TileB32 = TileShape<TILE_BF16, 1, 2, 2, 4, 4, 2>;      // bf16, 32 x 128
using TileB32n = TileShape<TILE_BF16, 1, 2, 2, 2, 5, 2>;     // bf16, 32 x 64

static_assert(TileB32::BM == kMinRowTile && TileB32n::BM == kMinRowTile && TileF32::BM == kMinRowTile && TileF32n::BM == kMinRowTile && LG_ROWS == kMinRowTile);

// Which tiles a GEMM uses: the shape with the least estimated time.  A CU works through ceil(tiles / CUs) tiles of
// (K chunks x time of a chunk + prologue and epilogue); a chunk takes the longer of
//   cost     its MFMAs and LDS traffic, us per chunk with the CU full, and
//   fetch    its weight bytes that come from HBM (row tiles of one expert share them through L2) at kCuFetch: what
//            one CU sustains against HBM, however deep its ring (a 64 x 128 ring of 6 chunks is no faster than one
//            of 3), so weight-bound layers need their bytes spread evenly over the CUs;
// and no launch is faster than its weights at kHbm.  Large tiles move the fewest operand bytes per flop, small ones
// leave no CU idle.  Measured against the estimate, us: 300 tokens Zipf(1.1), 16 experts, down 5632 -> 2048:
// 32 x 128 92, 64 x 128 108 (one expert has more than 64 rows: 272 tiles), 128 x 128 74; fp32, up / down: 64 x 128
// 213 / 238, 32 x 128 188 / 213, 32 x 64 165 / 168; 16 tokens, 8 experts, down 11008 -> 4096: 32 x 128 141, 32 x 64 133;
// 8 experts 4096 x 11008, K = 11008: 1230 rows 256 x 256 256, 256 x 128 178, 64 x 128 255.
// fp32: the split shapes' numbers are a fit to 260 layers timed in every pair of shapes (1e8 to 5e11 flop).  Of 600 others (5e7 to 3e11)
// the plan is 1.2 % off the best pair on average and 8.5 % faster than the three fp32 shapes were; 16 are 2 - 7 % slower than
// those: their rows per expert are not what the estimate expects, or each weight serves a row or two.
enum FfnShape { FFN_P256, FFN_256, FFN_128, FFN_64, FFN_32, FFN_32N, FFN_S128, FFN_S64, FFN_F64, FFN_F32, FFN_F32N, FFN_LONG };
struct ShapeInfo { int bm, brows; float cost, fixed, alone; };  // alone: of a chunk, where the CU has one workgroup (0: cost)
constexpr ShapeInfo kShape[] = {{256, 256, 1.45f, 5.0f}, {256, 128, 1.0f, 3.0f}, {128, 128, 0.62f, 2.0f},
                                {64, 128, 0.5f, 1.0f},   {32, 128, 0.4f, 1.0f},  {32, 64, 0.3f, 0.3f},
                                {128, 128, 1.37f, 1.1f, 2.8f}, {64, 128, 0.74f, 1.0f, 2.2f},  {64, 128, 1.05f, 1.0f},  {32, 128, 0.5f, 0.7f},  {32, 64, 0.26f, 0.5f},
                                {LG_ROWS, LG_COLS, 0.0f, 0.0f}};
constexpr float kCuFetch = 26e3f, kHbm = 5.9e6f;  // bytes per us
// the 256 x 256 kernel: its start, and a chunk of a tile of which a 1 / n share of the rows is there, n = 1 .. PK_MAX_CUT
constexpr float kPersistentStart = 6.0f, kCutCost[] = {1.0f, 0.72f, 0.6f, 0.53f, 0.5f, 0.47f, 0.45f, 0.43f};
static_assert(sizeof(kCutCost) / sizeof(float) == PK_MAX_CUT);
// the activation of a tile whose workgroup has the CU to itself (256 x 256: in `fixed`; smaller ones overlap theirs)
constexpr float kAct256 = 4.0f, kAct128 = 3.0f;

// Row tiles of height bm that the layer's rows are expected to make.
long long expected_row_tiles(const Dims &D, int bm) {
  // dispatched rows: the top-k assignments (a dropped token's re-routed row stands for its dropped ones)
  const long long want = (long long)D.T * D.k, R = want < D.Rmax ? want : D.Rmax, used = R < D.E ? R : D.E;
  if (used == 1) return (R + bm - 1) / bm;  // all rows are one expert's
  // a popular expert: its capacity and three times an even share of re-routed tokens; one expert in eight is one
  const long long popular = std::min((long long)D.T, D.C + (D.ir ? 3ll * D.T / D.E : 0)), n_popular = (used + 7) / 8;
  return 4 * R <= 3ll * bm * used ? used + n_popular * ((popular - 1) / bm) : R / bm + used / 2;
}

// Estimated time of a GEMM with tiles of shape q, us; < 0: not possible.  by_rows: 256 x 256 tiles of which only a share of
// the rows is there are priced like the parts of a cut tile (their K loop leaves the missing fragments out).
float shape_cost(const Dims &D, int K, int N, bool up, int q, bool by_rows = false) {
  constexpr int kCUs = 256;  // of the part: a host function, which cannot ask a device (the launch does, see cu_count)
  const bool bf16 = D.dtype == RR_BF16, gated = up && D.act == RR_ACT_SWIGLU;
  const ShapeInfo &s = kShape[q];
  if (q == FFN_P256 && !persistent_ok(K)) return -1.0f;
  const bool split = q == FFN_S128 || q == FFN_S64;
  const int es = bf16 ? 2 : 4, KT = (int)(((long long)K * es + GB_ROW_BYTES - 1) / GB_ROW_BYTES);
  // a tile's rows are addressed with 32-bit byte offsets (below kLongRow elements the narrowest shape always fits)
  if ((long long)K * std::max(s.bm, s.brows) * es >= 1ll << 31) return -1.0f;
  // fp32 rows of up to four chunks: fp32 MFMAs (a tile is mostly its start and end); longer ones: split operands or 32 x 64.  Past 2^20 split
  // tiles, passes of a tenth of a second, nothing was timed: fp32 MFMAs in any of their shapes, as for short rows.
  constexpr int kSplitChunks = 5;
  constexpr long long kSplitTiles = 1ll << 20;
  auto tiles_of = [&](int bm, int brows) { return expected_row_tiles(D, bm) * ((N + (gated ? brows / 2 : brows) - 1) / (gated ? brows / 2 : brows)); };
  const bool can_split = KT >= kSplitChunks && tiles_of(kShape[FFN_S128].bm, kShape[FFN_S128].brows) <= kSplitTiles;
  if (split && (!can_split || tiles_of(s.bm, s.brows) > kSplitTiles)) return -1.0f;
  if ((q == FFN_F64 || q == FFN_F32) && can_split) return -1.0f;
  const float used = (float)std::min<long long>({(long long)D.T * D.k, D.Rmax, D.E});
  const float stream = used * N * K * es * (gated ? 2 : 1) / kHbm;
  const int bn = gated ? s.brows / 2 : s.brows;
  const long long mt = expected_row_tiles(D, s.bm), tiles = mt * ((N + bn - 1) / bn), rounds = tiles / kCUs, left = tiles - rounds * kCUs;
  const float fetch = (float)(s.brows * GB_ROW_BYTES) / kCuFetch * used / (float)mt;
  const float filled = std::min(1.0f, (float)std::min<long long>((long long)D.T * D.k, D.Rmax) / (float)(mt * s.bm));
  const float fixed = s.fixed + filled * (up && q == FFN_256 ? kAct256 : (up && q == FFN_128 ? kAct128 : 0.0f));
  auto part_cost = [&](long long n) { return s.cost * kCutCost[std::min<long long>(n, PK_MAX_CUT) - 1]; };
  const float cost = by_rows ? part_cost((long long)(1.0f / filled)) : s.cost, chunk = std::max(cost, fetch);
  float busy = (float)rounds * (KT * chunk + fixed);
  if (split) {  // three or four workgroups per CU: their number evens out half of the last round
    const float all = (float)tiles / kCUs;
    busy = std::max((0.56f * all + 0.44f * ceilf(all)) * (KT * chunk + fixed), KT * s.alone + fixed);
  } else if (q == FFN_P256) {
    busy += kPersistentStart;
    if (left > 0) busy += KT * std::max(std::min(cost, part_cost(kCUs / left)), fetch) + fixed;
  } else if (left > 0) {  // several workgroups per CU: a round that is nearly empty runs partly under the one before
    busy += (KT * chunk + fixed) * (rounds ? std::min(1.0f, (float)left / kCUs + 0.5f) : 1.0f);
  }
  return std::max(busy, stream) + 0.1f * busy;
}

struct FfnPlan { FfnShape up, down; };
// The pair of shapes with the least cost.  Both GEMMs walk one table of row tiles, as high as the higher of the two: a
// lower shape cuts every row tile of the table (GemmArgs::sub) and launches a workgroup for the cuts that turn out
// to be empty too, about 30 ns each (300 tokens, up 2048 -> 5632: 32-row tiles in a table of 128 rows 269 us, 140 alone).
FfnPlan ffn_plan(const Dims &D) {
  if (std::max(D.d, D.F) >= kLongRow) return {FFN_LONG, FFN_LONG};
  constexpr float kEmpty = 0.031f;
  const int q0 = D.dtype == RR_BF16 ? FFN_P256 : FFN_S128, q1 = D.dtype == RR_BF16 ? FFN_32N : FFN_F32N;
  auto empty = [&](int q, int N, bool gated, int bm) {
    const ShapeInfo &s = kShape[q];
    const int bn = gated ? s.brows / 2 : s.brows;
    const long long cuts = expected_row_tiles(D, bm) * (bm / s.bm) - expected_row_tiles(D, s.bm);
    return kEmpty * (float)(std::max(0ll, cuts) * ((N + bn - 1) / bn));
  };
  // One GEMM in split tiles and the other, though it could be too, in 32 x 64 fp32 ones: only if well ahead.  256 tokens, 6 experts of
  // 77 - 123 rows, 1600 x 5696: 373 us, 329 in 32 x 64 tiles alone; 656 tokens, 12 experts, 1808 x 6632: 671, 642.  Of the 600 layers 23
  // are more than 2 % slower than in fp32 shapes without the margin (up to 12 %), 16 with it, and the mean of all gains 0.2 %.
  constexpr float kMixed = 1.1f;
  auto split = [](int q) { return q == FFN_S128 || q == FFN_S64; };
  FfnPlan best{(FfnShape)q1, (FfnShape)q1};
  float least = -1.0f, up[FFN_F32N + 1], down[FFN_F32N + 1];
  for (int q = q0; q <= q1; ++q) {
    up[q] = shape_cost(D, D.d, D.F, true, q);
    down[q] = shape_cost(D, D.F, D.d, false, q);
  }
  const bool both = D.dtype != RR_BF16 && up[FFN_S64] >= 0.0f && down[FFN_S64] >= 0.0f;
  for (int u = q0; u <= q1; ++u)
    for (int w = q0; w <= q1; ++w) {
      if (!(up[u] >= 0.0f) || !(down[w] >= 0.0f)) continue;
      const int bm = std::max(kShape[u].bm, kShape[w].bm);
      const float sure = both && split(u) != split(w) ? kMixed : 1.0f;
      const float cost = sure * (up[u] + down[w]) + empty(u, D.F, D.act == RR_ACT_SWIGLU, bm) + empty(w, D.d, false, bm);
      if (least < 0.0f || cost <= least) { least = cost; best = {(FfnShape)u, (FfnShape)w}; }
    }
  // Layers that their weights bound - more than the last-level cache holds, and some dozen to a tile's height of rows
  // for each expert: the estimate of lower tiles is at its weakest here, as an expert whose rows need one tile more
  // than expected reads its weights again (it knows no row counts).  One tile per expert, though mostly padding, does not care.
  // 1024 tokens, 32 experts, quotas, 3904 x 11840 SwiGLU: 1715 us in 32 x 128 tiles, 1486 in 256 x 256 ones; 896 tokens, 24
  // experts, 2112 x 6016: 462, 402.  Of 1300 layers timed in every pair of shapes 74 were more than 2 % slower than
  // in 256 x 256 tiles (30 more than 8 %), 47 and 13 with this rule; 5 lose by it, at most 9 %.
  constexpr float kSure = 0.85f;
  constexpr long long kLastLevelBytes = 256ll << 20;
  const long long R = std::min<long long>((long long)D.T * D.k, D.Rmax), used = std::min<long long>(R, D.E);
  if (D.dtype == RR_BF16 && up[FFN_P256] >= 0.0f && down[FFN_P256] >= 0.0f && R >= 24 * used && R <= 256 * used &&
      used * D.d * D.F * 2 >= kLastLevelBytes &&
      kSure * (shape_cost(D, D.d, D.F, true, FFN_P256, true) + shape_cost(D, D.F, D.d, false, FFN_P256, true)) < up[best.up] + down[best.down])
    best = {FFN_P256, FFN_P256};
  return best;
}

template <class S>
struct Tag { using type = S; };

template <class F>
void for_each_tile_kernel(F f) {
  auto shape = [&](auto tag) {
    using S = typename decltype(tag)::type;
    if constexpr (S::BF16) {
      f(gemm_tile_kernel<S, true, RR_ACT_SWIGLU, true, false>, S::SMEM);
      f(gemm_tile_kernel<S, true, RR_ACT_SWIGLU, false, false>, S::SMEM);
    }
    f(gemm_tile_kernel<S, true, -1, true, false>, S::SMEM);
    f(gemm_tile_kernel<S, true, -1, false, false>, S::SMEM);
    f(gemm_tile_kernel<S, false, RR_ACT_GELU, true, false>, S::SMEM);
    f(gemm_tile_kernel<S, false, RR_ACT_GELU, false, false>, S::SMEM);
    f(gemm_tile_kernel<S, false, -1, false, true>, S::SMEM);
  };
  shape(Tag<TileS128>{});
  shape(Tag<TileS64>{});
  shape(Tag<TileF64>{});
  shape(Tag<TileF32>{});
  shape(Tag<TileF32n>{});
  shape(Tag<TileB256>{});
  shape(Tag<TileB128>{});
  shape(Tag<TileB64>{});
  shape(Tag<TileB32>{});
  shape(Tag<TileB32n>{});
}

// bf16 SwiGLU layers whose activation is computed with a division, not the hardware's reciprocal
bool swiglu_divides(int K) { return K % GB_BK != 0 || K < 3 * GB_BK; }

// Grid of the small-tile kernel for `tiles` tiles: a grid dimension holds fewer than 2^32 threads (a layer of 2^20 fp32 tokens,
// d_ff 32768, in 32 x 64 outputs has 2^24 tiles of 256 threads), so more tiles make rows of whole XCD runs.
dim3 tile_grid(long long tiles) {
  constexpr long long kRow = 1ll << 20;
  return dim3((unsigned)((std::min(tiles, kRow) + 7) / 8 * 8), (unsigned)((tiles + kRow - 1) / kRow));
}
int column_tiles(const ShapeInfo &s, int N, bool gated) {
  const int bn = gated ? s.brows / 2 : s.brows;
  return (int)(((long long)N + bn - 1) / bn);
}

// One GEMM (UP or down) with tiles of shape S; grid: the most tiles there can be.
template <class S, bool UP>
void launch_tiles(const Dims &D, GemmArgs g, bool fuse, hipStream_t s) {
  const bool gated = UP && D.act == RR_ACT_SWIGLU;
  g.NT = column_tiles(ShapeInfo{S::BM, S::BROWS, 0.0f, 0.0f}, g.N, gated);
  g.sub = D.BM / S::BM;
  const dim3 grid = tile_grid((long long)g.NT * D.max_mtiles * g.sub);
  if constexpr (UP && S::BF16) {
    if (gated && swiglu_divides(g.K)) {
      if (fuse) gemm_tile_kernel<S, true, RR_ACT_SWIGLU, true, false><<<grid, S::THREADS, S::SMEM, s>>>(g);
      else gemm_tile_kernel<S, true, RR_ACT_SWIGLU, false, false><<<grid, S::THREADS, S::SMEM, s>>>(g);
      return;
    }
  }
  if constexpr (UP) {
    if (gated && fuse) gemm_tile_kernel<S, true, -1, true, false><<<grid, S::THREADS, S::SMEM, s>>>(g);
    else if (gated) gemm_tile_kernel<S, true, -1, false, false><<<grid, S::THREADS, S::SMEM, s>>>(g);
    else if (fuse) gemm_tile_kernel<S, false, RR_ACT_GELU, true, false><<<grid, S::THREADS, S::SMEM, s>>>(g);
    else gemm_tile_kernel<S, false, RR_ACT_GELU, false, false><<<grid, S::THREADS, S::SMEM, s>>>(g);
  } else {
    gemm_tile_kernel<S, false, -1, false, true><<<grid, S::THREADS, S::SMEM, s>>>(g);
  }
}

template <bool BF16, bool UP>
void launch_long(const Dims &D, GemmArgs g, bool fuse, hipStream_t s) {
  g.NT = (int)(((long long)g.N + LG_COLS - 1) / LG_COLS);
  const dim3 grid = tile_grid((long long)g.NT * D.max_mtiles);
  if constexpr (UP) {
    const bool gated = D.act == RR_ACT_SWIGLU;
    if (gated && fuse) gemm_long_kernel<BF16, true, -1, true, false><<<grid, LG_THREADS, 0, s>>>(g);
    else if (gated) gemm_long_kernel<BF16, true, -1, false, false><<<grid, LG_THREADS, 0, s>>>(g);
    else if (fuse) gemm_long_kernel<BF16, false, RR_ACT_GELU, true, false><<<grid, LG_THREADS, 0, s>>>(g);
    else gemm_long_kernel<BF16, false, RR_ACT_GELU, false, false><<<grid, LG_THREADS, 0, s>>>(g);
  } else {
    gemm_long_kernel<BF16, false, -1, false, true><<<grid, LG_THREADS, 0, s>>>(g);
  }
}

template <bool UP>
void launch_gemm(FfnShape shape, const Dims &D, GemmArgs g, bool fuse, hipStream_t s) {
  switch (shape) {
    case FFN_P256: {
      const bool gated = UP && D.act == RR_ACT_SWIGLU;
      g.NT = gated ? (g.N + 127) / 128 : (g.N + 255) / 256;
      const int cus = cu_count();
      if constexpr (UP) {
        const bool ragged = swiglu_divides(g.K);  // (ACT RR_ACT_SWIGLU: with the division)
        if (gated && fuse && ragged) gemm_bf16_persistent_kernel<true, RR_ACT_SWIGLU, true><<<cus, PK_THREADS, PK_SMEM, s>>>(g);
        else if (gated && ragged) gemm_bf16_persistent_kernel<true, RR_ACT_SWIGLU, false><<<cus, PK_THREADS, PK_SMEM, s>>>(g);
        else if (gated && fuse) gemm_bf16_persistent_kernel<true, -1, true><<<cus, PK_THREADS, PK_SMEM, s>>>(g);
        else if (gated) gemm_bf16_persistent_kernel<true, -1, false><<<cus, PK_THREADS, PK_SMEM, s>>>(g);
        else if (fuse) gemm_bf16_persistent_kernel<false, RR_ACT_GELU, true><<<cus, PK_THREADS, PK_SMEM, s>>>(g);
        else gemm_bf16_persistent_kernel<false, RR_ACT_GELU, false><<<cus, PK_THREADS, PK_SMEM, s>>>(g);
      } else {
        gemm_bf16_persistent_kernel<false, -1, false, true><<<cus, PK_THREADS, PK_SMEM, s>>>(g);
      }
      break;
    }
    case FFN_256: launch_tiles<TileB256, UP>(D, g, fuse, s); break;
    case FFN_128: launch_tiles<TileB128, UP>(D, g, fuse, s); break;
    case FFN_64: launch_tiles<TileB64, UP>(D, g, fuse, s); break;
    case FFN_32: launch_tiles<TileB32, UP>(D, g, fuse, s); break;
    case FFN_32N: launch_tiles<TileB32n, UP>(D, g, fuse, s); break;
    case FFN_S128: launch_tiles<TileS128, UP>(D, g, fuse, s); break;
    case FFN_S64: launch_tiles<TileS64, UP>(D, g, fuse, s); break;
    case FFN_F64: launch_tiles<TileF64, UP>(D, g, fuse, s); break;
    case FFN_F32: launch_tiles<TileF32, UP>(D, g, fuse, s); break;
    case FFN_F32N: launch_tiles<TileF32n, UP>(D, g, fuse, s); break;
    case FFN_LONG:
      if (D.dtype == RR_BF16) launch_long<true, UP>(D, g, fuse, s);
      else launch_long<false, UP>(D, g, fuse, s);
      break;
  }
}

}  // namespace

// The GEMM kernels use more dynamic LDS than the default limit.  Raising it is host-side set-up of the
// loaded code object on the current device (no stream work); the caller runs it once per device.
hipError_t ffn_kernel_attributes() {
  hipError_t e = hipSuccess;
  auto set = [&e](auto kern, int bytes) {
    if (e == hipSuccess) e = set_lds(kern, bytes);
  };
  set(gemm_bf16_persistent_kernel<true, RR_ACT_SWIGLU, true>, PK_SMEM);
  set(gemm_bf16_persistent_kernel<true, RR_ACT_SWIGLU, false>, PK_SMEM);
  set(gemm_bf16_persistent_kernel<true, -1, true>, PK_SMEM);
  set(gemm_bf16_persistent_kernel<true, -1, false>, PK_SMEM);
  set(gemm_bf16_persistent_kernel<false, RR_ACT_GELU, true>, PK_SMEM);
  set(gemm_bf16_persistent_kernel<false, RR_ACT_GELU, false>, PK_SMEM);
  set(gemm_bf16_persistent_kernel<false, -1, false, true>, PK_SMEM);
  for_each_tile_kernel(set);
  return e;
}

// Row-tile height of the layer's tile table: the higher of the two GEMMs' tiles.
int ffn_row_tile(const Dims &D) {
  const FfnPlan plan = ffn_plan(D);
  return std::max(kShape[plan.up].bm, kShape[plan.down].bm);
}

void ffn_describe(const Dims &D, FfnShapes *out) {
  const FfnPlan plan = ffn_plan(D);
  const FfnShape q[2] = {plan.up, plan.down};
  for (int i = 0; i < 2; ++i) {
    out->bm[i] = kShape[q[i]].bm;
    out->brows[i] = kShape[q[i]].brows;
    out->cost[i] = shape_cost(D, i ? D.F : D.d, i ? D.d : D.F, i == 0, q[i]);
  }
}

bool ffn_fuses_gather(const Dims &D) { return (long long)D.T * D.d * (D.dtype == RR_BF16 ? 2 : 4) < 0x7ffffff0ll; }

hipError_t launch_ffn(const Dims &D, const void *x, const rr_tables &tb, const void *w1, const void *w3,
                      const void *w2, const Work &W, void *out, hipStream_t s) {
  const bool fuse = ffn_fuses_gather(D);
  const FfnPlan plan = ffn_plan(D);
  const GemmArgs up{fuse ? x : W.x_disp, w1, w3, W.h, D.d, D.F, 0, 1, W.tiles, W.tile_ctl,
                    tb.slot_token, tb.ir_token, D.quota ? W.row_token : nullptr, D.C,
                    (long long)D.T * D.d * (D.dtype == RR_BF16 ? 2 : 4), nullptr, nullptr};
  const GemmArgs down{W.h, w2, nullptr, W.y, D.F, D.d, 0, 1, W.tiles, W.tile_ctl, nullptr, nullptr, nullptr, 0, 0, W.row_dest, out};
  prof_begin(K_FFN_UP, s);
  launch_gemm<true>(plan.up, D, up, fuse, s);
  prof_end(K_FFN_UP, s);
  prof_begin(K_FFN_DOWN, s);
  launch_gemm<false>(plan.down, D, down, fuse, s);
  prof_end(K_FFN_DOWN, s);
  return hipGetLastError();
}

}  // namespace rr

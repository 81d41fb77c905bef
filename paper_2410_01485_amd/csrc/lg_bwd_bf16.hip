// lg_bwd_bf16.hip — bf16 backward on the gfx950 matrix cores (paper Section 3.2: the
// backward step skips masked key blocks just like the forward; Table 1 counts both).
//
// Two kernels (the first one also forms Delta), or one for both where neither fills the GPU (bwd_both_bf16_kernel; the
// set-up kernel then forms Delta).  Sink + window without GQA uses no atomics and is
// bit-reproducible; strided patterns and GQA add float32 partial dk/dv sums of the column keys
// with atomics (see the dk/dv section).  Tiles travel global -> LDS directly (row-major,
// swizzled; lg_swz.h) and are read both with the contraction over dims (row reads) and with the
// contraction over tile rows (transposing LDS reads), so no tile is ever stored twice.
//
//  dq kernel (query-tile major, same tile walk as the forward; 4 waves x 32 query rows).  Per live key tile:
//     S^T  = K Q^T,  dP^T = V dO^T      (keys x queries; A = K / V rows from LDS,
//                                        B = Q / dO fragments kept in registers)
//     P^T  = exp2(S^T c - lse_i c'),  dS^T = P^T o (dP^T - Delta_i)   (one query per lane)
//     dQ^T += K^T dS^T                  (dims x queries; A = K through transposing reads,
//                                        B = dS^T straight from the accumulator registers)
//  dk/dv kernel (key-tile major; a wave for every 32 keys: 256 keys per workgroup for D = 128, 128 for D = 64; the K
//  fragment of a wave stays in registers, the V rows of the workgroup stay in LDS).  Per live query
//  tile of 64 rows, for every query head of the kv group:
//     S  = Q K^T,  dP = dO V^T          (queries x keys; A = Q / dO rows from LDS)
//     P, dS as above                    (one key per lane; S and dP start from the per-row
//                                        values -lse / scale and -Delta as their addend)
//     dV^T += dO^T P,  dK^T += Q^T dS   (dims x keys; A = dO / Q through transposing reads,
//                                        B = P / dS straight from the accumulators)
// 7 tile products instead of the minimal 5: S and dP are computed in both kernels.
//
// What bounds these two: a wave's matrix and vector work follow each other, so a SIMD needs waves in different phases.
// Workgroups are therefore as small as LDS and registers make several of them fit a CU (dq: 2 for D = 128, 3 for
// D = 64; dk/dv: 1 and 3), each with its own barriers, and operands from LDS are requested a few matrix instructions
// ahead.  Against one workgroup of 8 waves with a deeper ring and the compiler's order: dq, 32 heads of 128, 32768
// tokens, window 512: 805 -> 644 us; 64/8 heads, 9830 tokens, window 455: 489 -> 367 us; dk/dv, 32 heads of 64, 32768
// tokens, window 4096: 2441 -> 2104 us, window 512: 610 -> 475 us.
//
// What a workgroup reads and writes once (Q, dO, out, K; dq, dk, dv) goes through LDS in pieces of 1 KB: loaded or stored
// by each lane from or to its own row, an instruction touches 32 rows, and these instructions took as long as several
// tiles, with one workgroup per CU with nothing beside them.  32 heads of 128, 32768 tokens: window 64 dq 374 -> 328, dk/dv
// 461 -> 390 us; 512 590 -> 570, 830 -> 782; 2048 (64 rows per wave) 1545 -> 1493, 1910 -> 1875; 64 x 512 tokens 465 -> 380,
// 630 -> 495 (some of that from the order of the tiles, lg_order).
//
// For head dim 128 and long windows (dq 32 or more tiles, and 384 or more of 256 rows; dk/dv 16, in a launch of its own)
// both kernels have a second form with 64 rows (keys) per wave, one wave per SIMD and the accumulators in AGPRs (further
// down): every operand read from LDS then feeds two matrix instructions.
#include <algorithm>

#include "../../include/longgen_attn.h"
#include "lg_kernels.h"
#include "lg_mfma.h"
#include "lg_swz.h"
#include "lg_wide.h"

namespace {

// Keys of a dk/dv workgroup.
constexpr int btk_of(int D) { return D == 128 ? LG_BF16_BTK : LG_BF16_BTK64; }

constexpr float LOG2E = 1.44269504088896340736f;

// TOKEN (the 64-rows-per-wave kernels): the pattern is token-granular without strided columns (block <= 1, stride 0).  The
// mask fields that are then known let the compiler drop the block / stride arithmetic from the per-tile scheduling.
//
// Masks.  A lane's live pairs of a PARTIAL tile are runs: in dq a few of its 32 registers (lg_key_bits), in dk/dv one run of
// rows from its key on.  They are applied behind a real branch: as selects, which the compiler makes of a short condition
// on `full`, they cost every whole tile (dq, 32 heads of 128, window 512: 574 -> 517 us; head dim 64, window 1024: 503 ->
// 471).  A wave's class of a tile comes from bounds that it works out once (LgRows, LgKeys), and of the two blocks of 32
// that a PARTIAL tile has a dead one is left out (dk/dv 64 x 512 tokens 482 -> 460 us, with 64/8 heads of 64 and strided
// columns 1400 -> 1146).  With that, instances for token-granular patterns bring the 32-rows kernels nothing.

// Sequences of different lengths side by side in each head, in one set of launches, longest first: those that take
// the 64-rows-per-wave kernels are then the first ones, and long work items start first.  Lives in the workspace;
// bwd_setup_kernel writes it.
struct LgBwdSeqs {
  int n;
  int row0[LG_PACK_MAX];          // first row inside a head of the caller's tensors
  int wrow0[LG_PACK_MAX];         // ... and of the workspace's per-row arrays
  int len[LG_PACK_MAX];
  int ncol[LG_PACK_MAX];          // column groups split off (0: none)
  int nlone[LG_PACK_MAX];         // exactly one group: chunks of its column part (0 otherwise)
  int qtile0[LG_PACK_MAX + 1];    // query tiles (LG_BF16_TQ rows) of the sequences before
  int ktile0[LG_PACK_MAX + 1];    // key tiles (of a dk/dv workgroup)
  int grp0[LG_PACK_MAX + 1];      // 64-key groups: offset into col_of_group
  int col0[LG_PACK_MAX + 1];      // split-off column groups: offset into col_list and the partial sums
  int citem0[LG_PACK_MAX + 1];    // column work items (virtual tile x chunk), sequences with several groups
  int litem0[LG_PACK_MAX + 1];    // column work items (chunk), sequences with one group
};

// What tells a kernel which sequence and tile a work item is, and where partial sums are.
struct LgBwdWork {
  const LgBwdSeqs* seqs;  // nullptr: a batch of sequences of one length
  const int* items;       // packed dk/dv: (sequence << 24 | key tile)
  int B;
  int wld;                // rows from one head to the next in the workspace's per-row arrays
  int qt_first;           // packed dq: the launch's first query tile
  // column parts (see the dk/dv section)
  const int* col_of_group;
  const int* col_list;
  int ncol;               // split-off column groups of a head, of all packed sequences together
  int nlone;              // batch: chunks of a lone group's column part
  int chunk;              // query tiles per column work item where there are several groups
  float* colpart;         // [b x kv head][ncol] sums, one group slot each
  float* lonepart;        // Hq == Hkv: [b x kv head][lone chunks of all sequences] group slots
  int nlone_all;          // lone chunks of all sequences
  unsigned* arrived;      // Hq == Hkv: [b x kv head][sequence] chunks of a lone group that are done
  bool lone_joint;        // Hq == Hkv: beside dq and dk/dv: its key tile's window part counts as a chunk and waits in colpart
  int order;              // lg_order
  bool by_tile;           // dk/dv items: heads innermost (always for packed sequences and cut window parts)
  // window parts cut into `heads_cut` sets of query heads times `rows_cut` runs of query tiles
  int heads_cut, rows_cut;
  float* parts;           // [key tile][b x kv head][part] a group slot for each 64 keys
};

// Partial sums are kept the way the accumulators hold them, 64 keys ("group slot") at a time: [32-key block][dk, dv]
// [32-dim block][register][lane] floats, so that every store, load or atomic of a wave covers 256 consecutive bytes.
template <int D>
struct LgSlot {
  static constexpr int DB = D / 32;
  static constexpr int FLOATS = 64 * D * 2;
  __device__ __forceinline__ static int at(int kb, int which, int db) { return ((kb * 2 + which) * DB + db) * 1024; }
};

// The sequence that owns position t, given the n non-decreasing starts: the last one that starts at or before t.
// Called by whole waves; the answer is wave-uniform.
__device__ __forceinline__ int lg_uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int lg_seq_of(const int* __restrict__ start, int n, int t) {
  const int lane = threadIdx.x & 63;
  int c = 0;
#pragma unroll
  for (int x = 0; x < LG_PACK_MAX; x += 64)
    c += __popcll(__builtin_amdgcn_ballot_w64(x + lane < n && start[min(x + lane, n)] <= t));
  return lg_uniform(c - 1);
}

// sum over 8 bf16 pairs of x * y, added to s
__device__ __forceinline__ float lg_dot8(uint4 x, uint4 y, float s) {
  const unsigned xw[4] = {x.x, x.y, x.z, x.w}, yw[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    s = fmaf(__uint_as_float(xw[t] << 16), __uint_as_float(yw[t] << 16), s);
    s = fmaf(__uint_as_float(xw[t] & 0xffff0000u), __uint_as_float(yw[t] & 0xffff0000u), s);
  }
  return s;
}

// Sum over the aligned group of N lanes (8 or 16) that a lane is in.
template <int N>
__device__ __forceinline__ float lg_group_sum(float x) {
  auto add = [&](auto ctrl) {
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), decltype(ctrl)::value, 0xf, 0xf, false));
  };
  add(std::integral_constant<int, 0xB1>{});   // lane ^ 1
  add(std::integral_constant<int, 0x4E>{});   // lane ^ 2
  add(std::integral_constant<int, 0x141>{});  // 7 - lane, inside the group of 8
  if (N == 16) add(std::integral_constant<int, 0x140>{});  // 15 - lane
  return x;
}

// Delta = <dout, out> and the log-sum-exp of the ROWS rows from q0 on to LDS, by a workgroup of 256: dout from its tiles in
// LDS, out in pieces of 16 bytes, consecutive lanes consecutive pieces.  Rows past the end repeat the last one.
// Eight rows' products side by side and one store at the end: row after row, with a branch each, they waited for LDS and for
// each sum's steps (with the 64-rows-per-wave form's fragments read one by one as well 8000 cycles of an item's start, now
// 4900; 32 heads of 128: 32768 tokens, window 256 370 -> 363 us, 51 x 640 tokens 387 -> 383, 32 x 1024 497 -> 487).
template <int D, int ROWS>
__device__ __forceinline__ void lg_delta_rows(const unsigned char* tiles, const uint4 (&o)[ROWS * D / 2048], float* s_delta) {
  using T = LgSwzTile<D>;
  constexpr int P = ROWS * D / 2048, RPP = 256 / T::CPR, AT = P < 8 ? P : 8;  // pieces, rows of one; pieces side by side
  static_assert(P <= T::CPR, "a lane keeps one row");
  const int tid = threadIdx.x, c = tid % T::CPR;
  float mine = 0.f;
#pragma unroll
  for (int x0 = 0; x0 < P; x0 += AT) {
    uint4 gw[AT];
#pragma unroll
    for (int x = 0; x < AT; ++x) {
      const int r = (x0 + x) * RPP + tid / T::CPR;
      gw[x] = *reinterpret_cast<const uint4*>(tiles + r * T::ROW_BYTES + ((c ^ T::pi(r & 63)) << 4));
    }
#pragma unroll
    for (int x = 0; x < AT; ++x) {
      const float s = lg_group_sum<T::CPR>(lg_dot8(gw[x], o[x0 + x], 0.f));
      mine = c == x0 + x ? s : mine;
    }
  }
  if (c < P) s_delta[c * RPP + tid / T::CPR] = mine;
}
template <int D, int ROWS>
__device__ __forceinline__ void lg_load_pieces(const uint16_t* __restrict__ rows, int last, uint4 (&o)[ROWS * D / 2048]) {
  using T = LgSwzTile<D>;
  const int tid = threadIdx.x;
#pragma unroll
  for (int x = 0; x < ROWS * D / 2048; ++x)
    o[x] = *reinterpret_cast<const uint4*>(rows + (size_t)min(x * (256 / T::CPR) + tid / T::CPR, last) * D + tid % T::CPR * 8);
}

// In launches of their own both dq kernels also form Delta_i = <dout_i, out_i> of their rows (lg_delta_rows, from the dout
// that they bring to LDS anyway) and leave -Delta and -lse / scale in the workspace for the dk/dv kernels, which run after them on
// the same stream.  Where they share a launch with dk/dv, the set-up kernel leaves both there before.
// ------------------------------------------------------------------------- dq
// Waves per SIMD and operands requested ahead, as the registers of so many waves allow (256 for D = 128, 168 for D = 64).
template <int D>
struct LgDqTune {
  static constexpr int WAVES = D == 128 ? 2 : 3, AHEAD = D == 128 ? 3 : 2;
};
// A work item, 128 rows.  FORM: forms Delta; otherwise the set-up kernel has (launches that dq shares with dk/dv).  PAIR: of the
// eight waves four have half 0 of a 256-row tile and four half 1, with LDS of their own and the same barriers.
template <int D>
constexpr int DQ_LDS = 4 * LgSwzTile<D>::BYTES;
template <int D, bool FORM, bool PAIR>
__device__ __forceinline__ void dq_bf16_item(
    unsigned char* smem, float (*s_rows)[LG_BF16_TQ32], const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    const uint16_t* __restrict__ v, const uint16_t* __restrict__ out, const uint16_t* __restrict__ dout,
    const float* __restrict__ lse, float* __restrict__ ndelta, float* __restrict__ nlse, uint16_t* __restrict__ dq, int Hq, int Hkv,
    float scale, LgMask m, const LgBwdWork& wk, int b, int hk, int hq, int qt, int half, int x) {
  using T = LgSwzTile<D>;
  constexpr int NT = 256;
  using Dma = LgDma<D, NT>;
  constexpr int TQ = LG_BF16_TQ32, TK = LG_BF16_TK;
  static_assert(LG_BF16_TQ == 2 * TQ && TK == 64, "4 waves x 32 query rows, 64-key tiles");
  static_assert(!(FORM && PAIR), "a pair finds Delta formed");
  constexpr int DC = D / 16, DB = D / 32;
  constexpr int STAGE = 2 * T::BYTES;  // K tile + V tile
  static_assert(DQ_LDS<D> == 2 * STAGE, "two stages");
  int srow = 0, swrow = 0;  // packed: first row of the sequence inside its head, in the workspace
  if (wk.seqs) {
    const int t = wk.qt_first + x;
    const int sq = lg_seq_of(wk.seqs->qtile0, lg_uniform(wk.seqs->n), t);
    qt = lg_uniform(wk.seqs->qtile0[sq + 1]) - 1 - t;
    srow = lg_uniform(wk.seqs->row0[sq]);
    swrow = lg_uniform(wk.seqs->wrow0[sq]);
    m = lg_mask_for_length(m, lg_uniform(wk.seqs->len[sq]));
  }
  const int N = m.N;
  const int tid = PAIR ? threadIdx.x & 255 : threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, g = lane >> 5;
  const int q0 = (2 * qt + half) * TQ, q1 = min(q0 + TQ - 1, N - 1);
  if (!PAIR && q0 >= N) return;
  const int base = PAIR ? half * DQ_LDS<D> : 0;  // of this item's LDS
  const size_t row0 = (size_t)(b * Hq + hq) * m.ld + srow;       // the sequence's first row in this query head
  const size_t wrow0 = (size_t)(b * Hq + hq) * wk.wld + swrow;   // the same in the workspace
  const size_t qbase = row0 * D;
  const uint16_t* kh = k + ((size_t)(b * Hkv + hk) * m.ld + srow) * D;
  const uint16_t* vh = v + ((size_t)(b * Hkv + hk) * m.ld + srow) * D;
  const int i = q0 + wave * 32 + n;
  const int iq = min(i, N - 1);
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const bool idle = q0 + wave_s * 32 >= N;  // past the end
  const int qw0 = min(q0 + wave_s * 32, N - 1), qw1 = min(q0 + wave_s * 32 + 31, N - 1);  // this wave's rows

  f32x16_t acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;

  Dma dma;
  dma.init(tid);
  LgSwzReader<D> rd;
  rd.init(n, g);
  const uint32_t lds0 = (uint32_t)(uintptr_t)LG_LDS_PTR(unsigned char, smem) + base;
  const LgQSched qs = lg_qsched_init(m, q0, q1);
  const LgRows wrows = lg_rows(m, qw0, qw1);
  auto issue = [&](int t, int stage) {
    const size_t off = (size_t)t * TK * D;
    dma.issue(kh + off, N - t * TK, lds0 + stage * STAGE);
    dma.issue(vh + off, N - t * TK, lds0 + stage * STAGE + T::BYTES);
  };

  // patterns without strided columns walk the window run rotated (L2 sharing between neighbours)
  const LgQWalk qw = lg_qwalk_init(qs);
  auto walk = [&](const LgQSched& qs, const LgQWalk& qw, int prev) -> int {
    if (m.stride == 0) return prev < 0 ? lg_qwalk_first(qw) : lg_qwalk_next(qw, prev);
    return lg_qsched_next(m, qs, prev);
  };
  auto next_tile = [&](int prev) -> int { return walk(qs, qw, prev); };
  // the other half's walk: barriers as long as either has tiles
  const int o0 = (2 * qt + 1 - half) * TQ;
  const LgQSched qs_o = PAIR ? lg_qsched_init(m, min(o0, N - 1), min(o0 + TQ - 1, N - 1)) : qs;
  const LgQWalk qw_o = PAIR ? lg_qwalk_init(qs_o) : qw;
  // Q and dO rows through the two stages' places into registers, out and the log-sum-exp once per row
#pragma unroll
  for (int y = 0; y < 2; ++y)
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int rc = min(q0 + 64 * x, N - 1);  // a tile wholly past the end repeats the last row
      dma.issue((y ? q : dout) + qbase + (size_t)rc * D, N - rc, lds0 + y * STAGE + x * T::BYTES);
    }
  const int my_row = min(q0 + (tid & (TQ - 1)), N - 1);
  const float my_lse = lse[row0 + (FORM ? my_row : iq)];
  float di = 0.f, lse2 = 0.f;
  if constexpr (!FORM) {
    di = -ndelta[wrow0 + iq];
    lse2 = my_lse * LOG2E;
    LG_WAIT_VMCNT(0);
    __syncthreads();
  } else {
    uint4 o[TQ * D / 2048];
    lg_load_pieces<D, TQ>(out + qbase + (size_t)q0 * D, N - 1 - q0, o);
    LG_WAIT_VMCNT(0);
    __syncthreads();
    lg_delta_rows<D, TQ>(smem, o, s_rows[0]);
    if (tid < TQ) s_rows[1][tid] = my_lse;
  }
  bf16x8_t qf[DC], gf[DC];
#pragma unroll
  for (int dc = 0; dc < DC; ++dc) {
    gf[dc] = rd.read_rows(smem, base + (wave_s >> 1) * T::BYTES, wave_s & 1, dc);
    qf[dc] = rd.read_rows(smem, base + STAGE + (wave_s >> 1) * T::BYTES, wave_s & 1, dc);
  }
  // Touch everything loaded so far, so that the compiler's waits for these loads sit here and
  // not inside the tile loop (where they would drain the direct loads kept in flight).
#pragma unroll
  for (int dc = 0; dc < DC; ++dc) asm volatile("" ::"v"(qf[dc]), "v"(gf[dc]));
  __syncthreads();
  int t = !PAIR || q0 < N ? next_tile(-1) : -1, t_o = PAIR && o0 < N ? walk(qs_o, qw_o, -1) : -1;
  if (!PAIR || t >= 0) issue(t, 0);
  const float sl2 = scale * LOG2E;
  if constexpr (FORM) {
    di = s_rows[0][wave * 32 + n];
    lse2 = s_rows[1][wave * 32 + n] * LOG2E;
    if (tid < TQ && q0 + tid < N) {
      ndelta[wrow0 + q0 + tid] = -s_rows[0][tid];
      nlse[wrow0 + q0 + tid] = -my_lse / scale;
    }
  }
  asm volatile("" : "+v"(lse2), "+v"(di));

  int stage = 0;
  while (t >= 0 || (PAIR && t_o >= 0)) {
    LG_WAIT_VMCNT(0);
    __syncthreads();  // tile t landed for everyone; everyone is done with the one before
    if (PAIR) {
      if (t_o >= 0) t_o = walk(qs_o, qw_o, t_o);
      if (t < 0) continue;
    }
    const int t_next = next_tile(t);
    const int k0 = t * TK;
    // A tile that is not live throughout for the workgroup's 128 rows is classified again for
    // this wave's 32 rows: most waves then find it wholly live or wholly dead (they sit it out).
    int kind = LG_TILE_FULL;
    if (idle) kind = LG_TILE_DEAD;
    else if (!lg_qsched_full(m, qs, t)) kind = lg_rows_kind(m, wrows, k0, k0 + TK - 1);
    const bool full = kind == LG_TILE_FULL;
    // Whole tiles request the next one between matrix instructions instead of before them (32 heads of 128, 16 x 2048
    // tokens, causal 846 -> 826 us, 32 x 1024 499 -> 489, 2 of 24055 tokens, window 4032 160.8 -> 156.6; heads of 64: 482 ->
    // 470, 285 -> 279, 100.7 -> 96.8).
    const bool between = full && t_next >= 0 && N - t_next * TK >= TK;
    if (t_next >= 0 && !between) issue(t_next, stage ^ 1);
    const int sk = base + stage * STAGE, sv = sk + T::BYTES;
    const uint32_t bits = full ? ~0u : lg_key_bits(m, iq, k0, g);  // bit 16 kb + r: the key of register r of block kb is live

    if (kind != LG_TILE_DEAD)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      // (a PARTIAL tile may have a half without live pairs)
      if (!full && __builtin_amdgcn_ballot_w64(((bits >> (16 * kb)) & 0xffffu) != 0) == 0) continue;
      constexpr int AHEAD = LgDqTune<D>::AHEAD;
      f32x16_t sc, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[r] = dp[r] = 0.f;
      LgRing<2 * DC, AHEAD> rows;
      auto read_rows = [&](int u) { return rd.read_rows(smem, u & 1 ? sv : sk, kb, u >> 1); };
      rows.begin(read_rows);
      auto product = [&](int u, bf16x8_t a) {
        if (u & 1) dp = lg_mfma32(a, gf[u >> 1], dp);
        else sc = lg_mfma32(a, qf[u >> 1], sc);
      };
      if (kb == 0 && between) {
        const uint16_t *k1 = kh + (size_t)t_next * TK * D, *v1 = vh + (size_t)t_next * TK * D;
        const uint32_t to = lds0 + (stage ^ 1) * STAGE;
        rows.run(read_rows, [&](int u, bf16x8_t a) {
          product(u, a);
          static_assert(2 * Dma::CH == DC, "a request per two matrix instructions");
          const int x = u >> 1;
          if (u & 1) dma.load(x < Dma::CH ? k1 : v1, to + (x < Dma::CH ? 0 : T::BYTES), x % Dma::CH);
        });
      } else {
        rows.run(read_rows, product);
      }
      LgRing<2 * DB, AHEAD> cols;
      auto read_cols = [&](int u) { return rd.read_cols(smem, sk, u % DB, 2 * kb + u / DB); };
      cols.begin(read_cols);
      float ds[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) ds[r] = __builtin_amdgcn_exp2f(fmaf(sc[r], sl2, -lse2));
      if (!full) {
        asm volatile("; masked" ::: "memory");  // (a real branch: as selects the masks slowed whole tiles)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (!((bits >> (kb * 16 + r)) & 1)) ds[r] = 0.f;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) ds[r] *= dp[r] - di;
      const bf16x8_t bop[2] = {lg_pack8(ds), lg_pack8(ds + 8)};
      cols.run(read_cols, [&](int u, bf16x8_t a) { acc[u % DB] = lg_mfma32(a, bop[u / DB], acc[u % DB]); });
    }
    t = t_next;
    stage ^= 1;
  }

  // (everyone is done with the stage before the last tile's)
  unsigned char* rows = smem + base + stage * STAGE + wave_s * (32 * T::ROW_BYTES);
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    float a[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] = acc[db][r];
    lg_rows_put<D>(rows, lane, db, a, scale);
  }
  lg_rows_write<D>(rows, lane, dq + qbase + (size_t)(q0 + wave_s * 32) * D, N - (q0 + wave_s * 32));
}
template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(LgDqTune<D>::WAVES, LgDqTune<D>::WAVES))) void
dq_bf16_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ out, const uint16_t* __restrict__ dout, const float* __restrict__ lse,
    float* __restrict__ ndelta, float* __restrict__ nlse, uint16_t* __restrict__ dq, int Hq, int Hkv, float scale,
    LgMask m, int nqt, int total, LgRuns runs, LgBwdWork wk) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DQ_LDS<D>];
  __shared__ float s_rows[2][LG_BF16_TQ32];  // Delta, log-sum-exp

  const int L = lg_item_of(blockIdx.x, runs);
  if (L < 0 || L >= total) return;
  // logical order: (b, kv head) slowest, then query tile (longest rows first), then the query
  // heads of the GQA group: the G workgroups that walk the same K/V tiles run side by side
  const int G = Hq / Hkv;
  const int gq = L % G, rest = L / G;
  // (nqt, qtile0: in LG_BF16_TQ rows, two workgroups each)
  const int at = lg_order_at(wk.order, rest);
  int bhk = (at >> 1) / nqt, y = at - bhk * 2 * nqt;
  lg_in_order(wk.order, rest, 2 * nqt, &bhk, &y);
  const int half = 1 - (y & 1), x = y >> 1;
  const int b = bhk / Hkv, hk = bhk % Hkv;
  dq_bf16_item<D, true, false>(smem, s_rows, q, k, v, out, dout, lse, ndelta, nlse, dq, Hq, Hkv, scale, m, wk, b, hk, hk * G + gq,
                               nqt - 1 - x, half, x);
}

// ---------------------------------------------------------------------- dk, dv
// Column keys (sink tokens, keys of strided block columns) are seen by every later query.
// The query range of a key tile therefore has a dense window part (like every tile) and, if it
// holds column keys, a long column part: all later rows, but only its column keys live.
// The column parts are split off.  Where there are several column groups of 64 keys (strided patterns), the COLUMN
// instance of the kernel packs them into virtual tiles of the kernel's own size (four groups at head dim 128, two at
// 64), so that all waves have live keys and a Q / dO tile is used by as many keys again, cuts their query range into chunks that run as separate workgroups, and adds
// float32 sums into the workspace with hardware atomics (their order is not fixed, so the last bits of dk/dv of column
// keys can differ from run to run).  A lone group (the sink of a sink + window pattern) has a kernel of its own
// (dkdv_lone_bf16_kernel), without atomics where Hq == Hkv.  The main instance then handles the window part of every
// tile and folds the sums in before it rounds to bf16.  bwd_setup_kernel lists the column groups once per call.
// What the kernels below find in the workspace, written in one launch: the work queues' counters and the partial sums
// of the column parts cleared, the column tables, and for packed sequences their descriptor and the dk/dv work items.
//   col_of_group[c] = index of 64-key group c among the column groups, or -1; col_list = inverse
//   items: the key tiles of the first nwide sequences, then those of the others; within each the tiles farthest from
//          the end of their sequence, which the most query tiles see, come first
struct LgBwdSetup {
  int btk;       // keys of a dk/dv workgroup
  int n, nwide;  // packed sequences, longest first, and how many of them take the 64-keys-per-wave dk/dv kernel; n = 0: batch
  int row0[LG_PACK_MAX], len[LG_PACK_MAX], ncol[LG_PACK_MAX], citems[LG_PACK_MAX], nlone[LG_PACK_MAX];
};
constexpr int SETUP_NT = 512;

// Ranks from a ballot per wave plus the counts of the waves before it.  By a whole workgroup.
__device__ void column_table(int* __restrict__ col_of_group, int* __restrict__ col_list, const LgMask& m, int btk) {
  __shared__ int wcount[SETUP_NT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ngroups = (m.N + 63) / 64;
  int base = 0;
  for (int c0 = 0; c0 < ngroups; c0 += SETUP_NT) {
    const int c = c0 + tid;
    const bool is = c < ngroups && lg_is_column_group(m, c, btk, LG_BF16_BTQ);
    const unsigned long long bal = __ballot(is);
    if (lane == 0) wcount[wave] = __popcll(bal);
    __syncthreads();
    int off = base, all = 0;
    for (int w = 0; w < SETUP_NT / 64; ++w) {
      if (w < wave) off += wcount[w];
      all += wcount[w];
    }
    const int rank = off + __popcll(bal & ((1ull << lane) - 1ull));
    if (c < ngroups) col_of_group[c] = is ? rank : -1;
    if (is) col_list[rank] = c;
    base += all;
    __syncthreads();
  }
}

// What dq leaves for dk/dv, -Delta and -lse / scale, formed by workgroups of the set-up kernel where both share a launch: a
// workgroup per 64 rows of a sequence and query head, a row by 8 or 16 lanes as in lg_delta_rows, the same bits.
struct LgBwdDelta {
  int first, chunks;  // first workgroup (none: past the grid); 64-row chunks of all sequences
  int D, ld, wld;
  const uint16_t *out, *dout;
  const float* lse;
  float *ndelta, *nlse;
  float scale;
};
template <int D>
__device__ __forceinline__ void delta_rows(const LgBwdDelta& d, const LgBwdSetup& a, int N, int id) {
  constexpr int CPR = D / 8, RPP = SETUP_NT / CPR;
  const int tid = threadIdx.x, lane = tid & 63, head = id / d.chunks;
  int chunk = id - head * d.chunks, row0 = 0, wrow0 = 0;
  if (a.n > 0) {  // the sequence that has the chunk, by sums over the lanes
    int chunks = 0, rows = 0, found = -1;
    for (int x0 = 0; x0 < a.n && found < 0; x0 += 64) {
      const int len = x0 + lane < a.n ? a.len[x0 + lane] : 0;
      int c = (len + 63) / 64, r = len;
      for (int y = 1; y < 64; y <<= 1) {
        const int cu = __shfl_up(c, y), ru = __shfl_up(r, y);
        c += lane >= y ? cu : 0;
        r += lane >= y ? ru : 0;
      }
      const unsigned long long past = __builtin_amdgcn_ballot_w64(chunks + c > chunk);
      if (past != 0) {
        const int at = __builtin_ctzll(past);
        found = x0 + at;
        N = a.len[found];
        row0 = a.row0[found];
        wrow0 = rows + lg_uniform(__shfl(r, at)) - N;
        chunk -= chunks + lg_uniform(__shfl(c, at)) - (N + 63) / 64;
      }
      chunks += lg_uniform(__shfl(c, 63));
      rows += lg_uniform(__shfl(r, 63));
    }
  }
#pragma unroll
  for (int x = 0; x < 64 / RPP; ++x) {
    const int i = chunk * 64 + x * RPP + tid / CPR;
    const size_t row = (size_t)head * d.ld + row0 + min(i, N - 1);
    const size_t at = row * D + tid % CPR * 8;
    const uint4 g = *reinterpret_cast<const uint4*>(d.dout + at), o = *reinterpret_cast<const uint4*>(d.out + at);
    const float s = lg_group_sum<CPR>(lg_dot8(g, o, 0.f));
    if (tid % CPR == 0 && i < N) {
      d.ndelta[(size_t)head * d.wld + wrow0 + i] = -s;
      d.nlse[(size_t)head * d.wld + wrow0 + i] = -d.lse[row] / d.scale;
    }
  }
}

// Grid: one workgroup for the counters, the descriptor and the items, one per sequence (batch: one) for its column
// table, others clear the partial sums, the last ones form Delta (where dq does not).
__global__ __launch_bounds__(SETUP_NT) void bwd_setup_kernel(LgBwdSetup a, LgMask m, int* __restrict__ queue,
                                                             LgBwdSeqs* __restrict__ seqs, int* __restrict__ items,
                                                             int* __restrict__ col_of_group, int* __restrict__ col_list,
                                                             int ncol, unsigned* __restrict__ arrived, int narrived,
                                                             float* __restrict__ part, size_t part_floats, LgBwdDelta delta) {
  const int tid = threadIdx.x, nt = a.n > 0 ? a.n : 1;
  if ((int)blockIdx.x >= delta.first) {
    if (delta.D == 64) delta_rows<64>(delta, a, m.N, blockIdx.x - delta.first);
    else delta_rows<128>(delta, a, m.N, blockIdx.x - delta.first);
    return;
  }
  if ((int)blockIdx.x > nt) {  // (device-scope stores: atomics of every XCD add to these values)
    const size_t step = (size_t)(delta.first - 1 - nt) * SETUP_NT;
    for (size_t x = (size_t)(blockIdx.x - 1 - nt) * SETUP_NT + tid; x < part_floats / 2; x += step)
      lg_store_shared2(part + 2 * x, 0.f, 0.f);
    return;
  }
  if (blockIdx.x == 0) {
    if (tid < 16) queue[tid] = 0;
    for (int x = tid; x < narrived; x += SETUP_NT) arrived[x] = 0;
  }
  if (a.n == 0) {
    if (blockIdx.x == 1 && ncol > 0) column_table(col_of_group, col_list, m, a.btk);
    return;
  }
  // running sums over the sequences: query tiles, key tiles, groups, split-off column groups, column work items, rows
  // and chunks of lone groups
  __shared__ int sum[7][LG_PACK_MAX + 1];
  static_assert(SETUP_NT >= LG_PACK_MAX + 1, "a thread per sequence");
  const int len = tid < a.n ? a.len[tid] : 0;
  if (tid < 7) sum[tid][0] = 0;
  if (tid < LG_PACK_MAX) {
    sum[0][tid + 1] = (len + LG_BF16_TQ - 1) / LG_BF16_TQ;
    sum[1][tid + 1] = (len + a.btk - 1) / a.btk;
    sum[2][tid + 1] = (len + 63) / 64;
    sum[3][tid + 1] = tid < a.n ? a.ncol[tid] : 0;
    sum[4][tid + 1] = tid < a.n ? a.citems[tid] : 0;
    sum[5][tid + 1] = len;
    sum[6][tid + 1] = tid < a.n ? a.nlone[tid] : 0;
  }
  __syncthreads();
  for (int d = 1; d < LG_PACK_MAX; d <<= 1) {
    int y[7];
    for (int x = 0; x < 7; ++x) y[x] = tid < LG_PACK_MAX && tid + 1 > d ? sum[x][tid + 1 - d] : 0;
    __syncthreads();
    if (tid < LG_PACK_MAX)
      for (int x = 0; x < 7; ++x) sum[x][tid + 1] += y[x];
    __syncthreads();
  }
  if (blockIdx.x > 0) {
    const int sq = blockIdx.x - 1;
    if (a.ncol[sq] > 0)
      column_table(col_of_group + sum[2][sq], col_list + sum[3][sq], lg_mask_for_length(m, a.len[sq]), a.btk);
    return;
  }
  if (tid == 0) seqs->n = a.n;
  if (tid < a.n) {
    seqs->row0[tid] = a.row0[tid];
    seqs->wrow0[tid] = sum[5][tid];
    seqs->len[tid] = len;
    seqs->ncol[tid] = a.ncol[tid];
    seqs->nlone[tid] = a.nlone[tid];
  }
  if (tid <= a.n) {
    seqs->qtile0[tid] = sum[0][tid];
    seqs->ktile0[tid] = sum[1][tid];
    seqs->grp0[tid] = sum[2][tid];
    seqs->col0[tid] = sum[3][tid];
    seqs->citem0[tid] = sum[4][tid];
    seqs->litem0[tid] = sum[6][tid];
  }
  for (int t = tid; t < sum[1][a.n]; t += SETUP_NT) {
    int lo = 0, hi = a.n;  // the sequence of key tile t
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (sum[1][mid] <= t) lo = mid;
      else hi = mid;
    }
    const int kt = t - sum[1][lo], r = sum[1][lo + 1] - 1 - t;  // r: tiles of the sequence after this one
    const int c0 = lo < a.nwide ? 0 : a.nwide, c1 = lo < a.nwide ? a.nwide : a.n;  // its class
    int x0 = c0, x1 = c1;  // the sequences c0 .. x0 - 1 have more than r + 1 tiles (longest first)
    while (x0 < x1) {
      const int mid = (x0 + x1) >> 1;
      if (sum[1][mid + 1] - sum[1][mid] > r + 1) x0 = mid + 1;
      else x1 = mid;
    }
    // before it: of those sequences the tiles with more than r after them; of all with a tile at r, the ones before lo
    const int before = sum[1][x0] - sum[1][c0] - (x0 - c0) * (r + 1) + lo - c0;
    items[sum[1][c0] + before] = (lo << 24) | kt;
  }
}

// The sequence of a dk/dv work item: where its rows, key tiles and column groups start, how many groups are split off.
struct LgBwdItem {
  int row0, wrow0, ktile0, grp0, col0, ncol;
};
__device__ __forceinline__ LgBwdItem lg_bwd_item(const LgBwdSeqs* __restrict__ seqs, int sq, LgMask& m) {
  m = lg_mask_for_length(m, lg_uniform(seqs->len[sq]));
  return {lg_uniform(seqs->row0[sq]), lg_uniform(seqs->wrow0[sq]), lg_uniform(seqs->ktile0[sq]),
          lg_uniform(seqs->grp0[sq]), lg_uniform(seqs->col0[sq]), lg_uniform(seqs->ncol[sq])};
}

// A main work item: key tile, (b, kv head) and part of the window part.  Many items of a batch: in runs per XCD
// (lg_item_of), so that neighbouring key tiles share their Q / dO rows in one XCD's L2.  Otherwise (by_tile) heads
// innermost: the tiles with the most rows start first (with a multiple of 8 heads all tiles of a head still run on one
// XCD), packed sequences in the order of the item list.  False: an id of the padding.
struct LgBwdMain {
  int kt, bh, part;
};
__device__ __forceinline__ bool lg_bwd_main(const LgBwdWork& wk, int bid, int nkt, int total, int run, LgMask& m,
                                            LgBwdItem& it, LgBwdMain& w) {
  const int nbh = total / nkt, nparts = wk.heads_cut * wk.rows_cut;
  w.part = 0;
  if (wk.by_tile) {
    w.bh = bid % nbh;
    const int y = bid / nbh;
    w.part = y % nparts;
    w.kt = y / nparts;
    if (wk.seqs) {
      const int x = lg_uniform(wk.items[w.kt]);
      w.kt = x & 0xffffff;
      it = lg_bwd_item(wk.seqs, x >> 24, m);
    }
    return true;
  }
  const int L = lg_item_of(bid, run);
  const int at = lg_order_at(wk.order, L);
  w.bh = at / nkt;
  w.kt = at % nkt;
  lg_in_order(wk.order, L, nkt, &w.bh, &w.kt);
  return L < total;
}
// The query tiles [lo, hi] and query heads of the part: the window part of keys [k0, k1] (all query tiles that see them
// where no column parts are split off), rows and heads cut evenly.
__device__ __forceinline__ void lg_bwd_part_range(const LgBwdWork& wk, const LgMask& m, bool split, int k0, int k1, int part,
                                                  int G, int* lo, int* hi, int* head0, int* nheads) {
  lg_qtile_range(m, k0, k1, LG_BF16_BTQ, lo, hi);
  if (split) *hi = lg_qtile_window_hi(m, k1, LG_BF16_BTQ);
  *nheads = G / wk.heads_cut;
  *head0 = part / wk.rows_cut * *nheads;
  const int c = part % wk.rows_cut, len = *hi - *lo + 1, first = *lo;
  *lo = first + len * c / wk.rows_cut;
  *hi = first + len * (c + 1) / wk.rows_cut - 1;
}
// Where a part's sums go: a group slot for each 64 keys.
template <int D>
__device__ __forceinline__ float* lg_bwd_part_slot(const LgBwdWork& wk, const LgBwdItem& it, const LgBwdMain& w,
                                                   int nbh) {
  return wk.parts + (((size_t)(it.ktile0 + w.kt) * nbh + w.bh) * (wk.heads_cut * wk.rows_cut) + w.part) *
                        (btk_of(D) / 64 * LgSlot<D>::FLOATS);
}

// How many rows, from row j on, see key j (0 for keys past the end).
__device__ __forceinline__ unsigned lg_rows_seeing(const LgMask& m, int j) {
  if (j >= m.N) return 0;
  const bool column = j < m.sink || (m.stride > 0 && lg_strided(m, lg_div_b(m, j)));
  return (unsigned)((column ? m.N : lg_window_end(m, j)) - j);
}

// a[r] = the sum, in order, of n parts' values at src + 64 r, a part `step` floats after the one before, four of them asked for at a time.
template <typename Load>
__device__ __forceinline__ void lg_add_parts(const float* src, int n, size_t step, float (&a)[16], Load load) {
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = 0.f;
  int p = 0;
  const auto add = [&](auto count) {
    constexpr int P = decltype(count)::value;
    float x[P][16];
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) x[i][r] = load(src + (p + i) * step + 64 * r);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) a[r] += x[i][r];
    p += P;
  };
  while (p + 4 <= n) add(std::integral_constant<int, 4>{});
  if (p + 2 <= n) add(std::integral_constant<int, 2>{});
  if (p < n) add(std::integral_constant<int, 1>{});
}
// The sums of 32 keys and 32 dims (times f) to a lane's key row: dst its first dim of the block.
__device__ __forceinline__ void lg_put_keys(uint16_t* __restrict__ dst, const float (&a)[16], float f) {
#pragma unroll
  for (int r4 = 0; r4 < 4; ++r4) {
    uint2 w;
    w.x = lg_pack_bf16(a[4 * r4 + 0] * f, a[4 * r4 + 1] * f);
    w.y = lg_pack_bf16(a[4 * r4 + 2] * f, a[4 * r4 + 3] * f);
    *reinterpret_cast<uint2*>(dst + 8 * r4) = w;
  }
}

// After a workgroup has stored a chunk of a lone group (Hq == Hkv), or its key tile's window part where that counts as one: the
// last of them adds the chunks in order.  dk, dv: the sequence's first row.
template <int D>
__device__ __forceinline__ void lg_lone_done(const LgBwdWork& wk, int bh, int sq, int nseq, int nchunk, int lone0, int col0,
                                             uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int grp, int N, float scale) {
  using Slot = LgSlot<D>;
  constexpr int DB = D / 32;
  __shared__ int last;
  lg_shared_stores_done();
  __syncthreads();
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(wk.arrived + (size_t)bh * nseq + sq, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
           (unsigned)(nchunk - 1 + (wk.lone_joint ? 1 : 0));
  __syncthreads();
  if (!last) return;
  float* sum = wk.colpart + ((size_t)bh * wk.ncol + col0) * Slot::FLOATS;
  const float* chunks = wk.lonepart + ((size_t)bh * wk.nlone_all + lone0) * Slot::FLOATS;
  const int lane = threadIdx.x & 63, n = lane & 31, g = lane >> 5;
  for (int y = lg_uniform(threadIdx.x >> 6); y < 4 * DB; y += blockDim.x / 64) {  // blocks of 32 keys and 32 dims, dk's and dv's
    const int at = 1024 * y + lane, which = y / DB & 1;
    float a[16];
    lg_add_parts(chunks + at, nchunk, Slot::FLOATS, a, lg_load_shared1);
    if (!wk.lone_joint) {
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[at + 64 * r] = a[r];
      continue;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] += lg_load_shared1(sum + at + 64 * r);
    const int j = 64 * grp + 32 * (y / (2 * DB)) + n;
    if (j < N) lg_put_keys((which ? dv : dk) + (size_t)j * D + y % DB * 32 + 4 * g, a, which ? 1.f : scale);
  }
}

// 32 query rows against the wave's 32 keys, in an order that keeps few values alive at a time:
// S -> P -> (dV += dO^T P) -> dP -> dS -> (dK += Q^T dS), head dim 128: S -> dP and P -> (dV += dO^T P) -> dS -> (dK += Q^T dS), two
// exponentials behind each matrix instruction of dP.  sq, sg: the rows of Q and dO in LDS; sL: their -lse / scale, 64 floats further
// on their -Delta; voff: the V rows of the wave's keys.
// Exponentials by themselves, and behind dP's (backward, us): 8 heads of 128, 3500 tokens, window 600 55.9 -> 55.3; 4 x 8, 1111,
// causal 63.2 -> 61.8; 1, 1098 55.9 -> 54.2; 32, 16384, window 640 817 -> 808; 2 x 16/4, 1500 104.0 -> 102.5.  Head dim 64 has four
// of them for each of half as many matrix instructions and lost: 16, 1117 31.2 -> 32.5; 32, 16384, window 2048 947 -> 974.
template <int D, typename Dead>
__device__ __forceinline__ void lg_dkdv_block(const unsigned char* smem, const LgSwzReader<D>& rd, int sq, int sg, int voff,
                                              const float* sL, const bf16x8_t (&kf)[D / 16], f32x16_t (&ak)[D / 32],
                                              f32x16_t (&av)[D / 32], float sl2, int g, bool full, Dead dead) {
  constexpr int DC = D / 16, DB = D / 32, AHEAD = D == 128 ? 2 : 3;
  constexpr bool BEHIND = D == 128;  // P's exponentials behind dP's matrix instructions
  float p[16];
  f32x16_t sc, dp;  // start from -lse / scale and -Delta of their rows (register r <-> row 8 (r / 4) + 4g + r % 4)
  LgRing<DC, AHEAD> rows, vrows;
  LgRing<2 * DB, AHEAD> cols;
  auto q_rows = [&](int u) { return rd.read_rows(smem, sq, 0, u); };
  auto g_rows = [&](int u) { return rd.read_rows(smem, sg, 0, u); };
  auto v_rows = [&](int u) { return rd.read_rows(smem, voff, 0, u); };
  auto g_cols = [&](int u) { return rd.read_cols(smem, sg, u % DB, u / DB); };
  auto q_cols = [&](int u) { return rd.read_cols(smem, sq, u % DB, u / DB); };
  auto start = [&](f32x16_t& x, const float* from) {
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const float4 f = *reinterpret_cast<const float4*>(from + 8 * r4 + 4 * g);
      x[4 * r4 + 0] = f.x; x[4 * r4 + 1] = f.y; x[4 * r4 + 2] = f.z; x[4 * r4 + 3] = f.w;
    }
  };
  auto product_dp = [&](auto behind) {  // behind(u) goes behind matrix instruction u
    start(dp, sL + 64);
    rows.begin(g_rows);
    vrows.begin(v_rows);
    lg_static_for<DC>([&](auto U) {
      constexpr int u = decltype(U)::value, w = u + AHEAD, x = w % (AHEAD + 1), y = u % (AHEAD + 1);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (w < DC) {
        rows.op[x] = g_rows(w);
        vrows.op[x] = v_rows(w);
      }
      dp = lg_mfma32(rows.op[y], vrows.op[y], dp);
      behind(u);
    });
  };
  __builtin_amdgcn_sched_barrier(0);  // phases stay apart: bounds the operands held at once
  start(sc, sL);
  rows.begin(q_rows);
  rows.run(q_rows, [&](int u, bf16x8_t a) { sc = lg_mfma32(a, kf[u], sc); });
  if constexpr (BEHIND) {
    product_dp([&](int u) {
#pragma unroll
      for (int x = 0; x < 16 / DC; ++x) p[16 / DC * u + x] = __builtin_amdgcn_exp2f(sc[16 / DC * u + x] * sl2);
    });
    __builtin_amdgcn_sched_barrier(0);
    cols.begin(g_cols);
  } else {
    cols.begin(g_cols);
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] = __builtin_amdgcn_exp2f(sc[r] * sl2);
  }
  if (!full) {
    asm volatile("; masked" ::: "memory");  // (a real branch: as selects the masks cost whole tiles 5 % at head dim 64)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (dead(r)) p[r] = 0.f;
  }
  {
    const bf16x8_t pb[2] = {lg_pack8(p), lg_pack8(p + 8)};
    cols.run(g_cols, [&](int u, bf16x8_t a) { av[u % DB] = lg_mfma32(a, pb[u / DB], av[u % DB]); });
  }
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (!BEHIND) product_dp([](int) {});
  cols.begin(q_cols);
#pragma unroll
  for (int r = 0; r < 16; ++r) p[r] *= dp[r];  // p becomes dS
  {
    const bf16x8_t db_[2] = {lg_pack8(p), lg_pack8(p + 8)};
    cols.run(q_cols, [&](int u, bf16x8_t a) { ak[u % DB] = lg_mfma32(a, db_[u / DB], ak[u % DB]); });
  }
}

template <int D>
constexpr int DKDV_LDS = btk_of(D) / 64 * LgSwzTile<D>::BYTES + 2 * (2 * LgSwzTile<D>::BYTES + 1024);
template <int D, bool COLUMN, bool JOINT>
__device__ __forceinline__ void dkdv_bf16_item(
    unsigned char* smem, int bid,
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ dout, const float* __restrict__ nlse, const float* __restrict__ ndelta,
    uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int Hq, int Hkv, float scale, LgMask m_in,
    int nkt, int total, int run, const LgBwdWork& wk) {
  LgMask m = m_in;
  using T = LgSwzTile<D>;
  constexpr int TQ = LG_BF16_BTQ, TK = btk_of(D), NT = 2 * TK, NG = TK / 64;
  using Dma = LgDma<D, NT>;
  static_assert(TQ == 64, "64 query rows per step, a wave for every 32 keys");
  constexpr int DC = D / 16, DB = D / 32;
  constexpr int HALF = 32 * T::ROW_BYTES;
  constexpr int VRES = NG * T::BYTES;                // the workgroup's V rows
  constexpr int OFF_G = T::BYTES, OFF_L = 2 * T::BYTES;
  constexpr int STAGE = 2 * T::BYTES + 1024;         // Q tile, dO tile, -lse / scale | -Delta (2 x 64 floats)
  static_assert(DKDV_LDS<D> == VRES + 2 * STAGE, "V rows and two stages");

  const int G = Hq / Hkv;
  const float sl2 = scale * LOG2E;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, g = lane >> 5;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  // Work item.
  //   main: see lg_bwd_main.
  //   COLUMN: (chunk * nvt + virtual tile) * (heads) + (b x kv head) * G + query head of the group: with the heads
  //     innermost every XCD gets the same mix of long and short items (and of those that exit at once: a virtual tile
  //     has no rows in the chunks before its column part starts), and the virtual tiles of one head that walk the same
  //     chunk of query rows run on one XCD at about the same time.  Packed: one sequence after the other.
  int vt = 0, chunk = 0, gq = 0;
  LgBwdItem it = {0, 0, 0, 0, 0, wk.ncol};
  LgBwdMain w = {0, 0, 0};
  if (COLUMN) {
    const int nh = wk.B * Hq;
    int x = bid;
    const int hd = x % nh;
    x /= nh;
    if (wk.seqs) {
      const int sq = lg_seq_of(wk.seqs->citem0, lg_uniform(wk.seqs->n), x);
      x -= lg_uniform(wk.seqs->citem0[sq]);
      it = lg_bwd_item(wk.seqs, sq, m);
    }
    const int nvt = (it.ncol + NG - 1) / NG;
    vt = x % nvt;
    chunk = x / nvt;
    gq = hd % G;
    w.bh = hd / G;
  } else if (!lg_bwd_main(wk, bid, nkt, total, run, m, it, w)) {
    return;
  }
  const int bh = w.bh, kt = w.kt;
  const int N = m.N, ncol = it.ncol;
  const int* __restrict__ clist = wk.col_list + it.col0;
  const int b = bh / Hkv, hk = bh % Hkv;
  const int k0 = kt * TK, k1 = min(k0 + TK - 1, N - 1);
  const size_t kbase = ((size_t)(b * Hkv + hk) * m.ld + it.row0) * D;
  // this wave's 32 keys: part of the key tile, or half of one of the virtual tile's column groups
  int kw0 = k0 + wave_s * 32;
  int col_gi = 0;        // COLUMN: index of this wave's column group
  bool active = true;    // COLUMN: the virtual tile may have fewer groups
  int r0_w = 0;          // COLUMN: first row of the wave's column part
  if (COLUMN) {
    col_gi = NG * vt + (wave_s >> 1);
    active = col_gi < ncol;
    const int grp = clist[min(col_gi, ncol - 1)];
    kw0 = 64 * grp + 32 * (wave_s & 1);
    const int t1 = min((64 * grp / TK) * TK + TK - 1, N - 1);
    r0_w = (lg_qtile_window_hi(m, t1, TQ) + 1) * TQ;
  }
  const int j = kw0 + n;  // this lane's key
  const LgKeys wkeys = lg_keys(m, kw0, kw0 + 31);
  const unsigned seen = lg_rows_seeing(m, j);

  f32x16_t ak[DB], av[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) ak[db][r] = av[db][r] = 0.f;
  // query tiles of this work item
  int lo, hi, hq0 = hk * G, nheads = 1;
  if (COLUMN) {
    // the query tiles of chunk number `chunk` (chunks are cut at fixed tile numbers for all virtual
    // tiles, counted from the chunk in which the first column part starts) that come after the
    // window part of the virtual tile's first group
    const int tf = min((64 * clist[0] / TK) * TK + TK - 1, N - 1);
    const int c_abs = (lg_qtile_window_hi(m, tf, TQ) + 1) / wk.chunk + chunk;
    const int grp0 = clist[NG * vt];
    const int t1 = min((64 * grp0 / TK) * TK + TK - 1, N - 1);
    lo = max(lg_qtile_window_hi(m, t1, TQ) + 1, c_abs * wk.chunk);
    hi = min((N - 1) / TQ, c_abs * wk.chunk + wk.chunk - 1);
    if (lo > hi) return;
    hq0 += gq;
  } else {
    int head0;
    lg_bwd_part_range(wk, m, ncol > 0, k0, k1, w.part, G, &lo, &hi, &head0, &nheads);
    hq0 += head0;
  }
  const int per_head = hi - lo + 1;
  const int steps = per_head * nheads;

  const int voff = (wave >> 1) * T::BYTES + (wave & 1) * HALF;  // this wave's 32 V rows
  Dma dma;
  dma.init(tid);
  LgSwzReader<D> rd;
  rd.init(n, g);
  const uint32_t lds0 = (uint32_t)(uintptr_t)LG_LDS_PTR(unsigned char, smem);
  // K rows to registers, V rows resident.  K of head dim 64 goes through the stages' place; at 128, where one
  // workgroup fits a CU, its two barriers cost more than they save (window 256, 32768 tokens, 32 heads: 545 us direct, 568 through LDS; at 64 247 direct, 243).
  constexpr bool K_LDS = D == 64;
  static_assert(!K_LDS || NG * T::BYTES <= 2 * STAGE, "K rows fit the stages");
  bf16x8_t kf[DC];
  if constexpr (!K_LDS) {
    const int jk = min(j, N - 1);
#pragma unroll
    for (int dc = 0; dc < DC; ++dc)
      kf[dc] = lg_as_bf16x8(*reinterpret_cast<const uint4*>(k + kbase + (size_t)jk * D + dc * 16 + g * 8));
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) asm volatile("" ::"v"(kf[dc]));
  }
#pragma unroll
  for (int kv = K_LDS ? 0 : 1; kv < 2; ++kv)
#pragma unroll
    for (int x = 0; x < NG; ++x) {
      const int r0 = COLUMN ? 64 * clist[min(NG * vt + x, ncol - 1)] : k0 + 64 * x;
      const int rc = min(r0, N - 1);  // a tile wholly past the end repeats the last row
      dma.issue((kv ? v : k) + kbase + (size_t)rc * D, r0 < N ? N - r0 : 1, lds0 + (kv ? 0 : VRES) + x * T::BYTES);
    }
  if constexpr (K_LDS) {
    LG_WAIT_VMCNT(NG * Dma::CH);
    __syncthreads();
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) kf[dc] = rd.read_rows(smem, VRES + (wave_s >> 1) * T::BYTES, wave_s & 1, dc);
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) asm volatile("" ::"v"(kf[dc]));
    __syncthreads();
  }

  // (head, query tile) of a step advance incrementally: no divisions in the loop
  // rows of the query head whose step is requested next
  const uint16_t* qh = q + ((size_t)(b * Hq + hq0) * m.ld + it.row0) * D;
  const uint16_t* gh = dout + ((size_t)(b * Hq + hq0) * m.ld + it.row0) * D;
  const float* lh = nlse + (size_t)(b * Hq + hq0) * wk.wld + it.wrow0;
  const float* dh = ndelta + (size_t)(b * Hq + hq0) * wk.wld + it.wrow0;
  auto next_head = [&] {
    qh += (size_t)m.ld * D;
    gh += (size_t)m.ld * D;
    lh += wk.wld;
    dh += wk.wld;
  };
  auto issue_step = [&](int u, int buf) {
    const int q0 = u * TQ;
    const uint32_t st = lds0 + VRES + buf * STAGE;
    // the small per-row loads go first: anything the compiler makes them wait for must not
    // include the tile loads issued below
    if (wave < 2) {  // wave 0: -lse / scale rows, wave 1: -Delta rows (64 floats each)
      const float* src = (wave == 0 ? lh : dh) + min(q0 + lane, N - 1);
      lg_dma_f32x64(src, st + OFF_L + wave * 256);
    }
    dma.issue(qh + (size_t)q0 * D, N - q0, st);
    dma.issue(gh + (size_t)q0 * D, N - q0, st + OFF_G);
  };

  // The query tiles [lo, hi] of a head are walked rotated: at step x the tile congruent to x
  // modulo the range length.  Neighbouring key tiles, whose ranges overlap almost completely and
  // which run side by side, then read the same Q / dO tile at the same time and share it in L2.
  const int u0 = per_head > 0 ? lo + (per_head - lo % per_head) % per_head : lo;
  int u_i = u0;                  // step being issued
  int u_c = u0;                  // query tile of the step being computed
  int left_i = per_head;         // steps of the head being issued that are not issued yet
  if (steps > 0) issue_step(u_i, 0);
  else LG_WAIT_VMCNT(0);  // (a part without rows: nothing may still be on its way to LDS when it ends)
  for (int st = 0; st < steps; ++st) {
    const int buf = st & 1;
    LG_WAIT_VMCNT(0);
    __syncthreads();  // step st landed for everyone; everyone is done with step st-1
    if (st + 1 < steps) {
      u_i = (u_i == hi) ? lo : u_i + 1;
      if (--left_i == 0) {  // next query head of the group: same walk again
        left_i = per_head;
        u_i = u0;
        next_head();
      }
      issue_step(u_i, buf ^ 1);
    }
    const int q0 = u_c * TQ;
    u_c = (u_c == hi) ? lo : u_c + 1;
    // this wave's 32 keys against the step's two blocks of 32 queries, as far as they have live pairs (in most steps of the
    // sink key tile, once the queries are past its window, most waves have none)
    if (COLUMN && (!active || q0 < r0_w)) continue;  // no group, or rows of its window part
    const int kind = lg_keys_kind(wkeys, q0, q0 + TQ - 1);
    if (kind == LG_TILE_DEAD) continue;
    const int sq = VRES + buf * STAGE, sg = sq + OFF_G;
    const float* sL = reinterpret_cast<const float*>(smem + sq + OFF_L);
    auto block = [&](int qb, bool full) {
      // register r: row r0 + 4g + c, which sees the key if it is one of the `seen` rows from j on
      const int from = q0 + 32 * qb + 4 * g - j;
      lg_dkdv_block<D>(smem, rd, sq + qb * HALF, sg + qb * HALF, voff, sL + qb * 32, kf, ak, av, sl2, g, full,
                       [&](int r) { return !((unsigned)(from + lg_crow(r, 0)) < seen); });
    };
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      if (kind != LG_TILE_FULL && lg_keys_kind(wkeys, q0 + 32 * qb, q0 + 32 * qb + 31) == LG_TILE_DEAD) continue;
      block(qb, kind == LG_TILE_FULL);
    }
  }

  using Slot = LgSlot<D>;
  if (COLUMN) {
    if (!active) return;
    float* dst = wk.colpart + ((size_t)bh * wk.ncol + it.col0 + col_gi) * Slot::FLOATS + lane;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        unsafeAtomicAdd(dst + Slot::at(wave_s & 1, 0, db) + 64 * r, ak[db][r]);  // hardware float adds
        unsafeAtomicAdd(dst + Slot::at(wave_s & 1, 1, db) + 64 * r, av[db][r]);
      }
    return;
  }
  if (wk.heads_cut * wk.rows_cut > 1) {  // bwd_fold_kernel adds the parts
    float* dst = lg_bwd_part_slot<D>(wk, it, w, total / nkt) + (wave_s >> 1) * Slot::FLOATS + lane;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        dst[Slot::at(wave_s & 1, 0, db) + 64 * r] = ak[db][r];
        dst[Slot::at(wave_s & 1, 1, db) + 64 * r] = av[db][r];
      }
    return;
  }
  const int cid = (ncol > 0 && kw0 < N) ? wk.col_of_group[it.grp0 + (kw0 >> 6)] : -1;
  const bool joint = JOINT && wk.lone_joint && it.ncol == 1;
  if (joint && cid >= 0) {  // (its window part counts as one of the lone group's chunks: below)
    float* sum = wk.colpart + ((size_t)bh * wk.ncol + it.col0) * Slot::FLOATS + lane;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        lg_store_shared1(sum + Slot::at(wave_s & 1, 0, db) + 64 * r, ak[db][r]);
        lg_store_shared1(sum + Slot::at(wave_s & 1, 1, db) + 64 * r, av[db][r]);
      }
  } else {
    if (cid >= 0) {
      const float* src = wk.colpart + ((size_t)bh * wk.ncol + it.col0 + cid) * Slot::FLOATS + lane;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        __builtin_amdgcn_sched_barrier(0);  // (not all loads at once)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          ak[db][r] += lg_load_shared1(src + Slot::at(wave_s & 1, 0, db) + 64 * r);
          av[db][r] += lg_load_shared1(src + Slot::at(wave_s & 1, 1, db) + 64 * r);
        }
      }
    }
    unsigned char* rows = smem + voff;  // (its V rows' place: no other wave reads them)
#pragma unroll
    for (int which = 0; which < 2; ++which) {
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        float a[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) a[r] = which ? av[db][r] : ak[db][r];
        lg_rows_put<D>(rows, lane, db, a, which ? 1.f : scale);
      }
      lg_rows_write<D>(rows, lane, (which ? dv : dk) + kbase + (size_t)kw0 * D, N - kw0);
    }
  }
  if (joint) {
    const int grp = lg_uniform(wk.col_list[it.col0]);
    if (64 * grp / TK != w.kt) return;
    int sq = 0, nseq = 1, nchunk = wk.nlone, lone0 = 0;
    if (wk.seqs) {
      nseq = lg_uniform(wk.seqs->n);
      sq = lg_seq_of(wk.seqs->ktile0, nseq, it.ktile0);
      nchunk = lg_uniform(wk.seqs->nlone[sq]);
      lone0 = lg_uniform(wk.seqs->litem0[sq]);
    }
    lg_lone_done<D>(wk, bh, sq, nseq, nchunk, lone0, it.col0, dk + kbase, dv + kbase, grp, N, scale);
  }
}
template <int D, bool COLUMN>
__global__ __launch_bounds__(btk_of(D) * 2) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 3, D == 128 ? 2 : 3))) void
dkdv_bf16_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ dout, const float* __restrict__ nlse, const float* __restrict__ ndelta,
    uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int Hq, int Hkv, float scale, LgMask m_in,
    int nkt, int total, int run, LgBwdWork wk) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DKDV_LDS<D>];
  dkdv_bf16_item<D, COLUMN, false>(smem, blockIdx.x, q, k, v, dout, nlse, ndelta, dk, dv, Hq, Hkv, scale, m_in, nkt, total, run, wk);
}

// --------------------------------------------------------- dk, dv: the column part of a lone group
// A head's only column group (the sink keys) is seen by every later query: up to N / 64 query tiles for 64 keys.  Left
// to its key tile, one workgroup of the whole launch walks them with one wave in four (or two in eight) at work: with 2
// heads and 24000 tokens 1.0 ms beside 0.16 ms for all the rest.  Here the eight waves of a workgroup are the 2 blocks
// of 32 keys x the 4 blocks of 32 rows of two query tiles (head dim 64: four waves, a query tile, as many as share a launch with
// dq), double-buffered, and the range is cut into chunks.  Hq == Hkv: every chunk leaves its sums in the workspace, and the one that
// finishes last adds them in order (bit-reproducible; the cut depends on the sequence and its heads alone).  Groups of query
// heads: float32 atomics.
// A work item.  WAVES: 8, two query tiles at a time, or 4, one.  GROUPS: Hq != Hkv.  dk, dv: for wk.lone_joint.
template <int D, int WAVES>
constexpr int LONE_LDS = LgSwzTile<D>::BYTES + WAVES / 2 * (2 * LgSwzTile<D>::BYTES + 1024);  // V rows, two steps' tiles
template <int D, int WAVES, bool GROUPS>
__device__ __forceinline__ void dkdv_lone_item(
    unsigned char* smem, int id, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ dout, const float* __restrict__ nlse, const float* __restrict__ ndelta,
    uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int Hq, int Hkv, float scale, LgMask m, const LgBwdWork& wk) {
  using T = LgSwzTile<D>;
  using Slot = LgSlot<D>;
  constexpr int NT = 64 * WAVES, TILES = WAVES / 4;  // query tiles a step
  using Dma = LgDma<D, NT>;
  constexpr int TQ = LG_BF16_BTQ, TK = btk_of(D), DC = D / 16, DB = D / 32;
  constexpr int HALF = 32 * T::ROW_BYTES;
  constexpr int OFF_G = T::BYTES, OFF_L = 2 * T::BYTES, STAGE = 2 * T::BYTES + 1024;  // as in the kernel above
  static_assert(LONE_LDS<D, WAVES> == T::BYTES + 2 * TILES * STAGE, "V rows, two steps' tiles");

  const int nh = wk.B * Hq, hd = id % nh;
  int chunk = id / nh, nchunk = wk.nlone, lone0 = 0, sq = 0, nseq = 1;
  LgBwdItem it = {0, 0, 0, 0, 0, wk.ncol};
  if (wk.seqs) {
    nseq = lg_uniform(wk.seqs->n);
    sq = lg_seq_of(wk.seqs->litem0, nseq, chunk);
    lone0 = lg_uniform(wk.seqs->litem0[sq]);
    nchunk = lg_uniform(wk.seqs->nlone[sq]);
    chunk -= lone0;
    it = lg_bwd_item(wk.seqs, sq, m);
  }
  const int b = hd / Hq, hq = hd % Hq, hk = hq / (Hq / Hkv), bh = b * Hkv + hk;
  const int N = m.N, grp = lg_uniform(wk.col_list[it.col0]);
  const int first = lg_qtile_window_hi(m, min((64 * grp / TK) * TK + TK - 1, N - 1), TQ) + 1, last = (N - 1) / TQ;
  const int pairs = (last - first + 2) / 2;
  // steps [p0, p1) (never none: nchunk <= pairs)
  const int p0 = pairs * chunk / nchunk * (2 / TILES), p1 = min(pairs * (chunk + 1) / nchunk * (2 / TILES), TILES == 2 ? pairs : last - first + 1);

  const int tid = threadIdx.x, lane = tid & 63, wave = lg_uniform(tid >> 6);
  const int n = lane & 31, g = lane >> 5;
  const int kb = wave & 1, qb = (wave >> 1) & 1, tile = wave >> 2;
  const float sl2 = scale * LOG2E;
  const size_t kbase = ((size_t)bh * m.ld + it.row0) * D;
  const size_t row0 = (size_t)hd * m.ld + it.row0, wrow0 = (size_t)hd * wk.wld + it.wrow0;
  const int kw0 = 64 * grp + 32 * kb, j = kw0 + n;

  bf16x8_t kf[DC];
#pragma unroll
  for (int dc = 0; dc < DC; ++dc)
    kf[dc] = lg_as_bf16x8(*reinterpret_cast<const uint4*>(k + kbase + (size_t)min(j, N - 1) * D + dc * 16 + g * 8));
#pragma unroll
  for (int dc = 0; dc < DC; ++dc) asm volatile("" ::"v"(kf[dc]));
  f32x16_t ak[DB], av[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) ak[db][r] = av[db][r] = 0.f;

  Dma dma;
  dma.init(tid);
  LgSwzReader<D> rd;
  rd.init(n, g);
  const uint32_t lds0 = (uint32_t)(uintptr_t)LG_LDS_PTR(unsigned char, smem);
  dma.issue(v + kbase + (size_t)64 * grp * D, N - 64 * grp, lds0);
  auto issue = [&](int pr, int buf) {
#pragma unroll
    for (int x = 0; x < TILES; ++x) {
      const int q0 = min(first + TILES * pr + x, last) * TQ;  // (an odd range repeats its last tile; nobody uses it)
      const uint32_t st = lds0 + T::BYTES + (TILES * buf + x) * STAGE;
      if ((wave >> 1) == x)  // -lse / scale rows and -Delta rows (64 floats each)
        lg_dma_f32x64(((wave & 1) ? ndelta : nlse) + wrow0 + min(q0 + lane, N - 1), st + OFF_L + (wave & 1) * 256);
      dma.issue(q + (row0 + q0) * D, N - q0, st);
      dma.issue(dout + (row0 + q0) * D, N - q0, st + OFF_G);
    }
  };
  issue(p0, 0);
  for (int pr = p0; pr < p1; ++pr) {
    const int buf = (pr - p0) & 1;
    LG_WAIT_VMCNT(0);
    __syncthreads();  // this step's tiles landed for everyone; everyone is done with the one before
    if (pr + 1 < p1) issue(pr + 1, buf ^ 1);
    const int u = first + TILES * pr + tile, q0 = u * TQ + 32 * qb;
    if (u > last || q0 >= N) continue;
    const int kind = lg_tile_kind(m, q0, min(q0 + 31, N - 1), kw0, kw0 + 31);
    if (kind == LG_TILE_DEAD) continue;
    const bool full = kind == LG_TILE_FULL && q0 + 32 <= N;
    const uint32_t bits = full ? ~0u : lg_row_bits(m, j, q0, g);
    const int st = T::BYTES + (TILES * buf + tile) * STAGE;
    lg_dkdv_block<D>(smem, rd, st + qb * HALF, st + OFF_G + qb * HALF, kb * HALF,
                     reinterpret_cast<const float*>(smem + st + OFF_L) + 32 * qb, kf, ak, av, sl2, g, full,
                     [&](int r) { return !((bits >> r) & 1); });
  }

  // the row blocks' sums meet in waves 0 and 1, dk and then dv through the LDS of the tiles
  float* red = reinterpret_cast<float*>(smem + T::BYTES);
  static_assert((WAVES - 2) * DB * 4096 <= 2 * TILES * STAGE, "the other waves' blocks fit");
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    f32x16_t(&acc)[DB] = which ? av : ak;
    __syncthreads();
    if (wave >= 2)
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) red[((wave - 2) * DB + db) * 1024 + 64 * r + lane] = acc[db][r];
    __syncthreads();
    if (wave < 2)
#pragma unroll
      for (int x = 0; x < WAVES / 2 - 1; ++x)
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[db][r] += red[((2 * x + wave) * DB + db) * 1024 + 64 * r + lane];
  }

  float* sum = wk.colpart + ((size_t)bh * wk.ncol + it.col0) * Slot::FLOATS;
  if constexpr (GROUPS) {
    if (wave < 2)
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          unsafeAtomicAdd(sum + Slot::at(kb, 0, db) + 64 * r + lane, ak[db][r]);  // hardware float adds
          unsafeAtomicAdd(sum + Slot::at(kb, 1, db) + 64 * r + lane, av[db][r]);
        }
  } else {
    float* mine = wk.lonepart + ((size_t)bh * wk.nlone_all + lone0) * Slot::FLOATS;  // the sequence's first chunk
    if (wave < 2)
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float* dst = mine + (size_t)chunk * Slot::FLOATS + Slot::at(kb, 0, db) + 64 * r + lane;
          lg_store_shared1(dst, ak[db][r]);
          lg_store_shared1(dst + Slot::at(0, 1, 0), av[db][r]);
        }
    lg_lone_done<D>(wk, bh, sq, nseq, nchunk, lone0, it.col0, dk + kbase, dv + kbase, grp, N, scale);
  }
}
template <int D, int WAVES, bool GROUPS>
__global__ __launch_bounds__(64 * WAVES) void dkdv_lone_bf16_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ dout, const float* __restrict__ nlse, const float* __restrict__ ndelta, int Hq, int Hkv,
    float scale, LgMask m, LgBwdWork wk) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[LONE_LDS<D, WAVES>];
  dkdv_lone_item<D, WAVES, GROUPS>(smem, blockIdx.x, q, k, v, dout, nlse, ndelta, nullptr, nullptr, Hq, Hkv, scale, m, wk);
}

// dq and dk/dv in one launch, where neither fills the GPU (rule: bwd_both): the set-up kernel has formed Delta, and every work item does
// what it does in a launch of its own, with the same bits.  Head dim 128: dq's items two by two, for as many waves as dk/dv has.  LONE: and
// the column parts of lone groups (in one instance for all, calls without them lost up to 4 %).
enum { LONE_NONE, LONE_GROUPS, LONE_HEADS };
template <int D, int LONE>
__global__ __launch_bounds__(btk_of(D) * 2) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 3, D == 128 ? 2 : 3))) void
bwd_both_bf16_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ dout, const float* __restrict__ lse, float* __restrict__ nlse, float* __restrict__ ndelta,
    uint16_t* __restrict__ dq, uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int Hq, int Hkv, float scale, LgMask m,
    int nkt, int total, int run, LgBwdWork wk, int nqt, int nkv, int ndq, bool dq_first) {
  constexpr bool PAIR = D == 128;
  constexpr int LDS = std::max({(PAIR ? 2 : 1) * DQ_LDS<D>, DKDV_LDS<D>, LONE != LONE_NONE ? LONE_LDS<D, D / 16> : 0});
  __shared__ __attribute__((aligned(1024))) unsigned char smem[LDS];
  if (LONE != LONE_NONE && (int)blockIdx.x >= ndq + nkv) {
    if constexpr (LONE != LONE_NONE)
      dkdv_lone_item<D, D / 16, LONE == LONE_GROUPS>(smem, blockIdx.x - (ndq + nkv), q, k, v, dout, nlse, ndelta, dk, dv, Hq, Hkv, scale, m, wk);
    return;
  }
  const int id = dq_first ? (int)blockIdx.x : (int)blockIdx.x - nkv;
  if (id >= 0 && id < ndq) {  // heads innermost, longest rows first
    const int nh = wk.B * Hq, hd = id % nh, y = id / nh, x = PAIR ? y : y >> 1;
    const int half = PAIR ? lg_uniform(threadIdx.x >> 8) : 1 - (y & 1);
    const int b = hd / Hq, hq = hd - b * Hq;
    dq_bf16_item<D, false, PAIR>(smem, nullptr, q, k, v, nullptr, dout, lse, ndelta, nlse, dq, Hq, Hkv, scale, m, wk, b, hq / (Hq / Hkv), hq,
                                 nqt - 1 - x, half, x);
    return;
  }
  const int kv = dq_first ? (int)blockIdx.x - ndq : (int)blockIdx.x;
  dkdv_bf16_item<D, false, LONE == LONE_HEADS>(smem, kv, q, k, v, dout, nlse, ndelta, dk, dv, Hq, Hkv, scale, m, nkt, total, run, wk);
}

// Adds the parts of a key tile's window part, in order, and its column sums, and rounds: a wave for each 32 keys x 32 dims
// of dk or dv.  With few keys and many parts it is latency, so four parts are asked for at a time and the column sums with
// the first of them, and head dim 128 takes two workgroups per 32 keys.  One part after the other and one workgroup: 8 query
// heads on 1, 64, 3129 tokens 15.3 us, now 8.0; 16 on 2 of 128, 911 tokens 10.2, now 5.7; 4 x 16 on 2, 912 tokens (60 MB of
// parts) 10.2, now 9.6.
template <int D>
__global__ __launch_bounds__(256) void bwd_fold_kernel(uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int nbh,
                                                       float scale, LgMask m, LgBwdWork wk) {
  using Slot = LgSlot<D>;
  constexpr int DB = D / 32;
  constexpr int KB = btk_of(D) / 32;
  constexpr int WG = 2 * DB / 4;  // workgroups of a block of keys
  const int kb32 = blockIdx.x / WG % KB, x = blockIdx.x / (WG * KB), bh = x % nbh, t = x / nbh;
  const int nparts = wk.heads_cut * wk.rows_cut;
  LgBwdItem it = {0, 0, 0, 0, 0, wk.ncol};
  if (wk.seqs) it = lg_bwd_item(wk.seqs, lg_seq_of(wk.seqs->ktile0, lg_uniform(wk.seqs->n), t), m);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 31, g = lane >> 5;
  const int kw0 = (t - it.ktile0) * btk_of(D) + 32 * kb32, j = kw0 + n;
  if (kw0 >= m.N) return;
  const float* src = wk.parts + ((size_t)t * nbh + bh) * nparts * (KB / 2 * Slot::FLOATS) + (kb32 >> 1) * Slot::FLOATS + lane;
  const int cid = it.ncol > 0 ? wk.col_of_group[it.grp0 + (kw0 >> 6)] : -1;
  const float* csum = wk.colpart + ((size_t)bh * wk.ncol + it.col0 + max(cid, 0)) * Slot::FLOATS + lane;
  const int y = blockIdx.x % WG * 4 + wave, which = y / DB, db = y % DB, at = Slot::at(kb32 & 1, which, db);
  float a[16], c[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) c[r] = cid >= 0 ? lg_load_shared1(csum + at + 64 * r) : 0.f;
  lg_add_parts(src + at, nparts, KB / 2 * Slot::FLOATS, a, [](const float* p) { return *p; });
  if (cid >= 0)
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] += c[r];
  if (j < m.N) lg_put_keys((which ? dv : dk) + ((size_t)bh * m.ld + it.row0 + j) * D + db * 32 + 4 * g, a, which ? 1.f : scale);
}

// Work queue of the kernels that keep one workgroup per CU: queue[x] counts the items handed out
// with id % 8 == x (the ids that a grid launch would have placed on XCD x); a workgroup serves its
// own XCD's ids first, then the others'.  Returns the next id, or -1 once all eight counters have
// run out (every wave of every workgroup gets there).  Called by all threads of the workgroup; the
// barriers also separate two items' use of LDS.
__device__ __forceinline__ int lg_queue_take(int* __restrict__ queue, int nitems, int xcd, int* s_item) {
  __syncthreads();  // everyone is done with the previous item: its LDS, and *s_item
  if (threadIdx.x == 0) {
    int id = -1;
    for (int d = 0; d < 8 && id < 0; ++d) {
      const int x = (xcd + d) & 7;
      const int c = atomicAdd(queue + x, 1);
      if (c < (1 << 27) && 8 * c + x < nitems) id = 8 * c + x;
    }
    *s_item = id;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(*s_item);
}

// ------------------------------------------------- dk, dv: 64 keys per wave (D = 128)
// The main instance for D = 128.  Four waves of 64 keys each: every operand read from LDS (Q / dO
// rows, their transposed blocks) now feeds two matrix instructions, which halves the LDS traffic
// per product, the limit of the 32-keys-per-wave kernel above.  A wave then owns 256 accumulator
// registers (dk and dv of 64 keys x 128 dims); they live in the AGPR half of the register file
// for the whole kernel and only the matrix instructions touch them, while S / dP, which the
// vector unit has to read, use ordinary VGPRs.  The compiler picks one register form for all
// matrix instructions of a function, so the instructions are written out with their register
// classes here; that leaves their dependency waits, which the compiler otherwise provides, to
// this code (see the notes at lg_tie and in the step).
// COLUMN: the instance for the split-off column parts, as in the 32-keys-per-wave kernel: a virtual tile of
// four 64-key column groups, one group per wave, one chunk of the query range per workgroup,
// float32 atomics into the partial sums.
// bid: the work item, numbered like the block ids of the 32-keys-per-wave kernel's grid.
template <bool TOKEN, bool COLUMN>
__device__ __forceinline__ void dkdv_wide_item(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ dout, const float* __restrict__ nlse, const float* __restrict__ ndelta,
    uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int Hq, int Hkv, float scale, LgMask m_in,
    int nkt, int total, int run, const LgBwdWork& wk, const int bid) {
  LgMask m = m_in;
  if (TOKEN) {
    m.b = 1;
    m.stride = 0;
    m.bshift = 0;
    m.smask = -1;
    m.sb = m.sink;
    m.wb = m.window;
  }
  constexpr int D = 128;
  using T = LgSwzTile<D>;
  constexpr int NT = 256;
  using Dma = LgDma<D, NT>;
  constexpr int TQ = LG_BF16_BTQ, TK = LG_BF16_BTK;
  static_assert(TQ == 64 && TK == 256, "64 query rows per step, 4 waves x 64 keys");
  constexpr int DC = D / 16, DB = D / 32;
  constexpr int VRES = 4 * T::BYTES;                 // the workgroup's 256 V rows
  constexpr int OFF_G = T::BYTES, OFF_L = 2 * T::BYTES;
  constexpr int STAGE = 2 * T::BYTES + 1024;         // Q tile, dO tile, -lse / scale | -Delta (2 x 64 floats)
  __shared__ __attribute__((aligned(1024))) unsigned char smem[VRES + 2 * STAGE];

  const int G = Hq / Hkv;
  const float sl2 = scale * LOG2E;
  // (the thread index is made opaque per work item: what derives from it is recomputed for every item
  // instead of being kept in registers, or spilled, across the resident kernel's loop over items)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, g = lane >> 5;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  // work item: as in the kernel above
  int vt = 0, chunk = 0, gq = 0;
  LgBwdItem it = {0, 0, 0, 0, 0, wk.ncol};
  LgBwdMain w = {0, 0, 0};
  if (COLUMN) {
    // (the results of these divisions are pinned to scalar registers: the global->LDS copies take
    // their base addresses, which derive from them, as scalar operands)
    const int nh = wk.B * Hq;
    int x = bid;
    const int hd = x % nh;
    x /= nh;
    if (wk.seqs) {
      const int sq = lg_seq_of(wk.seqs->citem0, lg_uniform(wk.seqs->n), x);
      x -= lg_uniform(wk.seqs->citem0[sq]);
      it = lg_bwd_item(wk.seqs, sq, m);
    }
    const int nvt = (it.ncol + 3) / 4;
    vt = lg_uniform(x % nvt);
    chunk = lg_uniform(x / nvt);
    gq = lg_uniform(hd % G);
    w.bh = lg_uniform(hd / G);
  } else if (!lg_bwd_main(wk, bid, nkt, total, run, m, it, w)) {
    return;
  }
  const int bh = w.bh, kt = w.kt;
  const int N = m.N, ncol = it.ncol;
  const int* __restrict__ clist = wk.col_list + it.col0;
  const int b = bh / Hkv, hk = bh % Hkv;
  const int k0 = kt * TK, k1 = min(k0 + TK - 1, N - 1);
  const size_t kbase = ((size_t)(b * Hkv + hk) * m.ld + it.row0) * D;
  // this wave's 64 keys: a quarter of the key tile, or one column group of the virtual tile;
  // lane n holds keys kw0 + n and kw0 + 32 + n
  int kw0 = k0 + wave_s * 64;
  int col_gi = 0;        // COLUMN: index of this wave's column group
  bool active = true;    // COLUMN: the virtual tile may have fewer than 4 groups
  int r0_w = 0;          // COLUMN: first row of the wave's column part
  if (COLUMN) {
    col_gi = 4 * vt + wave_s;
    active = col_gi < ncol;
    const int grp = clist[min(col_gi, ncol - 1)];
    kw0 = 64 * grp;
    const int t1 = min((64 * grp / TK) * TK + TK - 1, N - 1);
    r0_w = (lg_qtile_window_hi(m, t1, TQ) + 1) * TQ;
  }
  const int j = kw0 + n;

  // accumulators: dk of key block kb, dim block db = block kb * 4 + db; dv = block 8 + kb * 4 + db
  bf16x8_t zero8 = lg_as_bf16x8(make_uint4(0u, 0u, 0u, 0u));
  // A matrix instruction must not read a register that a vector instruction wrote just before it
  // (the compiler spaces its own; an inline one that followed the write directly read stale lanes).
  asm volatile("s_nop 15" : "+v"(zero8));
#pragma unroll
  for (int i = 0; i < 16; ++i) lg_acc_zero(i, zero8);

  int lo, hi, hq0 = hk * G, nheads = 1;
  if (COLUMN) {
    // the query tiles of chunk number `chunk` (chunks are cut at fixed tile numbers for all virtual
    // tiles, counted from the chunk in which the first column part starts) that come after the
    // window part of the virtual tile's first group
    const int tf = min((64 * clist[0] / TK) * TK + TK - 1, N - 1);
    const int c_abs = (lg_qtile_window_hi(m, tf, TQ) + 1) / wk.chunk + chunk;
    const int grp0 = clist[4 * vt];
    const int t1 = min((64 * grp0 / TK) * TK + TK - 1, N - 1);
    lo = max(lg_qtile_window_hi(m, t1, TQ) + 1, c_abs * wk.chunk);
    hi = min((N - 1) / TQ, c_abs * wk.chunk + wk.chunk - 1);
    if (lo > hi) return;
    hq0 += gq;
  } else {
    int head0;
    lg_bwd_part_range(wk, m, ncol > 0, k0, k1, w.part, G, &lo, &hi, &head0, &nheads);
    hq0 += head0;
  }
  const int per_head = hi - lo + 1;
  const int steps = per_head * nheads;

  Dma dma;
  dma.init(tid);
  LgSwzReader<D> rd;
  rd.init(n, g);
  const uint32_t lds0 = (uint32_t)(uintptr_t)LG_LDS_PTR(unsigned char, smem);
  // K rows through the stages' place into registers, V rows resident
  static_assert(4 * T::BYTES <= 2 * STAGE, "K rows fit the stages");
#pragma unroll
  for (int kv = 0; kv < 2; ++kv)
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int r0 = COLUMN ? 64 * clist[min(4 * vt + x, ncol - 1)] : k0 + 64 * x;
      const int rc = min(r0, N - 1);  // a tile wholly past the end repeats the last row
      dma.issue((kv ? v : k) + kbase + (size_t)rc * D, r0 < N ? N - r0 : 1, lds0 + (kv ? 0 : VRES) + x * T::BYTES);
    }
  LG_WAIT_VMCNT(4 * Dma::CH);
  __syncthreads();
  bf16x8_t kf[2][DC];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) kf[kb][dc] = rd.read_rows(smem, VRES + wave_s * T::BYTES, kb, dc);
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) asm volatile("" ::"v"(kf[kb][dc]));
  __syncthreads();

  const int voff = wave * T::BYTES;  // this wave's 64 V rows
  const LgKeys wkeys = lg_keys(m, kw0, kw0 + 63);

  // rows of the query head whose step is requested next
  const uint16_t* qh = q + ((size_t)(b * Hq + hq0) * m.ld + it.row0) * D;
  const uint16_t* gh = dout + ((size_t)(b * Hq + hq0) * m.ld + it.row0) * D;
  const float* lh = nlse + (size_t)(b * Hq + hq0) * wk.wld + it.wrow0;
  const float* dh = ndelta + (size_t)(b * Hq + hq0) * wk.wld + it.wrow0;
  auto next_head = [&] {
    qh += (size_t)m.ld * D;
    gh += (size_t)m.ld * D;
    lh += wk.wld;
    dh += wk.wld;
  };
  auto issue_step = [&](int u, int buf) {
    const int q0 = u * TQ;
    const uint32_t st = lds0 + VRES + buf * STAGE;
    if (wave < 2) {  // wave 0: -lse / scale rows, wave 1: -Delta rows (64 floats each)
      const float* src = (wave == 0 ? lh : dh) + min(q0 + lane, N - 1);
      lg_dma_f32x64(src, st + OFF_L + wave * 256);
    }
    dma.issue(qh + (size_t)q0 * D, N - q0, st);
    dma.issue(gh + (size_t)q0 * D, N - q0, st + OFF_G);
  };

  const int u0 = per_head > 0 ? lo + (per_head - lo % per_head) % per_head : lo;  // rotated walk, as above
  int u_i = u0;
  int u_c = u0;
  int left_i = per_head;
  if (steps > 0) issue_step(u_i, 0);
  else LG_WAIT_VMCNT(0);  // (a part without rows: nothing may still be on its way to LDS when it ends)
  for (int st = 0; st < steps; ++st) {
    const int buf = st & 1;
    LG_WAIT_VMCNT(0);
    __syncthreads();  // step st landed for everyone; everyone is done with step st-1
    if (st + 1 < steps) {
      u_i = (u_i == hi) ? lo : u_i + 1;
      if (--left_i == 0) {
        left_i = per_head;
        u_i = u0;
        next_head();
      }
      issue_step(u_i, buf ^ 1);
    }
    const int q0 = u_c * TQ;
    u_c = (u_c == hi) ? lo : u_c + 1;
    if (COLUMN && (!active || q0 < r0_w)) continue;  // no group, or rows of its window part
    const int kind = lg_keys_kind(wkeys, q0, q0 + TQ - 1);
    if (kind == LG_TILE_DEAD) continue;
    const bool full = kind == LG_TILE_FULL;
    const int sq = VRES + buf * STAGE, sg = sq + OFF_G;
    const float* sL = reinterpret_cast<const float*>(smem + sq + OFF_L);
    // bit 16 qb + r of bits[kb]: pair (row of register r of query block qb, key j + 32 kb) is live
    uint32_t bits[2] = {~0u, ~0u};
    if (!full) {
      if (TOKEN) {
        // in tile coordinates (row = q0 + 4g + c): key j + 32 kb is seen by the rows c with
        // lo_c <= c < lo_c + window (no upper end for a sink key), below n_c
        const int n_c = N - q0 - 4 * g;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
          const int lo_c = j + 32 * kb - q0 - 4 * g;
          const long long end = j + 32 * kb < m.sink ? (long long)n_c : (long long)lo_c + m.window;
          bits[kb] = lg_reg_run(lo_c, (int)min(end, (long long)n_c));
        }
      } else {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) bits[kb] = lg_row_bits(m, j + 32 * kb, q0, g);
      }
    }
    auto dead = [&](int kb, int qb, int r) -> bool { return !((bits[kb] >> (qb * 16 + r)) & 1); };

    // One step = two 32-row query blocks (q) = 128 matrix instructions m, in pairs (units) that
    // share one operand read from LDS (one instruction for each key block); per block, m - 64 q:
    //    0..15  S  = Q K^T      16..31  dP = dO V^T      32..47  C: dV^T += dO^T P
    //   48..63  D: dK^T += Q^T dS
    // The instructions keep this order.  The LDS operand of unit u + DIST is requested before unit
    // u runs.  The vector work is cut into pieces of two elements (five instructions) and each
    // piece is placed after one matrix instruction, in whose shadow it then executes:
    //   22..29  P of rows h = 0 (both key blocks; S is final six instructions after its last one)
    //   32..39  P of rows h = 1           (C needs P of h = 0 from 32 on, of h = 1 from 40 on)
    //   40..47  dS of rows h = 0          (dP is final from 38 on; D needs dS of h = 0 from 48 on)
    //   48..55  dS of rows h = 1          (all vector work of a block ends before the next block's S)
    // S and dP start from the per-row values -lse / scale and -Delta (16 rows per lane, read from
    // LDS eight instructions before the chain starts), so P = exp2(c S') and dS = P dP'.
    f32x16_t sc[2], dp[2];
    uint32_t wP[2][2][4], wD[2][2][4];  // P / dS rounded to bf16, [key block][h][pair]
    constexpr int DIST = 2, NSL = DIST + 1;
    bf16x8_t ra[NSL], rv0[NSL], rv1[NSL];
    f32x16_t rowinit;
    auto row_init = [&](const float* base, int q) {  // register r <-> row 8 (r / 4) + 4g + r % 4 of block q
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const float4 x = *reinterpret_cast<const float4*>(base + q * 32 + 8 * r4 + 4 * g);
        rowinit[4 * r4 + 0] = x.x; rowinit[4 * r4 + 1] = x.y; rowinit[4 * r4 + 2] = x.z; rowinit[4 * r4 + 3] = x.w;
      }
    };
    auto reads = [&](int u) {  // u = 0..63: unit (m / 2) of the step
      const int sl = u % NSL, c = u & 7, q = u >> 5, ph = (u >> 3) & 3;
      if (ph == 0) {
        ra[sl] = rd.read_rows(smem, sq, q, c);
      } else if (ph == 1) {
        ra[sl] = rd.read_rows(smem, sg, q, c);
        rv0[sl] = rd.read_rows(smem, voff, 0, c);
        rv1[sl] = rd.read_rows(smem, voff, 1, c);
      } else if (ph == 2) {
        ra[sl] = rd.read_cols(smem, sg, c & 3, 2 * q + (c >> 2));  // dO^T, rows 32 q + 16 h ..
      } else {
        ra[sl] = rd.read_cols(smem, sq, c & 3, 2 * q + (c >> 2));  // Q^T
      }
    };
    // piece i (0..3) of (key block kb, half h): elements r = 8 h + 2 i, + 1
    auto sm_piece = [&](bool masked, int q, int kb, int h, int i) {
      const int r = 8 * h + 2 * i;
      float p0 = __builtin_amdgcn_exp2f(sc[kb][r] * sl2);
      float p1 = __builtin_amdgcn_exp2f(sc[kb][r + 1] * sl2);
      if (masked) {
        if (dead(kb, q, r)) p0 = 0.f;
        if (dead(kb, q, r + 1)) p1 = 0.f;
      }
      sc[kb][r] = p0;
      sc[kb][r + 1] = p1;
      wP[kb][h][i] = lg_pack_bf16(p0, p1);
    };
    auto ds_piece = [&](int kb, int h, int i) {
      const int r = 8 * h + 2 * i;
      wD[kb][h][i] = lg_pack_bf16(sc[kb][r] * dp[kb][r], sc[kb][r + 1] * dp[kb][r + 1]);
    };
    auto bop = [&](const uint32_t* w) { return lg_as_bf16x8(make_uint4(w[0], w[1], w[2], w[3])); };

    // two copies of the step: tiles that are live throughout skip the mask tests
    // Instruction numbers inside a 64-instruction block (see the table above): the chains' last
    // instructions, the anchors, and the first instruction after which each group of 8 pieces runs.
    constexpr int S_LAST = 15, DP_LAST = 31, C_FIRST = 32, D_FIRST = 48, NEXT_S = 64;
    constexpr int TIE_S = S_LAST + LG_MFMA_GAP, TIE_DP = DP_LAST + LG_MFMA_GAP;
    constexpr int P0 = 22, P1 = 32, DS0 = 40, DS1 = 48, NP = 8;  // P h0, P h1, dS h0, dS h1: NP pieces each
    static_assert(lg_readable_after(TIE_S, S_LAST) && P0 > TIE_S && P1 > TIE_S, "P reads S too early");
    static_assert(lg_readable_after(TIE_DP, DP_LAST) && DS0 > TIE_DP && DS1 > TIE_DP, "dS reads dP too early");
    static_assert(DS0 >= P0 + NP && DS1 >= P1 + NP, "dS of a half needs its P");
    // piece x of a group serves key block (x / 4) % 2; instruction C_FIRST + 8 h + 2 c' + kb reads the P of
    // (kb, h), D_FIRST + ... the dS: the last piece of key block 0 is number 3, of key block 1 number 7
    static_assert(lg_operand_ready(C_FIRST, P0 + 3) && lg_operand_ready(C_FIRST + 1, P0 + 7), "P (h0) late for dV");
    static_assert(lg_operand_ready(C_FIRST + 8, P1 + 3) && lg_operand_ready(C_FIRST + 9, P1 + 7), "P (h1) late for dV");
    static_assert(lg_operand_ready(D_FIRST, DS0 + 3) && lg_operand_ready(D_FIRST + 1, DS0 + 7), "dS (h0) late for dK");
    static_assert(lg_operand_ready(D_FIRST + 8, DS1 + 3) && lg_operand_ready(D_FIRST + 9, DS1 + 7), "dS (h1) late for dK");
    static_assert(DS1 + NP <= NEXT_S, "the vector work of a block ends before the next block's S overwrites it");
    auto run_step = [&](auto MASKED) {
    constexpr bool masked = decltype(MASKED)::value;
    __builtin_amdgcn_sched_barrier(0);
    row_init(sL, 0);
    lg_static_for<DIST>([&](auto U) { reads(decltype(U)::value); });
    lg_static_for<128>([&](auto M) {
      constexpr int m = decltype(M)::value;
      constexpr int u = m >> 1, kb = m & 1, sl = u % NSL, c = u & 7, q = m >> 6, mm = m & 63, ph = mm >> 4;
      if (kb == 0 && u + DIST < 64) reads(u + DIST);
      if (ph == 0) {
        if (c == 0) lg_mfma_vi(sc[kb], ra[sl], kf[kb][c], rowinit);
        else lg_mfma_v(sc[kb], ra[sl], kf[kb][c]);
      } else if (ph == 1) {
        if (c == 0) lg_mfma_vi(dp[kb], ra[sl], kb ? rv1[sl] : rv0[sl], rowinit);
        else lg_mfma_v(dp[kb], ra[sl], kb ? rv1[sl] : rv0[sl]);
      } else if (ph == 2) {
        lg_acc_fma(8 + 4 * kb + (c & 3), ra[sl], bop(wP[kb][c >> 2]));
      } else {
        lg_acc_fma(4 * kb + (c & 3), ra[sl], bop(wD[kb][c >> 2]));
      }
      if (mm == TIE_S) lg_tie(sc[0], sc[1]);
      if (mm == TIE_DP) lg_tie(dp[0], dp[1]);
      if (mm == 8) row_init(sL + 64, q);             // -Delta rows: dP starts at 16
      if (m == 56) row_init(sL, 1);                  // -lse / scale rows of the second block
      __builtin_amdgcn_sched_barrier(0);  // the piece follows its matrix instruction
      // pieces: P h0 at 22..29, P h1 at 32..39, dS h0 at 40..47, dS h1 at 48..55; key block = bit 2
      if (mm >= P0 && mm < P0 + NP) sm_piece(masked, q, ((mm - P0) >> 2) & 1, 0, (mm - P0) & 3);
      if (mm >= P1 && mm < P1 + NP) sm_piece(masked, q, ((mm - P1) >> 2) & 1, 1, (mm - P1) & 3);
      if (mm >= DS0 && mm < DS0 + NP) ds_piece(((mm - DS0) >> 2) & 1, 0, (mm - DS0) & 3);
      if (mm >= DS1 && mm < DS1 + NP) ds_piece(((mm - DS1) >> 2) & 1, 1, (mm - DS1) & 3);
      __builtin_amdgcn_sched_barrier(0);
    });
    };
    if (full) run_step(std::false_type{});
    else run_step(std::true_type{});
  }

  // the last matrix results must have landed before the blocks are copied out
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  using Slot = LgSlot<D>;
  unsigned char* rows = smem + voff;  // (its V rows' place: no other wave reads them)
  const bool cut = !COLUMN && wk.heads_cut * wk.rows_cut > 1;
  if (COLUMN && !active) return;
  float* slot = (cut ? lg_bwd_part_slot<D>(wk, it, w, total / nkt) + wave_s * Slot::FLOATS
                     : wk.colpart + ((size_t)bh * wk.ncol + it.col0 + col_gi) * Slot::FLOATS) + lane;
  const int cid = (!COLUMN && !cut && ncol > 0 && kw0 < N) ? wk.col_of_group[it.grp0 + (kw0 >> 6)] : -1;
  const float* csum = wk.colpart + ((size_t)bh * wk.ncol + it.col0 + max(cid, 0)) * Slot::FLOATS + lane;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    float c[2 * DB][16];  // the column part's sums, all of a key block in flight at once
    if (cid >= 0)
#pragma unroll
      for (int x = 0; x < 2 * DB; ++x)
#pragma unroll
        for (int r = 0; r < 16; ++r) c[x][r] = lg_load_shared1(csum + Slot::at(kb, x & 1, x >> 1) + 64 * r);
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      float akv[16], avv[16];
      lg_acc_get(kb * 4 + db, akv);
      lg_acc_get(8 + kb * 4 + db, avv);
      float* pk = slot + Slot::at(kb, 0, db);
      float* pv = slot + Slot::at(kb, 1, db);
      if (COLUMN) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          unsafeAtomicAdd(pk + 64 * r, akv[r]);  // hardware float adds
          unsafeAtomicAdd(pv + 64 * r, avv[r]);
        }
      } else if (cut) {  // bwd_fold_kernel adds the parts
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          pk[64 * r] = akv[r];
          pv[64 * r] = avv[r];
        }
      } else {
        if (cid >= 0)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            akv[r] += c[2 * db][r];
            avv[r] += c[2 * db + 1][r];
          }
        lg_rows_put<D>(rows, lane, db, akv, scale);
        lg_rows_put<D>(rows + 32 * T::ROW_BYTES, lane, db, avv, 1.f);
      }
    }
    if (!COLUMN && !cut) {
      lg_rows_write<D>(rows, lane, dk + kbase + (size_t)(kw0 + 32 * kb) * D, N - (kw0 + 32 * kb));
      lg_rows_write<D>(rows + 32 * T::ROW_BYTES, lane, dv + kbase + (size_t)(kw0 + 32 * kb) * D, N - (kw0 + 32 * kb));
    }
  }
}

// The column instance: one workgroup per work item.
template <bool TOKEN, bool COLUMN>
__global__ __launch_bounds__(256) void dkdv_wide_bf16_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ dout, const float* __restrict__ nlse, const float* __restrict__ ndelta,
    uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int Hq, int Hkv, float scale, LgMask m,
    int nkt, int total, int run, LgBwdWork wk) {
  dkdv_wide_item<TOKEN, COLUMN>(q, k, v, dout, nlse, ndelta, dk, dv, Hq, Hkv, scale, m, nkt, total, run, wk,
                                (int)blockIdx.x);
}

// The main instance: a workgroup holds a whole CU (4 x 512 registers, 130 KB of LDS), so the launch of
// the next one cannot overlap anything.  One workgroup per CU therefore stays and takes work items
// from a queue (lg_queue_take).
template <bool TOKEN>
__global__ __launch_bounds__(256) void dkdv_wide_bf16_kernel_q(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ dout, const float* __restrict__ nlse, const float* __restrict__ ndelta,
    uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int Hq, int Hkv, float scale, LgMask m,
    int nkt, int total, int run, LgBwdWork wk, int* __restrict__ queue, int nitems) {
  __shared__ int s_item;
  const int xcd = blockIdx.x & 7;
  for (;;) {
    const int id = lg_queue_take(queue, nitems, xcd, &s_item);
    if (id < 0) return;
    dkdv_wide_item<TOKEN, false>(q, k, v, dout, nlse, ndelta, dk, dv, Hq, Hkv, scale, m, nkt, total, run, wk, id);
  }
}

// ------------------------------------------------- dq: 64 query rows per wave (D = 128)
// Same idea as the wide dk/dv kernel: four waves of 64 query rows, so that every K / V operand
// read from LDS feeds two matrix instructions; same tile walk as the 32-rows-per-wave kernel, a 4-stage ring
// used as two pairs of tiles with one barrier per pair.  The AGPR half of the register file holds the dq
// accumulators (blocks 0..7 = a[0:127]: row block rb, dim block db -> block 4 rb + db) and the
// wave's Q and dO fragments (a[128:255], four registers per 32 rows x 16 dims), which the matrix
// instructions read as their second operand straight from there.
// bid: the work item, numbered like the block ids of the 32-rows-per-wave kernel's grid.
template <bool TOKEN>
__device__ __forceinline__ void dq_wide_item(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ out, const uint16_t* __restrict__ dout, const float* __restrict__ lse,
    float* __restrict__ ndelta, float* __restrict__ nlse, uint16_t* __restrict__ dq, int Hq, int Hkv, float scale,
    LgMask m_in, int nqt, int total, int run, const LgBwdWork& wk, const int bid) {
  LgMask m = m_in;
  if (TOKEN) {
    m.b = 1;
    m.stride = 0;
    m.bshift = 0;
    m.smask = -1;
    m.sb = m.sink;
    m.wb = m.window;
  }
  constexpr int D = 128;
  using T = LgSwzTile<D>;
  constexpr int NT = 256, STAGES = 4;
  using Dma = LgDma<D, NT>;
  constexpr int TQ = LG_BF16_TQ, TK = LG_BF16_TK;
  static_assert(TQ == 256 && TK == 64, "4 waves x 64 query rows, 64-key tiles");
  constexpr int DC = D / 16, DB = D / 32;
  constexpr int STAGE = 2 * T::BYTES;  // K tile + V tile
  __shared__ __attribute__((aligned(1024))) unsigned char smem[STAGES * STAGE];
  __shared__ float s_rows[2][TQ];  // Delta, log-sum-exp

  const int L = lg_item_of(bid, run);
  if (L >= total) return;
  const int G = Hq / Hkv;
  const int gq = L % G, rest = L / G;
  int qt = nqt - 1 - (rest % nqt);
  const int bhk = rest / nqt;
  const int b = bhk / Hkv, hk = bhk % Hkv;
  const int hq = hk * G + gq;
  int srow = 0, swrow = 0;  // packed: first row of the sequence inside its head, in the workspace
  if (wk.seqs) {
    const int t = wk.qt_first + rest % nqt;
    const int sq = lg_seq_of(wk.seqs->qtile0, lg_uniform(wk.seqs->n), t);
    qt = lg_uniform(wk.seqs->qtile0[sq + 1]) - 1 - t;
    srow = lg_uniform(wk.seqs->row0[sq]);
    swrow = lg_uniform(wk.seqs->wrow0[sq]);
    m = lg_mask_for_length(m, lg_uniform(wk.seqs->len[sq]));
  }
  const int N = m.N;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, g = lane >> 5;
  const int q0 = qt * TQ, q1 = min(q0 + TQ - 1, N - 1);
  const size_t row0 = (size_t)(b * Hq + hq) * m.ld + srow;       // the sequence's first row in this query head
  const size_t wrow0 = (size_t)(b * Hq + hq) * wk.wld + swrow;   // the same in the workspace
  const size_t qbase = row0 * D;
  const uint16_t* kh = k + ((size_t)(b * Hkv + hk) * m.ld + srow) * D;
  const uint16_t* vh = v + ((size_t)(b * Hkv + hk) * m.ld + srow) * D;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int qw0 = min(q0 + wave_s * 64, N - 1), qw1 = min(q0 + wave_s * 64 + 63, N - 1);  // this wave's rows
  const int i0 = q0 + wave * 64 + n;  // this lane's row of row block 0 (block 1: + 32)

  // Q and dO rows through the ring's place into fragments: Q of (rb, dc) -> fragment 8 rb + dc, dO -> 16 + 8 rb + dc
  Dma dma;
  dma.init(tid);
  LgSwzReader<D> rd;
  rd.init(n, g);
  const uint32_t lds0 = (uint32_t)(uintptr_t)LG_LDS_PTR(unsigned char, smem);
#pragma unroll
  for (int y = 0; y < 2; ++y)
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int rc = min(q0 + 64 * x, N - 1);  // a tile wholly past the end repeats the last row
      dma.issue((y ? q : dout) + qbase + (size_t)rc * D, N - rc, lds0 + (4 * y + x) * T::BYTES);
    }
  const float my_lse = lse[row0 + min(q0 + tid, N - 1)];
  const LgQSched qs = lg_qsched_init(m, q0, q1);
  const LgRows wrows = lg_rows(m, qw0, qw1);
  const LgQWalk qw = lg_qwalk_init(qs);
  auto next_tile = [&](int prev) -> int {
    if (TOKEN || m.stride == 0) return prev < 0 ? lg_qwalk_first(qw) : lg_qwalk_next(qw, prev);
    return lg_qsched_next(m, qs, prev);
  };
  int t = next_tile(-1);  // (while the rows are on their way)
  {
    uint4 o[16];
    lg_load_pieces<D, TQ>(out + qbase + (size_t)q0 * D, N - 1 - q0, o);
    LG_WAIT_VMCNT(0);
    __syncthreads();
    lg_delta_rows<D, TQ>(smem, o, s_rows[0]);
    s_rows[1][tid] = my_lse;
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    bf16x8_t f[DC];  // (all of a row block's reads in flight at once)
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) f[dc] = rd.read_rows(smem, ((x < 2 ? 0 : 4) + wave_s) * T::BYTES, x & 1, dc);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) lg_frag_set((x < 2 ? 16 : 0) + 8 * (x & 1) + dc, __builtin_bit_cast(uint4, f[dc]));
  }
  __syncthreads();
  auto issue = [&](int t, int stage) {
    const size_t off = (size_t)t * TK * D;
    dma.issue(kh + off, N - t * TK, lds0 + stage * STAGE);
    dma.issue(vh + off, N - t * TK, lds0 + stage * STAGE + T::BYTES);
  };
  // Tiles are handled in pairs: one barrier per two tiles (with one wave per SIMD nothing hides the
  // wait for the slowest wave, so fewer barriers matter more than a deeper ring).  Pair p lives in
  // stages 2 (p % 2), + 1; at its start the loads of pair p + 1 go into the other two stages.
  int t_issue = t;
  for (int x = 0; x < 2 && t_issue >= 0; ++x) {
    issue(t_issue, x);
    t_issue = next_tile(t_issue);
  }
  float lse2[2];
  f32x16_t ndl[2];  // -Delta of the lane's row in all 16 registers: the addend dP^T starts from
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    const int row = wave * 64 + 32 * rb + n;
    lse2[rb] = s_rows[1][row] * LOG2E;
    const float di = s_rows[0][row];
#pragma unroll
    for (int r = 0; r < 16; ++r) ndl[rb][r] = -di;
  }
  const float sl2 = scale * LOG2E;
  asm volatile("" : "+v"(lse2[0]), "+v"(lse2[1]), "+v"(ndl[0]), "+v"(ndl[1]));
  {  // The rows' -Delta and -lse / scale for the dk/dv kernels.  Every thread stores, without a branch: those past the end
     // hold (and store) the values of row N - 1, whose data they loaded.
    const size_t row = wrow0 + min(q0 + tid, N - 1);
    ndelta[row] = -s_rows[0][tid];
    nlse[row] = -my_lse * (1.f / scale);
  }
  bf16x8_t zero8 = lg_as_bf16x8(make_uint4(0u, 0u, 0u, 0u));
  asm volatile("s_nop 15" : "+v"(zero8));  // as in the dk/dv kernel: written well before it is read
#pragma unroll
  for (int x = 0; x < 8; ++x) lg_acc_zero(x, zero8);

  int stage = 0;
  while (t >= 0) {
    if ((stage & 1) == 0) {
      LG_WAIT_VMCNT(0);
      __syncthreads();  // this pair landed for everyone; everyone is done with the previous pair
#pragma unroll
      for (int x = 0; x < 2; ++x)
        if (t_issue >= 0) {
          issue(t_issue, (stage + 2 + x) % STAGES);
          t_issue = next_tile(t_issue);
        }
    }
    const int k0 = t * TK;
    int kind = LG_TILE_FULL;
    if (!lg_qsched_full(m, qs, t)) kind = lg_rows_kind(m, wrows, k0, k0 + TK - 1);
    const int sk = stage * STAGE, sv = sk + T::BYTES;
    t = next_tile(t);
    stage = (stage + 1) % STAGES;
    if (kind == LG_TILE_DEAD) continue;
    // bit 16 kb + r of bits[rb]: pair (row i0 + 32 rb, key of register r of key block kb) is live
    uint32_t bits[2] = {~0u, ~0u};
    if (kind == LG_TILE_PARTIAL) {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        const int i = i0 + 32 * rb;
        uint32_t w = 0;
        if (TOKEN) {
          // key = k0 + 4g + c: live if inside the window of row i, or a sink key not after i
          const int hi = i - k0 - 4 * g, lo = hi - (m.window - 1), se = m.sink - k0 - 4 * g;
          w = lg_reg_run(lo, hi + 1) | lg_reg_run(-1, min(se, hi + 1));
        } else {
          w = lg_key_bits(m, min(i, N - 1), k0, g);
        }
        bits[rb] = w;
      }
    }
    auto dead = [&](int rb, int kb, int r) -> bool { return !((bits[rb] >> (kb * 16 + r)) & 1); };

    // One tile = 96 matrix instructions mi, in pairs (units) that share one operand read from LDS
    // (one instruction for each 32-row block rb):
    //    0..15  S^T(0) = K Q^T    16..31  dP^T(0) = V dO^T    32..47  S^T(1)    48..63  dP^T(1)
    //   64..79  E(0): dQ^T += K^T dS^T(0)                     80..95  E(1)
    // (0), (1): key block of the tile.  S / dP of the two key blocks use separate registers, so the
    // vector work of key block 0 runs under the instructions of key block 1, two elements after
    // each instruction:  P(0) 22..37,  dS(0) 38..53,  P(1) 54..69,  dS(1) 70..85 (rows h = 0 of
    // both row blocks first: E(1) needs them from 80 on, h = 1 from 88 on).
    f32x16_t sc[2][2], dp[2][2];   // [key block][row block]
    uint32_t wD[2][2][2][4];       // dS rounded to bf16: [key block][row block][h][pair]
    constexpr int DIST = 2, NSL = DIST + 1;
    bf16x8_t ra[NSL];
    auto reads = [&](int u) {  // u = 0..47: unit (mi / 2) of the tile
      const int sl = u % NSL, c = u & 7, ph = u >> 3;
      if (ph == 0 || ph == 2) ra[sl] = rd.read_rows(smem, sk, ph >> 1, c);
      else if (ph == 1 || ph == 3) ra[sl] = rd.read_rows(smem, sv, ph >> 1, c);
      else ra[sl] = rd.read_cols(smem, sk, c & 3, 2 * (ph - 4) + (c >> 2));
    };
    // piece x (0..15) of key block kb: row block (x / 4) % 2, h = x / 8, elements 8 h + 2 (x % 4), + 1
    auto p_piece = [&](bool masked, int kb, int x) {
      const int rb = (x >> 2) & 1, r = 8 * (x >> 3) + 2 * (x & 3);
      float p0 = __builtin_amdgcn_exp2f(fmaf(sc[kb][rb][r], sl2, -lse2[rb]));
      float p1 = __builtin_amdgcn_exp2f(fmaf(sc[kb][rb][r + 1], sl2, -lse2[rb]));
      if (masked) {
        if (dead(rb, kb, r)) p0 = 0.f;
        if (dead(rb, kb, r + 1)) p1 = 0.f;
      }
      sc[kb][rb][r] = p0;
      sc[kb][rb][r + 1] = p1;
    };
    auto ds_piece = [&](int kb, int x) {
      const int rb = (x >> 2) & 1, h = x >> 3, r = 8 * h + 2 * (x & 3);
      wD[kb][rb][h][x & 3] = lg_pack_bf16(sc[kb][rb][r] * dp[kb][rb][r], sc[kb][rb][r + 1] * dp[kb][rb][r + 1]);
    };
    auto bop = [&](const uint32_t* w) { return lg_as_bf16x8(make_uint4(w[0], w[1], w[2], w[3])); };

    // Instruction numbers of the tile (see the table above): last instruction of each chain, anchors, first
    // instruction after which each group of 16 pieces runs.
    constexpr int S0_LAST = 15, DP0_LAST = 31, S1_LAST = 47, DP1_LAST = 63, E0_FIRST = 64, E1_FIRST = 80;
    constexpr int TIE_S0 = S0_LAST + LG_MFMA_GAP, TIE_DP0 = DP0_LAST + LG_MFMA_GAP, TIE_S1 = S1_LAST + LG_MFMA_GAP,
                  TIE_DP1 = DP1_LAST + LG_MFMA_GAP;
    constexpr int PP0 = 22, DSS0 = 38, PP1 = 54, DSS1 = 70, NPC = 16;
    static_assert(lg_readable_after(TIE_S0, S0_LAST) && PP0 > TIE_S0, "P(0) reads S too early");
    static_assert(lg_readable_after(TIE_DP0, DP0_LAST) && DSS0 > TIE_DP0 && DSS0 >= PP0 + NPC, "dS(0) too early");
    static_assert(lg_readable_after(TIE_S1, S1_LAST) && PP1 > TIE_S1, "P(1) reads S too early");
    static_assert(lg_readable_after(TIE_DP1, DP1_LAST) && DSS1 > TIE_DP1 && DSS1 >= PP1 + NPC, "dS(1) too early");
    // pieces 0..7 of a dS group are h = 0 (both row blocks), 8..15 are h = 1; E(kb) reads h = 0 in its first
    // eight instructions and h = 1 in its last eight
    static_assert(lg_operand_ready(E0_FIRST, DSS0 + 7) && lg_operand_ready(E0_FIRST + 8, DSS0 + 15), "dS(0) late for dQ");
    static_assert(lg_operand_ready(E1_FIRST, DSS1 + 7) && lg_operand_ready(E1_FIRST + 8, DSS1 + 15), "dS(1) late for dQ");
    auto run_tile = [&](auto MASKED) {
      constexpr bool masked = decltype(MASKED)::value;
      __builtin_amdgcn_sched_barrier(0);
      lg_static_for<DIST>([&](auto U) { reads(decltype(U)::value); });
      lg_static_for<96>([&](auto M) {
        constexpr int mi = decltype(M)::value;
        constexpr int u = mi >> 1, rb = mi & 1, sl = u % NSL, c = u & 7, ph = u >> 3;
        if (rb == 0 && u + DIST < 48) reads(u + DIST);
        constexpr int kb = ph < 4 ? ph >> 1 : ph - 4;  // key block of the unit
        if (ph == 0 || ph == 2) lg_frag_mfma(8 * rb + c, c == 0, sc[kb][rb], ra[sl]);
        else if ((ph == 1 || ph == 3) && c == 0) lg_frag_mfma_init(16 + 8 * rb, dp[kb][rb], ra[sl], ndl[rb]);
        else if (ph == 1 || ph == 3) lg_frag_mfma(16 + 8 * rb + c, false, dp[kb][rb], ra[sl]);
        else lg_acc_fma(4 * rb + (c & 3), ra[sl], bop(wD[kb][rb][c >> 2]));
        // S / dP are final six matrix instructions after their last one
        if (mi == TIE_S0) lg_tie(sc[0][0], sc[0][1]);
        if (mi == TIE_DP0) lg_tie(dp[0][0], dp[0][1]);
        if (mi == TIE_S1) lg_tie(sc[1][0], sc[1][1]);
        if (mi == TIE_DP1) lg_tie(dp[1][0], dp[1][1]);
        __builtin_amdgcn_sched_barrier(0);  // the piece follows its matrix instruction
        if (mi >= PP0 && mi < PP0 + NPC) p_piece(masked, 0, mi - PP0);
        if (mi >= DSS0 && mi < DSS0 + NPC) ds_piece(0, mi - DSS0);
        if (mi >= PP1 && mi < PP1 + NPC) p_piece(masked, 1, mi - PP1);
        if (mi >= DSS1 && mi < DSS1 + NPC) ds_piece(1, mi - DSS1);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    if (kind == LG_TILE_FULL) run_tile(std::false_type{});
    else run_tile(std::true_type{});
  }

  // the last matrix results must have landed before the blocks are copied out
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  // (into the stages of the pair before the last one, which everyone is done with)
  unsigned char* rows = smem + (((stage + 1) / 2 * 2) % STAGES) * STAGE + wave_s * (64 * T::ROW_BYTES);
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      float a[16];
      lg_acc_get(4 * rb + db, a);
      lg_rows_put<D>(rows + rb * (32 * T::ROW_BYTES), lane, db, a, scale);
    }
    const int r0 = q0 + wave_s * 64 + 32 * rb;
    lg_rows_write<D>(rows + rb * (32 * T::ROW_BYTES), lane, dq + qbase + (size_t)r0 * D, N - r0);
  }
}

// One resident workgroup per CU that takes its work items from a queue, as the dk/dv kernel above.
template <bool TOKEN>
__global__ __launch_bounds__(256) void dq_wide_bf16_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ out, const uint16_t* __restrict__ dout, const float* __restrict__ lse,
    float* __restrict__ ndelta, float* __restrict__ nlse, uint16_t* __restrict__ dq, int Hq, int Hkv, float scale,
    LgMask m, int nqt, int total, int run, LgBwdWork wk, int* __restrict__ queue, int nitems) {
  __shared__ int s_item;
  const int xcd = blockIdx.x & 7;
  for (;;) {
    const int id = lg_queue_take(queue, nitems, xcd, &s_item);
    if (id < 0) return;
    dq_wide_item<TOKEN>(q, k, v, out, dout, lse, ndelta, nlse, dq, Hq, Hkv, scale, m, nqt, total, run, wk, id);
  }
}

}  // namespace

namespace {

// The column groups of a sequence and the query tiles of their column parts.
struct Columns {
  int ncol;         // column groups
  int first, last;  // query tiles of the first group's column part, the longest
  // A lone group: its chunks, up to 8 and not below 8 pairs of tiles each; up to 16 heads, and with head dim 64, whose items take a
  // tile at a time, up to 16 (up to 16 heads of 64: 4 pairs).  By the sequence and its heads alone.  Backward in us, 8 : this, 8
  // heads of 64, 37511 tokens, window 600 268 : 241, 4 of 128 198 : 170; 32 of 64, window 128 503 : 493, but 2 x 32, window 300 1286 :
  // 1308.  Down to a pair each, 16 x 8 of 128, 3500 tokens 412 : 476.
  int lone(int D, int Hq) const {
    const int pairs = (last - first + 2) / 2, each = Hq <= 16 && D == 64 ? 4 : 8;
    return ncol != 1 ? 0 : std::min(std::max(pairs / each, 1), Hq <= 16 || D == 64 ? 16 : 8);
  }
  // ... with groups of G query heads and `heads` of them in all: more where that leaves CUs idle, not below a pair, up to 64 adders
  int lone_of_groups(int G, long long heads) const {
    const int pairs = (last - first + 2) / 2;
    return ncol != 1 ? 0 : std::max(lone(128, 64), (int)std::min<long long>({pairs, 64 / G, (256 + heads - 1) / heads}));
  }
  // several: work items (virtual tile x chunk) of a query head; chunks are cut at multiples of `chunk` tiles
  int items(int D, int chunk) const {
    const int ng = btk_of(D) / 64;
    return ncol < 2 ? 0 : (ncol + ng - 1) / ng * (last / chunk - first / chunk + 1);
  }
};
Columns columns_of(const LgMask& m, int D) {
  const int btk = btk_of(D);
  Columns c = {0, 0, 0};
  int first = -1;
  for (int grp = 0; grp < (m.N + 63) / 64; ++grp)
    if (lg_is_column_group(m, grp, btk, LG_BF16_BTQ)) {
      if (first < 0) first = grp;
      ++c.ncol;
    }
  if (c.ncol > 0) {
    const int t0 = first * 64 / btk * btk;
    const int t1 = t0 + btk - 1 < m.N - 1 ? t0 + btk - 1 : m.N - 1;
    c.first = lg_qtile_window_hi(m, t1, LG_BF16_BTQ) + 1;
    c.last = (m.N - 1) / LG_BF16_BTQ;
    if (c.ncol == 1 && c.last - c.first < 6) c.ncol = 0;  // a short one stays with its key tile
  }
  return c;
}

// Which kernels a sequence takes: the 64-rows-per-wave forms (head dim 128) start up and drain slower, so they
// need a number of steps per workgroup.
// dq: by the key tiles of an average query tile: its window, plus the strided columns below it.  In short runs the 32-rows
// form is the faster one up to 40 tiles (64/8 heads, 16001 tokens, window 2048 and strided columns 1415 : 1471 us), in long
// ones, at the power limit, what it draws more slows the kernels beside it (that whole training pass 4575 : 4515 us; 32
// heads, 32768 tokens, window 2048 4625 : 4619, 1100 2974 : 3017).  And only with enough work items of 256 rows, which at one
// per CU end one after the other (dq, causal, 64 rows per wave : 32; 4 heads, 6000 tokens 197 : 154, 24000 918 : 794; 12 heads,
// 7800 338 : 275; 16, 6000 (384 items) 225 : 228; 8/2, 12000 425 : 454).  Counted for one sequence, so that its dq has the same
// bits in every batch and pack; a batch has more work items, and what that costs it is: 2 x 4 heads, 16384 tokens 636 : 734 (the
// backward 1461 : 1561), 3 x 8/2, 10200 848 : 907, 8 x 4, 16384 2660 : 2700 (5975 : 6035), but 3 x 4, 20400 1735 : 1621, 4 x 16, 4096
// 410 : 369.
bool dq_wide(const LgMask& m, int D, int Hq) {
  const int col_tiles = m.stride > 0 ? (m.N / 2) / (m.b * m.stride) * ((m.b + LG_BF16_TK - 1) / LG_BF16_TK) : 0;
  return D == 128 && (m.wb * m.b + LG_BF16_TQ) / LG_BF16_TK + col_tiles >= 32 &&
         (long long)Hq * ((m.N + LG_BF16_TQ - 1) / LG_BF16_TQ) >= 384;
}
// dk/dv: by the query tiles of a key tile's window part
bool dkdv_wide(const LgMask& m, int D) { return D == 128 && (m.wb * m.b + LG_BF16_BTK) / LG_BF16_BTQ >= 16; }

constexpr int CUS = 256;  // compute units the cuts below are made for (they also decide the workspace's size)

// How the window parts are cut: heads x rows work items per key tile and kv head.
struct Cut {
  int heads, rows;
};
// Few key tiles leave the chip idle: each is one workgroup that walks its window part for every query head of the
// group.  They are cut so that the longest work item, or all of them over the CUs, takes least.  Measured: a query tile
// takes 3 us, starting an item 8 (head dim 64, three workgroups per CU: 1.5 and 8 for one, 1 and 3 for each of many), the
// pass that adds the parts 4 TB/s.  Only with groups of query heads or strided columns: elsewhere dk and dv do not
// depend on what else a launch holds.
//   nbh: b x kv heads; tiles: key tiles of a head; steps, longest: query tiles of all of a head's key tiles, and the most
//   of one; most: parts of a key tile that the workspace has room for; ndq: dq's work items, -1: not in a launch with dk/dv
// Where dq shares the launch, its items take as many rounds as dk/dv's, and more parts gain less than their sum takes: head dim 128
// then counts 2 us for a query tile, dq's as well, 3 TB/s for the sum, and does not ask for a tenth, up to three work items per CU
// before the cut (beyond that the launch may be cut in two: 4 x 16/2 heads, 4910 tokens, causal, 1440 items 1240 -> 1420).  23 shapes
// with groups, all cuts timed: the former rule's were 5.8 % from the best one (geometric mean), these 2.4.  Backward in us: 32/8
// heads, 1807 tokens, window 252 89.0 -> 79.9, 2 x 32/8, 370 43.1 -> 36.8, 4 x 16/2, 1786, causal 222 -> 209, 2 packed of up to 483,
// 64/8 64.4 -> 59.4; the least: 2/1, 1240, every 8th block 54.0 -> 55.6.  (Head dim 64: 5.2 % with the former rule, 6.0 with the best
// of this form.)  Parts of more than 200 query tiles, or of more than 64 with more than two work items per CU, outlast the others
// where they start late: half an average one is added to the rounds.  Without that and with it (and launches of their own): 16/8
// heads, 5529 tokens, window 4096 419, 398 (398), 4/1, 24000, causal 1936, 1821 (1835), 2/1, 48450, causal 3891, 3723 (3714); for all
// parts of more than 64 4/2, 16450, window 4096 would go from 418 to 466.  375 shapes with groups or strided columns are 1.317 times as
// fast as with launches of their own (geometric mean; without it 1.316, with the best cuts 1.355); slower are 9/3, 6407, window 500
// 96 : 99, 16/8, 5529, causal 426 : 437, 7450, window 1500 342 : 351, 4/2, 24200, causal 1844 : 1860.
Cut choose_cut(int D, int G, int nbh, size_t tiles, double steps, int longest, size_t most, long long ndq) {
  const double items = (double)tiles * nbh;
  const bool shared = D == 128 && ndq >= 0 && ndq + items <= 3 * CUS;
  const bool late = shared && (longest > 200 || (longest > 64 && ndq + items > 2 * CUS));  // items that start late end the launch alone
  const double each1 = shared ? 2.0 : D == 128 ? 3.0 : 1.5, each = shared ? 4.0 : D == 128 ? 3.0 : 1.0, start = D == 128 ? 8 : 3;
  Cut best = {1, 1};
  double least = 0;
  for (int heads = 1; heads <= G; ++heads) {
    if (G % heads) continue;
    for (int rows = 1; rows <= 8 && rows <= longest; ++rows) {
      const double parts = heads * rows;
      if (parts > 1 && (items * parts > (D == 128 ? 4 : 8) * CUS || parts > most)) break;
      const double one = (double)(G / heads) * ((longest + rows - 1) / rows) * each1 + (shared ? 4 : 8);
      const double all = (steps * G * nbh * each + items * parts * start) / CUS;
      const double fold = parts > 1 ? 5 + items * parts * (btk_of(D) * D * 8.0) / (shared ? 3e6 : 4e6) : 0;
      const double tail = late ? 0.5 * ((double)(G / heads) * steps / tiles / rows * each1 + 4) : 0;
      const double t = (one > all + tail ? one : all + tail) + fold;
      const bool level = shared && t == least && parts <= best.heads * best.rows;  // (of two alike the one of more heads)
      if (parts == 1 || t < (shared ? 1.0 : 0.9) * least || level) {
        least = t;
        best = {heads, rows};
      }
    }
  }
  return best;
}
bool may_cut(const LgShape& sh, bool strided, size_t items) {
  return (sh.Hq != sh.Hkv || strided) && items <= (sh.D == 128 ? 2 : 4) * CUS;
}
constexpr size_t MOST_PARTS = 8 * CUS;  // where the workspace is made for the cut: no limit
// query tiles of the window parts of a sequence's key tiles
void window_steps(const LgMask& m, int btk, double* steps, int* longest) {
  for (int k0 = 0; k0 < m.N; k0 += btk) {
    const int k1 = k0 + btk - 1 < m.N - 1 ? k0 + btk - 1 : m.N - 1;
    const int len = lg_qtile_window_hi(m, k1, LG_BF16_BTQ) - k0 / LG_BF16_BTQ + 1;  // (close enough without a split)
    *steps += len;
    *longest = len > *longest ? len : *longest;
  }
}

// The workspace of one set of launches.
struct BwdSize {
  size_t seqs = 0;    // sequences (the batch: 1)
  size_t rows = 0;    // tokens of a head
  size_t ktiles = 0;  // key tiles of a head
  size_t groups = 0;  // 64-key groups of a head
  size_t ncol = 0;    // split-off column groups of a head
  size_t lone = 0;    // chunks of lone groups
  void add(int n, int D, int Hq, const Columns& c) {
    ++seqs;
    rows += n;
    ktiles += (n + btk_of(D) - 1) / btk_of(D);
    groups += (n + 63) / 64;
    ncol += c.ncol;
    lone += c.lone(D, Hq);
  }
};
struct BwdLayout {  // offsets; -Delta is first
  size_t nlse, queue, arrived, seqs, items, col_of_group, col_list, colpart, lonepart, parts, end;
};
BwdLayout bwd_layout(const BwdSize& z, size_t B, size_t Hq, size_t Hkv, size_t D, const Cut& cut) {
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t slot = 64 * D * 2 * sizeof(float), nbh = B * Hkv, nparts = (size_t)cut.heads * cut.rows;
  BwdLayout l;
  l.nlse = up(B * Hq * z.rows * sizeof(float));
  l.queue = 2 * l.nlse;  // two work queues of 8 counters
  l.arrived = l.queue + 256;
  l.seqs = l.arrived + up(nbh * z.seqs * sizeof(unsigned));
  l.items = l.seqs + up(sizeof(LgBwdSeqs));
  l.col_of_group = l.items + up(z.ktiles * sizeof(int));
  l.col_list = l.col_of_group + z.groups * sizeof(int);
  l.colpart = l.col_of_group + up(2 * z.groups * sizeof(int));
  l.lonepart = l.colpart + nbh * z.ncol * slot;
  l.parts = l.lonepart + (Hq == Hkv ? nbh * z.lone * slot : 0);
  l.end = l.parts + (nparts > 1 ? nbh * z.ktiles * nparts * (btk_of(D) / 64) * slot : 0);
  return l;
}

// One set of launches: a batch of one length (setup.n = 0), or packed sequences.
struct BwdLaunch {
  LgBwdSetup setup;
  LgMask m;        // the batch's pattern; packed: the template
  int B, Hq, Hkv, D;
  float scale;
  BwdSize size;
  Cut cut;
  int qt_wide, qt_rest;   // query tiles of a head in each form of the dq kernel
  int kt_wide, kt_rest;   // key tiles of a head in each form of the dk/dv kernel
  int lone;               // chunks of lone groups
  int chunk, citems;      // column work items of a query head where there are several groups, and their query tiles
};

// dq and dk/dv share a launch (bwd_both_bf16_kernel) up to so many workgroups, where no sequence takes the 64-rows form of dq; dk/dv
// then takes its 32-keys form, which gives the same bits as the other.  One after the other both end with CUs idle, and a few
// heads of a few thousand tokens have workgroups for a part of the CUs either way.  Backward in us, launches of their own :
// this, of 64: 16 heads, 1117 tokens, causal 52 : 31, 8/4, 8 packed of up to 2186 89 : 62, 4 x 16, 997 58 : 46, 16/8, 1111, window
// 128 50 : 44, 2 x 64/16, 7479, window 200 (9568 workgroups) 437 : 434; of 128: 8, 3249, causal 224 : 150, 4 x 8, 1111 97 : 63, 16/8,
// 30 packed of up to 775 194 : 87, 1, 1098, causal 91 : 57, 16, 3707, window 186 93 : 90, 2 x 16/8, 8639, window 124 (1632) 254 : 241;
// 8, 30 packed of up to 3991, window 704 (1952) 317 : 323, 32/16, 30 of up to 3428, window 448 (5952) 992 : 1065.  Rows may be long:
// of 128, causal, 1, 49000 3073 : 2309, 4, 24000 1989 : 1805, 2, 48000 3904 : 3704, 1, 98000 8059 : 7855, window 4096 2, 24000 410 : 375.  Delta is a pass of
// its own then, over all of out and dO, which is got back up to 101 MB, of 64 up to 140: of 128, 129 (23 us), 2 x 32/16 heads, 3934
// tokens, window 182 221 : 236; 85, 2 x 8, 10341, window 128 159 : 159; 72, 32/8, 4408, window 320, every 8th block 301 : 248; of 64,
// 151, 32/16, 18467, window 192 214 : 223; 154, 4 x 64/8, 2349, causal 674 : 682; 107, 32/8, 13032, window 2930 986 : 954.
// Nor, of 128, where dq's rows are far longer than dk/dv's (strided columns, long sinks) and its items of 128 rows would have a CU
// each, or, with strided columns, half of them short rows beside: two by two they share one, and a tile takes about 0.4 us more; what
// there is of dk/dv to run beside them, 1.2 us a step, and the launch saved, 5, are less than that.  Every 2nd of 64-token blocks: 1
// head, 18047 tokens, window 128 401 : 474, 1, 58287, window 1024 1720 : 1895, 3, 15993, window 512 (189 pairs) 494 : 526; every 4th: 2,
// 16956, window 256 292 : 307; sink 2170, 2/1, 4340, window 200 78 : 81, but sink 3443, 8/4, 6887 (216 pairs) 1.13 times as fast
// shared.  The most that the rule costs: 4/1, every 4th block, 9776, window 256 218 : 215.
int both_dq_items(const BwdLaunch& a) { return (a.D == 128 ? 1 : 2) * a.qt_rest * a.Hq * a.B; }
struct Reach {
  int tiles, steps;  // of dq's longest rows, of dk/dv's window parts
};
Reach bwd_reach(const BwdLaunch& a) {
  const LgMask& m = a.m;
  const int N = a.setup.n > 0 ? a.setup.len[0] : m.N;  // (the longest)
  const long long reach = (long long)m.wb * m.b, cols = m.sink + (m.stride > 0 ? N / m.stride : 0);
  return {(int)(std::min<long long>(N, reach + cols) / 64) + 1, (int)(std::min<long long>(N, reach + btk_of(a.D)) / 64) + 1};
}
bool may_share(const BwdLaunch& a) {  // (however the window parts are cut)
  const double delta = 4.0 * a.size.rows * a.B * a.Hq * a.D;  // bytes of out and dO
  if (a.qt_wide > 0 || delta > (a.D == 128 ? 101e6 : 140e6)) return false;
  const Reach r = bwd_reach(a);
  return !(a.D == 128 && both_dq_items(a) <= (a.m.stride > 0 ? 255 : 128) && r.tiles > 3 * r.steps + 13);
}
bool bwd_both(const BwdLaunch& a) {
  const long long kv = (long long)(a.kt_wide + a.kt_rest) * a.Hkv * a.B * a.cut.heads * a.cut.rows;
  return may_share(a) && both_dq_items(a) + kv <= (a.D == 64 ? 8192 : 1536);
}
// Whether dq's items come first: those that take longer, by the products of a wave in a tile (3) and a step (4).  8/4 heads of 64, 8
// packed of up to 2186 tokens, causal, dq first 62, dk/dv first 68; 32/16, 8 of up to 1285, window 813 119, 94.
bool both_dq_first(const BwdLaunch& a) {
  const Reach r = bwd_reach(a);
  return 3 * r.tiles > 4 * ((r.steps + a.cut.rows - 1) / a.cut.rows) * (a.Hq / a.Hkv / a.cut.heads);
}

hipError_t launch_bwd(const uint16_t* uq, const uint16_t* uk, const uint16_t* uv, const uint16_t* uo, const float* lse,
                      const uint16_t* ug, uint16_t* dq, uint16_t* dk, uint16_t* dv, void* ws, const BwdLaunch& in,
                      hipStream_t s, hipEvent_t* ev) {
  BwdLaunch a = in;
  const size_t kv_bytes = (size_t)a.B * a.Hkv * a.m.ld * a.D * sizeof(uint16_t), lse_bytes = (size_t)a.B * a.Hq * a.m.ld * sizeof(float);
  bool both = bwd_both(a);
  for (const uint16_t* d : {dk, dv})
    both = both && !lg_overlap(d, kv_bytes, uk, kv_bytes) && !lg_overlap(d, kv_bytes, uv, kv_bytes) && !lg_overlap(d, kv_bytes, lse, lse_bytes);
  if (both) {
    a.kt_rest += a.kt_wide;
    a.kt_wide = a.setup.nwide = 0;
  }
  const LgMask& m = a.m;
  const int Hq = a.Hq, Hkv = a.Hkv, nbh = Hkv * a.B, ncol = (int)a.size.ncol, nlone = (int)a.size.lone;
  const float scale = a.scale;
  const BwdLayout l = bwd_layout(a.size, a.B, Hq, Hkv, a.D, a.cut);
  char* w = (char*)ws;
  // -Delta and -lse / scale: in this form the dk/dv kernels start the S and dP accumulators from them: S - lse / scale
  // needs one multiply before exp2, and dP - Delta comes out of the matrix pipe directly
  float* ndelta = (float*)w;
  float* nlse = (float*)(w + l.nlse);
  int* queue = (int*)(w + l.queue);
  unsigned* arrived = (unsigned*)(w + l.arrived);
  LgBwdSeqs* seqs = (LgBwdSeqs*)(w + l.seqs);
  int* items = (int*)(w + l.items);
  int* col_of_group = (int*)(w + l.col_of_group);
  int* col_list = (int*)(w + l.col_list);
  float* colpart = (float*)(w + l.colpart);
  const bool packed = a.setup.n > 0;
  const bool token = m.b == 1 && m.stride == 0;
  int cus = 0, dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    return hipErrorInvalidDevice;
  const int nparts = a.cut.heads * a.cut.rows;
  const long long most = 0x7fffffffLL - 8 * 16 * 64;  // (room for the padding of the last runs)
  if ((long long)(a.qt_wide + 2 * a.qt_rest) * Hq * a.B > most ||
      (long long)(a.kt_wide + a.kt_rest) * nbh * nparts * 8 > most || (long long)a.citems * Hq * a.B > most ||
      (long long)a.lone * Hq * a.B > most)
    return hipErrorInvalidValue;

  if (ev) (void)hipEventRecord(ev[0], s);
  // sums that atomics add to: all but those of lone groups with Hq == Hkv
  const size_t part_floats = a.citems > 0 || Hq != Hkv ? (l.lonepart - l.colpart) / sizeof(float) : 0;
  const size_t fill_wgs = (part_floats / 2 + 4 * SETUP_NT - 1) / (4 * SETUP_NT);
  LgBwdDelta delta = {(int)(1 + (packed ? a.setup.n : 1) + (fill_wgs < 1024 ? fill_wgs : 1024)), 0, a.D, m.ld, (int)(packed ? a.size.rows : m.N),
                      uo, ug, lse, ndelta, nlse, scale};
  for (int x = 0; x < (packed ? a.setup.n : 1); ++x) delta.chunks += ((packed ? a.setup.len[x] : m.N) + 63) / 64;
  bwd_setup_kernel<<<dim3((unsigned)(delta.first + (both ? delta.chunks * Hq * a.B : 0))), SETUP_NT, 0,
                     s>>>(a.setup, m, queue, seqs, items, col_of_group, col_list, ncol, arrived,
                          nlone > 0 ? nbh * (int)a.size.seqs : 0, colpart, part_floats, delta);
  if (ev) (void)hipEventRecord(ev[1], s);

  LgBwdWork wk;
  wk.seqs = packed ? seqs : nullptr;
  wk.items = items;
  wk.B = a.B;
  wk.wld = (int)(packed ? a.size.rows : m.N);
  wk.qt_first = 0;
  wk.col_of_group = col_of_group;
  wk.col_list = col_list;
  wk.ncol = ncol;
  wk.nlone = a.lone;
  wk.chunk = a.chunk;
  wk.colpart = colpart;
  wk.lonepart = Hq == Hkv ? (float*)(w + l.lonepart) : nullptr;
  wk.nlone_all = nlone;
  wk.arrived = arrived;
  wk.by_tile = packed || nparts > 1 || lg_dkdv_by_tile(m, nbh, (long long)(a.kt_wide + a.kt_rest) * nbh, both);
  wk.heads_cut = a.cut.heads;
  wk.rows_cut = a.cut.rows;
  wk.parts = (float*)(w + l.parts);
  wk.order = LG_BY_HEAD;
  if (a.qt_wide > 0) {
    const int total = a.qt_wide * Hq * a.B, run = lg_run_length(m, total, nbh, 8 * (Hq / Hkv), packed);
    const int nitems = (int)lg_run_grid(total, run);
    const dim3 grid((unsigned)(nitems < cus ? nitems : cus));
    if (token)
      dq_wide_bf16_kernel<true><<<grid, 256, 0, s>>>(uq, uk, uv, uo, ug, lse, ndelta, nlse, dq, Hq, Hkv, scale, m,
                                                     a.qt_wide, total, run, wk, queue, nitems);
    else
      dq_wide_bf16_kernel<false><<<grid, 256, 0, s>>>(uq, uk, uv, uo, ug, lse, ndelta, nlse, dq, Hq, Hkv, scale, m,
                                                      a.qt_wide, total, run, wk, queue, nitems);
  }
  if (a.qt_rest > 0 && !both) {
    const int total = 2 * a.qt_rest * Hq * a.B;
    const LgRuns runs = lg_runs(m, nbh, 2 * a.qt_rest, Hq / Hkv, packed);
    const dim3 grid((unsigned)lg_run_grid(runs, total));
    wk.qt_first = a.qt_wide;
    wk.order = lg_order(nbh, 2 * a.qt_rest, Hq / Hkv, a.D);
#define LG_DQ_LAUNCH(DD)                                                                                               \
  dq_bf16_kernel<DD><<<grid, 256, 0, s>>>(uq, uk, uv, uo, ug, lse, ndelta, nlse, dq, Hq, Hkv, scale, m, a.qt_rest, \
                                              total, runs, wk)
    if (a.D == 64) LG_DQ_LAUNCH(64);
    else LG_DQ_LAUNCH(128);
#undef LG_DQ_LAUNCH
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (ev) (void)hipEventRecord(ev[2], s);

#define LG_DKDV_ARGS uq, uk, uv, ug, nlse, ndelta, dk, dv, Hq, Hkv, scale, m
#define LG_DKDV_LAUNCH(DD, CC, GRID) \
  dkdv_bf16_kernel<DD, CC><<<GRID, 2 * btk_of(DD), 0, s>>>(LG_DKDV_ARGS, nkt, total, run, wk)
  // A lone group's items go with dq's and dk/dv's: where there are parts its sums are for the fold, with Hq == Hkv whoever comes last
  // adds them to the key tile's.  (Groups without parts: dk/dv adds what atomics have left, so they come before it.)  Backward in
  // us, a launch of their own : this, 4 heads of 128, 3500 tokens, window 128 58.3 : 36.9, 8, 3500, window 600 85.7 : 58.8, 16 x 4,
  // 900, window 128 73.6 : 62.7, 1, 37511, window 600 160.9 : 101.7; of 64, 2, 1700, window 128 36.1 : 18.7, 4 x 8, 1700 50.2 : 34.9,
  // 32, 900 32.8 : 26.4; with groups (and more chunks) 2/1 heads of 128, 2659 tokens, window 188 61.9 : 32.1, 16/2, 911, window 128 50.2 : 31.3,
  // 4 x 8/2, 1188, 64-token blocks, window 576 84.3 : 71.0; 8/2 of 64, 1162 tokens, window 205 40.0 : 23.0, 8/1, 3129, window 2201
  // 79.2 : 65.3, 4/2, 8 packed of up to 2456, window 194 63.0 : 53.5.
  const bool lone_too = both && (nparts > 1 || Hq == Hkv);
  wk.lone_joint = lone_too && nparts == 1;
  if (a.lone > 0 && !lone_too) {
    const dim3 grid((unsigned)(a.lone * Hq * a.B));
    // (groups have a chunk per CU: eight waves of head dim 64 as well.  32/16 heads, 8148 tokens 33 us with four, 26 with eight; 32/8,
    // 11624 47, 36)
#define LG_LONE_LAUNCH(DD, WAVES, GROUPS) \
  dkdv_lone_bf16_kernel<DD, WAVES, GROUPS><<<grid, 64 * WAVES, 0, s>>>(uq, uk, uv, ug, nlse, ndelta, Hq, Hkv, scale, m, wk)
    if (a.D == 64 && Hq == Hkv) LG_LONE_LAUNCH(64, 4, false);
    else if (a.D == 64) LG_LONE_LAUNCH(64, 8, true);
    else if (Hq == Hkv) LG_LONE_LAUNCH(128, 8, false);
    else LG_LONE_LAUNCH(128, 8, true);
#undef LG_LONE_LAUNCH
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (a.citems > 0) {
    const int nkt = 1, total = nbh, run = 1;
    const dim3 grid((unsigned)(a.citems * Hq * a.B));
    // column parts are long whatever the window is: the 64-keys form whenever it exists
    if (a.D == 128) dkdv_wide_bf16_kernel<false, true><<<grid, 256, 0, s>>>(LG_DKDV_ARGS, nkt, total, run, wk);
    else LG_DKDV_LAUNCH(64, true, grid);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (a.kt_wide > 0) {
    // one resident workgroup per CU, work items from the second queue
    wk.order = LG_BY_HEAD;  // (a queue hands them out)
    const int nkt = a.kt_wide, total = nkt * nbh, run = lg_run_length(m, total, nbh, 8, false);
    const int nitems = wk.by_tile ? total * nparts : (int)lg_run_grid(total, run);
    const dim3 grid((unsigned)(nitems < cus ? nitems : cus));
    if (token)
      dkdv_wide_bf16_kernel_q<true><<<grid, 256, 0, s>>>(LG_DKDV_ARGS, nkt, total, run, wk, queue + 8, nitems);
    else
      dkdv_wide_bf16_kernel_q<false><<<grid, 256, 0, s>>>(LG_DKDV_ARGS, nkt, total, run, wk, queue + 8, nitems);
  }
  if (a.kt_rest > 0) {
    const int nkt = a.kt_rest, total = nkt * nbh, run = lg_run_length(m, total, nbh, 8, false);
    const dim3 grid((unsigned)(wk.by_tile ? total * nparts : (int)lg_run_grid(total, run)));
    wk.items = items + a.kt_wide;
    wk.order = lg_order(nbh, nkt, 1, a.D);
    if (both) {
      const int ndq = both_dq_items(a), nkv = (int)grid.x, nlo = lone_too ? a.lone * Hq * a.B : 0;
#define LG_BOTH_LAUNCH(DD, LL)                                                                                                \
  bwd_both_bf16_kernel<DD, LL><<<dim3((unsigned)(nkv + ndq + nlo)), 2 * btk_of(DD), 0, s>>>(uq, uk, uv, ug, lse, nlse, ndelta, dq, dk, dv, Hq, Hkv, \
                                                                                  scale, m, nkt, total, run, wk, a.qt_rest, nkv, ndq, both_dq_first(a))
      const int lone = nlo == 0 ? LONE_NONE : Hq != Hkv ? LONE_GROUPS : LONE_HEADS;
      if (a.D == 64 && lone == LONE_NONE) LG_BOTH_LAUNCH(64, LONE_NONE);
      else if (a.D == 64 && lone == LONE_GROUPS) LG_BOTH_LAUNCH(64, LONE_GROUPS);
      else if (a.D == 64) LG_BOTH_LAUNCH(64, LONE_HEADS);
      else if (lone == LONE_NONE) LG_BOTH_LAUNCH(128, LONE_NONE);
      else if (lone == LONE_GROUPS) LG_BOTH_LAUNCH(128, LONE_GROUPS);
      else LG_BOTH_LAUNCH(128, LONE_HEADS);
#undef LG_BOTH_LAUNCH
    } else if (a.D == 64) LG_DKDV_LAUNCH(64, false, grid);
    else LG_DKDV_LAUNCH(128, false, grid);
  }
#undef LG_DKDV_LAUNCH
#undef LG_DKDV_ARGS
  if (nparts > 1) {
    const dim3 grid((unsigned)((a.kt_wide + a.kt_rest) * nbh * (btk_of(a.D) / 32) * (a.D / 64)));
    if (a.D == 64) bwd_fold_kernel<64><<<grid, 256, 0, s>>>(dk, dv, nbh, scale, m, wk);
    else bwd_fold_kernel<128><<<grid, 256, 0, s>>>(dk, dv, nbh, scale, m, wk);
  }
  e = hipGetLastError();
  if (ev) (void)hipEventRecord(ev[3], s);
  return e;
}

// Query tiles per column work item where there are several groups: 64, less where that leaves CUs idle, but not so few
// that more than 32 items add to the same sums, which then take longer than the products (64/8 heads of 128, 16001
// tokens, four groups: 32 adders 218 us, 64 adders 332 us).  items(chunk): work items of the launch; longest: query
// tiles of the longest column part; G: query heads per kv head.
template <typename F>
int choose_chunk(F items, int longest, int G) {
  int chunk = 64;
  while (chunk > 8 && items(chunk) < 2 * CUS && (long long)G * (longest / (chunk / 2) + 1) <= 32) chunk /= 2;
  return chunk;
}

// The launch of a batch: everything but the pointers (also decides the workspace's size).
BwdLaunch batch_launch(const LgShape& sh, const LgMask& m) {
  BwdLaunch a = {};
  a.m = m;
  a.B = sh.B;
  a.Hq = sh.Hq;
  a.Hkv = sh.Hkv;
  a.D = sh.D;
  a.scale = sh.scale;
  const Columns c = columns_of(m, sh.D);
  a.setup.btk = btk_of(sh.D);
  a.size.add(sh.N, sh.D, sh.Hq, c);
  a.chunk = choose_chunk([&](int chunk) { return (long long)c.items(sh.D, chunk) * sh.Hq * sh.B; },
                         c.last - c.first, sh.Hq / sh.Hkv);
  a.citems = c.items(sh.D, a.chunk);
  a.lone = sh.Hq == sh.Hkv ? c.lone(sh.D, sh.Hq) : c.lone_of_groups(sh.Hq / sh.Hkv, (long long)sh.Hq * sh.B);
  (dq_wide(m, sh.D, sh.Hq) ? a.qt_wide : a.qt_rest) = (sh.N + LG_BF16_TQ - 1) / LG_BF16_TQ;
  (dkdv_wide(m, sh.D) ? a.kt_wide : a.kt_rest) = (int)a.size.ktiles;
  a.cut = {1, 1};
  if (may_cut(sh, m.stride > 0, a.size.ktiles * sh.B * sh.Hkv)) {
    double steps = 0;
    int longest = 0;
    window_steps(m, a.setup.btk, &steps, &longest);
    a.cut = choose_cut(sh.D, sh.Hq / sh.Hkv, sh.B * sh.Hkv, a.size.ktiles, steps, longest, MOST_PARTS, may_share(a) ? both_dq_items(a) : -1);
  }
  return a;
}

// The next set of launches of a pack, for the sequences from `x` on: those that fit `budget` bytes of workspace together
// (the first one always counts as fitting), up to LG_PACK_MAX, sorted longest first.  Returns the first sequence that is
// not in it and the bytes it uses; a->setup.n is 0 when only empty sequences were left.  -1: too many work items.
int pack_launch(const LgShape& sh, const LgMask& tmpl, const int* cu_seqlens, int num_seqs, int x, size_t budget,
                BwdLaunch* out, size_t* bytes) {
  struct Seq {
    int row0, len;
    Columns c;
  } seq[LG_PACK_MAX];
  BwdLaunch& a = *out;
  a = {};
  a.m = tmpl;
  a.B = 1;
  a.Hq = sh.Hq;
  a.Hkv = sh.Hkv;
  a.D = sh.D;
  a.scale = sh.scale;
  a.cut = {1, 1};
  a.setup.btk = btk_of(sh.D);
  auto end = [&](const BwdSize& z) { return bwd_layout(z, 1, sh.Hq, sh.Hkv, sh.D, a.cut).end; };
  int& n = a.setup.n;
  for (; x < num_seqs && n < LG_PACK_MAX; ++x) {
    const int len = cu_seqlens[x + 1] - cu_seqlens[x];
    if (len == 0) continue;
    const Seq one = {cu_seqlens[x], len, columns_of(lg_mask_for_length(tmpl, len), sh.D)};
    BwdSize z = a.size;
    z.add(len, sh.D, sh.Hq, one.c);
    if (n > 0 && (end(z) > budget || z.ktiles > 0xffffff || (double)z.rows * sh.Hq > 1e9)) break;
    a.size = z;
    int y = n++;
    for (; y > 0 && seq[y - 1].len < len; --y) seq[y] = seq[y - 1];
    seq[y] = one;
  }
  if (n == 0) return x;
  auto citems = [&](int chunk) {
    long long all = 0;
    for (int y = 0; y < n; ++y) all += seq[y].c.items(sh.D, chunk);
    return all * sh.Hq;
  };
  int longest_col = 0;
  for (int y = 0; y < n; ++y)
    if (seq[y].c.last - seq[y].c.first > longest_col) longest_col = seq[y].c.last - seq[y].c.first;
  a.chunk = choose_chunk(citems, longest_col, sh.Hq / sh.Hkv);
  if (citems(a.chunk) > 0x7fffffffLL) return -1;
  double steps = 0;
  int longest = 0;
  bool strided = false;
  for (int y = 0; y < n; ++y) {
    const LgMask m = lg_mask_for_length(tmpl, seq[y].len);
    a.setup.row0[y] = seq[y].row0;
    a.setup.len[y] = seq[y].len;
    a.setup.ncol[y] = seq[y].c.ncol;
    a.setup.citems[y] = seq[y].c.items(sh.D, a.chunk);
    a.setup.nlone[y] = sh.Hq == sh.Hkv ? seq[y].c.lone(sh.D, sh.Hq) : seq[y].c.lone_of_groups(sh.Hq / sh.Hkv, (long long)sh.Hq * n);
    a.lone += a.setup.nlone[y];
    a.citems += a.setup.citems[y];
    // (both rules are monotone in the length: the wide ones come first)
    (dq_wide(m, sh.D, sh.Hq) ? a.qt_wide : a.qt_rest) += (seq[y].len + LG_BF16_TQ - 1) / LG_BF16_TQ;
    (dkdv_wide(m, sh.D) ? a.kt_wide : a.kt_rest) += (seq[y].len + a.setup.btk - 1) / a.setup.btk;
    a.setup.nwide += dkdv_wide(m, sh.D);
    strided = strided || m.stride > 0;
  }
  if (may_cut(sh, strided, a.size.ktiles * sh.Hkv)) {
    for (int y = 0; y < n; ++y) window_steps(lg_mask_for_length(tmpl, seq[y].len), a.setup.btk, &steps, &longest);
    const size_t tile = (size_t)sh.Hkv * a.size.ktiles * (a.setup.btk * 2 * sizeof(float)) * sh.D, used = end(a.size);
    a.cut = choose_cut(sh.D, sh.Hq / sh.Hkv, sh.Hkv, a.size.ktiles, steps, longest,
                       n == 1 ? MOST_PARTS : used < budget ? (budget - used) / tile : 0, may_share(a) ? both_dq_items(a) : -1);
  }
  *bytes = end(a.size);
  return x;
}
}  // namespace

// Sequences side by side in one set of launches are worth up to this much workspace: room for 85000 to 500000 tokens (64
// to 8 query heads).
constexpr size_t BWD_PACK_BYTES = 128u << 20;

size_t lg_bwd_bf16_workspace_bytes(const LgShape& sh, const LgMask& m) {
  const BwdLaunch a = batch_launch(sh, m);
  return bwd_layout(a.size, sh.B, sh.Hq, sh.Hkv, sh.D, a.cut).end;
}

bool lg_bwd_bf16_splits_columns(const LgMask& m, int D) { return columns_of(m, D).ncol > 0; }

size_t lg_bwd_bf16_pack_workspace_bytes(const LgShape& sh, const LgMask& tmpl, const int* cu_seqlens, int num_seqs,
                                        size_t least) {
  size_t need = least;
  BwdLaunch a;
  for (int x = 0; x >= 0 && x < num_seqs;) {
    size_t bytes = 0;
    x = pack_launch(sh, tmpl, cu_seqlens, num_seqs, x, std::max(least, BWD_PACK_BYTES), &a, &bytes);
    need = std::max(need, bytes);
  }
  return need;
}

void lg_bwd_bf16_plan(const LgShape& sh, const LgMask& m, const int* cu_seqlens, int num_seqs, size_t ws_bytes, int32_t* plan) {
  BwdLaunch a = {};
  size_t bytes = 0;
  if (!cu_seqlens) a = batch_launch(sh, m);
  else (void)pack_launch(sh, m, cu_seqlens, num_seqs, 0, std::max(ws_bytes, BWD_PACK_BYTES), &a, &bytes);
  const bool both = bwd_both(a);
  const int p[8] = {both, a.qt_wide, a.qt_rest, both ? 0 : a.kt_wide, both ? a.kt_wide + a.kt_rest : a.kt_rest, a.cut.heads, a.cut.rows, a.lone};
  std::copy(p, p + 8, plan);
}

hipError_t lg_launch_bwd_bf16(const void* q, const void* k, const void* v, const void* out, const float* lse,
                              const void* dout, void* dq, void* dk, void* dv, void* ws, const LgShape& sh,
                              const LgMask& m, hipStream_t s, hipEvent_t* ev) {
  return launch_bwd((const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)out, lse,
                    (const uint16_t*)dout, (uint16_t*)dq, (uint16_t*)dk, (uint16_t*)dv, ws, batch_launch(sh, m), s, ev);
}

// One set of launches for up to LG_PACK_MAX sequences.  Launched one sequence after the other, a document of 200 .. 8192
// tokens does not fill 256 CUs and its last wave of workgroups leaves most of them idle (24 documents, 32/8 heads of
// 128, window 4096: dq and dk/dv 11.7 ms; side by side 5.5 ms).
hipError_t lg_launch_bwd_bf16_pack(const void* q, const void* k, const void* v, const void* out, const float* lse,
                                   const void* dout, void* dq, void* dk, void* dv, void* ws, size_t ws_bytes,
                                   const LgShape& sh, const LgMask& tmpl, const int* cu_seqlens, int num_seqs,
                                   hipStream_t s) {
  BwdLaunch a;
  for (int x = 0; x < num_seqs;) {
    // (planned as for the size that was asked for, so that a workspace of that size or more gives one and the same plan
    // up to BWD_PACK_BYTES; again for what is there if that is less)
    size_t bytes = 0;
    int next = pack_launch(sh, tmpl, cu_seqlens, num_seqs, x, std::max(ws_bytes, BWD_PACK_BYTES), &a, &bytes);
    if (next >= 0 && bytes > ws_bytes) next = pack_launch(sh, tmpl, cu_seqlens, num_seqs, x, ws_bytes, &a, &bytes);
    if (next < 0 || bytes > ws_bytes) return hipErrorInvalidValue;
    x = next;
    if (a.setup.n == 0) break;
    const hipError_t e =
        launch_bwd((const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)out, lse,
                   (const uint16_t*)dout, (uint16_t*)dq, (uint16_t*)dk, (uint16_t*)dv, ws, a, s, nullptr);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// lg_fwd_bf16.h — bf16 prefill forward on the gfx950 matrix cores (paper Section
// 3.2: fused online-softmax attention that never loads key tiles whose mask is zero).
//
// Workgroup = 4 wavefronts = 128 query rows of one (b, hq); wave w owns 32 rows.  Per live key tile
// (64 keys, from the closed-form scheduler in lg_mask.h):
//   S^T = K Q^T     (keys x queries): A = K rows from LDS, B = Q kept in registers
//   softmax         on S^T: a lane holds 32 keys of ONE query, so row sum and (where it is
//                   looked at) row max are in-lane reductions plus one exchange with lane^32
//   O^T += V^T P^T  (dims x queries): A = V read from LDS through the transposing
//                   LDS load, B = P^T straight from the S^T accumulator registers
// Masking is applied only on PARTIAL tiles.
//
// What bounds it, and the shape that follows.  A tile costs a wave 1024 cycles of the matrix pipe (D = 128) and about
// as many of vector work, one after the other, so a SIMD needs several waves that are NOT in the same phase: three
// workgroups per CU for D = 128, four for D = 64, each with barriers of its own and little LDS (two K tiles and one V
// tile, 48 KB / 24 KB; K of tile t + 2 and V of tile t + 1 are requested as soon as tile t has left their place).
// One workgroup of 8 waves in step (two per SIMD) with a 128 KB ring needed 30 % more cycles; 6 or 12 waves per
// workgroup are slower as well, 6 because they do not spread evenly over four SIMDs.  Smaller workgroups also waste
// less on short sequences.  32 heads of 128, 131072 tokens, window 4096: 9.1 -> 8.45 ms, with the steps below 7.5 (1170 TFLOP/s;
// the clock settles at 1.8 GHz instead of 2.2 under the power limit); 8 x 1024 tokens 144 -> 116 us.
//
// Rows of few tiles are bound by what a workgroup does besides tiles, so Q and O go through LDS in pieces of 1 KB (a lane's
// own row, 16 bytes at a time, is 32 rows per instruction: address and cache-line work of 2000 cycles each way) and items
// are found without divisions: 32 heads of 128, 32768 tokens, window 64 216 -> 198 us (5.4 TB/s), 1024 633 -> 609; 64 x 512
// tokens 300 -> 269 us.  (Asking for the next item's Q lines while a tile is computed was slower: 198 -> 207 us.)
// What whole tiles cost depends on where the tile loop's code falls (5 % for 24055 tokens of 2 heads of 64, from a change
// that touched only the masks of PARTIAL tiles): its files are compiled with loops at 64-byte boundaries.
#ifndef LG_FWD_BF16_H_
#define LG_FWD_BF16_H_

#include "lg_kernels.h"
#include "lg_mfma.h"
#include "lg_swz.h"

namespace {

constexpr int TK = LG_BF16_TK;    // 64 keys per step
constexpr int TQ = LG_BF16_TQ32;  // 128 query rows per workgroup
constexpr int NT = TQ * 2;        // threads: one wave per 32 rows
// Waves per SIMD, and LDS operands of the two products requested ahead of the matrix instruction that uses them, as the
// registers of so many waves allow (168 for D = 128, 128 for D = 64).  Three ahead in both products of D = 128 instead of two
// and four: 32 heads, 131072 tokens, window 4096 7.84 -> 7.65 ms (four and three, four and four, three and two: 7.66 .. 7.72;
// five and three spill).
template <int D, bool FEW>
struct LgFwdTune {
    static constexpr int WAVES = FEW ? 2 : D == 128 ? 3 : 4, AHEAD = FEW ? 4 : 3, AHEAD_PV = FEW || D == 64 ? 4 : 3;
};

// FEW: the instance for launches that leave most SIMDs with one wave (LG_FWD_FEW work items, a workgroup or two per CU).
// Nothing then hides a wave's own waits: with the registers of two waves K is read four matrix instructions ahead, K and V of
// the next tile are both requested behind the one barrier of a tile (four tiles in LDS), for D = 128 between the matrix
// instructions of the first product, and V's first reads go out before the softmax.  Same operations in the same order on
// every row, so the results are those of the other instance bit for bit.  2 x 16 heads of 64, 1003 tokens 15.3 -> 14.5 us, of
// 128 19.6 -> 18.5; 4/1 heads of 128, 5000 tokens, causal 96.2 -> 88.8, of 64 73.4 -> 68.1; where workgroups share a CU it is
// slower (640 of them, D = 128: 90 -> 101).  Requests in between are slower for D = 64, as are reads further ahead; the second
// product in one phase with the next tile's exponentials was slower as well (98 -> 108: they do not overlap within a wave).
// Half of the CUs with two workgroups still gain (us, the other instance : this, heads of 128 and of 64): 288 items, 32/16 heads,
// 1086 tokens, window 237 16.3 : 14.2 and 12.4 : 10.2; 316, 4/1, 10000, causal 182 : 174 and 137 : 127; 352, 16/8, 2816, window 600
// 27.1 : 25.2 and 20.5 : 19.9; 384, 8, 6144, window 4096 86.7 : 83.5 and 63.7 : 58.6; 376, 6 packed of up to 1500, 8 heads 35.4 :
// 32.9 and 25.9 : 24.5 (least gain: 364, 2 packed of up to 6000, 4/1 heads of 128, causal 140.0 : 140.8).  Beyond that it depends on
// the rows: 448, 56/8, 1000, window 300 20.1 : 19.9 and 15.1 : 15.6; 512, 4 x 16, 960 24.0 : 25.0 and 17.7 : 18.2, but 16/4, 4000,
// causal 84.7 : 83.2 and 59.1 : 54.7; 592, 16/8, 4700, window 512 32.1 : 37.5 and 21.5 : 26.7.
constexpr int LG_FWD_FEW = 384, LG_FWD_ALONE = 256;  // (ALONE: up to so many have a CU each)
// PackT: LgNoPack for the batch layout (every (b, head) has the same query tiles), LgPackOf for
// sequences of different lengths side by side in each head (B = 1).
struct LgNoPack {};

// LIST (an instance of its own of FEW, by lg_fwd_lists): a wave's walk from its fourth tile on (strided columns: from the first), up
// to 64 tiles at a time worked out by its lanes as 4 * tile + class for the wave's rows.  The next tile and its class as scalar code
// are 60 instructions of a tile's 350, and nothing hides a lone wave's instructions: 1 head of 64, 4533 tokens, causal 62.9 -> 58.8
// us; 8 of 64, 2817 tokens, 64-token blocks, window 704, every 4th block 24.6 -> 22.4; 8/2 of 128, 3999 tokens, window 512 34.9 ->
// 31.4; 2 x 16 of 64, 1003 tokens, window 512 15.1 -> 14.7.  Rows of a few tiles pay for the list's start (scalar : list): 32/16
// heads of 64, 740 tokens, 64-token blocks, window 128 7.6 : 7.8, 16/4, 2265 8.5 : 9.6, of 128, 8/2, 5048, window 64 10.2 : 11.2, from
// ten tiles on the list is at least level (32/4, 758 tokens, causal 18.0 : 18.1); strided columns far apart leave a list one tile of
// 64 looked at: 1 head of 64, 24624 tokens, every 64th 64-token block 12.0 : 15.3, every 32nd 18.1 : 19.8, every 16th 30.1 : 29.1.
// (List or no list within one instance, by the row's length: slower for all.)
struct LgFewWalk {
  int list, at, count, pos;
  // after tile prev, the last one
  __device__ __forceinline__ int next(const LgMask& m, const LgQSched& s, const LgQWalk& w, const LgRows& rows, bool idle, int prev) {
    if (__builtin_expect(at == count, 0)) {
      asm volatile("; list tiles" ::: "memory");  // (a real branch)
      const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
      at = 0;
      int t = 0;
      if (m.stride == 0) {  // sink tiles, then the rotated run
        const int p = pos + lane, len = w.tmax - w.tws + 1;
        count = min(64, w.nsink + max(len, 0) - pos);
        if (count <= 0) return -1;
        pos += 64;
        t = p < w.nsink ? p : w.tstart + p - w.nsink;
        if (t > w.tmax) t -= len;
      } else {  // the live ones of 64 tiles, side by side
        unsigned long long live = 0;
        for (int x = ++prev >> 6; live == 0 && 64 * x <= s.tmax; ++x) {
          t = 64 * x + lane;
          live = __builtin_amdgcn_ballot_w64(t >= prev && lg_qsched_next(m, s, t - 1) == t);
        }
        const bool mine = (live >> lane) & 1;
        const int below = __builtin_amdgcn_mbcnt_hi((unsigned)(live >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)live, 0));
        count = __builtin_popcountll(live);
        t = __builtin_amdgcn_ds_permute(4 * (mine ? below : count + lane - below), t);
      }
      if (count <= 0) return -1;
      list = 4 * t + (idle ? LG_TILE_DEAD : lg_rows_kind(m, rows, t * TK, t * TK + TK - 1));
    }
    return __builtin_amdgcn_readlane(list, at++);
  }
};

template <int D, typename PackT, bool FEW, bool LIST>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(LgFwdTune<D, FEW>::WAVES, LgFwdTune<D, FEW>::WAVES))) void fwd_bf16_kernel(const uint16_t* __restrict__ q,
                                                      const uint16_t* __restrict__ k,
                                                      const uint16_t* __restrict__ v,
                                                      uint16_t* __restrict__ out,
                                                      float* __restrict__ lse, int Hq, int Hkv,
                                                      float scale_log2e, LgMask m_in, LgItems items,
                                                      PackT pack) {
  constexpr bool PACK = !__is_same(PackT, LgNoPack);
  LgMask m = m_in;
  using T = LgSwzTile<D>;
  using Dma = LgDma<D, NT, !FEW>;
  constexpr int DC = D / 16;            // 16-wide contraction chunks of the head dim
  constexpr int DB = D / 32;            // 32-row blocks of O^T
  using Tune = LgFwdTune<D, FEW>;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[(FEW ? 4 : 3) * T::BYTES];  // two K tiles, a V tile (FEW: two)

  const int L = lg_item_of(blockIdx.x, items);
  if (L < 0 || L >= items.total) return;
  const LgItem it = lg_item(items, L);
  const int b = it.b, hk = it.hk, hq = it.hq;
  int qt = (int)items.nqt.d - 1 - it.x;
  int seq_row0 = 0;  // first row of the sequence inside its head
  if constexpr (PACK) {
    // the sequence that owns query tile qt of the launch: the last one whose first tile is <= qt
    int lo = 0, hi = pack.n;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (pack.seq[mid].tile0() <= qt) lo = mid;
      else hi = mid;
    }
    const auto sq = pack.seq[lo];
    const int nt = (sq.len() + TQ - 1) / TQ;
    qt -= sq.tile0();
    // two sequences in four the other way round where their tiles are an even number (lg_order says why; sequence 0 comes last)
    if (nt % 2 == 0 && nt <= 64 && (lo & 2) != 0) qt = nt - 1 - qt;
    seq_row0 = sq.row0;
    m = lg_mask_for_length(m, sq.len());
  }
  const int N = m.N;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, g = lane >> 5;
  const int q0 = qt * TQ;
  const int q1 = min(q0 + TQ - 1, N - 1);
  const size_t qbase = ((size_t)(b * Hq + hq) * m.ld + seq_row0) * D;
  const uint16_t* kh = k + ((size_t)(b * Hkv + hk) * m.ld + seq_row0) * D;
  const uint16_t* vh = v + ((size_t)(b * Hkv + hk) * m.ld + seq_row0) * D;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const bool idle = q0 + wave_s * 32 >= N;  // past the end
  const int qw0 = min(q0 + wave_s * 32, N - 1), qw1 = min(q0 + wave_s * 32 + 31, N - 1);  // this wave's rows

  // Rows that grow along the sequence, hardly more of them than places: the longest decide when the launch ends, so they go
  // before their neighbours on the CU, the more the longer.  Full causal, without and with, us, and the rounds: 24 heads of 64,
  // 6000 tokens 169, 146 (1.1); 40, 3000 88, 74 (0.9); 24 of 128, 5400 tokens 204, 193 (1.3); 100 x 4, 300 30.2, 34.5 (1.6); four
  // heads side by side (lg_order), which even out by themselves: 2 x 32 of 64, 1300 tokens 29.4, 28.3 (0.7); of 128, 2048
  // tokens 76.8, 79.9 (1.3); 4 x 32 of 64, 2048 105, 115 (2).
  if (!PACK && !FEW && 5 * items.total <= (items.order >= LG_BY_FOUR ? 6 : 7) * 256 * Tune::WAVES && 2 * (long long)m.wb * m.b >= N) {
    const int third = (int)(3LL * q0 / N);
    if (third == 2) __builtin_amdgcn_s_setprio(2);
    else if (third == 1) __builtin_amdgcn_s_setprio(1);
  }
  f32x16_t oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
  float mref = -INFINITY, lrow = 0.f;
  bool watch = true;  // (FEW: not used) some row has no reference yet

  Dma dma;
  dma.init(tid);
  LgSwzReader<D> rd;
  rd.init(n, g);
  const uint32_t lds0 = (uint32_t)(uintptr_t)LG_LDS_PTR(unsigned char, smem);
  const bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};

  auto issue_k = [&](int t, int buf) { dma.issue(kh + (size_t)t * TK * D, N - t * TK, lds0 + buf * T::BYTES); };
  auto issue_v = [&](int t, int buf) { dma.issue(vh + (size_t)t * TK * D, N - t * TK, lds0 + (2 + buf) * T::BYTES); };
  // K tiles are requested up to two ahead of the one being computed, its own V tile behind the barrier that opens it
  const LgQSched qs = lg_qsched_init(m, q0, q1);
  const LgRows wrows = lg_rows(m, qw0, qw1);
  // patterns without strided columns walk the window run rotated (L2 sharing between neighbours)
  const LgQWalk qw = lg_qwalk_init(qs);
  auto next_tile = [&](int prev) -> int {
    if (m.stride == 0) return prev < 0 ? lg_qwalk_first(qw) : lg_qwalk_next(qw, prev);
    return lg_qsched_next(m, qs, prev);
  };
  LgFewWalk few = {0, 0, 0, 3};  // (LIST)
  int kind0 = 0, kind1 = 0, few2 = -1;  // (LIST) classes of tiles t, t1; the walk's entry after them
  auto kind_of = [&](int t) { return idle ? LG_TILE_DEAD : lg_rows_kind(m, wrows, t * TK, t * TK + TK - 1); };
  int t = next_tile(-1);  // tile to compute next
  int t1 = next_tile(t);
  issue_k(t, 0);
  // Q fragments (B operand): lane (n, g) holds dims 16*dc + 8g .. +7 of its row.  The workgroup's rows come through the
  // places of the second K tile and of V (loaded by each lane from its own row, an instruction touches 32 rows).
  bf16x8_t qf[DC];
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int r0 = min(q0 + 64 * x, N - 1);  // (rows past the end repeat the last one)
    dma.issue(q + qbase + (size_t)r0 * D, N - r0, lds0 + (1 + x) * T::BYTES);
  }
  if (LIST && m.stride > 0 && t1 >= 0) {  // (while the rows are under way)
    kind0 = few.next(m, qs, qw, wrows, idle, t - 1) & 3;
    kind1 = few.next(m, qs, qw, wrows, idle, t) & 3;
    few2 = few.next(m, qs, qw, wrows, idle, t1);
  } else if (LIST) {
    kind0 = kind_of(t);
    if (t1 >= 0) {
      kind1 = kind_of(t1);
      few2 = next_tile(t1);
      if (few2 >= 0) few2 = 4 * few2 + kind_of(few2);
    }
  }
  LG_WAIT_VMCNT(0);
  __syncthreads();
#pragma unroll
  for (int dc = 0; dc < DC; ++dc) qf[dc] = rd.read_rows(smem, (1 + (wave_s >> 1)) * T::BYTES, wave_s & 1, dc);
#pragma unroll
  for (int dc = 0; dc < DC; ++dc) asm volatile("" ::"v"(qf[dc]));
  __syncthreads();
  if (FEW) issue_v(t, 0);
  else if (t1 >= 0) issue_k(t1, 1);

  int buf = 0, t2 = -1;
  // One tile, t.  The exponents of a row are relative to a reference, on which softmax does not depend: its largest score in
  // the first tile that is live for it, or one that has moved since.  It moves, and the accumulators are rescaled, where a
  // score is more than 2^8 above it, so that a key that carries a row has the probability 1 and not a rounded one: the
  // log-sum-exp, and with it the gradients, are as exact as that.
  //   FOLLOW: every tile's maxima are looked at for that, a fifth of a tile's vector instructions.
  //   Otherwise the sums of the probabilities tell, which are there anyway: above 192 there may be one of 2^8 (less than that by
  // what P's exponent, a difference of rounded products, may be off), and the tile is left, returning true, and computed once
  // more by FOLLOW (resumed; K is still in its place), which also takes the wave's other tiles.  A reference moves at the same
  // scores either way, so results do not depend on which form took a tile.
  // Us with FOLLOW alone, and so: 8 heads of 128, 32768 tokens, window 4096 511, 486; 32 heads, 16384 tokens, causal 2017,
  // 1916; 32 heads, 32768 tokens, 64-token blocks, window 192, every 8th block 1160, 1120; 16 of 64, 8192 tokens, window 512 33.1,
  // 33.2.  With queries times 6, where scores outgrow the first ones in nearly every row: 522, 526; 2089, 2060; 1191, 1215;
  // 33.8, 36.6 (a tile more for rows of ten).  With one wave or two per SIMD (FEW) little hides the wait for the sums before the second
  // product, and FOLLOW alone is faster (2 x 16 heads of 64, 1003 tokens 15.0, 16.4).
  auto tile = [&](auto FOLLOW_, bool resumed) -> bool {
    constexpr bool FOLLOW = decltype(FOLLOW_)::value;
    if (!resumed) {
      if (!FEW && t1 >= 0) LG_WAIT_VMCNT(Dma::CH);
      else LG_WAIT_VMCNT(0);
      __syncthreads();  // K(t) landed; everyone is done with V(t-1); (FEW) V(t) landed as well
    }
    // (K's first operands are asked for before V's lines, whose four requests take 200 cycles: 7.57 -> 7.49 ms, head dim 64
    // 2.15 -> 2.13)
    const int sk = buf * T::BYTES;  // byte offsets of the K and V tiles inside smem
    auto read_k = [&](int u) { return rd.read_rows(smem, sk, u & 1, u >> 1); };
    LgRing<2 * DC, Tune::AHEAD> ring;
    ring.begin(read_k);
    __builtin_amdgcn_sched_barrier(0);
    if (!resumed) {
      if (!FEW) issue_v(t, 0);
      if (!LIST) t2 = t1 >= 0 ? next_tile(t1) : -1;
    }

    const int k0 = t * TK;
    // A tile that is not live throughout for the workgroup's 128 rows is classified again for
    // this wave's 32 rows: most waves then find it wholly live or wholly dead (they sit it out).
    int kind = LG_TILE_FULL, kind2 = 0;
    if (LIST) {
      kind = kind0;
      t2 = few2 >> 2;
      kind2 = few2 & 3;
      if (few2 >= 0) few2 = few.next(m, qs, qw, wrows, idle, t2);
    } else if (idle) kind = LG_TILE_DEAD;
    else if (!lg_qsched_full(m, qs, t)) kind = lg_rows_kind(m, wrows, k0, k0 + TK - 1);
    const bool full = kind == LG_TILE_FULL;
    const int sv = (FEW ? 2 + buf : 2) * T::BYTES;
    auto read_v = [&](int u) { return rd.read_cols(smem, sv, u % DB, u / DB); };
    LgRing<4 * DB, Tune::AHEAD_PV> vring;
    // (FEW) the next tiles' requests go between the matrix instructions of the first product, if both are whole
    const bool between = FEW && D == 128 && kind != LG_TILE_DEAD && t1 >= 0 && N - t1 * TK >= TK;
    if (FEW && t1 >= 0 && !between) {
      issue_k(t1, buf ^ 1);
      issue_v(t1, buf ^ 1);
    }
    bf16x8_t pf[4];  // P^T as bf16, B operand of the second product, per 16-key group
    if (kind != LG_TILE_DEAD) {

    // ---- S^T = K Q^T ----
    f32x16_t sacc[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[kb][r] = 0.f;
    // Each operand from LDS is requested some matrix instructions early (the compiler on its own asks for it just before
    // its use, which leaves the LDS latency in the wave's critical path sixteen times per product; for V that was 3 %
    // at 128K tokens, 10 % where a SIMD has one wave).
    {
      if (between) {
        const uint16_t *k1 = kh + (size_t)t1 * TK * D, *v1 = vh + (size_t)t1 * TK * D;
        const uint32_t to = lds0 + (buf ^ 1) * T::BYTES;
        ring.run(read_k, [&](int u, bf16x8_t k) {
          sacc[u & 1] = lg_mfma32(k, qf[u >> 1], sacc[u & 1]);
          static_assert(2 * Dma::CH == DC, "a request per two matrix instructions");
          const int x = u >> 1;
          if (u & 1) dma.load(x < Dma::CH ? k1 : v1, to + (x < Dma::CH ? 0 : 2 * T::BYTES), x % Dma::CH);
        });
      } else {
        ring.run(read_k, [&](int u, bf16x8_t k) { sacc[u & 1] = lg_mfma32(k, qf[u >> 1], sacc[u & 1]); });
      }
    }

    if (FEW) vring.begin(read_v);
    // ---- softmax (log2 domain) ----
    if (__builtin_expect(!full, 0)) {
      asm volatile("; masked" ::: "memory");  // (a real branch: nothing of it in whole tiles)
      int ln = lane;  // D = 128: asked for again here, kept from the start it was a register too many
      if (D == 128) asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
      const int row = min(q0 + wave_s * 32 + (ln & 31), N - 1);
      const uint32_t bits = lg_key_bits(m, row, k0, ln >> 5);  // a few runs of registers, in closed form
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          sacc[kb][r] = lg_keep_or(sacc[kb][r], bits, kb * 16 + r, -INFINITY);
    }
    if (FOLLOW || __builtin_expect(watch, 0)) {
      if (!FOLLOW) asm volatile("; reference" ::: "memory");  // keep this a real branch
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; r += 2) mx = fmaxf(fmaxf(sacc[kb][r], sacc[kb][r + 1]), mx);
      mx = fmaxf(mx, lg_other_half(mx));
      const bool none = mref == -INFINITY;
      if constexpr (FOLLOW) {
        if (__builtin_amdgcn_ballot_w64(!none && (mx - mref) * scale_log2e > 8.0f) != 0) {  // (one row's moves its neighbours')
          asm volatile("; rescale accumulators" ::: "memory");  // (likewise a real branch)
          const float mnew = fmaxf(mref, mx);
          const float alpha = mnew == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((mref - mnew) * scale_log2e);
          mref = mnew;
          lrow *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
        }
      }
      mref = none ? mx : mref;
      if (!FOLLOW) watch = __builtin_amdgcn_ballot_w64(mref == -INFINITY) != 0;
    }
    const float moff = (mref == -INFINITY) ? 0.f : mref * scale_log2e;
    float psum[2] = {0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint32_t w[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(sacc[kb][8 * h + 2 * x], scale_log2e, -moff));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(sacc[kb][8 * h + 2 * x + 1], scale_log2e, -moff));
          w[x] = lg_pack_bf16(p0, p1);
          // row sum of the ROUNDED probabilities: the same values the second product uses
          psum[kb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w[x]), ones, psum[kb], false);
        }
        pf[2 * kb + h] = lg_as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
      }
    const float sum = psum[0] + psum[1];
    // (not a number: left as well, so that its neighbours in the wave are treated as by FOLLOW)
    if (!FOLLOW && __builtin_expect(__builtin_amdgcn_ballot_w64(!(sum <= 192.f)) != 0, 0)) return true;
    lrow += sum;
    }
    if (!FEW) {
      LG_WAIT_VMCNT(0);
      __syncthreads();  // V(t) landed; everyone is done with K(t)
      if (t2 >= 0) issue_k(t2, buf);
    }
    if (kind != LG_TILE_DEAD) {
    // ---- O^T += V^T P^T ----
      if (!FEW) vring.begin(read_v);
      vring.run(read_v, [&](int u, bf16x8_t v) { oacc[u % DB] = lg_mfma32(v, pf[u / DB], oacc[u % DB]); });
    }  // kind != dead

    t = t1;
    t1 = t2;
    kind0 = kind1;
    kind1 = kind2;
    buf ^= 1;
    return false;
  };
  bool left = false;
  if constexpr (!FEW)
    while (t >= 0 && !left) left = tile(std::false_type{}, false);
  for (; t >= 0; left = false) tile(std::true_type{}, !FEW && left);

  if (FEW) __syncthreads();  // everyone is done with the K tiles
  // ---- epilogue: normalise, write O (bf16) and LSE (natural log) ----
  const float l = lrow + lg_other_half(lrow);
  const float inv = 1.f / l;
  // (the K tiles' place is free: nobody reads it behind the last tile's second barrier)
  unsigned char* rows = smem + wave_s * (32 * T::ROW_BYTES);
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    float o[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) o[r] = oacc[db][r];
    lg_rows_put<D>(rows, lane, db, o, inv);
  }
  lg_rows_write<D>(rows, lane, out + qbase + (size_t)(q0 + wave_s * 32) * D, N - (q0 + wave_s * 32));
  const int i = q0 + wave * 32 + n;  // this lane's query row
  if (lse != nullptr && g == 0 && i < N)
    lse[(size_t)(b * Hq + hq) * m.ld + seq_row0 + i] = (mref * scale_log2e + log2f(l)) * 0.69314718055994530942f;
}

}  // namespace

// The launches of LIST instances (lg_fwd_list_bf16.hip).  pack: NULL for the batch layout.
void lg_launch_fwd_list_bf16(const void* q, const void* k, const void* v, void* out, float* lse, const LgShape& sh, float scale_log2e,
                             const LgMask& m, const LgItems& items, const LgPackFew* pack, unsigned grid, hipStream_t s);

#endif  // LG_FWD_BF16_H_

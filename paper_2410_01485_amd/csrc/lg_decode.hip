// lg_decode.hip — decode over the sink + rolling-window KV cache (paper Section 3.2,
// second paragraph: at inference the bottleneck is loading the KV cache as fast as
// possible; the attention-sink variant keeps the window in a rolling buffer).
//
// One query per (b, hq); every valid cache slot is read exactly once, for all query heads of a kv head (up to 16) at
// once, on the matrix cores (decode_mfma_kernel).
// The slots of one (b, hkv) are split over workgroups so the chip is filled even for small batches; each leaves
// its normalised result and log-sum-exp in the workspace, and a second launch adds them (decode_add_kernel).
//
// The keys of a step are up to four runs of consecutive slots (LgDecSegs: sink tokens,
// live part of the rolling window, retained strided blocks); the kernels walk their
// concatenation.  The common case, one run starting at slot 0, has its own instance
// without the index translation.  A third instance serves paged caches with per-sequence
// context lengths: the runs are computed per sequence on the device and a slot goes through
// the sequence's page table.
//
// lg_kv_append_kernel stores new tokens into the cache rows by the same layout rule.
#include <hip/hip_bf16.h>

#include "../../include/longgen_attn.h"
#include "lg_kernels.h"
#include "lg_mask.h"
#include "lg_mfma.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace {

constexpr int WAVES = 4;
constexpr int WIDE = 12;  // waves of a workgroup that takes a whole row of few keys

// E elements of T loaded as one 16-byte vector, widened to float.  The loads are marked
// non-temporal: every cache byte is used exactly once per call, so keeping it in L2 / the
// memory-side cache only evicts something else (measured: 181 -> 164 us at B16 x 32 heads x
// 4160 slots).
typedef unsigned lg_u32x4 __attribute__((ext_vector_type(4)));
typedef float lg_f32x4 __attribute__((ext_vector_type(4)));
template <typename T, int E>
struct Frag;
template <>
struct Frag<float, 4> {
  __device__ static void load(const void* p, float* f) {
    const lg_f32x4 x = __builtin_nontemporal_load(reinterpret_cast<const lg_f32x4*>(p));
    f[0] = x.x; f[1] = x.y; f[2] = x.z; f[3] = x.w;
  }
};
template <>
struct Frag<__hip_bfloat16, 8> {
  __device__ static void load(const void* p, float* f) {
    const lg_u32x4 x = __builtin_nontemporal_load(reinterpret_cast<const lg_u32x4*>(p));
    const unsigned w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f[2 * t] = __uint_as_float(w[t] << 16);
      f[2 * t + 1] = __uint_as_float(w[t] & 0xffff0000u);
    }
  }
};

__device__ __forceinline__ void store_out(float* p, float x) { *p = x; }
__device__ __forceinline__ void store_out(__hip_bfloat16* p, float x) { *p = __float2bfloat16(x); }

// Running maxima are in the log2 domain: score * scale * log2(e).
// What a paged launch adds to the arguments.
struct LgPaged {
  const int* page_table;  // [B, pages_per_seq]
  const int* seq_lens;    // [B]
  int pages_per_seq, page_shift, n_max, num_pages, B;
  int keys_max;           // no sequence has more keys
  int few;                // workgroups of a small step
  LgMask cm;              // cache geometry (lg_make_cache_mask), N filled in per sequence
};

enum { LG_DEC_PLAIN = 0, LG_DEC_SEGS = 1, LG_DEC_PAGED = 2 };
// What an instance receives beyond the common arguments, and no more: a launch with 260 bytes of arguments takes the host
// 0.2 us longer than one with 12 (1 us when launches follow each other without a pause), and a short step waits for the
// host; with nothing but its own, the paged instance also needs fewer registers' worth of scalar loads (48 sequences of
// 20 .. 32768 tokens, 8 kv heads, with the append: 77.2 -> 71.1 us).
template <int MODE>
struct LgDecExtra {};
template <>
struct LgDecExtra<LG_DEC_SEGS> {
  LgDecSegs segs;
};
template <>
struct LgDecExtra<LG_DEC_PAGED> {
  LgPaged pg;
};

// ---------------------------------------------------------------- work of a decode launch
// The keys of every (b, kv head, head chunk) -- a "row" here -- are cut into `splits` parts of `chunk` keys; a
// workgroup takes one part.  (Paged: as many parts as the sequence's own length fills; the workgroups beyond leave.)
// Rows of several parts are added up by decode_add_kernel.
struct LgDecWork {
  int splits, chunk;  // (paged: the most parts of a row and the least keys of a part)
  float* o;           // [rows][splits][G][D]: normalised results of the parts
  float* lse2;        // [rows][splits][G]: their log2-sum-exp
  int* parts;         // [rows], paged: parts of the row
};
constexpr int LG_DEC_SPLITS_MAX = 64;
// Workgroups with keys that a paged step aims at: DEC_FULL less a quarter of its rows (b, kv head), a little below three per
// CU, what the matrix-core kernel's registers admit, or (bf16) one per CU when all rows together have so few keys that a
// workgroup's start and the final sum weigh more than its reads.  Rounding gives at most one part more per row.  With 768
// the last of 900 workgroups ran after the others: 64 sequences of 2000 .. 60000 tokens, 8 kv heads 184 us, with 720 165
// (float32 380, 331); 48 of 20 .. 32768 60 and 60 (136, 136), as are other batches; with 640 the latter lost 7 %, whole
// rounds missing on part of the CUs.
constexpr int DEC_FULL = 720, DEC_FEW = 256;
constexpr float DEC_MANY_KEYS = 300000.f;

struct LgDecPart {
  int b, q;           // sequence, and kv head * chunks + chunk
  int s0, s1;         // its keys
  int split, parts;   // of the row
  size_t row;
};

// Sums over the lanes up to and including each one (as shifts between the lanes of a row, no trip through LDS).
template <typename T>
__device__ __forceinline__ T lg_wave_scan(T x) {
  auto add = [&](auto ctrl, auto rows) {
    const int y = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
    x += __builtin_bit_cast(T, y);
  };
  add(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});  // lane - 1, in rows of 16 lanes
  add(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});  // lane - 2
  add(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});  // lane - 4
  add(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});  // lane - 8
  add(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});  // last lane of row 0 to row 1, of 2 to 3
  add(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});  // lane 31 to rows 2 and 3
  return x;
}

// The runs of a sequence of N tokens of a paged launch; returns the number of its keys.
__device__ __forceinline__ int lg_dec_sequence(const LgPaged& pg, int N, LgDecSegs& segs) {
  if (pg.cm.b == 1 && pg.cm.stride == 0) {  // token-granular: the slots in use are one run
    segs.start[0] = 0;
    segs.pre[1] = segs.pre[2] = segs.pre[3] = 0x7fffffff;
    return min(N, pg.cm.sink + pg.cm.window);
  }
  LgMask cm = pg.cm;
  cm.N = N;
  return lg_decode_runs(cm, segs);
}
// The part of this workgroup; false: none.  Grid: splits x rows of a sequence x B.  Paged (heads: rows of a sequence):
// one dimension, the parts of all sequences one after the other; segs receives the sequence's runs.
template <int MODE>
__device__ __forceinline__ bool lg_dec_part(const LgDecWork& wk, const LgPaged& pg, int heads, LgDecSegs& segs,
                                            int valid, LgDecPart& p) {
  if (MODE != LG_DEC_PAGED) {
    p.split = blockIdx.x;
    p.q = blockIdx.y;
    p.b = blockIdx.z;
    p.row = (size_t)p.b * heads + p.q;
    p.parts = wk.splits;
    p.s0 = p.split * wk.chunk;
    p.s1 = min(valid, p.s0 + wk.chunk);
    return p.s0 < valid;
  }
  // No row has parts (the longest context has too few keys): a workgroup per row, nothing to find out about the others.  With the
  // runs in registers, graph of append and decode, us: 8 kv heads, 1 sequence of 120 keys 8.1 -> 7.0, 300 10.5 -> 9.4; 32 of 300 14.3 ->
  // 12.8; 16 of 4160 (parts) 57.9 -> 55.9.
  if (wk.splits == 1) {
    p.row = blockIdx.x;
    p.b = p.row / heads;
    p.q = (int)p.row - p.b * heads;
    p.split = 0;
    p.parts = 1;
    p.s0 = 0;
    p.s1 = lg_dec_sequence(pg, min(max(pg.seq_lens[p.b], 1), pg.n_max), segs);
    return true;
  }
  // The lengths of the batch set the size of a part: about as many workgroups as the GPU holds at a time (fewer for a
  // step that is over in a few rounds anyway), no more parts per row than the workspace has room for.  As a grid of
  // (parts of the longest) x rows, with workgroups that find nothing to do, the others came out uneven over the CUs.
  const int lane = threadIdx.x & 63, B = pg.B;
  auto length = [&](int x) { return x < B ? pg.seq_lens[x] : 0; };
  auto keys = [&](int x, int n) { return x < B ? min(max(n, 1), pg.keys_max) : 0; };  // never too few
  const int first_n = length(lane), first = keys(lane, first_n);  // (a batch of up to 64: the only look at the lengths)
  float sum = (float)first;
  for (int x = 64 + lane; x < B; x += 64) sum += (float)keys(x, length(x));
  const float all = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(lg_wave_scan(sum)), 63)) * heads;
  const float target = all > DEC_MANY_KEYS ? fmaxf(DEC_FULL - 0.25f * B * heads, DEC_FEW) : (float)pg.few;
  const int chunk = max(wk.chunk, 128 * __builtin_amdgcn_readfirstlane((int)ceilf(all / (128.f * target))));
  // Rows are cut evenly.  What is left over goes to the others where the reads decide, up to a quarter of a part, and to a
  // row's only part always (no sum over parts then): a part of a few keys costs a workgroup's place for nothing (48
  // sequences of 20 .. 32768 tokens, 8 kv heads, with the append: 75.7 -> 71.3 us).
  const int spare = all > DEC_MANY_KEYS ? chunk >> 2 : 0;
  auto nparts = [&](int k) { return k <= chunk + (chunk >> 2) ? 1 : (k - spare + chunk - 1) / chunk; };
  const int w = blockIdx.x;
  int before = 0, N = 0;
  for (int c = 0; c < B; c += 64) {
    const int n = c == 0 ? first_n : length(c + lane), k = keys(c + lane, n);
    const int mine = k > 0 ? nparts(k) * heads : 0, upto = lg_wave_scan(mine);
    const unsigned long long past = __builtin_amdgcn_ballot_w64(before + upto > w);
    if (past != 0ull) {
      const int x = __builtin_ctzll(past);
      p.b = c + x;
      N = min(max(__builtin_amdgcn_readlane(n, x), 1), pg.n_max);
      const int at = w - before - __builtin_amdgcn_readlane(upto - mine, x);
      p.split = at / heads;
      p.q = at - p.split * heads;
      break;
    }
    before += __builtin_amdgcn_readlane(upto, 63);
    if (c + 64 >= B) return false;
  }
  p.row = (size_t)p.b * heads + p.q;
  valid = lg_dec_sequence(pg, N, segs);
  const int np = nparts(valid);
  if (np == 1) {
    p.parts = 1;
    p.s0 = 0;
    p.s1 = valid;
    return p.split == 0;
  }
  const int per = ((valid + np - 1) / np + 31) & ~31;
  p.parts = (valid + per - 1) / per;
  p.s0 = p.split * per;
  p.s1 = min(valid, p.s0 + per);
  return p.s0 < valid;
}

// What exponents are taken relative to: a maximum, or 0 where no score is finite (-inf - -inf is NaN; this way every
// weight is 0 there).
__device__ __forceinline__ float lg_finite_ref(float m) { return m == -INFINITY ? 0.f : m; }

// log2-sum-exp of head g from the waves' maxima and sums (-inf where every score is)
template <int W, int N>
__device__ __forceinline__ float lg_lse2(const float (&sM)[W][N], const float (&sL)[W][N], int g) {
  float M = -INFINITY, L = 0.f;
#pragma unroll
  for (int w = 0; w < W; ++w) M = fmaxf(M, sM[w][g]);
#pragma unroll
  for (int w = 0; w < W; ++w) L += sL[w][g] * exp2f(sM[w][g] - lg_finite_ref(M));
  return M + log2f(L);
}

// Cache row of key `slot` of the concatenated runs.
__device__ __forceinline__ int lg_dec_slot(const LgDecSegs& segs, int slot) {
  int shift = segs.start[0];
  if (slot >= segs.pre[1]) shift = segs.start[1] - segs.pre[1];
  if (slot >= segs.pre[2]) shift = segs.start[2] - segs.pre[2];
  if (slot >= segs.pre[3]) shift = segs.start[3] - segs.pre[3];
  return slot + shift;
}
// Row of slot `slot` of sequence b in a paged pool.  (A table entry outside the pool is clamped into it: a wrong
// result, never a stray read.)
__device__ __forceinline__ size_t lg_dec_page_row(const LgPaged& pg, int b, int Hkv, int hk, int slot) {
  const int page = min(max(pg.page_table[(size_t)b * pg.pages_per_seq + (slot >> pg.page_shift)], 0), pg.num_pages - 1);
  return (((size_t)page * Hkv + hk) << pg.page_shift) + (slot & ((1 << pg.page_shift) - 1));
}

// ---------------------------------------------------------------- matrix cores
// All G <= 16 query heads of a kv head at once.  On the vector ALUs every head costs a multiply-add per element of K
// and V and a reduction over the lanes of a row: with 8 heads that kernel ran at 1.2 TB/s, a sixth of what it reads
// at with one.  Here a wave takes a unit of 32 keys at a time on 16x16x32 instructions:
//   S (keys x heads) = K Q^T    A operand: lane (n, h) loads 16 bytes (dims 32 c + 8 h ..) of key row n straight from
//                               memory; the two 16-key blocks take rows so that register r of block x at lane group h
//                               is key 8 h + 4 x + r
//   O^T (dims x heads) += V^T P contraction slots 8 h .. 8 h + 7 = keys 8 h .. 8 h + 7: the B operand is the lane's
//                               own P values; for A a lane loads its VE dims of those 8 keys (whole rows over the 16
//                               lanes) and pairs them up with byte permutes
// No LDS on the way.  P enters the second product as three bf16 terms, which hold all 24 bits of the float32 value:
// K, V and Q are used as stored, sums are float32.  V goes past the caches (every byte is used once); K is read in
// half lines by two loads each, so it does not (both non-temporal: 94 instead of 86 us at 545 MB).  Bound: memory; per
// 16 KB (D = 128) a wave spends 512 matrix and about 600 vector cycles, several times less than the bytes take.
// Measured with the append (vector kernel -> this): 16 x 32 heads x 4160 slots 164 -> 161 us (6.8 TB/s); 8 x 8 kv heads of
// 8 query heads x 3648 slots 102 -> 26 us; 48 sequences of 20 .. 32768 tokens, 8 kv heads of 4 query heads, paged 112 -> 71.
// float32: units of 16 keys (as many bytes) on 16x16x4 float32 instructions: lane (n, h) loads dims 16 c + 4 h .. of key
// row n (contraction step (c, e): its element e; the four lane groups together dims 16 c + e, + 4, + 8, + 12), register r
// of S is key 4 h + r, which is the B operand of the second product's step r as it is; a lane loads dims 4 n .. (+ 64) of
// those 4 keys of V.  A unit takes 2048 matrix cycles, a third of what its bytes take at three workgroups per CU.
// Measured (vector kernel -> this): 8 x 8 kv heads of 8 query heads x 4160 slots 99 -> 51 us; 4 x 8 kv heads of 4 x 2112
// slots 40 -> 18 us; 8 x 32 heads x 4160 slots 197 -> 158 us; one head of 64, 364 slots 10.3 -> 6.8 us.
template <typename T>
struct LgDecElem {
  typedef T type;
};
template <>
struct LgDecElem<__hip_bfloat16> {
  typedef uint16_t type;
};
template <typename T, int D>
struct LgDecUnit {  // what a lane holds of a unit
  static constexpr int KEYS = 32;
  typedef unsigned vrow_t __attribute__((ext_vector_type(D / 32)));
  lg_u32x4 k[2][D / 32];
  vrow_t v[8];
};
template <int D>
struct LgDecUnit<float, D> {
  static constexpr int KEYS = 16;
  f32x4_t k[D / 16];
  f32x4_t v[4][D / 64];
};

template <typename TT, int D, int MODE, int W>
__global__ __launch_bounds__(W * 64, W == WAVES ? 3 : W / 4) void decode_mfma_kernel(
    const typename LgDecElem<TT>::type* __restrict__ q, const typename LgDecElem<TT>::type* __restrict__ kc,
    const typename LgDecElem<TT>::type* __restrict__ vc, TT* __restrict__ out, float* __restrict__ lse, LgDecWork wk,
    int Hq, int Hkv, int C, int valid, float qmul, float scale_log2e, float scale_pow2, LgDecExtra<MODE> extra) {
  constexpr bool F32 = sizeof(TT) == 4;
  constexpr int UNIT = LgDecUnit<TT, D>::KEYS;
  constexpr int DC = D / (F32 ? 16 : 32), VE = D / 16;  // loads of a key row; 16-dim blocks of O
  constexpr int PAGES = 1024;                           // page-table entries of a sequence kept in LDS
  __shared__ float sO[W][16][D + 4];
  __shared__ float sM[W][16], sL[W][16];
  __shared__ int spage[MODE == LG_DEC_PAGED ? PAGES : 1];

  LgDecSegs segs;  // (paged: of the sequence, from lg_dec_part)
  LgPaged pg;
  if constexpr (MODE == LG_DEC_SEGS) segs = extra.segs;
  if constexpr (MODE == LG_DEC_PAGED) pg = extra.pg;
  const int G = Hq / Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, h = lane >> 4;
  const int ka = 8 * (n >> 2) + (n & 3);  // this lane's key of block 0 (block 1: + 4)
  LgDecPart p;
  if (!lg_dec_part<MODE>(wk, pg, Hkv, segs, valid, p)) return;
  const int b = p.b, hk = p.q;
  const size_t out_row = (size_t)b * Hq + hk * G;
  uint4 qf[DC];  // (F32: dims 16 c + 4 h .., else 32 c + 8 h ..)
#pragma unroll
  for (int c = 0; c < DC; ++c) {
    qf[c] = make_uint4(0u, 0u, 0u, 0u);
    if (n < G) qf[c] = *reinterpret_cast<const uint4*>(q + (out_row + n) * D + (F32 ? 16 * c + 4 * h : 32 * c + 8 * h));
  }
  // Q takes the power of two of the scale, so that a score overflows where the scaled one does, not |1 / scale| earlier.
  // Exact but for products below the smallest normal number: at most 2^-133 |k| per term of a scaled score.
  auto scale_q = [&] {
#pragma unroll
    for (int c = 0; c < DC; ++c) {
      uint32_t w[4] = {qf[c].x, qf[c].y, qf[c].z, qf[c].w};
#pragma unroll
      for (int x = 0; x < 4; ++x)
        w[x] = F32 ? __float_as_uint(__uint_as_float(w[x]) * qmul)
                   : lg_pack_bf16(__uint_as_float(w[x] << 16) * qmul, __uint_as_float(w[x] & 0xffff0000u) * qmul);
      qf[c] = make_uint4(w[0], w[1], w[2], w[3]);
    }
  };
  f32x4_t acc[VE];
#pragma unroll
  for (int i = 0; i < VE; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float mref = -INFINITY, lrow = 0.f;
  float cl = scale_log2e, moff = 0.f;  // P = exp2(S cl - moff)

  const size_t head = MODE == LG_DEC_PAGED ? 0 : ((size_t)b * Hkv + hk) * C * D;
  const auto* kb_ = kc + head;
  const auto* vb_ = vc + head + (F32 ? 4 : VE) * n;
  const int r1 = p.s1;
  // The sequence's page-table entries go to LDS first (a table of more than PAGES entries is read in place: behind
  // each unit's loads, which keeps the next unit's waiting).
  const bool in_lds = MODE == LG_DEC_PAGED && pg.pages_per_seq <= PAGES;
  if (in_lds) {
    for (int x = tid; x < pg.pages_per_seq; x += W * 64)
      spage[x] = min(max(pg.page_table[(size_t)b * pg.pages_per_seq + x], 0), pg.num_pages - 1);
    __syncthreads();
  }
  // cache row of key key0 + lane % UNIT of a unit; the lanes hand them round
  auto resolve = [&](int key0, auto IN_LDS) -> unsigned {
    if (MODE == LG_DEC_PLAIN) return 0;
    const int slot = lg_dec_slot(segs, min(key0 + (lane & (UNIT - 1)), r1 - 1));
    if (MODE == LG_DEC_SEGS) return slot;
    // (rows of a pool that fits the memory: below 2^32)
    if (!decltype(IN_LDS)::value) return lg_dec_page_row(pg, b, Hkv, hk, slot);
    return (((unsigned)spage[slot >> pg.page_shift] * Hkv + hk) << pg.page_shift) + (slot & ((1 << pg.page_shift) - 1));
  };
    using Unit = LgDecUnit<TT, D>;
    auto load = [&](Unit& t, int key0, unsigned rows) {
      if constexpr (F32) {
        const unsigned r = MODE == LG_DEC_PLAIN ? (unsigned)min(key0 + n, r1 - 1) : __shfl(rows, n);
#pragma unroll
        for (int c = 0; c < DC; ++c)
          t.k[c] = *reinterpret_cast<const f32x4_t*>(kb_ + (size_t)r * D + 16 * c + 4 * h);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const unsigned rv = MODE == LG_DEC_PLAIN ? (unsigned)min(key0 + 4 * h + j, r1 - 1) : __shfl(rows, 4 * h + j);
#pragma unroll
          for (int x = 0; x < D / 64; ++x)
            t.v[j][x] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(vb_ + (size_t)rv * D + 64 * x));
        }
      } else {
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const unsigned r = MODE == LG_DEC_PLAIN ? (unsigned)min(key0 + ka + 4 * x, r1 - 1) : __shfl(rows, ka + 4 * x);
#pragma unroll
        for (int c = 0; c < DC; ++c)
          t.k[x][c] = *reinterpret_cast<const lg_u32x4*>(kb_ + (size_t)r * D + 32 * c + 8 * h);
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const unsigned r = MODE == LG_DEC_PLAIN ? (unsigned)min(key0 + 8 * h + j, r1 - 1) : __shfl(rows, 8 * h + j);
        t.v[j] = __builtin_nontemporal_load(reinterpret_cast<const typename Unit::vrow_t*>(vb_ + (size_t)r * D));
      }
      }
    };
    constexpr int NX = F32 ? 1 : 2;  // 16-key blocks of S
    auto compute = [&](const Unit& t, int key0) {
      f32x4_t s[NX];
#pragma unroll
      for (int x = 0; x < NX; ++x) {
        s[x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < DC; ++c)
          if constexpr (F32) {
            const f32x4_t qv = __builtin_bit_cast(f32x4_t, qf[c]);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.k[c][e], qv[e], s[x], 0, 0, 0);
          } else {
            s[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, t.k[x][c]), lg_as_bf16x8(qf[c]),
                                                           s[x], 0, 0, 0);
          }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (key0 + 4 * NX * h + 4 * x + r >= r1) s[x][r] = -INFINITY;
          mx = fmaxf(mx, s[x][r]);
        }
      // the exponent's reference moves only when a maximum has outgrown it by 2^8
      if (__builtin_amdgcn_ballot_w64((mx - mref) * scale_log2e > 8.0f) != 0) {
        float mnew = fmaxf(mx, mref);
        mnew = fmaxf(mnew, __shfl_xor(mnew, 16));
        mnew = fmaxf(mnew, lg_other_half(mnew));
        const float alpha = mnew == -INFINITY ? 1.f : exp2f((mref - mnew) * scale_log2e);
        mref = mnew;
        // From 2^30 on the rounding of mref * scale would show as a factor beyond the exponent's range.  Distinct scores
        // are then at least 2^5 apart, and the scale's power of two, with which the product is exact, serves as well.
        const bool far = fabsf(mref * scale_log2e) >= 0x1p30f;
        cl = far ? scale_pow2 : scale_log2e;
        moff = lg_finite_ref(mref) * cl;
        lrow *= alpha;
#pragma unroll
        for (int i = 0; i < VE; ++i) acc[i] *= alpha;
      }
      if constexpr (F32) {
        float pr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          pr[r] = exp2f(fmaf(s[0][r], cl, -moff));
          lrow += pr[r];
        }
#pragma unroll
        for (int i = 0; i < VE; ++i)  // dim 64 (i / 4) + 4 n + i % 4
#pragma unroll
          for (int r = 0; r < 4; ++r)
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.v[r][i / 4][i % 4], pr[r], acc[i], 0, 0, 0);
      } else {
      uint32_t w[3][4];  // P in three bf16 terms
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        float p0 = exp2f(fmaf(s[y >> 1][2 * (y & 1)], cl, -moff));
        float p1 = exp2f(fmaf(s[y >> 1][2 * (y & 1) + 1], cl, -moff));
        lrow += p0 + p1;
#pragma unroll
        for (int z = 0; z < 3; ++z) {
          w[z][y] = lg_pack_bf16(p0, p1);
          p0 -= __uint_as_float(w[z][y] << 16);
          p1 -= __uint_as_float(w[z][y] & 0xffff0000u);
        }
      }
      bf16x8_t pf[3];
#pragma unroll
      for (int z = 0; z < 3; ++z) pf[z] = lg_as_bf16x8(make_uint4(w[z][0], w[z][1], w[z][2], w[z][3]));
#pragma unroll
      for (int i = 0; i < VE; ++i) {  // dim VE n + i of keys 8 h .. 8 h + 7
        uint32_t a[4];
#pragma unroll
        for (int y = 0; y < 4; ++y)
          a[y] = __builtin_amdgcn_perm(t.v[2 * y + 1][i / 2], t.v[2 * y][i / 2], (i & 1) ? 0x07060302u : 0x05040100u);
        const bf16x8_t av = lg_as_bf16x8(make_uint4(a[0], a[1], a[2], a[3]));
#pragma unroll
        for (int z = 0; z < 3; ++z) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, pf[z], acc[i], 0, 0, 0);
      }
      }
    };
    constexpr int STEP = UNIT * W;
    auto all_units = [&](auto IN_LDS) {
      unsigned rows = resolve(p.s0 + UNIT * wave, IN_LDS);
      for (int key = p.s0 + UNIT * wave; key < r1; key += STEP) {
        Unit t;
        load(t, key, rows);
        rows = resolve(key + STEP, IN_LDS);
        __builtin_amdgcn_sched_barrier(0);  // all of the unit's loads are issued before anything waits for one
        if (key == p.s0 + UNIT * wave) scale_q();  // (here: while the first unit's loads are on their way)
        compute(t, key);
      }
    };
    if (MODE != LG_DEC_PAGED || in_lds) all_units(std::true_type{});
    else all_units(std::false_type{});

  // merge the waves: acc[i] register r is dim VE (4 h + r) + i of head n (float32: 64 (i / 4) + 4 (4 h + r) + i % 4)
  lrow += __shfl_xor(lrow, 16);
  lrow += lg_other_half(lrow);
  if (n < G) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int i = 0; i < VE; ++i) sO[wave][n][F32 ? 64 * (i / 4) + 4 * (4 * h + r) + i % 4 : VE * (4 * h + r) + i] = acc[i][r];
    if (h == 0) {
      sM[wave][n] = mref == -INFINITY ? -INFINITY : mref * scale_log2e;
      sL[wave][n] = lrow;
    }
  }
  __syncthreads();
  for (int e = tid; e < G * D / 2; e += W * 64) {
    const int g = e / (D / 2), d = 2 * (e % (D / 2));
    float M = -INFINITY;
#pragma unroll
    for (int x = 0; x < W; ++x) M = fmaxf(M, sM[x][g]);
    float L = 0.f, a0 = 0.f, a1 = 0.f;
#pragma unroll
    for (int x = 0; x < W; ++x) {
      const float f = exp2f(sM[x][g] - lg_finite_ref(M));
      L += sL[x][g] * f;
      a0 += sO[x][g][d] * f;
      a1 += sO[x][g][d + 1] * f;
    }
    const float inv = p.parts > 1 && L == 0.f ? 0.f : 1.f / L;  // (a part without a finite score adds nothing to its row)
    if (p.parts == 1) {
      if constexpr (F32) {
        *reinterpret_cast<float2*>(out + out_row * D + 2 * e) = make_float2(a0 * inv, a1 * inv);
      } else {
        *reinterpret_cast<uint32_t*>(out + out_row * D + 2 * e) = lg_pack_bf16(a0 * inv, a1 * inv);
      }
      if (lse != nullptr && d == 0) lse[out_row + g] = (M + log2f(L)) * 0.69314718055994530942f;
    } else {
      const size_t at = (p.row * wk.splits + p.split) * G;
      *reinterpret_cast<float2*>(wk.o + at * D + 2 * e) = make_float2(a0 * inv, a1 * inv);
    }
  }
  if (p.parts > 1 && tid < G) wk.lse2[(p.row * wk.splits + p.split) * G + tid] = lg_lse2(sM, sL, tid);
  if (MODE == LG_DEC_PAGED && wk.splits > 1 && p.split == 0 && tid == 0) wk.parts[p.row] = p.parts;
}

// Adds the parts of a row, a wave for each query head: the weights of up to 64 parts in its lanes, D / 64 dims in each.
// A launch of its own rather than the last of a row's workgroups to finish: nothing in the workspace is read that this
// call has not written, and the GPU gets through it no slower (1 sequence of 32/8 heads, 1500 tokens, append and decode
// replayed from a graph: 9.8 -> 9.1 us; 8 x 64/8 heads, 3648 slots: 27.0 -> 25.9).  A program that issues one short decode
// after the other waits for the host's third launch (the same sequence without a graph: 10.0 -> 12 us).
template <typename T, int D, bool PAGED>
__global__ __launch_bounds__(64) void decode_add_kernel(LgDecWork wk, int G, T* __restrict__ out, float* __restrict__ lse) {
  constexpr int E = D / 64, AHEAD = 16;  // loads in flight
  typedef float vec_t __attribute__((ext_vector_type(E)));
  const int lane = threadIdx.x, row = blockIdx.x / G, g = blockIdx.x - row * G;
  const size_t rec = (size_t)row * wk.splits;
  const float* po = wk.o + (rec * G + g) * D + E * lane;
  // (the first parts are requested before their number is known: every address is inside the workspace)
  const float mine = wk.lse2[(rec + min(lane, wk.splits - 1)) * G + g];
  const int np = PAGED ? min(__builtin_amdgcn_readfirstlane(wk.parts[row]), wk.splits) : wk.splits;
  vec_t x[AHEAD], acc = {};
  auto load = [&](int s0) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) x[u] = *reinterpret_cast<const vec_t*>(po + (size_t)min(s0 + u, wk.splits - 1) * G * D);
  };
  load(0);
  if (np == 1) return;  // (written by its workgroup)
  const float l = lane < np ? mine : -INFINITY;
  float M = l;
#pragma unroll
  for (int y = 1; y < 64; y <<= 1) M = fmaxf(M, __shfl_xor(M, y));
  float w = exp2f(l - lg_finite_ref(M)), sum = w;
#pragma unroll
  for (int y = 1; y < 64; y <<= 1) sum += __shfl_xor(sum, y);
  if (lse != nullptr && lane == 0) lse[(size_t)row * G + g] = (M + log2f(sum)) * 0.69314718055994530942f;
  w /= sum;
  for (int s0 = 0; s0 < np; s0 += AHEAD) {
    if (s0 > 0) load(s0);
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
      if (s0 + u < np) {
        const float wu = __shfl(w, s0 + u);
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = fmaf(wu, x[u][e], acc[e]);
      }
  }
#pragma unroll
  for (int e = 0; e < E; ++e) store_out(out + ((size_t)row * G + g) * D + E * lane + e, acc[e]);
}

// One thread per 16 bytes of a new token row (K and V): the token goes to its sink or ring
// slot unless a later token of the same call lands on that ring slot, and to its retained-block
// slot when its block is a strided column.  No two threads write the same bytes.
// Only rows that are stored are read, and without strided columns only they have threads (first: kept tokens at the start
// of the call, second: the first of those at its end): of a prompt longer than the window few are (1 x 32 heads of 128,
// 32768 tokens, window 4096: 110 -> 21 us; 1 x 16 heads of 64, 54868, window 741: 32 -> 3).
template <int LPR>
__global__ __launch_bounds__(256) void lg_kv_append_kernel(const uint4* __restrict__ kn,
                                                           const uint4* __restrict__ vn,
                                                           uint4* __restrict__ kc, uint4* __restrict__ vc,
                                                           int T, int pos, int slots, LgMask m, int first, int second) {
  int ti = blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
  if (ti >= first) ti += second - first;
  if (ti >= T) return;
  const int c = threadIdx.x % LPR;
  const size_t head = (size_t)blockIdx.z * gridDim.y + blockIdx.y;
  const size_t src = (head * T + ti) * LPR + c;
  const int p = pos + ti, last = pos + T - 1;
  const size_t row0 = head * slots;
  const bool ring = p < m.sink || (long long)p + m.window > last;
  const int kb = m.stride > 0 ? lg_div_b(m, p) : 0;
  const bool retained = m.stride > 0 && lg_strided(m, kb);
  if (!ring && !retained) return;
  const uint4 kx = kn[src], vx = vn[src];
  if (ring) {
    const int slot = p < m.sink ? p : m.sink + (p - m.sink) % m.window;
    kc[(row0 + slot) * LPR + c] = kx;
    vc[(row0 + slot) * LPR + c] = vx;
  }
  if (retained) {
    const int slot = m.sink + m.window + (kb / m.stride) * m.b + (p - kb * m.b);
    kc[(row0 + slot) * LPR + c] = kx;
    vc[(row0 + slot) * LPR + c] = vx;
  }
}

// The same for a paged cache: per-sequence start positions, slots go through the page table.
template <int LPR>
__global__ __launch_bounds__(256) void lg_kv_paged_append_kernel(const uint4* __restrict__ kn,
                                                                 const uint4* __restrict__ vn,
                                                                 uint4* __restrict__ kp, uint4* __restrict__ vp,
                                                                 const int* __restrict__ page_table,
                                                                 const int* __restrict__ positions, int T,
                                                                 int pages_per_seq, int page_shift, int num_pages,
                                                                 LgMask m) {
  const int ti = blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
  if (ti >= T) return;
  const int c = threadIdx.x % LPR;
  const int Hkv = gridDim.y, hk = blockIdx.y, b = blockIdx.z;
  const size_t src = (((size_t)b * Hkv + hk) * T + ti) * LPR + c;
  const uint4 kx = kn[src], vx = vn[src];
  const int pos = max(positions[b], 0);
  const int p = pos + ti, last = pos + T - 1;
  auto put = [&](int slot) {
    // (a table entry outside the pool is clamped into it: a misplaced row, never a stray write)
    const int page = min(max(page_table[(size_t)b * pages_per_seq + (slot >> page_shift)], 0), num_pages - 1);
    const size_t row = (((size_t)page * Hkv + hk) << page_shift) + (slot & ((1 << page_shift) - 1));
    kp[row * LPR + c] = kx;
    vp[row * LPR + c] = vx;
  };
  if (p < m.sink || (long long)p + m.window > last) put(p < m.sink ? p : m.sink + (p - m.sink) % m.window);
  if (m.stride > 0) {
    const int kb = lg_div_b(m, p);
    if (lg_strided(m, kb)) {
      const int slot = m.sink + m.window + (kb / m.stride) * m.b + (p - kb * m.b);
      if ((slot >> page_shift) < pages_per_seq) put(slot);  // positions beyond the table's reach are dropped
    }
  }
}

// ---------------------------------------------------------------- measurement aid
// The paper's decode design splits the LOADING OF THE HEAD DIMENSION across thread blocks instead
// of the cache slots (Section 3.2, second paragraph).  Read here as: block s of S loads dims
// [s*D/S, (s+1)*D/S) of every K row and produces partial scores; a second pass sums the S partial
// scores of a slot, runs the softmax and multiplies with its own dim slice of V.  K and V are
// still read once; the partial scores (S * slots floats per head) travel through the workspace.
// Kept as an A/B against the split over slots above, not used by any product entry point.
template <typename T, int D, int S>
__global__ __launch_bounds__(256) void decode_sd_scores_kernel(const T* __restrict__ q, const T* __restrict__ kc,
                                                               float* __restrict__ part, int Hq, int Hkv, int C,
                                                               int valid, float scale_log2e) {
  constexpr int E = 16 / sizeof(T), DS = D / S, LPR = DS / E, RPB = 256 / LPR;
  const int G = Hq / Hkv;
  const int s = blockIdx.y, bh = blockIdx.z, b = bh / Hkv, hk = bh % Hkv;
  const int slot = blockIdx.x * RPB + threadIdx.x / LPR;
  const int c = threadIdx.x % LPR;
  const int sl = min(slot, valid - 1);
  float kf[E];
  Frag<T, E>::load(kc + (((size_t)b * Hkv + hk) * C + sl) * D + s * DS + c * E, kf);
  for (int g = 0; g < G; ++g) {
    const int hq = hk * G + g;
    float qf[E];
    Frag<T, E>::load(q + ((size_t)b * Hq + hq) * D + s * DS + c * E, qf);
    float a = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) a = fmaf(qf[e], kf[e], a);
#pragma unroll
    for (int x = 1; x < LPR; x <<= 1) a += __shfl_xor(a, x);
    if (c == 0 && slot < valid) part[(((size_t)b * Hq + hq) * S + s) * C + slot] = a * scale_log2e;
  }
}

template <typename T, int D, int S>
__global__ __launch_bounds__(256) void decode_sd_out_kernel(const float* __restrict__ part, const T* __restrict__ vc,
                                                            T* __restrict__ out, float* __restrict__ lse, int Hq,
                                                            int Hkv, int C, int valid) {
  constexpr int E = 16 / sizeof(T), DS = D / S, LPR = DS / E, RPB = 256 / LPR;
  __shared__ float sM[RPB], sL[RPB], sO[RPB][DS];
  const int G = Hq / Hkv;
  const int s = blockIdx.x, row = blockIdx.y, b = row / Hq, hq = row % Hq, hk = hq / G;
  const int r = threadIdx.x / LPR, c = threadIdx.x % LPR;
  const float* pr = part + (size_t)row * S * C;
  const T* vb = vc + (((size_t)b * Hkv + hk) * C) * D + s * DS + c * E;
  float m = -INFINITY, l = 0.f, o[E];
#pragma unroll
  for (int e = 0; e < E; ++e) o[e] = 0.f;
  for (int slot = r; slot < valid; slot += RPB) {
    float sc = 0.f;
#pragma unroll
    for (int x = 0; x < S; ++x) sc += pr[(size_t)x * C + slot];
    float vf[E];
    Frag<T, E>::load(vb + (size_t)slot * D, vf);
    const float mn = fmaxf(m, sc);
    const float alpha = exp2f(m - mn), p = exp2f(sc - mn);
    m = mn;
    l = l * alpha + p;
#pragma unroll
    for (int e = 0; e < E; ++e) o[e] = fmaf(p, vf[e], o[e] * alpha);
  }
  if (c == 0) {
    sM[r] = m;
    sL[r] = l;
  }
#pragma unroll
  for (int e = 0; e < E; ++e) sO[r][c * E + e] = o[e];
  __syncthreads();
  for (int d = threadIdx.x; d < DS; d += 256) {
    float M = -INFINITY;
    for (int x = 0; x < RPB; ++x) M = fmaxf(M, sM[x]);
    float L = 0.f, acc = 0.f;
    for (int x = 0; x < RPB; ++x) {
      const float f = (sM[x] == -INFINITY) ? 0.f : exp2f(sM[x] - M);
      L += sL[x] * f;
      acc += sO[x][d] * f;
    }
    store_out(out + (size_t)row * D + s * DS + d, acc / L);
    if (lse != nullptr && s == 0 && d == 0) lse[row] = (M + log2f(L)) * 0.69314718055994530942f;
  }
}

template <typename T, int D>
hipError_t launch_split_headdim(const void* q, const void* kc, const void* vc, void* out, float* lse, void* ws,
                                int B, int Hq, int Hkv, int C, int valid, float scale, hipStream_t s) {
  constexpr int S = 2, E = 16 / sizeof(T), RPB = 256 / ((D / S) / E);
  const float sl2 = scale * 1.44269504088896340736f;
  decode_sd_scores_kernel<T, D, S><<<dim3((valid + RPB - 1) / RPB, S, B * Hkv), 256, 0, s>>>(
      (const T*)q, (const T*)kc, (float*)ws, Hq, Hkv, C, valid, sl2);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  decode_sd_out_kernel<T, D, S><<<dim3(S, B * Hq), 256, 0, s>>>((const float*)ws, (const T*)vc, (T*)out, lse, Hq,
                                                                Hkv, C, valid);
  return hipGetLastError();
}

struct DecPlan {
  int rows, most, splits, chunk;
  bool wide;          // a workgroup of WIDE waves for a row
  size_t part_bytes;  // workspace per part: most * rows * part_bytes serves every context up to the one given
};
// Rounds of keys up to which a workgroup of WIDE waves takes a whole row; 0: none does.
constexpr int wide_rounds(int dtype, int D) { return dtype == LG_F32 ? (D == 64 ? 3 : 0) : D == 64 ? 5 : 3; }
DecPlan dec_plan(int B, int Hq, int Hkv, int D, int valid, int dtype, bool paged) {
  const int G = Hq / Hkv;
  DecPlan p;
  p.rows = B * Hkv;
  p.part_bytes = ((size_t)G * (D + 1) + 1) * sizeof(float);  // results, log-sum-exps; LgDecWork::parts
  const int round = dtype == LG_F32 ? 64 : 128;  // keys of four units, one per wave
  const int rounds = (valid + round - 1) / round;
  // Most parts per row: five workgroups per CU; records within LG_DECODE_STATIC_SCRATCH_BYTES as long as that leaves
  // two workgroups per CU.  (Grows with the context, never falls: a workspace for the longest serves the shorter.)
  const int wgs = paged ? 2048 : 1280;
  long long most = wgs / p.rows;
  const long long fit = (long long)(LG_DECODE_STATIC_SCRATCH_BYTES / ((size_t)p.rows * p.part_bytes));
  if (most > fit) most = fit;
  const int two = (511 + p.rows) / p.rows;
  if (most < two) most = two;
  if (most > LG_DEC_SPLITS_MAX) most = LG_DEC_SPLITS_MAX;
  if (most > rounds) most = rounds;
  p.most = (int)most;
  int best_per = rounds;
  if (paged) {
    best_per = (rounds + p.most - 1) / p.most;
  } else {
    // time in us: the bytes at 6.6 GB/ms, more when the last workgroups find CUs idle or crowd them, or the rounds of
    // one workgroup at their latency; then the sum over the parts
    const float t_bytes = (float)p.rows * valid * (D * (dtype == LG_F32 ? 8 : 4)) / 6.6e6f;
    float best = 0.f;
    for (int n = 1; n <= p.most; ++n) {
      const int per = (rounds + n - 1) / n;
      if ((rounds + per - 1) / per != n) continue;
      const int wg = p.rows * n, k = (wg + 255) / 256;
      const float even = k * 256.f / wg;
      float t = t_bytes * (1.f + 0.35f * (even - 1.f) + 0.02f * (k - 1));
      if (t < 2.2f * per) t = 2.2f * per;
      if (n > 1) t += 3.5f + 0.1f * n + (k > 1 ? 2.f : 0.f);
      if (n == 1 || t < best) {
        best = t;
        best_per = per;
      }
    }
  }
  p.splits = (rounds + best_per - 1) / best_per;
  p.chunk = p.splits == 1 ? valid : round * best_per;
  // A row of few keys by one workgroup of WIDE waves, which leaves no parts to add (us per decode with its append, one after
  // the other and replayed from a graph; parts, wide; 8 kv heads): bf16 of 128, 384 keys 10.9, 8.8 and 8.9, 8.6, 500 keys 10.1,
  // 10.0 and 9.0, 9.8; of 64, 384 keys 11.2, 7.5 and 8.1, 6.6, 576 11.9, 8.1 and 8.1, 7.8, 768 10.9, 9.0 and 8.0, 8.7; float32
  // of 64, 192 keys 11.0, 8.2 and 8.4, 7.0, 384 11.0, 9.4 and 8.7, 9.1; of 128, 192 keys 10.7, 10.4 and 9.4, 10.2.
  // Up to 256 rows, each with a CU to itself (paged, without the append, 256 and 320 rows; parts, wide): bf16 of 128, 160 keys 8.7,
  // 6.9 and 10.1, 12.2, 384 12.8, 10.8 and 17.2, 18.7; of 64, 256 keys 7.8, 6.0 and 8.9, 9.7, 640 11.8, 8.8 and 14.1, 15.1; float32
  // of 64, 192 keys 11.1, 7.0 and 12.7, 11.7.  (Contiguous caches: rows are cut only where that leaves a workgroup per CU, at 320
  // rows no more.)
  p.wide = p.splits > 1 && rounds <= wide_rounds(dtype, D) && p.rows <= 256;
  if (p.wide) {
    p.splits = 1;
    p.chunk = valid;
  }
  return p;
}

template <typename T, int D>
hipError_t launch_typed(const void* q, const void* kc, const void* vc, void* out, float* lse, void* ws,
                        int B, int Hq, int Hkv, int C, const LgDecSegs& segs, float scale, hipStream_t s,
                        const LgPaged* paged) {
  constexpr int dtype = sizeof(T) == 4 ? LG_F32 : LG_BF16;
  const int valid = paged ? paged->keys_max : segs.pre[segs.n];
  const bool plain = segs.n == 1 && segs.start[0] == 0;
  LgPaged pg = {};
  if (paged) pg = *paged;
  const int G = Hq / Hkv;
  const DecPlan plan = dec_plan(B, Hq, Hkv, D, valid, dtype, paged != nullptr);
  const float sl2 = scale * 1.44269504088896340736f;
  const float qmul = sl2 < 1.f ? ldexpf(1.f, std::max(ilogbf(sl2), -126)) : 1.f, rest = sl2 / qmul;  // (exact)
  LgDecWork wk = {};
  wk.splits = plan.splits;
  wk.chunk = plan.chunk;
  if (plan.splits > 1) {
    wk.o = (float*)ws;
    wk.lse2 = wk.o + (size_t)plan.rows * plan.splits * G * D;
    wk.parts = (int*)(wk.lse2 + (size_t)plan.rows * plan.splits * G);
  }
  dim3 grid(plan.splits, plan.rows / B, B);
  if (paged) {
    pg.B = B;
    pg.few = dtype == LG_F32 ? DEC_FULL : DEC_FEW;
    // a part per 1 / DEC_FULL of all keys, and one more per row for what is left over
    const long long most = std::min<long long>((long long)plan.rows * plan.splits, (long long)DEC_FULL + plan.rows);
    grid = dim3((unsigned)most);
  }
  typedef typename LgDecElem<T>::type E;
#define LG_DECODE_LAUNCH(W, MODE, ...)                                                                               \
  decode_mfma_kernel<T, D, MODE, W><<<grid, (W) * 64, 0, s>>>((const E*)q, (const E*)kc, (const E*)vc, (T*)out, lse, wk, \
                                                              Hq, Hkv, C, valid, qmul, rest, ldexpf(1.f, ilogbf(rest)), \
                                                              LgDecExtra<MODE>{__VA_ARGS__})
  if constexpr (wide_rounds(dtype, D) > 0) {
    if (plan.wide) {
      if (paged) LG_DECODE_LAUNCH(WIDE, LG_DEC_PAGED, pg);
      else if (plain) LG_DECODE_LAUNCH(WIDE, LG_DEC_PLAIN);
      else LG_DECODE_LAUNCH(WIDE, LG_DEC_SEGS, segs);
      return hipGetLastError();
    }
  }
  if (paged) LG_DECODE_LAUNCH(WAVES, LG_DEC_PAGED, pg);
  else if (plain) LG_DECODE_LAUNCH(WAVES, LG_DEC_PLAIN);
  else LG_DECODE_LAUNCH(WAVES, LG_DEC_SEGS, segs);
#undef LG_DECODE_LAUNCH
  if (plan.splits > 1) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 heads((unsigned)(plan.rows * G));
    if (paged) decode_add_kernel<T, D, true><<<heads, 64, 0, s>>>(wk, G, (T*)out, lse);
    else decode_add_kernel<T, D, false><<<heads, 64, 0, s>>>(wk, G, (T*)out, lse);
  }
  return hipGetLastError();
}

}  // namespace

// Keys of a decode step at any context of up to m.N tokens, m from lg_make_cache_mask: at most this many.  (In block
// mode a shorter context can have a few more than the longest.)
int lg_decode_keys_max(const LgMask& m) { return (int)std::min<long long>(m.N, lg_cache_slots(m.N, m)); }

size_t lg_decode_workspace_bytes(int B, int Hq, int Hkv, int D, int valid, int dtype, bool paged) {
  const DecPlan p = dec_plan(B, Hq, Hkv, D, valid, dtype, paged);
  return p.most > 1 ? (size_t)p.rows * p.most * p.part_bytes : 0;
}

// paged: NULL for a contiguous cache [B, Hkv, C, D]; else page table, lengths and geometry of a
// paged cache [pages, Hkv, page size, D] (C unused), segs = the runs of the longest context.
hipError_t lg_launch_decode(const void* q, const void* kc, const void* vc, void* out, float* lse,
                            void* ws, int B, int Hq, int Hkv, int C, const LgDecSegs& segs, int D,
                            int dtype, float scale, hipStream_t s, const int* page_table, const int* seq_lens,
                            int pages_per_seq, int page_shift, int n_max, const LgMask* cache_mask,
                            int num_pages) {
  LgPaged pg = {};
  const LgPaged* pp = nullptr;
  if (page_table) {
    pg.page_table = page_table;
    pg.seq_lens = seq_lens;
    pg.pages_per_seq = pages_per_seq;
    pg.page_shift = page_shift;
    pg.n_max = n_max;
    pg.num_pages = num_pages;
    pg.cm = *cache_mask;
    pg.keys_max = lg_decode_keys_max(pg.cm);
    pp = &pg;
  }
  if (dtype == LG_F32) {
    return D == 64 ? launch_typed<float, 64>(q, kc, vc, out, lse, ws, B, Hq, Hkv, C, segs, scale, s, pp)
                   : launch_typed<float, 128>(q, kc, vc, out, lse, ws, B, Hq, Hkv, C, segs, scale, s, pp);
  }
  return D == 64
      ? launch_typed<__hip_bfloat16, 64>(q, kc, vc, out, lse, ws, B, Hq, Hkv, C, segs, scale, s, pp)
      : launch_typed<__hip_bfloat16, 128>(q, kc, vc, out, lse, ws, B, Hq, Hkv, C, segs, scale, s, pp);
}

// Workspace: S = 2 partial score rows of C floats per (b, hq).
size_t lg_decode_split_headdim_workspace_bytes(int B, int Hq, int C) { return (size_t)B * Hq * 2 * C * sizeof(float); }

hipError_t lg_launch_decode_split_headdim(const void* q, const void* kc, const void* vc, void* out, float* lse,
                                          void* ws, int B, int Hq, int Hkv, int C, int valid, int D, int dtype,
                                          float scale, hipStream_t s) {
  if (dtype == LG_F32) {
    return D == 64 ? launch_split_headdim<float, 64>(q, kc, vc, out, lse, ws, B, Hq, Hkv, C, valid, scale, s)
                   : launch_split_headdim<float, 128>(q, kc, vc, out, lse, ws, B, Hq, Hkv, C, valid, scale, s);
  }
  return D == 64
      ? launch_split_headdim<__hip_bfloat16, 64>(q, kc, vc, out, lse, ws, B, Hq, Hkv, C, valid, scale, s)
      : launch_split_headdim<__hip_bfloat16, 128>(q, kc, vc, out, lse, ws, B, Hq, Hkv, C, valid, scale, s);
}

hipError_t lg_launch_kv_paged_append(const void* k_new, const void* v_new, void* k_pages, void* v_pages,
                                     const int* page_table, const int* positions, int B, int Hkv,
                                     int row_bytes, int T, int pages_per_seq, int page_shift, int num_pages,
                                     const LgMask& m, hipStream_t s) {
  const int lpr = row_bytes / 16;
  const dim3 grid((T + 256 / lpr - 1) / (256 / lpr), Hkv, B);
  const uint4* kn = (const uint4*)k_new;
  const uint4* vn = (const uint4*)v_new;
  uint4* kp = (uint4*)k_pages;
  uint4* vp = (uint4*)v_pages;
#define LG_PA(L) lg_kv_paged_append_kernel<L><<<grid, 256, 0, s>>>(kn, vn, kp, vp, page_table, positions, T, \
                                                                   pages_per_seq, page_shift, num_pages, m)
  if (lpr == 8) LG_PA(8);
  else if (lpr == 16) LG_PA(16);
  else LG_PA(32);
#undef LG_PA
  return hipGetLastError();
}

hipError_t lg_launch_kv_append(const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                               int B, int Hkv, int row_bytes, int T, int pos, int slots,
                               const LgMask& m, hipStream_t s) {
  const int lpr = row_bytes / 16;  // 8, 16 or 32 lanes per token row
  int first = T, second = T;
  if (m.stride == 0) {  // the sink tokens of the call, and the last `window` of the others
    first = std::min(T, std::max(0, m.sink - pos));
    second = std::max(first, T - std::min(T, m.window));
  }
  const int kept = first + T - second;
  const dim3 grid((kept + 256 / lpr - 1) / (256 / lpr), Hkv, B);
  const uint4* kn = (const uint4*)k_new;
  const uint4* vn = (const uint4*)v_new;
  uint4* kc = (uint4*)k_cache;
  uint4* vc = (uint4*)v_cache;
  if (lpr == 8) lg_kv_append_kernel<8><<<grid, 256, 0, s>>>(kn, vn, kc, vc, T, pos, slots, m, first, second);
  else if (lpr == 16) lg_kv_append_kernel<16><<<grid, 256, 0, s>>>(kn, vn, kc, vc, T, pos, slots, m, first, second);
  else lg_kv_append_kernel<32><<<grid, 256, 0, s>>>(kn, vn, kc, vc, T, pos, slots, m, first, second);
  return hipGetLastError();
}

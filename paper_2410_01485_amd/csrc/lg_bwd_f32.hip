// lg_bwd_f32.hip — float32 backward (paper Section 3.2: masked key blocks are skipped in the backward step as
// well).
//
//   Delta_i = <dout_i, out_i>
//   P_ij = exp(scale <q_i,k_j> - lse_i),  dP_ij = <dout_i, v_j>,  dS_ij = P_ij (dP_ij - Delta_i)
//   dq_i = scale sum_j dS_ij k_j        (query-tile major, same tile walk as the forward; forms Delta too, or, where it shares a
//          launch with dk/dv because neither fills the GPU, a small kernel before both)
//   dk_j = scale sum_i dS_ij q_i,  dv_j = sum_i P_ij dout_i   (key-tile major, summed over the query heads of
//          the group)
// Precision path for float32 data: every product on the float32 matrix instruction (lg_f32.h).  dq uses 8 or 4 waves, as
// the forward: 4 or 2 groups of 16 rows x 2 halves of a tile's keys, summed through LDS at the end.  dk/dv uses 4 waves per 32 keys: 2 groups of 16 keys x 2 halves of a step's query rows (64, at head dim
// 128 32), two workgroups per CU: as 8 waves per 64 keys one workgroup fitted a CU (167 registers, 66 KB; at head dim 128
// 256 with spills), so that 280 work items were two rounds on 256 CUs, and every window had to be cut in two.  16/8 heads
// of 64, 1024 tokens, window 128: dk/dv 44 -> 29 us; 4 heads of 128, 4096 tokens, window 512: 168 -> 120.  Bound: the float32 matrix rate, 4096 cycles of a step's 6600; the rest is what one wave per
// SIMD cannot hide (masks, the next copies' issue, the barriers).
//
// The dk/dv work of a key tile is cut into parts: its window part (nsp equal runs of (head, query tile) steps,
// more than one only where key tiles x kv heads would leave CUs idle) and, for keys that every later query sees
// (sink, strided columns), its column part.  As one workgroup per key tile the sink tile of a 1024-token sequence
// with two query heads per kv head ran 32 steps where every other ran 6 and took 0.9 ms of a 1.1 ms pass.  Each
// part of a tile with several leaves float32 partial sums in the workspace; the workgroup that finishes last adds
// them in a fixed order, so the results stay bit-reproducible.
#include "../../include/longgen_attn.h"
#include "lg_f32.h"
#include "lg_kernels.h"

namespace {

constexpr float LOG2E = 1.44269504088896340736f;
using I0 = std::integral_constant<int, 0>;
using I1 = std::integral_constant<int, 1>;
using I2 = std::integral_constant<int, 2>;
static_assert(LG_F32_TK == 64, "two key halves of 32");
static_assert(LG_F32_KEYS == 32, "two groups of 16 keys");

// ------------------------------------------------------------------------- dq
// Delta of the 16 rows whose row n the lanes n, n + 16, .. hold a float4 each of every 16 dims of: the diagonal of out dO^T, in
// the order in which dP is summed: where out_i is v_j (a row with one live key) dP - Delta is then exactly zero, as it should be.
template <int D>
__device__ __forceinline__ float lg_delta_f32(const float* __restrict__ out, const float4 (&gf)[D / 16], int n, int h) {
  f32x4_t dl = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < D / 16; ++c) {
    const float4 ov = *reinterpret_cast<const float4*>(out + 16 * c + 4 * h);
    dl = lg_mfma16(ov.x, gf[c].x, dl);
    dl = lg_mfma16(ov.y, gf[c].y, dl);
    dl = lg_mfma16(ov.z, gf[c].z, dl);
    dl = lg_mfma16(ov.w, gf[c].w, dl);
  }
  // row n of column n is register n % 4 of lane (n, h = n / 4)
  return __shfl((n & 2) ? ((n & 1) ? dl[3] : dl[2]) : ((n & 1) ? dl[1] : dl[0]), 16 * (n >> 2) + n);
}

// FORM: also forms Delta for the dk/dv kernel (otherwise it is there) and clears its arrival counters.
template <int D>
constexpr int DQ_LDS = 4 * LgF32Tile<D>::BYTES;
template <int D, int TQ, bool FORM>
__device__ __forceinline__ void dq_f32_item(
    unsigned char* smem, int id, int ids, const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const float* __restrict__ out, const float* __restrict__ dout, const float* __restrict__ lse,
    float* __restrict__ delta, float* __restrict__ dq, int Hq, int Hkv, float scale, const LgMask& m, const LgItems& items,
    unsigned* __restrict__ arrived, int ncounters) {
  using T = LgF32Tile<D>;
  constexpr int RG = TQ / 16, NT = 128 * RG;  // as in the forward
  using Dma = LgTileDma<T, NT>;
  constexpr int TK = LG_F32_TK, DC = D / 16;
  constexpr int STAGE = 2 * T::BYTES, LPT = 2 * Dma::CH;

  const int tid = threadIdx.x;
  if (FORM)
    for (long long x = (long long)id * NT + tid; x < ncounters; x += (long long)ids * NT) arrived[x] = 0u;
  const int L = lg_item_of(id, items.run);
  if (L >= items.total) return;
  const LgItem it = lg_item(items, L);
  const int b = it.b, hk = it.hk, hq = it.hq, qt = (int)items.nqt.d - 1 - it.x;
  const int N = m.N;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, h = lane >> 4;
  const int rg = wave % RG, kh = wave / RG;
  const int q0 = qt * TQ, q1 = min(q0 + TQ - 1, N - 1);
  const int i = q0 + 16 * rg + n, iq = min(i, N - 1);
  const size_t qbase = (size_t)(b * Hq + hq) * m.ld * D;
  const size_t kbase = (size_t)(b * Hkv + hk) * m.ld * D;
  const float c2 = scale * LOG2E;

  float4 qf[DC], gf[DC];
#pragma unroll
  for (int c = 0; c < DC; ++c) {
    const size_t at = qbase + (size_t)iq * D + 16 * c + 4 * h;
    qf[c] = *reinterpret_cast<const float4*>(q + at);
    gf[c] = *reinterpret_cast<const float4*>(dout + at);
  }
  float* const my_delta = delta + (size_t)(b * Hq + hq) * N + iq;
  float lse2 = lse[(size_t)(b * Hq + hq) * m.ld + iq] * LOG2E, di;
  if constexpr (FORM) {
    di = lg_delta_f32<D>(out + qbase + (size_t)iq * D, gf, n, h);
    if (kh == 0 && h == 0 && i < N) *my_delta = di;
  } else {
    di = *my_delta;
  }
  asm volatile("" : "+v"(lse2), "+v"(di));  // everything loaded so far is waited for here, not in the tile loop
#pragma unroll
  for (int c = 0; c < DC; ++c) asm volatile("" ::"v"(qf[c].x), "v"(gf[c].x));

  f32x4_t acc[DC];
#pragma unroll
  for (int db = 0; db < DC; ++db) acc[db] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  Dma dma;
  dma.init(tid);
  LgF32Reader<D> rd;
  rd.init(n, h);
  const uint32_t lds0 = (uint32_t)(uintptr_t)LG_LDS_PTR(unsigned char, smem);
  auto issue = [&](int t, int stage) {
    dma.issue(k + kbase + (size_t)t * TK * D, N - t * TK, lds0 + stage * STAGE);
    dma.issue(v + kbase + (size_t)t * TK * D, N - t * TK, lds0 + stage * STAGE + T::BYTES);
  };
  const LgQSched qs = lg_qsched_init(m, q0, q1);
  LgF32Row row;
  row.init(m, i);
  int t = lg_qsched_next(m, qs, -1);
  issue(t, 0);
  int tn = lg_qsched_next(m, qs, t);
  if (tn >= 0) issue(tn, 1);
  for (int stage = 0; t >= 0; stage ^= 1) {
    if (tn >= 0) LG_WAIT_VMCNT(LPT);
    else LG_WAIT_VMCNT(0);
    __syncthreads();
    const int sk = stage * STAGE, sv = sk + T::BYTES;
    const int rb0 = 2 * kh, kk = t * TK + 32 * kh;
    // live keys of the lane's row in the wave's two 16-key blocks
    uint32_t bits = 0xffu;
    bool on0 = true, on1 = true, masked = false;
    if (!lg_qsched_full(m, qs, t)) {
      bits = row.bits(m, kk, h);
      on0 = __builtin_amdgcn_ballot_w64((bits & 0x0fu) != 0) != 0;
      on1 = __builtin_amdgcn_ballot_w64((bits & 0xf0u) != 0) != 0;
      masked = __builtin_amdgcn_ballot_w64(bits != 0xffu) != 0;
    }
    // as in the forward: units of matrix instructions, their LDS operands requested one unit ahead
    auto run = [&](auto B0_, auto NB_) {
      constexpr int B0 = decltype(B0_)::value, NB = decltype(NB_)::value;
      f32x4_t s[NB], dp[NB];
      float4 ka[2][NB], va[2][NB];
      float kc[2][DC];
      auto read_rows = [&](int c) {
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          ka[c & 1][x] = rd.row4(smem, sk, rb0 + B0 + x, c);
          va[c & 1][x] = rd.row4(smem, sv, rb0 + B0 + x, c);
        }
      };
      auto read_cols = [&](int u) {  // unit u = 4 x + r
#pragma unroll
        for (int db = 0; db < DC; ++db) kc[u & 1][db] = rd.col(smem, sk, rb0 + B0 + (u >> 2), u & 3, db);
      };
#pragma unroll
      for (int x = 0; x < NB; ++x) s[x] = dp[x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      read_rows(0);
#pragma unroll
      for (int c = 0; c < DC; ++c) {
        if (c + 1 < DC) read_rows(c + 1);
        else read_cols(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          s[x] = lg_mfma16(ka[c & 1][x].x, qf[c].x, s[x]);
          dp[x] = lg_mfma16(va[c & 1][x].x, gf[c].x, dp[x]);
        }
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          s[x] = lg_mfma16(ka[c & 1][x].y, qf[c].y, s[x]);
          dp[x] = lg_mfma16(va[c & 1][x].y, gf[c].y, dp[x]);
        }
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          s[x] = lg_mfma16(ka[c & 1][x].z, qf[c].z, s[x]);
          dp[x] = lg_mfma16(va[c & 1][x].z, gf[c].z, dp[x]);
        }
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          s[x] = lg_mfma16(ka[c & 1][x].w, qf[c].w, s[x]);
          dp[x] = lg_mfma16(va[c & 1][x].w, gf[c].w, dp[x]);
        }
      }
#pragma unroll
      for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[x][r] = __builtin_amdgcn_exp2f(fmaf(s[x][r], c2, -lse2));
      if (masked) {
        asm volatile("; masked" ::: "memory");  // (a real branch: nothing of it in whole tiles)
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            s[x][r] = lg_keep_or(s[x][r], bits, 4 * (B0 + x) + r, 0.f);
      }
#pragma unroll
      for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[x][r] *= dp[x][r] - di;
#pragma unroll
      for (int u = 0; u < 4 * NB; ++u) {
        if (u + 1 < 4 * NB) read_cols(u + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int db = 0; db < DC; ++db) acc[db] = lg_mfma16(kc[u & 1][db], s[u >> 2][u & 3], acc[db]);
      }
    };
    if (on0 && on1) run(I0{}, I2{});
    else if (on0) run(I0{}, I1{});
    else if (on1) run(I1{}, I1{});
    __syncthreads();  // everyone is done with this stage
    const int t2 = tn >= 0 ? lg_qsched_next(m, qs, tn) : -1;
    if (t2 >= 0) issue(t2, stage);
    t = tn;
    tn = t2;
  }

  float4* so = reinterpret_cast<float4*>(smem);  // add the two key halves
  if (kh == 1)
#pragma unroll
    for (int db = 0; db < DC; ++db)
      so[(rg * DC + db) * 64 + lane] = make_float4(acc[db][0], acc[db][1], acc[db][2], acc[db][3]);
  __syncthreads();
  if (kh == 0 && i < N)
#pragma unroll
    for (int db = 0; db < DC; ++db) {
      const float4 x = so[(rg * DC + db) * 64 + lane];
      *reinterpret_cast<float4*>(dq + qbase + (size_t)i * D + 16 * db + 4 * h) =
          make_float4((acc[db][0] + x.x) * scale, (acc[db][1] + x.y) * scale, (acc[db][2] + x.z) * scale,
                      (acc[db][3] + x.w) * scale);
    }
}

template <int D, int TQ>
__global__ __launch_bounds__(8 * TQ, (D == 64 ? 4 : 2) * TQ / 64) void dq_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const float* __restrict__ out, const float* __restrict__ dout, const float* __restrict__ lse,
    float* __restrict__ delta, float* __restrict__ dq, int Hq, int Hkv, float scale, LgMask m, LgItems items,
    unsigned* __restrict__ arrived, int ncounters) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DQ_LDS<D>];
  dq_f32_item<D, TQ, true>(smem, blockIdx.x, gridDim.x, q, k, v, out, dout, lse, delta, dq, Hq, Hkv, scale, m, items, arrived, ncounters);
}

// ---------------------------------------------------------------------- dk, dv
// How the dk/dv work is cut (a function of the shape and the pattern alone, so that a sequence's results do not
// depend on what else runs).
struct F32Parts {
  int nkt, nqt;  // key tiles; query tiles of a dk/dv step's size
  int nsp;    // window parts per key tile
  int ncand;  // leading key tiles that may hold column keys
  int ncc;    // column parts per such tile
  int longest;  // steps of the longest part
  LgDiv heads, Hkv, dsp, dcc;  // divisions by the kv heads of the batch, of a sequence, by nsp and ncc
  size_t counters_off, part_off, end;  // workspace: Delta | arrival counters | partial dk, dv
};

__host__ __device__ __forceinline__ int ceil_div(int a, int b) { return (int)(((unsigned)a + (unsigned)b - 1u) / (unsigned)b); }
// query rows of a step of the dk/dv kernel: two stages of Q and dO then take 66 KB, and two workgroups fit a CU
__host__ __device__ constexpr int btq_of(int D) { return D == 64 ? 64 : 32; }

F32Parts f32_parts(const LgShape& sh, const LgMask& m) {
  F32Parts p;
  const int TK = LG_F32_KEYS, TQ = btq_of(sh.D);
  p.nkt = ceil_div(sh.N, TK);
  p.nqt = ceil_div(sh.N, TQ);
  const int G = sh.Hq / sh.Hkv;
  const long long base = (long long)p.nkt * sh.Hkv * sh.B;
  int w = (m.wb * m.b + TQ - 1) / TQ + 1;  // query tiles the window of a key tile reaches
  if (w > p.nqt) w = p.nqt;
  const long long steps = (long long)w * G;
  // In steps (2 us): the longest part and the one beside it, or all of them over the CUs (two workgroups on one share its
  // matrix pipes, but one's start and end run beside the other's steps).  Starting costs two steps, partial sums and their
  // addition three more.  Beside the longest: with two per CU at once the one that is dealt out 256 later (causal, 8 heads of
  // 64, 2048 tokens, dk/dv: in one part 122 us, in two 106; 16/8 of 128 457, 373; 12 of 64, 1024 61, 53.5).
  const double total = base * G * (w - 0.5 * w * w / p.nqt);
  double least = 0;
  p.nsp = 1;
  for (int n = 1; n <= steps / 3 + 1 && n <= 64; ++n) {
    const double one = (double)((steps + n - 1) / n) + (n > 1 ? 5 : 2);
    const double all = (total + base * n * (n > 1 ? 3 : 1.5)) / 256;
    const double later = p.nqt * (1 - 256.0 / (base * n));  // query tiles from that one's first key on
    const double beside = base * n > 256 && base * n <= 512 ? (later < w ? later : w) * G / n : 0;
    const double t = one + beside > all ? one + beside : all;
    if (n == 1 || t < least) {
      least = t;
      p.nsp = n;
    }
  }
  // (the window of key tile 0 ends first: if it reaches the last row, no tile has a column part)
  const int whi0 = lg_qtile_window_hi(m, sh.N < TK ? sh.N - 1 : TK - 1, TQ);
  p.ncand = 0;
  if (whi0 < p.nqt - 1) p.ncand = m.stride > 0 ? p.nkt : ceil_div(m.sink, TK);
  if (p.ncand > p.nkt) p.ncand = p.nkt;
  // A column part is about as long as a window part, four steps at least (below that its own start and the final
  // sum weigh more).  Strided patterns have many column tiles: a few parts each fill the GPU and keep the partial
  // sums small.
  const long long csteps = (long long)(p.nqt - 1 - whi0) * G;
  long long len = (steps + p.nsp - 1) / p.nsp;
  if (len < 4) len = 4;
  if (m.stride == 0 && m.sink <= 16 && sh.D == 64) len *= 2;  // (a step with one key group takes half the time)
  long long ncc = (csteps + len - 1) / len;
  const int most = m.stride > 0 ? 8 : 64;
  p.ncc = p.ncand == 0 ? 0 : (int)(ncc < 1 ? 1 : ncc > most ? most : ncc);
  p.longest = (int)((steps + p.nsp - 1) / p.nsp);
  if (p.ncc > 0 && (csteps + p.ncc - 1) / p.ncc > p.longest) p.longest = (int)((csteps + p.ncc - 1) / p.ncc);
  const size_t rows = (((size_t)sh.B * sh.Hq * sh.N * sizeof(float)) + 255) & ~(size_t)255;
  const bool split = p.nsp > 1 || p.ncand > 0;
  const size_t heads = (size_t)sh.B * sh.Hkv;
  p.heads = lg_make_div((int)heads);
  p.Hkv = lg_make_div(sh.Hkv);
  p.dsp = lg_make_div(p.nsp);
  p.dcc = lg_make_div(p.ncc > 0 ? p.ncc : 1);
  p.counters_off = rows;
  p.part_off = p.counters_off + (split ? (heads * p.nkt * sizeof(unsigned) + 255) & ~(size_t)255 : 0);
  p.end = p.part_off + (split ? heads * ((size_t)p.nkt * p.nsp + (size_t)p.ncand * p.ncc) * 2 * TK * sh.D * sizeof(float) : 0);
  return p;
}

constexpr int BNT = 256;
template <int D>
constexpr int DKDV_LDS = 2 * (2 * LgF32Tile<D, btq_of(D)>::BYTES + 1024);
template <int D>
__device__ __forceinline__ void dkdv_f32_item(
    unsigned char* smem, int id, const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const float* __restrict__ dout, const float* __restrict__ lse, const float* __restrict__ delta,
    float* __restrict__ dk, float* __restrict__ dv, int Hq, int Hkv, float scale, const LgMask& m, const F32Parts& pt, int heads,
    unsigned* __restrict__ arrived, float* __restrict__ part) {
  constexpr int TQ = btq_of(D), TK = LG_F32_KEYS, DC = D / 16, NB2 = TQ / 32;  // NB2: 16-row blocks of a wave
  using T = LgF32Tile<D, TQ>;
  using Dma = LgTileDma<T, BNT>;
  constexpr int OFF_G = T::BYTES, OFF_L = 2 * T::BYTES, STAGE = 2 * T::BYTES + 1024, LPT = 2 * Dma::CH;
  static_assert(DKDV_LDS<D> == 2 * STAGE, "two stages");
  __shared__ unsigned s_before;

  // work item: the column parts first (they are there for few tiles and as long as any), then the window parts
  const int G = Hq / Hkv, N = m.N;
  const int ncol = heads * pt.ncand * pt.ncc;
  const bool column = id < ncol;
  // heads innermost, first key tiles (the longest, where the window is) first
  int bh, pi, hk;
  const int x = lg_divmod(pt.heads, column ? id : id - ncol, &bh);
  const LgDiv np = column ? pt.dcc : pt.dsp;
  const int kt = lg_divmod(np, x, &pi), b = lg_divmod(pt.Hkv, bh, &hk);
  const int k0 = kt * TK, k1 = min(k0 + TK - 1, N - 1);
  const int wlo = k0 / TQ, whi = lg_qtile_window_hi(m, k1, TQ);
  const bool has_col = pt.ncand > 0 && whi < pt.nqt - 1 && lg_has_column_key(m, k0, k1);
  if (column && !has_col) return;
  // steps of the whole part group: (query head, query tile), head slowest
  const int lo = column ? whi + 1 : wlo, per_head = column ? pt.nqt - 1 - whi : whi - wlo + 1;
  const int steps = per_head * G, len = lg_div(np, steps + (int)np.d - 1);
  const int s0 = pi * len, s1 = min(steps, s0 + len);
  if (s0 >= s1) return;
  const int wsteps = (whi - wlo + 1) * G, csteps = has_col ? (pt.nqt - 1 - whi) * G : 0;
  const int nmain = pt.nsp > 1 ? ceil_div(wsteps, lg_div(pt.dsp, wsteps + pt.nsp - 1)) : 1;
  const int ncols = has_col ? ceil_div(csteps, lg_div(pt.dcc, csteps + pt.ncc - 1)) : 0;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, h = lane >> 4;
  // A wave's 16 keys and its row blocks of a step: key group wave % 2 and half of the blocks, or, in a column part with
  // column keys in one group only (a sink of up to 16 tokens), that group, with one block for each wave there is one for.
  int kg = wave & 1, ngrp = 0;
  for (int x = 0; x < 2; ++x)
    if (column && k0 + 16 * x < N && lg_has_column_key(m, k0 + 16 * x, min(k0 + 16 * x + 15, N - 1))) {
      ++ngrp;
      kg = x;
    }
  const bool narrow = ngrp == 1;
  if (!narrow) kg = wave & 1;
  const int rb0 = narrow ? wave : NB2 * (wave >> 1);
  const bool idle = narrow && wave >= TQ / 16;
  const bool owner = narrow ? wave == 0 : wave < 2;  // holds the sum over the row blocks at the end
  const int j = k0 + 16 * kg + n, jk = min(j, N - 1);
  // The rows that see the lane's key are one run (as in lg_row_bits): from j on, `seen` of them.  Of the wave's keys: the
  // first and the last one, the ends of the run that ends first and of the one that ends last.  (With lg_tile_kind and
  // lg_live for every block and element, class and mask were 1000 and 1500 of a step's 8900 cycles: 3 of the 44 us above.)
  const int kw0 = k0 + 16 * kg, kw1 = kw0 + 15, kbj = lg_div_b(m, jk);
  const bool to_end = jk < m.sink || (m.stride > 0 && lg_strided(m, kbj)) || kbj + m.wb >= lg_div_b(m, N - 1) + 1;
  const int end_j = j >= N ? 0 : to_end ? N : (kbj + m.wb) * m.b;
  const unsigned seen = (unsigned)max(end_j - j, 0);
  int first_end = end_j, last_end = end_j;
#pragma unroll
  for (int x = 1; x < 16; x <<= 1) {
    first_end = min(first_end, __shfl_xor(first_end, x));
    last_end = max(last_end, __shfl_xor(last_end, x));
  }
  first_end = __builtin_amdgcn_readfirstlane(first_end);
  last_end = __builtin_amdgcn_readfirstlane(last_end);
  const size_t kbase = (size_t)(b * Hkv + hk) * m.ld * D;
  const float c2 = scale * LOG2E;

  Dma dma;
  dma.init(tid);
  LgF32Reader<D> rd;
  rd.init(n, h);
  const uint32_t lds0 = (uint32_t)(uintptr_t)LG_LDS_PTR(unsigned char, smem);
  auto issue = [&](int hq, int u, int stage) {
    const int q0 = u * TQ;
    const uint32_t st = lds0 + stage * STAGE;
    const size_t urow = (size_t)(b * Hq + hq) * m.ld;
    if (wave < 2) {  // wave 0: lse rows, wave 1: Delta rows (dense in the workspace)
      const int r = min(q0 + lane, N - 1);
      lg_dma_f32x64(wave == 0 ? lse + urow + r : delta + (size_t)(b * Hq + hq) * N + r, st + OFF_L + wave * 256);
    }
    dma.issue(q + (urow + q0) * D, N - q0, st);
    dma.issue(dout + (urow + q0) * D, N - q0, st + OFF_G);
  };
  const int hq_0 = (unsigned)s0 / (unsigned)per_head;
  int hq_c = hk * G + hq_0, u_c = lo + s0 - hq_0 * per_head;    // step being computed
  int hq_i = hq_c, u_i = u_c;                                   // step being issued
  auto advance = [&](int& hq, int& u) {
    if (++u == lo + per_head) {
      u = lo;
      ++hq;
    }
  };
  issue(hq_i, u_i, 0);
  advance(hq_i, u_i);
  if (s0 + 1 < s1) issue(hq_i, u_i, 1);
  // (K and V rows to registers, behind the first steps' copies)
  float4 kf[DC], vf[DC];
#pragma unroll
  for (int c = 0; c < DC; ++c) {
    kf[c] = *reinterpret_cast<const float4*>(k + kbase + (size_t)jk * D + 16 * c + 4 * h);
    vf[c] = *reinterpret_cast<const float4*>(v + kbase + (size_t)jk * D + 16 * c + 4 * h);
  }
#pragma unroll
  for (int c = 0; c < DC; ++c) asm volatile("" ::"v"(kf[c].x), "v"(vf[c].x));
  f32x4_t ak[DC], av[DC];
#pragma unroll
  for (int db = 0; db < DC; ++db) ak[db] = av[db] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  for (int st = s0; st < s1; ++st) {
    const int stage = (st - s0) & 1;
    if (st + 1 < s1) LG_WAIT_VMCNT(LPT);
    else LG_WAIT_VMCNT(0);
    __syncthreads();
    const int sq = stage * STAGE, sg = sq + OFF_G;
    const float* sL = reinterpret_cast<const float*>(smem + sq + OFF_L);
    const int r0 = u_c * TQ + 16 * rb0;
    // this wave's 16-row blocks (two; narrow, and at head dim 128: one) against its 16 keys
    auto some_live = [&](int r) { return r + 15 >= kw0 && r < last_end; };
    const bool on0 = !idle && some_live(r0), on1 = NB2 == 2 && !narrow && some_live(r0 + 16);
    const bool masked = r0 < kw1 || r0 + 16 * NB2 > first_end;
    auto run = [&](auto B0_, auto NB_) {
      constexpr int B0 = decltype(B0_)::value, NB = decltype(NB_)::value;
      f32x4_t s[NB], dp[NB];
      float4 qa[2][NB], ga[2][NB];
      float qc[2][DC], gc[2][DC];
      auto read_rows = [&](int c) {
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          qa[c & 1][x] = rd.row4(smem, sq, rb0 + B0 + x, c);
          ga[c & 1][x] = rd.row4(smem, sg, rb0 + B0 + x, c);
        }
      };
      auto read_cols = [&](int u) {  // unit u = 4 x + r
#pragma unroll
        for (int db = 0; db < DC; ++db) {
          gc[u & 1][db] = rd.col(smem, sg, rb0 + B0 + (u >> 2), u & 3, db);
          qc[u & 1][db] = rd.col(smem, sq, rb0 + B0 + (u >> 2), u & 3, db);
        }
      };
      float4 l4[NB], d4[NB];
#pragma unroll
      for (int x = 0; x < NB; ++x) {
        s[x] = dp[x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        l4[x] = *reinterpret_cast<const float4*>(sL + 16 * (rb0 + B0 + x) + 4 * h);
        d4[x] = *reinterpret_cast<const float4*>(sL + 64 + 16 * (rb0 + B0 + x) + 4 * h);
      }
      read_rows(0);
#pragma unroll
      for (int c = 0; c < DC; ++c) {
        if (c + 1 < DC) read_rows(c + 1);
        else read_cols(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          s[x] = lg_mfma16(qa[c & 1][x].x, kf[c].x, s[x]);
          dp[x] = lg_mfma16(ga[c & 1][x].x, vf[c].x, dp[x]);
        }
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          s[x] = lg_mfma16(qa[c & 1][x].y, kf[c].y, s[x]);
          dp[x] = lg_mfma16(ga[c & 1][x].y, vf[c].y, dp[x]);
        }
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          s[x] = lg_mfma16(qa[c & 1][x].z, kf[c].z, s[x]);
          dp[x] = lg_mfma16(ga[c & 1][x].z, vf[c].z, dp[x]);
        }
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          s[x] = lg_mfma16(qa[c & 1][x].w, kf[c].w, s[x]);
          dp[x] = lg_mfma16(ga[c & 1][x].w, vf[c].w, dp[x]);
        }
      }
#pragma unroll
      for (int x = 0; x < NB; ++x) {
        const float ls[4] = {l4[x].x, l4[x].y, l4[x].z, l4[x].w};
#pragma unroll
        for (int r = 0; r < 4; ++r) s[x][r] = __builtin_amdgcn_exp2f(fmaf(s[x][r], c2, -ls[r] * LOG2E));
      }
      if (masked) {
        asm volatile("; masked" ::: "memory");
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (!((unsigned)(r0 + 16 * (B0 + x) + 4 * h + r - j) < seen)) s[x][r] = 0.f;
      }
#pragma unroll
      for (int x = 0; x < NB; ++x) {
        const float de[4] = {d4[x].x, d4[x].y, d4[x].z, d4[x].w};
#pragma unroll
        for (int r = 0; r < 4; ++r) dp[x][r] = s[x][r] * (dp[x][r] - de[r]);
      }
#pragma unroll
      for (int u = 0; u < 4 * NB; ++u) {
        if (u + 1 < 4 * NB) read_cols(u + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int db = 0; db < DC; ++db) {
          av[db] = lg_mfma16(gc[u & 1][db], s[u >> 2][u & 3], av[db]);
          ak[db] = lg_mfma16(qc[u & 1][db], dp[u >> 2][u & 3], ak[db]);
        }
      }
    };
    if constexpr (NB2 == 2) {
      if (on0 && on1) run(I0{}, I2{});
      else if (on0) run(I0{}, I1{});
      else if (on1) run(I1{}, I1{});
    } else {
      if (on0) run(I0{}, I1{});
    }
    __syncthreads();  // everyone is done with this stage
    advance(hq_c, u_c);
    if (st + 2 < s1) {
      advance(hq_i, u_i);
      issue(hq_i, u_i, stage);
    }
  }

  // add the row blocks
  float4* so = reinterpret_cast<float4*>(smem);
  constexpr int GIVERS = TQ / 16 - 1;             // narrow: waves that are neither the owner nor idle
  static_assert((GIVERS > 2 ? GIVERS : 2) * 2 * DC * 1024 <= 2 * STAGE, "their sums fit");
  const int give = narrow ? wave - 1 : wave - 2;  // LDS slot of a wave that is not an owner
  if (!owner && !idle)
#pragma unroll
    for (int db = 0; db < DC; ++db) {
      so[(give * 2 * DC + db) * 64 + lane] = make_float4(ak[db][0], ak[db][1], ak[db][2], ak[db][3]);
      so[(give * 2 * DC + DC + db) * 64 + lane] = make_float4(av[db][0], av[db][1], av[db][2], av[db][3]);
    }
  __syncthreads();
  if (owner)
    for (int y = narrow ? 0 : wave; y < (narrow ? GIVERS : wave + 1); ++y)
#pragma unroll
      for (int db = 0; db < DC; ++db) {
        const float4 a = so[(y * 2 * DC + db) * 64 + lane], c = so[(y * 2 * DC + DC + db) * 64 + lane];
        ak[db] += f32x4_t{a.x, a.y, a.z, a.w};
        av[db] += f32x4_t{c.x, c.y, c.z, c.w};
      }
  auto put = [&](int key, int db, f32x4_t a, f32x4_t c) {
    const size_t at = kbase + (size_t)key * D + 16 * db + 4 * h;
    *reinterpret_cast<float4*>(dk + at) = make_float4(a[0] * scale, a[1] * scale, a[2] * scale, a[3] * scale);
    *reinterpret_cast<float4*>(dv + at) = make_float4(c[0], c[1], c[2], c[3]);
  };
  if (nmain + ncols == 1) {
    if (owner && j < N)
#pragma unroll
      for (int db = 0; db < DC; ++db) put(j, db, ak[db], av[db]);
    return;
  }
  // partial sums: slot of (tile, part), then [dk | dv][key group][dim block][lane] float4
  const size_t pslot = 2 * (size_t)TK * D;
  const size_t main0 = ((size_t)bh * pt.nkt + kt) * pt.nsp;
  const size_t col0 = (size_t)heads * pt.nkt * pt.nsp + ((size_t)bh * pt.ncand + kt) * pt.ncc;
  // does a column part serve keys of group g?  (no other group's slot of a column part is written or read)
  auto col_group = [&](int g) {
    const int a = k0 + 16 * g;
    return has_col && a < N && lg_has_column_key(m, a, min(a + 15, N - 1));
  };
  float* mine = part + (column ? col0 + pi : main0 + pi) * pslot;
  if (owner && (!column || col_group(kg)))
#pragma unroll
    for (int db = 0; db < DC; ++db) {
      lg_store_shared4(mine + ((kg * DC + db) * 64 + lane) * 4, ak[db]);
      lg_store_shared4(mine + (((2 + kg) * DC + db) * 64 + lane) * 4, av[db]);
    }
  lg_shared_stores_done();
  __syncthreads();
  if (tid == 0)
    s_before = __hip_atomic_fetch_add(arrived + (size_t)bh * pt.nkt + kt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (s_before != (unsigned)(nmain + ncols - 1)) return;  // another part will be the last
  // the last one adds all parts in their order: wave = (key group, half of the dims), four parts' loads in flight
  constexpr int HB = DC / 2, AHEAD = 4;
  const int g = wave & 1, db0 = (wave >> 1) * HB;
  const int nsum = nmain + (col_group(g) ? ncols : 0);
  f32x4_t sk_[HB], sv_[HB];
#pragma unroll
  for (int y = 0; y < HB; ++y) sk_[y] = sv_[y] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int p0 = 0; p0 < nsum; p0 += AHEAD) {
    f32x4_t a[AHEAD][HB], c[AHEAD][HB];
#pragma unroll
    for (int x = 0; x < AHEAD; ++x) {
      const int p = min(p0 + x, nsum - 1);
      const float* src = part + (p < nmain ? main0 + p : col0 + p - nmain) * pslot;
#pragma unroll
      for (int y = 0; y < HB; ++y) {
        a[x][y] = lg_load_shared4(src + ((g * DC + db0 + y) * 64 + lane) * 4);
        c[x][y] = lg_load_shared4(src + (((2 + g) * DC + db0 + y) * 64 + lane) * 4);
      }
    }
#pragma unroll
    for (int x = 0; x < AHEAD; ++x)
      if (p0 + x < nsum)
#pragma unroll
        for (int y = 0; y < HB; ++y) {
          sk_[y] += a[x][y];
          sv_[y] += c[x][y];
        }
  }
  if (k0 + 16 * g + n < N)
#pragma unroll
    for (int y = 0; y < HB; ++y) put(k0 + 16 * g + n, db0 + y, sk_[y], sv_[y]);
}

template <int D>
__global__ __launch_bounds__(BNT, 2) void dkdv_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const float* __restrict__ dout, const float* __restrict__ lse, const float* __restrict__ delta,
    float* __restrict__ dk, float* __restrict__ dv, int Hq, int Hkv, float scale, LgMask m, F32Parts pt, int heads,
    unsigned* __restrict__ arrived, float* __restrict__ part) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DKDV_LDS<D>];
  dkdv_f32_item<D>(smem, blockIdx.x, q, k, v, dout, lse, delta, dk, dv, Hq, Hkv, scale, m, pt, heads, arrived, part);
}

// Both in one launch (f32_both), the same bits.  Delta and the cleared arrival counters, which dk/dv needs from the start, come from
// bwd_prep_f32_kernel, a wave for every 16 rows.
template <int D>
__global__ __launch_bounds__(256) void bwd_prep_f32_kernel(const float* __restrict__ out, const float* __restrict__ dout,
                                                           float* __restrict__ delta, int N, int ld, int tiles,
                                                           unsigned* __restrict__ arrived, int ncounters) {
  for (long long x = (long long)blockIdx.x * 256 + threadIdx.x; x < ncounters; x += (long long)gridDim.x * 256) arrived[x] = 0u;
  const int lane = threadIdx.x & 63, n = lane & 15, h = lane >> 4;
  const int head = blockIdx.x / tiles, i = (blockIdx.x - head * tiles) * 64 + 16 * (threadIdx.x >> 6) + n;
  const size_t row = ((size_t)head * ld + min(i, N - 1)) * D;
  float4 gf[D / 16];
#pragma unroll
  for (int c = 0; c < D / 16; ++c) gf[c] = *reinterpret_cast<const float4*>(dout + row + 16 * c + 4 * h);
  const float di = lg_delta_f32<D>(out + row, gf, n, h);
  if (h == 0 && i < N) delta[(size_t)head * N + i] = di;
}
template <int D>
__global__ __launch_bounds__(BNT, 2) void bwd_both_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ dout,
    const float* __restrict__ lse, float* __restrict__ delta, float* __restrict__ dq, float* __restrict__ dk,
    float* __restrict__ dv, int Hq, int Hkv, float scale, LgMask m, F32Parts pt, int heads, unsigned* __restrict__ arrived,
    float* __restrict__ part, LgItems items, int nkv, int ndq, bool dq_first) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DQ_LDS<D> > DKDV_LDS<D> ? DQ_LDS<D> : DKDV_LDS<D>];
  // (ndq is a multiple of 8, so that dq's workgroups keep their XCDs)
  const int id = dq_first ? (int)blockIdx.x : (int)blockIdx.x - ((nkv + 7) & ~7);
  if (id >= 0 && id < ndq)
    dq_f32_item<D, 32, false>(smem, id, 0, q, k, v, nullptr, dout, lse, delta, dq, Hq, Hkv, scale, m, items, nullptr, 0);
  const int kv = dq_first ? (int)blockIdx.x - ndq : (int)blockIdx.x;
  if (kv >= 0 && kv < nkv) dkdv_f32_item<D>(smem, kv, q, k, v, dout, lse, delta, dk, dv, Hq, Hkv, scale, m, pt, heads, arrived, part);
}

// Up to how many workgroups dq (32 rows each) and dk/dv share a launch.  One after the other they end twice with CUs idle, and a
// sequence of a few hundred tokens has work for a fraction of them either way.  Backward in us, two launches : this, of 64: 2
// heads, 510 tokens, causal 35 : 23, 4 x 4, 1036 101 : 56, 2, 3000 165 : 121, 2 x 8/4, 1024, window 128 45 : 41, 8, 2048 210 : 152,
// 8/1, 3216, window 231 175 : 139, 4, 8000, window 300 129 : 126, 2 x 2/1, 5033, every 4th block 209 : 171; of 128: 1 head, 715
// tokens, window 217 51 : 31, 8/1, 297 59 : 39, 2, 695, causal 76 : 50, 4, 1384, window 143 42 : 42.  One workgroup of head dim
// 128 fills a CU's LDS (dk/dv alone: two): 4 x 4 heads, 502 tokens, 768 workgroups 77 : 83, 2 x 16/4, 578, 1408 94 : 100.  Which of
// the two comes first: the one whose longest item takes longer, that is 3 : 2 in dq's tiles (2 heads of 64, 3000 tokens 176 with
// dk/dv first; 8/2, 4096, window 512 169, dq first 214).
bool f32_both(const LgShape& sh, const F32Parts& pt) {
  const long long items = (long long)sh.B * sh.Hkv * ((long long)pt.nkt * pt.nsp + (long long)pt.ncand * pt.ncc);
  return (long long)ceil_div(sh.N, 32) * sh.Hq * sh.B + items <= (sh.D == 64 ? 4096 : 512);
}
template <int D>
hipError_t launch_bwd(const float* q, const float* k, const float* v, const float* out, const float* lse,
                      const float* dout, float* dq, float* dk, float* dv, void* ws, const LgShape& sh,
                      const LgMask& m, hipStream_t s, hipEvent_t* ev) {
  const F32Parts pt = f32_parts(sh, m);
  const int heads = sh.B * sh.Hkv;
  float* delta = (float*)ws;
  unsigned* arrived = (unsigned*)((char*)ws + pt.counters_off);
  float* part = (float*)((char*)ws + pt.part_off);
  const long long ncnt = pt.part_off > pt.counters_off ? (long long)heads * pt.nkt : 0;
  const int TQ = lg_f32_rows(sh, m), nqt = ceil_div(sh.N, TQ);
  const long long tl = (long long)nqt * sh.Hq * sh.B;
  const long long items = (long long)heads * ((long long)pt.nkt * pt.nsp + (long long)pt.ncand * pt.ncc);
  if (tl > 0x7fffffffLL - 8 || items > 0x7fffffffLL || ncnt > 0x7fffffffLL) return hipErrorInvalidValue;
  if (ev) (void)hipEventRecord(ev[0], s);
  const int nqt32 = ceil_div(sh.N, 32);
  const size_t kv_bytes = (size_t)heads * m.ld * D * sizeof(float);
  bool both = f32_both(sh, pt);
  for (const float* d : {dk, dv}) both = both && !lg_overlap(d, kv_bytes, k, kv_bytes) && !lg_overlap(d, kv_bytes, v, kv_bytes);
  if (both) {
    const int tiles = ceil_div(sh.N, 64);
    bwd_prep_f32_kernel<D><<<dim3((unsigned)(tiles * sh.Hq * sh.B)), 256, 0, s>>>(out, dout, delta, sh.N, m.ld, tiles, arrived, (int)ncnt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (ev) {
      (void)hipEventRecord(ev[1], s);
      (void)hipEventRecord(ev[2], s);  // (dq and dk/dv: one figure)
    }
    const int total = nqt32 * sh.Hq * sh.B, run = lg_run_length(m, total, sh.B * sh.Hkv, 8 * (sh.Hq / sh.Hkv), false);
    const int nkv = (int)items, ndq = (int)lg_run_grid(total, run);
    const long long reach = (long long)m.wb * m.b + m.sink + (m.stride > 0 ? sh.N / m.stride : 0);
    const int tiles_dq = (int)((reach < sh.N ? reach : sh.N) / 64) + 1;
    const bool dq_first = 2 * tiles_dq > 3 * pt.longest;
    bwd_both_f32_kernel<D><<<dim3((unsigned)(((nkv + 7) & ~7) + ndq)), BNT, 0, s>>>(
        q, k, v, dout, lse, delta, dq, dk, dv, sh.Hq, sh.Hkv, sh.scale, m, pt, heads, arrived, part,
        lg_make_items(total, run, nqt32, sh.Hq, sh.Hkv, sh.D), nkv, ndq, dq_first);
    e = hipGetLastError();
    if (ev) (void)hipEventRecord(ev[3], s);
    return e;
  }
  if (ev) (void)hipEventRecord(ev[1], s);  // (nothing to set up)
  const int total = (int)tl, run = lg_run_length(m, total, sh.B * sh.Hkv, 256 / TQ * (sh.Hq / sh.Hkv), false);
  const auto kernel = TQ == 64 ? dq_f32_kernel<D, 64> : dq_f32_kernel<D, 32>;
  kernel<<<dim3((unsigned)lg_run_grid(total, run)), 8 * TQ, 0, s>>>(q, k, v, out, dout, lse, delta, dq, sh.Hq, sh.Hkv, sh.scale, m,
                                                    lg_make_items(total, run, nqt, sh.Hq, sh.Hkv, sh.D), arrived, (int)ncnt);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (ev) (void)hipEventRecord(ev[2], s);
  dkdv_f32_kernel<D><<<dim3((unsigned)items), BNT, 0, s>>>(q, k, v, dout, lse, delta, dk, dv, sh.Hq, sh.Hkv, sh.scale,
                                                          m, pt, heads, arrived, part);
  e = hipGetLastError();
  if (ev) (void)hipEventRecord(ev[3], s);
  return e;
}

}  // namespace

size_t lg_bwd_workspace_bytes(const LgShape& sh, const LgMask& m, int dtype) {
  if (dtype == LG_F32) return f32_parts(sh, m).end;
  return lg_bwd_bf16_workspace_bytes(sh, m);
}

bool lg_bwd_f32_shares(const LgShape& sh, const LgMask& m) { return f32_both(sh, f32_parts(sh, m)); }

hipError_t lg_launch_bwd_f32(const float* q, const float* k, const float* v, const float* out,
                             const float* lse, const float* dout, float* dq, float* dk, float* dv,
                             void* ws, const LgShape& sh, const LgMask& m, hipStream_t s,
                             hipEvent_t* ev) {
  return sh.D == 64 ? launch_bwd<64>(q, k, v, out, lse, dout, dq, dk, dv, ws, sh, m, s, ev)
                    : launch_bwd<128>(q, k, v, out, lse, dout, dq, dk, dv, ws, sh, m, s, ev);
}

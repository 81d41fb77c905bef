// lg_fwd_f32.hip — float32 prefill forward (paper Section 3.2: fused online-softmax
// attention that only visits key tiles the mask leaves live).
//
// Precision path: float32 inputs, products, sums and softmax.  The products run on the float32 matrix
// instruction (lg_f32.h).  As vector multiply-adds with an LDS operand each, the forward of 16 heads x 1024 tokens
// (D = 64, window 128) took 86 us; this form takes 17.
//
// One workgroup = 8 waves = 4 groups of 16 query rows of one (b, hq) x 2 halves of every 64-key tile (two waves per SIMD: one's
// softmax runs under the other's matrix work), merged at the end; where that is few workgroups 4 waves = 2 groups x 2 halves
// (lg_f32_rows).  What a wave does, and with it every bit of the result, is the same in both.  Per wave and 16-key block:
//   S^T = K Q^T (keys x queries), online softmax with a lane owning one query, O^T += V^T P^T with P^T straight
//   from the accumulator registers.
// Bound: the float32 matrix rate (4096 cycles per 64 x 64 tile at D = 64); measured 98 TFLOP/s on full causal
// attention, 8 heads x 4096 tokens, D = 128.
#include "lg_f32.h"
#include "lg_kernels.h"

namespace {

constexpr int TK = LG_F32_TK;
static_assert(TK == 64, "two key halves of 32");

// TQ: query rows of a workgroup, 64 or 32.  Two workgroups per CU where LDS allows it (D = 64: 64 KB each)
template <int D, int TQ>
__global__ __launch_bounds__(8 * TQ, (D == 64 ? 4 : 2) * TQ / 64) void fwd_f32_kernel(const float* __restrict__ q,
                                                                      const float* __restrict__ k,
                                                                      const float* __restrict__ v,
                                                                      float* __restrict__ out,
                                                                      float* __restrict__ lse, int Hq, int Hkv,
                                                                      float scale, LgMask m, LgItems items) {
  using T = LgF32Tile<D>;
  constexpr int RG = TQ / 16, NT = 128 * RG;  // row groups of two waves each
  using Dma = LgTileDma<T, NT>;
  constexpr int DC = D / 16;
  constexpr int STAGE = 2 * T::BYTES, LPT = 2 * Dma::CH;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * STAGE];

  const int L = lg_item_of(blockIdx.x, items.run);
  if (L >= items.total) return;
  const LgItem it = lg_item(items, L);
  const int b = it.b, hk = it.hk, hq = it.hq, qt = (int)items.nqt.d - 1 - it.x;
  const int N = m.N;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, h = lane >> 4;
  const int rg = wave % RG, kh = wave / RG;
  const int q0 = qt * TQ, q1 = min(q0 + TQ - 1, N - 1);
  const int i = q0 + 16 * rg + n, iq = min(i, N - 1);
  const size_t qbase = (size_t)(b * Hq + hq) * m.ld * D;
  const size_t kbase = (size_t)(b * Hkv + hk) * m.ld * D;
  const float c2 = scale * 1.44269504088896340736f;
  const float c2_pow2 = __uint_as_float(__float_as_uint(c2) & 0x7f800000u);

  float4 qf[DC];
#pragma unroll
  for (int c = 0; c < DC; ++c) qf[c] = *reinterpret_cast<const float4*>(q + qbase + (size_t)iq * D + 16 * c + 4 * h);
#pragma unroll
  for (int c = 0; c < DC; ++c) asm volatile("" ::"v"(qf[c].x));  // wait for them here, not inside the tile loop

  f32x4_t o[DC];
#pragma unroll
  for (int db = 0; db < DC; ++db) o[db] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float mref = -INFINITY, lrow = 0.f;
  float cl = c2, moff = 0.f;  // P = exp2(S cl - moff)

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
  const LgRows rows = lg_rows(m, min(q0 + 16 * rg, N - 1), min(q0 + 16 * rg + 15, N - 1));
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
    int kind0 = LG_TILE_FULL, kind1 = LG_TILE_FULL;
    if (!lg_qsched_full(m, qs, t)) {
      kind0 = lg_rows_kind(m, rows, kk, kk + 15);
      kind1 = lg_rows_kind(m, rows, kk + 16, kk + 31);
    }
    const bool on0 = kind0 != LG_TILE_DEAD, on1 = kind1 != LG_TILE_DEAD, masked = kind0 == LG_TILE_PARTIAL || kind1 == LG_TILE_PARTIAL;
    // Blocks B0 .. B0 + NB - 1 of the half tile, as a straight sequence of units whose LDS operands are requested one
    // unit ahead: DC units of the first product, then 4 NB of the second.
    auto run = [&](auto B0_, auto NB_) {
      constexpr int B0 = decltype(B0_)::value, NB = decltype(NB_)::value;
      f32x4_t s[NB];
      float4 ka[2][NB];
      float va[2][DC];
      auto read_k = [&](int c) {
#pragma unroll
        for (int x = 0; x < NB; ++x) ka[c & 1][x] = rd.row4(smem, sk, rb0 + B0 + x, c);
      };
      auto read_v = [&](int u) {  // unit u = 4 x + r
#pragma unroll
        for (int db = 0; db < DC; ++db) va[u & 1][db] = rd.col(smem, sv, rb0 + B0 + (u >> 2), u & 3, db);
      };
#pragma unroll
      for (int x = 0; x < NB; ++x) s[x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      read_k(0);
#pragma unroll
      for (int c = 0; c < DC; ++c) {
        if (c + 1 < DC) read_k(c + 1);
        else read_v(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < NB; ++x) s[x] = lg_mfma16(ka[c & 1][x].x, qf[c].x, s[x]);
#pragma unroll
        for (int x = 0; x < NB; ++x) s[x] = lg_mfma16(ka[c & 1][x].y, qf[c].y, s[x]);
#pragma unroll
        for (int x = 0; x < NB; ++x) s[x] = lg_mfma16(ka[c & 1][x].z, qf[c].z, s[x]);
#pragma unroll
        for (int x = 0; x < NB; ++x) s[x] = lg_mfma16(ka[c & 1][x].w, qf[c].w, s[x]);
      }
      if (masked) {
        asm volatile("; masked" ::: "memory");  // (a real branch: nothing of it in whole tiles)
        const uint32_t bits = row.bits(m, kk, h);
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
          for (int r = 0; r < 4; ++r) s[x][r] = lg_keep_or(s[x][r], bits, 4 * (B0 + x) + r, -INFINITY);
      }
      float mx = -INFINITY;
#pragma unroll
      for (int x = 0; x < NB; ++x) mx = fmaxf(mx, fmaxf(fmaxf(s[x][0], s[x][1]), fmaxf(s[x][2], s[x][3])));
      // the exponent's reference moves only when a maximum has outgrown it by 2^8 (lse holds for any reference)
      if (__builtin_amdgcn_ballot_w64((mx - mref) * c2 > 8.0f) != 0) {
        const float mnew = lg_col_max(fmaxf(mx, mref));
        const float alpha = mnew == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((mref - mnew) * c2);
        mref = mnew;
        // From 2^30 on the rounding of mref * c2 would show as a factor beyond the exponent's range.  Distinct scores are
        // then at least 2^5 apart, and c2's power of two, with which the product is exact, serves as well.
        cl = fabsf(mref * c2) >= 0x1p30f ? c2_pow2 : c2;
        moff = mref == -INFINITY ? 0.f : mref * cl;
        lrow *= alpha;
#pragma unroll
        for (int db = 0; db < DC; ++db) o[db] *= alpha;
      }
#pragma unroll
      for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          s[x][r] = __builtin_amdgcn_exp2f(fmaf(s[x][r], cl, -moff));
          lrow += s[x][r];
        }
#pragma unroll
      for (int u = 0; u < 4 * NB; ++u) {
        if (u + 1 < 4 * NB) read_v(u + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int db = 0; db < DC; ++db) o[db] = lg_mfma16(va[u & 1][db], s[u >> 2][u & 3], o[db]);
      }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    if (on0 && on1) run(I0{}, I2{});
    else if (on0) run(I0{}, I1{});
    else if (on1) run(I1{}, I1{});
    __syncthreads();  // everyone is done with this stage
    const int t2 = tn >= 0 ? lg_qsched_next(m, qs, tn) : -1;
    if (t2 >= 0) issue(t2, stage);
    t = tn;
    tn = t2;
  }

  // merge the two key halves of the rows
  float l = lg_col_sum(lrow);
  float4* so = reinterpret_cast<float4*>(smem);
  float2* sml = reinterpret_cast<float2*>(smem + RG * DC * 64 * 16);
  static_assert(RG * (DC * 64 * 16 + 64 * 8) <= 2 * STAGE, "a half's results fit the stages");
  if (kh == 1) {
#pragma unroll
    for (int db = 0; db < DC; ++db) so[(rg * DC + db) * 64 + lane] = make_float4(o[db][0], o[db][1], o[db][2], o[db][3]);
    sml[rg * 64 + lane] = make_float2(mref, l);
  }
  __syncthreads();
  if (kh == 0 && i < N) {
    const float2 ml = sml[rg * 64 + lane];
    const float M = fmaxf(mref, ml.x), Ms = M == -INFINITY ? 0.f : M;  // (no finite score: weights 0, lse -inf)
    const float wa = __builtin_amdgcn_exp2f((mref - Ms) * c2), wb = __builtin_amdgcn_exp2f((ml.x - Ms) * c2);
    l = l * wa + ml.y * wb;
    const float fa = wa / l, fb = wb / l;
#pragma unroll
    for (int db = 0; db < DC; ++db) {
      const float4 x = so[(rg * DC + db) * 64 + lane];
      *reinterpret_cast<float4*>(out + qbase + (size_t)i * D + 16 * db + 4 * h) =
          make_float4(o[db][0] * fa + x.x * fb, o[db][1] * fa + x.y * fb, o[db][2] * fa + x.z * fb, o[db][3] * fa + x.w * fb);
    }
    if (lse != nullptr && h == 0)
      lse[(size_t)(b * Hq + hq) * m.ld + i] = (M * c2 + log2f(l)) * 0.69314718055994530942f;
  }
}

}  // namespace

hipError_t lg_launch_fwd_f32(const float* q, const float* k, const float* v, float* out, float* lse,
                             const LgShape& sh, const LgMask& m, hipStream_t s) {
  const int TQ = lg_f32_rows(sh, m), nqt = (sh.N + TQ - 1) / TQ;
  const long long tl = (long long)nqt * sh.Hq * sh.B;
  if (tl > 0x7fffffffLL - 8) return hipErrorInvalidValue;
  const int total = (int)tl, run = lg_run_length(m, total, sh.B * sh.Hkv, 256 / TQ * (sh.Hq / sh.Hkv), false);
  const LgItems items = lg_make_items(total, run, nqt, sh.Hq, sh.Hkv, sh.D);
  const dim3 grid((unsigned)lg_run_grid(total, run));
#define LG_FWD_LAUNCH(DD, ROWS) \
  fwd_f32_kernel<DD, ROWS><<<grid, 8 * ROWS, 0, s>>>(q, k, v, out, lse, sh.Hq, sh.Hkv, sh.scale, m, items)
  if (sh.D == 64 && TQ == 64) LG_FWD_LAUNCH(64, 64);
  else if (sh.D == 64) LG_FWD_LAUNCH(64, 32);
  else if (TQ == 64) LG_FWD_LAUNCH(128, 64);
  else LG_FWD_LAUNCH(128, 32);
#undef LG_FWD_LAUNCH
  return hipGetLastError();
}

// lg_fwd_list_bf16.hip — the instances of the bf16 prefill forward (lg_fwd_bf16.h) whose waves list their key tiles.
#include "lg_fwd_bf16.h"

void lg_launch_fwd_list_bf16(const void* q, const void* k, const void* v, void* out, float* lse, const LgShape& sh, float scale_log2e,
                             const LgMask& m, const LgItems& items, const LgPackFew* pack, unsigned grid, hipStream_t s) {
#define LG_FWD_LAUNCH(DD, Pack, pack)                                                                               \
  fwd_bf16_kernel<DD, Pack, true, true><<<dim3(grid), NT, 0, s>>>((const uint16_t*)q, (const uint16_t*)k,            \
                                                                  (const uint16_t*)v, (uint16_t*)out, lse, sh.Hq,   \
                                                                  sh.Hkv, scale_log2e, m, items, pack)
  if (sh.D == 64 && pack) LG_FWD_LAUNCH(64, LgPackFew, *pack);
  else if (sh.D == 64) LG_FWD_LAUNCH(64, LgNoPack, LgNoPack{});
  else if (pack) LG_FWD_LAUNCH(128, LgPackFew, *pack);
  else LG_FWD_LAUNCH(128, LgNoPack, LgNoPack{});
#undef LG_FWD_LAUNCH
}

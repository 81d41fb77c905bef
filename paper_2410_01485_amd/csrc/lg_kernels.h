// lg_kernels.h — internal interface between the C ABI (lg_api.hip) and the kernel
// translation units.  Tile sizes live here because the host-side tile map (lg_debug_tile_map) lists tiles of these sizes: bf16
// exactly those that the kernels walk, float32 those of 64 x 64 that the kernels' smaller ones lie in.
#ifndef LG_KERNELS_H_
#define LG_KERNELS_H_

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "lg_mask.h"

// Kernel tile sizes (query rows x keys per step).  Independent of the pattern's
// `block`: they never change results, only which tiles count as PARTIAL.
enum {
  LG_F32_TQ = 64, LG_F32_TK = 64,        // float32 forward / dq (half the rows where workgroups are few: lg_f32_rows)
  LG_F32_BTQ = 64, LG_F32_BTK = 64,      // float32 dk/dv (key-tile major), as listed by the host view
  LG_F32_KEYS = 32,                      // keys of a float32 dk/dv workgroup (a step: 64 rows, at head dim 128 32)
  LG_BF16_TQ = 256, LG_BF16_TK = 64,     // bf16 dq kernel with 64 rows per wave
  LG_BF16_TQ32 = 128,                    // bf16 forward, dq kernel with 32 rows per wave (64 keys per step as well)
  LG_BF16_BTQ = 64, LG_BF16_BTK = 256,   // bf16 dk/dv kernels (key-tile major), head dim 128
  LG_BF16_BTK64 = 128                    // ... head dim 64
};

struct LgShape {
  int B, Hq, Hkv, N, D;
  float scale;  // already resolved (> 0)
};

// float32 forward and dq: query rows of a workgroup, 64 (8 waves) or 32 (4 waves, which do the same work each: every bit of a
// sequence's results is the same in both, so the choice may depend on the batch).  32 halve the time of a row's chain of tiles,
// whose matrix instructions two waves of a SIMD otherwise share, and give twice the workgroups, but load the keys twice as
// often.  They pay where 64 rows leave CUs without work: up to 128 workgroups (forward / dq, us: 1 head of 64, 2000 tokens,
// causal 84 -> 53 / 115 -> 70; 4 heads of 64, 2048 tokens, window 300 22.6 -> 16.4 / 32.7 -> 23.1; of 128 38 -> 27 / 55 -> 39; 192
// workgroups, causal, of 128 160 -> 186 / 229 -> 254), and where they would need a second round for less than half the CUs
// and rows are long enough for that to matter (34 x 500 tokens of 64 43 -> 34 / 64 -> 48, of 128 88 -> 71 / 127 -> 98; 384
// workgroups, window 1000, of 64 87 -> 82 / 128 -> 112, of 128 180 -> 170 / 261 -> 238; window 100, of 64 23 -> 26 / 35 -> 37;
// 512 workgroups, window 300, of 64 39 -> 45 / 59 -> 64).
inline int lg_f32_rows(const LgShape& sh, const LgMask& m) {
  const long long n = (long long)sh.B * sh.Hq * ((sh.N + LG_F32_TQ - 1) / LG_F32_TQ);
  const long long reach = (long long)m.wb * m.b < sh.N ? (long long)m.wb * m.b : sh.N;
  return n <= 128 || (n > 256 && n <= 384 && reach >= 256) ? LG_F32_TQ / 2 : LG_F32_TQ;
}

// Each launcher enqueues on `s` and returns hipGetLastError().
hipError_t lg_launch_fwd_f32(const float* q, const float* k, const float* v, float* out, float* lse,
                             const LgShape& sh, const LgMask& m, hipStream_t s);
hipError_t lg_launch_fwd_bf16(const void* q, const void* k, const void* v, void* out, float* lse,
                              const LgShape& sh, const LgMask& m, hipStream_t s);

// Several sequences of different lengths, packed along the token axis of every head, in ONE forward launch.  Passed to the
// kernel by value (1 KB of kernel arguments for launches of few work items, else 3 KB); what a workgroup reads of a sequence
// lies side by side.
enum { LG_PACK_MAX = 128, LG_FWD_PACK_MAX = 256, LG_FWD_PACK_FEW = 128 };  // sequences of a backward, of a forward launch
struct LgPackSeq {
  int row0;            // its first row inside each head
  int tile0_, len_;    // the launch's query tiles before its own; its rows
  LG_HD int tile0() const { return tile0_; }
  LG_HD int len() const { return len_; }
};
struct LgPackSeqFew {  // (one word for both: scalar loads are of whole words)
  int row0;
  uint32_t tile0_len;
  LG_HD int tile0() const { return (int)(tile0_len >> 16); }
  LG_HD int len() const { return (int)(tile0_len & 0xffffu); }
};
template <typename Seq, int MAX>
struct LgPackOf {
  int n, tiles;  // sequences, none of them empty; query tiles of all
  Seq seq[MAX];
};
typedef LgPackOf<LgPackSeq, LG_FWD_PACK_MAX> LgPack;
typedef LgPackOf<LgPackSeqFew, LG_FWD_PACK_FEW> LgPackFew;
// Orders the sequences and fills in their tile0 (bf16 forward tile size); returns the number of query tiles.
long long lg_fwd_bf16_pack_tiles(LgPack* pack, int Hq);
// sh: B = 1, N unused; tmpl: the pattern made for a length no sequence exceeds, ld = rows per head.
hipError_t lg_launch_fwd_bf16_pack(const void* q, const void* k, const void* v, void* out, float* lse,
                                   const LgShape& sh, const LgMask& tmpl, const LgPack& pack, hipStream_t s);

size_t lg_bwd_workspace_bytes(const LgShape& sh, const LgMask& m, int dtype);
size_t lg_bwd_bf16_workspace_bytes(const LgShape& sh, const LgMask& m);
// Are the column keys of the pattern's key tiles split off (walked by workgroups of their own)?
bool lg_bwd_bf16_splits_columns(const LgMask& m, int D);
// For the packed launch below; least: the most that any of its sequences needs by itself, with which it runs as well.
size_t lg_bwd_bf16_pack_workspace_bytes(const LgShape& sh, const LgMask& tmpl, const int* cu_seqlens, int num_seqs,
                                        size_t least);
// Do two ranges of bytes overlap?  dk and dv may be written over k and v (a key tile is read by the workgroup that writes it, and
// before that): dq and dk/dv then keep launches of their own, one after the other.
inline bool lg_overlap(const void* a, size_t na, const void* b, size_t nb) {
  return (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}
// The kernels of a shape, or of the first set of launches of a pack (cu_seqlens), as lg_debug_bwd_plan tells them.
void lg_bwd_bf16_plan(const LgShape& sh, const LgMask& m, const int* cu_seqlens, int num_seqs, size_t ws_bytes, int32_t* plan);
bool lg_bwd_f32_shares(const LgShape& sh, const LgMask& m);
// ev: NULL, or 4 events recorded before the set-up, before the dq kernel, before the dk/dv kernels and after the
// last one (measurement aid).
hipError_t lg_launch_bwd_f32(const float* q, const float* k, const float* v, const float* out,
                             const float* lse, const float* dout, float* dq, float* dk, float* dv,
                             void* ws, const LgShape& sh, const LgMask& m, hipStream_t s,
                             hipEvent_t* ev);
hipError_t lg_launch_bwd_bf16(const void* q, const void* k, const void* v, const void* out,
                              const float* lse, const void* dout, void* dq, void* dk, void* dv,
                              void* ws, const LgShape& sh, const LgMask& m, hipStream_t s,
                              hipEvent_t* ev);
// sh, tmpl: as for the packed forward.  ws_bytes: at least what the longest sequence needs; more lets more sequences
// share a set of launches.
hipError_t lg_launch_bwd_bf16_pack(const void* q, const void* k, const void* v, const void* out, const float* lse,
                                   const void* dout, void* dq, void* dk, void* dv, void* ws, size_t ws_bytes,
                                   const LgShape& sh, const LgMask& tmpl, const int* cu_seqlens, int num_seqs,
                                   hipStream_t s);

// Decode: C = sink + window cache slots per (b, hkv), `valid` of them in use.
int lg_decode_keys_max(const LgMask& m);
size_t lg_decode_workspace_bytes(int B, int Hq, int Hkv, int D, int valid, int dtype, bool paged);
hipError_t lg_launch_decode(const void* q, const void* kc, const void* vc, void* out, float* lse,
                            void* ws, int B, int Hq, int Hkv, int C, const LgDecSegs& segs, int D,
                            int dtype, float scale, hipStream_t s, const int* page_table = nullptr,
                            const int* seq_lens = nullptr, int pages_per_seq = 0, int page_shift = 0,
                            int n_max = 0, const LgMask* cache_mask = nullptr, int num_pages = 0);
size_t lg_decode_split_headdim_workspace_bytes(int B, int Hq, int C);
hipError_t lg_launch_decode_split_headdim(const void* q, const void* kc, const void* vc, void* out, float* lse,
                                          void* ws, int B, int Hq, int Hkv, int C, int valid, int D, int dtype,
                                          float scale, hipStream_t s);
hipError_t lg_launch_kv_paged_append(const void* k_new, const void* v_new, void* k_pages, void* v_pages,
                                     const int* page_table, const int* positions, int B, int Hkv,
                                     int row_bytes, int T, int pages_per_seq, int page_shift, int num_pages,
                                     const LgMask& m, hipStream_t s);
hipError_t lg_launch_kv_append(const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                               int B, int Hkv, int row_bytes, int T, int pos, int slots,
                               const LgMask& m, hipStream_t s);

#endif  // LG_KERNELS_H_

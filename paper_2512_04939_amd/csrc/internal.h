// Host-side launch functions of the kernel files; the C ABI in api.hip calls these
// after validating arguments.  All pointers are device pointers unless noted.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

#include "../../include/litevggt.h"

namespace lv {

struct Dims {
  int F, H, W, S, C, heads, P, T;
  int64_t N;
};

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Raise a kernel's dynamic LDS limit on the current device to the most that any of its launches takes (a
// constant: it is set by the first launch alone).  The attribute is per device, so
// `done` (one per kernel, zero-initialised) remembers the devices that have it; setting it
// twice is harmless, which makes concurrent first calls safe.
template <size_t BYTES>
inline int allow_dynamic_lds(const void *kernel, std::atomic<uint64_t> &done) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return LV_ERR_HIP;
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return LV_OK;
  if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)BYTES) != hipSuccess)
    return LV_ERR_HIP;
  done.fetch_or(bit, std::memory_order_release);
  return LV_OK;
}

// importance.hip
int launch_grad_map(const void *images, int img_dtype, const Dims &d, int patch, float *psi_g,
                    hipStream_t st);
// both maps
int launch_maps(const void *images, int img_dtype, const uint16_t *x, const Dims &d, int patch, int pool, float *psi_g, float *psi_v,
                hipStream_t st);
int launch_naive_score(const Dims &d, int policy, uint32_t seed, float *score, hipStream_t st);
int launch_var_map(const uint16_t *x, const Dims &d, int pool, float *psi_v, hipStream_t st);
int launch_ga_fuse(const float *psi_g, const float *psi_v, const Dims &d, float alpha, float beta,
                   float *score, hipStream_t st);

// Capacity of the library-owned variance-map scratch of litevggt_importance_static, and the
// device address of that scratch on the current device (looked up once per device).
constexpr size_t kStaticScoreFloats = LV_STATIC_SCORE_MAX;
int static_importance_scratch(float **out);

// select.hip
int launch_select(const float *score, const Dims &d, const litevggt_plan_t &pl,
                  const litevggt_index &ix, hipStream_t st);

// launch_ga_fuse and launch_select in one
int launch_fuse_select(const float *psi_g, const float *psi_v, float alpha, float beta, float *score, const Dims &d,
                       const litevggt_plan_t &pl, const litevggt_index &ix, hipStream_t st);

// match.hip
// Scratch that the call asks for or, with `least`, that it does with: calls choose between ways by the
// room there is, so that scratch of a longer sequence always serves a shorter one.
size_t match_ws_bytes(const Dims &d, const litevggt_plan_t &pl, bool least = false);
int launch_match(const uint16_t *x, const Dims &d, const litevggt_plan_t &pl,
                 const litevggt_index &ix, float *best_sim, void *ws, size_t ws_bytes, hipStream_t st);

// rows 0..n-1 of a row-major [n, C] bf16 matrix -> fragment-major (1 KB per 32 rows x 16
// channels), padded with zero rows to n_pad
int launch_pack_rows(const uint16_t *x, int64_t n, int64_t n_pad, int C, void *packed,
                     hipStream_t st);

// block.hip
size_t block_ws_bytes(int64_t M, int C, int heads, int attn_dtype, bool least = false);
size_t block_wpack_bytes(int C);
// delta = Block(z) - z for M tokens; the two events (optional) are recorded around the
// attention kernel inside the block.  wpack_keep (optional, block_wpack_bytes(C)): receives the
// weights in the linear kernel's operand order (FP8 layers: quantised, with their amaxes), or, with
// wpack_ready, already holds them from an earlier call with the same weights.
int launch_global_block(const uint16_t *z, int64_t M, int C, int heads, float scale, int attn_dtype,
                        int qk_norm, const litevggt_block_weights &bw, uint16_t *delta, void *ws,
                        size_t ws_bytes, hipStream_t st, hipEvent_t after_pack = nullptr,
                        hipEvent_t after_attn = nullptr, void *wpack_keep = nullptr,
                        bool wpack_ready = false);

// merge.hip
int launch_merge(const uint16_t *x, const Dims &d, int64_t M, const litevggt_index &ix,
                 uint16_t *z, hipStream_t st);
int launch_unmerge(const uint16_t *y, const Dims &d, const litevggt_index &ix,
                   const uint16_t *residual, uint16_t *out, hipStream_t st);
// launch_unmerge(y, x -> x) and launch_merge(x -> z) in one; y and z are different buffers
int launch_unmerge_merge(const uint16_t *y, const Dims &d, int64_t M, const litevggt_index &ix, uint16_t *x, uint16_t *z,
                         hipStream_t st);

// attn.hip
size_t attn_ws_bytes(int heads, int64_t n_tokens, int attn_dtype, int n_seq = 1, bool least = false);
// What a layer that produces q, k and v can do for the attention over them (one sequence): bf16: write K, normalised
// when qk_norm, and V straight into the order the attention reads (kp, vp; n_kt tiles of 32 keys per head); E4M3:
// raise the amaxes of (normalised) q, k and v (words 0 to 2).  It needs the two ranges of words cleared before.
struct AttnKV {
  void *kp = nullptr, *vp = nullptr;
  int n_kt = 0, qk_norm = 0;
  uint32_t *amax = nullptr;
  uint32_t *clear[2] = {nullptr, nullptr};
  int n_clear[2] = {0, 0};
};
int attn_kv_target(AttnKV &kv, int64_t n_tokens, int heads, float scale, int attn_dtype, int qk_norm, const void *q, const void *o,
                   void *ws, size_t ws_bytes);
// A linear layer's activation operand buffer for align_up(n_tokens, 256) rows of K = 64 heads channels, in that layer's
// fragment order.  inv: as E4M3 codes with the scale *inv, the largest |value| raised in *amax; NULL: as bf16.
struct AttnOperand {
  void *at;
  const uint32_t *inv = nullptr;
  uint32_t *amax = nullptr;
  bool written = false;
};
// `after_pack`, when not NULL, is recorded between the K/V re-layout and the main kernel;
// n_seq sequences of n_tokens each; res: optional residual added to the output.  operand (optional; one sequence, no
// residual): where the kernels can they write the output there instead of to o, and set `written`.  ready: an
// attn_kv_target() of the same arguments whose work has been done.
int launch_attn(const uint16_t *q, const uint16_t *k, const uint16_t *v, uint16_t *o,
                int64_t n_tokens, int heads, float scale, int attn_dtype, int qk_norm, void *ws,
                size_t ws_bytes, hipStream_t st, hipEvent_t after_pack = nullptr, int n_seq = 1,
                const uint16_t *res = nullptr, AttnOperand *operand = nullptr,
                const AttnKV *ready = nullptr);

}  // namespace lv

// Token partition (Sec. 3.4 "GA Token Partitioning"): one workgroup per frame keeps the
// frame's scores in LDS, picks one dst token per grid cell (lowest score), finds the score of
// the last GA token (the n_ga-th highest among the rest) by radix selection, and writes the
// ascending index lists with ballot prefix sums.  All per-frame counts are closed-form, so every
// frame knows its output offsets without any cross-frame communication.
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace lv {

// fp32 score -> uint32 key with the same order (-0 folded onto +0; key 0 is reserved).
__device__ __forceinline__ uint32_t order_key(float s) {
  uint32_t b = __float_as_uint(s + 0.0f);
  uint32_t k = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
  return k == 0u ? 1u : k;
}

// sum of the lanes up to this one, in registers (a shuffle is a round trip to LDS)
__device__ __forceinline__ uint32_t lanes_scan(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);   // row_bcast 15 into rows 1 and 3
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);   // row_bcast 31 into rows 2 and 3
  return x;
}

struct Tri {
  int k, d, s;
};

// What bounds this kernel is the latency of one frame: a frame is a few KB, and short sequences
// have fewer frames than the chip has CUs.  Hence 16 waves per frame; the GA threshold by four
// 8-bit histogram passes over the keys (P reads each; counting every token's rank against all
// others read P^2 keys from LDS: 221 us per call for 32 frames of 37 x 37 patches, now about 9);
// and index lists written in token order, 64 tokens per wave and step, with ballots
// giving the positions (coalesced stores, no barrier between steps).  A pass has one barrier: every digit has
// counters of its own, and every wave finds the digit for itself, by a scan in registers (three barriers, the
// first wave's scan by shuffles: 2 frames of 16 x 16 7.2 us, now 6.2, 32 of 37 x 37 9.5, now 8.9; every wave's scan
// by shuffles 8.3 and 10.2; equal digits of a step counted by ballot first, which cost 0.8 us more again).
// 8 waves where a frame gives 16 too little to do (2 frames of 16 x 16 6.4 us with 16, 6.2 with 8; of 28 x 37 7.9
// and 8.4) and where there are more frames than the chip holds of 16 waves each, two per CU (1000 frames of
// 37 x 37 22.8 and 17.2 us, before 22.6).
constexpr int kFewTokens = 512, kManyFrames = 512;
constexpr int kFewSteps = 2048;   // (40 frames of 6,000 tokens 16.6 and 20.7 us)

// FUSE: the frame's scores are made here from its two maps (k_ga_fuse, the same bits) and stored: one launch
// and one read of the scores less in the layer driver (two layers of two 16 x 16 frames 69.9 -> 67.5 us).
template <bool FUSE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_select(
    const float *__restrict__ psi_g, const float *__restrict__ psi_v, float alpha, float beta,
    float *__restrict__ score, int H, int W, int S, int cell, int n_ga, int n_dst_pf,
    int n_src_pf, uint8_t *__restrict__ role_out, int32_t *__restrict__ kept_idx,
    int32_t *__restrict__ dst_idx, int32_t *__restrict__ src_idx,
    int32_t *__restrict__ anchor_of, int32_t *__restrict__ slot_of) {
  extern __shared__ uint32_t key[];           // [P] order keys; 0 marks a dst token
  __shared__ __attribute__((aligned(16))) uint32_t hist[4][256];           // one per digit
  __shared__ int eq_cnt[WAVES];
  __shared__ Tri wtot[WAVES];
  constexpr int kThreads = 64 * WAVES;
  const int P = H * W, T = P + S, f = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool all_dst = (f == 0) || (n_src_pf == 0);
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));   // the lanes before this one

  if constexpr (FUSE) {
    __shared__ float red[WAVES][4];
    const float *g = psi_g + (size_t)f * P, *v = psi_v + (size_t)f * P;
    float glo = INFINITY, ghi = -INFINITY, vlo = INFINITY, vhi = -INFINITY;
    for (int t = tid; t < P; t += kThreads) {
      const float a = g[t], b = v[t];
      glo = fminf(glo, a);
      ghi = fmaxf(ghi, a);
      vlo = fminf(vlo, b);
      vhi = fmaxf(vhi, b);
    }
    glo = wave_min(glo);
    ghi = wave_max(ghi);
    vlo = wave_min(vlo);
    vhi = wave_max(vhi);
    if (lane == 0) {
      red[wave][0] = glo;
      red[wave][1] = ghi;
      red[wave][2] = vlo;
      red[wave][3] = vhi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      glo = fminf(glo, red[w][0]);
      ghi = fmaxf(ghi, red[w][1]);
      vlo = fminf(vlo, red[w][2]);
      vhi = fmaxf(vhi, red[w][3]);
    }
    for (int t = tid; t < P; t += kThreads) {
      const float s = ga_score(g[t], v[t], glo, ghi - glo, vlo, vhi - vlo, alpha, beta);
      score[(size_t)f * P + t] = s;
      key[t] = all_dst ? 0u : order_key(s);
    }
  } else {
    for (int t = tid; t < P; t += kThreads) key[t] = all_dst ? 0u : order_key(score[(size_t)f * P + t]);
  }
  for (int i = tid; i < 4 * 256; i += kThreads) (&hist[0][0])[i] = 0u;
  __syncthreads();
  if (!all_dst) {
    // cells are disjoint: the thread that owns one is the only reader and writer of its keys
    const int ncw = (W + cell - 1) / cell, nch = (H + cell - 1) / cell;
    for (int c = tid; c < nch * ncw; c += kThreads) {
      const int ci = (c / ncw) * cell, cj = (c % ncw) * cell;
      uint32_t best = 0xffffffffu;
      int bt = -1;
      for (int i = ci; i < min(H, ci + cell); ++i)
        for (int j = cj; j < min(W, cj + cell); ++j) {
          uint32_t k = key[i * W + j];
          if (bt < 0 || k < best) {
            best = k;
            bt = i * W + j;
          }
        }
      key[bt] = 0u;
    }
    __syncthreads();
  }
  // The n_ga-th largest key of the tokens that are left (there are at least n_ga; keys of
  // tokens are never 0): digit by digit from the top, among the keys that share the digits so far.
  // Every wave finds the digit for itself: one barrier per digit.
  const bool pick = !all_dst && n_ga > 0;
  uint32_t prefix = 0u, need = (uint32_t)n_ga;   // digits fixed so far, rank left inside them
  if (pick) {
#pragma unroll
    for (int shift = 24; shift >= 0; shift -= 8) {
      uint32_t *const bins = hist[shift >> 3];
      const uint32_t mask = shift == 24 ? 0u : ~0u << (shift + 8);
      for (int t = tid; t < P; t += kThreads) {
        const uint32_t k = key[t];
        if (k != 0u && (k & mask) == prefix) atomicAdd(&bins[(k >> shift) & 255u], 1u);
      }
      __syncthreads();
      const u32x4 h4 = *(const u32x4 *)(bins + 252 - 4 * lane);   // lane l: bins 255 - 4l down to 252 - 4l
      const uint32_t h[4] = {h4.w, h4.z, h4.y, h4.x}, sum = (h[0] + h[1]) + (h[2] + h[3]);
      const uint32_t inc = lanes_scan(sum);
      uint32_t above = inc - sum, to = prefix, rank = need;   // above: keys in higher bins
      const uint64_t here = __builtin_amdgcn_ballot_w64(above < need && need <= inc);   // exactly one lane
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (above < need && need <= above + h[i]) {
          to = prefix | ((uint32_t)(255 - 4 * lane - i) << shift);
          rank = need - above;
        }
        above += h[i];
      }
      if (here != 0) {
        const int at = __builtin_ctzll(here);
        prefix = (uint32_t)__builtin_amdgcn_readlane((int)to, at);
        need = (uint32_t)__builtin_amdgcn_readlane((int)rank, at);
      }
    }
  }
  const uint32_t last = pick ? prefix : 0xffffffffu;   // key of the last GA token; of those equal to it ...
  const int n_eq = pick ? (int)need : 0;               // ... the n_eq lowest token numbers are GA tokens

  // Each wave owns a run of whole 64-token steps of the frame's T tokens.
  const int steps = (T + 63) / 64, per = (steps + WAVES - 1) / WAVES;
  const int t0 = wave * per * 64, t1 = min(t0 + per * 64, T);
  int eq = 0;
  for (int tb = t0; tb < t1; tb += 64) {
    const int t = tb + lane - S;
    eq += __popcll(__builtin_amdgcn_ballot_w64(tb + lane < t1 && t >= 0 && key[t] == last));
  }
  if (lane == 0) eq_cnt[wave] = eq;
  __syncthreads();
  int eq_before = 0;
  for (int w = 0; w < wave; ++w) eq_before += eq_cnt[w];
  // role of this lane's token of the step that starts at tb (seen: equal keys before the step)
  auto role_at = [&](int tb, int &seen) {
    const int t = tb + lane - S;
    const bool on = tb + lane < t1;
    const uint32_t k = on && t >= 0 ? key[t] : 0u;
    const uint64_t eqm = __builtin_amdgcn_ballot_w64(on && t >= 0 && k == last);
    int r = LV_ROLE_PROTECTED;
    if (t >= 0) {
      const bool ga = k > last || (k == last && seen + (int)__popcll(eqm & below) < n_eq);
      r = k == 0u ? LV_ROLE_DST : ga ? LV_ROLE_PROTECTED : LV_ROLE_SRC;
    }
    seen += __popcll(eqm);
    return on ? r : -1;
  };
  Tri mine = {0, 0, 0};
  int seen = eq_before;
  for (int tb = t0; tb < t1; tb += 64) {
    const int r = role_at(tb, seen);
    const int d = __popcll(__builtin_amdgcn_ballot_w64(r == LV_ROLE_DST));
    const int sn = __popcll(__builtin_amdgcn_ballot_w64(r == LV_ROLE_SRC));
    mine.d += d;
    mine.s += sn;
    mine.k += min(64, t1 - tb) - sn;
  }
  if (lane == 0) wtot[wave] = mine;
  __syncthreads();
  Tri pos = {0, 0, 0};
  for (int w = 0; w < wave; ++w) {
    pos.k += wtot[w].k;
    pos.d += wtot[w].d;
    pos.s += wtot[w].s;
  }
  const int K = n_dst_pf + n_ga;
  const int64_t kb = f == 0 ? 0 : (int64_t)T + (int64_t)(f - 1) * (S + K);
  const int64_t db = f == 0 ? 0 : (int64_t)P + (int64_t)(f - 1) * n_dst_pf;
  const int64_t sb = f == 0 ? 0 : (int64_t)(f - 1) * n_src_pf;
  seen = eq_before;
  for (int tb = t0; tb < t1; tb += 64) {
    const int r = role_at(tb, seen);
    const uint64_t dm = __builtin_amdgcn_ballot_w64(r == LV_ROLE_DST), sm = __builtin_amdgcn_ballot_w64(r == LV_ROLE_SRC);
    const uint64_t km = __builtin_amdgcn_ballot_w64(r >= 0) & ~sm;
    const int64_t g = (int64_t)f * T + tb + lane;
    if (r >= 0) {
      role_out[g] = (uint8_t)r;
      if (r == LV_ROLE_SRC) {
        src_idx[sb + pos.s + __popcll(sm & below)] = (int32_t)g;
      } else {
        const int64_t slot = kb + pos.k + __popcll(km & below);
        kept_idx[slot] = (int32_t)g;
        slot_of[g] = (int32_t)slot;
        anchor_of[g] = (int32_t)g;
        if (r == LV_ROLE_DST) dst_idx[db + pos.d + __popcll(dm & below)] = (int32_t)g;
      }
    }
    pos.k += __popcll(km);
    pos.d += __popcll(dm);
    pos.s += __popcll(sm);
  }
}

template <bool FUSE>
static int select_frames(const float *psi_g, const float *psi_v, float alpha, float beta, float *score, const Dims &d,
                         const litevggt_plan_t &pl, const litevggt_index &ix, hipStream_t st) {
  // the limit on P of the earlier layout (9 bytes of LDS per patch within 60 KB) is kept
  if (align_up((size_t)d.P * 9, 16) > 60 * 1024) return LV_ERR_SHAPE;
  const size_t lds = align_up((size_t)d.P * sizeof(uint32_t), 16);
  auto launch = [&](auto waves) {
    constexpr int WAVES = decltype(waves)::value;
    hipLaunchKernelGGL((k_select<FUSE, WAVES>), dim3((unsigned)d.F), dim3(64 * WAVES), lds, st, psi_g, psi_v, alpha, beta, score,
                       d.H, d.W, d.S, pl.cell, pl.n_ga_per_frame, pl.n_dst_per_frame, pl.n_src_per_frame, ix.role, ix.kept_idx,
                       ix.dst_idx, ix.src_idx, ix.anchor_of, ix.slot_of);
  };
  if (d.P <= kFewTokens || (d.F > kManyFrames && d.P <= kFewSteps)) launch(std::integral_constant<int, 8>{});
  else launch(std::integral_constant<int, 16>{});
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

int launch_select(const float *score, const Dims &d, const litevggt_plan_t &pl, const litevggt_index &ix, hipStream_t st) {
  return select_frames<false>(nullptr, nullptr, 0.f, 0.f, const_cast<float *>(score), d, pl, ix, st);   // only read
}

int launch_fuse_select(const float *psi_g, const float *psi_v, float alpha, float beta, float *score, const Dims &d,
                       const litevggt_plan_t &pl, const litevggt_index &ix, hipStream_t st) {
  return select_frames<true>(psi_g, psi_v, alpha, beta, score, d, pl, ix, st);
}

}  // namespace lv

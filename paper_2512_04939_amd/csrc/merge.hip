// Merge (Sec. 3.4 merge equation) and unmerge (Sec. 3.4 "Token Unmerging").
// Both are pure HBM streaming: every token row (dim bf16 values, 2 KB at dim 1024) is
// read or written exactly once with 16-byte accesses per lane, whole rows per wave (large groups
// in the pass that does both: slices of rows, 4 or 8 bytes per lane).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace lv {

__device__ __forceinline__ void acc_row(float (&a)[2], const uint32_t w) {
  a[0] += bf16_lo(w);
  a[1] += bf16_hi(w);
}

__device__ __forceinline__ void acc_row(float (&a)[4], const u32x2 w) {
  a[0] += bf16_lo(w.x);
  a[1] += bf16_hi(w.x);
  a[2] += bf16_lo(w.y);
  a[3] += bf16_hi(w.y);
}

__device__ __forceinline__ void acc_row(float (&a)[8], const u32x4 w) {
  a[0] += bf16_lo(w.x);
  a[1] += bf16_hi(w.x);
  a[2] += bf16_lo(w.y);
  a[3] += bf16_hi(w.y);
  a[4] += bf16_lo(w.z);
  a[5] += bf16_hi(w.z);
  a[6] += bf16_lo(w.w);
  a[7] += bf16_hi(w.w);
}

// ADD (k_merge): the token rows are written as well
template <bool ADD> struct MergeX { typedef const uint16_t *__restrict__ type; };
template <> struct MergeX<true> { typedef uint16_t *__restrict__ type; };

#ifndef LV_MERGE_COOP
#define LV_MERGE_COOP 64
#endif
constexpr int kCoopSize = LV_MERGE_COOP;   // groups larger than this are summed by all 4 waves of a workgroup

// two pieces of rows added, one rounding
__device__ __forceinline__ uint32_t add_row(const uint32_t v, const uint32_t w) {
  return pack_bf16(bf16_lo(v) + bf16_lo(w), bf16_hi(v) + bf16_hi(w));
}
__device__ __forceinline__ u32x2 add_row(const u32x2 v, const u32x2 w) {
  return u32x2{pack_bf16(bf16_lo(v.x) + bf16_lo(w.x), bf16_hi(v.x) + bf16_hi(w.x)),
               pack_bf16(bf16_lo(v.y) + bf16_lo(w.y), bf16_hi(v.y) + bf16_hi(w.y))};
}
__device__ __forceinline__ u32x4 add_row(const u32x4 v, const u32x4 w) {
  return u32x4{pack_bf16(bf16_lo(v.x) + bf16_lo(w.x), bf16_hi(v.x) + bf16_hi(w.x)),
               pack_bf16(bf16_lo(v.y) + bf16_lo(w.y), bf16_hi(v.y) + bf16_hi(w.y)),
               pack_bf16(bf16_lo(v.z) + bf16_lo(w.z), bf16_hi(v.z) + bf16_hi(w.z)),
               pack_bf16(bf16_lo(v.w) + bf16_lo(w.w), bf16_hi(v.w) + bf16_hi(w.w))};
}

// acc += rows group_mem[lo..hi) of x, this lane's chunks; R member rows in flight per lane.
// Rows are taken in batches of R; the last batch is masked (lo, hi are wave-uniform), so its
// loads are issued together as well.  The member indices of a batch are fetched while the rows
// of the batch before it are in flight, so a batch costs one memory round trip, not two.
template <int CPL, int R>
__device__ __forceinline__ void sum_rows(const uint16_t *__restrict__ x,
                                         const int32_t *__restrict__ group_mem, int lo, int hi,
                                         int C, int nch, int lane, float (&a)[CPL][8]) {
  int r[R];
#pragma unroll
  for (int u = 0; u < R; ++u) r[u] = lo + u < hi ? group_mem[lo + u] : -1;
  for (int j = lo; j < hi; j += R) {
    u32x4 w[R][CPL];
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int ch = lane + 64 * c;
        w[u][c] = (r[u] >= 0 && ch < nch) ? ((const u32x4 *)(x + (size_t)r[u] * C))[ch] : u32x4{0u, 0u, 0u, 0u};
      }
#pragma unroll
    for (int u = 0; u < R; ++u) r[u] = j + R + u < hi ? group_mem[j + R + u] : -1;
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
      for (int c = 0; c < CPL; ++c) acc_row(a[c], w[u][c]);
  }
}

// The same with row i becoming x[i] + y first (rounded to bf16 and stored; y: the slot's row).  V: the piece of a
// row that a lane holds, 64 CPL pieces in all from x on.  The
// loads of a batch are issued ahead of the stores of the batch before it: loads and stores of a wave are
// waited for in the order of their issue, so behind them they would wait for the stores as well.
// The two batches' registers decide how many waves a SIMD holds (four with 4 KB in flight each).  A wave has 512 channels of
// eight rows there rather than whole rows of 1024, four of them: twice the waves, half as long each, where a wave's time
// is that of its slot's batches one after the other (32 frames of 37 x 37 have 5,776 slots of 1 to 95 members).  C = 1024, whole rows
// and halves, us: 8 frames 22.4 and 16.5, 32 46.4 and 39.1, 100 132 and 124, 200 254 and 244, 24 of 28 x 37 at ratio 0.5 32.4
// and 27.9; C = 768, 48 of 37 x 37 at 0.75 55.4 and 48.9.  (256 channels of 8, 12 or 16 rows: 38 to 39 for the 32 frames, 36 to 52
// at ratio 0.5; four rows of 512 channels 40.6.)  Up to 512 channels four rows: 16 frames of 16 x 16, C = 256, 5.3, with eight 6.1.
constexpr int kAddRows = 8, kAddRowsFew = 4, kAddRowsCoop = 16;
template <typename V, int CPL, int R>
__device__ __forceinline__ void add_sum_rows(uint16_t *x, const V (&y)[CPL], const int32_t *__restrict__ group_mem,
                                             int lo, int hi, int C, int nch, int lane, float (&a)[CPL][sizeof(V) / 2]) {
  int r[2][R];
  V w[2][R][CPL];
  auto index = [&](int j, int (&q)[R]) {
#pragma unroll
    for (int u = 0; u < R; ++u) q[u] = j + u < hi ? group_mem[j + u] : -1;
  };
  auto load = [&](const int (&q)[R], V(&v)[R][CPL]) {
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int ch = lane + 64 * c;
        v[u][c] = (q[u] >= 0 && ch < nch) ? ((const V *)(x + (size_t)q[u] * C))[ch] : V{};
      }
  };
  auto step = [&](int j, int (&q)[R], V(&v)[R][CPL], int (&qn)[R], V(&vn)[R][CPL]) {
    load(qn, vn);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int ch = lane + 64 * c;
        if (q[u] >= 0 && ch < nch) {
          v[u][c] = add_row(y[c], v[u][c]);
          ((V *)(x + (size_t)q[u] * C))[ch] = v[u][c];
        }
        acc_row(a[c], v[u][c]);
      }
    index(j + 2 * R, q);
  };
  index(lo, r[0]);
  load(r[0], w[0]);
  index(lo + R, r[1]);
  for (int j = lo; j < hi; j += 2 * R) {
    step(j, r[0], w[0], r[1], w[1]);
    if (j + R < hi) step(j + R, r[1], w[1], r[0], w[0]);
  }
}

template <int CPL, int VALS>
__device__ __forceinline__ void store_mean(uint16_t *__restrict__ z, int m, int C, int nch, int lane,
                                           const float (&a)[CPL][VALS], float inv) {
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int ch = lane + 64 * c;
    if (ch < nch) {
      uint32_t o[VALS / 2];
#pragma unroll
      for (int i = 0; i < VALS / 2; ++i) o[i] = pack_bf16(a[c][2 * i] * inv, a[c][2 * i + 1] * inv);
      uint32_t *row = (uint32_t *)(z + (size_t)m * C);
      if constexpr (VALS == 8) ((u32x4 *)row)[ch] = u32x4{o[0], o[1], o[2], o[3]};
      else if constexpr (VALS == 4) ((u32x2 *)row)[ch] = u32x2{o[0], o[1]};
      else row[ch] = o[0];
    }
  }
}

// Slots with at most kCoopSize members are summed by one wave each, in ascending member
// order (a workgroup takes 4 consecutive slots).  Larger groups (a heavy tail: a few percent of
// the slots hold most of the tokens once the features have been through some layers) are
// summed by all 4 waves of a workgroup, each taking a contiguous quarter of the members, and
// the four partial sums are added in wave order -- the order of additions depends only on the
// group size, so results are reproducible.  The large groups are the long jobs, so they are
// started first: workgroups 0 .. nb0-1 scan kScan slots each (nb0 apart) and sum the large
// groups among them, workgroups nb0 .. take the small ones behind them.
//
// ADD: the unmerge of one layer and the merge of the next in one pass over the tokens, where both use
// the same groups: row i of slot m becomes x[i] + y[m] (the sum that k_unmerge stores, bit for bit) and
// enters the mean of its slot as it is stored.  Bound by HBM like its two halves, which read x twice and
// gather y per token; C = 1024, 37 x 37 patches, both halves -> together: 32 frames at ratio 0.9
// 56 -> 39 us (5.2 TB/s), 200 frames 358 -> 244 (5.2 TB/s); two frames of 16 x 16, C = 256 7.2 -> 3.9.
// Its large groups are bound by the rows that a workgroup has in flight, a quarter of merge's where a wave holds two
// batches of four whole rows.  So a workgroup takes a slice of the channels (128 up to 512 channels, else 256) of
// 16 rows per batch and wave, in the same registers, and there are at least 512 of them, or as many as make sets of 8 slots
// each.  Both halves, together with whole rows by M / 64 workgroups, like this (us): still scenes, 100 frames of 28 x 37 at ratio
// 0.98 (groups of 100), C = 256 82, 135, 33, C = 1024 190, 244, 81; 500 of 16 x 16 (up to 645), C = 256, ratio 0.98
// 63, 104, 35; moving, 300 frames of 37 x 37 over 20 layers (at last 1,718 groups with 60 % of the tokens, up to 749)
// 546, 415, 370.  One group with nearly all tokens is one workgroup's in every way and stays slower than
// the two halves: 38,193 of C = 1024 1,338, 3,755, 1,535, 8,625 of C = 256 181, 530, 315.
constexpr int kScan = 64;

template <int CPL, bool ADD>
__global__ __launch_bounds__(256) void k_merge(typename MergeX<ADD>::type x, const uint16_t *__restrict__ y,
                                               const int32_t *__restrict__ group_off,
                                               const int32_t *__restrict__ group_mem, int M,
                                               int C, int nb0, uint16_t *__restrict__ z) {
  // cooperative pass: a lane's piece of a row, how many of them, values in one, and channels of a workgroup
  using V = std::conditional_t<ADD, std::conditional_t<CPL == 1, uint32_t, u32x2>, u32x4>;
  constexpr int kPieces = ADD ? 1 : CPL, kVals = sizeof(V) / 2, kSlice = 64 * kVals * kPieces;
  __shared__ float part[3][kPieces * 64 * kVals];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nch = C >> 3;
  const int slices = (C + kSlice - 1) / kSlice;
  if ((int)blockIdx.x < nb0 * slices) {  // cooperative pass over the large groups of kScan slots
    const int set = (int)blockIdx.x / slices, ch0 = ((int)blockIdx.x - set * slices) * kSlice;   // first channel
    const int pieces = (C - ch0) / kVals;
    // strided: neighbouring slots (the all-dst first frame) hold the largest groups
    const int64_t ms = (int64_t)set + (int64_t)lane * nb0;
    const int bl = ms < M ? group_off[ms] : 0, el = ms < M ? group_off[ms + 1] : 0;
    uint64_t big = __builtin_amdgcn_ballot_w64(el - bl > kCoopSize);   // same in every wave
    while (big) {
      const int s = __builtin_ctzll(big);
      big &= big - 1;
      const int m = (int)(set + (int64_t)s * nb0);   // < M: its lane passed the range check
      const int b = __builtin_amdgcn_readlane(bl, s), e = __builtin_amdgcn_readlane(el, s), n = e - b;
      const int per = (n + 3) >> 2;
      const int lo = min(b + wave * per, e), hi = min(lo + per, e);
      float a[kPieces][kVals];
#pragma unroll
      for (int c = 0; c < kPieces; ++c)
#pragma unroll
        for (int i = 0; i < kVals; ++i) a[c][i] = 0.f;
      if constexpr (ADD) {
        const V ym[1] = {lane < pieces ? ((const V *)(y + (size_t)m * C + ch0))[lane] : V{}};
        add_sum_rows<V, 1, kAddRowsCoop>(x + ch0, ym, group_mem, lo, hi, C, pieces, lane, a);
      } else {
        sum_rows<CPL, 16>(x, group_mem, lo, hi, C, pieces, lane, a);
      }
      if (wave > 0) {
#pragma unroll
        for (int c = 0; c < kPieces; ++c)
#pragma unroll
          for (int i = 0; i < kVals; ++i) part[wave - 1][(c * kVals + i) * 64 + lane] = a[c][i];
      }
      __syncthreads();
      if (wave == 0) {
#pragma unroll
        for (int w = 0; w < 3; ++w)
#pragma unroll
          for (int c = 0; c < kPieces; ++c)
#pragma unroll
            for (int i = 0; i < kVals; ++i) a[c][i] += part[w][(c * kVals + i) * 64 + lane];
        store_mean(z + ch0, m, C, pieces, lane, a, 1.0f / (float)n);
      }
      __syncthreads();
    }
    return;
  }
  const int own = ((int)blockIdx.x - nb0 * slices) * 4 + wave;   // own slot, if small; ADD: 512 channels of it
  if constexpr (ADD) {
    const int m = own / CPL, ch0 = (own - m * CPL) * 512, pieces = (C - ch0) >> 3;
    if (m < M) {
      const int b = group_off[m], e = group_off[m + 1];
      if (e - b <= kCoopSize) {
        float a[1][8] = {{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}};
        const u32x4 ym[1] = {lane < pieces ? ((const u32x4 *)(y + (size_t)m * C + ch0))[lane] : u32x4{0u, 0u, 0u, 0u}};
        add_sum_rows<u32x4, 1, CPL == 1 ? kAddRowsFew : kAddRows>(x + ch0, ym, group_mem, b, e, C, pieces, lane, a);
        store_mean(z + ch0, m, C, pieces, lane, a, 1.0f / (float)(e - b));
      }
    }
    return;
  }
  const int m = own;
  if (m < M) {
    const int b = group_off[m], e = group_off[m + 1];
    if (e - b <= kCoopSize) {
      float a[CPL][8];
#pragma unroll
      for (int c = 0; c < CPL; ++c)
#pragma unroll
        for (int i = 0; i < 8; ++i) a[c][i] = 0.f;
      sum_rows<CPL, 8>(x, group_mem, b, e, C, nch, lane, a);
      store_mean(z, m, C, nch, lane, a, 1.0f / (float)(e - b));
    }
  }
}

template <bool ADD>
static int merge_rows(typename MergeX<ADD>::type x, const uint16_t *y, const Dims &d, int64_t M, const litevggt_index &ix,
                      uint16_t *z, hipStream_t st) {
  const int cpl = (d.C / 8 + 63) / 64;
  int64_t nb0 = (M + kScan - 1) / kScan;
  const int slice = cpl == 1 ? 128 : 256, slices = ADD ? (d.C + slice - 1) / slice : 1;   // kSlice
  if (ADD) nb0 = std::max(nb0, std::min<int64_t>(512 / slices, (M + 7) / 8));
  const int parts = ADD ? cpl : 1;            // waves of a small slot
  const unsigned grid = (unsigned)(nb0 * slices + (M * parts + 3) / 4);
#define LV_MERGE(CPL)                                                                                     \
  hipLaunchKernelGGL((k_merge<CPL, ADD>), dim3(grid), dim3(256), 0, st, x, y, ix.group_off, ix.group_mem, \
                     (int)M, d.C, (int)nb0, z)
  switch (cpl) {
    case 1: LV_MERGE(1); break;
    case 2: LV_MERGE(2); break;
    case 3: LV_MERGE(3); break;
    case 4: LV_MERGE(4); break;
    default: return LV_ERR_SHAPE;
  }
#undef LV_MERGE
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

int launch_merge(const uint16_t *x, const Dims &d, int64_t M, const litevggt_index &ix, uint16_t *z, hipStream_t st) {
  return merge_rows<false>(x, nullptr, d, M, ix, z, st);
}

int launch_unmerge_merge(const uint16_t *y, const Dims &d, int64_t M, const litevggt_index &ix, uint16_t *x, uint16_t *z,
                         hipStream_t st) {
  return merge_rows<true>(x, y, d, M, ix, z, st);
}

#ifndef LV_UNMERGE_ROWS
#define LV_UNMERGE_ROWS 2
#endif
// out[i] = y[slot_of[i]] (+ residual[i]); a wave moves LV_UNMERGE_ROWS token rows per step
// (all loads of a step are issued before its stores), grid-stride over row groups.
template <bool RES>
__global__ __launch_bounds__(256) void k_unmerge(const uint16_t *__restrict__ y,
                                                 const int32_t *__restrict__ slot_of,
                                                 const uint16_t *residual, int64_t N, int C,
                                                 uint16_t *out) {
  constexpr int R = LV_UNMERGE_ROWS;
  const int lane = threadIdx.x & 63;
  const int nch = C >> 3;
  const int wpb = blockDim.x >> 6;
  for (int64_t i0 = ((int64_t)blockIdx.x * wpb + (threadIdx.x >> 6)) * R; i0 < N;
       i0 += (int64_t)gridDim.x * wpb * R) {
    int slot[R];
#pragma unroll
    for (int r = 0; r < R; ++r) slot[r] = slot_of[min(i0 + r, N - 1)];
    for (int ch = lane; ch < nch; ch += 64) {
      u32x4 w[R], res[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        w[r] = ((const u32x4 *)(y + (size_t)slot[r] * C))[ch];
        if (RES) res[r] = ((const u32x4 *)(residual + (size_t)min(i0 + r, N - 1) * C))[ch];
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (i0 + r >= N) break;
        u32x4 v = w[r];
        if (RES) v = add_row(v, res[r]);
        __builtin_nontemporal_store(v, (u32x4 *)(out + (size_t)(i0 + r) * C) + ch);
      }
    }
  }
}

int launch_unmerge(const uint16_t *y, const Dims &d, const litevggt_index &ix,
                   const uint16_t *residual, uint16_t *out, hipStream_t st) {
  const int64_t want = (d.N + 4 * LV_UNMERGE_ROWS - 1) / (4 * LV_UNMERGE_ROWS);
  const unsigned grid = (unsigned)(want < 256 * 64 ? want : 256 * 64);
  if (residual)
    hipLaunchKernelGGL(k_unmerge<true>, dim3(grid), dim3(256), 0, st, y, ix.slot_of, residual, d.N,
                       d.C, out);
  else
    hipLaunchKernelGGL(k_unmerge<false>, dim3(grid), dim3(256), 0, st, y, ix.slot_of, residual,
                       d.N, d.C, out);
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

}  // namespace lv

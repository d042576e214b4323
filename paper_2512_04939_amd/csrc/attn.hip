// Full (unmasked) self-attention over the merged sequence of all frames, per head
// (Sec. 3.1 "Bottleneck Analysis": every token attends to every token of every frame).
//
// Flash-style: scores never leave registers, softmax is computed online in fp32.
// Layout choices for CDNA4 (wave64, v_mfma_f32_32x32x16_bf16):
//   * the score tile is computed transposed, S^T = K Q^T, so that a lane owns one query
//     column: row max / row sum are in-lane reductions plus one exchange between the two
//     lane halves, and the exponentiated tile is already in the B-operand layout of the
//     second contraction O^T += V^T P^T -- probabilities go from accumulator registers
//     to MFMA operands without touching LDS;
//   * K and V are re-laid out once per call into "fragment-major" order (each MFMA A
//     operand is 1 KB contiguous), V with the key permutation that the accumulator layout
//     of S^T induces.  A K/V tile is then a straight 16 KB copy into LDS, read back
//     conflict-free with ds_read_b128;
//   * a wave owns 64 queries (two 32-wide MFMA column blocks) so every K/V fragment read
//     from LDS feeds two MFMAs; a workgroup owns 256 queries;
//   * workgroups are dealt to the 8 XCDs round-robin by hardware, so the grid is ordered
//     to give each XCD whole heads: all CUs of an XCD stream the same K/V through one L2.
#include "common.h"
#include "internal.h"

#include <type_traits>

namespace lv {

constexpr int kKT = 32;              // keys per MFMA tile
constexpr int kKV = 64;              // keys per LDS stage (2 MFMA tiles)
constexpr int kSlots = 64;           // workgroups resident on an XCD: 32 CUs, 2 each
constexpr int kSyncWords = 2 * kXcd * kSlots;   // per cut block (AttnCut): pieces that have arrived, sums are there
constexpr int kQW = 64;              // queries per wave
constexpr int kQB = 512;             // queries per workgroup (8 waves)
constexpr int kFragU4 = 64;          // one fragment = 64 lanes x 16 B

constexpr float kRaise = 8.0f;       // log2 headroom before the softmax reference is raised

// RMS-normalise a 64-value head row that is spread over 2^log2_lanes neighbouring lanes (8
// bf16 values each, or several such chunks per lane): returns this lane's chunk scaled by
// 1/sqrt(mean(x^2) + eps), rounded to bf16.
__device__ __forceinline__ u32x4 rms_scale8(const u32x4 w, int log2_lanes) {
  float ss = sumsq8(w);
  for (int o = 1; o < (1 << log2_lanes); o <<= 1) ss += __shfl_xor(ss, o, 64);
  return scale8(w, 1.0f / sqrtf(ss * (1.0f / 64.0f) + kQkEps));
}

// K -> [head][key tile][k-step s][lane] : lane (h*32+r) holds K[tile*32+r][16s+8h .. +8]
// V -> [head][key tile][u][dt][lane]    : lane (h*32+dr) holds, for e = 0..7,
//      V[tile*32 + 16u + 8(e/4) + 4h + e%4][32dt + dr]   (the key order in which a lane of
//      the S^T accumulator holds its rows, so P needs no shuffle before the second MFMA)
// With several sequences of n tokens each in one call (frame attention: one per frame) the
// second grid dimension runs over (sequence, head) pairs and so do the packed arrays.
// SYNC: also clears the words that workgroups meet at (pieces of cut blocks, the next blocks' counters); FLAGS: and the flags of the online
// kernel, n_flags (<= n_kt) per (sequence, head) pair, which took a launch of 2 us (kernels of their own:
// behind a run-time test it cost every call 2 %, 42.8 -> 43.7 us for 32 frames of 1374 tokens).
// V false: K only (k_attn_bf16_stream takes V's rows as they lie).
template <bool SYNC, bool FLAGS, bool V>
__global__ __launch_bounds__(256) void k_attn_pack(const uint16_t *__restrict__ k,
                                                   const uint16_t *__restrict__ v, int64_t n,
                                                   int heads, int n_kt, int qk_norm,
                                                   u32x4 *__restrict__ kp,
                                                   u32x4 *__restrict__ vp, uint32_t *sync, int n_sync,
                                                   uint32_t *flags, int n_flags) {
  __shared__ __attribute__((aligned(16))) uint16_t vt[kKT][72];
  const int kt = blockIdx.x, t = threadIdx.x;
  if constexpr (SYNC)
    if (blockIdx.x == 0 && blockIdx.y == 0)
      for (int i = t; i < n_sync; i += 256) sync[i] = 0u;
  if constexpr (FLAGS)
    if (t == 0 && kt < n_flags) flags[(size_t)blockIdx.y * n_flags + kt] = 0u;
  const int seq = blockIdx.y / heads, head = blockIdx.y - seq * heads;
  const int C = heads * 64;
  k += (size_t)seq * n * C;
  v += (size_t)seq * n * C;
  const int key = t >> 3, chunk = t & 7;
  const int64_t row = (int64_t)kt * kKT + key;
  u32x4 wk = {0u, 0u, 0u, 0u}, wv = {0u, 0u, 0u, 0u};
  if (row < n) {
    wk = *(const u32x4 *)(k + (size_t)row * C + head * 64 + chunk * 8);
    if constexpr (V) wv = *(const u32x4 *)(v + (size_t)row * C + head * 64 + chunk * 8);
  }
  if (qk_norm) wk = rms_scale8(wk, 3);   // the 8 lanes that share a key hold its 64 values
  const size_t tile = ((size_t)blockIdx.y * n_kt + kt) * 4 * kFragU4;
  kp[tile + (chunk >> 1) * kFragU4 + (chunk & 1) * 32 + key] = wk;
  if constexpr (!V) return;
  *(u32x4 *)&vt[key][chunk * 8] = wv;
  __syncthreads();
  const int u = t >> 7, dt = (t >> 6) & 1, lane = t & 63, h = lane >> 5, dr = lane & 31;
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const int k0 = 16 * u + 8 * (e >> 2) + 4 * h + (e & 3);
    w[e >> 1] = (uint32_t)vt[k0][32 * dt + dr] | ((uint32_t)vt[k0 + 1][32 * dt + dr] << 16);
  }
  vp[tile + (u * 2 + dt) * kFragU4 + lane] = u32x4{w[0], w[1], w[2], w[3]};
}

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

constexpr int kKSlots = 2;           // LDS ring slots of 64-key K tiles
constexpr int kVSlots = 3;           // LDS ring slots of 64-key V tiles

// One workgroup = 8 waves = two groups of 4 (one wave of each group per SIMD), 512 queries.
// A wave alternates between a matrix phase (O^T += V^T P^T of the previous key tile, then the
// scores K Q^T of the next one) and a vector phase (softmax of those scores: exp2, bf16 pack,
// row sums).  The two groups run exactly one phase apart, with a workgroup barrier at every
// phase boundary, so on every SIMD one wave feeds the matrix pipe while the other feeds the
// VALU -- deterministically, not by luck of the wave scheduler.
__global__ __launch_bounds__(512) void k_attn_bf16(
    const uint16_t *q, const u32x4 *__restrict__ kp, const u32x4 *__restrict__ vp, uint16_t *o,
    const uint16_t *res, int64_t n, int heads, int n_seq, int n_kt, int nqb, float c,
    int qk_norm, const uint32_t *__restrict__ redo) {
  __shared__ u32x4 ks[kKSlots][8 * kFragU4];
  __shared__ u32x4 vs[kVSlots][8 * kFragU4];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ql = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2;           // phase group
  const int C = heads * 64;
  int sh, qb;   // (sequence, head) pair and query block; each XCD gets whole pairs
  if (((heads * n_seq) & 7) == 0) {
    const int hp = (heads * n_seq) >> 3, xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    sh = xcd * hp + local / nqb;
    qb = local % nqb;
  } else {
    sh = blockIdx.x / nqb;
    qb = blockIdx.x % nqb;
  }
  // second pass behind the per-row-reference kernel: only the query blocks it left undone (one
  // flag per 256 queries; the whole workgroup takes the same branch, before any barrier)
  if (redo && redo[(size_t)sh * (2 * nqb) + 2 * qb] == 0u && redo[(size_t)sh * (2 * nqb) + 2 * qb + 1] == 0u) return;
  const int seq = sh / heads, head = sh - seq * heads;
  q += (size_t)seq * n * C;
  o += (size_t)seq * n * C;
  if (res) res += (size_t)seq * n * C;
  const int64_t q0 = (int64_t)qb * kQB + wave * kQW;

  // Q^T fragments (B operand): lane (h*32+ql) holds Q[q0+32*sub+ql][16s+8h .. +8]
  bf16x8 qf[2][4];
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const int64_t row = min(q0 + sub * 32 + ql, n - 1);
    const uint16_t *qp = q + (size_t)row * C + head * 64 + 8 * h;
    u32x4 w[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) w[s] = *(const u32x4 *)(qp + 16 * s);
    if (qk_norm) {   // this lane holds 32 of the row's 64 values, lane^32 the other 32
      float ss = (sumsq8(w[0]) + sumsq8(w[1])) + (sumsq8(w[2]) + sumsq8(w[3]));
      ss += __shfl_xor(ss, 32, 64);
      const float r = 1.0f / sqrtf(ss * (1.0f / 64.0f) + kQkEps);
#pragma unroll
      for (int s = 0; s < 4; ++s) w[s] = scale8(w[s], r);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[sub][s] = __builtin_bit_cast(bf16x8, w[s]);
  }

  f32x16 oacc[2][2];   // [query block][d tile]
#pragma unroll
  for (int sub = 0; sub < 2; ++sub)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[sub][dt][r] = 0.f;
  float mref[2] = {-INFINITY, -INFINITY}, lrow[2] = {0.f, 0.f};
  const bf16x2 kOnes = {(__bf16)1.0f, (__bf16)1.0f};

  const int nkv = n_kt >> 1;           // 64-key tiles
  const u32x4 *kh = kp + (size_t)sh * n_kt * 4 * kFragU4;
  const u32x4 *vh = vp + (size_t)sh * n_kt * 4 * kFragU4;
  u32x4 rk, rv;
  auto g2r = [&](int j) {              // global -> registers, 64-key tile j (16 B of K and V per thread)
    const size_t off = (size_t)j * 8 * kFragU4;
    rk = kh[off + tid];
    rv = vh[off + tid];
  };
  auto r2s = [&](int j) {              // registers -> LDS ring slots of tile j
    ks[j % kKSlots][tid] = rk;
    vs[j % kVSlots][tid] = rv;
  };

  f32x16 sacc[2][2];   // [key half][query block]: scores of one 64-key tile
  u32x4 pb[2][2][2];   // [query block][key half][u]: its bf16 weights

  // ---- matrix phase j: PV of tile j-1 (if any), scores of tile j (if any).  All LDS
  // fragment reads of a half-phase are issued before its MFMAs so that LDS latency is paid
  // once, not once per fragment.
  auto phase_m = [&](int j) {
    __builtin_amdgcn_sched_barrier(0);
    if (j > 0) {
      const u32x4 *vt = &vs[(j - 1) % kVSlots][lane];
      u32x4 vf[8];
#pragma unroll
      for (int f = 0; f < 8; ++f) vf[f] = vt[f * kFragU4];
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int dt = 0; dt < 2; ++dt) {
            const bf16x8 a = __builtin_bit_cast(bf16x8, vf[(kt2 * 2 + u) * 2 + dt]);
            oacc[0][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                a, __builtin_bit_cast(bf16x8, pb[0][kt2][u]), oacc[0][dt], 0, 0, 0);
            oacc[1][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                a, __builtin_bit_cast(bf16x8, pb[1][kt2][u]), oacc[1][dt], 0, 0, 0);
          }
      __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (j < nkv) {
      const u32x4 *kt = &ks[j % kKSlots][lane];
      u32x4 kf[8];
#pragma unroll
      for (int f = 0; f < 8; ++f) kf[f] = kt[f * kFragU4];
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2) {
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
          for (int r = 0; r < 16; ++r) sacc[kt2][sub][r] = 0.f;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const bf16x8 a = __builtin_bit_cast(bf16x8, kf[kt2 * 4 + s]);
          sacc[kt2][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[0][s], sacc[kt2][0], 0, 0, 0);
          sacc[kt2][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[1][s], sacc[kt2][1], 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);
    }
    // The phase discipline only works if this phase's MFMAs are really issued here: make
    // their results opaque so that nothing is sunk past the barrier into the vector phase.
    asm volatile("" : "+v"(sacc[0][0]), "+v"(sacc[0][1]), "+v"(sacc[1][0]), "+v"(sacc[1][1]),
                 "+v"(oacc[0][0]), "+v"(oacc[0][1]), "+v"(oacc[1][0]), "+v"(oacc[1][1]));
    __builtin_amdgcn_sched_barrier(0);
  };
  // ---- vector phase j: online softmax of tile j, one query column per lane.  The running
  // reference mref is only raised (and O, l rescaled) when some lane's tile maximum exceeds
  // it by more than kRaise in log2 units, so weights stay below 2^kRaise and rescaling is rare.
  auto phase_v = [&](int j) {
    __builtin_amdgcn_sched_barrier(0);
    if (j == nkv - 1) {   // keys beyond the sequence end in the last tile
      const int64_t kbase = (int64_t)j * kKV;
      if (kbase + kKV > n) {
#pragma unroll
        for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int64_t key = kbase + kt2 * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
            if (key >= n) {
              sacc[kt2][0][r] = -INFINITY;
              sacc[kt2][1][r] = -INFINITY;
            }
          }
      }
    }
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      {
        float mx = -INFINITY;
#pragma unroll
        for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
          for (int r = 0; r < 16; r += 2) mx = max3(mx, sacc[kt2][sub][r], sacc[kt2][sub][r + 1]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        if (__builtin_amdgcn_ballot_w64((mx - mref[sub]) * c > kRaise) != 0) {
          const float mnew = fmaxf(mref[sub], mx);
          const float alpha = __builtin_amdgcn_exp2f((mref[sub] - mnew) * c);
          mref[sub] = mnew;
          lrow[sub] *= alpha;
#pragma unroll
          for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[sub][dt][r] *= alpha;
        }
      }
      float ls = lrow[sub];
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          uint32_t w[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float s0 = sacc[kt2][sub][8 * u + 2 * e], s1 = sacc[kt2][sub][8 * u + 2 * e + 1];
            // the difference first: scores are of any size here, and c * s - c * mref with the
            // second product rounded is off by 2^-24 of it, i.e. by thousands once scores reach 1e11
            const float p0 = __builtin_amdgcn_exp2f((s0 - mref[sub]) * c);
            const float p1 = __builtin_amdgcn_exp2f((s1 - mref[sub]) * c);
            w[e] = pack_bf16(p0, p1);
            // row sum of the bf16-rounded weights (what the second MFMA really multiplies)
            ls = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w[e]), kOnes, ls, false);
          }
          pb[sub][kt2][u] = u32x4{w[0], w[1], w[2], w[3]};
        }
      }
      lrow[sub] = ls;
    }
    // likewise the weights must exist before the barrier, not be recomputed lazily after it
    asm volatile("" : "+v"(pb[0][0][0]), "+v"(pb[0][0][1]), "+v"(pb[0][1][0]), "+v"(pb[0][1][1]),
                 "+v"(pb[1][0][0]), "+v"(pb[1][0][1]), "+v"(pb[1][1][0]), "+v"(pb[1][1][1]),
                 "+v"(lrow[0]), "+v"(lrow[1]));
    __builtin_amdgcn_sched_barrier(0);
  };

  g2r(0);
  r2s(0);
  __syncthreads();
  // Global phases p = 0 .. 2*nkv+1; group g works on local phase p-g: even local phases are
  // matrix phases, odd ones vector phases.  Every wave passes every barrier (2 per j, for
  // j = 0 .. nkv).  Tile j+1 is fetched during phase 2j and written to LDS during phase
  // 2j+1: its K slot held tile j-1 (last read in phase 2j-1) and its V slot tile j-2 (last
  // read in phase 2j-1).  The two groups run separate copies of the loop so that each is
  // straight-line code for the register allocator.
  if (grp == 0) {
    for (int j = 0; j < nkv; ++j) {
      if (j + 1 < nkv) g2r(j + 1);
      phase_m(j);                        // phase 2j
      __syncthreads();
      if (j + 1 < nkv) r2s(j + 1);
      phase_v(j);                        // phase 2j+1
      __syncthreads();
    }
    phase_m(nkv);                        // phase 2*nkv: last PV
    __syncthreads();
    __syncthreads();
  } else {
    if (nkv > 1) g2r(1);
    __syncthreads();                     // phase 0: idle
    if (nkv > 1) r2s(1);
    phase_m(0);                          // phase 1
    __syncthreads();
    for (int j = 1; j < nkv; ++j) {
      if (j + 1 < nkv) g2r(j + 1);
      phase_v(j - 1);                    // phase 2j
      __syncthreads();
      if (j + 1 < nkv) r2s(j + 1);
      phase_m(j);                        // phase 2j+1
      __syncthreads();
    }
    phase_v(nkv - 1);                    // phase 2*nkv
    __syncthreads();
    phase_m(nkv);                        // phase 2*nkv+1: last PV
    __syncthreads();
  }

  // ---- normalise and store: lane holds query column ql, rows d = 32dt + 8g + 4h + i
  // second pass: the 256-query half that the first pass completed keeps its rows (with a fused
  // residual in place they already hold the sum)
  const bool mine = !redo || redo[(size_t)sh * (2 * nqb) + 2 * qb + grp] != 0u;
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const float l = lrow[sub] + __shfl_xor(lrow[sub], 32, 64);
    const float inv = 1.0f / l;
    const int64_t row = q0 + sub * 32 + ql;
    if (row < n && mine) {
      uint16_t *op = o + (size_t)row * C + head * 64 + 4 * h;
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float r0 = oacc[sub][dt][4 * g] * inv, r1 = oacc[sub][dt][4 * g + 1] * inv;
          float r2 = oacc[sub][dt][4 * g + 2] * inv, r3 = oacc[sub][dt][4 * g + 3] * inv;
          if (res) {   // out = res + attention, one rounding (res may be the output buffer)
            const u32x2 x = *(const u32x2 *)(res + (size_t)row * C + head * 64 + 4 * h + 32 * dt + 8 * g);
            r0 += bf16_lo(x.x);
            r1 += bf16_hi(x.x);
            r2 += bf16_lo(x.y);
            r3 += bf16_hi(x.y);
          }
          const u32x2 w = {pack_bf16(r0, r1), pack_bf16(r2, r3)};
          *(u32x2 *)(op + 32 * dt + 8 * g) = w;
        }
    }
  }
}

// ---------------------------------------------------------------------------------------
// The main attention kernel.  A wave owns two 32-query blocks that run half a 32-key step
// apart, which gives every stretch of the instruction stream independent VALU (exp2, bf16
// pack, row sum of one block) and MFMA work (PV and next scores of the other):
//   A(t): weights of block 0, tile t   ||  PV of block 1, tile t-1;  scores of block 1, tile t
//   B(t): weights of block 1, tile t   ||  PV of block 0, tile t;    scores of block 0, tile t+1
// The MFMAs are interleaved with the VALU work by an explicit scheduling recipe.
//
// The softmax scale (in log2 units) is folded into q before its one bf16 rounding, so a
// score leaves the MFMA ready for exp2.  What the exponent is taken against:
//   ONLINE = false (unit-RMS q and k whose scores cannot exceed 64 in log2 units): nothing;
//     softmax is invariant to the reference and exp2 of a bounded score cannot overflow.  The
//     loop has no maximum, no subtraction, no rescale and no branch.
//   ONLINE = true: online softmax with one running reference R per wave, raised lazily.  The
//     score accumulators start from -R (the MFMA's C operand), so the steady state costs the
//     same instructions plus one compare and branch per phase: a tile whose weights push a row
//     sum beyond 2^40 (some score more than ~40 above R, or not finite) triggers a raise: R
//     moves to that tile's maximum, O and the row sums of both blocks are rescaled by 2^-(R' - R),
//     the scores still pending are re-based, the tile's weights are recomputed.  fp32 covers
//     rows up to ~100 binades apart in one wave; a 256-query block in which some row ends with a
//     sum below 2^-60 (all its scores far below its wave's reference), or whose reference grows
//     beyond kRefUseful (where the bf16 rounding of the scaled q no longer resolves the
//     scores), writes nothing, sets its flag, and the per-row kernel k_attn_bf16 redoes it.
// ---------------------------------------------------------------------------------------
// waits until every LDS operation issued so far has completed
__device__ __forceinline__ void lds_wait(u32x4 (&a)[4], u32x4 (&b)[4]) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]),
                 "+v"(b[3])
               :
               : "memory");
}

constexpr int kBQB = 256;            // queries per workgroup (4 waves)
constexpr float kRefUseful = 256.0f; // largest reference (log2 units) the folded scale resolves scores against
constexpr float kSumRaise = 1.0995116e12f;   // 2^40: a row sum beyond it raises the wave's reference
constexpr int kBStages = 4;          // LDS ring of 64-key K/V stages


// ---- Cutting the blocks of a short sequence.  A workgroup (256 queries of one head, all keys) takes
// as long as any other and two fit on a CU, so fewer than 512 leave CUs idle: 368 blocks (5776 tokens,
// 16 heads) put two on 112 CUs and one, which runs 1.5 times as fast alone, on 144: 149 us.  The
// blocks are therefore cut in two along the keys, the first piece as long as k second pieces, so that
// the slots the first pieces leave idle take k second pieces each (137 us).  The piece that comes to
// its end first leaves its fp32 sums (O, row sums, ONLINE: the waves' references) in the workspace,
// the other one waits until they are there (it is a workgroup that is running, and writing them is
// the last thing it does), adds them to its own and finishes the block.  The sum of two is the same
// in either order.  XCD x's blocks are those of its heads (heads a multiple of 8), so the same cut
// serves every XCD.
struct AttnCut {
  int n_cut;                                 // blocks per XCD, all of them cut (0: none is)
  int small;                                 // stages of a second piece
};
constexpr size_t kPieceFloats = (size_t)256 * 64 + 2 * 256 * 2;   // O, row sums, references of one piece

// The end of a piece (every wave of its workgroup comes here, except those beyond the sequence end):
// false: the other piece finishes the block; true: the sums now cover all keys.
template <bool ONLINE>
__device__ __forceinline__ bool join_pieces(f32x16 (&oacc)[2][2], float (&lsub)[2], float ref, uint32_t *sync,
                                            float *partial, int wave, int lane) {
#pragma clang fp contract(off)
  __shared__ uint32_t arrived;
  const bool lead = lane == 0 && __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0;   // wave 0 is never beyond the end
  if (lead) arrived = __hip_atomic_fetch_add(sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  // The sums travel in relaxed agent-scope atomics of 8 bytes, which go to where every XCD sees them
  // and are there when the wave's store counter says so.  (Plain stores between fences of that scope
  // write back and invalidate the whole L2 each time: 150 us became 228.)
  auto put = [&](size_t at, float x, float y) {
    const uint64_t v = (uint64_t)__float_as_uint(x) | (uint64_t)__float_as_uint(y) << 32;
    __hip_atomic_store((uint64_t *)partial + at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto get = [&](size_t at) {
    const uint64_t v = __hip_atomic_load((uint64_t *)partial + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return f32x2{__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32))};
  };
  const size_t row = (size_t)256 * 32 + wave * 64 + lane;   // after O: per wave and lane (row sum, reference)
  if (arrived == 0u) {
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          put((((wave * 2 + sub) * 2 + dt) * 8 + e) * 64 + lane, oacc[sub][dt][2 * e], oacc[sub][dt][2 * e + 1]);
    put(row, lsub[0], lsub[1]);
    if (ONLINE) put(row + 256, ref, 0.f);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (lead) __hip_atomic_store(sync + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
  }
  if (lead)
    while (__hip_atomic_load(sync + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) __builtin_amdgcn_s_sleep(1);
  __syncthreads();
  float mine = 1.0f, theirs = 1.0f;
  if (ONLINE) {                              // both to the larger of the two references
    const float r = get(row + 256)[0], top = fmaxf(ref, r);
    mine = __builtin_amdgcn_exp2f(ref - top);
    theirs = __builtin_amdgcn_exp2f(r - top);
  }
  const f32x2 l = get(row);
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) {
      f32x2 v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = get((((wave * 2 + sub) * 2 + dt) * 8 + e) * 64 + lane);
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          oacc[sub][dt][2 * e + i] = ONLINE ? oacc[sub][dt][2 * e + i] * mine + v[e][i] * theirs : oacc[sub][dt][2 * e + i] + v[e][i];
    }
    lsub[sub] = ONLINE ? lsub[sub] * mine + l[sub] * theirs : lsub[sub] + l[sub];
  }
  return true;
}

// PACKED (one sequence, no residual, not ONLINE): `o` is a linear layer's activation operand
// buffer and receives the output rows in that layer's fragment order, [row / 32][k-step of 16
// channels][lane = row % 32 + 32 * (second 8 of the 16)], 16 bytes each.
// CUT: the blocks are pieces (AttnCut).
template <bool ONLINE, bool PACKED, bool CUT>
__device__ __forceinline__ void attn_bf16_main(
    const uint16_t *q, const u32x4 *__restrict__ kp, const u32x4 *__restrict__ vp, uint16_t *o,
    const uint16_t *res, int64_t n, int heads, int n_seq, int n_kt, int nqb, float c, int qk_norm,
    uint32_t *__restrict__ redo, int redo_stride, AttnCut cut, uint32_t *sync, float *partial) {
  __shared__ u32x4 ks[kBStages][8 * kFragU4];
  __shared__ u32x4 vs[kBStages][8 * kFragU4];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ql = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C = heads * 64;
  int sh, qb;   // (sequence, head) pair and query block; each XCD gets whole pairs
  int first = 0, nkv = n_kt >> 1;   // the stages this workgroup takes (a piece: not all of them)
  int piece = -1;                   // number of the cut block
  if (((heads * n_seq) & 7) == 0) {
    const int hp = (heads * n_seq) >> 3, xcd = blockIdx.x & 7;
    int local = blockIdx.x >> 3;
    if constexpr (CUT) {            // first all first pieces, then all second ones
      if (local < cut.n_cut) {
        nkv -= cut.small;
      } else {
        local -= cut.n_cut;
        first = nkv - cut.small;
        nkv = cut.small;
      }
      piece = xcd * cut.n_cut + local;
    }
    sh = xcd * hp + local / nqb;
    qb = local % nqb;
  } else {
    sh = blockIdx.x / nqb;
    qb = blockIdx.x % nqb;
  }
  const int seq = sh / heads, head = sh - seq * heads;
  q += (size_t)seq * n * C;
  o += (size_t)seq * n * C;
  if (res) res += (size_t)seq * n * C;
  const int64_t q0 = (int64_t)qb * kBQB + wave * kQW;

  const int nkt = 2 * nkv;
  const int64_t n_keys = n - (int64_t)first * kKV;   // keys from the first one of these stages to the sequence end
  const u32x4 *kh = kp + ((size_t)sh * n_kt + 2 * first) * 4 * kFragU4;
  const u32x4 *vh = vp + ((size_t)sh * n_kt + 2 * first) * 4 * kFragU4;
  // Stage `stage` of this head's packed K and V (64 keys, 8 KB each) goes from global memory
  // straight into its ring slot, 1 KB per wave and instruction (global_load_lds_dwordx4: lane l
  // of a wave lands at the wave's LDS base + 16 l).  No registers are staged, so a stage can be
  // fetched three iterations before its first use.  Completion is per wave (vmcnt) and is
  // published to the workgroup by the barrier of the steady-state loop.
  auto fetch = [&](int stage) {
    const int slot = stage & (kBStages - 1);
    const size_t off = (size_t)stage * 8 * kFragU4 + tid;
    __builtin_amdgcn_global_load_lds(kh + off, &ks[slot][wave * 64], 16, 0, 0);
    __builtin_amdgcn_global_load_lds(kh + off + 256, &ks[slot][256 + wave * 64], 16, 0, 0);
    __builtin_amdgcn_global_load_lds(vh + off, &vs[slot][wave * 64], 16, 0, 0);
    __builtin_amdgcn_global_load_lds(vh + off + 256, &vs[slot][256 + wave * 64], 16, 0, 0);
  };
  // the first two stages are requested before q is loaded and normalised: one memory round
  // trip for both (short sequences, e.g. frame attention, have few stages to hide it behind)
  fetch(0);
  fetch(min(1, nkv - 1));

  // Q^T fragments with the softmax scale (log2 units) folded in, RMS-normalised per head when
  // qk_norm is set
  bf16x8 qf[2][4];
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const int64_t row = min(q0 + sub * 32 + ql, n - 1);
    const uint16_t *qp = q + (size_t)row * C + head * 64 + 8 * h;
    u32x4 w[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) w[s] = *(const u32x4 *)(qp + 16 * s);
    float ss = (sumsq8(w[0]) + sumsq8(w[1])) + (sumsq8(w[2]) + sumsq8(w[3]));
    ss += __shfl_xor(ss, 32, 64);
    const float r = qk_norm ? c / sqrtf(ss * (1.0f / 64.0f) + kQkEps) : c;
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[sub][s] = __builtin_bit_cast(bf16x8, scale8(w[s], r));
  }

  f32x16 oacc[2][2];   // [query block][d tile]
#pragma unroll
  for (int sub = 0; sub < 2; ++sub)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[sub][dt][r] = 0.f;
  float lrow[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
  // what the score accumulators start from: 0, or minus the wave's running reference (16
  // registers that stay live through the loop; one per query block would not fit, a subtraction
  // per score would cost a fifth of the kernel's VALU time)
  f32x16 s_start = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float ref_run = 0.f;         // ONLINE: the reference R (uniform over the wave)
  bool over = false;           // ONLINE: R went beyond kRefUseful
  float lnew[2] = {0.f, 0.f};  // ONLINE: row sums including the tile whose weights were just taken

  f32x16 sacc[2];      // [query block]: scores of its current 32-key tile
  u32x4 pb[2][2];      // [query block][u]: bf16 weights of its current 32-key tile
  // Fragments held in registers feed both query blocks: fv[t & 1] = V fragments of tile t
  // (used in B(t), A(t+1)), fk[t & 1] = K fragments of tile t (used in B(t-1), A(t)).
  u32x4 fv[2][4], fk[2][4];

  auto load_v = [&](int t, u32x4(&dst)[4]) {
    const u32x4 *vt = &vs[(t >> 1) & (kBStages - 1)][(t & 1) * 4 * kFragU4 + lane];
#pragma unroll
    for (int f = 0; f < 4; ++f) dst[f] = vt[f * kFragU4];
  };
  auto load_k = [&](int t, u32x4(&dst)[4]) {
    const u32x4 *kt = &ks[(t >> 1) & (kBStages - 1)][(t & 1) * 4 * kFragU4 + lane];
#pragma unroll
    for (int f = 0; f < 4; ++f) dst[f] = kt[f * kFragU4];
  };
  auto mma_s = [&](int sub, const u32x4(&kf)[4]) {
    f32x16 acc = s_start;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[s]), qf[sub][s],
                                                    acc, 0, 0, 0);
    sacc[sub] = acc;
  };
  auto mma_pv = [&](int sub, const u32x4(&vf)[4]) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
        oacc[sub][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8, vf[u * 2 + dt]), __builtin_bit_cast(bf16x8, pb[sub][u]),
            oacc[sub][dt], 0, 0, 0);
  };
  auto mask_tail = [&](int t, int sub) {   // keys beyond the sequence end
    if ((int64_t)(t + 1) * kKT > n_keys) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t key = (int64_t)t * kKT + (r >> 2) * 8 + h * 4 + (r & 3);
        if (key >= n_keys) sacc[sub][r] = -INFINITY;
      }
    }
  };
  // exp2 of the scaled scores, bf16 pack, row sums.  The sums are plain fp32 adds of the
  // unrounded weights in two chains: v_dot2c_f32_bf16 on the packed pairs would halve the
  // instruction count, but it does not overlap with MFMAs (measured: a phase with dot2 row sums
  // takes as long as its MFMA and VALU parts one after the other, with adds it takes 1.1x its
  // MFMA part).
  auto weights = [&](int sub) {
    float l0 = lrow[sub][0], l1 = lrow[sub][1];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p0 = __builtin_amdgcn_exp2f(sacc[sub][8 * u + 2 * e]);
        const float p1 = __builtin_amdgcn_exp2f(sacc[sub][8 * u + 2 * e + 1]);
        w[e] = pack_bf16(p0, p1);
        l0 += p0;
        l1 += p1;
      }
      pb[sub][u] = u32x4{w[0], w[1], w[2], w[3]};
    }
    if (ONLINE) {      // held back until settle() has seen them
      lnew[0] = l0;
      lnew[1] = l1;
    } else {
      lrow[sub][0] = l0;
      lrow[sub][1] = l1;
    }
  };
  // ONLINE, at the end of the phase that took the weights of block `sub`: accept the new row
  // sums, or raise the reference first.  At this point the other block's weights have been
  // consumed (its PV was issued in this phase), its scores of the next tile are pending, and no
  // MFMA of `sub`'s tile has been issued yet.
  auto settle = [&](int sub) {
    if (!ONLINE) return;
    __builtin_amdgcn_sched_barrier(0);
    if (__builtin_amdgcn_ballot_w64(!(lnew[0] + lnew[1] <= kSumRaise)) != 0) {
      // fragment reads issued by hand may be in flight: let them land before anything else
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      float mx = sacc[sub][0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sacc[sub][r]);
      const float delta = fmaxf(wave_max(mx), 0.f);      // how far the tile's maximum lies above R
      const float alpha = __builtin_amdgcn_exp2f(-delta);
      ref_run += delta;
      over |= !(ref_run <= kRefUseful);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        lrow[b][0] *= alpha;
        lrow[b][1] *= alpha;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[b][dt][r] *= alpha;
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[b][r] -= delta;   // own tile: redone below; other block: pending scores
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) s_start[r] = -ref_run;
      weights(sub);
    }
    lrow[sub][0] = lnew[0];
    lrow[sub][1] = lnew[1];
    __builtin_amdgcn_sched_barrier(0);
  };
  // One phase = 8 MFMAs + the weights of 16 scores per lane (16 exp2, 8 pack, 16 add).  The
  // recipe asks the scheduler to spread the MFMAs over the VALU work; A phases re-fill fv
  // after their 4 PV MFMAs and fk after their 4 score MFMAs.  (Forcing a strict
  // exp2/exp2/MFMA/pack/sum order with opaque pins was measured slower than this.)
  auto recipe = [&]() {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);   // 2 exp2
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // 1 MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);   // pack + 2 adds
    }
  };
  // In the steady state the fragment reads are issued by hand (lds_read4_async): V(t) and
  // K(t+1) at the start of A(t); B(t) is their first user and waits for them a whole phase
  // later.  Both are double-buffered, so the registers a read overwrites were last used by
  // MFMAs a whole phase before it is issued.
  const uint32_t ks_lane = lds_addr(&ks[0][lane]), vs_lane = lds_addr(&vs[0][lane]);
  auto frag_off = [&](int t) {   // byte offset of tile t's four fragments in a ring array
    return (uint32_t)((((t >> 1) & (kBStages - 1)) * 8 + (t & 1) * 4) * kFragU4 * 16);
  };
  // A(t), t >= 1: weights of block 0 || PV(t-1) and scores(t) of block 1
  int fslot = 0;       // ring slot and source offset of the stage being fetched
  size_t foff = 0;
  auto fetch1 = [&](int q) {   // one of the four fetch instructions of a stage
    const u32x4 *src = (q < 2 ? kh : vh) + foff + (q & 1) * 256;
    u32x4 *dst = (q < 2 ? &ks[fslot][0] : &vs[fslot][0]) + (q & 1) * 256 + wave * 64;
    __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
  };
  auto phase_a = [&](int t, const u32x4(&v_prev)[4], u32x4(&v_cur)[4], const u32x4(&k_cur)[4],
                     u32x4(&k_next)[4], int fq = -1) {
    lds_read4_async(v_cur, vs_lane + frag_off(t));
    lds_read4_async(k_next, ks_lane + frag_off(t + 1));   // past the last tile: a stale slot, never used
    if (fq >= 0) fetch1(fq);
    __builtin_amdgcn_sched_barrier(0);
    weights(0);
    mma_pv(1, v_prev);
    mma_s(1, k_cur);
    recipe();
    settle(0);
  };
  // B(t), t <= nkt-2: weights of block 1 || PV(t) and scores(t+1) of block 0
  auto phase_b = [&](u32x4(&v_cur)[4], u32x4(&k_next)[4], int fq = -1) {
    __builtin_amdgcn_sched_barrier(0);     // the work of A(t) stays ahead of the wait
    lds_wait(v_cur, k_next);
    if (fq >= 0) {
      fetch1(fq);
      __builtin_amdgcn_sched_barrier(0);
    }
    weights(1);
    mma_pv(0, v_cur);
    mma_s(0, k_next);
    recipe();
    settle(1);
  };

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  fetch(min(2, nkv - 1));                  // in flight during the prologue and the first iteration
  if (q0 >= n) {
    // All 64 queries of this wave lie beyond the sequence end (the ragged last block: 1374
    // tokens per frame are 5.4 blocks).  The wave only moves its share of the K/V stages and
    // keeps the workgroup's barriers company, leaving both pipes of its SIMD to the other
    // workgroup resident there.
    if (ONLINE && __syncthreads_or(0)) {     // the other waves' first-tile check
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      return;
    }
    for (int i = 0; i < nkv - 2; ++i) {
      fslot = (i + 3) & (kBStages - 1);
      foff = (size_t)min(i + 3, nkv - 1) * 8 * kFragU4 + tid;
      fetch1(0);
      fetch1(1);
      fetch1(2);
      asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      fetch1(3);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (ONLINE) __syncthreads_or(0);         // the other waves' final check
    return;
  }
  // prologue: scores of tile 0 for both blocks, weights of block 0, then V(0) and K(1)
  load_k(0, fk[0]);
  mma_s(0, fk[0]);
  mask_tail(0, 0);
  if (ONLINE) {
    // the reference starts at the largest score of the first tile (both blocks)
    mma_s(1, fk[0]);
    mask_tail(0, 1);
    float mx = fmaxf(sacc[0][0], sacc[1][0]);
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, fmaxf(sacc[0][r], sacc[1][r]));
    ref_run = wave_max(mx);
    // A reference this large cannot serve (and one that is not finite cannot at all): the block
    // goes to the second pass without being computed here first.
    if (__syncthreads_or(!(ref_run <= kRefUseful))) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the stages already requested land before the workgroup ends
      if (tid == 0) redo[(size_t)sh * redo_stride + qb] = 1u;
      return;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s_start[r] = -ref_run;
      sacc[0][r] -= ref_run;
      sacc[1][r] -= ref_run;
    }
    weights(0);
    lrow[0][0] = lnew[0];
    lrow[0][1] = lnew[1];
  } else {
    weights(0);
    mma_s(1, fk[0]);
  }
  load_v(0, fv[0]);
  load_k(1, fk[1]);
  if (!ONLINE && nkv == 1) mask_tail(0, 1);
  // steady state: stage i holds tiles 2i, 2i+1; iteration i reads stages i and i+1, stage i+2
  // is in flight since the previous iteration and stage i+3 is fetched now, into the slot of
  // stage i-1, which every wave finished reading before the previous barrier.  (Past the end
  // the last stage is fetched again into a slot nobody reads: the loop body has no branches.)
  for (int i = 0; i < nkv - 2; ++i) {
    // one fetch instruction at the head of each phase
    fslot = (i + 3) & (kBStages - 1);
    foff = (size_t)min(i + 3, nkv - 1) * 8 * kFragU4 + tid;
    phase_b(fv[0], fk[1], 0);                           // B(2i)
    phase_a(2 * i + 1, fv[0], fv[1], fk[1], fk[0], 1);  // A(2i+1)
    phase_b(fv[1], fk[0], 2);                           // B(2i+1)
    // this wave's part of stage i+2 has landed (the three newest loads, of stage i+3, may still
    // be in flight); after the barrier all of stage i+2 is readable: first read in A(2i+3)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    phase_a(2 * i + 2, fv[1], fv[0], fk[0], fk[1], 3);  // A(2i+2)
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing may land after the workgroup ends
  if (nkv >= 2) {                          // stage nkv-2; it enters the last stage, whose tiles may be ragged
    const int i = nkv - 2;
    phase_b(fv[0], fk[1]);
    phase_a(2 * i + 1, fv[0], fv[1], fk[1], fk[0]);
    phase_b(fv[1], fk[0]);
    mask_tail(2 * i + 2, 0);
    phase_a(2 * i + 2, fv[1], fv[0], fk[0], fk[1]);
    mask_tail(2 * i + 2, 1);
  }
  // last stage: tiles nkt-2, nkt-1
  phase_b(fv[0], fk[1]);                   // B(nkt-2)
  mask_tail(nkt - 1, 0);
  phase_a(nkt - 1, fv[0], fv[1], fk[1], fk[0]);   // A(nkt-1)
  mask_tail(nkt - 1, 1);
  lds_wait(fv[1], fk[0]);
  weights(1);
  mma_pv(0, fv[1]);
  settle(1);
  mma_pv(1, fv[1]);

  float lsub[2];
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const float lsum = lrow[sub][0] + lrow[sub][1];
    lsub[sub] = lsum + __shfl_xor(lsum, 32, 64);
  }
  __shared__ int any_low;     // CUT only
  if constexpr (CUT) {
    if (ONLINE && __syncthreads_or(over)) {   // the block is the second pass's; the other piece waits for nobody
      if (tid == 0) redo[(size_t)sh * redo_stride + qb] = 1u;
      return;
    }
    if (ONLINE && tid == 0) any_low = 0;
    if (!join_pieces<ONLINE>(oacc, lsub, ref_run, sync + 2 * piece, partial + (size_t)piece * kPieceFloats, wave, lane)) return;
  }
  if (ONLINE) {
    // A row whose scores all lie ~60 binades or more below its wave's reference has lost its
    // weights to underflow, and a reference beyond kRefUseful is not resolved: the whole
    // 256-query block is left to the per-row kernel, and nothing of it is written here (the
    // output may alias the residual).
    bool low = over;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) low |= q0 + sub * 32 + ql < n && !(lsub[sub] >= 8.67e-19f);   // 2^-60
    bool redo_block;
    if constexpr (CUT) {      // the waves beyond the sequence end are gone by now: a plain barrier
      if (__builtin_amdgcn_ballot_w64(low) != 0 && lane == 0) any_low = 1;
      __syncthreads();
      redo_block = any_low != 0;
    } else {
      redo_block = __syncthreads_or(low);
    }
    if (redo_block) {
      if (tid == 0) redo[(size_t)sh * redo_stride + qb] = 1u;
      return;
    }
  }
  if constexpr (PACKED) {
    // a lane holds channels 8g + 4h .. + 3 of its query per group of four registers: lanes l and
    // l + 32 trade halves (first operand's lanes 32-63 <-> second operand's lanes 0-31), after
    // which lane l has channels 0-7 and lane l + 32 channels 8-15 of a k-step: 1 KB per store
    u32x4 *op = (u32x4 *)o;
    const int KS = C >> 4;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      const bool live = q0 + sub * 32 + ql < n;
      const float inv = live ? 1.0f / lsub[sub] : 0.f;
      const size_t base = ((size_t)((q0 + sub * 32) >> 5) * KS + head * 4) * 64 + lane;
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
          float r[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) r[i] = live ? oacc[sub][dt][8 * gp + i] * inv : 0.f;
          const auto s0 = __builtin_amdgcn_permlane32_swap(pack_bf16(r[0], r[1]), pack_bf16(r[4], r[5]), false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(pack_bf16(r[2], r[3]), pack_bf16(r[6], r[7]), false, false);
          op[base + (size_t)(dt * 2 + gp) * 64] = u32x4{s0[0], s1[0], s0[1], s1[1]};
        }
    }
    return;
  }
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const float l = lsub[sub];
    const float inv = 1.0f / l;
    const int64_t row = q0 + sub * 32 + ql;
    if (row < n) {
      uint16_t *op = o + (size_t)row * C + head * 64 + 4 * h;
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float r0 = oacc[sub][dt][4 * g] * inv, r1 = oacc[sub][dt][4 * g + 1] * inv;
          float r2 = oacc[sub][dt][4 * g + 2] * inv, r3 = oacc[sub][dt][4 * g + 3] * inv;
          if (res) {   // out = res + attention, one rounding (res may be the output buffer)
            const u32x2 x = *(const u32x2 *)(res + (size_t)row * C + head * 64 + 4 * h + 32 * dt + 8 * g);
            r0 += bf16_lo(x.x);
            r1 += bf16_hi(x.x);
            r2 += bf16_lo(x.y);
            r3 += bf16_hi(x.y);
          }
          const u32x2 w = {pack_bf16(r0, r1), pack_bf16(r2, r3)};
          *(u32x2 *)(op + 32 * dt + 8 * g) = w;
        }
    }
  }
}

template <bool ONLINE, bool PACKED = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_attn_bf16_main(
    const uint16_t *q, const u32x4 *__restrict__ kp, const u32x4 *__restrict__ vp, uint16_t *o,
    const uint16_t *res, int64_t n, int heads, int n_seq, int n_kt, int nqb, float c, int qk_norm,
    uint32_t *__restrict__ redo, int redo_stride) {
  attn_bf16_main<ONLINE, PACKED, false>(q, kp, vp, o, res, n, heads, n_seq, n_kt, nqb, c, qk_norm, redo, redo_stride,
                                        AttnCut{0, 0}, nullptr, nullptr);
}
template <bool ONLINE, bool PACKED = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_attn_bf16_cut(
    const uint16_t *q, const u32x4 *__restrict__ kp, const u32x4 *__restrict__ vp, uint16_t *o,
    int64_t n, int heads, int n_kt, int nqb, float c, int qk_norm,
    uint32_t *__restrict__ redo, int redo_stride, AttnCut cut, uint32_t *sync, float *partial) {
  attn_bf16_main<ONLINE, PACKED, true>(q, kp, vp, o, nullptr, n, heads, 1, n_kt, nqb, c, qk_norm, redo, redo_stride, cut,
                                       sync, partial);
}

// ---------------------------------------------------------------------------------------
// More blocks than the chip holds at once.  The main kernel's loop without a running reference, in
// workgroups that stay: one per slot of the chip takes block after block, and the seam between two blocks is part of
// the stream.  The next block's number comes from a counter per XCD; its first two K/V stages are fetched during
// the last two of this one, into the ring as if they followed them; its q rows and this block's
// residual rows are requested while the last weights are taken: neither a workgroup start nor a round trip
// to memory stands between them, and the other workgroup of the CU has less time to run alone in.  K/V
// stages, slots and phases as in attn_bf16_main (the scores' MFMAs stand first in a phase's source, or the
// scheduler leaves them to the phase's end: 3 % in long sequences).  Bound like the main kernel by the MFMA and VALU issue of the loop.
// One launch per block -> this: frame attention, 16 heads, 100 frames of 37 x 37 943 -> 911 us, 50 of 28 x 37 321 ->
// 307, 200 of 16 x 16 261 -> 209; one sequence of 9000 tokens 348 -> 333, 15432 821 -> 802, 60000 11685 -> 11632.
// ---------------------------------------------------------------------------------------
constexpr int kStreamStages = 4;     // key stages of a sequence, at least
constexpr int kStreamMost = 1024;    // ... and at most (65,536 keys): the seam is nothing beside a longer block (100,000
                                     // tokens level, 143,232 level on one box and 3 % slower on another)
constexpr int kVRowsStages = 64;     // key stages of a sequence whose V is read as it lies, at most
constexpr int kStreamWords = 8 * 8;  // counters: one per XCD, 32 bytes apart
constexpr int kGiveWayStages = 32;   // (2,525 tokens, up to two rounds: 0.98 of one launch per block with, 0.96 without; 1,805
                                     // 0.98 and 1.00, 765 0.99 and 1.06)

// VROWS: V is not re-laid out, which takes as long as K (100 frames of 37 x 37, 16 heads: 133 us for both, 90 for K).  Its rows
// go into the ring as they lie, 64 of 128 bytes per stage, and the fragments come out by transposing reads, 16 per stage
// in place of 8.  The loop pays 1 to 3 % for them, so it is for sequences short enough that the copy weighs more, us:
// 200 frames of 16 x 16 207.8 -> 183.3, 100 of 37 x 37 941.5 -> 908.7, 20 of 60 x 60 1020 -> 1011, one sequence of 8,200 tokens
// 302.9 and 300.3, of 9,000 335.6 and 338.4, of 30,000 3102 and 3143.  (K's fragments asked for a phase earlier than V's, to spread the
// reads: level, and 2 to 4 registers short in the forms without a residual.)
// A sequence's last block, with at most half of its queries there, gives every wave 32 of them instead of 64 to one or two
// waves: the block's waves do half the work, and the SIMDs that had none of it share it, us: 200 frames of 16 x 16 (5 queries
// of 256) 190 -> 181, 50 of 28 x 37 (17) 299 -> 289, 100 of 37 x 37 (94) 874 -> 856.  The same additions in the same order.
// Both go for calls whose output lies apart from V: in place, as the layer driver has its frame attention, a block's output
// would take rows that another one still reads, and V is re-laid out.
// (In the forms with packed V, whose sequences are longer, the second loop costs 20 registers in scratch.)

// Eight transposing reads: the four fragments of 32 keys of V from its rows in LDS (k_attn_bf16_stream), two 8-byte
// halves each, not waited for.  addr: where channels 0-31 of the lane's row lie; channels 32-63 are at addr ^ 64 (rows of
// 128 bytes, at multiples of kVRowBytes).
constexpr size_t kVRowBytes = 128;
__device__ __forceinline__ void lds_read_vt_async(u32x2 (&dst)[8], uint32_t addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:1024\n\t"
               "ds_read_b64_tr_b16 %2, %9\n\tds_read_b64_tr_b16 %3, %9 offset:1024\n\t"
               "ds_read_b64_tr_b16 %4, %8 offset:2048\n\tds_read_b64_tr_b16 %5, %8 offset:3072\n\t"
               "ds_read_b64_tr_b16 %6, %9 offset:2048\n\tds_read_b64_tr_b16 %7, %9 offset:3072"
               : "=&v"(dst[0]), "=&v"(dst[1]), "=&v"(dst[2]), "=&v"(dst[3]), "=&v"(dst[4]), "=&v"(dst[5]), "=&v"(dst[6]), "=&v"(dst[7])
               : "v"(addr), "v"(addr ^ 64u)
               : "memory");
}

template <bool PACKED, bool RES, bool VROWS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_attn_bf16_stream(
    const uint16_t *q, const u32x4 *__restrict__ kp, const u32x4 *__restrict__ vp, const uint16_t *vrows, uint16_t *o,
    const uint16_t *res, int64_t n, int heads, int n_seq, int n_kt, int nqb, float c, int qk_norm, uint32_t *ctr) {
  __shared__ u32x4 ks[kBStages][8 * kFragU4];
  __shared__ __attribute__((aligned(kVRowBytes))) u32x4 vs[kBStages][8 * kFragU4];
  __shared__ int next_block;
  static_assert(__alignof__(vs) % kVRowBytes == 0, "lds_read_vt_async");
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ql = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C = heads * 64, nkv = n_kt >> 1, nkt = n_kt;
  // each XCD's list: the blocks of its (sequence, head) pairs; else one list for all
  const int pairs = heads * n_seq, lists = (pairs & 7) == 0 ? 8 : 1, list = lists == 8 ? blockIdx.x & 7 : 0;
  const int in_list = pairs / lists * nqb, slots = gridDim.x / lists;
  int blk = lists == 8 ? blockIdx.x >> 3 : blockIdx.x;

  int sh = 0, qb = 0;
  const u32x4 *kh, *vh;
  // VROWS: the head's columns of the sequence's rows; what lies beyond reads as zeros.  (Whole offsets are the lanes': the
  // scalar offset of a buffer load is left out of its check against the range.)
  __amdgpu_buffer_rsrc_t vb;
  // thread tid moves the 16-byte piece c of rows tid / 8 and tid / 8 + 32 to place c ^ 4 (row / 2 % 2) of the row in LDS, so
  // that the four rows that 32 lanes of a transposing read take 64 bytes each from lie in different banks
  const int v_off = VROWS ? (tid >> 3) * C * 2 + ((tid & 7) ^ (tid >> 4 & 1) * 4) * 16 : 0;
  auto place = [&](int b) {          // block b of the list: its pair, query block and packed K and V
    sh = list * (pairs / lists) + b / nqb;
    qb = b % nqb;
    kh = kp + (size_t)sh * n_kt * 4 * kFragU4 + tid;
    if constexpr (VROWS) {
      const int seq = sh / heads, head = sh - seq * heads;
      vb = __builtin_amdgcn_make_buffer_rsrc((void *)(vrows + (size_t)seq * n * C + head * 64), 0, (int)((n - 1) * C * 2 + 128),
                                             0x00020000);
    } else {
      vh = vp + (size_t)sh * n_kt * 4 * kFragU4 + tid;
    }
  };
  int base = 0;                      // ring slot of the block's stage 0
  int fslot = 0, fstage = 0;
  size_t foff = 0;
  auto fetch1 = [&](int part) {      // one of the four fetch instructions of a stage
    u32x4 *dst = (part < 2 ? &ks[fslot][0] : &vs[fslot][0]) + (part & 1) * 256 + wave * 64;
    if (VROWS && part >= 2) {
      int rows = (2 * fstage + (part & 1)) * 64 * C;
      asm volatile("" : "+s"(rows));   // (added here: the sums of the first stages would stay in registers all along)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vb, dst, 16, v_off + rows, 0, 0, 0);
    } else {
      const u32x4 *src = (part < 2 ? kh : vh) + foff + (part & 1) * 256;
      __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
    }
  };
  auto at_stage = [&](int src, int ring) {
    fslot = (base + ring) & (kBStages - 1);
    foff = (size_t)src * 8 * kFragU4;
    fstage = src;
  };
  auto fetch = [&](int stage) {
    at_stage(stage, stage);
    fetch1(0);
    fetch1(1);
    fetch1(2);
    fetch1(3);
  };
  auto narrow = [&]() { return VROWS && n - (int64_t)qb * kBQB <= kBQB / 2; };   // the block's waves take 32 queries each
  u32x4 qraw[2][4];
  auto load_q = [&]() {
    const int seq = sh / heads, head = sh - seq * heads, qw = narrow() ? kQW / 2 : kQW;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      const int64_t row = (int64_t)seq * n + min((int64_t)qb * kBQB + wave * qw + sub * 32 + ql, n - 1);
      const uint16_t *qp = q + (size_t)row * C + head * 64 + 8 * h;
#pragma unroll
      for (int s = 0; s < 4; ++s) qraw[sub][s] = *(const u32x4 *)(qp + 16 * s);
    }
  };

  bf16x8 qf[2][4];
  f32x16 oacc[2][2], sacc[2];
  float lrow[2][2];
  u32x4 pb[2][2], fk[2][4];
  using VF = std::conditional_t<VROWS, u32x2[8], u32x4[4]>;   // V fragments of a tile: as halves, or whole
  VF fv[2];
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // (of_sub: the query block; sub: whose registers hold its scores and weights)
  auto mma_s_of = [&](int of_sub, int sub, const u32x4(&kf)[4]) {
    f32x16 acc = zero;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[s]), qf[of_sub][s], acc, 0, 0, 0);
    sacc[sub] = acc;
  };
  auto mma_s = [&](int sub, const u32x4(&kf)[4]) { mma_s_of(sub, sub, kf); };
  auto frag_v = [&](const VF &vf, int f) {
    if constexpr (VROWS) return u32x4{vf[2 * f].x, vf[2 * f].y, vf[2 * f + 1].x, vf[2 * f + 1].y};
    else return vf[f];
  };
  auto mma_pv_of = [&](int of_sub, int sub, const VF &vf) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
        oacc[of_sub][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, frag_v(vf, u * 2 + dt)),
                                                                   __builtin_bit_cast(bf16x8, pb[sub][u]), oacc[of_sub][dt], 0, 0, 0);
  };
  auto mma_pv = [&](int sub, const VF &vf) { mma_pv_of(sub, sub, vf); };
  const int n_last = (int)(n - (int64_t)(nkv - 1) * kKV) - 4 * h;   // keys of the last stage, from this lane half's first row
  auto mask_tail = [&](int tile, int sub) {                         // tile 0, 1 of the last stage
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (tile * kKT + (r >> 2) * 8 + (r & 3) >= n_last) sacc[sub][r] = -INFINITY;
  };
  auto weights_of = [&](int of_sub, int sub) {
    float l0 = lrow[of_sub][0], l1 = lrow[of_sub][1];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p0 = __builtin_amdgcn_exp2f(sacc[sub][8 * u + 2 * e]);
        const float p1 = __builtin_amdgcn_exp2f(sacc[sub][8 * u + 2 * e + 1]);
        w[e] = pack_bf16(p0, p1);
        l0 += p0;
        l1 += p1;
      }
      pb[sub][u] = u32x4{w[0], w[1], w[2], w[3]};
    }
    lrow[of_sub][0] = l0;
    lrow[of_sub][1] = l1;
  };
  auto weights = [&](int sub) { weights_of(sub, sub); };
  auto recipe = [&]() {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);   // 2 exp2
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // 1 MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);   // pack + 2 adds
    }
  };
  const uint32_t ks_lane = lds_addr(&ks[0][lane]);
  const uint32_t vs_lane = VROWS ? lds_addr(&vs[0][0]) + (4 * h + (lane >> 2 & 3)) * 128 + (lane >> 3 & 1) * 64 + (lane >> 4 & 1) * 32 +
                                       (lane & 3) * 8
                                 : lds_addr(&vs[0][lane]);
  auto read_v = [&](VF &dst, uint32_t addr) {
    if constexpr (VROWS) lds_read_vt_async(dst, addr);
    else lds_read4_async(dst, addr);
  };
  // The fragments are there.  VROWS: the operands beside V's halves are kept behind the wait in their place (two halves are
  // one operand: a copy of each otherwise).  Nothing then tells the compiler not to move or copy a half between its read and
  // the wait; tests/test_isa_lds_waits.py looks for that in the built code.
  auto wait_frags = [&](VF &v, u32x4(&k)[4]) {
    if constexpr (VROWS) {
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(k[0]), "+v"(k[1]), "+v"(k[2]), "+v"(k[3]), "+v"(oacc[0][0]), "+v"(oacc[0][1]), "+v"(oacc[1][0]), "+v"(oacc[1][1])
                   :
                   : "memory");
      __builtin_amdgcn_sched_barrier(0);
    } else {
      lds_wait(v, k);
    }
  };
  auto wait_k = [&](u32x4(&k)[4]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(k[0]), "+v"(k[1]), "+v"(k[2]), "+v"(k[3]) : : "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto frag_off = [&](int t) {   // byte offset of tile t's four fragments in a ring array
    return (uint32_t)(((((t >> 1) + base) & (kBStages - 1)) * 8 + (t & 1) * 4) * kFragU4 * 16);
  };
  auto phase_a = [&](int t, const VF &v_prev, VF &v_cur, const u32x4(&k_cur)[4], u32x4(&k_next)[4], int fq = -1) {
    read_v(v_cur, vs_lane + frag_off(t));
    lds_read4_async(k_next, ks_lane + frag_off(t + 1));   // past the last tile: a slot that may be arriving, never used
    if (fq >= 0) fetch1(fq);
    __builtin_amdgcn_sched_barrier(0);
    mma_s(1, k_cur);
    weights(0);
    mma_pv(1, v_prev);
    recipe();
  };
  auto phase_b = [&](VF &v_cur, u32x4(&k_next)[4], int fq = -1) {
    __builtin_amdgcn_sched_barrier(0);
    wait_frags(v_cur, k_next);
    if (fq >= 0) {
      fetch1(fq);
      __builtin_amdgcn_sched_barrier(0);
    }
    mma_s(0, k_next);
    weights(1);
    mma_pv(0, v_cur);
    recipe();
  };
  // One query block: tile t's weights beside the scores of tile t + 1 and the output of tile t - 1; the registers
  // that hold a second query block's scores, weights and fragments hold every other tile's.  The wait is for the reads of the step before.
  auto step = [&](auto first, auto last, auto odd, int t, int fq0 = -1, int fq1 = -1) {
    constexpr int P = decltype(odd)::value;               // t % 2
    __builtin_amdgcn_sched_barrier(0);
    wait_frags(fv[P ^ 1], fk[P ^ 1]);
    read_v(fv[P], vs_lane + frag_off(t));
    if constexpr (!decltype(last)::value) lds_read4_async(fk[P], ks_lane + frag_off(t + 2));
    if (fq0 >= 0) fetch1(fq0);
    if (fq1 >= 0) fetch1(fq1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!decltype(last)::value) mma_s_of(0, P ^ 1, fk[P ^ 1]);
    weights_of(0, P);
    if constexpr (!decltype(first)::value) mma_pv_of(0, P ^ 1, fv[P ^ 1]);
    if constexpr (!decltype(first)::value && !decltype(last)::value) recipe();
  };
  // outside the loop: the row sums are taken where they stand (else the additions are moved to the
  // end of the block and the weights that wait for them to scratch)
  auto pin = [&]() { asm volatile("" : "+v"(lrow[0][0]), "+v"(lrow[0][1]), "+v"(lrow[1][0]), "+v"(lrow[1][1])); };
  // this wave's part of the stage after the next has landed (all but the newest fetches); after the barrier all of it
  auto publish = [&](auto newest) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(newest)::value) : "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  // The next block's number is asked for as late as the answer can be waited for, so that who is ahead takes it.
  // (At a block's first stage where the last round fills no more than half of the slots, in the hope that its blocks then
  // go to one workgroup per CU: level with this at best where every XCD has its own counter, and now and then, behind a
  // kernel that leaves the slots in another order, two to a CU after all: blocks of E4M3 layers, 12,000 tokens, 900 or 960 us, late
  // 900.  Where all XCDs share a counter they went to those that it answered first: 12 heads, one launch per block, early,
  // late, us: 16,384 tokens (1.5 rounds) 710 883 701, 35,384 (3.3) 3312 3530 3192; 16 heads, 16,384 (2) 936 972 920.)
  bool more = true;
  auto turn = [&]() {      // the workgroup's next block (or none: this one's stages again, into slots nobody reads)
    int nb;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(nb) : "v"(lds_addr(&next_block)) : "memory");
    nb = __builtin_amdgcn_readfirstlane(nb);
    more = nb < in_list;
    if (more) blk = nb;
    place(blk);
  };

  // Of a CU's two workgroups the hardware lets the older one issue first.  One that takes block after block would stay the
  // older one, be ahead for good and leave its partner alone with most of a block at the end.  So a workgroup gives way
  // with each block it takes, as a new workgroup would to the one beside it.  Not up to two rounds where the last one fills no
  // more than half of the slots, which the workgroups that are ahead take one per CU, nor with long blocks there (2 to 4 %
  // the other way).  One launch per block, without, with, us: 16 heads, 20 frames of 760 tokens (1.9 rounds) 74.6 82.7 74.1,
  // 17 of 1600 (3.7) 220 230 215, 12 heads, 15 of 28 x 37 83.2 90.9 81.2.
  const int rounds = (in_list - 1) / slots, last_round = in_list - rounds * slots;   // full rounds, blocks of the last one
  const bool give_way = rounds >= 2 || (last_round * 2 > slots && nkv <= kGiveWayStages);
  int taken_blocks = 0;
  auto take_turn = [&]() {
    switch (taken_blocks++ & 3) {
      case 0: __builtin_amdgcn_s_setprio(3); break;
      case 1: __builtin_amdgcn_s_setprio(2); break;
      case 2: __builtin_amdgcn_s_setprio(1); break;
      default: __builtin_amdgcn_s_setprio(0);
    }
  };

  place(blk);
  fetch(0);
  fetch(1);
  load_q();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  while (true) {
    if (give_way) take_turn();
    const bool one_sub = narrow();
    const int64_t q0 = (int64_t)qb * kBQB + wave * (one_sub ? kQW / 2 : kQW);
    const int seq = sh / heads, head = sh - seq * heads;
    uint16_t *const ob = o + (size_t)seq * n * C;
    const uint16_t *const rb = RES ? res + (size_t)seq * n * C : nullptr;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      float ss = (sumsq8(qraw[sub][0]) + sumsq8(qraw[sub][1])) + (sumsq8(qraw[sub][2]) + sumsq8(qraw[sub][3]));
      ss += __shfl_xor(ss, 32, 64);
      const float r = qk_norm ? c / sqrtf(ss * (1.0f / 64.0f) + kQkEps) : c;
#pragma unroll
      for (int s = 0; s < 4; ++s) qf[sub][s] = __builtin_bit_cast(bf16x8, scale8(qraw[sub][s], r));
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) oacc[sub][dt] = zero;
      lrow[sub][0] = lrow[sub][1] = 0.f;
    }
    // stages 0 and 1 were requested ahead of q (and the last block's stores, eight at most, after it):
    // this wave's parts have landed; after the barrier all of them, and nobody reads the last block's any more
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    fetch(2);
    // lanes l and l + 32 trade halves: lane l then has channels 0-7, lane l + 32 channels 8-15 of 16
    auto store = [&](int sub, const u32x4(&rs)[4]) {
      float l = lrow[sub][0] + lrow[sub][1];
      l += __shfl_xor(l, 32, 64);
      const int64_t row = q0 + sub * 32 + ql;
      const bool live = row < n;
      const float inv = PACKED && !live ? 0.f : 1.0f / l;
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
          float r[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) r[i] = PACKED && !live ? 0.f : oacc[sub][dt][8 * gp + i] * inv;
          if constexpr (RES) {   // out = res + attention, one rounding: halves traded the other way first
            const u32x4 x = rs[dt * 2 + gp];
            const auto a = __builtin_amdgcn_permlane32_swap(x.x, x.z, false, false);
            const auto b = __builtin_amdgcn_permlane32_swap(x.y, x.w, false, false);
            r[0] += bf16_lo(a[0]);
            r[1] += bf16_hi(a[0]);
            r[2] += bf16_lo(b[0]);
            r[3] += bf16_hi(b[0]);
            r[4] += bf16_lo(a[1]);
            r[5] += bf16_hi(a[1]);
            r[6] += bf16_lo(b[1]);
            r[7] += bf16_hi(b[1]);
          }
          const auto s0 = __builtin_amdgcn_permlane32_swap(pack_bf16(r[0], r[1]), pack_bf16(r[4], r[5]), false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(pack_bf16(r[2], r[3]), pack_bf16(r[6], r[7]), false, false);
          const u32x4 w = u32x4{s0[0], s1[0], s0[1], s1[1]};
          if constexpr (PACKED)
            ((u32x4 *)o)[((size_t)((q0 + sub * 32) >> 5) * (C >> 4) + head * 4 + dt * 2 + gp) * 64 + lane] = w;
          else if (live)
            *(u32x4 *)(ob + (size_t)row * C + head * 64 + 32 * dt + 16 * gp + 8 * h) = w;
        }
    };
    auto load_res = [&](int sub, u32x4(&rs)[4]) {
      const int64_t row = min(q0 + sub * 32 + ql, n - 1);
#pragma unroll
      for (int i = 0; i < 4; ++i) rs[i] = *(const u32x4 *)(rb + (size_t)row * C + head * 64 + 16 * i + 8 * h);
    };
    using Yes = std::true_type;
    using No = std::false_type;
    if (q0 >= n) {
      // no queries: the wave only moves its share of the stages
      for (int i = 0; i < nkv - 3; ++i) {
        at_stage(i + 3, i + 3);
        fetch1(0);
        fetch1(1);
        fetch1(2);
        publish(std::integral_constant<int, 3>{});
        fetch1(3);
      }
      publish(std::integral_constant<int, 0>{});
      turn();
      for (int i = 0; i < 2; ++i) {
        at_stage(i, nkv + i);
        fetch1(0);
        fetch1(1);
        fetch1(2);
        fetch1(3);
      }
      load_q();
    } else if (one_sub) {
      lds_read4_async(fk[0], ks_lane + frag_off(0));
      wait_k(fk[0]);
      lds_read4_async(fk[1], ks_lane + frag_off(1));
      mma_s_of(0, 0, fk[0]);
      step(Yes{}, No{}, No{}, 0);
      pin();
      uint32_t taken = 0u;
#pragma unroll 1
      for (int i = 0; i < nkv - 3; ++i) {
        if (i == nkv - kStreamStages && tid == 0)
          taken = __hip_atomic_fetch_add(ctr + list * 8, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int st = i + 3;
        asm volatile("" : "+s"(st));
        at_stage(st, st);
        step(No{}, No{}, Yes{}, 2 * i + 1, 0, 1);
        fetch1(2);
        wait_frags(fv[1], fk[1]);
        publish(std::integral_constant<int, 3>{});
        step(No{}, No{}, No{}, 2 * i + 2, 3);
      }
      if (tid == 0) next_block = slots + (int)taken;
      step(No{}, No{}, Yes{}, nkt - 5);
      pin();
      wait_frags(fv[1], fk[1]);
      publish(std::integral_constant<int, 0>{});
      turn();                                               // from here on the next block's stages 0 and 1 are fetched
      at_stage(0, nkv);
      step(No{}, No{}, No{}, nkt - 4, 0, 1);
      pin();
      step(No{}, No{}, Yes{}, nkt - 3, 2, 3);
      pin();
      if (n_last + 4 * h < kKV) mask_tail(0, 0);
      at_stage(1, nkv + 1);
      step(No{}, No{}, No{}, nkt - 2, 0, 1);
      pin();
      if (n_last + 4 * h < kKV) mask_tail(1, 1);
      step(No{}, Yes{}, Yes{}, nkt - 1, 2, 3);
      pin();
      wait_frags(fv[1], fk[1]);
      u32x4 rw[4];
      if constexpr (RES) load_res(0, rw);
      load_q();
      __builtin_amdgcn_sched_barrier(0);
      mma_pv_of(0, 1, fv[1]);
      store(0, rw);
    } else {
      lds_read4_async(fk[0], ks_lane + frag_off(0));
      read_v(fv[0], vs_lane + frag_off(0));
      wait_frags(fv[0], fk[0]);
      lds_read4_async(fk[1], ks_lane + frag_off(1));
      mma_s(0, fk[0]);
      weights(0);
      mma_s(1, fk[0]);
      pin();
      uint32_t taken = 0u;
#pragma unroll 1
      for (int i = 0; i < nkv - 3; ++i) {
        if (i == nkv - kStreamStages && tid == 0)
          taken = __hip_atomic_fetch_add(ctr + list * 8, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int st = i + 3;
        asm volatile("" : "+s"(st));   // (addresses from the stage number, not carried along: the recipe counts their arithmetic)
        at_stage(st, st);
        phase_b(fv[0], fk[1], 0);                           // B(2i)
        phase_a(2 * i + 1, fv[0], fv[1], fk[1], fk[0], 1);  // A(2i+1)
        phase_b(fv[1], fk[0], 2);                           // B(2i+1)
        publish(std::integral_constant<int, 3>{});
        phase_a(2 * i + 2, fv[1], fv[0], fk[0], fk[1], 3);  // A(2i+2)
      }
      if (tid == 0) next_block = slots + (int)taken;        // (wave 0 always has queries)
      phase_b(fv[0], fk[1]);                                // stage nkv - 3: nothing of this block is left to fetch
      pin();
      phase_a(nkt - 5, fv[0], fv[1], fk[1], fk[0]);
      pin();
      phase_b(fv[1], fk[0]);
      pin();
      publish(std::integral_constant<int, 0>{});
      phase_a(nkt - 4, fv[1], fv[0], fk[0], fk[1]);
      pin();
      wait_frags(fv[0], fk[1]);
      turn();                                               // from here on the next block's stages 0 and 1 are fetched
      at_stage(0, nkv);
      phase_b(fv[0], fk[1], 0);
      pin();
      phase_a(nkt - 3, fv[0], fv[1], fk[1], fk[0], 1);
      pin();
      phase_b(fv[1], fk[0], 2);
      pin();
      if (n_last + 4 * h < kKV) mask_tail(0, 0);
      phase_a(nkt - 2, fv[1], fv[0], fk[0], fk[1], 3);
      pin();
      if (n_last + 4 * h < kKV) mask_tail(0, 1);
      at_stage(1, nkv + 1);
      phase_b(fv[0], fk[1], 0);
      fetch1(1);
      pin();
      if (n_last + 4 * h < kKV) mask_tail(1, 0);
      phase_a(nkt - 1, fv[0], fv[1], fk[1], fk[0], 2);
      fetch1(3);
      pin();
      if (n_last + 4 * h < kKV) mask_tail(1, 1);
      wait_frags(fv[1], fk[0]);
      weights(1);
      pin();
      // this block's residual rows and the next block's q rows, in the registers of the fragments and scores
      __builtin_amdgcn_sched_barrier(0);
      u32x4 rw[2][4];
      if constexpr (RES) {
        load_res(0, rw[0]);
        load_res(1, rw[1]);
      }
      load_q();
      __builtin_amdgcn_sched_barrier(0);
      mma_pv(0, fv[1]);
      mma_pv(1, fv[1]);
      store(0, rw[0]);
      store(1, rw[1]);
    }
    base = (base + nkv) & (kBStages - 1);
    if (!more) break;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may land after the workgroup ends
}

// ---------------------------------------------------------------------------------------
// Short sequences.  Blocks of 256 queries are few (394 tokens of 4 heads: 8) and each walks all keys
// alone.  Here a workgroup has 64 queries and its four waves take a quarter of the keys each, every
// wave as in the main kernel (two 32-query blocks half a step apart, the same weights and references);
// a wave's K and V fragments come straight from L2 into its registers, a whole tile ahead of their
// use: no wave reads what another one does, so there is no ring, and no barrier before the end.  There
// the partial sums meet in LDS: wave w adds up quarter w of the output (query block w / 2, channels
// 32 (w % 2) .. + 31) in pairs and stores it.  Bound by latency: kernel start, one round trip for
// q, K and V each, a few tiles per wave (394 tokens of 4 heads, the call with its K/V re-layout, 14.1 ->
// 9.8 us).  Eight waves with an eighth of the keys each gave nothing (9.8 -> 10.7; 4000 tokens 28.1 -> 28.5).
// attn_is_short says where it is used.
// ---------------------------------------------------------------------------------------
constexpr int kShortWaves = 4;   // (sum4 below)
// ROWS: K and V are not re-laid out before.  A wave normalises the keys of its tiles itself, as k_attn_pack does, and V's rows pass
// through its own 4 KB of LDS per tile, read transposed; both are asked for two tiles ahead.  That takes a launch away and
// pays with every block's own normalisation of all keys, so it is for few blocks per sequence, with the re-layout and without, us:
// 394 tokens of 16 heads 11.8 and 9.7, 700 12.9 and 11.9, 800 of 8 heads 12.1 and 12.3, 1,500 of 16 23.3 and 25.9; 25 frames of 15 x 17, 4
// heads, 21.1 and 13.0, 6 of 16 x 16, 16 heads, 16.4 and 13.0, 2 of 37 x 37, 8 heads, 22.7 and 25.0.  (Its two
// arguments stand last: in front they push others out of the first 64 bytes, and every form waits 0.2 us longer.)
constexpr int kRowsBlocks = 12;  // 64-query blocks of a sequence, at most
template <bool ONLINE, bool PACKED, bool ROWS>
__global__ __launch_bounds__(64 * kShortWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_attn_bf16_short(
    const uint16_t *q, const u32x4 *__restrict__ kp, const u32x4 *__restrict__ vp, uint16_t *o,
    const uint16_t *res, int64_t n, int heads, int n_seq, int n_kt, int nqs, float c, int qk_norm,
    uint32_t *__restrict__ redo, int redo_stride, const uint16_t *krows, const uint16_t *vrows) {
  constexpr int WAVES = kShortWaves, R = 64 / WAVES;   // of a lane's 64 output registers (query block, channels 32 dt .., row) a
                                             // wave adds up and stores R
  // [wave][whose registers, its own left out][group of 4][lane]; ROWS: V's rows before
  __shared__ __attribute__((aligned(kVRowBytes))) f32x4 part[WAVES][WAVES - 1][R / 4 * 64];
  static_assert(__alignof__(part) % kVRowBytes == 0 && sizeof(part[0]) % kVRowBytes == 0, "lds_read_vt_async");
  __shared__ f32x2 psum[WAVES][64];          // row sums of the two query blocks
  __shared__ float pref[WAVES];              // ONLINE: the waves' references
  __shared__ int any_low;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ql = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C = heads * 64;
  int sh, qs;   // (sequence, head) pair and 64-query block; each XCD gets whole pairs
  if (((heads * n_seq) & 7) == 0) {
    const int hp = (heads * n_seq) >> 3, xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    sh = xcd * hp + local / nqs;
    qs = local % nqs;
  } else {
    sh = blockIdx.x / nqs;
    qs = blockIdx.x % nqs;
  }
  const int seq = sh / heads, head = sh - seq * heads;
  q += (size_t)seq * n * C;
  o += (size_t)seq * n * C;
  if (res) res += (size_t)seq * n * C;
  const int64_t q0 = (int64_t)qs * kQW;
  const int nt = (int)((n + kKT - 1) / kKT);                       // tiles with keys in them
  // a wave takes whole steps of its loop, two tiles; of four tiles or fewer one at most (33 to 64 tokens, one
  // launch of 256-query blocks 6.9 us, both tiles by one wave 7.2, like this 7.0)
  const int unit = nt <= WAVES ? 1 : 2;
  const int64_t units = (nt + unit - 1) / unit;
  const int t0 = min(nt, unit * (int)(units * wave / WAVES)), t1 = min(nt, unit * (int)(units * (wave + 1) / WAVES));
  const u32x4 *kh = kp + (size_t)sh * n_kt * 4 * kFragU4 + lane;
  const u32x4 *vh = vp + (size_t)sh * n_kt * 4 * kFragU4 + lane;
  auto load = [&](const u32x4 *from, int t, u32x4(&dst)[4]) {      // past the wave's last tile: that one again
    const u32x4 *p = from + (size_t)min(t, t1 - 1) * 4 * kFragU4;
#pragma unroll
    for (int f = 0; f < 4; ++f) dst[f] = p[f * kFragU4];
  };
  // ROWS: a lane's 64 bytes of its key's row; V's 32 rows into one of three places in what will hold this wave's sums, in
  // k_attn_bf16_stream's order there (rows beyond the sequence as zeros)
  const uint16_t *const krow = ROWS ? krows + (size_t)seq * n * C + head * 64 + 8 * h : nullptr;
  auto load_k = [&](int t, u32x4(&dst)[4]) {
    if constexpr (ROWS) {
      const uint16_t *p = krow + (size_t)min((int64_t)min(t, t1 - 1) * kKT + ql, n - 1) * C;
#pragma unroll
      for (int f = 0; f < 4; ++f) dst[f] = *(const u32x4 *)(p + 16 * f);
    } else {
      load(kh, t, dst);
    }
  };
  __amdgpu_buffer_rsrc_t vb;
  if constexpr (ROWS)
    vb = __builtin_amdgcn_make_buffer_rsrc((void *)(vrows + (size_t)seq * n * C + head * 64), 0, (int)((n - 1) * C * 2 + 128), 0x00020000);
  const int v_off = ROWS ? (lane >> 3) * C * 2 + ((lane & 7) ^ (lane >> 4 & 1) * 4) * 16 : 0;
  auto fetch_v = [&](int t) {              // (ahead of the same tile of K: once that is there, so is this)
    if (t < t1)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(vb, (u32x4 *)part[wave] + (t % 3) * 256 + i * 64, 16, v_off + (4 * t + i) * 16 * C, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
  };
  const uint32_t v_lane = ROWS ? lds_addr(&part[wave]) + (4 * h + (lane >> 2 & 3)) * 128 + (lane >> 3 & 1) * 64 + (lane >> 4 & 1) * 32 +
                                     (lane & 3) * 8
                               : 0u;
  u32x2 vt[8];
  auto read_v = [&](int t) {
    __builtin_amdgcn_sched_barrier(0);
    lds_read_vt_async(vt, v_lane + (t % 3) * 4096);
  };
  auto wait_v = [&](u32x4(&v)[4]) {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(vt[0]), "+v"(vt[1]), "+v"(vt[2]), "+v"(vt[3]), "+v"(vt[4]), "+v"(vt[5]), "+v"(vt[6]), "+v"(vt[7])
                 :
                 : "memory");
#pragma unroll
    for (int f = 0; f < 4; ++f) v[f] = u32x4{vt[2 * f].x, vt[2 * f].y, vt[2 * f + 1].x, vt[2 * f + 1].y};
  };
  auto norm_k = [&](u32x4(&k)[4]) {        // k_attn_pack's values: chunks of 8 channels, added in pairs
    if constexpr (ROWS) {
      float pair_sum[4];
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        const float cs = sumsq8(k[f]);
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(cs), __float_as_uint(cs), false, false);
        pair_sum[f] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
      }
      const float r = 1.0f / sqrtf(((pair_sum[0] + pair_sum[1]) + (pair_sum[2] + pair_sum[3])) * (1.0f / 64.0f) + kQkEps);
#pragma unroll
      for (int f = 0; f < 4; ++f) k[f] = scale8(k[f], r);
    }
  };
  u32x4 fv[2][4], fk[2][4];            // [tile & 1]
  bf16x8 qf[2][4];
  f32x16 oacc[2][2], sacc[2], s_start;
  float lrow[2][2] = {{0.f, 0.f}, {0.f, 0.f}}, lnew[2] = {0.f, 0.f}, ref_run = ONLINE ? -INFINITY : 0.f;
  bool over = false;
  u32x4 pb[2][2];
#pragma unroll
  for (int sub = 0; sub < 2; ++sub)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[sub][dt][r] = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) s_start[r] = 0.f;
  if (ONLINE && tid == 0) any_low = 0;

  auto mma_s = [&](int sub, const u32x4(&kf)[4]) {
    f32x16 acc = s_start;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[s]), qf[sub][s], acc, 0, 0, 0);
    sacc[sub] = acc;
  };
  auto mma_pv = [&](int sub, const u32x4(&vf)[4]) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
        oacc[sub][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vf[u * 2 + dt]),
                                                                __builtin_bit_cast(bf16x8, pb[sub][u]), oacc[sub][dt], 0, 0, 0);
  };
  auto mask_tail = [&](int t, int sub) {   // keys beyond the sequence end
    const int left = (int)(n - (int64_t)t * kKT) - 4 * h;
    if (left + 4 * h < kKT) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if ((r >> 2) * 8 + (r & 3) >= left) sacc[sub][r] = -INFINITY;
    }
  };
  auto weights = [&](int sub) {
    float l0 = lrow[sub][0], l1 = lrow[sub][1];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p0 = __builtin_amdgcn_exp2f(sacc[sub][8 * u + 2 * e]);
        const float p1 = __builtin_amdgcn_exp2f(sacc[sub][8 * u + 2 * e + 1]);
        w[e] = pack_bf16(p0, p1);
        l0 += p0;
        l1 += p1;
      }
      pb[sub][u] = u32x4{w[0], w[1], w[2], w[3]};
    }
    lnew[0] = l0;
    lnew[1] = l1;
  };
  // ONLINE: accept the new row sums, or raise the reference first (settle() of the main kernel)
  auto settle = [&](int sub) {
    if (ONLINE && __builtin_amdgcn_ballot_w64(!(lnew[0] + lnew[1] <= kSumRaise)) != 0) {
      float mx = sacc[sub][0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sacc[sub][r]);
      const float delta = fmaxf(wave_max(mx), 0.f);
      const float alpha = __builtin_amdgcn_exp2f(-delta);
      ref_run += delta;
      over |= !(ref_run <= kRefUseful);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        lrow[b][0] *= alpha;
        lrow[b][1] *= alpha;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[b][dt][r] *= alpha;
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[b][r] -= delta;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) s_start[r] = -ref_run;
      weights(sub);
    }
    lrow[sub][0] = lnew[0];
    lrow[sub][1] = lnew[1];
  };

  if (t0 < t1) {
    if constexpr (ROWS) fetch_v(t0);
    load_k(t0, fk[0]);
    if constexpr (ROWS) fetch_v(t0 + 1);
    else load(vh, t0, fv[0]);
    load_k(t0 + 1, fk[1]);
    __builtin_amdgcn_sched_barrier(0);
    // both blocks' q rows at once, but for the plain form behind a re-layout, which takes them one after the other sooner
    // (1,130 tokens of 8 heads 13.1 us at once, 12.9)
    constexpr bool kQAtOnce = ROWS || ONLINE || PACKED;
    u32x4 qw[2][4];
    auto load_q = [&](int sub) {
      const int64_t row = min(q0 + sub * 32 + ql, n - 1);
      const uint16_t *qp = q + (size_t)row * C + head * 64 + 8 * h;
#pragma unroll
      for (int s = 0; s < 4; ++s) qw[sub][s] = *(const u32x4 *)(qp + 16 * s);
    };
    if constexpr (kQAtOnce) {
      load_q(0);
      load_q(1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {      // q as in the main kernel
      if constexpr (!kQAtOnce) load_q(sub);
      const u32x4(&w)[4] = qw[sub];
      float ss = (sumsq8(w[0]) + sumsq8(w[1])) + (sumsq8(w[2]) + sumsq8(w[3]));
      ss += __shfl_xor(ss, 32, 64);
      const float r = qk_norm ? c / sqrtf(ss * (1.0f / 64.0f) + kQkEps) : c;
#pragma unroll
      for (int s = 0; s < 4; ++s) qf[sub][s] = __builtin_bit_cast(bf16x8, scale8(w[s], r));
    }
    norm_k(fk[0]);
    mma_s(0, fk[0]);
    mma_s(1, fk[0]);
    mask_tail(t0, 0);
    mask_tail(t0, 1);
    if (ONLINE) {
      float mx = fmaxf(sacc[0][0], sacc[1][0]);
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, fmaxf(sacc[0][r], sacc[1][r]));
      ref_run = wave_max(mx);
      over = !(ref_run <= kRefUseful);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s_start[r] = -ref_run;
        sacc[0][r] -= ref_run;
        sacc[1][r] -= ref_run;
      }
    }
    weights(0);
    lrow[0][0] = lnew[0];
    lrow[0][1] = lnew[1];
    // B(t): weights of block 1, tile t || PV(t) and scores(t + 1) of block 0;  A(t + 1): weights of block 0,
    // tile t + 1 || PV(t) and scores(t + 1) of block 1.  V(t + 1) and K(t + 2) are requested ahead of both.
    auto tile = [&](int t, u32x4(&v)[4], u32x4(&v2)[4], u32x4(&k1)[4], u32x4(&k2)[4]) {
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (ROWS) {
        read_v(t);                             // (K(t) has been used)
        fetch_v(t + 2);
      } else {
        load(vh, t + 1, v2);
      }
      load_k(t + 2, k2);
      __builtin_amdgcn_sched_barrier(0);
      weights(1);
      if constexpr (ROWS) wait_v(v);
      mma_pv(0, v);
      norm_k(k1);
      mma_s(0, k1);
      mask_tail(t + 1, 0);
      settle(1);
      weights(0);
      mma_pv(1, v);
      mma_s(1, k1);
      mask_tail(t + 1, 1);
      settle(0);
    };
    int t = t0;
    for (; t + 2 < t1; t += 2) {
      tile(t, fv[0], fv[1], fk[1], fk[0]);
      tile(t + 1, fv[1], fv[0], fk[0], fk[1]);
    }
    if (t + 1 < t1) {
      tile(t, fv[0], fv[1], fk[1], fk[0]);
      ++t;
#pragma unroll
      for (int f = 0; f < 4; ++f) fv[0][f] = fv[1][f];
    }
    if constexpr (ROWS) read_v(t);
    weights(1);                              // the last tile
    if constexpr (ROWS) wait_v(fv[0]);
    mma_pv(0, fv[0]);
    settle(1);
    mma_pv(1, fv[0]);
  }

  // ---- the four waves' sums meet
  float lsub[2];
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const float l = lrow[sub][0] + lrow[sub][1];
    lsub[sub] = l + __shfl_xor(l, 32, 64);
  }
#pragma unroll
  for (int w = 0; w < WAVES; ++w)
    if (w != wave) {
      f32x4 *dst = part[wave][w < wave ? w : w - 1] + lane;
#pragma unroll
      for (int g = 0; g < R / 4; ++g) {
        const int at = w * R + 4 * g;
        const f32x16 &a = oacc[at >> 5][(at >> 4) & 1];
        dst[g * 64] = f32x4{a[at & 15], a[(at & 15) + 1], a[(at & 15) + 2], a[(at & 15) + 3]};
      }
    }
  psum[wave][lane] = f32x2{lsub[0], lsub[1]};
  if (ONLINE && lane == 0) pref[wave] = over ? __builtin_nanf("") : ref_run;
  __syncthreads();
  float scale[WAVES];
  bool low = false;
  if (ONLINE) {
    float top = -INFINITY;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      low |= pref[w] != pref[w];             // a reference that does not serve
      top = fmaxf(top, pref[w]);
    }
#pragma unroll
    for (int w = 0; w < WAVES; ++w) scale[w] = __builtin_amdgcn_exp2f(pref[w] - top);
  }
  const int sub = wave * R >> 5, dt = (wave * R >> 4) & 1, r0 = wave * R & 15;
  const int64_t row = q0 + sub * 32 + ql;
  const bool live = row < n;
  float own[R], l = 0.f;
#pragma unroll
  for (int w = 0; w < WAVES; ++w)            // (wave is uniform: one copy runs)
    if (w == wave)
#pragma unroll
      for (int r = 0; r < R; ++r) own[r] = oacc[(w * R + r) >> 5][((w * R + r) >> 4) & 1][(w * R + r) & 15];
  float acc[R], lw[WAVES];
  auto sum4 = [&](const float (&x)[WAVES]) {   // neighbours first, whoever adds
    return ONLINE ? (x[0] * scale[0] + x[1] * scale[1]) + (x[2] * scale[2] + x[3] * scale[3]) : (x[0] + x[1]) + (x[2] + x[3]);
  };
#pragma unroll
  for (int w = 0; w < WAVES; ++w) lw[w] = psum[w][lane][sub];
  l = sum4(lw);
#pragma unroll
  for (int g = 0; g < R / 4; ++g) {
    f32x4 v[WAVES];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) v[w] = part[w][w == wave ? 0 : wave < w ? wave : wave - 1][g * 64 + lane];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float x[WAVES];
#pragma unroll
      for (int w = 0; w < WAVES; ++w) x[w] = w == wave ? own[4 * g + i] : v[w][i];
      acc[4 * g + i] = sum4(x);
    }
  }
  if (ONLINE) {                              // as in the main kernel: rows lost to underflow go to the second pass
    low |= live && !(l >= 8.67e-19f);        // 2^-60
    if (__builtin_amdgcn_ballot_w64(low) != 0 && lane == 0) any_low = 1;
    __syncthreads();
    if (any_low != 0) {
      if (tid == 0) redo[(size_t)sh * redo_stride + (q0 / kBQB)] = 1u;
      return;
    }
  }
  const float inv = live ? 1.0f / l : 0.f;
  if constexpr (PACKED) {
    u32x4 *op = (u32x4 *)o + ((size_t)((q0 + sub * 32) >> 5) * (C >> 4) + head * 4 + dt * 2 + (r0 >> 3)) * 64 + lane;
#pragma unroll
    for (int gp = 0; gp < R / 8; ++gp) {
      float r[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) r[i] = live ? acc[8 * gp + i] * inv : 0.f;
      const auto s0 = __builtin_amdgcn_permlane32_swap(pack_bf16(r[0], r[1]), pack_bf16(r[4], r[5]), false, false);
      const auto s1 = __builtin_amdgcn_permlane32_swap(pack_bf16(r[2], r[3]), pack_bf16(r[6], r[7]), false, false);
      op[gp * 64] = u32x4{s0[0], s1[0], s0[1], s1[1]};
    }
    return;
  }
  if (live) {
    const size_t at = (size_t)row * C + head * 64 + 32 * dt + 2 * r0 + 4 * h;
#pragma unroll
    for (int g = 0; g < R / 4; ++g) {
      float r[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = acc[4 * g + i] * inv;
      if (res) {   // out = res + attention, one rounding
        const u32x2 x = *(const u32x2 *)(res + at + 8 * g);
        r[0] += bf16_lo(x.x);
        r[1] += bf16_hi(x.x);
        r[2] += bf16_lo(x.y);
        r[3] += bf16_hi(x.y);
      }
      *(u32x2 *)(o + at + 8 * g) = u32x2{pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3])};
    }
  }
}

// ---------------------------------------------------------------------------------------
// FP8 (E4M3, OCP "fn": bias 7, max 448) variant: q, k, v are quantised per tensor with
// scale = amax/448 taken in the same call, the softmax weights with a fixed scale 2^8; the
// MFMAs are v_mfma_f32_32x32x64_f8f6f4, everything else (scores, max, sums, O) stays fp32.
// ---------------------------------------------------------------------------------------
constexpr float kFp8PShift = 8.0f;   // weights are stored as 2^8 * p, p <= 1 at the reference
constexpr float kFp8Raise = 0.75f;   // 2^(8 + 0.75) < 448: the reference follows the maximum closely

// bf16 values of w scaled by r and rounded to bf16 (the normalised q/k as the bf16 path sees them)
__device__ __forceinline__ u32x4 norm8(const u32x4 w, float ss_head, int qk_norm) {
  return qk_norm ? scale8(w, 1.0f / sqrtf(ss_head * (1.0f / 64.0f) + kQkEps)) : w;
}

// part[workgroup] = max |q^|, |k^|, |v| over its share of the call's tensors (q^, k^ normalised when
// qk_norm); k_attn_amax_final reduces them.  One thread per 8-value chunk; the 8 lanes of a (row, head) combine
// their sums of squares.  No atomics: a few thousand workgroups end together and all find the words at 0, and
// how many of them send one varies (15,432 tokens of 16 heads 19-26 us with conditional atomics on three words,
// now 17.5; a call of 600 tokens 28.1 -> 24.1 with the launch that only cleared words gone as well).
__global__ __launch_bounds__(256) void k_attn_amax(const uint16_t *__restrict__ q,
                                                   const uint16_t *__restrict__ k,
                                                   const uint16_t *__restrict__ v, int64_t n, int C,
                                                   int qk_norm, f32x4 *__restrict__ part) {
  __shared__ float red[3][4];
  const int64_t nchunks = n * (C >> 3);
  float mq = 0.f, mk = 0.f, mv = 0.f;
  // the 8 lanes that share a (row, head) hold consecutive chunk indices, so they enter and
  // leave this loop together and the xor-shuffles below only read lanes that are active
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nchunks;
       i += (int64_t)gridDim.x * blockDim.x) {
    const u32x4 wq = ((const u32x4 *)q)[i], wk = ((const u32x4 *)k)[i], wv = ((const u32x4 *)v)[i];
    float sq = sumsq8(wq), sk = sumsq8(wk);
    for (int o = 1; o < 8; o <<= 1) {
      sq += __shfl_xor(sq, o, 64);
      sk += __shfl_xor(sk, o, 64);
    }
    mq = fmaxf(mq, absmax8(norm8(wq, sq, qk_norm)));
    mk = fmaxf(mk, absmax8(norm8(wk, sk, qk_norm)));
    mv = fmaxf(mv, absmax8(wv));
  }
  mq = wave_max(mq);
  mk = wave_max(mk);
  mv = wave_max(mv);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) {
    red[0][wave] = mq;
    red[1][wave] = mk;
    red[2][wave] = mv;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    f32x4 m = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 3; ++t) m[t] = fmaxf(fmaxf(red[t][0], red[t][1]), fmaxf(red[t][2], red[t][3]));
    part[blockIdx.x] = m;
  }
}

// amax[0..2] from the n_part parts
__global__ __launch_bounds__(256) void k_attn_amax_final(const f32x4 *__restrict__ part, int n_part, uint32_t *__restrict__ amax) {
  __shared__ float red[3][4];
  f32x4 m = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int p = threadIdx.x; p < n_part; p += 256) {
    const f32x4 v = part[p];
#pragma unroll
    for (int t = 0; t < 3; ++t) m[t] = fmaxf(m[t], v[t]);
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    m[t] = wave_max(m[t]);
    if (lane == 0) red[t][wave] = m[t];
  }
  __syncthreads();
  if (threadIdx.x < 3)
    amax[threadIdx.x] = __float_as_uint(fmaxf(fmaxf(red[threadIdx.x][0], red[threadIdx.x][1]),
                                              fmaxf(red[threadIdx.x][2], red[threadIdx.x][3])));
}

// fp8 counterpart of k_attn_pack: same fragment-major orders with 8 bytes per lane.
__global__ __launch_bounds__(256) void k_attn_pack_fp8(const uint16_t *__restrict__ k,
                                                       const uint16_t *__restrict__ v, int64_t n,
                                                       int heads, int n_kt, int qk_norm,
                                                       const uint32_t *__restrict__ amax,
                                                       u32x2 *__restrict__ kp, u32x2 *__restrict__ vp) {
  __shared__ __attribute__((aligned(8))) uint8_t vt[kKT][72];
  const int kt = blockIdx.x, head = blockIdx.y, t = threadIdx.x;
  const int C = heads * 64;
  const int key = t >> 3, chunk = t & 7;
  const int64_t row = (int64_t)kt * kKT + key;
  u32x4 wk = {0u, 0u, 0u, 0u}, wv = {0u, 0u, 0u, 0u};
  if (row < n) {
    wk = *(const u32x4 *)(k + (size_t)row * C + head * 64 + chunk * 8);
    wv = *(const u32x4 *)(v + (size_t)row * C + head * 64 + chunk * 8);
  }
  float ss = sumsq8(wk);
  for (int o = 1; o < 8; o <<= 1) ss += __shfl_xor(ss, o, 64);
  wk = norm8(wk, ss, qk_norm);
  const size_t tile = ((size_t)head * n_kt + kt) * 4 * kFragU4;
  kp[tile + (chunk >> 1) * kFragU4 + (chunk & 1) * 32 + key] = quant8(wk, fp8_scale_inv(amax[1]));
  *(u32x2 *)&vt[key][chunk * 8] = quant8(wv, fp8_scale_inv(amax[2]));
  __syncthreads();
  const int u = t >> 7, dt = (t >> 6) & 1, lane = t & 63, h = lane >> 5, dr = lane & 31;
  uint32_t w[2] = {0u, 0u};
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k0 = 16 * u + 8 * (e >> 2) + 4 * h + (e & 3);
    w[e >> 2] |= (uint32_t)vt[k0][32 * dt + dr] << (8 * (e & 3));
  }
  vp[tile + (u * 2 + dt) * kFragU4 + lane] = u32x2{w[0], w[1]};
}

// four 8-byte operand pieces side by side: the 32-byte operand of v_mfma_f32_32x32x64_f8f6f4
__device__ __forceinline__ i32x8 cat_fp8(u32x2 a, u32x2 b, u32x2 c, u32x2 d) {
  return i32x8{(int)a.x, (int)a.y, (int)b.x, (int)b.y, (int)c.x, (int)c.y, (int)d.x, (int)d.y};
}

// Where the output of the E4M3 kernels goes: rows, or a linear layer's activation operand (rows beyond the sequence end
// up to whole blocks of 256 zero): in bf16, or as E4M3 codes of the values rounded to bf16 (scale *inv), whose largest
// magnitude is raised in *amax.  The layer's own pass over the rows took 10.6 us at 15,432 tokens of 16 heads.
// (The bounded kernel leaves each wave's magnitude, four per flag, in wave_max: the second pass knows which blocks
// keep their rows and raises theirs.)
enum AttnOut { kOutRows, kOutBf16, kOutE4M3 };
struct AttnOutArgs {
  const uint32_t *inv;
  uint32_t *amax;
  float *wave_max;
};
// 32 queries from row0 on (query lane % 32) x the head's 64 channels, as a lane's accumulators hold them, times the lane's inv;
// returns the largest |value| of a live row
template <AttnOut OUT>
__device__ __forceinline__ float store_head(const f32x16 (&acc)[2], float inv, int64_t row0, int64_t n, int C, int head,
                                            uint16_t *o, float code_inv, int lane) {
  const int h = lane >> 5;
  const int64_t row = row0 + (lane & 31);
  const bool live = row < n;
  float m = 0.f;
  if constexpr (OUT == kOutRows) {
    if (live) {
      uint16_t *op = o + (size_t)row * C + head * 64 + 4 * h;
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const u32x2 w = {pack_bf16(acc[dt][4 * g] * inv, acc[dt][4 * g + 1] * inv),
                           pack_bf16(acc[dt][4 * g + 2] * inv, acc[dt][4 * g + 3] * inv)};
          *(u32x2 *)(op + 32 * dt + 8 * g) = w;
        }
    }
  } else {
    if (row0 >= (n + kBQB - 1) / kBQB * kBQB) return 0.f;   // beyond the operand (uniform)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) {
      uint32_t p[4][2];                // channels 8g + 4h .. + 3 of 32 dt
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        p[g][0] = live ? pack_bf16(acc[dt][4 * g] * inv, acc[dt][4 * g + 1] * inv) : 0u;
        p[g][1] = live ? pack_bf16(acc[dt][4 * g + 2] * inv, acc[dt][4 * g + 3] * inv) : 0u;
      }
      if constexpr (OUT == kOutBf16) {
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
          const auto s0 = __builtin_amdgcn_permlane32_swap(p[2 * gp][0], p[2 * gp + 1][0], false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(p[2 * gp][1], p[2 * gp + 1][1], false, false);
          ((u32x4 *)o)[((size_t)(row0 >> 5) * (C >> 4) + head * 4 + dt * 2 + gp) * 64 + lane] = u32x4{s0[0], s1[0], s0[1], s1[1]};
        }
      } else {
        uint32_t d[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float a = bf16_lo(p[g][0]), b = bf16_hi(p[g][0]), c = bf16_lo(p[g][1]), e = bf16_hi(p[g][1]);
          m = fmaxf(m, fmaxf(fmaxf(fabsf(a), fabsf(b)), fmaxf(fabsf(c), fabsf(e))));
          d[g] = cvt4_fp8(clamp448(a * code_inv), clamp448(b * code_inv), clamp448(c * code_inv), clamp448(e * code_inv));
        }
        const auto s0 = __builtin_amdgcn_permlane32_swap(d[0], d[2], false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(d[1], d[3], false, false);
        ((u32x4 *)o)[((size_t)(row0 >> 5) * (C >> 5) + head * 2 + dt) * 64 + lane] = u32x4{s0[0], s0[1], s1[0], s1[1]};
      }
    }
  }
  return m;
}

// Same structure as k_attn_bf16 (two phase groups, lazily raised reference) on fp8 operands.
// Each contraction is one v_mfma_f32_32x32x64_f8f6f4 (contraction length 64: all channels of a
// head for the scores, all keys of a stage for the output), which runs at twice the rate of the
// 32x32x16 fp8 form; the order of the 64 contraction indices inside an operand is the same for
// both operands (piece p of the packed fragments = indices 16p .. 16p+15 in fragment order).
// SECOND: the pass behind the bounded kernel, over that kernel's packed K and V (k_attn_pack_fp8b).
template <bool SECOND, AttnOut OUT>
__global__ __launch_bounds__(512) void k_attn_fp8(
    const uint16_t *__restrict__ q, const u32x2 *__restrict__ kp, const u32x2 *__restrict__ vp,
    uint16_t *__restrict__ o, int64_t n, int heads, int n_kt, int nqb, float c_in, int qk_norm,
    const uint32_t *__restrict__ amax, const uint32_t *__restrict__ redo, AttnOutArgs oa) {
  __shared__ u32x2 ks[kKSlots][8 * kFragU4];
  __shared__ u32x2 vs[kVSlots][8 * kFragU4];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ql = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2;
  const int C = heads * 64;
  int head, qb;
  if ((heads & 7) == 0) {
    const int hp = heads >> 3, xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    head = xcd * hp + local / nqb;
    qb = local % nqb;
  } else {
    head = blockIdx.x / nqb;
    qb = blockIdx.x % nqb;
  }
  // second pass behind the bounded kernel: only the query blocks it has flagged (one flag per
  // 256 queries; the whole workgroup takes the same branch, before any barrier)
  if (SECOND && redo[(size_t)head * (2 * nqb) + 2 * qb] == 0u && redo[(size_t)head * (2 * nqb) + 2 * qb + 1] == 0u) {
    if (OUT == kOutE4M3 && wave == 0) {
      const bool there = lane < kQB / kQW && (int64_t)qb * kQB + lane * kQW < n;   // (the last flag may have no block)
      const float m = wave_max(there ? oa.wave_max[((size_t)head * (2 * nqb) + 2 * qb) * (kBQB / kQW) + lane] : 0.f);
      if (lane == 0) raise_max(oa.amax, m);
    }
    return;
  }
  const int64_t q0 = (int64_t)qb * kQB + wave * kQW;
  const float inv_sq = fp8_scale_inv(amax[0]);
  // scores come out in units of scale_q*scale_k; fold both into the exponent scale
  const float c = c_in * (1.0f / inv_sq) * (1.0f / fp8_scale_inv(amax[1]));
  const float out_scale = 1.0f / fp8_scale_inv(amax[2]);

  i32x8 qf8[2];
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const int64_t row = min(q0 + sub * 32 + ql, n - 1);
    const uint16_t *qp = q + (size_t)row * C + head * 64 + 8 * h;
    u32x4 w[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) w[s] = *(const u32x4 *)(qp + 16 * s);
    float ss = (sumsq8(w[0]) + sumsq8(w[1])) + (sumsq8(w[2]) + sumsq8(w[3]));
    ss += __shfl_xor(ss, 32, 64);
    u32x2 q8[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) q8[s] = quant8(norm8(w[s], ss, qk_norm), inv_sq);
    qf8[sub] = cat_fp8(q8[0], q8[1], q8[2], q8[3]);
  }

  f32x16 oacc[2][2];
#pragma unroll
  for (int sub = 0; sub < 2; ++sub)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[sub][dt][r] = 0.f;
  float mref[2] = {-INFINITY, -INFINITY}, lrow[2] = {0.f, 0.f};

  const int nkv = n_kt >> 1;
  const u32x2 *kh = kp + (size_t)head * n_kt * 4 * kFragU4;
  const u32x2 *vh = vp + (size_t)head * n_kt * 4 * kFragU4;
  u32x2 rk, rv;
  // SECOND: where the piece that lies at tid in LDS, fragment (kt2, s) of K, (kt2, u, dt) of V, is in 16-byte pieces
  const int kt2_ = wave >> 2, k_at = SECOND ? ((kt2_ * 2 + ((wave >> 1) & 1)) * 64 + lane) * 2 + (wave & 1) : tid;
  const int v_at = SECOND ? (((wave & 1) * 2 + kt2_) * 64 + lane) * 2 + ((wave >> 1) & 1) : tid;
  auto g2r = [&](int j) {
    const size_t off = (size_t)j * 8 * kFragU4;
    rk = kh[off + k_at];
    rv = vh[off + v_at];
  };
  auto r2s = [&](int j) {
    ks[j % kKSlots][tid] = rk;
    vs[j % kVSlots][tid] = rv;
  };

  f32x16 sacc[2][2];
  u32x2 pb[2][2][2];

  auto phase_m = [&](int j) {
    __builtin_amdgcn_sched_barrier(0);
    if (j > 0) {
      const u32x2 *vt = &vs[(j - 1) % kVSlots][lane];
      u32x2 vf[8];
#pragma unroll
      for (int f = 0; f < 8; ++f) vf[f] = vt[f * kFragU4];
      // one MFMA per (query block, d tile) over all 64 keys: the operands are the four 16-key
      // pieces (kt2, u) side by side, in the same order for V and for the weights
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) {
        const i32x8 a = cat_fp8(vf[0 * 2 + dt], vf[1 * 2 + dt], vf[2 * 2 + dt], vf[3 * 2 + dt]);
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
          oacc[sub][dt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
              a, cat_fp8(pb[sub][0][0], pb[sub][0][1], pb[sub][1][0], pb[sub][1][1]), oacc[sub][dt], 0, 0, 0,
              0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (j < nkv) {
      const u32x2 *kt = &ks[j % kKSlots][lane];
      u32x2 kf[8];
#pragma unroll
      for (int f = 0; f < 8; ++f) kf[f] = kt[f * kFragU4];
      // one MFMA per (key tile, query block) over all 64 channels: the four k-step pieces side by side
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2) {
        const i32x8 a = cat_fp8(kf[kt2 * 4], kf[kt2 * 4 + 1], kf[kt2 * 4 + 2], kf[kt2 * 4 + 3]);
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
          sacc[kt2][sub] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, qf8[sub], zero, 0, 0, 0, 0, 0, 0);
      }
    }
    asm volatile("" : "+v"(sacc[0][0]), "+v"(sacc[0][1]), "+v"(sacc[1][0]), "+v"(sacc[1][1]),
                 "+v"(oacc[0][0]), "+v"(oacc[0][1]), "+v"(oacc[1][0]), "+v"(oacc[1][1]));
    __builtin_amdgcn_sched_barrier(0);
  };
  auto phase_v = [&](int j) {
    __builtin_amdgcn_sched_barrier(0);
    if (j == nkv - 1) {
      const int64_t kbase = (int64_t)j * kKV;
      if (kbase + kKV > n) {
#pragma unroll
        for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int64_t key = kbase + kt2 * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
            if (key >= n) {
              sacc[kt2][0][r] = -INFINITY;
              sacc[kt2][1][r] = -INFINITY;
            }
          }
      }
    }
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      float mx = -INFINITY;
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
        for (int r = 0; r < 16; r += 2) mx = max3(mx, sacc[kt2][sub][r], sacc[kt2][sub][r + 1]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      if (__builtin_amdgcn_ballot_w64((mx - mref[sub]) * c > kFp8Raise) != 0) {
        const float mnew = fmaxf(mref[sub], mx);
        const float alpha = __builtin_amdgcn_exp2f((mref[sub] - mnew) * c);
        mref[sub] = mnew;
        lrow[sub] *= alpha;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[sub][dt][r] *= alpha;
      }
      float ls = lrow[sub];
      // exp2(c (s - mref) + shift).  As one fma on c * mref - shift while that product is small
      // enough to be exact to 2^-10 (this kernel is bound by its VALU instructions); beyond that
      // (scores of any size come in here) the difference is taken first.
      const float mc = mref[sub] * c - kFp8PShift;
      if (__builtin_amdgcn_ballot_w64(!(fabsf(mc) < 16384.0f)) == 0) {
#pragma unroll
        for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            float pv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              pv[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kt2][sub][8 * u + e], c, -mc));
              ls += pv[e];   // row sum of the fp32 weights, before the cast
            }
            pb[sub][kt2][u] = u32x2{cvt4_fp8(pv[0], pv[1], pv[2], pv[3]), cvt4_fp8(pv[4], pv[5], pv[6], pv[7])};
          }
      } else {
#pragma unroll
        for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            float pv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              pv[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kt2][sub][8 * u + e] - mref[sub], c, kFp8PShift));
              ls += pv[e];
            }
            pb[sub][kt2][u] = u32x2{cvt4_fp8(pv[0], pv[1], pv[2], pv[3]), cvt4_fp8(pv[4], pv[5], pv[6], pv[7])};
          }
      }
      lrow[sub] = ls;
    }
    asm volatile("" : "+v"(pb[0][0][0]), "+v"(pb[0][0][1]), "+v"(pb[0][1][0]), "+v"(pb[0][1][1]),
                 "+v"(pb[1][0][0]), "+v"(pb[1][0][1]), "+v"(pb[1][1][0]), "+v"(pb[1][1][1]),
                 "+v"(lrow[0]), "+v"(lrow[1]));
    __builtin_amdgcn_sched_barrier(0);
  };

  g2r(0);
  r2s(0);
  __syncthreads();
  if (grp == 0) {
    for (int j = 0; j < nkv; ++j) {
      if (j + 1 < nkv) g2r(j + 1);
      phase_m(j);
      __syncthreads();
      if (j + 1 < nkv) r2s(j + 1);
      phase_v(j);
      __syncthreads();
    }
    phase_m(nkv);
    __syncthreads();
    __syncthreads();
  } else {
    if (nkv > 1) g2r(1);
    __syncthreads();
    if (nkv > 1) r2s(1);
    phase_m(0);
    __syncthreads();
    for (int j = 1; j < nkv; ++j) {
      if (j + 1 < nkv) g2r(j + 1);
      phase_v(j - 1);
      __syncthreads();
      if (j + 1 < nkv) r2s(j + 1);
      phase_m(j);
      __syncthreads();
    }
    phase_v(nkv - 1);
    __syncthreads();
    phase_m(nkv);
    __syncthreads();
  }

  const float code_inv = OUT == kOutE4M3 ? __uint_as_float(*oa.inv) : 1.0f;
  float m = 0.f;
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const float l = lrow[sub] + __shfl_xor(lrow[sub], 32, 64);
    m = fmaxf(m, store_head<OUT>(oacc[sub], out_scale / l, q0 + sub * 32, n, C, head, o, code_inv, lane));
  }
  if constexpr (OUT == kOutE4M3) {
    m = wave_max(m);
    if (lane == 0) raise_max(oa.amax, m);
  }
}

// ---------------------------------------------------------------------------------------
// Bounded-score FP8 kernel (qk_norm).  With unit-RMS heads a score cannot exceed
// B = 73 * softmax_scale (Cauchy-Schwarz, with room for the bf16 and E4M3 roundings of the
// normalised rows), so the weights are exponentiated against the fixed reference B: stored weight =
// 2^(score - B) * 2^8.75 <= 430, no running maximum, no rescaling, no branches.  E4M3 keeps 3
// mantissa bits down to 2^-6 and flushes below 2^-10, so a row is served well when the scores
// that carry its mass are within ~15 binades of B.  The sum L of a row's stored weights
// tells: rows with L < 1 (the total mass of the row sits more than 8.75 binades below the bound,
// where single weights lose precision and nothing averages the loss out) are flagged per 256-
// query block, and k_attn_fp8 (running maximum) recomputes the flagged blocks afterwards.  With
// q = k (the layer driver) every row has the weight 2^8.75 of its own key and nothing is flagged.
//
// Structure as k_attn_bf16_main with a 64-key stage in place of a 32-key tile (the FP8 MFMA
// contracts 64 keys at once): a wave owns two 32-query blocks half a stage apart,
//   A(t): weights of block 0, stage t   ||  PV of block 1, stage t-1;  scores of block 1, stage t
//   B(t): weights of block 1, stage t   ||  PV of block 0, stage t;    scores of block 0, stage t+1
// Bound by the issue of the loop: per stage and SIMD 128 exp2 and 64 packs of 9 cycles each, and every FP8 MFMA takes
// about 30 cycles from a VALU that runs beside it (a loop of 16 exp2 and 8 packs alone 172 ns, 2 MFMAs alone 113, both
// 227).  Scores of both blocks alive, MFMAs spread among the VALU part, row sums in half an MFMA, packs into stale
// registers, against MFMAs at the ends of a phase, one block's scores alive, a whole MFMA per row sum, 16 heads:
// 1,500 tokens 35.0 -> 31.0 us, 5,776 129 -> 115, 15,432 588 -> 521, 143,232 42.9 -> 38.3 ms; the same bits.
// K and V are packed so that an MFMA operand is two 16-byte pieces per lane:
//   K piece (stage, kt2, j): lane (h*32+key) holds channels 32j+8h .. +8 and 32j+16+8h .. +8 of
//                            key 64 stage + 32 kt2 + key
//   V piece (stage, dt, kt2): lane (h*32+dr) holds column 32dt+dr of the 16 keys of tile
//                            2 stage + kt2 that the lane's accumulator rows map to (u = 0, 1)
// ---------------------------------------------------------------------------------------
constexpr int kF8Stages = 8;          // LDS ring of 64-key stages (4 KB of K, 4 KB of V each)
constexpr int kF8Ahead = 5;           // stages fetched ahead
constexpr float kF8Bound = 73.0f;     // |q.k| <= 64 (1 + 2^-8)^2 (1 + 2^-4)^2 < 73: unit-RMS rows rounded to bf16,
                                      // then to E4M3 (every element at most 2^-4 off, all in the same direction)
constexpr float kF8Top = 8.75f;       // a weight at the bound is stored as 2^8.75

__global__ __launch_bounds__(256) void k_attn_pack_fp8b(const uint16_t *__restrict__ k,
                                                        const uint16_t *__restrict__ v, int64_t n,
                                                        int heads, int n_kt,
                                                        const uint32_t *__restrict__ amax,
                                                        u32x2 *__restrict__ kp, u32x2 *__restrict__ vp,
                                                        uint32_t *__restrict__ flags) {
  __shared__ __attribute__((aligned(8))) uint8_t vt[kKT][72];
  const int kt = blockIdx.x, head = blockIdx.y, t = threadIdx.x;
  const int C = heads * 64;
  const int key = t >> 3, chunk = t & 7;
  const int64_t row = (int64_t)kt * kKT + key;
  // two flags per 512 tokens, fewer than key tiles.  (From n: one argument more would take the others past 64 bytes, 0.2 us.)
  const int n_flags = 2 * (int)((n + kQB - 1) / kQB);
  if (t == 0 && kt < n_flags) flags[(size_t)head * n_flags + kt] = 0u;
  u32x4 wk = {0u, 0u, 0u, 0u}, wv = {0u, 0u, 0u, 0u};
  if (row < n) {
    wk = *(const u32x4 *)(k + (size_t)row * C + head * 64 + chunk * 8);
    wv = *(const u32x4 *)(v + (size_t)row * C + head * 64 + chunk * 8);
  }
  float ss = sumsq8(wk);
  for (int o = 1; o < 8; o <<= 1) ss += __shfl_xor(ss, o, 64);
  wk = norm8(wk, ss, 1);
  const int stage = kt >> 1, kt2 = kt & 1;
  const size_t base = ((size_t)head * (n_kt >> 1) + stage) * 4 * 64;   // in 16-byte pieces
  const int s = chunk >> 1, hh = chunk & 1;
  kp[2 * (base + (size_t)(kt2 * 2 + (s >> 1)) * 64 + hh * 32 + key) + (s & 1)] = quant8(wk, fp8_scale_inv(amax[1]));
  *(u32x2 *)&vt[key][chunk * 8] = quant8(wv, fp8_scale_inv(amax[2]));
  __syncthreads();
  const int u = t >> 7, dt = (t >> 6) & 1, lane = t & 63, h = lane >> 5, dr = lane & 31;
  uint32_t w[2] = {0u, 0u};
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k0 = 16 * u + 8 * (e >> 2) + 4 * h + (e & 3);
    w[e >> 2] |= (uint32_t)vt[k0][32 * dt + dr] << (8 * (e & 3));
  }
  vp[2 * (base + (size_t)(dt * 2 + kt2) * 64 + lane) + u] = u32x2{w[0], w[1]};
}

template <AttnOut OUT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_attn_fp8_bounded(
    const uint16_t *__restrict__ q, const u32x4 *__restrict__ kp, const u32x4 *__restrict__ vp,
    uint16_t *__restrict__ o, int64_t n, int heads, int nkv, int nqb, float c_in,
    const uint32_t *__restrict__ amax, uint32_t *__restrict__ redo, int redo_stride, AttnOutArgs oa) {
  __shared__ u32x4 ks[kF8Stages][4 * 64];
  __shared__ u32x4 vs[kF8Stages][4 * 64];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ql = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C = heads * 64;
  int head, qb;
  if ((heads & 7) == 0) {
    const int hp = heads >> 3, xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    head = xcd * hp + local / nqb;
    qb = local % nqb;
  } else {
    head = blockIdx.x / nqb;
    qb = blockIdx.x % nqb;
  }
  const int64_t q0 = (int64_t)qb * kBQB + wave * kQW;
  // The score MFMA delivers log2-domain scores minus the reference directly: its accumulator
  // starts at -ref, and the factor between a product of codes and a log2-domain score, c / (scale
  // of q * scale of k), is made a power of two 2^e by quantising q with a scale up to 2x smaller
  // than 448 / amax (same relative precision, floating point); 2^e is the MFMA's block scale.
  const float inv_sk = fp8_scale_inv(amax[1]);
  const float e_f = fminf(fmaxf(ceilf(log2f(c_in / (fp8_scale_inv(amax[0]) * inv_sk))), -100.f), 100.f);
  const float inv_sq = c_in / (inv_sk * exp2f(e_f));
  const int scale_k = 127 + (int)e_f;       // E8M0: 2^(scale_k - 127), applied to the K operand
  const float ref = kF8Bound * c_in - kF8Top;
  const float out_scale = 1.0f / fp8_scale_inv(amax[2]);

  i32x8 qf8[2];
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const int64_t row = min(q0 + sub * 32 + ql, n - 1);
    const uint16_t *qp = q + (size_t)row * C + head * 64 + 8 * h;
    u32x4 w[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) w[s] = *(const u32x4 *)(qp + 16 * s);
    float ss = (sumsq8(w[0]) + sumsq8(w[1])) + (sumsq8(w[2]) + sumsq8(w[3]));
    ss += __shfl_xor(ss, 32, 64);
    u32x2 q8[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) q8[s] = quant8(norm8(w[s], ss, 1), inv_sq);
    qf8[sub] = cat_fp8(q8[0], q8[1], q8[2], q8[3]);
  }

  f32x16 oacc[2][2];
#pragma unroll
  for (int sub = 0; sub < 2; ++sub)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[sub][dt][r] = 0.f;
  // Row sums come from the matrix pipe as well: a fragment of ones (E4M3 1.0 = 0x38) against the weights sums
  // the E4M3 weights of the lane's query.  The normaliser is then the sum of exactly the weights that
  // multiply V: with a fixed reference the largest weight of a row is not a power of two (as it is relative to a
  // running maximum) and carries up to 3 % rounding error, which cancels in this ratio and would not against
  // the fp32 sum.  The 16x16x128 form does it in half the cycles of another 32x32x64 and in 4 registers: fed with the
  // operand of that form, its column c and k chunk of 32 are lane 16 * chunk + c, so even chunks hold query c and odd ones
  // query c + 16.  Ones in the even chunks of even rows and in the odd chunks of odd rows keep them apart.
  f32x4 lacc[2];
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) lacc[sub] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int one = ((lane ^ (lane >> 4)) & 1) ? 0 : 0x38383838;
  const i32x8 ones8 = {one, one, one, one, one, one, one, one};
  const float nr = -ref;
  const f32x16 kStart = {nr, nr, nr, nr, nr, nr, nr, nr, nr, nr, nr, nr, nr, nr, nr, nr};

  const u32x4 *kh = kp + (size_t)head * nkv * 4 * 64;
  const u32x4 *vh = vp + (size_t)head * nkv * 4 * 64;
  // one stage = 256 pieces of K and 256 of V: one direct-to-LDS load of each per thread
  // (stage `src` goes to the ring slot of stage `as`: past the end the last stage is fetched
  // again, into a slot nobody reads, so that the loop body has no branches)
  auto fetch = [&](int as) {
    const int src = min(as, nkv - 1);
    __builtin_amdgcn_global_load_lds(kh + (size_t)src * 256 + tid, &ks[as & (kF8Stages - 1)][wave * 64], 16, 0, 0);
    __builtin_amdgcn_global_load_lds(vh + (size_t)src * 256 + tid, &vs[as & (kF8Stages - 1)][wave * 64], 16, 0, 0);
  };

  f32x16 sacc[2][2];   // [query block][32-key half]: scores
  i32x8 pb[2] = {};    // [query block]: E4M3 weights of its current stage
  u32x4 fv[4], fk[4];  // the pieces of one stage of V and of K

  auto mma_s = [&](int sub, int kt2) {
    sacc[sub][kt2] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(cat8(fk[2 * kt2], fk[2 * kt2 + 1]), qf8[sub],
                                                                     kStart, 0, 0, 0, scale_k, 0, 127);
  };
  auto mma_pv = [&](int sub, int dt) {
    oacc[sub][dt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(cat8(fv[2 * dt], fv[2 * dt + 1]), pb[sub],
                                                                    oacc[sub][dt], 0, 0, 0, 0, 0, 0);
  };
  auto mma_l = [&](int sub) {
    lacc[sub] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(ones8, pb[sub], lacc[sub], 0, 0, 0, 0, 0, 0);
  };
  auto mask_tail = [&](int t, int sub) {   // keys beyond the sequence end
    if ((int64_t)(t + 1) * kKV > n) {
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int64_t key = (int64_t)t * kKV + kt2 * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
          if (key >= n) sacc[sub][kt2][r] = -INFINITY;
        }
    }
  };
  // a quarter of a stage's weights of one block: exp2 against the fixed reference, E4M3 pack
  auto weights = [&](int sub, int i) {
    float pv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) pv[e] = __builtin_amdgcn_exp2f(sacc[sub][i >> 1][8 * (i & 1) + e]);
    // (into the stale codes, not into a cleared register: all four bytes are written, and clearing took 16 moves per stage)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int w = __builtin_amdgcn_cvt_pk_fp8_f32(pv[4 * j], pv[4 * j + 1], pb[sub][i * 2 + j], false);
      pb[sub][i * 2 + j] = __builtin_amdgcn_cvt_pk_fp8_f32(pv[4 * j + 2], pv[4 * j + 3], w, true);
    }
  };
  // Fragment reads but the newest `newer` are there.  `with`: the other operands of the MFMAs that need them, which keep
  // those behind this wait (the fragments themselves in their place would cost a copy of each: two form one operand).  A
  // fragment that the compiler moved or copied ahead of it would be lost: tests/test_isa_lds_waits.py reads the built code for that.
  auto wait_frags = [&](i32x8(&with)[2], auto newer) {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(with[0]), "+v"(with[1]) : "n"(decltype(newer)::value) : "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  using None = std::integral_constant<int, 0>;
  using Four = std::integral_constant<int, 4>;
  // A phase turns one block's scores into weights (32 exp2 and 16 packs, 8 cycles each: the longer pipe) while the
  // matrix pipe works on the other block: the weights' product with V and their sum, and that block's next
  // scores (4 x 64 + 32 cycles).  A MFMA stands between any two quarters of the VALU part, so that a wave waits for none of its
  // own; the scores of both blocks are alive.  Fragments are read by hand, V(t+1) and K(t+2) in A(t+1) once the
  // MFMAs that had their registers are issued, and waited for in B(t+1).
  const uint32_t ks_lane = lds_addr(&ks[0][lane]), vs_lane = lds_addr(&vs[0][lane]);
  auto slot_off = [&](int t) { return (uint32_t)((t & (kF8Stages - 1)) * 4 * 64 * 16); };
#define LV_PIN() __builtin_amdgcn_sched_barrier(0)
  // B(t): PV(t) and scores(t+1) of block 0; weights of block 1 (stage t)
  auto phase_b = [&](int t, bool last) {
    LV_PIN();
    wait_frags(pb, Four{});
    mma_pv(0, 0);
    LV_PIN();
    weights(1, 0);
    LV_PIN();
    mma_pv(0, 1);
    LV_PIN();
    weights(1, 1);
    LV_PIN();
    wait_frags(qf8, None{});
    mma_s(0, 0);
    LV_PIN();
    weights(1, 2);
    LV_PIN();
    mma_s(0, 1);
    LV_PIN();
    weights(1, 3);
    LV_PIN();
    mma_l(0);
    if (last) mask_tail(t + 1, 0);
  };
  // A(t): PV(t-1) and scores(t) of block 1; weights of block 0 (stage t); reads V(t) and K(t+1)
  auto phase_a = [&](int t, bool last) {
    LV_PIN();
    mma_pv(1, 0);
    LV_PIN();
    weights(0, 0);
    LV_PIN();
    mma_pv(1, 1);
    LV_PIN();
    lds_read4_async(fv, vs_lane + slot_off(t));
    LV_PIN();
    weights(0, 1);
    LV_PIN();
    mma_s(1, 0);
    LV_PIN();
    weights(0, 2);
    LV_PIN();
    mma_s(1, 1);
    LV_PIN();
    lds_read4_async(fk, ks_lane + slot_off(t + 1));   // past the end: a slot that may be arriving, never used
    LV_PIN();
    weights(0, 3);
    LV_PIN();
    mma_l(1);
    if (last) mask_tail(t, 1);
  };

  // stages 0 and 1 complete and the next ones in flight before the loop; iteration t fetches stage t + kF8Ahead
  // into a slot that nobody has read since stage t + kF8Ahead - kF8Stages
#pragma unroll
  for (int i = 0; i < kF8Ahead; ++i) fetch(i);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * (kF8Ahead - 2)) : "memory");
  __builtin_amdgcn_s_barrier();
  // A(0) without a PV
  LV_PIN();
  lds_read4_async(fk, ks_lane);
  lds_read4_async(fv, vs_lane);
  wait_frags(qf8, Four{});
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    mma_s(sub, 0);
    mma_s(sub, 1);
    if (nkv == 1) mask_tail(0, sub);
  }
  LV_PIN();
  lds_read4_async(fk, ks_lane + slot_off(1));
  LV_PIN();
#pragma unroll
  for (int i = 0; i < 4; ++i) weights(0, i);
  // steady state: B(t), A(t+1) for t <= nkv-3: the stages they read (t+1, t+2) are complete ones
  for (int t = 0; t < nkv - 2; ++t) {
    // this wave's parts of stage t+2 have landed (the newest loads may be in flight); after the barrier all of
    // stage t+2 is readable
    LV_PIN();
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * (kF8Ahead - 3)) : "memory");
    __builtin_amdgcn_s_barrier();
    LV_PIN();
    fetch(t + kF8Ahead);
    phase_b(t, false);
    phase_a(t + 1, false);
  }
  if (nkv >= 2) {                                         // enters the last stage, which may be ragged
    phase_b(nkv - 2, true);
    phase_a(nkv - 1, true);
  }
  // B(nkv-1) without scores of a next stage, and the last PV of block 1
  LV_PIN();
  wait_frags(pb, None{});
  asm volatile("" ::"v"(fk[0]), "v"(fk[1]), "v"(fk[2]), "v"(fk[3]));   // (the last K read ends before its registers do)
#pragma unroll
  for (int i = 0; i < 4; ++i) weights(1, i);
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    mma_pv(sub, 0);
    mma_pv(sub, 1);
    mma_l(sub);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // nothing may land after the workgroup ends
#undef LV_PIN

  const float code_inv = OUT == kOutE4M3 ? __uint_as_float(*oa.inv) : 1.0f;
  bool low = false;
  float m = 0.f;
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const float l = (lane & 16) ? lacc[sub][1] : lacc[sub][0];
    low |= q0 + sub * 32 + ql < n && !(l >= 1.0f);
    m = fmaxf(m, store_head<OUT>(oacc[sub], out_scale / l, q0 + sub * 32, n, C, head, o, code_inv, lane));
  }
  const size_t at = (size_t)head * redo_stride + qb;
  if (__builtin_amdgcn_ballot_w64(low) != 0 && lane == 0) atomicOr(&redo[at], 1u);
  if constexpr (OUT == kOutE4M3) {
    m = wave_max(m);
    if (lane == 0) oa.wave_max[at * (kBQB / kQW) + wave] = m;
  }
}

static int n_key_tiles(int64_t n) { return (int)(2 * ((n + kKV - 1) / kKV)); }

// flags of the bounded FP8 kernel: one word per (head, 256-query block), rows padded to two per
// 512-query block of the second pass
static size_t fp8_flag_words(int heads, int64_t n) { return (size_t)heads * 2 * ((n + kQB - 1) / kQB); }

// Whether and how (see AttnCut): b blocks for kSlots slots per XCD; a slot without a first piece takes
// k = ceil(b / idle slots) second pieces, each with a start of its own (about 6 stages of 64 keys).
// A stage takes about 1 us with one workgroup per CU and 1.55 with two, and a cut about 9 us in all.
// (Sequences whose 64-query blocks all fit, attn_is_short, do not come here.)
// Measured with 16 heads, whole against cut: 1500 tokens 26 -> 22 us, 4500 111 -> 100, 5776 149 -> 137,
// 3500 57.4 -> 56.  With a full round before them, blocks do not end together and the last round's
// idle slots are not there to be had (15432 tokens 866 -> 876 us, 20000 1356 -> 1364): not cut.  Nor
// are the blocks of many sequences.
// The bounded kernel (no running reference) takes 0.87 us per stage where a quarter of the CUs or more idle,
// and sharing CUs then costs more than the cut gives: 8 heads, whole against cut, 4500 tokens 65.0 and
// 67.1 us, 5000 72.3 and 74.7, 6000 86.6 and 87.0, from 6500 on 96.2 and 94.8 (the online kernel gains 8 %
// there).  Scratch is asked for as if by the online kernel, which is cut wherever the bounded one is.
static AttnCut attn_cut(int heads, int64_t n, bool bounded = false) {
  const int64_t nqb = (n + kBQB - 1) / kBQB, nkv = (n + kKV - 1) / kKV, b = heads / kXcd * nqb;
  if (heads % kXcd != 0 || b >= kSlots) return {0, 0};
  const int64_t idle = kSlots - b, k = (b + idle - 1) / idle;
  const int64_t small = (nkv - 6 * (k - 1)) / (k + 1);
  if (small < 6) return {0, 0};
  const auto stage_us = [](int64_t per_xcd) { return per_xcd <= kSlots / 2 ? 1.0 : 1.55; };
  const int64_t chain = k * (small + 6) - 6, longest = nkv - small > chain ? nkv - small : chain;
  const double alone = bounded && b <= kSlots * 3 / 8 && 2 * b > kSlots / 2 ? 0.87 : 1.0;
  const double whole = (double)nkv * stage_us(b) * alone, cut = (double)longest * stage_us(2 * b) + 9.0;
  if (cut > 0.97 * whole) return {0, 0};
  return {(int)b, (int)small};
}
static size_t cut_bytes(int heads, int64_t n, int n_seq) {
  const AttnCut c = n_seq == 1 ? attn_cut(heads, n) : AttnCut{0, 0};
  return c.n_cut ? kSyncWords * sizeof(uint32_t) + align_up((size_t)kXcd * c.n_cut * kPieceFloats * sizeof(float), 256) : 0;
}

// Whether the blocks of 64 queries (k_attn_bf16_short) are used: as long as all of them are on the chip at once,
// two per CU.  One call, otherwise against this way, us: 16 heads with q, k normalised 394 tokens 14.6 and
// 10.9, 700 18.3 and 11.8, 1024 (256 blocks) 22.1 and 13.5, 2000 (512) 32.8 and 28.3, 2500 (640) 45.3 and
// 43.5, 4000 (1008) 73.2 and 83.6; 4 heads, which are never cut, 4000 tokens 59.6 and 28.2, 8190 (512) 107.5 and 76.9, 9000 119 and
// 112; 2 frames of 37 x 37 of 8 heads (352) 30.0 and 20.8.  The online kernel's steady loop is the slower one here
// (its references are registers the loop would need): where its blocks can be cut, only up to one
// per CU (8 heads: 2000 tokens 31.5 and 26.1, 3000 39.4 and 39.6, 4000 48.9 and 51.0).  A block that it leaves to
// the second pass has sisters that are stored by then: not where o may be q, from which that pass starts again (a
// residual may be added in place).
static bool attn_is_short(int64_t blocks, bool bounded, bool can_be_cut, bool in_place, int n_cu) {
  if (!bounded && in_place) return false;
  return blocks <= (bounded || !can_be_cut ? 2 * n_cu : n_cu);
}

size_t attn_ws_bytes(int heads, int64_t n_tokens, int attn_dtype, int n_seq, bool least) {
  const size_t elem = attn_dtype == LV_ATTN_FP8_E4M3 ? sizeof(u32x2) : sizeof(u32x4);
  const size_t per = (size_t)heads * n_seq * n_key_tiles(n_tokens) * 4 * kFragU4 * elem;
  // [amax block][K fragments][V fragments]; FP8: the first pair is the running-maximum kernel's (with qk_norm the
  // workgroups' maxima lie there until K is written, or a block's, of its attention's output), the second the bounded
  // kernel's and its second pass', then the flags.  No call uses K and V of both pairs; they stay apart because callers
  // have sized their scratch by this.
  size_t total = 256 + 2 * align_up(per, 256);
  if (attn_dtype == LV_ATTN_FP8_E4M3) total += 2 * align_up(per, 256) + align_up(fp8_flag_words(heads, n_tokens) * 4, 256);
  // bf16: the flags of the online-softmax pass (one word per 256-query block)
  else total += align_up(fp8_flag_words(heads * n_seq, n_tokens) * 4, 256) + (least ? 0 : cut_bytes(heads, n_tokens, n_seq));
  return total;
}

namespace {
// Where a call's parts lie in its scratch.
struct AttnPlan {
  bool bounded, is_short = false, stream = false;
  AttnCut cut = {0, 0};
  size_t per, words;
  int n_kt, nqb, nqb2, nqs, n_cu = 0;
  uint32_t *head;           // 64 words: E4M3 the amaxes, else the counters of a stream's blocks
  char *frag;
  uint32_t *redo, *sync;
  float *partial;
};
}  // namespace

static int attn_plan(AttnPlan &a, int64_t n, int heads, float scale, int attn_dtype, int qk_norm, const void *q, const void *o,
                     void *ws, size_t ws_bytes, int n_seq, const void *res) {
  if (n_seq < 1 || (int64_t)heads * n_seq > 65535) return LV_ERR_SHAPE;
  if ((n_seq > 1 || res) && attn_dtype != LV_ATTN_BF16) return LV_ERR_DTYPE;
  if (attn_dtype != LV_ATTN_BF16 && attn_dtype != LV_ATTN_FP8_E4M3) return LV_ERR_DTYPE;
  const float c = scale * 1.4426950408889634f;
  const bool f8 = attn_dtype == LV_ATTN_FP8_E4M3;
  a.n_kt = n_key_tiles(n);
  a.nqb = (int)((n + kQB - 1) / kQB);
  a.nqb2 = (int)((n + kBQB - 1) / kBQB);
  a.nqs = (int)((n + kQW - 1) / kQW);
  a.head = (uint32_t *)ws;
  a.frag = (char *)ws + 256;
  a.per = align_up((size_t)heads * n_seq * a.n_kt * 4 * kFragU4 * (f8 ? sizeof(u32x2) : sizeof(u32x4)), 256);
  a.words = fp8_flag_words(heads * n_seq, n);
  a.redo = (uint32_t *)(a.frag + (f8 ? 4 : 2) * a.per);
  a.sync = a.redo + align_up(a.words * 4, 256) / 4;
  a.partial = (float *)(a.sync + kSyncWords);
  // two ways: q, k normalised with exponents that stay in range: the branch-free kernel with
  // no (E4M3: a fixed) reference; otherwise (q, k as given, or a softmax scale beyond that range) the same kernel
  // as online softmax with a per-wave running reference, then the per-row kernel on the query
  // blocks the first pass flagged (normally none: its workgroups return at once)
  a.bounded = qk_norm && (f8 ? kF8Bound : 64.25f) * c <= 64.0f;
  if (f8) return LV_OK;
  int dev = 0;   // (not for E4M3: calls of few tokens are bound by the host, and its answer takes 0.2 us of their 20)
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&a.n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return LV_ERR_HIP;
  a.is_short = attn_is_short((int64_t)a.nqs * heads * n_seq, a.bounded, n_seq == 1 && heads % kXcd == 0, res || o == q, a.n_cu);
  if (!a.is_short && n_seq == 1 && !res && 2 * a.n_cu == kXcd * kSlots && ws_bytes >= attn_ws_bytes(heads, n, attn_dtype))
    a.cut = attn_cut(heads, n, a.bounded);
  // more blocks than slots: workgroups that stay (their rows are written and the residual's read 16 bytes
  // at a time, the main kernel's 8)
  const int64_t n_blocks = (int64_t)a.nqb2 * heads * n_seq;
  a.stream = a.bounded && a.n_kt / 2 >= kStreamStages && a.n_kt / 2 <= kStreamMost && n_blocks > 2 * a.n_cu &&
             n_blocks < ((int64_t)1 << 30) && a.n_cu % 4 == 0 && (((uintptr_t)o | (uintptr_t)res) & 15u) == 0;
  return LV_OK;
}

int attn_kv_target(AttnKV &kv, int64_t n, int heads, float scale, int attn_dtype, int qk_norm, const void *q, const void *o, void *ws,
                   size_t ws_bytes) {
  AttnPlan a;
  if (int rc = attn_plan(a, n, heads, scale, attn_dtype, qk_norm, q, o, ws, ws_bytes, 1, nullptr)) return rc;
  kv = AttnKV{};
  kv.qk_norm = qk_norm;
  kv.clear[0] = a.head;
  kv.n_clear[0] = kStreamWords;
  if (attn_dtype == LV_ATTN_FP8_E4M3) {
    kv.amax = a.head;
    return LV_OK;
  }
  kv.kp = a.frag;
  kv.vp = a.frag + a.per;
  kv.n_kt = a.n_kt;
  kv.clear[1] = a.bounded ? a.sync : a.redo;   // the flags and, behind them, the words that pieces of cut blocks meet at
  kv.n_clear[1] = (a.bounded ? 0 : (int)(a.sync - a.redo)) + (a.cut.n_cut ? kSyncWords : 0);
  return LV_OK;
}

// n_seq independent sequences of n tokens each, stored one after the other (n_seq = 1: the
// global attention over the merged sequence; n_seq = frames: frame attention).  Several
// sequences and the fused residual (o = res + attention, res may be o: a workgroup reads the
// rows it writes and nothing else of them) are supported by the bf16 kernels only.
int launch_attn(const uint16_t *q, const uint16_t *k, const uint16_t *v, uint16_t *o,
                int64_t n, int heads, float scale, int attn_dtype, int qk_norm, void *ws, size_t ws_bytes,
                hipStream_t st, hipEvent_t after_pack, int n_seq, const uint16_t *res,
                AttnOperand *operand, const AttnKV *ready) {
  if (operand && (n_seq != 1 || res)) return LV_ERR_PARAM;
  AttnPlan a;
  if (int rc = attn_plan(a, n, heads, scale, attn_dtype, qk_norm, q, o, ws, ws_bytes, n_seq, res)) return rc;
  const bool bounded = a.bounded, is_short = a.is_short, stream = a.stream;
  const int n_kt = a.n_kt, nqb = a.nqb, nqb2 = a.nqb2, nqs = a.nqs, n_cu = a.n_cu;
  const float c = scale * 1.4426950408889634f;
  const AttnCut cut = a.cut;
  uint32_t *const redo = a.redo;
  if (attn_dtype == LV_ATTN_FP8_E4M3) {
    uint32_t *const amax = a.head;
    u32x2 *kp = (u32x2 *)a.frag, *vp = (u32x2 *)(a.frag + a.per);
    const int C = heads * 64;
    if (!(ready && ready->amax)) {   // (else the layer that produced q, k and v has taken them)
      const int64_t nchunks = n * (C / 8);
      const unsigned ag = (unsigned)(((nchunks + 255) / 256) < 2048 ? ((nchunks + 255) / 256) : 2048);
      f32x4 *const part = (f32x4 *)kp;   // (16 bytes per 2048 of K, gone before K is written)
      hipLaunchKernelGGL(k_attn_amax, dim3(ag), dim3(256), 0, st, q, k, v, n, C, qk_norm, part);
      hipLaunchKernelGGL(k_attn_amax_final, dim3(1), dim3(256), 0, st, (const f32x4 *)part, (int)ag, amax);
    }
    u32x2 *kpb = (u32x2 *)(a.frag + 2 * a.per), *vpb = (u32x2 *)(a.frag + 3 * a.per);
    if (bounded)
      hipLaunchKernelGGL(k_attn_pack_fp8b, dim3((unsigned)n_kt, (unsigned)heads), dim3(256), 0, st, k, v, n,
                         heads, n_kt, amax, kpb, vpb, redo);
    else
      hipLaunchKernelGGL(k_attn_pack_fp8, dim3((unsigned)n_kt, (unsigned)heads), dim3(256), 0, st, k,
                         v, n, heads, n_kt, qk_norm, amax, kp, vp);
    if (after_pack && hipEventRecord(after_pack, st) != hipSuccess) return LV_ERR_HIP;
    auto kernels = [&](auto kind, uint16_t *out) {
      constexpr AttnOut OUT = decltype(kind)::value;
      // (the running-maximum kernel's K, which the bounded one does without, has room for its waves' maxima)
      const AttnOutArgs oa = {operand ? operand->inv : nullptr, operand ? operand->amax : nullptr, (float *)kp};
      if (bounded) {
        // the branch-free kernel against the fixed reference first, then the running-maximum kernel on the query
        // blocks the first one flagged (normally none: its workgroups return at once)
        hipLaunchKernelGGL(k_attn_fp8_bounded<OUT>, dim3((unsigned)(nqb2 * heads)), dim3(256), 0, st, q, (const u32x4 *)kpb,
                           (const u32x4 *)vpb, out, n, heads, n_kt / 2, nqb2, c, amax, redo, 2 * nqb, oa);
        hipLaunchKernelGGL((k_attn_fp8<true, OUT>), dim3((unsigned)(nqb * heads)), dim3(512), 0, st, q, kpb, vpb, out, n,
                           heads, n_kt, nqb, c, qk_norm, amax, (const uint32_t *)redo, oa);
      } else {
        hipLaunchKernelGGL((k_attn_fp8<false, OUT>), dim3((unsigned)(nqb * heads)), dim3(512), 0, st, q, kp, vp, out, n,
                           heads, n_kt, nqb, c, qk_norm, amax, (const uint32_t *)nullptr, oa);
      }
    };
    if (operand) operand->written = true;
    if (!operand) kernels(std::integral_constant<AttnOut, kOutRows>{}, o);
    else if (operand->inv) kernels(std::integral_constant<AttnOut, kOutE4M3>{}, (uint16_t *)operand->at);
    else kernels(std::integral_constant<AttnOut, kOutBf16>{}, (uint16_t *)operand->at);
    LV_HIP_CHECK_LAUNCH();
    return LV_OK;
  }
  u32x4 *kp = (u32x4 *)a.frag, *vp = (u32x4 *)(a.frag + a.per);
  uint32_t *const sync = a.sync, *const ctr = a.head;
  float *const partial = a.partial;
  // K and V as they lie: not where a block's output may take the place of rows that another one still reads
  const size_t bytes = (size_t)n_seq * n * heads * 128;
  const bool kv_ready = ready && ready->kp;
  const auto apart = [&](const void *x) { return (uintptr_t)o >= (uintptr_t)x + bytes || (uintptr_t)x >= (uintptr_t)o + bytes; };
  const bool as_is = !kv_ready && !(operand && !operand->inv) && n * heads * 128 < ((int64_t)1 << 31) && apart(v);
  const bool vrows = stream && n_kt / 2 <= kVRowsStages && as_is;
  const bool rows = is_short && bounded && as_is && apart(k) && nqs <= kRowsBlocks;
  auto pack_kernel = [&](auto has_sync) {
    constexpr bool SYNC = decltype(has_sync)::value;
    uint32_t *const cleared = stream ? ctr : sync;
    const int n_cleared = stream ? kStreamWords : kSyncWords;
    const dim3 grid((unsigned)n_kt, (unsigned)(heads * n_seq));
    if (vrows)
      hipLaunchKernelGGL((k_attn_pack<true, false, false>), grid, dim3(256), 0, st, k, v, n, heads, n_kt, qk_norm, kp, vp, cleared,
                         n_cleared, redo, 0);
    else if (bounded)
      hipLaunchKernelGGL((k_attn_pack<SYNC, false, true>), grid, dim3(256), 0, st, k, v, n, heads, n_kt, qk_norm, kp, vp, cleared,
                         n_cleared, redo, 0);
    else
      hipLaunchKernelGGL((k_attn_pack<SYNC, true, true>), grid, dim3(256), 0, st, k, v, n, heads, n_kt, qk_norm, kp, vp, cleared,
                         n_cleared, redo, 2 * nqb);
  };
  if (kv_ready || rows) {}  // the layer that produced k and v has packed them, and what they clear is cleared
  else if (cut.n_cut || stream) pack_kernel(std::true_type{});
  else pack_kernel(std::false_type{});
  if (after_pack && hipEventRecord(after_pack, st) != hipSuccess) return LV_ERR_HIP;
  auto main_kernel = [&](auto online, auto packed, uint16_t *out) {
    constexpr bool ON = decltype(online)::value, PK = decltype(packed)::value;
    uint32_t *const flags = ON ? redo : nullptr;
    const int stride = ON ? 2 * nqb : 0;
    if (is_short)
      hipLaunchKernelGGL((rows ? k_attn_bf16_short<false, false, true> : k_attn_bf16_short<ON, PK, false>),
                         dim3((unsigned)(nqs * heads * n_seq)), dim3(256), 0, st, q, kp, vp, out, res, n, heads, n_seq, n_kt,
                         nqs, c, qk_norm, flags, stride, k, v);
    else if (!ON && stream)
      hipLaunchKernelGGL((vrows ? res ? k_attn_bf16_stream<false, true, true> : k_attn_bf16_stream<false, false, true>
                                : res ? k_attn_bf16_stream<PK, !PK, false> : k_attn_bf16_stream<PK, false, false>),
                         dim3((unsigned)(2 * n_cu)), dim3(256), 0, st, q, kp, vp, v, out, res, n, heads, n_seq, n_kt, nqb2, c,
                         qk_norm, ctr);
    else if (cut.n_cut)
      hipLaunchKernelGGL((k_attn_bf16_cut<ON, PK>), dim3((unsigned)(kXcd * 2 * cut.n_cut)), dim3(256), 0, st, q, kp, vp, out,
                         n, heads, n_kt, nqb2, c, qk_norm, flags, stride, cut, sync, partial);
    else
      hipLaunchKernelGGL((k_attn_bf16_main<ON, PK>), dim3((unsigned)(nqb2 * heads * n_seq)), dim3(256), 0, st, q, kp, vp, out,
                         res, n, heads, n_seq, n_kt, nqb2, c, qk_norm, flags, stride);
  };
  if (bounded && operand && !operand->inv) {
    main_kernel(std::false_type{}, std::true_type{}, (uint16_t *)operand->at);
    operand->written = true;
  } else if (bounded) {
    main_kernel(std::false_type{}, std::false_type{}, o);
  } else {
    main_kernel(std::true_type{}, std::false_type{}, o);
    hipLaunchKernelGGL(k_attn_bf16, dim3((unsigned)(nqb * heads * n_seq)), dim3(512), 0, st, q, kp,
                       vp, o, res, n, heads, n_seq, n_kt, nqb, c, qk_norm, (const uint32_t *)redo);
  }
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

}  // namespace lv

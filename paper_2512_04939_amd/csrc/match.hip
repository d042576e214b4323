// Cosine matching of src tokens to dst tokens (Sec. 3.4 "Cached Token Merging") and the
// construction of the merge index (CSR groups).
//
// The similarity is a dense contraction dst[n_dst,C] x src[n_src,C]^T that is never
// materialised (see k_match_sim).  bf16 x bf16 products are exact in fp32, only the
// accumulation order differs from an exact dot product; rows whose two best candidates are
// closer than kRescoreGap are re-decided from float64 dot products in a cheap second kernel.
#include "common.h"
#include "internal.h"

namespace lv {

constexpr float kRescoreGap = 2e-4f; // similarity gap below which float64 decides

struct Top2 {
  float v1;
  int i1;
  float v2;
  int i2;
};

// Rows 0..n-1 of x into fragment-major order: fragment (tile t of 32 rows, k-step s of 16
// channels) is 1 KB contiguous, lane (h*32 + r) holds row r, channels 16s+8h .. 16s+8h+7.  Rows
// beyond n are zero.
// A wave writes whole fragments (1 KB stores); it takes 4 consecutive k-steps of its 32 rows,
// so the 128 bytes it needs of a row are one cache line read by 4 back-to-back loads.
// Grid: (row tiles, ceil(KS / 16)); a workgroup's 4 waves take 4 k-steps each.
__global__ __launch_bounds__(256) void k_pack_rows(const uint16_t *__restrict__ x, int n, int C,
                                                   u32x4 *__restrict__ packed) {
  const int KS = C >> 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, r = lane & 31;
  const int t = blockIdx.x, row = t * 32 + r;
  const int s0 = (blockIdx.y * 4 + wave) * 4;
  u32x4 w[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    w[u] = u32x4{0u, 0u, 0u, 0u};
    if (row < n && s0 + u < KS) w[u] = ((const u32x4 *)(x + (size_t)row * C))[(s0 + u) * 2 + h];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (s0 + u < KS) packed[((size_t)t * KS + s0 + u) * 64 + lane] = w[u];
}

// The operands of the similarity kernel: dst rows and src rows gathered into the same order, and
// each row's 1 / max(|x|, 1e-12), the norm accumulated in float64 from the registers that are
// being moved.  Workgroups 0 .. dst_tiles - 1 take 32 dst rows each, the others 32 src rows;
// a wave takes every fourth group of 4 k-steps, all its loads (at most 16, C <= 1024) in flight
// at once.  Bound by HBM: every row is read once and written once.  (One launch instead of a
// norm pass over all tokens and two packs, which read every row twice: 55 -> 29 us at 32 frames
// of 37 x 37 patches, 124 -> 76 us at 100 frames of 28 x 37, C = 1024.)
__global__ __launch_bounds__(256) void k_match_pack(const uint16_t *__restrict__ x,
                                                    const int32_t *__restrict__ dst_idx, int n_dst, int dst_tiles,
                                                    const int32_t *__restrict__ src_idx, int n_src, int C,
                                                    u32x4 *__restrict__ dstp, u32x4 *__restrict__ srcp,
                                                    float *__restrict__ invd, float *__restrict__ invs,
                                                    uint32_t *__restrict__ team_ctr) {
  __shared__ double part[4][32];
  const int KS = C >> 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, r = lane & 31;
  const bool is_dst = (int)blockIdx.x < dst_tiles;
  const int t = is_dst ? blockIdx.x : (int)blockIdx.x - dst_tiles, j = t * 32 + r;
  if (blockIdx.x == 0) team_ctr[threadIdx.x] = 0u;   // the similarity kernel's team counters
  int row = -1;
  if (j < (is_dst ? n_dst : n_src)) row = is_dst ? dst_idx[j] : src_idx[j];
  u32x4 w[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int s0 = (i * 4 + wave) * 4;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      w[i][u] = u32x4{0u, 0u, 0u, 0u};
      if (row >= 0 && s0 + u < KS) w[i][u] = ((const u32x4 *)(x + (size_t)row * C))[(s0 + u) * 2 + h];
    }
  }
  u32x4 *packed = is_dst ? dstp : srcp;
  double ss = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int s0 = (i * 4 + wave) * 4;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s0 + u < KS) {
        const u32x4 v = w[i][u];
        packed[((size_t)t * KS + s0 + u) * 64 + lane] = v;
        const uint32_t b[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double lo = bf16_lo(b[q]), hi = bf16_hi(b[q]);
          ss += lo * lo + hi * hi;
        }
      }
  }
  ss += __shfl_xor(ss, 32, 64);
  if (h == 0) part[wave][r] = ss;
  __syncthreads();
  if (threadIdx.x < 32) {   // row r of the tile; rows beyond the list get NaN: no comparison picks them
    const double n2 = (part[0][r] + part[1][r]) + (part[2][r] + part[3][r]);
    (is_dst ? invd : invs)[j] = row >= 0 ? (float)(1.0 / fmax(sqrt(n2), 1e-12)) : __builtin_nanf("");
  }
}

__device__ __forceinline__ void top2_insert_any(Top2 &t, float v, int i) {
  if (i < 0) return;
  if (v > t.v1 || (v == t.v1 && (t.i1 < 0 || i < t.i1))) {
    t.v2 = t.v1;
    t.i2 = t.i1;
    t.v1 = v;
    t.i1 = i;
  } else if (v > t.v2 || (v == t.v2 && (t.i2 < 0 || i < t.i2))) {
    t.v2 = v;
    t.i2 = i;
  }
}

int launch_pack_rows(const uint16_t *x, int64_t n, int64_t n_pad, int C, void *packed, hipStream_t st) {
  if (n_pad >= ((int64_t)1 << 31) || n_pad % 32 != 0 || C % 16 != 0) return LV_ERR_SHAPE;
  hipLaunchKernelGGL(k_pack_rows, dim3((unsigned)(n_pad / 32), (unsigned)((C / 16 + 15) / 16)), dim3(256), 0, st, x,
                     (int)n, C, (u32x4 *)packed);
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

// The same for an element of a higher row than every one before it: equal values lose.  A NaN
// (rows beyond the list) is never taken.
__device__ __forceinline__ void top2_insert_later(Top2 &t, float v, int i) {
  const bool c1 = v > t.v1, c2 = v > t.v2;
  t.v2 = c1 ? t.v1 : c2 ? v : t.v2;
  t.i2 = c1 ? t.i1 : c2 ? i : t.i2;
  t.v1 = c1 ? v : t.v1;
  t.i1 = c1 ? i : t.i1;
}

// ---------------------------------------------------------------------------------
// Similarity kernel.  A workgroup (8 waves) computes 256 src x 256 dst tiles of the similarity
// matrix with the channel dimension as the inner loop: both operands come pre-packed in
// fragment-major order, go from global memory straight into a 4-stage LDS ring (2 k-steps =
// 32 KB per stage, fetched 3 stages ahead) and are read from there as MFMA fragments, so every
// byte fetched from L2 feeds 128 flop (a src-resident design with streamed dst reaches 64 and
// was bound by the L2 -> CU rate).  Wave (wd, ws) owns the 64 dst x 128 src sub-tile: dst is
// the MFMA row dimension, so a lane owns one src column per 32-column block and folds every
// finished tile into its running (best, second best) pair without cross-lane traffic.
//
// The kernel is persistent: one workgroup per CU.  The workgroups the hardware deals to one
// XCD (block index mod 8) form a team of (src tiles) x (sweeps), 8 x 4 where nothing speaks
// against it; in every full round the team takes its own super-row of src tiles, and in it
// workgroup (src tile, sweep dl) visits the dst tiles dl, dl + n, dl + 2n, ... of n sweeps.  The
// team moves from one dst tile to the next together (a bounded, advisory wait on a counter in the
// XCD's L2), so its workgroups ask for the same src and dst tiles within a few microseconds of
// each other and 4 of 5 requests hit that L2.  The src tiles that do not fill a round of all the
// teams are shared out in a last round over the whole chip, as many sweeps per src tile as there
// are workgroups for it (MatchSched: which shape).  The partial results of a src row, one per
// sweep, are merged by k_match_finish.
// ---------------------------------------------------------------------------------
constexpr int kGTile = 256;          // src and dst rows per workgroup tile
constexpr int kGStages = 4;          // LDS ring depth
constexpr int kGStageU4 = 2 * 2 * 8 * 64;   // u32x4 per stage: [src|dst][2 k-steps][8 fragments][64 lanes]
constexpr int kTeamSpin = 512;       // polls of the team counter before a workgroup goes on alone
constexpr int kInvBufs = 8;          // per-wave LDS buffers of 64 inverse dst norms
constexpr int kTeam = 32;            // workgroups per team: the CUs of an XCD
constexpr int kMaxLists = 64;        // candidate lists of one src row, at most
constexpr int kFewLists = 4;         // ... at least, and at most where the scratch was sized for another sequence:
                                     // many lists come and go with the tile counts, these grow with them

// How the src tiles are dealt out.  Rounds 0 .. n_full - 1: team x takes the sr src tiles from
// (round * 8 + x) * sr on, each with n_sweeps sweeps.  Then the n_rest tiles from `full` on, each
// with rest_sweeps sweeps.  A sweep hands over one list of two candidates per row, or, so that near-equal
// rows are told apart among at least kFewLists lists whatever the shape, one per half or quarter of the
// workgroup's dst rows.  Each list is the two best of its own rows: the fold's bound is shared inside a
// list only (32 frames, two sweeps for most src tiles: 423 -> 427 us against one bound per sweep).
// They lie full_lists * full tiles of rows, list by list, then rest_lists * n_rest.
struct MatchSched {
  int n_sweeps, sr, n_full, rest_sweeps, n_rest, full, full_lists, rest_lists;
};
inline int div_up(int a, int b) { return (a + b - 1) / b; }
static int lists_of(int sweeps) { return sweeps == 1 ? 4 : sweeps < kFewLists ? 2 * sweeps : sweeps; }

// A tile step (256 x 256 rows, all channels) takes the same time on every CU, so the time of a
// shape is its number of steps: rounds * ceil(dst tiles / sweeps).  With 8 x 4 teams alone a last
// round with one super-row in it costs as much as a full one, and a dst tile count that is no
// multiple of 4 idles a part of the team: 32 frames of 37 x 37 patches (150 x 18 tiles) took 15
// steps for 10.5 steps' worth of tiles and 542 us, now 11; 100 frames of 28 x 37 patches under
// the fixed rule (258 x 107) 135 for 107.8 and 4090 us, now 109.  Among shapes of nearly equal
// step counts the one that asks its L2 for the fewest distinct tiles wins: 8 x 4 and 4 x 8 ask
// for 12, and at 1000 frames 8 x 4 was 1 % faster than 16 x 2 and 3 % faster than 4 x 8.
static MatchSched match_sched(int src_tiles, int dst_tiles, int team, int max_lists = kMaxLists) {
  MatchSched best = {1, 1, 0, 1, 0, 0, 4, 4};
  double best_cost = 1e300;
  for (int l = 1; l <= team && l <= dst_tiles; ++l) {
    if (lists_of(l) > max_lists) continue;
    const int sr = team / l, per_round = sr * kXcd;
    const double share = 1.0 + 0.04 * ((sr + l) / 12.0 - 1.0) + (l == 4 ? 0.0 : 0.01);
    const int most = src_tiles / per_round;
    for (int f = most; f >= 0 && f >= most - 1; --f) {
      const int rest = src_tiles - f * per_round;
      if (rest > team * kXcd) break;
      int rs = rest ? team * kXcd / rest : 1;
      if (rs > dst_tiles) rs = dst_tiles;
      if (rs > max_lists) rs = max_lists;
      while (lists_of(rs) > max_lists) --rs;
      // + a few percent of a step per round for filling the pipeline and writing the result
      const double cost = f * (div_up(dst_tiles, l) * share + 0.1) + (rest ? div_up(dst_tiles, rs) * 1.03 + 0.1 : 0.0);
      if (cost < best_cost) {
        best_cost = cost;
        best = {l, sr, f, rs, rest, f * per_round, lists_of(l), lists_of(rs)};
      }
    }
  }
  return best;
}
static size_t sched_partials(const MatchSched &s) {   // tiles of 256 partial results
  return (size_t)s.full_lists * s.full + (size_t)s.rest_lists * s.n_rest;
}

__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_match_sim(
    const u32x4 *__restrict__ srcp, const u32x4 *__restrict__ dstp, const float *__restrict__ invd,
    int n_dst_tiles, MatchSched sched, int KS, int spin_budget, uint32_t *team_ctr,
    Top2 *__restrict__ top2p) {
  extern __shared__ u32x4 ring[];    // kGStages stages
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wd = wave & 3, wsrc = wave >> 2;
  const int team = blockIdx.x & (kXcd - 1), rank = blockIdx.x >> 3;
  const int per_team = gridDim.x >> 3, team_size = sched.n_sweeps * sched.sr;
  const int SPT = KS >> 1;           // stages per tile
  uint32_t *ctr = team_ctr + team * 32;      // one counter per team, 128 bytes apart
  uint32_t rounds = 0;                       // sweep steps of the rounds the team has finished
  const int n_rounds = sched.n_full + (sched.n_rest ? 1 : 0);

  for (int rd = 0; rd < n_rounds; ++rd) {
  const bool in_team = rd < sched.n_full;    // else the last round, over the whole chip
  // chip-wide the workgroups of an XCD are neighbours: few src tiles with many sweeps each
  const int id = in_team ? rank : team * per_team + rank;
  const int n_lanes = in_team ? sched.n_sweeps : sched.rest_sweeps;
  const int dl = id % n_lanes, sti = id / n_lanes;
  const int st = in_team ? (rd * kXcd + team) * sched.sr + sti : sched.full + sti;
  const int nt_max = (n_dst_tiles + n_lanes - 1) / n_lanes;
  const int nt = dl < n_dst_tiles ? (n_dst_tiles - dl + n_lanes - 1) / n_lanes : 0;   // my dst tiles
  const int total = nt * SPT;
  const bool member = sti < (in_team ? sched.sr : sched.n_rest);
  const bool active = member && total > 0;
  const int lists = (in_team ? sched.full_lists : sched.rest_lists) / n_lanes;   // of this sweep: 1, 2 or 4
  Top2 best[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) best[b] = Top2{-INFINITY, -1, -INFINITY, -1};

  if (active) {
    // fetch: this wave moves fragments f = 4*wave .. 4*wave+3 of a stage (f = op*16 + ks*8 + a)
    const int f_op = wave >> 2, f_ks = (wave >> 1) & 1, f_a0 = (wave & 1) * 4;
    int pf_tile = dl, pf_s = 0, pf_g = 0;      // next stage to fetch: dst tile, stage in tile, flat index
    int pf_t = 0;                              // tiles whose first stage has been requested
    // the inverse norms of this wave's 64 dst rows travel with the first stage of their tile
    // into a wave-private LDS buffer, so the fold at the end of the tile has them without a
    // memory round trip.  kInvBufs buffers in turn: stages are requested up to kGStages ahead,
    // which with one stage per tile (C = 32) is that many tiles not yet folded.
    float *inv_lds = (float *)(ring + (size_t)kGStages * kGStageU4) + wave * (kInvBufs * 64);
    // fetch_part<0>: the inverse norms and fragments 0, 1 of the stage; fetch_part<1>: fragments
    // 2, 3 and the bookkeeping.
    auto fetch_part = [&](auto part) {
      constexpr int P = decltype(part)::value;
      if (P == 0 && pf_s == 0 && pf_g < total) {
        __builtin_amdgcn_global_load_lds(invd + (size_t)pf_tile * kGTile + wd * 64 + lane,
                                         inv_lds + (pf_t & (kInvBufs - 1)) * 64, 4, 0, 0);
        ++pf_t;
      }
      const int tile = f_op ? pf_tile : st;
      const u32x4 *src = (f_op ? dstp : srcp) +
                         ((size_t)(tile * 8 + f_a0) * KS + (size_t)(pf_s * 2 + f_ks)) * 64 + lane;
      u32x4 *dst = ring + (size_t)(pf_g & (kGStages - 1)) * kGStageU4 + (size_t)(wave * 4) * 64;
#pragma unroll
      for (int i = 2 * P; i < 2 * P + 2; ++i)
        __builtin_amdgcn_global_load_lds(src + (size_t)i * KS * 64, dst + i * 64, 16, 0, 0);
      if (P == 1) {
        ++pf_g;
        // past the end the last stage is fetched again (into a free slot nobody reads)
        if (pf_g < total && ++pf_s == SPT) {
          pf_s = 0;
          pf_tile += n_lanes;
        }
      }
    };
    auto fetch = [&]() {
      fetch_part(std::integral_constant<int, 0>{});
      fetch_part(std::integral_constant<int, 1>{});
    };
    const uint32_t ring_lane = lds_addr(&ring[lane]);
    // byte offsets of this wave's fragments inside a stage, k-step 0: src (B operand) fragments
    // 4*wsrc .. +3, dst (A operand) fragments 2*wd, 2*wd+1; k-step 1 is 8 KB further
    const uint32_t b_off = (uint32_t)((0 * 16 + wsrc * 4) * 1024), a_off = (uint32_t)((16 + wd * 2) * 1024);
    u32x4 fb[2][4], fa[2][2];
    auto read_frags = [&](int g, int ks, u32x4(&b)[4], u32x4(&a)[2]) {
      const uint32_t base = ring_lane + (uint32_t)((g & (kGStages - 1)) * kGStageU4 * 16 + ks * 8 * 1024);
      lds_read4_async(b, base + b_off);
      lds_read2_async(a, base + a_off);
    };
    auto wait_frags = [&](u32x4(&b)[4], u32x4(&a)[2]) {
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]), "+v"(a[0]), "+v"(a[1])
                   :
                   : "memory");
    };
    f32x16 acc[2][4];
    auto clear_acc = [&]() {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    };
    auto mma = [&](const u32x4(&b)[4], const u32x4(&a)[2]) {
#pragma unroll
      for (int bi = 0; bi < 4; ++bi)
#pragma unroll
        for (int ai = 0; ai < 2; ++ai)
          acc[ai][bi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[ai]),
                                                               __builtin_bit_cast(bf16x8, b[bi]),
                                                               acc[ai][bi], 0, 0, 0);
    };
    auto mma_first = [&](const u32x4(&b)[4], const u32x4(&a)[2]) {   // first k-step of a tile: starts from zero
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int bi = 0; bi < 4; ++bi)
#pragma unroll
        for (int ai = 0; ai < 2; ++ai)
          acc[ai][bi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[ai]),
                                                               __builtin_bit_cast(bf16x8, b[bi]), zero, 0, 0, 0);
    };
    auto mma_pair = [&](const u32x4(&b)[4], const u32x4(&a)[2], int bi) {   // the two MFMAs of column block bi
#pragma unroll
      for (int ai = 0; ai < 2; ++ai)
        acc[ai][bi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[ai]),
                                                             __builtin_bit_cast(bf16x8, b[bi]),
                                                             acc[ai][bi], 0, 0, 0);
    };
    // Fold the eight finished 32x32 tiles into the running top-2 of this lane's four columns.
    // Almost no element beats its column's second best once a few tiles have been seen, but
    // with 64 columns per wave "some lane of the wave has such an element in this tile" is true
    // nearly always, so the test is made per element: a compare per element and one branch per
    // tile in the common case, the insertion code only for the elements that need it.
    //
    // A column's rows are spread over eight running pairs (four waves, two lane halves), each
    // of which alone would let through about 2 ln(rows / 8) elements.  The test is therefore
    // made against thr >= the largest second best that any pair of the same list had at the end
    // of the previous tile (exchanged through LDS once per tile; a list is all four waves, two or
    // one): an element at or below it cannot be one of the list's two best, and with equal
    // values it has the higher row index, because earlier tiles hold lower rows.  Two buffers by tile parity: a wave that is already done
    // with this tile writes the other one (bounds from this tile's rows could tie with a lower
    // row that a slower wave has yet to see), and nobody is more than one tile-end barrier apart.
    float *share = (float *)(ring + (size_t)kGStages * kGStageU4) + 8 * kInvBufs * 64;   // [parity][wsrc][b][wd][column]
    const int peers = 4 / lists - 1, w0 = wd & ~peers;   // the waves of this one's list: w0 .. w0 + peers
    float thr[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int b = 0; b < 4; ++b) {   // before the first barrier of the round
      share[((wsrc * 4 + b) * 4 + wd) * 32 + (lane & 31)] = -INFINITY;
      share[1024 + ((wsrc * 4 + b) * 4 + wd) * 32 + (lane & 31)] = -INFINITY;
    }
    auto fold = [&](int tile, int buf, int parity) {
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int w = 0; w < 4; ++w)
          thr[b] = fmaxf(thr[b], share[parity * 1024 + ((wsrc * 4 + b) * 4 + w0 + (w & peers)) * 32 + (lane & 31)]);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int row0 = tile * kGTile + wd * 64 + a * 32 + h * 4;
        const f32x4 *ip = (const f32x4 *)(inv_lds + buf * 64 + a * 32 + h * 4);
        f32x4 iv[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) iv[g] = ip[2 * g];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          float v[16];
          uint64_t hit[16], any = 0;       // lanes whose element r beats their second best (scalar masks)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            v[r] = acc[a][b][r] * iv[r >> 2][r & 3];
            hit[r] = __builtin_amdgcn_ballot_w64(v[r] > thr[b]);
            any |= hit[r];
          }
          if (any != 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              if (hit[r] != 0) {   // insertions only raise the thresholds: the masks stay a superset
                top2_insert_later(best[b], v[r], row0 + (r >> 2) * 8 + (r & 3));
              }
            }
            thr[b] = fmaxf(thr[b], best[b].v2);
          }
        }
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        thr[b] = fmaxf(thr[b], __shfl_xor(thr[b], 32, 64));   // the other half of the wave has the same column
        share[(parity ^ 1) * 1024 + ((wsrc * 4 + b) * 4 + wd) * 32 + (lane & 31)] = thr[b];
      }
    };

    clear_acc();
#pragma unroll
    for (int i = 0; i < kGStages; ++i) fetch();                // stages 0..3
    asm volatile("s_waitcnt vmcnt(12)" ::: "memory");          // stage 0 has landed (this wave's part)
    __builtin_amdgcn_s_barrier();
    read_frags(0, 0, fb[0], fa[0]);
    int tile = dl, sidx = 0, steps = 0;
    for (int g = 0; g < total; ++g) {
      // k-step 0 of stage g
      __builtin_amdgcn_sched_barrier(0);
      wait_frags(fb[0], fa[0]);
      read_frags(g, 1, fb[1], fa[1]);
      __builtin_amdgcn_sched_barrier(0);
      if (sidx == 0) mma_first(fb[0], fa[0]);
      else mma(fb[0], fa[0]);
      // k-step 1 of stage g: its fragments are in registers, so the slot of stage g is free once
      // every wave is here; stage g+1 is published by the same barrier.  The barrier, the
      // fetch instructions and the fragment reads sit between pairs of MFMAs, so that the MFMA
      // pipe still has queued work from this wave while it does them.
      __builtin_amdgcn_sched_barrier(0);
      wait_frags(fb[1], fa[1]);
      mma_pair(fb[1], fa[1], 0);
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt vmcnt(8)" ::: "memory");         // stage g+1 has landed; g+2, g+3 may be in flight
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      mma_pair(fb[1], fa[1], 1);
      __builtin_amdgcn_sched_barrier(0);
      // The stage's loads go out in two halves with an MFMA pair and the fragment reads between
      // them: eight waves issuing all five loads at once right behind the barrier was measured
      // 1 % slower.  (Anything moved ahead of the barrier, into k-step 0, costs 2-6 %.)
      fetch_part(std::integral_constant<int, 0>{});            // stage g+4 -> slot of stage g, first half
      __builtin_amdgcn_sched_barrier(0);
      mma_pair(fb[1], fa[1], 2);
      __builtin_amdgcn_sched_barrier(0);
      read_frags(g + 1, 0, fb[0], fa[0]);                      // past the end: a stale slot, never used
      __builtin_amdgcn_sched_barrier(0);
      fetch_part(std::integral_constant<int, 1>{});            // second half
      __builtin_amdgcn_sched_barrier(0);
      mma_pair(fb[1], fa[1], 3);
      if (++sidx == SPT) {
        // Team step: the workgroups of a team finish a dst tile at about the same time and
        // start the next one together, so that what one of them fetches is still in their
        // XCD's L2 when the others ask for it.  The wait is advisory: it is bounded, and no
        // result depends on it.
        if (in_team && tid == 0) __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        fold(tile, steps & (kInvBufs - 1), steps & 1);
        sidx = 0;
        tile += n_lanes;
        ++steps;
        if (in_team && tid == 0) {
          const uint32_t target = (uint32_t)team_size * (rounds + (uint32_t)steps);
          for (int spin = 0; spin < spin_budget; ++spin) {
            if (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= target) break;
            __builtin_amdgcn_s_sleep(8);
          }
        }
        __builtin_amdgcn_s_barrier();
      }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // nothing may land in LDS any more
  }
  __syncthreads();
  // sweep steps this workgroup did not take still count for its team
  if (in_team && member) {
    const uint32_t missing = (uint32_t)(nt_max - nt);
    if (tid == 0 && missing)
      __hip_atomic_fetch_add(ctr, missing, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    rounds += (uint32_t)nt_max;
  }
  if (member) {
    // merge the two half-wave copies of a column and the four dst quarters (waves wd = 0..3)
    Top2 *cand = (Top2 *)ring;
#pragma unroll
    for (int b = 0; b < 4; ++b) cand[(wave * 4 + b) * 64 + lane] = best[b];
    __syncthreads();
    if (tid < kGTile) {
      const int ws2 = tid >> 7, b = (tid >> 5) & 3, c = tid & 31;
      for (int g = 0, w = 0; g < lists; ++g) {
        Top2 t = Top2{-INFINITY, -1, -INFINITY, -1};
        for (; w < 4 * (g + 1) / lists; ++w)
          for (int hh = 0; hh < 2; ++hh) {
            const Top2 cd = cand[((ws2 * 4 + w) * 4 + b) * 64 + hh * 32 + c];
            top2_insert_any(t, cd.v1, cd.i1);
            top2_insert_any(t, cd.v2, cd.i2);
          }
        const size_t at = in_team ? (size_t)(dl * lists + g) * sched.full + st
                                  : (size_t)sched.full_lists * sched.full + (size_t)(dl * lists + g) * sched.n_rest + sti;
        top2p[at * kGTile + tid] = t;
      }
    }
    __syncthreads();   // the ring is reused by the next round
  }
  }   // rounds
}

// ---------------------------------------------------------------------------------
// Few tokens.  A handful of 256 x 256 tiles leaves most CUs idle while each takes a whole tile step (1024 channels:
// 28 us, and the fold's code for eight blocks comes in cold).  Here a workgroup has 64 src x 64 dst
// rows and four waves: wave (kg, wn) multiplies half of the channels for 32 src rows with both halves
// of the dst rows, fragments straight from L2 into registers, three batches of two k-steps ahead of
// their use; the two channel halves meet in LDS, wave (kg, .) folds dst rows 32 kg .. + 31, and the
// 64 dst rows of a tile are one candidate list.  Bound by the latency of its chain: the operands'
// round trips, the fold, two barriers.
// ---------------------------------------------------------------------------------
constexpr int kSmallTile = 64;       // src and dst rows of a workgroup
// Workgroups at most, four rounds of two per CU.  One refresh, otherwise -> this way: 2 frames of 16 x 16, C = 256 (10 of
// them) 39.4 -> 24.2 us; C = 1024: 2 frames of 37 x 37 (460) 68.1 -> 44.0, 3 (975) 79.0 -> 60.2, 4 (1566) 86.0 -> 75.9, 5
// (2156) 85.8 and 85.7, 6 (2910) 85.4 and 100.4.  The line lies here at every width: C = 256, 24 frames of 16 x 16 at the fixed
// rule (1647) 57.6 -> 52.1, 32 at ratio 0.5 (2170) 58.3 and 57.8, 6 of 37 x 37 (2910) 63.1 and 68.7; C = 64 (1647) 50.8 -> 47.4,
// (2170) 49.6 and 49.2, (2910) 55.3 and 59.3.
constexpr int kSmallTiles = 2048;

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_match_small(
    const u32x4 *__restrict__ srcp, const u32x4 *__restrict__ dstp, const float *__restrict__ invd, int n_st,
    int n_dt, int KS, int stride, Top2 *__restrict__ top2p) {
  __shared__ f32x4 part[2][2][4 * 64];       // [kg][wn][register group][lane]: the sums the other group finishes
  __shared__ Top2 cand[2][kSmallTile];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wn = wave & 1, kg = wave >> 1;
  const uint32_t lb = xcd_contiguous(blockIdx.x, (uint32_t)(n_st * n_dt));   // an XCD's workgroups share src tiles
  if (lb >= (uint32_t)(n_st * n_dt)) return;
  const int st = lb / n_dt, dt = lb % n_dt;
  const int nb = KS >> 2;                    // batches of two k-steps in this wave's half of the channels (C % 64 == 0)
  const u32x4 *ap = dstp + ((size_t)(dt * 2) * KS + kg * (KS >> 1)) * 64 + lane;
  const u32x4 *bp = srcp + ((size_t)(st * 2 + wn) * KS + kg * (KS >> 1)) * 64 + lane;
  u32x4 fa[4][2][2], fb[4][2];               // [batch & 3][k-step][dst half]
  auto load = [&](int i, u32x4(&a)[2][2], u32x4(&b)[2]) {   // past the end the last batch again
    const size_t at = (size_t)min(i, nb - 1) * 2 * 64;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      b[k] = bp[at + k * 64];
#pragma unroll
      for (int d = 0; d < 2; ++d) a[k][d] = ap[at + k * 64 + (size_t)d * KS * 64];
    }
  };
  f32x16 acc[2];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[d][r] = 0.f;
#pragma unroll
  for (int j = 0; j < 3; ++j) load(j, fa[j], fb[j]);
  for (int i = 0; i < nb; i += 4) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (i + j < nb) {
        load(i + j + 3, fa[(j + 3) & 3], fb[(j + 3) & 3]);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int d = 0; d < 2; ++d)
            acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[j][k][d]),
                                                             __builtin_bit_cast(bf16x8, fb[j][k]), acc[d], 0, 0, 0);
      }
    }
  }
  // the inverse norms of the rows this wave folds, 8g + 4h .. + 3 of its half
  f32x4 iv[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) iv[g] = *(const f32x4 *)(invd + dt * kSmallTile + kg * 32 + 8 * g + 4 * h);
#pragma unroll
  for (int d = 0; d < 2; ++d)
    if (d != kg)                             // (uniform: one copy runs)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        part[kg][wn][g * 64 + lane] = f32x4{acc[d][4 * g], acc[d][4 * g + 1], acc[d][4 * g + 2], acc[d][4 * g + 3]};
  __syncthreads();
  Top2 t = Top2{-INFINITY, -1, -INFINITY, -1};
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 o = part[1 - kg][wn][g * 64 + lane];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float own = kg == 0 ? acc[0][4 * g + i] : acc[1][4 * g + i];
      top2_insert_later(t, (own + o[i]) * iv[g][i], dt * kSmallTile + kg * 32 + 8 * g + 4 * h + i);
    }
  }
  const Top2 u = Top2{__shfl_xor(t.v1, 32, 64), __shfl_xor(t.i1, 32, 64), __shfl_xor(t.v2, 32, 64), __shfl_xor(t.i2, 32, 64)};
  top2_insert_any(t, u.v1, u.i1);
  top2_insert_any(t, u.v2, u.i2);
  if (h == 0) cand[kg][wn * 32 + lane] = t;
  __syncthreads();
  if (tid < kSmallTile) {
    Top2 b = cand[0][tid];
    const Top2 o = cand[1][tid];
    top2_insert_any(b, o.v1, o.i1);
    top2_insert_any(b, o.v2, o.i2);
    top2p[(size_t)dt * stride + st * kSmallTile + tid] = b;
  }
}

// Final decision per src row.  Every list (MatchSched) holds its two best candidates by fp32 similarity.
// If the runner-up is closer than kRescoreGap to the best, every candidate inside that gap is
// recomputed in float64 and the decision is taken on those values rounded to fp32, lowest token
// index on a tie: the rule the fp32 accumulation order cannot disturb.  A row with more
// near-equal candidates than one list's two best can still lose its true best inside a list;
// what it picks instead is within twice the fp32 accumulation error of it (C / 16 additions of
// exact 16-product sums).
//
// Bound by the latency of its index chain: a wave takes kFinRows consecutive rows at once, 8 lanes
// per row reading the row's lists, and only the rows with near-equal candidates one after the
// other with all 64 lanes (a wave per row: 32 us for 38,192 rows none of which is near-equal).
// 8 rows and no more, because in late refreshes most rows are near-equal and want many waves.  (Up to 256 rows by the one
// workgroup that sorts the groups behind them, a launch less: us, matching of 2 frames of 16 x 16, C = 256, tokens that differ 19.6
// and 18.5 at ratio 0.5, 18.4 and 20.7 at 0.9; all alike 62 and 134, 63 and 244.)
constexpr int kFinRows = 8;

// A row that goes to 64 bits is a chain of round trips, and a wave with a few of them is what the launch waits for: two candidates
// and the src row itself are read at once, and their five sums cross the lanes side by side by DPP (one after the other,
// by LDS shuffles: refreshes of 5 frames of 16 x 16, C = 1024, 38.1 -> 36.0 us, 12 of 37 x 37 154.4 -> 152.0; matching of 2 frames of
// 16 x 16 with tokens all alike, C = 256, 79 -> 62, 1024 108 -> 81, of 37 x 37 484 -> 356; the same bits).
__global__ __launch_bounds__(256) void k_match_finish(
    const uint16_t *__restrict__ x, const int32_t *__restrict__ src_idx,
    const int32_t *__restrict__ dst_idx, const float *__restrict__ inv_src,
    const Top2 *__restrict__ top2p, MatchSched sched, int n_src, int C,
    int32_t *__restrict__ anchor_of, int32_t *slot_of, float *__restrict__ best_sim) {
  const int lane = threadIdx.x & 63, nch = C >> 3, sub = lane & 7;
  const int64_t p0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kFinRows;
  if (p0 >= n_src) return;
  const int p = (int)min(p0 + (lane >> 3), (int64_t)n_src - 1);
  // the sweeps of the rows of this wave (a tile of 256 rows holds whole waves' rows)
  const int tile = (int)(p0 / kGTile);
  const bool in_full = tile < sched.full;
  const int n_lists = in_full ? sched.full_lists : sched.rest_lists;
  const size_t stride = (size_t)(in_full ? sched.full : sched.n_rest) * kGTile;
  const Top2 *part = in_full ? top2p : top2p + (size_t)sched.full_lists * sched.full * kGTile - (size_t)sched.full * kGTile;
  const int s = src_idx[p];
  Top2 t = Top2{-INFINITY, -1, -INFINITY, -1};
  for (int l = sub; l < n_lists; l += 8) {
    const Top2 o = part[l * stride + p];
    top2_insert_any(t, o.v1, o.i1);
    top2_insert_any(t, o.v2, o.i2);
  }
  const float invs = inv_src[p];
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) {
    const Top2 u = Top2{__shfl_xor(t.v1, o, 64), __shfl_xor(t.i1, o, 64), __shfl_xor(t.v2, o, 64), __shfl_xor(t.i2, o, 64)};
    top2_insert_any(t, u.v1, u.i1);
    top2_insert_any(t, u.v2, u.i2);
  }
  int choose = t.i1 < 0 ? 0 : t.i1;
  float sim = t.i1 < 0 ? 0.f : t.v1 * invs;
  const bool near = t.i1 >= 0 && t.i2 >= 0 && (t.v1 - t.v2) * invs < kRescoreGap;
  uint64_t rows = __builtin_amdgcn_ballot_w64(near && sub == 0 && p0 + (lane >> 3) < n_src);
  while (rows) {
    const int r = __builtin_ctzll(rows);       // first lane of the row's eight
    rows &= rows - 1;
    const int rp = __builtin_amdgcn_readlane(p, r), rs = __builtin_amdgcn_readlane(s, r);
    const float v1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, t.v1), r));
    const float is32 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, invs), r));
    // lane l holds the two candidates of list l
    Top2 o = Top2{-INFINITY, -1, -INFINITY, -1};
    if (lane < n_lists) o = part[lane * stride + rp];
    uint64_t c1 = __builtin_amdgcn_ballot_w64(o.i1 >= 0 && (v1 - o.v1) * is32 < kRescoreGap);
    uint64_t c2 = __builtin_amdgcn_ballot_w64(o.i2 >= 0 && (v1 - o.v2) * is32 < kRescoreGap);
    float bs = -INFINITY;
    int bd = 0x7fffffff, bi = 0;
    auto take = [&]() {                        // the next candidate inside the gap
      const bool first = c1 != 0;
      const int l = __builtin_ctzll(first ? c1 : c2);
      if (first) c1 &= c1 - 1;
      else c2 &= c2 - 1;
      return first ? __builtin_amdgcn_readlane(o.i1, l) : __builtin_amdgcn_readlane(o.i2, l);
    };
    while (c1 | c2) {                          // two at a time (never none: the best is one; an odd last one twice)
      int ci[2];
      ci[0] = take();
      ci[1] = c1 | c2 ? take() : ci[0];
      const int d[2] = {dst_idx[ci[0]], dst_idx[ci[1]]};
      double ss = 0, nn[2] = {0, 0}, pp[2] = {0, 0};
      for (int ch = lane; ch < nch; ch += 64) {
        const u32x4 w = ((const u32x4 *)(x + (size_t)rs * C))[ch];
        const u32x4 wd[2] = {((const u32x4 *)(x + (size_t)d[0] * C))[ch], ((const u32x4 *)(x + (size_t)d[1] * C))[ch]};
        const uint32_t us[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double sl = bf16_lo(us[q]), sh = bf16_hi(us[q]);
          ss += sl * sl + sh * sh;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const uint32_t ud = q == 0 ? wd[k].x : q == 1 ? wd[k].y : q == 2 ? wd[k].z : wd[k].w;
            const double al = bf16_lo(ud), ah = bf16_hi(ud);
            nn[k] += al * al + ah * ah;
            pp[k] += sl * al + sh * ah;
          }
        }
      }
      ss = wave_sum_ordered(ss);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        nn[k] = wave_sum_ordered(nn[k]);
        pp[k] = wave_sum_ordered(pp[k]);
      }
      const double is = 1.0 / fmax(sqrt(ss), 1e-12);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const float sc = (float)(pp[k] * is * (1.0 / fmax(sqrt(nn[k]), 1e-12)));
        if (sc > bs || (sc == bs && d[k] < bd)) {
          bs = sc;
          bd = d[k];
          bi = ci[k];
        }
      }
    }
    if (lane == r && bd != 0x7fffffff) {       // (NaN similarities leave the fp32 choice)
      choose = bi;
      sim = bs;
    }
  }
  if (sub == 0 && p0 + (lane >> 3) < n_src) {
    const int a = dst_idx[choose];
    anchor_of[s] = a;
    slot_of[s] = slot_of[a];
    if (best_sim) best_sim[p] = sim;
  }
}

// ---------------------------------------------------------------------------------
// CSR groups: a stable LSD radix sort of (slot_of[i], i) gives the members of every slot in
// ascending token order.  All of it is latency: a few MB at the most per pass, three launches per
// pass.  Digits are as narrow as the number of passes allows (fewer counters to scan); a
// workgroup takes a chunk of 1024 elements, each of its 4 waves 256 consecutive ones, so the
// scatter is a chain of 4 steps and not of 16; the last pass writes group_mem itself.
// Together 56 -> 34 us at 32 frames of 37 x 37 patches, 73 -> 41 us at 100 frames of 28 x 37 (before the
// three-launch way, which takes both of these sizes now: 15 and 26 us under the trace).
// ---------------------------------------------------------------------------------
constexpr int kSortChunk = 1024;
constexpr int kScanPer = 16;     // counters per thread and tile of the scan

__global__ __launch_bounds__(256) void k_radix_hist(const uint32_t *__restrict__ keys, int64_t N,
                                                    int shift, int bins, int nchunks,
                                                    uint32_t *__restrict__ hist) {
  __shared__ uint32_t h[256];
  const int tid = threadIdx.x;
  h[tid] = 0u;
  __syncthreads();
  const int64_t b = (int64_t)blockIdx.x * kSortChunk;
#pragma unroll
  for (int i = 0; i < kSortChunk / 256; ++i) {
    const int64_t g = b + i * 256 + tid;
    if (g < N) atomicAdd(&h[(keys[g] >> shift) & (uint32_t)(bins - 1)], 1u);
  }
  __syncthreads();
  if (tid < bins) hist[(size_t)tid * nchunks + blockIdx.x] = h[tid];
}

// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ uint32_t wave_scan(uint32_t v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t up = __shfl_up(v, o, 64);
    if (lane >= o) v += up;
  }
  return v;
}

// exclusive prefix sum over hist[bins*nchunks] in place (digit-major), single workgroup: tiles
// of 16384 elements, 16 consecutive elements per thread, the running total carried from tile to tile
__global__ __launch_bounds__(1024) void k_radix_scan(uint32_t *__restrict__ hist, int64_t n) {
  __shared__ uint32_t wtot[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t carry = 0;
  for (int64_t t0 = 0; t0 < n; t0 += 1024 * kScanPer) {
    const int64_t i = t0 + (int64_t)tid * kScanPer;
    uint32_t v[kScanPer], sum = 0u;
#pragma unroll
    for (int u = 0; u < kScanPer; u += 4) {
      u32x4 q = u32x4{0u, 0u, 0u, 0u};
      if (i + u + 3 < n) {   // the array starts on a 256-byte boundary
        q = *(const u32x4 *)(hist + i + u);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (i + u + e < n) q[e] = hist[i + u + e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[u + e] = q[e];
        sum += q[e];
      }
    }
    const uint32_t inc = wave_scan(sum, lane);
    if (lane == 63) wtot[wave] = inc;
    __syncthreads();
    uint32_t base = 0, total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const uint32_t wt = wtot[w];
      if (w < wave) base += wt;
      total += wt;
    }
    uint32_t run = carry + base + inc - sum;
#pragma unroll
    for (int u = 0; u < kScanPer; u += 4) {
      u32x4 q;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        q[e] = run;
        run += v[u + e];
      }
      if (i + u + 3 < n) {
        *(u32x4 *)(hist + i + u) = q;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (i + u + e < n) hist[i + u + e] = q[e];
      }
    }
    carry += total;
    __syncthreads();   // wtot is rewritten by the next tile
  }
}

// the lanes that are on and hold the same digit as this one
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, int bits, bool on) {
  uint64_t peers = __builtin_amdgcn_ballot_w64(on);
  for (int bit = 0; bit < bits; ++bit) {
    const uint64_t bal = __builtin_amdgcn_ballot_w64((d >> bit) & 1u);
    peers &= ((d >> bit) & 1u) ? bal : ~bal;
  }
  return peers;
}
// A wave's own LDS accesses complete in program order; this keeps the compiler to that order.
__device__ __forceinline__ void wave_lds_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// vals_in NULL: element i carries i.
__global__ __launch_bounds__(256) void k_radix_scatter(const uint32_t *__restrict__ keys,
                                                       const int32_t *__restrict__ vals_in, int64_t N,
                                                       int shift, int bits, int nchunks,
                                                       const uint32_t *__restrict__ hist,
                                                       uint32_t *__restrict__ keys_out,
                                                       int32_t *__restrict__ vals_out) {
  __shared__ uint32_t base[4][256];   // per wave: elements of a digit counted, then the next position
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t mask = (1u << bits) - 1u;
  const int64_t b = (int64_t)blockIdx.x * kSortChunk + wave * 256;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  uint32_t key[4];
  int32_t val[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t g = b + i * 64 + lane;
    key[i] = g < N ? keys[g] : 0u;
    val[i] = g < N ? (vals_in ? vals_in[g] : (int32_t)g) : 0;
  }
#pragma unroll
  for (int w = 0; w < 4; ++w) base[w][tid] = 0u;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (b + i * 64 + lane < N) atomicAdd(&base[wave][(key[i] >> shift) & mask], 1u);
  __syncthreads();
  if (tid <= (int)mask) {
    uint32_t run = hist[(size_t)tid * nchunks + blockIdx.x];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t c = base[w][tid];
      base[w][tid] = run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool ok = b + i * 64 + lane < N;
    const uint32_t d = (key[i] >> shift) & mask;
    const uint64_t peers = digit_peers(d, bits, ok);
    const uint32_t rank = (uint32_t)__popcll(peers & below), cnt = (uint32_t)__popcll(peers);
    const uint32_t at = base[wave][d];
    wave_lds_order();
    if (ok && rank == cnt - 1) base[wave][d] = at + cnt;   // one lane per digit present
    wave_lds_order();
    if (ok) {
      keys_out[at + rank] = key[i];
      vals_out[at + rank] = val[i];
    }
  }
}

// ---- Two passes in three launches (k_radix_first, two k_radix_move), where the counters are few enough
// for every workgroup to sum them itself: at these sizes a launch costs more than what it does. Counters lie [chunk][digit].  The first move counts the second one's digits on the way, at
// the places where its elements come to lie, and the second one finds the groups' starts as the lowest
// place of each slot; both by integer atomics, whose order leaves no trace.
// One refresh call, seven launches -> three: 12 frames of 37 x 37 patches 94.7 -> 90.5 us, 64 of 16 x 16
// 79.5 -> 73.7, 100 of 28 x 37 (13,056 counters) 1226.0 -> 1221.3; above 16,384 counters, 100 of 28 x 37,
// C = 256, at ratio 0.5 952 -> 937, 52 of 37 x 37, C = 256 369 -> 361, 200 of 28 x 37, C = 512 (52,480) 2853 -> 2813, 200 of
// 37 x 37 (68,864) level: what every workgroup reads grows with the tokens' square.
constexpr int kMoveCounters = 65536;   // chunks x digits, at most

// Counts the first pass' digits, clears the second pass' counters, and sets group_off to no place yet.
__global__ __launch_bounds__(256) void k_radix_first(const uint32_t *__restrict__ keys, int N, int M, int bits,
                                                     uint32_t *__restrict__ hist, uint32_t *__restrict__ hist2,
                                                     int32_t *__restrict__ group_off) {
  __shared__ uint32_t h[256];
  const int tid = threadIdx.x, bins = 1 << bits;
  h[tid] = 0u;
  __syncthreads();
  const int b = blockIdx.x * kSortChunk;
#pragma unroll
  for (int i = 0; i < kSortChunk / 256; ++i) {
    const int g = b + i * 256 + tid;
    if (g < N) atomicAdd(&h[keys[g] & (uint32_t)(bins - 1)], 1u);
    if (g <= M) group_off[g] = g == M ? N : 0x7fffffff;   // M <= N
  }
  if (N == M && blockIdx.x == gridDim.x - 1 && tid == 0) group_off[M] = N;
  __syncthreads();
  if (tid < bins) {
    hist[blockIdx.x * bins + tid] = h[tid];
    hist2[blockIdx.x * bins + tid] = 0u;
  }
}

// FIRST: element i carries i, and the elements' second digits are counted.  Else: the low digits are sorted
// and vals_out is group_mem.  16 waves of 64 elements: the counters of all chunks are read in two or three
// batches, and no wave has a chain of steps.
constexpr int kMoveWaves = kSortChunk / 64;

template <bool FIRST>
__global__ __launch_bounds__(kSortChunk) void k_radix_move(const uint32_t *__restrict__ keys,
                                                           const int32_t *__restrict__ vals_in, int N, int M, int bits,
                                                           int nchunks, const uint32_t *__restrict__ hist,
                                                           uint32_t *__restrict__ hist2, uint32_t *__restrict__ keys_out,
                                                           int32_t *__restrict__ vals_out, int32_t *__restrict__ group_off) {
  __shared__ uint32_t base[kMoveWaves][256];   // per wave: elements of a digit, then the place of its first one
  __shared__ uint32_t total[256], before[256], wtot[4];
  const int tid = threadIdx.x, lane = tid & 63, bins = 1 << bits, chunk = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t mask = (uint32_t)bins - 1u;
  const int g = chunk * kSortChunk + tid;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const bool ok = g < N;
  const uint32_t key = ok ? keys[g] : 0u;
  const int32_t val = ok ? (FIRST ? g : vals_in[g]) : 0;
  // of digit tid & mask, in every (1024 / bins)-th chunk: all elements, and those of earlier chunks
  uint32_t all = 0u, early = 0u;
  const int groups = kSortChunk >> bits;
  for (int c = tid >> bits; c < nchunks; c += 8 * groups) {
    uint32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = c + u * groups < nchunks ? hist[(c + u * groups) * bins + (tid & (int)mask)] : 0u;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      all += v[u];
      early += c + u * groups < chunk ? v[u] : 0u;
    }
  }
#pragma unroll
  for (int i = 0; i < kMoveWaves * 256 / kSortChunk; ++i) (&base[0][0])[i * kSortChunk + tid] = 0u;
  if (tid < 256) total[tid] = before[tid] = 0u;
  __syncthreads();
  const uint32_t d = (FIRST ? key : key >> bits) & mask;
  const uint64_t peers = digit_peers(d, bits, ok);
  const uint32_t rank = (uint32_t)__popcll(peers & below);
  if (ok && rank == 0u) base[wave][d] = (uint32_t)__popcll(peers);
  atomicAdd(&total[tid & (int)mask], all);
  atomicAdd(&before[tid & (int)mask], early);
  __syncthreads();
  // first place of a digit = all elements of lower digits + its elements in earlier chunks
  const uint32_t mine = tid < bins ? total[tid] : 0u;
  uint32_t inc = 0u;
  if (wave < 4) {
    inc = wave_scan(mine, lane);
    if (lane == 63) wtot[wave] = inc;
  }
  __syncthreads();
  if (tid < bins) {
    uint32_t run = inc - mine + before[tid];
    for (int w = 0; w < wave; ++w) run += wtot[w];
#pragma unroll
    for (int w = 0; w < kMoveWaves; ++w) {
      const uint32_t c = base[w][tid];
      base[w][tid] = run;
      run += c;
    }
  }
  __syncthreads();
  const uint32_t to = base[wave][d] + rank;
  if constexpr (FIRST) {
    if (ok) {
      keys_out[to] = key;
      vals_out[to] = val;
      atomicAdd(&hist2[(to / kSortChunk) * bins + ((key >> bits) & mask)], 1u);
    }
  } else {
    // lower lanes of the same high digit have no larger low digits: the nearest one tells whether the
    // slot has been here already
    const uint64_t lower = peers & below;
    const uint32_t prev = __shfl(key, lower ? 63 - __builtin_clzll(lower) : lane, 64);
    if (ok) {
      vals_out[to] = val;
      if ((!lower || prev != key) && key < (uint32_t)M) atomicMin(&group_off[key], (int32_t)to);
    }
  }
}

// group_off from the sorted slots (every slot has a member: its own kept token)
__global__ __launch_bounds__(256) void k_csr_finish(const uint32_t *__restrict__ keys, int64_t N,
                                                    int64_t M, int32_t *__restrict__ group_off) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= N) return;
  const uint32_t k = keys[j];
  if ((j == 0 || keys[j - 1] != k) && (int64_t)k < M) group_off[k] = (int32_t)j;
  if (j == N - 1) group_off[M] = (int32_t)N;
}

// Short sequences: the whole sort in one workgroup.  An element is slot << 14 | token; wave w
// owns elements w * per .. in steps of 64, ranks them against the earlier ones of its own with
// the same digit (two passes of 7 bits), and the positions follow from one scan over the
// counters of all digits and waves.  The elements are in registers while they are moved, so one
// LDS array serves both passes.  Up to kCsrSmall tokens, where its time on one CU is below the three
// launches of the general way.  One refresh call, this way against that: 2,748 tokens 53.5 and 61.3 us, 4,122 58.3 and
// 61.3, 6,870 63.7 and 61.5, 10,992 84.3 and 75.1, 15,114 95.6 and 78.5.  With at most 256 slots the general way is one digit
// pass in four launches: 2,448 tokens 35.0 and 37.8, 4,320 38.3 and 38.0, 6,400 39.8 and 33.1.
constexpr int kCsrSmall = 5120;
constexpr int kCsrSteps = kCsrSmall / 1024;   // 64-element steps per wave, at most

__global__ __launch_bounds__(1024) void k_csr_small(const int32_t *__restrict__ slot_of, int N, int M,
                                                    int32_t *__restrict__ group_off,
                                                    int32_t *__restrict__ group_mem) {
  extern __shared__ uint32_t elem[];            // [N]
  __shared__ uint32_t cnt[128 * 16];            // [digit][wave]
  __shared__ uint32_t wtot[16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const int steps = (N + 1023) / 1024, b = wave * steps * 64 + lane;
  uint32_t e[kCsrSteps], rk[kCsrSteps];
#pragma unroll
  for (int i = 0; i < kCsrSteps; ++i) {
    const int g = b + i * 64;
    e[i] = i < steps && g < N ? (uint32_t)slot_of[g] << 14 | (uint32_t)g : 0u;
  }
  for (int pass = 0; pass < 2; ++pass) {
    const int shift = 14 + 7 * pass;
    cnt[tid] = 0u;
    cnt[tid + 1024] = 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kCsrSteps; ++i) {
      if (i < steps) {
        const bool ok = b + i * 64 < N;
        const uint32_t d = (e[i] >> shift) & 127u;
        const uint64_t peers = digit_peers(d, 7, ok);
        const uint32_t r = (uint32_t)__popcll(peers & below), n = (uint32_t)__popcll(peers);
        const uint32_t at = cnt[d * 16 + wave];
        wave_lds_order();
        if (ok && r == n - 1) cnt[d * 16 + wave] = at + n;
        wave_lds_order();
        rk[i] = at + r;
      }
    }
    __syncthreads();
    const uint32_t c0 = cnt[2 * tid], c1 = cnt[2 * tid + 1];
    const uint32_t inc = wave_scan(c0 + c1, lane);
    if (lane == 63) wtot[wave] = inc;
    __syncthreads();
    uint32_t run = inc - c0 - c1;
    for (int w = 0; w < wave; ++w) run += wtot[w];
    cnt[2 * tid] = run;
    cnt[2 * tid + 1] = run + c0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kCsrSteps; ++i)
      if (i < steps && b + i * 64 < N) elem[cnt[((e[i] >> shift) & 127u) * 16 + wave] + rk[i]] = e[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kCsrSteps; ++i)
      if (i < steps && b + i * 64 < N) e[i] = elem[b + i * 64];
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < kCsrSteps; ++i) {
    const int j = b + i * 64;
    if (i < steps && j < N) {
      const int slot = (int)(e[i] >> 14);
      group_mem[j] = (int32_t)(e[i] & 0x3fffu);
      if (slot < M && (j == 0 || (int)(elem[j - 1] >> 14) != slot)) group_off[slot] = j;
    }
  }
  if (tid == 0) group_off[M] = N;
}

// ---------------------------------------------------------------------------------
static int small_tiles(int rows) { return (rows + kSmallTile - 1) / kSmallTile; }
// few tokens: k_match_small, with a list per dst tile
static bool match_is_small(int n_src, int n_dst) {
  return small_tiles(n_dst) <= kMaxLists && (int64_t)small_tiles(n_src) * small_tiles(n_dst) <= kSmallTiles;
}

struct MatchWs {
  u32x4 *dstp, *srcp;
  float *invd, *invs;
  Top2 *top2p;
  uint32_t *keys[2];
  int32_t *vals[2];
  uint32_t *hist, *team_ctr;
  size_t bytes;
  size_t partials;       // tiles of 256 partial results that top2p holds
  int n_dst_pad, n_src_pad, nchunks;
};

static MatchWs carve(const Dims &d, const litevggt_plan_t &pl, bool least, char *base) {
  MatchWs w;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char *p = base ? base + off : nullptr;
    off += align_up(bytes, 256);
    return p;
  };
  w.n_dst_pad = (int)align_up((size_t)pl.n_dst, kGTile);
  w.n_src_pad = (int)align_up((size_t)pl.n_src, kGTile);
  w.nchunks = (int)((d.N + kSortChunk - 1) / kSortChunk);
  w.dstp = (u32x4 *)take((size_t)w.n_dst_pad * d.C * 2);
  w.srcp = (u32x4 *)take((size_t)w.n_src_pad * d.C * 2);
  w.invd = (float *)take((size_t)w.n_dst_pad * 4);
  w.invs = (float *)take((size_t)w.n_src_pad * 4);
  const int src_tiles = w.n_src_pad / kGTile, dst_tiles = w.n_dst_pad / kGTile;
  w.partials = (size_t)kFewLists * src_tiles;
  const size_t ideal = match_is_small((int)pl.n_src, (int)pl.n_dst) ? (size_t)small_tiles((int)pl.n_dst) * src_tiles
                                                                    : sched_partials(match_sched(src_tiles, dst_tiles, kTeam));
  if (!least && ideal > w.partials) w.partials = ideal;
  w.top2p = (Top2 *)take(w.partials * kGTile * sizeof(Top2));
  for (int i = 0; i < 2; ++i) {
    w.keys[i] = (uint32_t *)take((size_t)d.N * 4);
    w.vals[i] = (int32_t *)take((size_t)d.N * 4);
  }
  w.hist = (uint32_t *)take((size_t)256 * w.nchunks * 4);
  w.team_ctr = (uint32_t *)take(256 * 4);
  w.bytes = off;
  return w;
}

size_t match_ws_bytes(const Dims &d, const litevggt_plan_t &pl, bool least) { return carve(d, pl, least, nullptr).bytes; }

int launch_match(const uint16_t *x, const Dims &d, const litevggt_plan_t &pl,
                 const litevggt_index &ix, float *best_sim, void *ws, size_t ws_bytes, hipStream_t st) {
  MatchWs w = carve(d, pl, ws_bytes < match_ws_bytes(d, pl), (char *)ws);
  const int n_src = (int)pl.n_src, n_dst = (int)pl.n_dst;
  if (n_src > 0) {
    if (d.C % 64 != 0 || n_dst <= 0) return LV_ERR_SHAPE;   // (64: k_match_small)
    // 128 KB ring (reused for the final merge) + per wave kInvBufs buffers of 64 inverse norms
    // and two buffers of 8 x 4 x 32 second-best bounds the waves of a column exchange
    constexpr size_t lds = (size_t)kGStages * kGStageU4 * 16 + 8 * kInvBufs * 64 * sizeof(float) + 2 * 1024 * sizeof(float);
    static std::atomic<uint64_t> lds_done{0};
    if (int rc = allow_dynamic_lds<lds>((const void *)k_match_sim, lds_done)) return rc;
    const int pack_dst = w.n_dst_pad / 32, pack_src = w.n_src_pad / 32;
    hipLaunchKernelGGL(k_match_pack, dim3((unsigned)(pack_dst + pack_src)), dim3(256), 0, st, x, ix.dst_idx, n_dst,
                       pack_dst, ix.src_idx, n_src, d.C, w.dstp, w.srcp, w.invd, w.invs, w.team_ctr);
    // One workgroup per CU, all resident at once; the workgroups the hardware deals to one
    // XCD (block index mod 8) form a team of (src tiles per super-row) x (sweeps).
    const int src_tiles = w.n_src_pad / kGTile, dst_tiles = w.n_dst_pad / kGTile;
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return LV_ERR_HIP;
    const int per_team = n_cu >= kXcd ? n_cu / kXcd : 1;
    const int n_st = small_tiles(n_src), n_dt = small_tiles(n_dst);
    MatchSched sched;
    if (match_is_small(n_src, n_dst) && (size_t)n_dt * src_tiles <= w.partials) {
      sched = {1, 1, 0, 1, src_tiles, 0, 1, n_dt};   // one list per dst tile of every src row
      hipLaunchKernelGGL(k_match_small, dim3((unsigned)align_up((size_t)n_st * n_dt, kXcd)), dim3(256), 0, st, w.srcp, w.dstp,
                         w.invd, n_st, n_dt, d.C / 16, src_tiles * kGTile, w.top2p);
    } else {
      sched = match_sched(src_tiles, dst_tiles, per_team);
      if (sched_partials(sched) > w.partials) sched = match_sched(src_tiles, dst_tiles, per_team, kFewLists);
      hipLaunchKernelGGL(k_match_sim, dim3((unsigned)(per_team * kXcd)), dim3(512), lds, st, w.srcp, w.dstp, w.invd, dst_tiles,
                         sched, d.C / 16, kTeamSpin, w.team_ctr, w.top2p);
    }
    const unsigned fin = (unsigned)((n_src + 4 * kFinRows - 1) / (4 * kFinRows));
    hipLaunchKernelGGL(k_match_finish, dim3(fin), dim3(256), 0, st, x, ix.src_idx, ix.dst_idx,
                       w.invs, w.top2p, sched, n_src, d.C, ix.anchor_of, ix.slot_of, best_sim);
    LV_HIP_CHECK_LAUNCH();
  }
  // CSR groups by stable radix sort of slot_of
  if (d.N <= kCsrSmall) {   // M <= N: slots fit 14 bits
    const size_t lds = align_up((size_t)d.N * sizeof(uint32_t), 16);
    static std::atomic<uint64_t> lds_done{0};
    if (int rc = allow_dynamic_lds<kCsrSmall * sizeof(uint32_t)>((const void *)k_csr_small, lds_done)) return rc;
    hipLaunchKernelGGL(k_csr_small, dim3(1), dim3(1024), lds, st, (const int32_t *)ix.slot_of, (int)d.N, (int)pl.M,
                       ix.group_off, ix.group_mem);
    LV_HIP_CHECK_LAUNCH();
    return LV_OK;
  }
  int bits = 1;
  while (((int64_t)1 << bits) < pl.M) ++bits;
  const int passes = (bits + 7) / 8, per_pass = (bits + passes - 1) / passes;
  const uint32_t *kin = (const uint32_t *)ix.slot_of;
  const int32_t *vin = nullptr;
  if (passes == 2 && (w.nchunks << per_pass) <= kMoveCounters) {
    uint32_t *hist2 = w.keys[1];   // (at least as many words as counters: N > kCsrSmall)
    const int N = (int)d.N, M = (int)pl.M;
    hipLaunchKernelGGL(k_radix_first, dim3((unsigned)w.nchunks), dim3(256), 0, st, kin, N, M, per_pass, w.hist, hist2,
                       ix.group_off);
    hipLaunchKernelGGL(k_radix_move<true>, dim3((unsigned)w.nchunks), dim3(kSortChunk), 0, st, kin, vin, N, M, per_pass, w.nchunks,
                       (const uint32_t *)w.hist, hist2, w.keys[0], w.vals[0], ix.group_off);
    hipLaunchKernelGGL(k_radix_move<false>, dim3((unsigned)w.nchunks), dim3(kSortChunk), 0, st, (const uint32_t *)w.keys[0],
                       (const int32_t *)w.vals[0], N, M, per_pass, w.nchunks, (const uint32_t *)hist2, (uint32_t *)nullptr,
                       (uint32_t *)nullptr, ix.group_mem, ix.group_off);
    LV_HIP_CHECK_LAUNCH();
    return LV_OK;
  }
  for (int p = 0; p < passes; ++p) {
    uint32_t *kout = w.keys[p & 1];
    int32_t *vout = p == passes - 1 ? ix.group_mem : w.vals[p & 1];
    hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)w.nchunks), dim3(256), 0, st, kin, d.N, per_pass * p,
                       1 << per_pass, w.nchunks, w.hist);
    hipLaunchKernelGGL(k_radix_scan, dim3(1), dim3(1024), 0, st, w.hist, (int64_t)w.nchunks << per_pass);
    hipLaunchKernelGGL(k_radix_scatter, dim3((unsigned)w.nchunks), dim3(256), 0, st, kin, vin, d.N,
                       per_pass * p, per_pass, w.nchunks, w.hist, kout, vout);
    kin = kout;
    vin = vout;
  }
  hipLaunchKernelGGL(k_csr_finish, dim3((unsigned)((d.N + 255) / 256)), dim3(256), 0, st, kin, d.N, pl.M,
                     ix.group_off);
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

}  // namespace lv

// Geometry-aware map (Sec. 3.4 "Geometry-aware Feature Map"): Sobel gradient map,
// local token-variance map, per-frame min-max normalisation and fusion.
// All three kernels are HBM-bound streaming passes; arithmetic is fp32.
#include "common.h"
#include "internal.h"

namespace lv {

// ---------------------------------------------------------------------------------
// Psi_g.  One workgroup per (frame, patch row); neighbouring patch rows run on the same XCD, whose
// L2 then has the two pixel rows they share.  The patch + 2 pixel rows (border rows replicated)
// are one contiguous run of each colour plane: four pixels per load, all planes' loads of four
// steps in flight, their luma kept in LDS.  Then a thread walks down its pixel column with the
// three rows of its three columns in registers (3 LDS reads per pixel, not 8) and the columns of a
// patch are added up.  Both sums are chains and run in float64, a pair of pixels per step; only the
// pairs, the column sums and the result are rounded (chains in fp32: 7.0e-8 relative error against 64
// bits on white noise, patch 14, now 2.9e-8; fp32 images take the same time, 8-bit ones 1.5 % more).
// Bound by HBM, as long as enough loads are in flight: 140 us for 100 frames
// of 518 x 518 in fp32 (2.3 TB/s) with one pixel per load and a division per pixel, now 57.
// VEC: the planes are whole numbers of 4-pixel pieces from an aligned base, so pieces never leave
// a plane; else one pixel at a time.
// ---------------------------------------------------------------------------------
template <typename PixT> struct Quad;
template <> struct Quad<float> { typedef f32x4 type; };
template <> struct Quad<uint8_t> { typedef uint32_t type; };
__device__ __forceinline__ f32x4 quad_f32(f32x4 v) { return v; }
__device__ __forceinline__ f32x4 quad_f32(uint32_t v) {
  return f32x4{(float)(v & 255u), (float)((v >> 8) & 255u), (float)((v >> 16) & 255u), (float)(v >> 24)};
}

// PIECES: pieces of every plane whose loads a thread has in flight.
template <typename PixT, bool VEC, int PIECES>
__device__ __forceinline__ void grad_rows(const PixT *__restrict__ img, int F, int H, int W, int patch,
                                          float *__restrict__ psi_g, uint32_t block, f32x4 *luma4) {
  float *luma = (float *)luma4;              // luma of the pixel rows, from the last multiple of 4 pixels on
  const int Hi = H * patch, Wi = W * patch;
  const uint32_t nblk = (uint32_t)F * H, lb = xcd_contiguous(block, nblk);
  if (lb >= nblk) return;
  const int f = lb / H, ph = lb % H, tid = threadIdx.x, nt = blockDim.x;
  const size_t plane = (size_t)Hi * Wi;
  const PixT *base = img + (size_t)f * 3 * plane;
  const float unit = sizeof(PixT) == 1 ? (1.0f / 255.0f) : 1.0f;
  const int y0 = max(ph * patch - 1, 0), y1 = min(ph * patch + patch + 1, Hi);   // pixel rows [y0, y1)
  const int p0 = y0 * Wi, p1 = y1 * Wi;      // (a plane has less than 2^31 pixels: its rows fit LDS)
  const int q0 = VEC ? p0 >> 2 : p0;
  if constexpr (VEC) {
    typedef typename Quad<PixT>::type Q;
    const Q *r4 = (const Q *)base, *g4 = (const Q *)(base + plane), *b4 = (const Q *)(base + 2 * plane);
    const int q1 = (p1 + 3) >> 2;
    for (int q = q0 + tid; q < q1; q += PIECES * nt) {
      Q v[PIECES][3];
#pragma unroll
      for (int u = 0; u < PIECES; ++u) {
        const int at = min(q + u * nt, q1 - 1);
        v[u][0] = r4[at];
        v[u][1] = g4[at];
        v[u][2] = b4[at];
      }
#pragma unroll
      for (int u = 0; u < PIECES; ++u) {
        const f32x4 r = quad_f32(v[u][0]) * unit, g = quad_f32(v[u][1]) * unit, b = quad_f32(v[u][2]) * unit;
        f32x4 l;
#pragma unroll
        for (int e = 0; e < 4; ++e) l[e] = 0.299f * r[e] + 0.587f * g[e] + 0.114f * b[e];
        if (q + u * nt < q1) luma4[q + u * nt - q0] = l;
      }
    }
  } else {
    for (int i = p0 + tid; i < p1; i += nt) {
      const float r = (float)base[i] * unit, g = (float)base[plane + i] * unit, b = (float)base[2 * plane + i] * unit;
      luma[i - q0] = 0.299f * r + 0.587f * g + 0.114f * b;
    }
  }
  __syncthreads();
  const int rows = ((y1 - y0) * Wi + 3 + 3) & ~3;          // floats before the column sums
  float *colsum = luma + rows;                             // [Wi]
  const float *top = luma + (VEC ? p0 & 3 : 0);            // pixel row y0
  for (int x = tid; x < Wi; x += nt) {
    const int xl = max(x - 1, 0), xr = min(x + 1, Wi - 1);
    auto row = [&](int y) { return top + (min(max(y, 0), Hi - 1) - y0) * Wi; };
    const float *c = row(ph * patch - 1);
    float al = c[xl], am = c[x], ar = c[xr];
    c = row(ph * patch);
    float bl = c[xl], bm = c[x], br = c[xr];
    auto step = [&](int py) {
      c = row(ph * patch + py + 1);
      const float cl = c[xl], cm = c[x], cr = c[xr];
      const float gx = (ar + 2.f * br + cr) - (al + 2.f * bl + cl);
      const float gy = (cl + 2.f * cm + cr) - (al + 2.f * am + ar);
      al = bl, am = bm, ar = br;
      bl = cl, bm = cm, br = cr;
      return sqrtf(gx * gx + gy * gy);
    };
    double acc = 0.0;
    int py = 0;
    for (; py + 1 < patch; py += 2) {
      const float g0 = step(py);
      acc += g0 + step(py + 1);
    }
    if (py < patch) acc += step(py);
    colsum[x] = (float)acc;
  }
  __syncthreads();
  const double pp = (double)(patch * patch);
  for (int pw = tid; pw < W; pw += nt) {
    double acc = 0.0;
    for (int i = 0; i < patch; ++i) acc += colsum[pw * patch + i];
    psi_g[((size_t)f * H + ph) * W + pw] = (float)(acc / pp);
  }
}
template <typename PixT, bool VEC>
__global__ __launch_bounds__(640) void k_grad_map(const PixT *__restrict__ img, int F, int H, int W,
                                                  int patch, float *__restrict__ psi_g) {
  extern __shared__ f32x4 luma4[];
  grad_rows<PixT, VEC, 4>(img, F, H, W, patch, psi_g, blockIdx.x, luma4);
}

int launch_grad_map(const void *images, int img_dtype, const Dims &d, int patch, float *psi_g,
                    hipStream_t st) {
  // the limit of the earlier layout ((patch + 2) rows of Wi + 2 luma values within 64 KB) is kept
  const int Wi = d.W * patch;
  if ((size_t)(patch + 2) * (Wi + 2) * sizeof(float) > 64 * 1024) return LV_ERR_SHAPE;
  const size_t lds = ((size_t)(patch + 2) * Wi + Wi + 8) * sizeof(float);   // pixel rows, column sums
  const int passes = (Wi + 639) / 640;       // a thread per pixel column, as few idle as may be
  const unsigned threads = (unsigned)(((Wi + passes - 1) / passes + 63) / 64 * 64);
  const dim3 grid((unsigned)align_up((size_t)d.F * d.H, kXcd));
  const size_t pix = img_dtype == LV_IMG_F32 ? 4 : 1;
  const bool vec = (size_t)d.H * patch * Wi % 4 == 0 && (uintptr_t)images % (4 * pix) == 0;
  static std::atomic<uint64_t> lds_done[4];
  int rc;
#define LV_GRAD(T, V, I)                                                                          \
  do {                                                                                            \
    if ((rc = allow_dynamic_lds<96 * 1024>((const void *)k_grad_map<T, V>, lds_done[I]))) return rc; \
    hipLaunchKernelGGL((k_grad_map<T, V>), grid, dim3(threads), lds, st, (const T *)images, d.F, d.H, d.W, patch, psi_g); \
  } while (0)
  if (img_dtype == LV_IMG_F32) {
    if (vec) LV_GRAD(float, true, 0);
    else LV_GRAD(float, false, 1);
  } else {
    if (vec) LV_GRAD(uint8_t, true, 2);
    else LV_GRAD(uint8_t, false, 3);
  }
#undef LV_GRAD
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

// ---------------------------------------------------------------------------------
// Psi_v.  One workgroup (2 waves) per (frame, grid row); thread t owns channels 8t..8t+7 (+1024k).
// The workgroup slides along the row: for every grid column it loads the K tokens of that
// column (rows i-R..i+R, clipped) once and keeps their per-channel sum and sum of squares
// for the last K columns in registers; the window of an output column is the sum of those K
// column partials, its variance E[d^2] - E[d]^2 in fp32 with d = x - (the frame's first patch
// token), so that the cancellation costs ~1e-7 of the spread and not of a channel's offset.
// Workgroups of consecutive grid rows are placed on the same XCD so the two neighbouring rows
// they share are found in that XCD's L2.
// ---------------------------------------------------------------------------------
template <int K>
__global__ __launch_bounds__(128) void k_var_map(const uint16_t *__restrict__ x, int F, int H,
                                                 int W, int S, int C, float *__restrict__ psi_v) {
  extern __shared__ float part[];            // [W][2 waves]
  const uint32_t nblk = (uint32_t)F * H;
  const uint32_t lb = xcd_contiguous(blockIdx.x, nblk);
  if (lb >= nblk) return;
  const int f = lb / H, i = lb % H;
  constexpr int R = K / 2;
  const int T = H * W + S;
  const uint16_t *frame = x + ((size_t)f * T + S) * C;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i0 = max(i - R, 0), i1 = min(i + R, H - 1);
  const int nrow = i1 - i0 + 1;
  for (int c0 = threadIdx.x * 8, pass = 0; c0 < (C + 1023) / 1024 * 1024; c0 += 1024, ++pass) {
    const bool on = c0 < C;                  // every thread walks every pass: part[] is per wave
    float s1[K][8], s2[K][8];                // column partials of the last K columns; slot = column % K
#pragma unroll
    for (int u = 0; u < K; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) s1[u][e] = s2[u][e] = 0.f;
    // Sums are taken of x - pivot, the pivot being the frame's first patch token: the variance
    // does not change, and a channel that sits at a large offset (mean >> spread) no longer loses
    // its spread in the rounding of E[x^2] - E[x]^2.
    const u32x4 pbits = on ? *(const u32x4 *)(frame + c0) : u32x4{0u, 0u, 0u, 0u};
    const float pv[8] = {bf16_lo(pbits.x), bf16_hi(pbits.x), bf16_lo(pbits.y), bf16_hi(pbits.y),
                         bf16_lo(pbits.z), bf16_hi(pbits.z), bf16_lo(pbits.w), bf16_hi(pbits.w)};
    // the K tokens of a column are requested one column ahead of their use
    auto load_col = [&](int jj, u32x4(&w)[K]) {
#pragma unroll
      for (int a = 0; a < K; ++a) {          // rows outside the grid read as the pivot: they add nothing
        const int ii = i - R + a;
        w[a] = pbits;
        if (on && jj < W && ii >= i0 && ii <= i1) w[a] = *(const u32x4 *)(frame + ((size_t)ii * W + jj) * C + c0);
      }
    };
    u32x4 wcur[K], wnext[K];
    load_col(0, wcur);
    for (int jb = 0; jb < W + R; jb += K) {
#pragma unroll
      for (int u = 0; u < K; ++u) {
        const int jj = jb + u;               // column entering the window; output column is jj - R
        load_col(jj + 1, wnext);
        float a1[8], a2[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) a1[e] = a2[e] = 0.f;
#pragma unroll
        for (int a = 0; a < K; ++a) {        // (the pivot beyond the row end)
          const float v[8] = {bf16_lo(wcur[a].x), bf16_hi(wcur[a].x), bf16_lo(wcur[a].y), bf16_hi(wcur[a].y),
                              bf16_lo(wcur[a].z), bf16_hi(wcur[a].z), bf16_lo(wcur[a].w), bf16_hi(wcur[a].w)};
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float dlt = v[e] - pv[e];
            a1[e] += dlt;
            a2[e] = __builtin_fmaf(dlt, dlt, a2[e]);
          }
        }
#pragma unroll
        for (int a = 0; a < K; ++a) wcur[a] = wnext[a];
#pragma unroll
        for (int e = 0; e < 8; ++e) {        // columns beyond the row end enter as zeros of x - pivot
          s1[u][e] = a1[e];
          s2[u][e] = a2[e];
        }
        const int j = jj - R;
        if (j >= 0 && j < W) {
          const int j0 = max(j - R, 0), j1 = min(j + R, W - 1);
          const float inv_cnt = 1.0f / (float)(nrow * (j1 - j0 + 1));
          float tot = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float t1 = 0.f, t2 = 0.f;
#pragma unroll
            for (int q = 0; q < K; ++q) {
              t1 += s1[q][e];
              t2 += s2[q][e];
            }
            const float m = t1 * inv_cnt;
            tot += __builtin_fmaf(-m, m, t2 * inv_cnt);
          }
          tot = wave_sum(tot);
          if (lane == 0) part[j * 2 + wave] = (pass ? part[j * 2 + wave] : 0.f) + tot;
        }
      }
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < W; j += blockDim.x)
    psi_v[((size_t)f * H + i) * W + j] = (part[j * 2] + part[j * 2 + 1]) / (float)C;
}

// ---------------------------------------------------------------------------------
// Psi_v for the 3 x 3 window, every token row read once (plus a one-column halo on each side
// of a strip).  A workgroup (2 waves, lane = 8 channels, wave = 512 channels) owns a strip of
// kSeg grid columns of one frame and walks down the grid rows.  When row i arrives the window
// sums of output row i - 1 follow from
//   sum_c var_c = (1/n) sum_window e  -  (1/n^2) sum_c (sum_window d_c)^2,
// d = x - (the frame's first patch token), e = sum_c d_c^2 of one token: only the first moment
// needs per-channel window sums, the second moment is a window sum of one number per token.
// Per column the lane keeps d of row i-1 and the pair sum d(i-1) + d(i-2) in fp32, so every
// token is widened once: vertical sum = d(i) + pair, then pair <- d(i) + d(i-1); the horizontal
// 3-sum slides over the strip's columns.  Cells outside the grid are fed as the pivot token
// (d = 0) and n counts the cells inside.  The bits of row i+2 are requested into a column's
// registers as soon as that column of row i has been widened.
// A strip is a chain of one memory round trip after the other, about 1.7 us per row, so short
// sequences, whose strips do not fill the 1024 workgroup slots, cut the rows into segments, each
// with one more row read on either side (var_row_segments; 63 -> 36 us for 32 frames of 37 x 37,
// 25 -> 9 for 2 of 16 x 16).  Whole strips are a kernel of their own (SEG false): with the bounds of a
// segment in registers 1000 frames took 800 us, without them 760.
// ---------------------------------------------------------------------------------
constexpr int kSeg = 4;                        // (wave_sum4)
constexpr int kVarWaves = 2;                   // waves per workgroup: 512 channels each, 8 per lane

// Sums of four values over the 64 lanes, with DPP moves and permlane swaps only: butterflies inside the rows of 16 lanes, then rows
// change places so that one addition serves two values, and four.  Value q ends up in all lanes of row q.  (One after the other each value's six steps
// waited for one another, 42 idle slots in two grid rows, and a move or a lane read each: importance of 32 frames of
// 37 x 37, C = 1024, 54.7 -> 51.7 us, 60 of 16 x 16, C = 512, 26.9 -> 25.3, 100 of 37 x 37 138.6 -> 133.8, 1000 1213 -> 1172.
// The pivot kept out of the fetches that do not need it, 12 % fewer instructions, loses 4 % there to the branches.)
__device__ __forceinline__ float wave_sum4(float (&v)[4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] += dpp_take<0xB1, 0xF>(v[q]);    // quad_perm [1,0,3,2]
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] += dpp_take<0x4E, 0xF>(v[q]);    // quad_perm [2,3,0,1]
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] += dpp_take<0x141, 0xF>(v[q]);   // row_half_mirror
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] += dpp_take<0x140, 0xF>(v[q]);   // row_mirror
  float t[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {              // rows 0 + 1 and 2 + 3: of v[2p] in rows 0 and 2, of v[2p + 1] in rows 1 and 3
    const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[2 * p]), __float_as_uint(v[2 * p + 1]), false, false);
    t[p] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
  }
  const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(t[0]), __float_as_uint(t[1]), false, false);
  return __uint_as_float(y[0]) + __uint_as_float(y[1]);
}

// STRIPS (SEG only): strips of the workgroup, `block` STRIPS + 0, 1, ..., two waves each; they walk one number of rows.
template <bool SEG, int STRIPS>
__device__ __forceinline__ void var_strip(
    const uint16_t *__restrict__ x, int F, int H, int W, int S, int C, int nseg, int row_segs,
    float *__restrict__ psi_v, uint32_t block) {
  constexpr int NC = kSeg + 2;               // columns a strip reads: its own and one on each side
  __shared__ float comb_[STRIPS][2][kVarWaves][kSeg]; // the waves' partial sums of a grid row, by row parity
  const int strip = STRIPS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * kVarWaves));
  auto &comb = comb_[strip];
  if constexpr (!SEG) row_segs = 1;
  const uint32_t nblk = (uint32_t)F * row_segs * nseg;
  uint32_t lb = STRIPS == 1 ? xcd_contiguous(block, nblk) : block * STRIPS + strip;   // neighbouring strips share an L2
  const bool spare = lb >= nblk;             // (of several: goes through the motions of the last one)
  if (STRIPS == 1 && spare) return;
  if (spare) lb = nblk - 1;
  const int fr = lb / nseg, j0 = (int)(lb % nseg) * kSeg;
  const int f = fr / row_segs, rs = fr % row_segs;
  // output rows [r0, r1), and the grid rows that are read
  const int r0 = SEG ? (int)((int64_t)H * rs / row_segs) : 0, r1 = SEG ? (int)((int64_t)H * (rs + 1) / row_segs) : H;
  const int ib = SEG ? max(r0 - 1, 0) : 0, row_end = SEG ? min(r1 + 1, H) : H;
  // of several strips one number, at least r1 + 1 - ib of each (a whole strip has no row ahead of it)
  const int steps = STRIPS == 1 ? r1 + 1 - ib : (H + row_segs - 1) / row_segs + (row_segs > 1 ? 2 : 1);
  const int wave = (threadIdx.x >> 6) % kVarWaves, lane = threadIdx.x & 63;
  const int T = H * W + S;
  const uint16_t *frame = x + ((size_t)f * T + S) * C;
  float *out = psi_v + (size_t)f * H * W;
  const float inv_c = 1.0f / (float)C;
  for (int cbase = 0; cbase < C; cbase += 512 * kVarWaves) {
    const int c0 = cbase + wave * 512 + lane * 8;
    const bool on = c0 < C;
    const u32x4 pbits = on ? *(const u32x4 *)(frame + c0) : u32x4{0u, 0u, 0u, 0u};
    const float pv[8] = {bf16_lo(pbits.x), bf16_hi(pbits.x), bf16_lo(pbits.y), bf16_hi(pbits.y),
                         bf16_lo(pbits.z), bf16_hi(pbits.z), bf16_lo(pbits.w), bf16_hi(pbits.w)};
    u32x4 raw[2][NC];                          // bits of rows i and i+1, by row parity; a column's
                                               // registers are refilled with row i+2 once used
    float d1[NC][8], pair[NC][8];              // d(i-1) and d(i-1) + d(i-2) per column
    float e1[NC], epair[NC];                   // the same for this lane's share of e
    auto fetch = [&](int i, int a, u32x4 &dst) {   // column a of the strip in grid row i, or the pivot
      const int jj = j0 - 1 + a;
      dst = pbits;
      if (on && i < row_end && jj >= 0 && jj < W) dst = *(const u32x4 *)(frame + ((size_t)i * W + jj) * C + c0);
    };
#pragma unroll
    for (int a = 0; a < NC; ++a) {
      fetch(ib, a, raw[0][a]);
      fetch(ib + 1, a, raw[1][a]);
      e1[a] = epair[a] = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) d1[a][e] = pair[a][e] = 0.f;
    }
    auto step = [&](auto parity, int i) {      // grid row i arrives, output row i - 1 leaves
      u32x4(&rw)[NC] = raw[decltype(parity)::value];
      const int io = i - 1;
      const int nrow = min(io + 1, H - 1) - max(io - 1, 0) + 1;
      const float inv_r = nrow == 3 ? (1.0f / 3.0f) : nrow == 2 ? 0.5f : 1.0f;
      float v0[8], v1[8], v2[8];               // vertical sums of the last three columns
      float ve0 = 0.f, ve1 = 0.f, ve2 = 0.f;
      float res[kSeg];
#pragma unroll
      for (int e = 0; e < 8; ++e) v0[e] = v1[e] = v2[e] = 0.f;
#pragma unroll
      for (int a = 0; a < NC; ++a) {
        const u32x4 w = rw[a];
        const float xv[8] = {bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y),
                             bf16_lo(w.z), bf16_hi(w.z), bf16_lo(w.w), bf16_hi(w.w)};
        fetch(i + 2, a, rw[a]);
        float e_new = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {          // slide: columns a - 2, a - 1 stay
          v0[e] = v1[e];
          v1[e] = v2[e];
          const float dn = xv[e] - pv[e];
          e_new = __builtin_fmaf(dn, dn, e_new);
          v2[e] = dn + pair[a][e];
          pair[a][e] = dn + d1[a][e];
          d1[a][e] = dn;
        }
        ve0 = ve1;
        ve1 = ve2;
        ve2 = e_new + epair[a];
        epair[a] = e_new + e1[a];
        e1[a] = e_new;
        if (a >= 2) {                          // output column j0 + a - 2
          const int jo = j0 + a - 2;
          const int ncol = min(jo + 1, W - 1) - max(jo - 1, 0) + 1;
          const float inv_n = (ncol == 3 ? (1.0f / 3.0f) : ncol == 2 ? 0.5f : 1.0f) * inv_r;   // scalar work
          float sq = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float h = v0[e] + v1[e] + v2[e];
            sq = __builtin_fmaf(h, h, sq);
          }
          const float m2 = (ve0 + ve1 + ve2) * inv_n;
          res[a - 2] = __builtin_fmaf(-sq * inv_n, inv_n, m2);
        }
      }
      // every lane holds its 8 channels' share of the strip's kSeg outputs of row io
      float r = wave_sum4(res);                // output q in row q of 16 lanes
      const int par = SEG ? decltype(parity)::value : i & 1;
      if ((lane & 15) == 0) comb[par][wave][lane >> 4] = r;
      __syncthreads();
      if (wave == 0 && lane < kSeg && io >= r0 && io < r1 && j0 + lane < W && !spare) {
        r = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < kVarWaves; ++w2) r += comb[par][w2][lane];
        r *= inv_c;
        float *o = out + (size_t)io * W + j0 + lane;
        *o = cbase ? *o + r : r;
      }
    };
    // rows ib .. r1; row H is a row of pivots that flushes output row H - 1 (a step beyond r1 sees
    // pivots only and writes nothing)
    for (int i = ib; i < ib + steps; i += 2) {
      step(std::integral_constant<int, 0>{}, i);
      step(std::integral_constant<int, 1>{}, i + 1);
    }
    __syncthreads();                           // comb is reused by the next channel pass
  }
}

template <bool SEG>
__global__ __launch_bounds__(64 * kVarWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_var_map3(
    const uint16_t *__restrict__ x, int F, int H, int W, int S, int C, int nseg, int row_segs,
    float *__restrict__ psi_v) {
  var_strip<SEG, 1>(x, F, H, W, S, C, nseg, row_segs, psi_v, blockIdx.x);
}

// Both maps of a short sequence in one launch, side by side: workgroups of 256 threads, first the strips, two each, then the
// patch rows.  While all of them are on the chip at once (two per CU) the gradient map costs next to nothing beside the
// variance map: with the fusion, apart and like this, us, 2 frames of 16 x 16, C = 256 15.0 and 12.1, 8 of them 16.9 and 12.3,
// 2 of 37 x 37, C = 1024 (444 workgroups) 20.3 and 16.9.  Beyond, the strips' 250 registers leave the patch rows too few waves:
// 588 workgroups 20.9 and 22.5, 1024 18.7 and 20.1, 100 frames of 37 x 37 143 and 160 at best, in any order of the two.
constexpr int kBothStrips = 2, kBothThreads = 64 * kVarWaves * kBothStrips;
template <typename PixT>
__global__ __launch_bounds__(kBothThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_both_maps(
    const PixT *__restrict__ img, int patch, float *__restrict__ psi_g, const uint16_t *__restrict__ x, int F, int H, int W, int S,
    int C, int nseg, int row_segs, float *__restrict__ psi_v, int strip_blocks) {
  extern __shared__ f32x4 luma4[];
  if ((int)blockIdx.x < strip_blocks) var_strip<true, kBothStrips>(x, F, H, W, S, C, nseg, row_segs, psi_v, blockIdx.x);
  else grad_rows<PixT, true, 8>(img, F, H, W, patch, psi_g, blockIdx.x - strip_blocks, luma4);
}

// Row segments per strip: rounds of 1024 workgroups (256 CUs, 2 waves per SIMD, 2 waves each), a
// segment costing its rows, the two rows around them and about two rows' time to start.
static int var_row_segments(int64_t strips, int H) {
  int best = 1;
  int64_t best_cost = 0;
  for (int k = 1; k <= H && k <= 64; ++k) {
    const int64_t cost = (strips * k + 1023) / 1024 * ((H + k - 1) / k + (k > 1 ? 2 : 0) + 2);
    if (k == 1 || cost < best_cost) {
      best = k;
      best_cost = cost;
    }
  }
  return best;
}

int launch_maps(const void *images, int img_dtype, const uint16_t *x, const Dims &d, int patch, int pool, float *psi_g, float *psi_v,
                hipStream_t st) {
  const int Wi = d.W * patch, nseg = (d.W + kSeg - 1) / kSeg;
  const size_t pix = img_dtype == LV_IMG_F32 ? 4 : 1, lds = ((size_t)(patch + 2) * Wi + Wi + 8) * sizeof(float);
  const bool vec = (size_t)d.H * patch * Wi % 4 == 0 && (uintptr_t)images % (4 * pix) == 0;
  const int64_t strips = (int64_t)d.F * nseg, rows = (int64_t)d.F * d.H;
  const int row_segs = var_row_segments(strips, d.H);
  const int64_t strip_blocks = (strips * row_segs + kBothStrips - 1) / kBothStrips, row_blocks = (int64_t)align_up((size_t)rows, kXcd);
  int dev = 0, n_cu = 0;   // (launch_grad_map has the limit of image rows)
  const bool can = pool == 3 && vec && lds <= 64 * 1024;
  if (can && (hipGetDevice(&dev) != hipSuccess ||
              hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess))
    return LV_ERR_HIP;
  if (!can || strip_blocks + row_blocks > 2 * n_cu) {
    if (int rc = launch_grad_map(images, img_dtype, d, patch, psi_g, st)) return rc;
    return launch_var_map(x, d, pool, psi_v, st);
  }
  const dim3 grid((unsigned)(strip_blocks + row_blocks));
  static std::atomic<uint64_t> lds_done[2];
  int rc;
#define LV_BOTH(T, I)                                                                                            \
  if ((rc = allow_dynamic_lds<64 * 1024>((const void *)k_both_maps<T>, lds_done[I]))) return rc;                   \
  hipLaunchKernelGGL((k_both_maps<T>), grid, dim3(kBothThreads), lds, st, (const T *)images, patch, psi_g, x, d.F, d.H, d.W, \
                     d.S, d.C, nseg, row_segs, psi_v, (int)strip_blocks)
  if (img_dtype == LV_IMG_F32) {
    LV_BOTH(float, 0);
  } else {
    LV_BOTH(uint8_t, 1);
  }
#undef LV_BOTH
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

int launch_var_map(const uint16_t *x, const Dims &d, int pool, float *psi_v, hipStream_t st) {
  if (pool == 3) {
    const int nseg = (d.W + kSeg - 1) / kSeg, row_segs = var_row_segments((int64_t)d.F * nseg, d.H);
    const dim3 grid((unsigned)align_up((size_t)d.F * row_segs * nseg, kXcd));
    if (row_segs > 1)
      hipLaunchKernelGGL(k_var_map3<true>, grid, dim3(64 * kVarWaves), 0, st, x, d.F, d.H, d.W, d.S, d.C, nseg, row_segs,
                         psi_v);
    else
      hipLaunchKernelGGL(k_var_map3<false>, grid, dim3(64 * kVarWaves), 0, st, x, d.F, d.H, d.W, d.S, d.C, nseg, 1, psi_v);
    LV_HIP_CHECK_LAUNCH();
    return LV_OK;
  }
  dim3 grid((unsigned)(align_up((size_t)d.F * d.H, kXcd)));
  size_t lds = (size_t)d.W * 2 * sizeof(float);
  switch (pool) {
    case 1:
      hipLaunchKernelGGL(k_var_map<1>, grid, dim3(128), lds, st, x, d.F, d.H, d.W, d.S, d.C, psi_v);
      break;
    case 5:
      hipLaunchKernelGGL(k_var_map<5>, grid, dim3(128), lds, st, x, d.F, d.H, d.W, d.S, d.C, psi_v);
      break;
    default:
      return LV_ERR_PARAM;
  }
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

// ---------------------------------------------------------------------------------
// Fusion: one workgroup per frame finds min/max of both maps, then writes
// alpha*norm(Psi_g) + beta*norm(Psi_v).
// ---------------------------------------------------------------------------------
// A frame is a few KB: while there are CUs to spare its latency counts (100 frames 5.5 -> 4.1 us with 16
// waves in place of 4), with more frames than CUs the launch of its waves (1000 frames 12.2 us against
// 9.5).  The number of waves is a template argument: as a launch parameter it cost the four waves 3 %
// (1000 frames 8.8 us, 8.5 like this).
constexpr int kFuseWavesFew = 16, kFuseWavesMany = 4;
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_ga_fuse(const float *__restrict__ psi_g,
                                                        const float *__restrict__ psi_v, int P,
                                                        float alpha, float beta,
                                                        float *__restrict__ score) {
  __shared__ float red[WAVES][4];
  const float *g = psi_g + (size_t)blockIdx.x * P, *v = psi_v + (size_t)blockIdx.x * P;
  float glo = INFINITY, ghi = -INFINITY, vlo = INFINITY, vhi = -INFINITY;
  for (int t = threadIdx.x; t < P; t += 64 * WAVES) {
    float a = g[t], b = v[t];
    glo = fminf(glo, a);
    ghi = fmaxf(ghi, a);
    vlo = fminf(vlo, b);
    vhi = fmaxf(vhi, b);
  }
  glo = wave_min(glo);
  ghi = wave_max(ghi);
  vlo = wave_min(vlo);
  vhi = wave_max(vhi);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
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
  const float gr = ghi - glo, vr = vhi - vlo;
  for (int t = threadIdx.x; t < P; t += 64 * WAVES) {
    score[(size_t)blockIdx.x * P + t] = ga_score(g[t], v[t], glo, gr, vlo, vr, alpha, beta);
  }
}

int launch_ga_fuse(const float *psi_g, const float *psi_v, const Dims &d, float alpha, float beta,
                   float *score, hipStream_t st) {
  if (d.F > 256)
    hipLaunchKernelGGL(k_ga_fuse<kFuseWavesMany>, dim3((unsigned)d.F), dim3(64 * kFuseWavesMany), 0, st, psi_g, psi_v, d.P,
                       alpha, beta, score);
  else
    hipLaunchKernelGGL(k_ga_fuse<kFuseWavesFew>, dim3((unsigned)d.F), dim3(64 * kFuseWavesFew), 0, st, psi_g, psi_v, d.P, alpha,
                       beta, score);
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

// Scores of the geometry-blind partitions (Sec. 3.2 "Naive Token Merging"): a fixed
// low-discrepancy pattern over the token index, or an independent hash per (frame, token).
// 24-bit values, exact in fp32.
__global__ __launch_bounds__(256) void k_naive_score(int F, int P, int policy, uint32_t seed,
                                                     float *__restrict__ score) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)F * P) return;
  const uint32_t f = (uint32_t)(idx / P), t = (uint32_t)(idx % P);
  uint32_t hsh;
  if (policy == LV_POLICY_FIXED) {
    hsh = (t + 1u) * 2654435769u;                 // multiplicative hash by 2^32 / golden ratio
  } else {
    hsh = seed ^ (f * 0x9E3779B9u) ^ (t * 0x85EBCA6Bu);
    hsh ^= hsh >> 16;                             // 32-bit finaliser of MurmurHash3
    hsh *= 0x85EBCA6Bu;
    hsh ^= hsh >> 13;
    hsh *= 0xC2B2AE35u;
    hsh ^= hsh >> 16;
  }
  score[idx] = (float)(hsh >> 8) * (1.0f / 16777216.0f);
}

int launch_naive_score(const Dims &d, int policy, uint32_t seed, float *score, hipStream_t st) {
  const int64_t n = (int64_t)d.F * d.P;
  hipLaunchKernelGGL(k_naive_score, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d.F, d.P,
                     policy, seed, score);
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

}  // namespace lv

// ---------------------------------------------------------------------------------
// Scratch for callers that cannot hand over a workspace (litevggt_importance_static): the
// variance map of one call lives in this file-scope device array.  Every GPU holds its own
// copy at its own address, so the address is looked up once per device, with that device
// current, and host code only ever uses the looked-up pointer (the array's name is a host-side
// stand-in, not a device address).
// ---------------------------------------------------------------------------------
namespace lv {

static __device__ __align__(256) float g_static_psi_v[kStaticScoreFloats];

int static_importance_scratch(float **out) {
  static std::atomic<float *> per_device[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return LV_ERR_HIP;
  if (dev < 0 || dev >= 64) return LV_ERR_HIP;
  float *p = per_device[dev].load(std::memory_order_acquire);
  if (!p) {
    void *sym = nullptr;
    if (hipGetSymbolAddress(&sym, HIP_SYMBOL(g_static_psi_v)) != hipSuccess || !sym) return LV_ERR_HIP;
    p = (float *)sym;
    per_device[dev].store(p, std::memory_order_release);   // the same value from every thread
  }
  *out = p;
  return LV_OK;
}

}  // namespace lv

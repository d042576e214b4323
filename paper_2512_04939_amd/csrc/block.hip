// The transformer block around the global attention core, on the merged sequence (Sec. 3.1:
// the aggregator's global layers are standard pre-norm attention + MLP blocks; the paper does
// not restate their details and there are no trained weights here, so the block is the plain
// one with synthetic weights):
//   h  = LN(z; g1, b1)                       q|k|v = h Wqkv^T + bqkv
//   a  = Attn(q, k, v)   (q, k RMS-normalised per head when qk_norm)
//   u1 = a Wo^T + bo                         h2 = LN(z + u1; g2, b2)
//   u2 = GELU(h2 W1^T + b1m) W2^T + b2m      delta = u1 + u2        (Block(z) = z + delta)
// Every intermediate is stored as bf16; the four linear layers run on one tiled MFMA kernel,
// with bf16 operands or (supplementary "FP8 Quantization Details") with FP8 E4M3 operands
// quantised per tensor, the input's scale taken from the tensor itself or from an 80-step amax
// history (delayed scaling).
#include "common.h"
#include "internal.h"

namespace lv {

// ---------------------------------------------------------------------------------------
// LayerNorm over the channel dimension, one wave per row, statistics in fp32 (two passes over
// registers: mean, then the centred sum of squares).  `add` (optional) is added to x first.
// ---------------------------------------------------------------------------------------
constexpr float kLnEps = 1e-6f;

// one row: lane holds the 16-byte pieces lane, lane + 64, ... of x (and of add); o = the normalised row
template <int CPL>
__device__ __forceinline__ void ln_row(const u32x4 (&w)[CPL], const u32x4 (&a)[CPL],
                                       const float *__restrict__ gamma, const float *__restrict__ beta,
                                       int lane, int nch, int C, u32x4 (&o)[CPL]) {
  float v[CPL][8];
  float sum = 0.f;
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const uint32_t uw[4] = {w[c].x, w[c].y, w[c].z, w[c].w}, ua[4] = {a[c].x, a[c].y, a[c].z, a[c].w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[c][2 * i] = bf16_lo(uw[i]) + bf16_lo(ua[i]);
      v[c][2 * i + 1] = bf16_hi(uw[i]) + bf16_hi(ua[i]);
      sum += v[c][2 * i] + v[c][2 * i + 1];
    }
  }
  const float mean = wave_sum_ordered(sum) / (float)C;
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < CPL; ++c)
    if (lane + 64 * c < nch)
#pragma unroll
      for (int i = 0; i < 8; ++i) ss += (v[c][i] - mean) * (v[c][i] - mean);
  const float rstd = 1.0f / sqrtf(wave_sum_ordered(ss) / (float)C + kLnEps);
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int ch = lane + 64 * c;
    o[c] = u32x4{0u, 0u, 0u, 0u};
    if (ch < nch) {
      const f32x4 g0 = ((const f32x4 *)gamma)[2 * ch], g1 = ((const f32x4 *)gamma)[2 * ch + 1];
      const f32x4 b0 = ((const f32x4 *)beta)[2 * ch], b1 = ((const f32x4 *)beta)[2 * ch + 1];
      o[c].x = pack_bf16((v[c][0] - mean) * rstd * g0[0] + b0[0], (v[c][1] - mean) * rstd * g0[1] + b0[1]);
      o[c].y = pack_bf16((v[c][2] - mean) * rstd * g0[2] + b0[2], (v[c][3] - mean) * rstd * g0[3] + b0[3]);
      o[c].z = pack_bf16((v[c][4] - mean) * rstd * g1[0] + b1[0], (v[c][5] - mean) * rstd * g1[1] + b1[1]);
      o[c].w = pack_bf16((v[c][6] - mean) * rstd * g1[2] + b1[2], (v[c][7] - mean) * rstd * g1[3] + b1[3]);
    }
  }
}

template <int CPL>
__device__ __forceinline__ void ln_load(const uint16_t *__restrict__ x, const uint16_t *__restrict__ add,
                                        int64_t row, int C, int lane, int nch, u32x4 (&w)[CPL], u32x4 (&a)[CPL]) {
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int ch = lane + 64 * c;
    w[c] = u32x4{0u, 0u, 0u, 0u};
    a[c] = u32x4{0u, 0u, 0u, 0u};
    if (ch < nch) {
      w[c] = ((const u32x4 *)(x + (size_t)row * C))[ch];
      if (add) a[c] = ((const u32x4 *)(add + (size_t)row * C))[ch];
    }
  }
}

template <int CPL>
__global__ __launch_bounds__(256) void k_layernorm(const uint16_t *__restrict__ x,
                                                   const uint16_t *__restrict__ add,
                                                   const float *__restrict__ gamma,
                                                   const float *__restrict__ beta, int64_t M, int C,
                                                   uint16_t *__restrict__ out) {
  const int lane = threadIdx.x & 63, nch = C >> 3;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  u32x4 w[CPL], a[CPL], o[CPL];
  ln_load<CPL>(x, add, row, C, lane, nch, w, a);
  ln_row<CPL>(w, a, gamma, beta, lane, nch, C, o);
#pragma unroll
  for (int c = 0; c < CPL; ++c)
    if (lane + 64 * c < nch) ((u32x4 *)(out + (size_t)row * C))[lane + 64 * c] = o[c];
}

// The same LayerNorm with the result written as a linear layer's activation operand (the
// fragment order k_pack_rows produces: [row / 32][k-step of 16 channels][lane = row % 32 + 32 *
// (second 8 of the 16)], 16 bytes each).  A workgroup owns the 32 rows of one fragment row, a
// wave 4 of them (their loads are all issued before the first row is reduced, and more waves
// per workgroup would leave a wave too few; 8 rows per wave and sums through LDS shuffles: 15.2 us
// for 5776 rows of 1024 channels in bf16, now 10.1; 38 for 15432 in FP8, now 20); the normalised
// rows meet in LDS (row stride C * 2 + 16 bytes: the 32 rows a wave reads back at one channel
// piece then lie in different banks) and leave as one contiguous run of 32 * C * 2 bytes.
// Rows beyond M are written as zeros.
//
// FP8: the normalised row (rounded to bf16, as if it had been stored) is quantised with the
// scale *inv to E4M3 codes and leaves in the FP8 operand order of k_quant_pack_fp8 (units of 32
// rows x 32 channels, lane h * 32 + r holds the 16 codes of channels 32u + 16h .. + 15 of row
// r); the largest |value| of the rows below M is kept for the history.  Row stride in LDS: C + 16 bytes.
constexpr int kLnWaves = 8;
// Row tile `tile`; FP8: quantised with r, the rows' largest |value| is returned in thread 0 (0 in bf16).
template <int CPL, bool FP8>
__device__ __forceinline__ float ln_packed_tile(const uint16_t *__restrict__ x, const uint16_t *__restrict__ add,
                                                const float *__restrict__ gamma, const float *__restrict__ beta, int64_t M, int C,
                                                int tile, u32x4 *__restrict__ packed, float r, u32x4 *ln_stage) {
  constexpr int kRows = 32 / kLnWaves;            // rows of a wave
  constexpr int RB = CPL <= 2 ? kRows : kRows / 2;   // rows whose loads are in flight together
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nch = C >> 3, stride = nch + 1;
  if constexpr (FP8) {
    const int stride8 = (C >> 3) + 2;   // u32x2 per row
    u32x2 *stage8 = (u32x2 *)ln_stage;
    float m = 0.f;
#pragma unroll 1
    for (int j0 = 0; j0 < kRows; j0 += RB) {
      u32x4 w[RB][CPL], a[RB][CPL];
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        const int64_t row = (int64_t)tile * 32 + wave * kRows + j0 + j;
        ln_load<CPL>(x, add, row < M ? row : 0, C, lane, row < M ? nch : 0, w[j], a[j]);
      }
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        const int rr = wave * kRows + j0 + j;
        u32x4 o[CPL];
        ln_row<CPL>(w[j], a[j], gamma, beta, lane, nch, C, o);
        const bool live = (int64_t)tile * 32 + rr < M;
#pragma unroll
        for (int c = 0; c < CPL; ++c)
          if (lane + 64 * c < nch) {
            if (live) m = fmaxf(m, absmax8(o[c]));
            stage8[rr * stride8 + lane + 64 * c] = live ? quant8(o[c], r) : u32x2{0u, 0u};
          }
      }
    }
    __shared__ float red[kLnWaves];
    m = wave_max(m);
    if (lane == 0) red[wave] = m;
    __syncthreads();
    const int pieces = 32 * (C >> 4);   // = (C / 32) units x 64 lanes
    for (int p = threadIdx.x; p < pieces; p += 64 * kLnWaves) {
      const int u = p >> 6, lp = p & 63;
      const u32x2 *src = stage8 + (lp & 31) * stride8 + 4 * u + 2 * (lp >> 5);
      const u32x2 lo = src[0], hi = src[1];
      packed[(size_t)tile * pieces + p] = u32x4{lo.x, lo.y, hi.x, hi.y};
    }
#pragma unroll
    for (int i = 0; i < kLnWaves; ++i) m = fmaxf(m, red[i]);
    return m;
  }
#pragma unroll 1
  for (int j0 = 0; j0 < kRows; j0 += RB) {
    u32x4 w[RB][CPL], a[RB][CPL];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      const int64_t row = (int64_t)tile * 32 + wave * kRows + j0 + j;
      ln_load<CPL>(x, add, row < M ? row : 0, C, lane, row < M ? nch : 0, w[j], a[j]);
    }
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      const int rr = wave * kRows + j0 + j;
      u32x4 o[CPL];
      ln_row<CPL>(w[j], a[j], gamma, beta, lane, nch, C, o);
      const bool live = (int64_t)tile * 32 + rr < M;
#pragma unroll
      for (int c = 0; c < CPL; ++c)
        if (lane + 64 * c < nch) ln_stage[rr * stride + lane + 64 * c] = live ? o[c] : u32x4{0u, 0u, 0u, 0u};
    }
  }
  __syncthreads();
  const int pieces = 32 * nch;   // = (C / 16) k-steps x 64 lanes
  for (int p = threadIdx.x; p < pieces; p += 64 * kLnWaves) {
    const int ks = p >> 6, lp = p & 63;
    packed[(size_t)tile * pieces + p] = ln_stage[(lp & 31) * stride + 2 * ks + (lp >> 5)];
  }
  return 0.f;
}

// what 32 rows take in LDS
static constexpr size_t ln_packed_lds(int C, bool fp8) { return fp8 ? (size_t)32 * (C / 8 + 2) * 8 : (size_t)32 * (C / 8 + 1) * 16; }

template <int CPL, bool FP8>
__global__ __launch_bounds__(64 * kLnWaves) void k_layernorm_packed(const uint16_t *__restrict__ x,
                                                          const uint16_t *__restrict__ add,
                                                          const float *__restrict__ gamma,
                                                          const float *__restrict__ beta, int64_t M, int C,
                                                          u32x4 *__restrict__ packed,
                                                          const uint32_t *__restrict__ inv,
                                                          uint32_t *__restrict__ amax) {
  extern __shared__ u32x4 ln_stage[];
  const float m = ln_packed_tile<CPL, FP8>(x, add, gamma, beta, M, C, blockIdx.x, packed, FP8 ? __uint_as_float(*inv) : 1.0f, ln_stage);
  if (FP8 && threadIdx.x == 0) raise_max(amax, m);
}

// packed: the result goes there in a linear layer's operand order (Mp rows, the ones beyond M
// zero) instead of to out; with fp8_inv / fp8_amax as E4M3 codes (scale *fp8_inv, the largest
// |value| reduced into *fp8_amax), else as bf16
static int launch_layernorm(const uint16_t *x, const uint16_t *add, const float *gamma,
                            const float *beta, int64_t M, int C, uint16_t *out, hipStream_t st,
                            u32x4 *packed = nullptr, int64_t Mp = 0, const uint32_t *fp8_inv = nullptr,
                            uint32_t *fp8_amax = nullptr) {
  const int cpl = (C / 8 + 63) / 64;
  if (C % 32 != 0 || cpl > 4) return LV_ERR_SHAPE;
  if (packed) {
    if (Mp % 32 != 0 || Mp < M || !fp8_inv != !fp8_amax) return LV_ERR_SHAPE;
    const size_t lds = ln_packed_lds(C, fp8_inv != nullptr);
    static std::atomic<uint64_t> lds_done[8];
    const unsigned grid = (unsigned)(Mp / 32);
    int rc;
#define LV_LNP(CPL, F8)                                                                                       \
  if ((rc = allow_dynamic_lds<ln_packed_lds(512 * CPL, F8)>((const void *)k_layernorm_packed<CPL, F8>, lds_done[(CPL - 1) * 2 + F8]))) \
    return rc;                                                                                                \
  hipLaunchKernelGGL((k_layernorm_packed<CPL, F8>), dim3(grid), dim3(64 * kLnWaves), lds, st, x, add, gamma, beta, M, C,  \
                     packed, fp8_inv, fp8_amax)
    if (fp8_inv) {
      switch (cpl) {
        case 1: LV_LNP(1, true); break;
        case 2: LV_LNP(2, true); break;
        case 3: LV_LNP(3, true); break;
        default: LV_LNP(4, true); break;
      }
    } else {
      switch (cpl) {
        case 1: LV_LNP(1, false); break;
        case 2: LV_LNP(2, false); break;
        case 3: LV_LNP(3, false); break;
        default: LV_LNP(4, false); break;
      }
    }
#undef LV_LNP
    LV_HIP_CHECK_LAUNCH();
    return LV_OK;
  }
  const unsigned grid = (unsigned)((M + 3) / 4);
#define LV_LN(CPL) \
  hipLaunchKernelGGL(k_layernorm<CPL>, dim3(grid), dim3(256), 0, st, x, add, gamma, beta, M, C, out)
  switch (cpl) {
    case 1: LV_LN(1); break;
    case 2: LV_LN(2); break;
    case 3: LV_LN(3); break;
    case 4: LV_LN(4); break;
    default: return LV_ERR_SHAPE;
  }
#undef LV_LN
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

// ---------------------------------------------------------------------------------------
// FP8 E4M3 operands.  Scalars of one linear layer (device memory, 8 words):
//   [0] amax of the input (bits of a non-negative float, reduced with atomic max)
//   [1] amax of the weight     [2] 448 / amax used for the input    [3] the same for the weight
//   [4] product of the two scales (what the accumulators are multiplied with)
// ---------------------------------------------------------------------------------------
constexpr int kFp8Words = 8;

// The workgroup's maximum of m, in thread 0
__device__ __forceinline__ float block_max4(float m, float (&red)[4]) {
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}
// amax of a bf16 tensor of n16 16-byte pieces
__global__ __launch_bounds__(256) void k_amax_bf16(const u32x4 *__restrict__ x, int64_t n16,
                                                   uint32_t *__restrict__ amax) {
  __shared__ float red[4];
  float m = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16;
       i += (int64_t)gridDim.x * blockDim.x)
    m = fmaxf(m, absmax8(x[i]));
  m = block_max4(m, red);
  if (threadIdx.x == 0) raise_max(amax, m);
}

// One wave: picks the scales of a layer from the tensors' own amax (current scaling; the weight's
// are in place already).
__global__ __launch_bounds__(64) void k_fp8_scales(uint32_t *__restrict__ sc) {
  if (threadIdx.x == 0) {
    const float ia = fp8_scale_inv(sc[0]), iw = __uint_as_float(sc[3]);
    sc[2] = __float_as_uint(ia);
    sc[4] = __float_as_uint((1.0f / ia) * (1.0f / iw));
  }
}

// Quantise rows 0..n-1 of a row-major [n, K] bf16 matrix with the scale in *inv and store them
// fragment-major for the FP8 MFMA: a unit (32 rows x 32 consecutive k, 1 KB) holds, in lane
// (h*32 + r), the 16 codes k = 32u + 16h .. + 15 of row r; an MFMA operand of 64 k is two
// units.  (Both operands use the same k order inside an operand, which is all a dot product
// needs.)  The byte layout equals that of the bf16 packing of a matrix with K/2 columns, so
// the tiled kernel fetches and reads both types the same way.  Rows n..n_pad-1 are zero.
// A wave writes whole units (1 KB stores) and takes the 4 units from s0 on of its 32 rows (256
// bytes of each bf16 row).  k_quant_pack_fp8's grid: (row tiles, ceil(units / 16)).
// amax != NULL: the largest |x| read is reduced into *amax on the way (delayed scaling needs
// it only afterwards, for the history, so no pass of its own).
// scale() is asked once the loads have been issued (a block's head reduces 96 or 128 maxima for it; ahead of them: whole blocks of 200
// rows with current scaling, C = 1536 122.5 us, now 119.5, 2048 146.7 and 143.5, of which the fewer registers in launch_block_head 0.5).
template <typename Scale>
__device__ __forceinline__ void quant_pack_units(const uint16_t *__restrict__ x, int n, int K, Scale scale, int t, int s0,
                                                 u32x4 *__restrict__ packed, uint32_t *__restrict__ amax) {
  const int KS = K >> 5;
  const int lane = threadIdx.x & 63, h = lane >> 5, rr = lane & 31;
  const int j = t * 32 + rr;
  u32x4 src[4][2];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    src[u][0] = src[u][1] = u32x4{0u, 0u, 0u, 0u};
    if (j < n && s0 + u < KS) {
      const u32x4 *p = (const u32x4 *)(x + (size_t)j * K) + 2 * ((s0 + u) * 2 + h);
      src[u][0] = p[0];
      src[u][1] = p[1];
    }
  }
  const float r = scale();
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (s0 + u < KS) {
      const u32x2 lo = quant8(src[u][0], r), hi = quant8(src[u][1], r);
      packed[((size_t)t * KS + s0 + u) * 64 + lane] = u32x4{lo.x, lo.y, hi.x, hi.y};
    }
  if (amax) {   // rows and units outside the matrix were read as zeros
    float m = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) m = fmaxf(m, fmaxf(absmax8(src[u][0]), absmax8(src[u][1])));
    __shared__ float red[4];
    m = block_max4(m, red);
    if (threadIdx.x == 0) raise_max(amax, m);
  }
}
__global__ __launch_bounds__(256) void k_quant_pack_fp8(const uint16_t *__restrict__ x, int n,
                                                        int K, const uint32_t *__restrict__ inv,
                                                        u32x4 *__restrict__ packed,
                                                        uint32_t *__restrict__ amax) {
  quant_pack_units(x, n, K, [&] { return __uint_as_float(*inv); }, blockIdx.x, (blockIdx.y * 4 + (threadIdx.x >> 6)) * 4, packed, amax);
}

// ---- The block's four weight matrices (qkv, output, MLP 1, MLP 2: 3C x C, C x C, 4C x C, C x 4C): their
// amaxes in one launch, 24 MB at C = 1024 (four launches took 78 us with one atomic per workgroup on one
// word, now about 8).
struct BlockWeights4 {
  const uint16_t *w[4];
  u32x4 *dst[4];
};
constexpr int kWAmaxUnit = 32;                     // workgroups per C x C elements of weights
constexpr int kWAmaxParts = 12 * kWAmaxUnit;       // partial maxima, layer by layer
__device__ __forceinline__ int weight_first_unit(int l) { return l == 0 ? 0 : l == 1 ? 3 : l == 2 ? 4 : l == 3 ? 8 : 12; }

__global__ __launch_bounds__(256) void k_weights_amax(BlockWeights4 bw, int C, uint32_t *__restrict__ partial) {
  __shared__ float red[4];
  const int unit = blockIdx.x / kWAmaxUnit, l = unit < 3 ? 0 : unit < 4 ? 1 : unit < 8 ? 2 : 3;
  const int u0 = weight_first_unit(l), n_wg = (weight_first_unit(l + 1) - u0) * kWAmaxUnit;
  const u32x4 *x = (const u32x4 *)bw.w[l];
  const int64_t n16 = (int64_t)(n_wg / kWAmaxUnit) * C * C / 8;
  float m = 0.f;
  for (int64_t i = (int64_t)((int)blockIdx.x - u0 * kWAmaxUnit) * 256 + threadIdx.x; i < n16; i += (int64_t)n_wg * 256 * 4) {
    u32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = i + (int64_t)u * n_wg * 256 < n16 ? x[i + (int64_t)u * n_wg * 256] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int u = 0; u < 4; ++u) m = fmaxf(m, absmax8(v[u]));
  }
  m = block_max4(m, red);
  if (threadIdx.x == 0) partial[blockIdx.x] = __float_as_uint(m);
}

// ---- The head of a block: what its first linear layer waits for, in one launch.  Workgroups by number: the
// first LayerNorm's row tiles (n_ln; the longest chain, so they start first), the weights on their way into operand
// order (n_pack; per weight (rows / 32) row tiles x ceil(k-steps / 32) groups, one weight after the other), and
// one for the layers' scalars (FP8) and for words that the attention needs cleared.  All three depend on inputs only: with FP8 a workgroup takes the scale it needs from
// the weights' partial maxima or the amax history itself.  Apart they were three launches one after the other that
// each left most of the chip waiting: C = 1024, us, 5,776 rows in bf16 10.9 + 10.3, now 16.4; 15,432 rows in E4M3
// 4.5 + 8.5 + 19.1, now 26.9; whole blocks of 394 rows in bf16 74.7 -> 70.0, in E4M3 (delayed scaling) 81.2 -> 73.6.
struct Fp8Head {
  uint32_t *sc;              // the four layers' scalars (8 words each)
  const float *state;        // amax histories (delayed scaling), or NULL: every input's scale is 1 for now
  uint32_t *wamax;           // the weights' amaxes: written (partial != NULL), or read
  const uint32_t *partial;   // the weights' partial maxima, or NULL
  uint32_t *ln_part;         // receives every row tile's largest |value| (the history's; no word to clear before)
};
struct ClearWords {          // what the attention (AttnKV) finds cleared
  uint32_t *at[2];
  int n[2];
};
__device__ __forceinline__ float weight_amax(const Fp8Head &hd, int l) {
  if (!hd.partial) return __uint_as_float(hd.wamax[l]);
  float m = 0.f;
  const int e = weight_first_unit(l + 1) * kWAmaxUnit;
  for (int i = weight_first_unit(l) * kWAmaxUnit + (threadIdx.x & 63); i < e; i += 64) m = fmaxf(m, __uint_as_float(hd.partial[i]));
  return wave_max(m);
}
// 448 / the largest recorded input amax of layer l (a history with nothing recorded yet gives 1)
__device__ __forceinline__ float history_inv(const Fp8Head &hd, int l) {
  if (!hd.state) return 1.0f;
  const float *hist = hd.state + (size_t)l * (LV_FP8_HISTORY + 2);
  const int lane = threadIdx.x & 63;
  return fp8_scale_inv(__float_as_uint(wave_max(fmaxf(hist[lane], lane + 64 < LV_FP8_HISTORY ? hist[lane + 64] : 0.f))));
}

template <int CPL, bool FP8>
__global__ __launch_bounds__(64 * kLnWaves) void k_block_head(const uint16_t *__restrict__ z, const float *__restrict__ gamma,
                                                              const float *__restrict__ beta, int64_t M, int C, int n_ln,
                                                              u32x4 *__restrict__ packed, BlockWeights4 bw, int n_pack, Fp8Head hd,
                                                              ClearWords cw) {
  extern __shared__ u32x4 ln_stage[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int b = blockIdx.x;
  if (b < n_ln) {
    const float m = ln_packed_tile<CPL, FP8>(z, nullptr, gamma, beta, M, C, b, packed, FP8 ? history_inv(hd, 0) : 1.0f, ln_stage);
    if (FP8 && threadIdx.x == 0) hd.ln_part[b] = __float_as_uint(m);
    return;
  }
  b -= n_ln;
  if (b < n_pack) {
    constexpr int kPer = 4 * kLnWaves;                                 // k-steps (units) of a workgroup
    const int g1 = (C / (FP8 ? 32 : 16) + kPer - 1) / kPer, g4 = (4 * C / (FP8 ? 32 : 16) + kPer - 1) / kPer;   // groups at K = C, 4C
    const int rt = C / 32;
    int l = 0;
    if (b >= 3 * rt * g1) b -= 3 * rt * g1, l = 1;
    if (l == 1 && b >= rt * g1) b -= rt * g1, l = 2;
    if (l == 2 && b >= 4 * rt * g1) b -= 4 * rt * g1, l = 3;
    const int groups = l == 3 ? g4 : g1, K = l == 3 ? 4 * C : C, t = b / groups, s0 = (b % groups * kLnWaves + wave) * 4;
    if constexpr (FP8) {
      quant_pack_units(bw.w[l], t * 32 + 32, K, [&] { return fp8_scale_inv(__float_as_uint(weight_amax(hd, l))); }, t, s0, bw.dst[l],
                       nullptr);
    } else {
      const int KS = K >> 4;
      const u32x4 *row = (const u32x4 *)(bw.w[l] + (size_t)(t * 32 + (lane & 31)) * K);
      u32x4 w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = s0 + u < KS ? row[(s0 + u) * 2 + (lane >> 5)] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (s0 + u < KS) bw.dst[l][((size_t)t * KS + s0 + u) * 64 + lane] = w[u];
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
    for (int i = threadIdx.x; i < cw.n[r]; i += 64 * kLnWaves) cw.at[r][i] = 0u;
  if constexpr (FP8) {
    if (wave < 4) {
      const float wm = weight_amax(hd, wave), ia = history_inv(hd, wave), iw = fp8_scale_inv(__float_as_uint(wm));
      if (lane == 0) {
        uint32_t *s = hd.sc + wave * kFp8Words;
        s[0] = 0u;
        s[1] = __float_as_uint(wm);
        s[2] = __float_as_uint(ia);
        s[3] = __float_as_uint(iw);
        s[4] = __float_as_uint((1.0f / ia) * (1.0f / iw));
        if (hd.partial) hd.wamax[wave] = __float_as_uint(wm);
      }
    }
  }
}

static int launch_block_head(const uint16_t *z, const float *gamma, const float *beta, int64_t M, int64_t Mp, int C, u32x4 *packed,
                             const BlockWeights4 *bw, bool fp8, const Fp8Head &hd, const AttnKV &kv, hipStream_t st) {
  // without a LayerNorm the form of the fewest registers: more waves stream the weights
  const int cpl = packed ? (C / 8 + 63) / 64 : 1;
  if (C % 32 != 0 || C > 2048 || Mp % 32 != 0 || Mp < M) return LV_ERR_SHAPE;
  const int per = (fp8 ? 32 : 16) * 4 * kLnWaves, n_ln = packed ? (int)(Mp / 32) : 0;
  const int n_pack = bw ? C / 32 * (8 * ((C + per - 1) / per) + (4 * C + per - 1) / per) : 0;
  const unsigned grid = (unsigned)(n_ln + n_pack + 1);
  const ClearWords cw = {{kv.clear[0], kv.clear[1]}, {kv.n_clear[0], kv.n_clear[1]}};
  const size_t lds = packed ? ln_packed_lds(C, fp8) : 0;
  static std::atomic<uint64_t> lds_done[8];
  const BlockWeights4 w4 = bw ? *bw : BlockWeights4{};
  int rc;
#define LV_HEAD(CPL, F8)                                                                                       \
  if ((rc = allow_dynamic_lds<ln_packed_lds(512 * CPL, F8)>((const void *)k_block_head<CPL, F8>, lds_done[(CPL - 1) * 2 + F8]))) \
    return rc;                                                                                                 \
  hipLaunchKernelGGL((k_block_head<CPL, F8>), dim3(grid), dim3(64 * kLnWaves), lds, st, z, gamma, beta, M, C, n_ln, packed, w4, n_pack, hd, cw)
#define LV_HEADS(F8)                   \
  switch (cpl) {                       \
    case 1: LV_HEAD(1, F8); break;     \
    case 2: LV_HEAD(2, F8); break;     \
    case 3: LV_HEAD(3, F8); break;     \
    default: LV_HEAD(4, F8); break;    \
  }
  if (fp8) {
    LV_HEADS(true)
  } else {
    LV_HEADS(false)
  }
#undef LV_HEADS
#undef LV_HEAD
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

// ---------------------------------------------------------------------------------------
// Y[M, Nout] = A[M, K] W[Nout, K]^T + bias (optionally GELU), bf16 in and out, fp32
// accumulation.  Output tiles of BM rows x BN columns, waves of 64 rows x BN / 2 columns; both
// operands come pre-packed fragment-major and are fetched straight into an LDS ring (2 k-steps
// per stage).  256 x 256: 8 waves, 4 stages, one workgroup per CU, 128 flop per fetched byte.
// 128 x 256 and 128 x 128: 4 waves, 3 and 4 stages, two workgroups per CU, whose epilogues run
// beside each other's main loops: for row counts that fill the chip badly with larger tiles
// (tile_shape).  KG = 2 (64 x 64, 128 x 128): two groups of waves with a ring each take half of K each and
// meet in LDS: for row counts that do not fill it at all (one tile per workgroup).  Bound by
// the matrix pipe and what keeps a wave from feeding it: issuing the fetches, the barrier, the
// fragment reads; the MFMAs alone take 70 % of the loop's time.  The finished tile goes from the accumulators straight to global
// memory (bias, optional GELU, one rounding to bf16); `addend` (optional, shaped like the
// output) is added to the rounded result on the way out.  The ring is free meanwhile, so the
// next tile's first stages are fetched during the epilogue.
// `split`: the output is Nout / split row-major blocks of [M, split] one after the other
// (split = Nout: one plain matrix; split = C for the fused q|k|v projection).
// PACKED: the output, through GELU, is the activation operand of a following layer with K = Nout and is
// written in that layer's operand order straight from the accumulators (bf16 fragments, or,
// with FP8, E4M3 codes quantised with *out_inv while the largest |value| goes to *out_amax).
// kQkvAmax, kQkvPacked (the fused q|k|v projection, whole heads of 64 channels): the epilogue holds the bf16 values that
// the attention's passes over q, k and v would read again, so it does their work: the amaxes that E4M3 attention scales
// by (a pass of 17.6 us at 15,432 x 1024 and a launch of 4.7 for its sums), or K and V in fragment order (9 us at 5,776 x 1024).  Same
// bits: values are rounded first, sums taken in the same order.  (k_attn_pack stays for q, k, v that come without the layer.)
// FP8: the same ring and the same byte traffic per stage, but a stage (two 1 KB units per
// fragment) is one k-step of 64 for v_mfma_f32_32x32x64_f8f6f4, whose operands are the two
// units of a fragment side by side in 8 registers: per stage a wave issues 8 MFMAs of twice
// the work.  `alpha` (FP8: the product of the two scales) multiplies the
// accumulators before the bias.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void lds_read1_async(u32x4 &dst, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1" : "=&v"(dst) : "v"(addr) : "memory");
}
constexpr int kTile = 256;                   // what rows are padded to and output channels are a multiple of
// Shape of a workgroup (KG = 2: of a K group) with tiles of BM rows x BN columns: (BM / 64) x 2 waves of 64 rows x
// BN / 2 columns.
template <int BM, int BN>
struct GemmShape {
  static constexpr int kWaves = BM / 32, kThreads = kWaves * 64;
  static constexpr int kB = BN / 64;                      // weight fragments of a wave per k-step (2 of activations)
  static constexpr int kFragW = BN / 32, kFragA = BM / 32;   // fragments of the tile per k-step
  static constexpr int kStageU4 = 2 * (kFragW + kFragA) * 64;   // [weights: 2 k-steps x kFragW | activations: 2 x kFragA][64 lanes]
  static constexpr int kStages = BM == 128 && BN == 256 ? 3 : 4;   // LDS ring: 128 KB, one workgroup per CU; 72 or 64 KB, two
  static constexpr int kLoads = 2 * (kFragW + kFragA) / kWaves;   // fragments a wave fetches per stage
  static constexpr int kLoadsW = kWaves == 8 ? kLoads : 2 * kFragW / kWaves;   // ... of these of the weights (8 waves: all or none)
  static constexpr size_t kLds = (size_t)kStages * kStageU4 * 16 + 2 * BN * sizeof(float);   // + two tiles' bias values
};

// GELU in its erf form, v * Phi(v) = max(v, 0) - |v| erfc(|v| / sqrt 2) / 2.  erfc by the rational-times-exponential form
// of Abramowitz & Stegun 7.1.26 (absolute error <= 1.5e-7, four orders below a bf16 step) with sqrt 2 and the
// half in its constants; the negative side uses erfc itself, so nothing cancels there.  The epilogue of the
// first MLP layer evaluates it 65536 times per tile, where it is as long as an E4M3 main loop: 12 VALU instructions and
// two transcendental ones (as v / 2 * (2 - erfc) with a select 17 and two; C = 1024, E4M3, the layer at M = 5,776 46.6 -> 39.7 us, 15,432 107 -> 99).  Against 64 bits on
// [-12, 12] at most 3.3e-7 off and 7.6e-8 rms, that form 4.2e-7 and 8.1e-8 (9 % of the points are further off, 26 % closer).  (|v| beyond 64, where the product is 0, is held there: infinity stays.)
__device__ __forceinline__ float gelu_erf(float v) {
  const float a = fminf(fabsf(v), 64.0f);
  const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.23164189f, a, 1.0f));
  float p = __builtin_fmaf(0.5307027145f, t, -0.7265760135f);
  p = __builtin_fmaf(p, t, 0.7107068705f);
  p = __builtin_fmaf(p, t, -0.142248368f);
  p = __builtin_fmaf(p, t, 0.127414796f);
  const float half_erfc = p * t * __builtin_amdgcn_exp2f(-0.72134752f * v * v);
  return __builtin_fmaf(-a, half_erfc, fmaxf(v, 0.f));
}

// What the block's last layer leaves behind under delayed scaling: the four layers' input amaxes go into their
// histories (a launch of their own took 4.5 us; every amax is known once the third layer has run).
struct Fp8Record {
  float *state = nullptr;             // NULL: nothing to record
  const uint32_t *sc = nullptr;       // layers 1 to 3: word 0
  const uint32_t *ln_part = nullptr;  // layer 0: n_part row tiles' maxima
  int n_part = 0;
};
__device__ __forceinline__ void record_amaxes(const Fp8Record &rec, int lane) {
  float m = 0.f;
  for (int i = lane; i < rec.n_part; i += 64) m = fmaxf(m, __uint_as_float(rec.ln_part[i]));
  m = wave_max(m);
  if (lane < 4) {
    float *hist = rec.state + (size_t)lane * (LV_FP8_HISTORY + 2);
    uint32_t *step = (uint32_t *)(hist + LV_FP8_HISTORY);
    hist[*step % LV_FP8_HISTORY] = lane == 0 ? m : __uint_as_float(rec.sc[lane * kFp8Words]);
    *step += 1;
  }
}

// max(m, |a|, |b|) in one instruction (written as fmaxf of fabsf, values taken from their bits are made canonical first)
__device__ __forceinline__ float max3_abs(float m, float a, float b) {
  float r;
  asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(r) : "v"(m), "v"(a), "v"(b));
  return r;
}

// What becomes of the output (see above): rows; the next layer's operand; q|k|v as rows with their amaxes taken; q as
// rows, K and V in the order the attention reads.
enum GemmOut { kRows, kOperand, kQkvAmax, kQkvPacked };
struct QkvOut {
  u32x4 *kp = nullptr, *vp = nullptr;
  uint32_t *amax = nullptr;
  int n_kt = 0, qk_norm = 0;
};

template <bool FP8, GemmOut OUT, int BM, int BN, int KG = 1>
__global__ __launch_bounds__((GemmShape<BM, BN>::kThreads * KG)) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_bt(
    const u32x4 *__restrict__ ap, const u32x4 *__restrict__ wp, int64_t M, int KS, int nt_n,
    const float *__restrict__ bias, int gelu, uint16_t *__restrict__ out, int split,
    const float *__restrict__ alpha_p, int n_tiles, int rows_by_xcd, const uint16_t *__restrict__ addend,
    const uint32_t *__restrict__ out_inv, uint32_t *__restrict__ out_amax, Fp8Record rec, QkvOut qkv) {
  using S = GemmShape<BM, BN>;
  constexpr bool PACKED = OUT == kOperand, QKV = OUT == kQkvAmax || OUT == kQkvPacked;
  static_assert(OUT != kQkvPacked || BM == BN, "V's tiles swap rows and columns");
  constexpr int kStages = S::kStages, kStageU4 = S::kStageU4, kB = S::kB;
  // 256 x 256: two groups of four waves, one wave of each on every SIMD, take turns.  One reads the fragments of its next
  // stage and fetches while the other's MFMAs run, a barrier ends both.  (All eight waves in step, reads, fetches and
  // MFMAs mixed as below: every wave of a SIMD waited for the same barrier and address unit at once, 1,450 cycles
  // per E4M3 stage of 1,024 MFMA cycles on a chip that is mostly idle, 1,250 in turns; on a full one the clock takes a part
  // back.)  The ring runs on from tile to tile: a tile's last stages fetch the next one's first, nothing is
  // drained between them.  us for qkv / out / MLP 1 / MLP 2, C = 1024, in step and in turns: E4M3, M = 15,432 62.0 26.8 102.6
  // 71.8, 58.6 26.5 96.2 67.8, 30,000 113 43.7 196 134, 111 41.1 181 125; bf16, 30,000 176 65.9 268 233, 165 62.1 251 221.
  constexpr bool kTurns = BM == 256 && BN == 256;
  constexpr bool kTwoSets = !kTurns && (!FP8 || kB <= 2);   // registers for two sets of weight fragments
  constexpr int kAhead = kTurns ? kStages - 1 : kStages;   // stages fetched ahead
  extern __shared__ u32x4 rings[];             // one ring per K group
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
  const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / S::kWaves;   // this wave's part of K
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) - kg * S::kWaves;
  u32x4 *const ring = rings + (size_t)kg * kStages * kStageU4;
  const int wd = wave % (BM / 64), wn = wave / (BM / 64);
  const int total = (KS >> 1) / KG;
  // persistent: one workgroup per CU walks the tiles (a workgroup owns a whole CU's LDS, so a
  // launch per tile would pay a dispatch between any two tiles of a CU)
  // Workgroup w runs on XCD w % 8.  An XCD takes the row tiles tm = x, x + 8, ..., so an
  // activation tile is fetched into one L2 only, and walks its tiles one group of G = 4 column
  // tiles after the other, row by row inside a group: the G weight tiles of a group (2 MB at
  // K = 1024) stay in that L2 meanwhile, and an activation tile is shared by G workgroups.  Its
  // workgroups take this list in turn, so they differ by one tile at most.  (Few rows: plain order.)
  const int nt_m = n_tiles / nt_n;
  const int xcd = blockIdx.x & (kXcd - 1);
  const bool by_xcd = rows_by_xcd != 0 && (gridDim.x & (kXcd - 1)) == 0;
  const int my_rows = by_xcd ? (nt_m - xcd + kXcd - 1) / kXcd : nt_m;   // row tiles of this XCD
  const int my_tiles = my_rows * nt_n, stride = by_xcd ? (int)gridDim.x >> 3 : (int)gridDim.x;
  const int n_group = my_rows * 4;                                     // tiles of a full column group
  auto tile_at = [&](int v, int &tm_, int &tn_) {                      // tile v of the list (v < my_tiles)
    if (by_xcd) {
      const int cg = v / n_group, in = v - cg * n_group, width = min(4, nt_n - cg * 4);
      tm_ = in / width * kXcd + xcd;
      tn_ = cg * 4 + in % width;
    } else {
      tm_ = v / nt_n;
      tn_ = v % nt_n;
    }
  };
  __shared__ uint32_t wg_amax;   // FP8 && PACKED: the largest |value| this workgroup has written
  if (FP8 && PACKED && tid == 0) wg_amax = 0u;   // (many barriers before its first use)
  __shared__ uint32_t qkv_amax[OUT == kQkvAmax ? 3 : 1];   // kQkvAmax: of q, k and v
  if (OUT == kQkvAmax && tid < 3) qkv_amax[tid] = 0u;
  __shared__ float half_head[QKV && kB == 1 ? 2 * 2 * 32 : 1];   // two waves share a head: their sums of squares
  bool primed = false;   // this tile's first stages have been issued by the previous tile('s epilogue)
  bool stored = false;   // kTurns: the previous tile has ended with at least kStores stores behind its last fetch
  constexpr int kStores = FP8 && PACKED ? 2 * kB : 4 * kB;
  // (kTurns: the scalars once for all tiles, nothing waits in an epilogue; else there, a short tile's first loads come first)
  float alpha = 1.0f, r = 1.0f;
  auto load_scalars = [&]() {
    if (alpha_p) alpha = *alpha_p;
    if constexpr (FP8 && PACKED) r = __uint_as_float(*out_inv);
  };
  if constexpr (kTurns) load_scalars();
  int parity = 0;
  int tm = 0, tn = 0, tm2 = 0, tn2 = 0;
  for (int v = by_xcd ? (int)blockIdx.x >> 3 : (int)blockIdx.x; v < my_tiles; v += stride, parity ^= 1) {
  tile_at(v, tm, tn);
  const bool more = v + stride < my_tiles;
  if (more) tile_at(v + stride, tm2, tn2);
  // this tile's bias values wait in LDS behind the ring (read in the epilogue, many barriers
  // later); two buffers in turn, so a wave still in the previous tile's epilogue reads its own
  float *bias_lds = (float *)(rings + (size_t)KG * kStages * kStageU4) + parity * BN;
  if (tid < BN) {                            // (whole waves; straight to LDS: nobody waits for it, nor for the stores before it)
    if (bias) __builtin_amdgcn_global_load_lds(bias + tn * BN + tid, bias_lds + (tid & ~63), 4, 0, 0);
    else bias_lds[tid] = 0.f;
  }

  // fetch: with 8 waves, waves 0-3 move 4 weight fragments of a stage each, waves 4-7 4 activation
  // fragments; with 4 waves each moves kB weight and 2 activation fragments
  const int f_ks = S::kWaves == 2 ? wave : (wave >> 1) & 1, f_half = S::kWaves == 2 ? 0 : wave & 1;
  int pf_g = 0, f_tm = tm, f_tn = tn;
  if (kTurns && primed) pf_g = kAhead;
  auto slot_of = [](int g) { return kStages == 4 ? g & 3 : g % kStages; };
  // kQkvPacked: the tiles of V take activations and weights the other way round, so that a lane has one channel of four
  // consecutive tokens per register group
  const int third = split / BN;
  auto swapped = [&](int t) { return OUT == kQkvPacked && t >= 2 * third; };
  const u32x4 *f_src[2];   // this wave's next weight and activation fragments (8 waves: [0] is either)
  u32x4 *f_dst[2];
  auto fetch_begin = [&]() {
    int s = pf_g < total ? pf_g : total - 1;   // past the end: the last stage again, into a free slot ...
    if (kTurns && pf_g >= total && more) {     // ... or the next tile's first ones
      s = pf_g - total;
      f_tm = tm2;
      f_tn = tn2;
    }
    const size_t at = (size_t)((kg * total + s) * 2 + f_ks) * 64;   // uniform: the lane is added in the load
    u32x4 *stage = ring + (size_t)slot_of(pf_g) * kStageU4;
    if constexpr (S::kWaves == 8) {
      const int a0 = (wave & 1) * 4;
      const bool second = swapped(f_tn) != (wave >> 2 != 0);   // the activations' fragments
      f_src[0] = (second ? ap + (size_t)(f_tm * 8 + a0) * KS * 64 : wp + (size_t)(f_tn * 8 + a0) * KS * 64) + at;
      f_dst[0] = stage + (size_t)(wave * 4) * 64;
    } else {
      const bool sw = swapped(f_tn);
      f_src[0] = (sw ? ap : wp) + (size_t)((sw ? f_tm : f_tn) * S::kFragW + f_half * kB) * KS * 64 + at;
      f_src[1] = (sw ? wp : ap) + (size_t)((sw ? f_tn : f_tm) * S::kFragA + f_half * 2) * KS * 64 + at;
      f_dst[0] = stage + (size_t)(wave * S::kLoadsW) * 64;
      f_dst[1] = stage + (size_t)(2 * S::kFragW + wave * 2) * 64;
    }
    ++pf_g;
  };
  auto fetch_one = [&](auto idx) {
    constexpr int i = decltype(idx)::value;
    constexpr int part = i >= S::kLoadsW ? 1 : 0, j = i - part * S::kLoadsW;
    if constexpr (i < S::kLoads)
      __builtin_amdgcn_global_load_lds(f_src[part] + (size_t)j * KS * 64 + lane, f_dst[part] + j * 64, 16, 0, 0);
  };
  auto fetch = [&]() {
    fetch_begin();
    fetch_one(std::integral_constant<int, 0>{});
    fetch_one(std::integral_constant<int, 1>{});
    fetch_one(std::integral_constant<int, 2>{});
    fetch_one(std::integral_constant<int, 3>{});
    fetch_one(std::integral_constant<int, 4>{});
    fetch_one(std::integral_constant<int, 5>{});
  };
  const uint32_t ring_lane = lds_addr(&ring[lane]);
  // byte offsets of this wave's fragments inside a stage, k-step 0, and from k-step 0 to k-step 1
  const uint32_t b_off = (uint32_t)((wn * kB) * 1024), a_off = (uint32_t)((2 * S::kFragW + wd * 2) * 1024);
  constexpr uint32_t b_ks = S::kFragW * 1024, a_ks = S::kFragA * 1024;
  u32x4 fb[kTwoSets ? 2 : 1][2][kB], fa[kTurns ? 1 : 2][2][2];   // [set][k-step (FP8: unit of 32)][fragment]
  auto read_frags = [&](int g, int ks, u32x4(&b)[kB], u32x4(&a)[2]) {
    const uint32_t base = ring_lane + (uint32_t)(slot_of(g) * kStageU4 * 16);
    if constexpr (kB == 4) lds_read4_async(b, base + b_off + ks * b_ks);
    else if constexpr (kB == 2) lds_read2_async(b, base + b_off + ks * b_ks);
    else lds_read1_async(b[0], base + b_off + ks * b_ks);
    lds_read2_async(a, base + a_off + ks * a_ks);
  };
  f32x16 acc[2][kB];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < kB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
  if (kTurns && primed) {
    // (landed: the last tile's last stage has waited for stage 0)
  } else if (primed) {
    pf_g = kAhead;
    // the stages were issued ahead of the previous epilogue's stores: wait for everything
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
#pragma unroll
    for (int i = 0; i < kAhead; ++i) fetch();                // the ring's stages
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kAhead - 1) * S::kLoads) : "memory");   // stage 0 has landed (this wave's part)
  }
  if (!kTurns || !primed) __builtin_amdgcn_s_barrier();
  // Steady state of the smaller tiles: all fragments of a stage are in registers while its MFMAs run, and those of the
  // next stage are read meanwhile: into a second set, a whole stage ahead of their use (bf16), or,
  // where the registers do not hold two sets of weight fragments beside the 8-register operands
  // (FP8), the activations into a second set and each weight fragment into its own registers once
  // its MFMAs have been issued.  The barrier, the reads and the fetch instructions, one or two at a
  // time (a wave that issues a stage's 4 or 6 back to back waits for the address unit, and its
  // MFMAs with it), sit between pairs of MFMAs, so that the MFMA pipe has queued work of this wave
  // while it does them.  (All of it behind the barrier at the head of a k-step: 1046 us for the qkv
  // layer at M = 143,232, C = 1024 in bf16, 900 like this.)
  auto wait_set = [&](u32x4(&b)[2][kB], u32x4(&a)[2][2]) {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(b[0][0]), "+v"(b[1][0]), "+v"(a[0][0]), "+v"(a[0][1]), "+v"(a[1][0]), "+v"(a[1][1])
                 :
                 : "memory");
    if constexpr (kB >= 2) asm volatile("" : "+v"(b[0][1]), "+v"(b[1][1]) : : "memory");
    if constexpr (kB == 4)
      asm volatile("" : "+v"(b[0][2]), "+v"(b[0][3]), "+v"(b[1][2]), "+v"(b[1][3]) : : "memory");
  };
  // the two MFMAs of column block bi: of k-step u, or (FP8) of both, whose units lie side by side
  auto pair = [&](const u32x4(&b)[2][kB], const u32x4(&a)[2][2], int u, int bi) {
#pragma unroll
    for (int ai = 0; ai < 2; ++ai) {
      if constexpr (FP8)
        acc[ai][bi] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(cat8(b[0][bi], b[1][bi]), cat8(a[0][ai], a[1][ai]),
                                                                      acc[ai][bi], 0, 0, 0, 0, 0, 0);
      else
        acc[ai][bi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[u][bi]),
                                                             __builtin_bit_cast(bf16x8, a[u][ai]), acc[ai][bi], 0, 0, 0);
    }
  };
  auto ld = [&](auto i) {
    __builtin_amdgcn_sched_barrier(0);
    fetch_one(i);
    __builtin_amdgcn_sched_barrier(0);
  };
#define LV_LD(i) ld(std::integral_constant<int, i>{})
  auto stage = [&](int g, u32x4(&bc)[2][kB], u32x4(&ac)[2][2], u32x4(&bn)[2][kB], u32x4(&an)[2][2]) {
    __builtin_amdgcn_sched_barrier(0);
    wait_set(bc, ac);
    if constexpr (kTwoSets) pair(bc, ac, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kStages - 2) * S::kLoads) : "memory");   // stage g+1 has landed; later ones may be in flight
    __builtin_amdgcn_s_barrier();                            // and nobody reads stage g from LDS any more
    __builtin_amdgcn_sched_barrier(0);
    // stage g + kStages goes to the slot of stage g; past the end the reads get a stale slot, never used
    if constexpr (!kTwoSets) {
      const uint32_t base = ring_lane + (uint32_t)(slot_of(g + 1) * kStageU4 * 16);
      auto again = [&](int bi) {                             // the next stage's weight fragment bi
        __builtin_amdgcn_sched_barrier(0);
        lds_read1_async(bn[0][bi], base + b_off + bi * 1024);
        lds_read1_async(bn[1][bi], base + b_ks + b_off + bi * 1024);
      };
      lds_read2_async(an[0], base + a_off);
      lds_read2_async(an[1], base + a_ks + a_off);
      fetch_begin();
      LV_LD(0);
      pair(bc, ac, 0, 0);
      again(0);
      LV_LD(1);
      pair(bc, ac, 0, 1);
      again(1);
      LV_LD(2); LV_LD(4);
      pair(bc, ac, 0, 2);
      again(2);
      LV_LD(3); LV_LD(5);
      pair(bc, ac, 0, 3);
      again(3);
    } else if constexpr (FP8) {                              // kB <= 2
      read_frags(g + 1, 0, bn[0], an[0]);
      read_frags(g + 1, 1, bn[1], an[1]);
      fetch_begin();
      LV_LD(0); LV_LD(1);
      if constexpr (kB == 2) pair(bc, ac, 0, 1);
      LV_LD(2); LV_LD(3);
    } else if constexpr (kB == 1) {
      read_frags(g + 1, 0, bn[0], an[0]);
      read_frags(g + 1, 1, bn[1], an[1]);
      fetch_begin();
      LV_LD(0); LV_LD(1);
      pair(bc, ac, 1, 0);
      LV_LD(2); LV_LD(3);
    } else {
      pair(bc, ac, 0, 1);
      __builtin_amdgcn_sched_barrier(0);
      read_frags(g + 1, 0, bn[0], an[0]);
      fetch_begin();
      LV_LD(0);
      if constexpr (kB == 4) {
        pair(bc, ac, 0, 2);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(g + 1, 1, bn[1], an[1]);
        __builtin_amdgcn_sched_barrier(0);
        pair(bc, ac, 0, 3);
        LV_LD(1);
        pair(bc, ac, 1, 0);
        LV_LD(2);
        pair(bc, ac, 1, 1);
        LV_LD(3);
        pair(bc, ac, 1, 2);
        LV_LD(4);
        pair(bc, ac, 1, 3);
        LV_LD(5);
      } else {
        pair(bc, ac, 1, 0);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(g + 1, 1, bn[1], an[1]);
        LV_LD(1);
        pair(bc, ac, 1, 1);
        LV_LD(2); LV_LD(3);
      }
    }
  };
#undef LV_LD
  if constexpr (kTurns) {
    const bool late = wave >= 4;             // this group is one barrier behind the other; level again in the epilogue,
    if (late) __builtin_amdgcn_s_barrier();  // where both at once hide each other's latencies
    // A stage: [reads of stage g, fetch of stage g + 3 into the slot of g - 1 | barrier | its MFMAs | barrier].  Both groups
    // have read stage g - 1 by then: the late one in the turn before.
    auto turn = [&](int g, auto younger) {
      __builtin_amdgcn_sched_barrier(0);
      read_frags(g, 0, fb[0][0], fa[0][0]);
      read_frags(g, 1, fb[0][1], fa[0][1]);
      fetch();
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * S::kLoads + decltype(younger)::value) : "memory");   // stage g+1 has landed
      wait_set(fb[0], fa[0]);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int u = 0; u < (FP8 ? 1 : 2); ++u)
#pragma unroll
        for (int b = 0; b < kB; ++b) pair(fb[0], fa[0], u, b);
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
    };
    int g = 0;
    if (stored) {                            // the last tile's stores may still be on their way
      turn(0, std::integral_constant<int, kStores>{});
      turn(1, std::integral_constant<int, kStores>{});
      g = 2;
    }
    for (; g < total; ++g) turn(g, std::integral_constant<int, 0>{});
    if (!late) __builtin_amdgcn_s_barrier();
  } else {
  read_frags(0, 0, fb[0][0], fa[0][0]);
  read_frags(0, 1, fb[0][1], fa[0][1]);
  constexpr int kSetB = kTwoSets ? 1 : 0;   // the weight set of odd stages
  for (int g = 0; g < total; g += 2) {       // (an even number of stages in each K group: K is a multiple of 256)
    stage(g, fb[0], fa[0], fb[kSetB], fa[1]);
    stage(g + 1, fb[kSetB], fa[1], fb[0], fa[0]);
  }
  // the reads issued by the last stage are waited for before their registers die
  wait_set(fb[0], fa[0]);
  wait_set(fb[kSetB], fa[1]);
  }
  if constexpr (!kTurns) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // nothing may land in LDS any more
    __syncthreads();
  }
  // Two K groups trade sums through their rings: group kg finishes row block a = kg, group 0's sum first.
  auto mine = [&](int a) { return KG == 1 || a == kg; };
  if constexpr (KG == 2) {
    auto at = [&](int from, int b, int g) {
      return (f32x4 *)(rings + (size_t)from * kStages * kStageU4) + (size_t)((wave * kB + b) * 4 + g) * 64 + lane;
    };
#pragma unroll
    for (int a = 0; a < 2; ++a)
      if (a != kg)                           // (uniform: one copy runs)
#pragma unroll
        for (int b = 0; b < kB; ++b)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            *at(kg, b, g) = f32x4{acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2], acc[a][b][4 * g + 3]};
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 2; ++a)
      if (a == kg)
#pragma unroll
        for (int b = 0; b < kB; ++b)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 x = *at(1 - a, b, g);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[a][b][4 * g + i] += x[i];
          }
  }

  // Epilogue: bias, activation, bf16, straight from the accumulators to global memory; nothing
  // goes through LDS, so the next tile's first stages are issued first and land while the
  // arithmetic runs.  The weights are the first MFMA operand, so a lane holds one token (column)
  // and, per group of four accumulator registers, four consecutive output channels 8g + 4h .. + 3:
  // lanes l and l + 32 trade halves (one v_permlane32_swap per register pair: the first operand's
  // lanes 32-63 against the second operand's lanes 0-31), after which lane l has channels 0-7 and
  // lane l + 32 channels 8-15 of a run of 16, 16 bytes per lane.
  if constexpr (!kTurns) load_scalars();
  int anchor = 0;   // opaque zero: keeps the address arithmetic below inside this tile's epilogue
  asm volatile("" : "+v"(anchor));   // (hoisted out of the tile loop it would stay live through the main loop)
  if (kTurns) {
    primed = true;
    stored = (int64_t)(tm + 1) * BM <= M;
  } else if (KG == 1 && more) {
    f_tn = tn2;
    f_tm = tm2;
    pf_g = 0;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) fetch();
    primed = true;
  } else {
    primed = false;
  }
  if constexpr (PACKED) {
    // The output is the next linear layer's activation operand and is written in that kernel's
    // fragment order: out[(row / 32) * KSn + k-step][lane], where a k-step is 16 of this layer's
    // output channels and lane = row % 32 + 32 * (second 8 of the 16), which is exactly what the
    // lanes hold after the swap: a wave stores 1 KB in a row.
    if constexpr (FP8) {
      // E4M3 codes for an FP8 layer with K = Nout (units of 32 rows x 32 channels, lane h * 32 + r
      // holds the 16 codes of channels 32u + 16h .. + 15 of row r): every value is rounded to
      // bf16 as if it had been stored, then scaled by *out_inv; a lane has one dword of four codes
      // per register group g, lanes l and l + 32 trade groups 2, 3 against groups 0, 1.  The
      // largest |value| of the rows below M goes into *out_amax; the tile's rows beyond M are written as zeros.
      const int KSn = nt_n * (BN / 32);
      u32x4 *op = (u32x4 *)out + ((size_t)(tm * S::kFragA + wd * 2) * KSn + tn * (BN / 32) + wn * kB) * 64 + lane + anchor;
      float m = 0.f;
#pragma unroll
      for (int b = 0; b < kB; ++b)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          if (!mine(a)) continue;
          uint32_t keep = (int64_t)tm * BM + wd * 64 + 32 * a + (lane & 31) < M ? ~0u : 0u;
          asm volatile("" : "+v"(keep));     // (a mask: as a condition it becomes a branch around every four values)
          uint32_t d[4];
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 bv = *(const f32x4 *)(bias_lds + wn * 32 * kB + 32 * b + 8 * g + 4 * h);
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = gelu_erf(acc[a][b][4 * g + i] * alpha + bv[i]);
            const uint32_t p0 = pack_bf16(v[0], v[1]) & keep, p1 = pack_bf16(v[2], v[3]) & keep;
            m = max3_abs(m, bf16_lo(p0), bf16_hi(p0));
            m = max3_abs(m, bf16_lo(p1), bf16_hi(p1));
            d[g] = cvt4_fp8(clamp448(bf16_lo(p0) * r), clamp448(bf16_hi(p0) * r), clamp448(bf16_lo(p1) * r), clamp448(bf16_hi(p1) * r));
          }
          const auto s0 = __builtin_amdgcn_permlane32_swap(d[0], d[2], false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(d[1], d[3], false, false);
          op[((size_t)a * KSn + b) * 64] = u32x4{s0[0], s0[1], s1[0], s1[1]};
        }
      m = wave_max(m);
      if (lane == 0) atomicMax(&wg_amax, __float_as_uint(m));   // in LDS; once per workgroup to memory
      continue;
    }
    const int KSn = nt_n * (BN / 16);
    u32x4 *op = (u32x4 *)out + ((size_t)(tm * S::kFragA + wd * 2) * KSn + tn * (BN / 16) + wn * 2 * kB) * 64 + lane + anchor;
#pragma unroll
    for (int b = 0; b < kB; ++b)
#pragma unroll
      for (int gp = 0; gp < 2; ++gp) {
        const int ch0 = wn * 32 * kB + 32 * b + 16 * gp + 4 * h;
        const f32x4 bv0 = *(const f32x4 *)(bias_lds + ch0), bv1 = *(const f32x4 *)(bias_lds + ch0 + 8);
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          if (!mine(a)) continue;
          float v0[4], v1[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v0[i] = gelu_erf(acc[a][b][8 * gp + i] + bv0[i]);
            v1[i] = gelu_erf(acc[a][b][8 * gp + 4 + i] + bv1[i]);
          }
          // first operand's lanes 32-63 <-> second operand's lanes 0-31
          const auto s0 = __builtin_amdgcn_permlane32_swap(pack_bf16(v0[0], v0[1]), pack_bf16(v1[0], v1[1]), false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(pack_bf16(v0[2], v0[3]), pack_bf16(v1[2], v1[3]), false, false);
          op[((size_t)a * KSn + 2 * b + gp) * 64] = u32x4{s0[0], s1[0], s0[1], s1[1]};
        }
      }
    continue;
  }
  // row-major rows of `split` channels: per store instruction a wave writes 32 bytes of each of
  // 32 rows; the four stores that complete a 128-byte line follow each other
  const int blk = (tn * BN) / split, col0 = (tn * BN) % split;   // a tile never straddles two blocks
  if constexpr (QKV) {
    const int n_tok = tm * BM, ch_tile = col0 + anchor;
    if (OUT == kQkvPacked && blk == 2) {
      // V, rows and columns swapped: lane h * 32 + dr holds channel 32 dt + dr and, per 16 keys u, the 8 keys 16u + 8 (e / 4) +
      // 4h + e % 4 of a tile: a fragment of the attention's V operand as it stands
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        if (!mine(a)) continue;
        const int ch = wd * 64 + 32 * a;
        const float bv = bias_lds[ch + (lane & 31)];
        const size_t head = (size_t)(ch_tile + ch) >> 6;
#pragma unroll
        for (int b = 0; b < kB; ++b) {
          const int kt = (n_tok + wn * 32 * kB + 32 * b) >> 5;
          if (kt >= qkv.n_kt) continue;
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
              w[i] = FP8 ? pack_bf16(acc[a][b][8 * u + 2 * i] * alpha + bv, acc[a][b][8 * u + 2 * i + 1] * alpha + bv)
                         : pack_bf16(acc[a][b][8 * u + 2 * i] + bv, acc[a][b][8 * u + 2 * i + 1] + bv);
            qkv.vp[((head * qkv.n_kt + kt) * 4 + u * 2 + (ch >> 5 & 1)) * 64 + lane] = u32x4{w[0], w[1], w[2], w[3]};
          }
        }
      }
      continue;
    }
    // q and k (and v as rows): a lane has 8 channels of its token per chunk of 16, lane l + 32 the other 8; kB column blocks
    // are whole heads, or (kB = 1) half of one
    constexpr int kHeads = kB == 1 ? 1 : kB / 2, kChunks = kB == 1 ? 2 : 4;   // of a wave, and of a (part of a) head
    float top = 0.f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int j = 0; j < kHeads; ++j) {
        u32x4 t[kChunks];
        float ss = 0.f;
        const int64_t m = (int64_t)n_tok + wd * 64 + 32 * a + (lane & 31);
        if (mine(a)) {
#pragma unroll
          for (int s = 0; s < kChunks; ++s) {
            const int b = j * 2 + (s >> 1), gp = s & 1;
            const int ch0 = wn * 32 * kB + 32 * b + 16 * gp + 4 * h;
            const f32x4 bv0 = *(const f32x4 *)(bias_lds + ch0), bv1 = *(const f32x4 *)(bias_lds + ch0 + 8);
            float v0[4], v1[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              v0[i] = FP8 ? acc[a][b][8 * gp + i] * alpha + bv0[i] : acc[a][b][8 * gp + i] + bv0[i];
              v1[i] = FP8 ? acc[a][b][8 * gp + 4 + i] * alpha + bv1[i] : acc[a][b][8 * gp + 4 + i] + bv1[i];
            }
            const auto s0 = __builtin_amdgcn_permlane32_swap(pack_bf16(v0[0], v0[1]), pack_bf16(v1[0], v1[1]), false, false);
            const auto s1 = __builtin_amdgcn_permlane32_swap(pack_bf16(v0[2], v0[3]), pack_bf16(v1[2], v1[3]), false, false);
            t[s] = u32x4{s0[0], s1[0], s0[1], s1[1]};
          }
          // the sum of a head row's squares, as k_attn_pack takes it: chunks of 8, added in pairs
          float pair_sum[kChunks];
#pragma unroll
          for (int s = 0; s < kChunks; ++s) {
            const float cs = sumsq8(t[s]);
            const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(cs), __float_as_uint(cs), false, false);
            pair_sum[s] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
          }
          ss = pair_sum[0] + pair_sum[1];
          if constexpr (kB > 1) ss += pair_sum[2] + pair_sum[3];
        }
        if constexpr (kB == 1) {             // (KG = 2: row block a is K group a's; the two waves of a group share its rows)
          if (j == 0 && mine(a)) half_head[(kg * 2 + wn) * 32 + (lane & 31)] = ss;
          __syncthreads();
          if (mine(a)) ss = half_head[kg * 64 + (lane & 31)] + half_head[kg * 64 + 32 + (lane & 31)];
        }
        if (!mine(a)) continue;
        const float r = qkv.qk_norm && blk < 2 ? 1.0f / sqrtf(ss * (1.0f / 64.0f) + kQkEps) : 1.0f;
        if (OUT == kQkvPacked && blk == 1) {
          const int64_t kt = m >> 5;         // (the same for all lanes)
          const size_t head = (size_t)(ch_tile + wn * 32 * kB + 64 * j) >> 6;
          if (kt < qkv.n_kt) {
#pragma unroll
            for (int s = 0; s < kChunks; ++s) {
              const int step = s + (kB == 1 ? 2 * wn : 0);
              const u32x4 w = qkv.qk_norm ? scale8(t[s], r) : t[s];
              qkv.kp[((head * qkv.n_kt + kt) * 4 + step) * 64 + lane] = m < M ? w : u32x4{0u, 0u, 0u, 0u};
            }
          }
          continue;
        }
        if (OUT == kQkvAmax && m < M) {      // rounding keeps the order, so the largest is rounded alone
          float big = 0.f;
#pragma unroll
          for (int s = 0; s < kChunks; ++s) big = fmaxf(big, absmax8(t[s]));
          top = fmaxf(top, bf16_lo(pack_bf16(big * r, 0.f)));
        }
        if (m < M)
#pragma unroll
          for (int s = 0; s < kChunks; ++s)
            *(u32x4 *)(out + (size_t)blk * M * split + ch_tile + wn * 32 * kB + 64 * j + 16 * s + 8 * h + (size_t)m * split) = t[s];
      }
    if constexpr (OUT == kQkvAmax) {
      top = wave_max(top);
      if (lane == 0) atomicMax(&qkv_amax[blk], __float_as_uint(top));
    }
    continue;
  }
  uint16_t *ob = out + (size_t)blk * M * split + col0 + wn * 32 * kB + 8 * h + anchor;
#pragma unroll
  for (int b = 0; b < kB; ++b)
#pragma unroll
    for (int gp = 0; gp < 2; ++gp) {
      const int ch0 = wn * 32 * kB + 32 * b + 16 * gp + 4 * h;
      const f32x4 bv0 = *(const f32x4 *)(bias_lds + ch0), bv1 = *(const f32x4 *)(bias_lds + ch0 + 8);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        if (!mine(a)) continue;
        float v0[4], v1[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v0[i] = FP8 ? acc[a][b][8 * gp + i] * alpha + bv0[i] : acc[a][b][8 * gp + i] + bv0[i];
          v1[i] = FP8 ? acc[a][b][8 * gp + 4 + i] * alpha + bv1[i] : acc[a][b][8 * gp + 4 + i] + bv1[i];
        }
        if (gelu) {                          // (one branch for eight values)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v0[i] = gelu_erf(v0[i]);
            v1[i] = gelu_erf(v1[i]);
          }
        }
        const auto s0 = __builtin_amdgcn_permlane32_swap(pack_bf16(v0[0], v0[1]), pack_bf16(v1[0], v1[1]), false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(pack_bf16(v0[2], v0[3]), pack_bf16(v1[2], v1[3]), false, false);
        u32x4 t = u32x4{s0[0], s1[0], s0[1], s1[1]};
        const int64_t m = (int64_t)tm * BM + wd * 64 + 32 * a + (lane & 31);
        if (addend) {   // out = addend + (this layer's output, already rounded to bf16): one more rounding
          const u32x4 y = m < M ? *(const u32x4 *)(addend + (ob - out) + (size_t)m * split + 32 * b + 16 * gp)
                                : u32x4{0u, 0u, 0u, 0u};
          t.x = pack_bf16(bf16_lo(t.x) + bf16_lo(y.x), bf16_hi(t.x) + bf16_hi(y.x));
          t.y = pack_bf16(bf16_lo(t.y) + bf16_lo(y.y), bf16_hi(t.y) + bf16_hi(y.y));
          t.z = pack_bf16(bf16_lo(t.z) + bf16_lo(y.z), bf16_hi(t.z) + bf16_hi(y.z));
          t.w = pack_bf16(bf16_lo(t.w) + bf16_lo(y.w), bf16_hi(t.w) + bf16_hi(y.w));
        }
        if (m < M) *(u32x4 *)(ob + (size_t)m * split + 32 * b + 16 * gp) = t;
      }
    }
  }   // tiles
  if constexpr (kTurns) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may land in LDS once the workgroup has ended
  if constexpr (FP8 && PACKED) {
    __syncthreads();
    if (tid == 0) raise_max(out_amax, __uint_as_float(wg_amax));
  }
  if constexpr (OUT == kQkvAmax) {
    __syncthreads();
    if (tid < 3 && qkv_amax[tid] != 0u) raise_max(qkv.amax + tid, __uint_as_float(qkv_amax[tid]));
  }
  if constexpr (FP8 && OUT == kRows)
    if (rec.state && blockIdx.x == gridDim.x - 1 && tid < 64) record_amaxes(rec, lane);
}

// ---------------------------------------------------------------------------------------
struct BlockWs {
  uint16_t *h, *qkv, *a, *u1, *h3;
  u32x4 *apack, *wpack;
  uint32_t *fp8sc, *wpart;
  void *attn;
  size_t attn_bytes, bytes;
  int64_t Mp;
};

// the four weight matrices in operand order, one after the other (qkv, output, MLP 1, MLP 2),
// then a 256-byte tail for their four amaxes (FP8 layers)
size_t block_wpack_bytes(int C) { return align_up((size_t)12 * C * C * 2, 256) + 256; }

static BlockWs carve_block(int64_t M, int C, int heads, int attn_dtype, bool least, char *base) {
  BlockWs w;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char *p = base ? base + off : nullptr;
    off += align_up(bytes, 256);
    return p;
  };
  w.Mp = (int64_t)align_up((size_t)M, kTile);
  w.h = (uint16_t *)take((size_t)M * C * 2);
  w.qkv = (uint16_t *)take((size_t)3 * M * C * 2);
  w.a = (uint16_t *)take((size_t)M * C * 2);
  w.u1 = (uint16_t *)take((size_t)M * C * 2);
  w.h3 = (uint16_t *)take((size_t)w.Mp * 4 * C * 2);   // row-major (FP8 layers) or in fragment order (bf16 layers)
  w.apack = (u32x4 *)take((size_t)w.Mp * 4 * C);       // a layer's activation operand: bf16 with K = C, FP8 with K <= 4C
  w.wpack = (u32x4 *)take(block_wpack_bytes(C));
  w.fp8sc = (uint32_t *)take(4 * kFp8Words * sizeof(uint32_t));   // one set per linear layer
  w.wpart = (uint32_t *)w.h3;   // the weights' partial maxima, gone before the first MLP layer writes there
  w.attn_bytes = attn_ws_bytes(heads, M, attn_dtype, 1, least);
  w.attn = take(w.attn_bytes);
  w.bytes = off;
  return w;
}

size_t block_ws_bytes(int64_t M, int C, int heads, int attn_dtype, bool least) {
  return carve_block(M, C, heads, attn_dtype, least, nullptr).bytes;
}

// What a linear layer finds ready and what it leaves behind.
struct LinearOpts {
  bool fp8 = false;
  const u32x4 *a_packed = nullptr;     // the activation operand, already in operand order (then A is unused)
  // out receives the next layer's (K = Nout) operand instead of row-major rows: the rows of whole tiles (64,
  // 128 or 256 each), rows M and up undefined; the next layer may read up to Mp rows, into outputs it drops
  bool pack_out = false;
  const uint16_t *addend = nullptr;    // row-major, same shape as out: out = addend + result
  const u32x4 *w_packed = nullptr;     // the weight operand
  // FP8: this layer's scalars, prepared by k_block_head.  A, unless a_packed, is quantised with
  // sc[2] and its amax reduced into sc[0]; `current`: sc[2] and sc[4] are taken from that amax first
  uint32_t *sc = nullptr;
  bool current = false;
  const uint32_t *out_inv = nullptr;   // FP8 pack_out: the next layer's input scale ...
  uint32_t *out_amax = nullptr;        // ... and where the largest |output| is reduced into
  Fp8Record rec;                       // FP8, not pack_out: what to record once it has run
  const AttnKV *kv = nullptr;          // the q|k|v layer: do this for the attention, if the tiles' shape allows it ...
  bool *kv_done = nullptr;             // ... and tell whether it was
};

// Which output tile suits M rows and Nout columns: 256 x 256 (one workgroup per CU), 128 x 256 or
// 128 x 128 (two), by estimated time in units of a 256 x 256 tile's on one CU (24-36 us at K = 1024).
// Whole rounds of workgroups cost 0.97, 1.03 and 0.6 (smaller tiles fetch 1.5 and 2 times as much into
// LDS per product); what is left over costs less where every CU gets one at most, and less still
// where it is the only round.  Fitted to (C = 1024, bf16, us for the layers qkv / out / MLP 1 / MLP 2)
//   M =    394: 25 24 29 75   19 16 21 50   13 12 15 32        M =  9000: 62 29 100  92   65 30  81  97   62 27  85  92
//   M =   2200: 28 24 33 77   22 18 32 52   20 12 34 36        M = 15432: 99 36 143 116  100 35 139 119  112 38 159 133
//   M =   5776: 54 27 66 83   43 19 54 59   42 19 58 56        M = 143232: 890 282 1183 1015  952 311 1242 1172
// with the three tiles in that order, and the first one's waves in step.  In turns (k_gemm_bt) it takes, M = 3000, 9000, 15432, 30000:
//   bf16   29 23 33 72   61 28 95 86   94 35 134 116   175 63 254 222     E4M3   21 16 27 42   39 19 70 50   59 25 96 67   110 40 181 124
// (128 x 256 in E4M3: 23 14 27 36   42 20 57 56   61 23 96 73   112 44 170 139).  E4M3 through GELU, whose epilogue is half as long as the
// tile's loop: two workgroups per CU run one's beside the other's loop, so there the whole tile keeps its 1.
// Over 23 sizes (C = 512, 768, 1024, M = 3,000 to 30,000) the choice is 0.6 % (bf16) and 0.8 % (E4M3) above the best of the three.
// Where even the 128 x 128 tiles leave CUs idle, what counts is how long one workgroup is at a tile: it
// gets 16 KB per stage at 150 GB/s and pays the barrier of every stage.  64 x 64 tiles in two K groups halve both, as
// long as all of them are on the chip at once (two per CU); longer rows (K >= 2048 in bf16) gain from two K groups of 128 x 128
// tiles, one per CU.  us for qkv / out / MLP 1 / MLP 2, 128 x 128 and as chosen:
//   M =  394: 11.2 10.7 13.8 30.9    9.8 6.4 11.0 14.9      M = 2200: 19.8 12.2 33.7 36.5   (the same) (the same) (the same) 31.6
//   M = 1000: 12.2 11.2 14.5 30.9   (the same) 7.7 (the same) 16.7     E4M3, M = 394: 8.5 8.4 13.4 19.6    7.4 5.4 8.9 9.8
// (64 x 64 without groups 22.6 for MLP 2 at M = 394, 128 x 128 with them 25.7, 64 x 64 in four groups 14.7.)
// Whole blocks with and without the 64 x 64 tiles, bf16 and E4M3 layers (delayed scaling), us: C = 256, where the output layers take them
// up to 8,192 rows: M = 394 42.6 and 53.4, 55.9 and 65.3; 2048 55.6 and 64.8, 73.7 and 79.7; 4096 69.7 and 74.9, 87.2 and 92.5;
// 8192 131.2 and 133.6, E4M3 level.  C = 512: 1000 61.9 and 73.1, 72.8 and 80.8; 4096 112.4 and 114.3, 124.7 and 126.7.
enum TileShape { kTile256x256, kTile128x256, kTile128x128, kTile128x128K2, kTile64x64K2 };
static TileShape tile_shape(int64_t M, int Nout, int K, bool fp8, bool gelu, int n_cu) {
  if ((M + 63) / 64 * (Nout / 64) <= 2 * n_cu) return kTile64x64K2;
  if (!fp8 && K >= 2048 && (M + 127) / 128 * (Nout / 128) <= n_cu) return kTile128x128K2;
  int64_t rest = 0;
  const auto rounds = [&](int bm, int bn, int slots) {   // full rounds (of the XCD with the most tiles), and what is left
    const int64_t nt_m = (M + bm - 1) / bm, nt_n = Nout / bn, tiles = nt_m * nt_n;
    if (tiles <= slots) {
      rest = tiles;
      return (int64_t)0;
    }
    const int64_t per = (nt_m + kXcd - 1) / kXcd * nt_n, s = slots / kXcd > 0 ? slots / kXcd : 1;
    rest = per % s * kXcd;
    return per / s;
  };
  const int64_t r256 = rounds(256, 256, n_cu);
  const double round256 = fp8 && gelu ? 1.0 : 0.97, only256 = fp8 && gelu ? 1.0 : 0.85;
  const double t256 = round256 * (double)r256 + (rest == 0 ? 0.0 : r256 ? round256 : only256);
  const int64_t r128 = rounds(128, 256, 2 * n_cu);
  const double t128 = 1.03 * (double)r128 + (rest == 0 ? 0.0 : rest > n_cu ? 1.03 : r128 ? 0.55 : 0.72);
  const int64_t r64 = rounds(128, 128, 2 * n_cu);
  const double more = rest > n_cu ? (double)(rest - n_cu) / n_cu : 0.0;
  const double t64 = 0.6 * (double)r64 + (rest == 0 ? 0.0 : r64 ? (rest > n_cu ? 0.6 : 0.3) : rest > n_cu ? 0.64 + 0.1 * more : 0.48);
  return t64 < t128 && t64 < t256 ? kTile128x128 : t128 < t256 ? kTile128x256 : kTile256x256;
}

// Y = A W^T + bias: brings the activation into operand order where it is not yet (FP8: quantised,
// current scaling after taking its amax), then the tiled kernel.
static int launch_linear(const uint16_t *A, int64_t M, int K, int Nout,
                         const float *bias, int gelu, uint16_t *out, int split, BlockWs &w,
                         hipStream_t st, const LinearOpts &o) {
  if (!o.w_packed || (o.fp8 && !o.sc) || (o.current && (o.a_packed || o.pack_out))) return LV_ERR_PARAM;
  if (o.pack_out && (!gelu || o.addend || split != Nout || (o.fp8 && (!o.out_inv || !o.out_amax)))) return LV_ERR_PARAM;
  if (o.kv && (o.pack_out || o.addend || gelu || Nout != 3 * split)) return LV_ERR_PARAM;
  if (K % 256 != 0 || Nout % kTile != 0 || split % kTile != 0 || Nout % split != 0) return LV_ERR_SHAPE;
  int rc;
  if (w.Mp / 128 * (Nout / 128) >= ((int64_t)1 << 30) || w.Mp >= ((int64_t)1 << 31)) return LV_ERR_SHAPE;
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
    return LV_ERR_HIP;
  const TileShape shape = tile_shape(M, Nout, K, o.fp8, gelu != 0, n_cu);
  QkvOut qkv;
  if (o.kv) qkv = QkvOut{(u32x4 *)o.kv->kp, (u32x4 *)o.kv->vp, o.kv->amax, o.kv->n_kt, o.kv->qk_norm};
  auto gemm = [&](auto fp8, auto kind, auto bm, auto bn, auto kg, const u32x4 *act, int KS, const float *alpha) -> int {
    constexpr bool F8 = decltype(fp8)::value;
    constexpr GemmOut PK = decltype(kind)::value;
    constexpr int BM = decltype(bm)::value, BN = decltype(bn)::value, KG = decltype(kg)::value;
    using S = GemmShape<BM, BN>;
    constexpr size_t kLds = S::kLds + (KG - 1) * (size_t)S::kStages * S::kStageU4 * 16;
    static std::atomic<uint64_t> lds_done{0};
    if (int rc2 = allow_dynamic_lds<kLds>((const void *)k_gemm_bt<F8, PK, BM, BN, KG>, lds_done)) return rc2;
    const int nt_m = (int)((M + BM - 1) / BM), nt_n = Nout / BN, n_tiles = nt_m * nt_n;
    const int slots = n_cu * (KG == 1 ? 256 / BM : BM == 64 ? 2 : 1);   // KG = 2: tile_shape() leaves one tile per workgroup
    // One round only: row tiles still go to one XCD each (M = 5776, K = 4096: 69 us dealt out in
    // plain order, 56 like this) unless the fullest XCD would then have more than its share of CUs or slots.
    const int fullest = (nt_m + kXcd - 1) / kXcd * nt_n, share = (n_tiles <= n_cu ? n_cu : slots) / kXcd;
    const bool by_xcd = n_tiles > slots || (nt_m >= 2 * kXcd && fullest <= share);
    const unsigned grid = (unsigned)(n_tiles > slots ? slots : by_xcd ? fullest * kXcd : n_tiles);
    hipLaunchKernelGGL((k_gemm_bt<F8, PK, BM, BN, KG>), dim3(grid), dim3(S::kThreads * KG), kLds, st, act,
                       o.w_packed, M, KS, nt_n, bias, gelu, out, split, alpha, n_tiles, by_xcd ? 1 : 0, o.addend, o.out_inv,
                       o.out_amax, o.rec, qkv);
    return LV_OK;
  };
  auto launch = [&](auto fp8, const u32x4 *act, int KS, const float *alpha) -> int {
    using N128 = std::integral_constant<int, 128>;
    using N256 = std::integral_constant<int, 256>;
    using N64 = std::integral_constant<int, 64>;
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    auto tiles = [&](auto kind) -> int {
      if (shape == kTile64x64K2) return gemm(fp8, kind, N64{}, N64{}, Two{}, act, KS, alpha);
      if (shape == kTile128x128K2) return gemm(fp8, kind, N128{}, N128{}, Two{}, act, KS, alpha);
      if (shape == kTile128x128) return gemm(fp8, kind, N128{}, N128{}, One{}, act, KS, alpha);
      if constexpr (decltype(kind)::value != kQkvPacked)
        if (shape == kTile128x256) return gemm(fp8, kind, N128{}, N256{}, One{}, act, KS, alpha);
      return gemm(fp8, kind, N256{}, N256{}, One{}, act, KS, alpha);
    };
    const bool kv = o.kv && (o.kv->amax || shape != kTile128x256);
    if (o.kv_done) *o.kv_done = kv;
    if (kv && o.kv->amax) return tiles(std::integral_constant<GemmOut, kQkvAmax>{});
    if (kv) return tiles(std::integral_constant<GemmOut, kQkvPacked>{});
    if (o.pack_out) return tiles(std::integral_constant<GemmOut, kOperand>{});
    return tiles(std::integral_constant<GemmOut, kRows>{});
  };
  const u32x4 *a_packed = o.a_packed;
  if (o.fp8) {
    uint32_t *const sc = o.sc;
    if (!a_packed) {
      if (o.current) {   // the tensor's own amax first
        const int64_t n16 = M * (K / 8);
        const unsigned g = (unsigned)(((n16 + 255) / 256) < 1024 ? ((n16 + 255) / 256) : 1024);
        hipLaunchKernelGGL(k_amax_bf16, dim3(g), dim3(256), 0, st, (const u32x4 *)A, n16, sc);
        hipLaunchKernelGGL(k_fp8_scales, dim3(1), dim3(64), 0, st, sc);
      }
      hipLaunchKernelGGL(k_quant_pack_fp8, dim3((unsigned)(w.Mp / 32), (unsigned)((K / 32 + 15) / 16)), dim3(256), 0, st, A, (int)M,
                         K, (const uint32_t *)(sc + 2), w.apack, o.current ? (uint32_t *)nullptr : sc);
      a_packed = w.apack;
    }
    if ((rc = launch(std::true_type{}, a_packed, K / 32, (const float *)(sc + 4)))) return rc;
  } else {
    if (!a_packed) {
      if ((rc = launch_pack_rows(A, M, w.Mp, K, w.apack, st))) return rc;
      a_packed = w.apack;
    }
    if ((rc = launch(std::false_type{}, a_packed, K / 16, nullptr))) return rc;
  }
  LV_HIP_CHECK_LAUNCH();
  return LV_OK;
}

int launch_global_block(const uint16_t *z, int64_t M, int C, int heads, float scale, int attn_dtype,
                        int qk_norm, const litevggt_block_weights &bw, uint16_t *delta, void *ws,
                        size_t ws_bytes, hipStream_t st, hipEvent_t after_pack, hipEvent_t after_attn, void *wpack_keep,
                        bool wpack_ready) {
  if (C % kTile != 0) return LV_ERR_SHAPE;
  BlockWs w = carve_block(M, C, heads, attn_dtype, ws_bytes < block_ws_bytes(M, C, heads, attn_dtype), (char *)ws);
  int rc;
  const bool f8 = bw.linear_dtype == LV_LINEAR_FP8_E4M3;
  const bool delayed = f8 && bw.fp8_recipe == LV_FP8_DELAYED;
  // The weights in operand order: in the workspace, or in a buffer of the caller's that outlives
  // the call and may already hold them (bf16 layers, and FP8 layers under delayed scaling, where
  // a weight's scale depends on nothing but the weight; the four amaxes follow the matrices).
  const bool keep = wpack_keep && (!f8 || delayed);
  u32x4 *const wp = keep ? (u32x4 *)wpack_keep : w.wpack;
  const bool pack_w = !(keep && wpack_ready);
  const size_t cc16 = (size_t)C * C * 2 / 16;
  u32x4 *const wp_l[4] = {wp, wp + 3 * cc16, wp + 4 * cc16, wp + 8 * cc16};
  uint32_t *const wamax = (uint32_t *)(wp + 12 * cc16);
  const BlockWeights4 bw4 = {{(const uint16_t *)bw.w_qkv, (const uint16_t *)bw.w_o, (const uint16_t *)bw.w_1,
                              (const uint16_t *)bw.w_2},
                             {wp_l[0], wp_l[1], wp_l[2], wp_l[3]}};
  const float *const bias[4] = {bw.b_qkv, bw.b_o, bw.b_1, bw.b_2};
  const uint16_t *q = w.qkv, *k = w.qkv + (size_t)M * C, *v = w.qkv + (size_t)2 * M * C;

  // the weights' amaxes, then every layer's scalars, the weights into operand order and (bf16 layers and delayed
  // scaling, where its scale is known) the first LayerNorm into the first layer's operand
  AttnKV kv;                 // what the first layer does for the attention (kv_ready: has done)
  bool kv_ready = false;
  if ((rc = attn_kv_target(kv, M, heads, scale, attn_dtype, qk_norm, q, w.a, w.attn, w.attn_bytes))) return rc;
  Fp8Head hd{};
  if (f8) {
    if (pack_w) hipLaunchKernelGGL(k_weights_amax, dim3(kWAmaxParts), dim3(256), 0, st, bw4, C, w.wpart);
    hd = Fp8Head{w.fp8sc, delayed ? (const float *)bw.fp8_state : nullptr, wamax, pack_w ? (const uint32_t *)w.wpart : nullptr,
                 (uint32_t *)w.h};
  }
  u32x4 *const ln_packed = f8 && !delayed ? nullptr : w.apack;
  if ((rc = launch_block_head(z, bw.ln1_g, bw.ln1_b, M, w.Mp, C, ln_packed, pack_w ? &bw4 : nullptr, f8, hd, kv, st))) return rc;

  if (delayed) {
    // FP8 layers, delayed scaling: every input scale is known before its tensor exists, so the
    // LayerNorms and the first MLP layer quantise their results themselves (taking the amax for
    // the history on the way), and so does E4M3 attention; bf16 attention's output goes through k_quant_pack_fp8.
    uint32_t *const sc = w.fp8sc;
    auto layer = [&](int l) {
      LinearOpts o;
      o.fp8 = true;
      o.sc = sc + l * kFp8Words;
      o.w_packed = wp_l[l];
      return o;
    };
    LinearOpts o = layer(0);
    o.a_packed = w.apack;
    o.kv = &kv;
    o.kv_done = &kv_ready;
    if ((rc = launch_linear(nullptr, M, C, 3 * C, bias[0], 0, w.qkv, C, w, st, o))) return rc;
    AttnOperand a_op{w.apack, sc + kFp8Words + 2, sc + kFp8Words};
    if ((rc = launch_attn(q, k, v, w.a, M, heads, scale, attn_dtype, qk_norm, w.attn, w.attn_bytes, st, after_pack, 1, nullptr,
                          &a_op, kv_ready ? &kv : nullptr)))
      return rc;
    if (after_attn && hipEventRecord(after_attn, st) != hipSuccess) return LV_ERR_HIP;
    o = layer(1);
    o.a_packed = a_op.written ? w.apack : nullptr;
    if ((rc = launch_linear(w.a, M, C, C, bias[1], 0, w.u1, C, w, st, o))) return rc;
    if ((rc = launch_layernorm(z, w.u1, bw.ln2_g, bw.ln2_b, M, C, nullptr, st, w.apack, w.Mp,
                               sc + 2 * kFp8Words + 2, sc + 2 * kFp8Words)))
      return rc;
    o = layer(2);
    o.a_packed = w.apack;
    o.pack_out = true;
    o.out_inv = sc + 3 * kFp8Words + 2;
    o.out_amax = sc + 3 * kFp8Words;
    if ((rc = launch_linear(nullptr, M, C, 4 * C, bias[2], 1, w.h3, 4 * C, w, st, o))) return rc;
    o = layer(3);
    o.a_packed = (const u32x4 *)w.h3;
    o.addend = w.u1;
    o.rec.state = (float *)bw.fp8_state;
    o.rec.sc = sc;
    o.rec.ln_part = hd.ln_part;
    o.rec.n_part = (int)(w.Mp / 32);
    return launch_linear(nullptr, M, 4 * C, C, bias[3], 0, delta, C, w, st, o);
  }

  auto layer = [&](int l) {
    LinearOpts o;
    o.fp8 = o.current = f8;
    o.sc = f8 ? w.fp8sc + l * kFp8Words : nullptr;
    o.w_packed = wp_l[l];
    return o;
  };
  // bf16 layers: the LayerNorms write their result in the following layer's operand order
  if (f8 && (rc = launch_layernorm(z, nullptr, bw.ln1_g, bw.ln1_b, M, C, w.h, st))) return rc;
  LinearOpts o = layer(0);
  o.a_packed = ln_packed;
  o.kv = &kv;
  o.kv_done = &kv_ready;
  if ((rc = launch_linear(w.h, M, C, 3 * C, bias[0], 0, w.qkv, C, w, st, o))) return rc;
  // bf16 layers: where the attention kernel can, it writes the output projection's operand itself
  AttnOperand a_op{w.apack};
  if ((rc = launch_attn(q, k, v, w.a, M, heads, scale, attn_dtype, qk_norm, w.attn, w.attn_bytes, st, after_pack, 1, nullptr,
                        f8 ? nullptr : &a_op, kv_ready ? &kv : nullptr)))
    return rc;
  if (after_attn && hipEventRecord(after_attn, st) != hipSuccess) return LV_ERR_HIP;
  o = layer(1);
  o.a_packed = a_op.written ? w.apack : nullptr;
  if ((rc = launch_linear(w.a, M, C, C, bias[1], 0, w.u1, C, w, st, o))) return rc;
  if ((rc = launch_layernorm(z, w.u1, bw.ln2_g, bw.ln2_b, M, C, w.h, st, ln_packed, w.Mp))) return rc;
  // bf16 layers: the first MLP layer writes its output in the second one's operand order.  All
  // layers: the second one's epilogue adds u1 (delta = u1 + u2, u2 rounded to bf16 first as if
  // it had been stored).
  o = layer(2);
  o.a_packed = ln_packed;
  o.pack_out = !f8;
  if ((rc = launch_linear(w.h, M, C, 4 * C, bias[2], 1, w.h3, 4 * C, w, st, o))) return rc;
  o = layer(3);
  o.a_packed = f8 ? nullptr : (const u32x4 *)w.h3;
  o.addend = w.u1;
  return launch_linear(w.h3, M, 4 * C, C, bias[3], 0, delta, C, w, st, o);
}

}  // namespace lv

// Target occupancy predictor (Sec. 3.2, Eq. 5) on gfx950, in the configured
// form: per voxel of a scale, the 11 input bits [delta, parent code] (target
// embedding, Eqs. 7-8), L submanifold 3x3x3 sparse conv + ReLU layers on the
// target coordinates (Eq. 9) and a linear head to 256 logits with the softmax
// normaliser (Eq. 10).  The first layer, whose input is 11 bits, is a sum of
// table rows (k_first); the others are matrix products (k_conv).
//
// Matrix layers: a wavefront owns 16 voxels of one scale (in small launches a quad
// of waves shares them, or a block's waves a few tiles).  Each layer is computed
// transposed, out^T[c_out][16] = sum_k W_k^T in_k^T, on fp16 MFMA 16x16x32
// with split operands (below): the A operand is the offset's weights (staged
// once per block in LDS), the B operand the gathered neighbour rows (lane
// (r, g) holds a slice of the row of voxel r's neighbour).  Only offsets with at
// least one occupied neighbour in the tile are issued.  A
// lane ends with 8 consecutive channels of its voxel, which is exactly the B
// operand of the head, so the head (16 x 256 logits per tile) runs from
// registers, followed by a row max / sum of exp over the 64 logits a lane
// holds and the 4 lanes sharing a voxel.
// Output-stationary: no atomics, a fixed summation order per voxel (4 offset
// groups, each chained from zero and added in group order; the softmax
// normaliser merged per 64-symbol group in group order), so an encoder and a
// decoder evaluating the same scale get bit-identical results however a launch
// shares its tiles among waves.

#include <type_traits>

#include "ctx.h"

namespace reno {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

// fp16 planes of split weights: [hi][lo], and at C = 16, where a gathered row
// fills one operand, a third one: its sums are so short that the weights' 2^-23
// would show beside fp32 rounding
__host__ __device__ constexpr int weight_planes(int C) { return C == 16 ? 3 : 2; }

constexpr int CONV_THREADS = 1024;
constexpr int CONV_WAVES = CONV_THREADS / 64;

// ---- split-fp16 arithmetic ----
// A row x of fp32 features is carried as x = f (hi + lo): f the power of two
// that brings the row's largest entry to [2^14, 2^15), hi = fp16(x / f) and lo
// = fp16(x / f - hi), both rounded to nearest, 22 bits of every entry within
// 2^-17 of the row's largest (smaller ones keep an absolute 2^-40 of it).
// Weights are split the same way, with one factor per output channel or symbol.
// A product is lo*hi + hi*lo + hi*hi on v_mfma_f32_16x16x32_f16 with fp32
// accumulation, smallest terms first (lo*lo, 2^-22 of the product, is dropped
// except at C = 16, where it fits in), 48 cycles per 16 x 16 x 32 block against
// 256 on fp32 MFMA.  An output sums one fma per offset instead of C / 4
// chained roundings, so its error against fp64 is about half that of the fp32
// MFMA chain (one layer of 6 neighbours, C = 32: 0.96e-7 against 1.76e-7
// relative; a whole 3-layer model's logits: 1.6e-7 against 1.7e-7).
// In fp32 a channel's magnitude is arbitrary: scaled by 2^k, and the weights that
// read it by 2^-k, every product is the same.  A shared factor would lose bits to
// that once channels lie 2^17 apart, so the matrices are balanced as they are
// packed: input channel c is divided by b_c, the power of two at or below its
// largest weight (0 where all are 0), and the rows split for that matrix carry
// channel c times b_c, exactly.  Entries and weights are then small beside others
// only where their products are.  The balance of a layer's output is part of its
// own weights' factors and bias (of the first layer's table, of the embeddings);
// where two matrices read a row, it carries the balance of one and is multiplied
// by the ratio (k_feature_balance) for the other.  With every row multiplied as it
// is split, the 14-bit scan's calls were 2 to 5 % slower.
__device__ __forceinline__ f4 mfma_h(const uint4& a, const uint4& b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}
__device__ __forceinline__ uint32_t pack_h2(float x0, float x1) {
  const h2 v = {(_Float16)x0, (_Float16)x1};
  return __builtin_bit_cast(uint32_t, v);
}

// The larger of two magnitudes; NaN if one is (a maximum would lose it, and the
// entry with it).
__device__ __forceinline__ float max_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// What maps a largest magnitude m to [2^14, 2^15), and a row's factor in units of
// 2^-14: the weights' factors are kept in units of 2^14, so that sums stay near
// the magnitude of their terms and overflow where those do.  From the exponent
// bits (exponents below 14 share the smallest factor; a denormal factor is exact).
__device__ __forceinline__ void split_scale(float m, float& mul, float& fac) {
  const uint32_t ex = max(__float_as_uint(m) >> 23, 14u);
  mul = __uint_as_float((268u - ex) << 23);                                       // 2^(14 - e)
  fac = __uint_as_float(ex > 28u ? (ex - 28u) << 23 : 1u << (ex - 6u));           // 2^(e - 28)
}

template <int N>
__device__ __forceinline__ float abs_max(const float (&x)[N], float m = 0.0f) {
#pragma unroll
  for (int i = 0; i < N; ++i) m = max_nan(m, fabsf(x[i]));
  return m;
}

// Factors of a row from a lane's largest magnitude, whose other entries are in
// the lanes STEP and 2 STEP away (16: lanes r + 16 g; 1: lanes 4 r + g).  A row
// with an infinite entry keeps that one at 2^15 against (practically) zero others
// and gets the factor infinity, so that what it adds to an output is infinite as
// in fp32; a row with a NaN gets the factor NaN.
template <int STEP = 16>
__device__ __forceinline__ void row_scale(float m, float& mul, float& fac) {
  m = max_nan(m, __shfl_xor(m, STEP));
  m = max_nan(m, __shfl_xor(m, 2 * STEP));
  split_scale(m, mul, fac);
  fac = m < INFINITY ? fac : m;
}

// Packed words of hi and lo of entries x0, x1 of a row.
__device__ __forceinline__ void split_words(float x0, float x1, float mul, uint32_t& hi, uint32_t& lo) {
  const float v0 = __builtin_amdgcn_fmed3f(x0 * mul, -32768.0f, 32768.0f);
  const float v1 = __builtin_amdgcn_fmed3f(x1 * mul, -32768.0f, 32768.0f);
  const h2 h = {(_Float16)v0, (_Float16)v1};
  hi = __builtin_bit_cast(uint32_t, h);
  lo = pack_h2(v0 - (float)h[0], v1 - (float)h[1]);
}

// A whole row: packed words of hi and lo, and the row's factor.
template <int N, int STEP = 16>
__device__ __forceinline__ float row_split(const float (&x)[N], uint32_t (&hi)[N / 2], uint32_t (&lo)[N / 2]) {
  float mul, fac;
  row_scale<STEP>(abs_max(x), mul, fac);
#pragma unroll
  for (int i = 0; i < N; i += 2) split_words(x[i], x[i + 1], mul, hi[i / 2], lo[i / 2]);
  return fac;
}

// ---------------------------------------------------------------------------
// Weight packing.

// The balance b_c of C input channels (above) from their largest magnitudes over
// W [kv][C][NS] (a head: kv = 1), one block per channel.  Infinite or NaN
// weights leave their channel as it is.
__global__ void __launch_bounds__(256) k_balance(const float* __restrict__ W, int kv, int C, int NS,
                                                 float* __restrict__ bal) {
  __shared__ float s_m[256];
  const int c = blockIdx.x;
  float m = 0.0f;
  for (int i = threadIdx.x; i < kv * NS; i += 256) m = max_nan(m, fabsf(W[((size_t)(i / NS) * C + c) * NS + i % NS]));
  s_m[threadIdx.x] = m;
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int i = 1; i < 256; ++i) m = max_nan(m, s_m[i]);
  const uint32_t ex = max(__float_as_uint(m) >> 23, 1u);
  bal[c] = m == 0.0f ? 0.0f : m < INFINITY ? __uint_as_float(ex << 23) : 1.0f;
}

// 1 / b_c (b_c = 0: no weight is scaled by it)
__device__ __forceinline__ float unbalance(float b) { return b > 0.0f ? 1.0f / b : 0.0f; }

// The features' balance, which the last layer's rows carry (hbal; with the full
// predictor also its child rows X_B): the first head matrix's, for channels that
// this one does not read the second's (hbal + C ..., two-stage), then that of the
// conv that reads X_B (b1; full predictor).  Those two become the features'
// balance times a ratio (hrat, xrat), a power of two inside fp32.
__device__ __forceinline__ float ratio(float a, float b) {
  if (!(a > 0.0f) || !(b > 0.0f)) return 0.0f;
  const int e = (int)(__float_as_uint(a) >> 23) - (int)(__float_as_uint(b) >> 23);
  return __uint_as_float((uint32_t)(min(max(e, -126), 126) + 127) << 23);
}
__global__ void __launch_bounds__(128) k_feature_balance(int C, float* __restrict__ hbal, float* __restrict__ hbal2,
                                                         float* __restrict__ hrat, float* __restrict__ b1,
                                                         float* __restrict__ xrat) {
  const int c = threadIdx.x;
  if (c >= C) return;
  float f = hbal[c];
  if (hbal2 && f == 0.0f) f = hbal2[c];
  if (b1 && f == 0.0f) f = b1[c];
  hbal[c] = f;
  if (hbal2) {
    hrat[c] = ratio(hbal2[c], f);
    hbal2[c] = f * hrat[c];
  }
  if (b1) {
    xrat[c] = ratio(b1[c], f);
    b1[c] = f * xrat[c];
  }
}

// What brings an output channel's (or symbol's) balanced weights to fp16 and the
// factor that takes it back, in units of 2^14 (split_scale); infinite or NaN
// weights are kept as they are, so they reach the products.
__device__ __forceinline__ void weight_scale(float m, float& mul, float& fac) {
  const uint32_t ex = min(max(__float_as_uint(m) >> 23, 15u), 254u);
  mul = m < INFINITY ? __uint_as_float((268u - ex) << 23) : 1.0f;   // 2^(14 - e)
  fac = m < INFINITY ? __uint_as_float(ex << 23) : 0x1p14f;         // 2^e
}

// Largest balanced magnitude of every output channel of W [n][C] (row i of input
// channel i % C) over each block's share of the n rows: part [gridDim.x][C].
constexpr int WMAX_BLOCKS = 64;
__global__ void __launch_bounds__(256) k_weight_max(const float* __restrict__ W, int n, int C,
                                                    const float* __restrict__ bal, float* __restrict__ part) {
  __shared__ float s_m[256];
  const int co = threadIdx.x % C, per = 256 / C;
  float m = 0.0f;
  for (int i = blockIdx.x * per + threadIdx.x / C; i < n; i += gridDim.x * per)
    m = max_nan(m, fabsf(W[(size_t)i * C + co] * unbalance(bal[i % C])));
  s_m[threadIdx.x] = m;
  __syncthreads();
  if ((int)threadIdx.x >= C) return;
  for (int j = 1; j < per; ++j) m = max_nan(m, s_m[j * C + co]);
  part[(size_t)blockIdx.x * C + co] = m;
}

// Conv layer W [kv][C][C]: the output channels' factors (from k_weight_max; times
// the output's balance obal) and the split A operands.  Lane l = (m, g) of column block cb carries an output
// channel such that the lane (r, g) that ends with rows 4g .. 4g + 3 of the
// column blocks holds channels 32 ch + 8g .. + 7 of voxel r (C = 16: channel m).
// K slot 8g + j: C >= 32 input channel 32 ch + 8g + j of piece ch, planes
// [hi][lo]; C = 16 the two halves of a gathered row [16 hi][16 lo], planes
// [W1 | W1], [W2 | W2] and [W3 | W3].  Packed [kv][C/16][ch][plane][64][8] fp16.
template <int C>
__global__ void __launch_bounds__(256) k_pack_conv(const float* __restrict__ W, int kv, const float* __restrict__ part,
                                                   const float* __restrict__ bal, const float* __restrict__ obal,
                                                   uint16_t* __restrict__ out, float* __restrict__ fac_out) {
  constexpr int NCB = C / 16, NCH = C >= 32 ? C / 32 : 1, PL = weight_planes(C);
  __shared__ float s_mul[C];
  if ((int)threadIdx.x < C) {
    float m = 0.0f, mul, fac;
    for (int i = 0; i < WMAX_BLOCKS; ++i) m = max_nan(m, part[i * C + threadIdx.x]);
    weight_scale(m, mul, fac);
    s_mul[threadIdx.x] = mul;
    if (blockIdx.x == 0) fac_out[threadIdx.x] = fac * obal[threadIdx.x];
  }
  __syncthreads();
  const int64_t n = (int64_t)kv * C * C;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int co = (int)(i % C), ci = (int)(i / C % C), k = (int)(i / (C * C));
    const int cb = C >= 32 ? 2 * (co >> 5) + ((co >> 2) & 1) : 0;
    const int row = C >= 32 ? 4 * ((co & 31) >> 3) + (co & 3) : co;  // m of the A operand
    uint16_t* o = out + ((size_t)(k * NCB + cb) * NCH + (C >= 32 ? ci >> 5 : 0)) * PL * 64 * 8;
    const int at = (((ci & 31) >> 3) * 16 + row) * 8 + (ci & 7);  // lane (row, group of ci), slot ci % 8
    float rest = W[i] * unbalance(bal[ci]) * s_mul[co];
#pragma unroll
    for (int pl = 0; pl < PL; ++pl) {
      const _Float16 h = (_Float16)rest;
      rest -= (float)h;
      o[pl * 64 * 8 + at] = __builtin_bit_cast(uint16_t, h);
      if (C == 16) o[pl * 64 * 8 + at + 2 * 16 * 8] = __builtin_bit_cast(uint16_t, h);  // groups 2, 3: the row's lo half
    }
  }
}

// Largest balanced magnitude of every symbol of a head H [C][NS].
__global__ void __launch_bounds__(64) k_head_max(const float* __restrict__ H, int C, int NS, const float* __restrict__ bal,
                                                 float* __restrict__ smax) {
  const int sym = blockIdx.x * 64 + threadIdx.x;
  if (sym >= NS) return;
  float m = 0.0f;
  for (int c = 0; c < C; ++c) m = max_nan(m, fabsf(H[(size_t)c * NS + sym] * unbalance(bal[c])));
  smax[sym] = m;
}

// Head H [C][NS] (NS = 256, or 16 per stage of the two-stage head), one block
// per 16-symbol block sb: the symbols' factors and the split A operands, lane
// (m, g) carrying symbol 16 sb + m.  C >= 32: K slot 8g + j of chunk ch is
// channel 32 ch + 8g + j, planes [hi][lo]; C = 16: slots 8g .. 8g + 3 and 8g +
// 4 .. 8g + 7 both carry channels 4g .. 4g + 3 (a lane's operand is [4 hi][4
// lo] of them), planes [H1 | H1], [H2 | H2] and [H3 | H3].  Packed
// [NS/16][max(C/32, 1)][plane][64][8] fp16.
// 256 symbols whose largest weights lie within 2^8 of each other share the factor
// of the largest: a symbol's entries down to 2^-9 of its own largest keep their 22
// bits, and a logit's smaller terms an absolute 2^-32 of the largest one.  Where
// they do, fac_out[256] is that factor, else 0.  With the factors read per symbol
// always (and rows balanced as they are split) the logits of the 14-bit scan took
// 180 us, with one factor (and balance folded into the weights) 170.
__global__ void __launch_bounds__(256) k_pack_head(const float* __restrict__ H, int C, int NS,
                                                   const float* __restrict__ bal, const float* __restrict__ smax,
                                                   uint16_t* __restrict__ out, float* __restrict__ fac_out) {
  __shared__ float s_mul[16];
  const int nch = C >= 32 ? C / 32 : 1, sb = blockIdx.x, planes = weight_planes(C);
  if (threadIdx.x < 16) {
    float m = smax[sb * 16 + threadIdx.x], mul, fac;
    bool shared = NS == 256;
    if (shared) {
      float hi = 0.0f, lo = INFINITY;
      for (int i = 0; i < NS; ++i) {
        hi = max_nan(hi, smax[i]);
        lo = fminf(lo, smax[i]);
      }
      shared = hi < INFINITY && lo >= hi * 0x1p-8f;
      if (shared) m = hi;
    }
    weight_scale(m, mul, fac);
    s_mul[threadIdx.x] = mul;
    fac_out[sb * 16 + threadIdx.x] = fac;
    if (NS == 256 && sb == 0 && threadIdx.x == 0) fac_out[256] = shared ? fac : 0.0f;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nch * 64 * 8; i += 256) {
    const int j = i & 7, lane = (i >> 3) & 63, ch = i >> 9, g = lane >> 4;
    const int c = C >= 32 ? 32 * ch + 8 * g + j : 4 * g + (j & 3);
    uint16_t* o = out + (size_t)((sb * nch + ch) * planes) * 64 * 8 + (i & 511);
    float rest = H[(size_t)c * NS + sb * 16 + (lane & 15)] * unbalance(bal[c]) * s_mul[lane & 15];
    for (int pl = 0; pl < planes; ++pl) {
      const _Float16 h = (_Float16)rest;
      rest -= (float)h;
      o[pl * 64 * 8] = __builtin_bit_cast(uint16_t, h);
    }
  }
}

// Transposes H [C][NS] into rows row0 .. row0+NS-1 of a [*][C] table.
// divided by the balance of the features.
__global__ void k_transpose_head(const float* __restrict__ H, const float* __restrict__ bal, int C, int NS, int row0,
                                 float* __restrict__ out) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < C * NS; i += gridDim.x * blockDim.x) {
    const int c = i / NS, s = i % NS;
    out[(size_t)(row0 + s) * C + c] = H[i] * unbalance(bal[c]);
  }
}

// A head [C][NS] divided by the balance of the features, into columns col0 .. of
// a [C][stride] table.
__global__ void k_unbalance_head(const float* __restrict__ H, const float* __restrict__ bal, int C, int NS, int stride,
                                 int col0, float* __restrict__ out) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < C * NS; i += gridDim.x * blockDim.x)
    out[(i / NS) * stride + col0 + i % NS] = H[i] * unbalance(bal[i / NS]);
}

// Rows [n][C] (a bias, an embedding) times a balance.
__global__ void k_balance_rows(const float* __restrict__ src, const float* __restrict__ bal, int n, int C,
                               float* __restrict__ dst) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n * C; i += gridDim.x * blockDim.x) dst[i] = src[i] * bal[i % C];
}

// ---------------------------------------------------------------------------
// Head pieces, shared by the last conv layer, the head on stored features and
// the decoder's stage-2 kernel, so that all produce identical bits.  A lane
// (r, g) holds C / 4 features of voxel r: x[8 ch + j] = channel 32 ch + 8g + j
// (C = 16: x[j] = channel 4g + j).

// The lane's C / 4 entries of a row of C floats, in the order above.
template <int C>
__device__ __forceinline__ void load_row(const float* __restrict__ row, int g, float (&x)[C / 4]) {
  constexpr int Q = C >= 32 ? 2 : 1;  // f4 words per chunk
#pragma unroll
  for (int ch = 0; ch < (C >= 32 ? C / 32 : 1); ++ch)
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const f4 t = *reinterpret_cast<const f4*>(row + 32 * ch + 4 * Q * g + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[8 * ch + 4 * q + e] = t[e];
    }
}

// Stores a lane's entries of a row of C floats.
template <int C>
__device__ __forceinline__ void store_row(const float (&x)[C / 4], int g, float* __restrict__ row) {
  constexpr int Q = C >= 32 ? 2 : 1;
#pragma unroll
  for (int ch = 0; ch < (C >= 32 ? C / 32 : 1); ++ch)
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = 8 * ch + 4 * q;
      *reinterpret_cast<f4*>(row + 32 * ch + 4 * Q * g + 4 * q) = f4{x[i], x[i + 1], x[i + 2], x[i + 3]};
    }
}

// x + the same entries of another row (Emb(S1), Emb_D).
template <int C>
__device__ __forceinline__ void add_row(const float (&x)[C / 4], const float* __restrict__ row, int g,
                                        float (&out)[C / 4]) {
  load_row<C>(row, g, out);
#pragma unroll
  for (int i = 0; i < C / 4; ++i) out[i] = x[i] + out[i];
}

// x times the same entries of a row (a balance); out may be x.
template <int C>
__device__ __forceinline__ void mul_row(const float (&x)[C / 4], const float* __restrict__ row, int g,
                                        float (&out)[C / 4]) {
  float b[C / 4];
  load_row<C>(row, g, b);
#pragma unroll
  for (int i = 0; i < C / 4; ++i) out[i] = x[i] * b[i];
}

// B operand of a head from a lane's (balanced) features.
template <int C>
struct HeadOp {
  static constexpr int NCH = C >= 32 ? C / 32 : 1;
  static constexpr int BLOCK = NCH * weight_planes(C) * 64;  // 16-byte words of one packed 16-symbol block
  uint4 hi[NCH], lo[C >= 32 ? NCH : 1];
  float fac;
  __device__ __forceinline__ void set(const float (&x)[C / 4]) {
    uint32_t h[C / 8], l[C / 8];
    fac = row_split<C / 4>(x, h, l);
    if constexpr (C >= 32) {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        hi[ch] = make_uint4(h[4 * ch], h[4 * ch + 1], h[4 * ch + 2], h[4 * ch + 3]);
        lo[ch] = make_uint4(l[4 * ch], l[4 * ch + 1], l[4 * ch + 2], l[4 * ch + 3]);
      }
    } else {
      hi[0] = make_uint4(h[0], h[1], l[0], l[1]);
    }
  }
};

// H^T x of one 16-symbol block in units of the row's and the symbols' factors: lane (r, g) ends
// with symbols 4g .. 4g + 3 of voxel r.  hp: the block's packed operands.
template <int C>
__device__ __forceinline__ f4 head_block(const uint4* hp, int lane, const HeadOp<C>& b) {
  constexpr int NCH = HeadOp<C>::NCH;
  f4 p = f4{0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (C >= 32) {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) p = mfma_h(hp[(2 * ch + 1) * 64 + lane], b.hi[ch], p);
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) p = mfma_h(hp[2 * ch * 64 + lane], b.lo[ch], p);
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) p = mfma_h(hp[2 * ch * 64 + lane], b.hi[ch], p);
  } else {
#pragma unroll
    for (int pl = weight_planes(C) - 1; pl >= 0; --pl) p = mfma_h(hp[pl * 64 + lane], b.hi[0], p);
  }
  return p;
}

// 16 logits of one stage of the two-stage head.
template <int C>
__device__ __forceinline__ f4 head16(const uint4* hp, const float* __restrict__ hfac,
                                     const float* __restrict__ hb, const float (&x)[C / 4], int lane, int g) {
  HeadOp<C> b;
  b.set(x);
  const f4 p = head_block<C>(hp, lane, b);
  const f4 f = *reinterpret_cast<const f4*>(hfac + 4 * g);
  f4 z = *reinterpret_cast<const f4*>(hb + 4 * g);
#pragma unroll
  for (int e = 0; e < 4; ++e) z[e] = fmaf(p[e] * b.fac, f[e], z[e]);
  return z;
}

// Natural-log normaliser of the 16 logits spread over lanes r, r+16, r+32, r+48.
__device__ __forceinline__ float lse16(const f4& z) {
  float m = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
  m = fmaxf(m, __shfl_xor(m, 16));
  m = fmaxf(m, __shfl_xor(m, 32));
  float s = (__expf(z[0] - m) + __expf(z[1] - m)) + (__expf(z[2] - m) + __expf(z[3] - m));
  s += __shfl_xor(s, 16);
  s += __shfl_xor(s, 32);
  return m + __logf(s);
}

__global__ void k_copy_f32(const float* __restrict__ src, float* __restrict__ dst, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    dst[i] = src[i];
}

// ---------------------------------------------------------------------------
struct ConvArgs {
  int b_lo, b_hi, b0;
  const int32_t* count;
  const int32_t* moff;
  int64_t cap_pts, cap_model;
  const int32_t* nbr;     // neighbour map [rows][stride]
  const float* h_in;      // conv input: split rows (k_headw: fp32 rows); row cap_model all zero
  const float* r_in;      // factors of the split rows
  float* h_out;           // fp32 output rows [rows][C], or NULL
  uint32_t* s_out;        // split output rows, or NULL
  float* r_out;           // their factors
  uint32_t* next;         // groups taken of each XCD's share [8], zero at launch (k_convw)
  const float* w;         // packed conv weights
  const float* wfac;      // their factors [C]
  const float* bias;      // [C]
  const uint4* hw;        // packed head weights (last layer)
  const float* hfac;      // the symbols' factors, as hb; [256]: the one they share, or 0 (one-stage)
  const float* hrat;      // two-stage head: what takes the features to stage 2's balance [C]
  const float* hb;        // [256]
  float* lse;             // [cap_model]
  float* logits;          // optional [rows][256] (two-stage: [rows][32]), row = packed row - moff[b_lo]
  // two-stage head
  const float* emb;       // [16][C]
  const uint8_t* s1_code; // codes of the per-scale regions (S1 = O & 15), or NULL: stage 1 only
  float* lse2;            // [cap_model]
  uint8_t* s1_out;        // [cap_model] the S1 stage 2 used
  const int32_t* perm;    // k_convw: tile order, tile slot -> packed row
  // full predictor
  const float* res;       // residual input added before the ReLU (same rows as h_out), or NULL; see emb_o
  int b_ext;              // scale whose rows live past the zero row (the base scale), or -1
  int64_t ext_off;        // first packed row of that scale (cap_model + 1)
  int64_t cap_rows;       // rows of the feature buffers
  // replication + octant embedding fused into the epilogue (Eqs. 7-8): each
  // voxel's result F, plus Emb_D[delta], goes to the rows of its children
  float* xb;              // child rows' input X_B (rows of scale b + 1), or NULL
  uint32_t* xb_s;         // X_B as split rows
  float* xb_r;            // their factors
  const float* xrat;      // what takes X_B to the balance of the conv that reads them [C]
  const float* emb_d;     // [8][C]
  const float* emb_o;     // [256][C]: the residual input X_A of that layer
  const uint8_t* code;    // per-scale regions: O_b
  const int32_t* fc;      // per-scale regions: first child row in V_{b+1}
};

// Packed-row layout of the scales: scale b at moff[b] .. below the reserved
// zero row cap_model; the full predictor also models the base scale, whose
// rows sit past the zero row at ext_off.
struct RowMap {
  const int32_t* count;
  const int32_t* moff;
  int64_t cap_model;
  int b_ext;
  int64_t ext_off, cap_rows;
};

// First packed row and voxel count of scale b; a scale that would not fit
// reads as empty (the overflow was latched where its size was made).
__device__ __forceinline__ void scale_span(const RowMap& m, int b, int64_t& mo, int64_t& n) {
  n = m.count[b];
  if (b == m.b_ext) {
    mo = m.ext_off;
    if (mo + n > m.cap_rows) n = 0;
  } else {
    mo = m.moff[b];
    if (mo + n > m.cap_model) n = 0;
  }
}

// Register-staged copy of N16 16-byte words into LDS, in two halves: the
// loads (issued early, so that their latency overlaps other work) and the
// stores.
template <int N16, int THREADS>
struct Staged {
  static constexpr int PER = (N16 + THREADS - 1) / THREADS;
  f4 v[PER];
  __device__ __forceinline__ void load(const f4* __restrict__ src, int tid) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int idx = i * THREADS + tid;
      if (idx < N16) v[i] = src[idx];
    }
  }
  __device__ __forceinline__ void store(f4* dst, int tid) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int idx = i * THREADS + tid;
      if (idx < N16) dst[idx] = v[i];
    }
  }
};

// Where the neighbour search reads: the coordinate hash and the per-scale
// arrays (scale b at (b - b0) * cap_pts).
struct CellArgs {
  const HashSlot* hash;
  int hash_lg;
  const uint64_t* hreg;  // hash region starts of a frame batch (null: one frame)
  int fb;                // frame-id bits above the Morton bits
  int b0;
  int64_t cap_pts;
  const uint8_t* code;
  const int32_t* fc;
};

// (first child, code) of N cells of scale s, all of the frame of bits fr (in
// place above the 3 s Morton bits): code 0 where ok is false or the cell is
// absent.  The hash maps the cells of scale s - 1, so a cell is found as the
// child of its own parent cell, and its code and first child are read by row.
// Neighbouring cells share parents (8 cells around a voxel lie in 3.4 of them
// on average) and the finest parent scale, the largest, is never inserted, so
// the probes of absent cells, each a random line of the table, mostly hit
// lines in use; the hash build, bound by its inserts, halves (10 frames of the
// 14-bit scan: 111 -> 64 us; 64 frames: 679 -> 414 us).  Probing every cell of
// a scale below the finest directly instead costs the same at one frame and
// 1 to 4 % more at 10.  The base scale has no stored parent and is probed
// directly.
template <int N>
__device__ __forceinline__ void find_cells(const CellArgs& a, int s, uint64_t fr, const uint64_t (&cell)[N],
                                           const bool (&ok)[N], uint2 (&hit)[N]) {
  const HashReg reg = hash_region(a.hreg, a.hash_lg, frame_part(fr, s));
  uint64_t tk[N];
  if (s == a.b0) {
#pragma unroll
    for (int i = 0; i < N; ++i) tk[i] = ok[i] ? tag_key(fr | cell[i], s, a.fb) : 0ull;
    hash_find_n<N>(a.hash, a.hash_lg, reg, tk, hit);
    return;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) tk[i] = ok[i] ? tag_key((fr | cell[i]) >> 3, s - 1, a.fb) : 0ull;
  hash_find_n<N>(a.hash, a.hash_lg, reg, tk, hit);
  const uint8_t* code = a.code + (int64_t)(s - a.b0) * a.cap_pts;
  const int32_t* fc = a.fc + (int64_t)(s - a.b0) * a.cap_pts;
  uint32_t c[N];
  int32_t f[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint32_t d = (uint32_t)cell[i] & 7u;
    const bool in = (hit[i].y >> d) & 1u;
    const uint32_t row = in ? hit[i].x + __popc(hit[i].y & ((1u << d) - 1u)) : 0u;
    c[i] = in ? code[row] : 0u;
    f[i] = in ? fc[row] : 0;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) hit[i] = make_uint2((uint32_t)f[i], c[i]);
}

// Neighbour rows of a voxel from the parent scale.  The 27 cells around v lie
// in at most 8 cells of the parent scale: the parent p and, per axis, the
// neighbour of p on v's side.  Lane (r, g) looks up cells e = 2g and 2g+1
// (e = ex + 2ey + 4ez) of its voxel r; each hit gives the cell's code and
// first-child row, from which every neighbour row follows by the FCG order.
// par is the 8-entry LDS slot of voxel r (shared by the 4 lanes of r); the
// lane ends with the rows of offsets 8g .. 8g+7 (-1: absent or off-grid).
//
// The cells are stepped to directly on the Morton key (dilated-integer
// increments and decrements of one axis's bits), so no coordinate is ever
// unpacked; a step off the grid leaves the probe empty, and every neighbour
// in such a cell reads as absent, so the offsets need no bounds of their own.

// OR over each row of 16 lanes.
__device__ __forceinline__ uint32_t or_row16(uint32_t v) {
  v |= dpp<0x128>(v);  // row_ror:8, 4, 2, 1
  v |= dpp<0x124>(v);
  v |= dpp<0x122>(v);
  v |= dpp<0x121>(v);
  return v;
}

// Stores a voxel's row of the 3x3x3 neighbour map as k_conv reads it: lane 4r + g
// holds offsets 8g .. 8g + 7 of voxel r; entry MAP_MASK of the row's padding
// takes the mask of its occupied offsets.
constexpr int MAP_MASK = 27;
__device__ __forceinline__ void store_map(int32_t* nbr, int64_t prow, bool valid, int g, const int32_t (&nb)[8]) {
  uint32_t own = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) own |= (nb[j] >= 0 ? 1u : 0u) << j;
  own <<= 8 * g;
  own |= (uint32_t)__shfl_xor((int)own, 1);
  own |= (uint32_t)__shfl_xor((int)own, 2);
  if (!valid) return;
  int4* dst = reinterpret_cast<int4*>(nbr + prow * NBR_STRIDE + 8 * g);
  dst[0] = make_int4(nb[0], nb[1], nb[2], g == MAP_MASK / 8 ? (int)own : nb[3]);
  dst[1] = make_int4(nb[4], nb[5], nb[6], nb[7]);
}

// Per entry slot j of the 8 a lane holds, the four lane groups' offsets
// k = 8g + j packed one byte each: bit 6 the offset exists (k < 27), bits 3..5
// the axes it moves up, bits 0..2 the axes it moves at all (k = dx+1 +
// 3 (dy+1) + 9 (dz+1)).
__host__ __device__ constexpr uint32_t offset_moves(int j) {
  uint32_t v = 0;
  for (int g = 0; g < 4; ++g) {
    const int k = 8 * g + j;
    if (k < 27) {
      const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = k / 9 - 1;
      const uint32_t nz = (dx != 0 ? 1u : 0u) | (dy != 0 ? 2u : 0u) | (dz != 0 ? 4u : 0u);
      const uint32_t up = (dx == 1 ? 1u : 0u) | (dy == 1 ? 2u : 0u) | (dz == 1 ? 4u : 0u);
      v |= (64u | (up << 3) | nz) << (8 * g);
    }
  }
  return v;
}

// One step of the cell with Morton key k (axis bits m) towards +1 (up) or -1
// along that axis; `off` is set when the step leaves the grid.
__device__ __forceinline__ uint64_t morton_step(uint64_t k, uint64_t m, bool up, bool& off) {
  const uint64_t a = k & m, rest = k & ~m;
  off = up ? a == m : a == 0ull;
  const uint64_t na = up ? ((a | ~m) + 1ull) & m : (a - 1ull) & m;
  return na | rest;
}

__device__ __forceinline__ void parent_cell_rows(uint64_t kf, int b, int g, const CellArgs& a,
                                                 uint64_t* par, int32_t (&nb)[8]) {
  const uint64_t key = morton_part(kf, b), fr = frame_part(kf, b) << (3 * (b - 1));
  const uint32_t oct = (uint32_t)key & 7u;  // v's octant in its parent: the side of each neighbour cell
  const uint64_t pk = key >> 3;
  const uint64_t all = (1ull << (3 * (b - 1))) - 1ull;
  const uint64_t mx = 0x1249249249249249ull & all, my = (mx << 1) & all, mz = (mx << 2) & all;
  // lane group g looks up cells 2g and 2g + 1: the y and z steps of g, then x
  bool off_y = false, off_z = false, off_x = false;
  uint64_t c0 = pk;
  if (g & 1) c0 = morton_step(c0, my, (oct & 2u) != 0u, off_y);
  if (g & 2) c0 = morton_step(c0, mz, (oct & 4u) != 0u, off_z);
  const uint64_t c1 = morton_step(c0, mx, (oct & 1u) != 0u, off_x);
  const bool ok0 = !(off_y || off_z);
  const uint64_t cells[2] = {c0, c1};
  const bool ok[2] = {ok0, ok0 && !off_x};
  uint2 hit[2];
  find_cells<2>(a, b - 1, fr, cells, ok, hit);
  // cross-lane exchange through LDS within the wave
  wave_lds_fence();  // earlier reads of the slots are done
  par[2 * g] = ((uint64_t)hit[0].y << 32) | hit[0].x;
  par[2 * g + 1] = ((uint64_t)hit[1].y << 32) | hit[1].x;
  wave_lds_fence();
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t c = (offset_moves(j) >> (8 * g)) & 0xFFu;
    const uint32_t nz = c & 7u, up = (c >> 3) & 7u;
    // the parent-scale cell of the neighbour: a moved axis leaves v's parent
    // when the move points to v's side; its octant flips every moved axis
    const uint32_t e = nz & ~(oct ^ up), d = oct ^ nz;
    const uint64_t pc = par[e];
    const uint32_t first = (uint32_t)pc, code = (uint32_t)(pc >> 32);
    nb[j] = ((c & 64u) && ((code >> d) & 1u)) ? (int32_t)(first + __popc(code & ((1u << d) - 1u))) : -1;
  }
}

constexpr float LOG2E_F = 1.4426950408889634f;

// One group of 64 symbols of the 256-way head (symbol blocks 4 grp .. 4 grp
// + 3, 16 symbols each) for a tile: logits z = H^T x + b, stored when requested
// (lo, or NULL), and the group's normaliser terms per lane: gm = the max of the
// lane's 16 logits, part = the sum of exp(z - gm).
template <int C>
__device__ __forceinline__ void head_group(const uint4* s_h, const float* __restrict__ hb, const float* __restrict__ hfac,
                                           const HeadOp<C>& op, float* lo, int lane, int g, int grp, float& gm,
                                           float& part) {
  f4 zz[4];
  const float shared = hfac[256];
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    const int sb = grp * 4 + q4;
    const f4 bias = *reinterpret_cast<const f4*>(hb + 16 * sb + 4 * g);
    const f4 p = head_block<C>(s_h + (size_t)sb * HeadOp<C>::BLOCK, lane, op);
    const float f1 = op.fac * shared;
    f4 f = f4{f1, f1, f1, f1};
    if (shared == 0.0f) f = *reinterpret_cast<const f4*>(hfac + 16 * sb + 4 * g) * op.fac;  // uniform
#pragma unroll
    for (int e = 0; e < 4; ++e) zz[q4][e] = fmaf(p[e], f[e], bias[e]);
  }
  float mx = zz[0][0];
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
    for (int e = 0; e < 4; ++e) mx = fmaxf(mx, zz[q4][e]);
  // exp(z - gm) as 2^(z log2(e) - gm log2(e)): one fused multiply-add per term
  const float ml = mx * LOG2E_F;
  float s = __builtin_amdgcn_exp2f(fmaf(zz[0][0], LOG2E_F, -ml));
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (q4 || e) s += __builtin_amdgcn_exp2f(fmaf(zz[q4][e], LOG2E_F, -ml));
  gm = mx;
  part = s;
  if (lo) {
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) *reinterpret_cast<f4*>(lo + 16 * (grp * 4 + q4)) = zz[q4];
  }
}

// Running normaliser (m, s) of the logits seen so far, extended by a group
// with terms (gm, part); starts from (-inf, 0).
__device__ __forceinline__ void lse_merge(float& m, float& s, float gm, float part) {
  const float mn = fmaxf(m, gm);
  s = s * __expf(m - mn) + part * __expf(gm - mn);
  m = mn;
}

// The 4 lanes r, r+16, r+32, r+48 hold the 4 quarters of voxel r's symbols:
// merged by lane exchange, then lse = m + log(s) stored at row prow.
__device__ __forceinline__ void lse_finish(const ConvArgs& a, float m, float ssum, int g, bool valid, int64_t prow) {
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) {
    const float om = __shfl_xor(m, o), os = __shfl_xor(ssum, o);
    const float mn = fmaxf(m, om);
    ssum = ssum * __expf(m - mn) + os * __expf(om - mn);
    m = mn;
  }
  if (valid && g == 0) a.lse[prow] = m + __logf(ssum);
}

// A tile as the epilogue and the head need it (per lane: voxel r).
struct TileRef {
  int b;
  int64_t mo, lvb, prow;
  bool valid;
};

// The two-stage head (Eqs. 11-13) on a tile's features: stage 1 over S1; stage
// 2 over S2 with x + Emb(S1) when the codes of the scale are known.
template <int C>
__device__ __forceinline__ void head_two(const ConvArgs& a, const float (&x)[C / 4], const uint4* s_h, int lane, int g,
                                         const TileRef& tr, int64_t mo_first) {
  constexpr int BLK = HeadOp<C>::BLOCK;
  float rt[C / 4];
  load_row<C>(a.hrat, g, rt);  // before the stores of stage 1, which it would wait behind
  const f4 z1 = head16<C>(s_h, a.hfac, a.hb, x, lane, g);
  const float l1 = lse16(z1);
  if (tr.valid && g == 0) a.lse[tr.prow] = l1;
  float* lo = (a.logits && tr.valid) ? a.logits + (tr.prow - mo_first) * 32 + 4 * g : nullptr;
  if (lo) *reinterpret_cast<f4*>(lo) = z1;
  if (!a.s1_code) return;
  const int s1 = a.s1_code[tr.lvb + (tr.prow - tr.mo)] & 15;
  float x2[C / 4];
  add_row<C>(x, a.emb + s1 * C, g, x2);
#pragma unroll
  for (int i = 0; i < C / 4; ++i) x2[i] *= rt[i];
  const f4 z2 = head16<C>(s_h + BLK, a.hfac + 16, a.hb + 16, x2, lane, g);
  const float l2 = lse16(z2);
  if (tr.valid && g == 0) {
    a.lse2[tr.prow] = l2;
    a.s1_out[tr.prow] = (uint8_t)s1;
  }
  if (lo) *reinterpret_cast<f4*>(lo + 16) = z2;
}

// The head on a tile's features in registers: the one-stage 256-way head with its
// softmax normaliser (Eq. 10), or the two-stage head.  Writes lse (lse2, S1) at
// the tile's rows and, when requested, the logits at row prow - mo_first.
template <int C, bool TWO>
__device__ __forceinline__ void head_epilogue(const ConvArgs& a, const float (&x)[C / 4], const uint4* s_h, int lane,
                                              int g, const TileRef& tr, int64_t mo_first) {
  if constexpr (TWO) {
    head_two<C>(a, x, s_h, lane, g, tr, mo_first);
  } else {
    HeadOp<C> op;
    op.set(x);
    float* lo = (a.logits && tr.valid) ? a.logits + (tr.prow - mo_first) * 256 + 4 * g : nullptr;
    float m = -INFINITY, ssum = 0.0f;
#pragma unroll 1
    for (int grp = 0; grp < 4; ++grp) {
      float gm, part;
      head_group<C>(s_h, a.hb, a.hfac, op, lo, lane, g, grp, gm, part);
      lse_merge(m, ssum, gm, part);
    }
    lse_finish(a, m, ssum, g, tr.valid, tr.prow);
  }
}

// The k-th tile of an XCD's share.
__device__ __forceinline__ int64_t xcd_tile(int xcd, int64_t k, int64_t tch) {
  return ((k / tch) * 8 + xcd) * tch + k % tch;
}

// Tile of a block's slot, XCD-aware: workgroups are dealt round-robin to the
// 8 XCDs (block b runs on XCD b % 8), so chunks of tch consecutive tiles are
// dealt to the XCDs in turn and the blocks of one XCD sweep that XCD's chunks
// together: tiles that gather the same neighbour rows run on one L2 at about
// the same time.  Increasing in the slot for a fixed block.
__device__ __forceinline__ int64_t conv_tile(int64_t slot, int64_t tch) {
  return xcd_tile(blockIdx.x & 7, (blockIdx.x >> 3) + (int64_t)(gridDim.x >> 3) * slot, tch);
}

// Offsets of group i of the conv's fixed summation order: k in [7i, 7i + 7),
// the last group [21, 27).
__device__ __forceinline__ uint32_t group_offsets(int i) {
  const int lo = 7 * i, hi = i < 3 ? 7 * i + 7 : 27;
  return ((1u << hi) - 1u) & ~((1u << lo) - 1u);
}

// Split row of C channels: [C fp16 hi][C fp16 lo], C 32-bit words.  The slice a
// lane of k_conv feeds: C = 32 channels 8g .. 8g + 7 of both planes; C = 16 the 8
// halves 8g .. 8g + 7 of the whole row (K slots of k_pack_conv).
template <int C>
struct SplitRow {
  uint4 hi, lo;  // C = 16: hi alone
  float fac;
};

// Stores piece ch of a lane's entries (32 channels of the row, all of it at C =
// 16) as split words.
template <int C>
__device__ __forceinline__ void store_split_piece(const float* x, float mul, int ch, int g, uint32_t* row) {
  constexpr int W = C >= 32 ? 4 : 2;  // words of a lane's piece in each plane
  uint32_t h[W], l[W];
#pragma unroll
  for (int i = 0; i < W; ++i) split_words(x[2 * i], x[2 * i + 1], mul, h[i], l[i]);
  if constexpr (C >= 32) {
    *reinterpret_cast<uint4*>(row + 16 * ch + 4 * g) = make_uint4(h[0], h[1], h[2], h[3]);
    *reinterpret_cast<uint4*>(row + C / 2 + 16 * ch + 4 * g) = make_uint4(l[0], l[1], l[2], l[3]);
  } else {
    *reinterpret_cast<uint2*>(row + 2 * g) = make_uint2(h[0], h[1]);
    *reinterpret_cast<uint2*>(row + 8 + 2 * g) = make_uint2(l[0], l[1]);
  }
}

// Entries of a row that a lane works on at once: all of its C / 4, at C = 128 a
// piece, whose work ends at piece_end: the registers do not hold that of all four.
constexpr int at_once(int C) { return C > 64 ? 8 : C / 4; }
template <int C>
__device__ __forceinline__ void piece_end() {
  if constexpr (C > 64) __builtin_amdgcn_sched_barrier(0);
}

// Stores a lane's entries of a row as a split row and, from lane group 0, its
// factor.  part(c0, y) gives entries c0 .. of the row (twice for each piece at C =
// 128).
template <int C, int STEP = 16, typename Part>
__device__ __forceinline__ void store_split(Part part, int g, uint32_t* row, float* fac) {
  constexpr int N = C / 4, NC = at_once(C);
  float m = 0.0f, mul, f, y[NC];
#pragma unroll
  for (int c0 = 0; c0 < N; c0 += NC) {
    part(c0, y);
    m = abs_max(y, m);
    piece_end<C>();
  }
  row_scale<STEP>(m, mul, f);
#pragma unroll
  for (int c0 = 0; c0 < N; c0 += NC) {
    if constexpr (N > NC) part(c0, y);
#pragma unroll
    for (int q = 0; q < NC; q += 8) store_split_piece<C>(y + q, mul, (c0 + q) / 8, g, row);
    piece_end<C>();
  }
  if (g == 0) *fac = f;
}

// Out-of-range byte offset of a buffer load, which then returns zeros without
// an access; the row's 128-byte (64) and 4-byte offsets derived from it stay
// out of range of a scale of up to CONV_BUF_ROWS rows and do not wrap.
constexpr uint32_t NO_ROW = 0xFFFFFF00u;
constexpr int64_t CONV_BUF_ROWS = (int64_t(1) << 25) - 8;

__device__ __forceinline__ uint4 buf_load16(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0));
}
__device__ __forceinline__ float buf_load4(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 0));
}

// Conv sums of a tile of 16 voxels (lane (r, g): row row0 + r of a scale of n
// rows whose first packed row is mo), in units of the weights' factors: all 4
// offset groups added in group order (grp < 0), or one group's sum alone (a
// wave of a quad).  The tile's neighbours go to tbl (LDS of this wave,
// [offset][16], as byte offsets of their rows in the scale), where a lane
// reads the row of any offset; with a table of 16 offsets only, the second
// half replaces the first when the walk reaches it.  The tile's occupied
// offsets are walked in ascending order, PCH at a time, the next PCH gathered
// before the products of the current ones.  Each offset's products are chained
// on MFMA from zero and added with the neighbour row's factor by one fma.
//
// What bounds it (the 14-bit scan's middle layer, all scales in one launch): the
// L1 access rate and the LDS.  In the operand's layout 16 consecutive lanes name 16
// rows, so a gather costs one L1 access per lane: with both planes and the factor
// loaded that way, 28 M accesses, 57 us.  Absent rows (60 % of those named) are
// therefore out-of-range buffer loads, which return zeros without an access and,
// unlike skipped loads, keep the compiler's wait counts exact; and the hi plane
// goes through 4 lane exchanges (LDS) instead: 11.5 M accesses, 43 us.  Exchanging
// both planes moves the bound to the LDS, none back to the L1: 47 and 50 us.  8
// waves with 8 to 16 rows gathered ahead each: 54 us.  Tiles sorted by
// neighbourhood, which halved the fp32 MFMA work, no longer pay for their pass.
//
// BIG: a scale may hold more than CONV_BUF_ROWS rows (4 GB); rows are then
// read through 64-bit addresses and absent ones from the zero row.
template <int C, int TBL, bool BIG>
__device__ __forceinline__ void conv_sum(const ConvArgs& a, const uint4* s_w, uint32_t (*tbl)[16], int lane, int mo,
                                         int n, int row0, int grp, f4 (&out)[C / 16]) {
  constexpr int NCB = C / 16, PL = weight_planes(C);
  constexpr int PCH = 3;
  constexpr uint32_t ROWB = 4 * C;  // bytes of a split row
  const int r = lane & 15, g = lane >> 4;
  const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.h_in) + (int64_t)mo * C, 0,
                                                      BIG ? 0 : (int)((uint32_t)n * ROWB), 0x00027000);
  const auto facs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.r_in) + mo, 0, BIG ? 0 : n * 4, 0x00027000);
  // map row of voxel lane / 4, entries 4p .. 4p + 3 and 16 + 4p .. of its piece p =
  // lane % 4 (the 4 lanes of a voxel read 64 consecutive bytes)
  const bool have4 = row0 + (lane >> 2) < n;
  uint32_t nb[8], offs;
  {
    const int4* src =
        reinterpret_cast<const int4*>(a.nbr + (int64_t)(mo + (have4 ? row0 + (lane >> 2) : 0)) * NBR_STRIDE) + (lane & 3);
    const int4 lo = src[0], hi = src[4];
    const int32_t e8[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    // the union of the 16 voxels' masks (entry 27, the last of piece 2's second half)
    uint32_t m = have4 && (lane & 3) == 2 ? (uint32_t)hi.w : 0u;
    m = or_row16(m);
    offs = (uint32_t)(__builtin_amdgcn_readlane((int)m, 0) | __builtin_amdgcn_readlane((int)m, 16) |
                      __builtin_amdgcn_readlane((int)m, 32) | __builtin_amdgcn_readlane((int)m, 48));
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const bool has = have4 && e8[j] >= 0;
      if constexpr (BIG) nb[j] = has ? (uint32_t)(mo + e8[j]) : (uint32_t)a.cap_model;
      else nb[j] = has ? (uint32_t)e8[j] * ROWB : NO_ROW;
    }
  }
  if (grp >= 0) offs &= group_offsets(grp);
  auto table = [&](int half) {
    wave_lds_fence();  // earlier reads of the table are done
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (TBL == 32 || (j >> 2) == half) tbl[(16 * (j >> 2) + 4 * (lane & 3) + (j & 3)) % TBL][lane >> 2] = nb[j];
    wave_lds_fence();
  };
  table(0);
  int next_half = TBL == 32 ? 32 : 16;  // first offset not in the table
  f4 acc[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) out[cb] = acc[cb] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  int gcur = grp >= 0 ? grp : 0;  // group whose sum acc holds
  auto fold = [&]() {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      out[cb] += acc[cb];
      acc[cb] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    ++gcur;
  };
  // The next PCH offsets (-1 beyond the last) and the gathers of their rows.
  // The hi plane (C = 16: the row) and the factor are loaded by lane 4v + p,
  // piece p of voxel v's neighbour: one L1 access per row; the lo plane by lane
  // (r, g) as the operand has it.
  auto gather = [&](int (&ks)[PCH], SplitRow<C> (&x)[PCH]) {
    constexpr uint32_t NONE = NO_ROW;
    uint32_t at[PCH], at4[PCH];
#pragma unroll
    for (int c = 0; c < PCH; ++c) {
      ks[c] = offs ? __builtin_ctz(offs) : -1;
      offs &= offs ? offs - 1u : 0u;
      if (TBL < 32 && ks[c] >= next_half) {  // uniform
        table(1);
        next_half = 32;
      }
      const uint32_t (*t)[16] = tbl + (ks[c] & 31) % TBL;
      const uint32_t none = BIG ? (uint32_t)a.cap_model : NONE;
      at4[c] = ks[c] < 0 ? none : (*t)[lane >> 2];
      if constexpr (C == 32) at[c] = ks[c] < 0 ? none : (*t)[r];
    }
#pragma unroll
    for (int c = 0; c < PCH; ++c) {
      if constexpr (BIG) {
        x[c].hi = reinterpret_cast<const uint4*>(a.h_in + (int64_t)at4[c] * C)[lane & 3];
        if constexpr (C == 32) x[c].lo = reinterpret_cast<const uint4*>(a.h_in + (int64_t)at[c] * C)[4 + g];
        x[c].fac = a.r_in[at4[c]];
      } else {
        x[c].hi = buf_load16(rows, at4[c] + 16u * (lane & 3));
        if constexpr (C == 32) x[c].lo = buf_load16(rows, at[c] + 64u + 16u * g);
        x[c].fac = buf_load4(facs, at4[c] / C);
      }
    }
  };
  const int from = 4 * (4 * r + g);  // lane 4r + g, for lane (r, g) = r + 16g
  auto exchange = [&](uint32_t v, int at) { return (uint32_t)__builtin_amdgcn_ds_bpermute(at, (int)v); };
  auto mma = [&](const int (&ks)[PCH], const SplitRow<C> (&x)[PCH]) {
#pragma unroll
    for (int c = 0; c < PCH; ++c) {
      const int k = ks[c];
      if (k < 0) break;
      while (k >= (gcur < 3 ? 7 * (gcur + 1) : 27)) fold();
      uint4 wv[PL][NCB];
#pragma unroll
      for (int pl = 0; pl < PL; ++pl)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) wv[pl][cb] = s_w[((k * NCB + cb) * PL + pl) * 64 + lane];
      const uint4 hi = make_uint4(exchange(x[c].hi.x, from), exchange(x[c].hi.y, from), exchange(x[c].hi.z, from),
                                  exchange(x[c].hi.w, from));
      const float fac = __uint_as_float(exchange(__float_as_uint(x[c].fac), 16 * r));
      f4 p[NCB];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) p[cb] = mfma_h(wv[PL - 1][cb], hi, f4{0.0f, 0.0f, 0.0f, 0.0f});
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) p[cb] = mfma_h(C == 32 ? wv[0][cb] : wv[1][cb], C == 32 ? x[c].lo : hi, p[cb]);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) p[cb] = mfma_h(wv[0][cb], hi, p[cb]);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[cb][e] = fmaf(p[cb][e], fac, acc[cb][e]);
    }
  };
  int kA[PCH], kB[PCH];
  SplitRow<C> xA[PCH], xB[PCH];
  gather(kA, xA);
  while (true) {
    gather(kB, xB);
    mma(kA, xA);
    if (kB[0] < 0) break;
    gather(kA, xA);
    mma(kB, xB);
    if (kA[0] < 0) break;
  }
  if (grp < 0) {
    while (gcur < 4) fold();  // every group added, also the empty ones
  } else {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) out[cb] = acc[cb];
  }
}

// Bias, residual, ReLU, the children's X_B rows (full predictor) and the output
// rows of a tile from its conv sums: x ends with the lane's features.
template <int C, bool XB>
__device__ __forceinline__ void conv_epilogue(const ConvArgs& a, const f4 (&sum)[C / 16], int g, const TileRef& tr,
                                              float (&x)[C / 4]) {
  constexpr int N = C / 4, NC = at_once(C);
  // residual block: ReLU(x + conv(.)), x read at the voxel's own row; X_A (the
  // block that feeds the children) is a row of Emb_O
  uint32_t code = 0;
  if constexpr (XB) code = a.code[tr.lvb + (tr.prow - tr.mo)];
  const float* res = XB ? a.emb_o + code * C : a.res ? a.res + tr.prow * C : nullptr;
#pragma unroll
  for (int c0 = 0; c0 < N; c0 += NC) {
    float wf[NC], bs[NC];
    load_row<4 * NC>(a.wfac + 4 * c0, g, wf);
    load_row<4 * NC>(a.bias + 4 * c0, g, bs);
#pragma unroll
    for (int i = 0; i < NC; ++i) x[c0 + i] = fmaf(sum[(c0 + i) / 4][i % 4], wf[i], bs[i]);
    if (res) {
      float rs[NC];
      load_row<4 * NC>(res + 4 * c0, g, rs);
#pragma unroll
      for (int i = 0; i < NC; ++i) x[c0 + i] += rs[i];
    }
    piece_end<C>();
  }
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = fmaxf(x[i], 0.0f);
  if (!tr.valid) return;
  if constexpr (XB) {  // children v of this voxel u: X_B[v] = F[u] + Emb_D[delta(v)]
    int64_t cmo = a.moff[tr.b + 1];
    const int64_t cn = a.count[tr.b + 1];
    const int64_t first = a.fc[tr.lvb + (tr.prow - tr.mo)];
    if (cmo + cn > a.cap_model) cmo = -1;  // overflow (latched where the size was made): no writes
    float rt[NC];
    if constexpr (N == NC) load_row<4 * NC>(a.xrat, g, rt);
    int rank = 0;
    for (int d = 0; d < 8; ++d) {
      if (cmo >= 0 && ((code >> d) & 1u)) {
        const int64_t row = cmo + first + rank;
        auto child = [&](int c0, float (&y)[NC]) {
          load_row<4 * NC>(a.emb_d + d * C + 4 * c0, g, y);
#pragma unroll
          for (int i = 0; i < NC; ++i) y[i] = x[c0 + i] + y[i];
        };
        float y[NC];
#pragma unroll
        for (int c0 = 0; c0 < N; c0 += NC) {
          child(c0, y);
          store_row<4 * NC>(y, g, a.xb + row * C + 4 * c0);
          piece_end<C>();
        }
        auto split = [&](int c0, float (&z)[NC]) {
          if constexpr (N > NC) {
            child(c0, z);
            mul_row<4 * NC>(z, a.xrat + 4 * c0, g, z);
          } else {
#pragma unroll
            for (int i = 0; i < NC; ++i) z[i] = y[i] * rt[i];
          }
        };
        store_split<C>(split, g, a.xb_s + row * C, a.xb_r + row);
        ++rank;
      }
    }
  }
  if (a.s_out) {
    auto own = [&](int c0, float (&y)[NC]) {
#pragma unroll
      for (int i = 0; i < NC; ++i) y[i] = x[c0 + i];
    };
    store_split<C>(own, g, a.s_out + tr.prow * C, a.r_out + tr.prow);
  }
  if (a.h_out) store_row<C>(x, g, a.h_out + tr.prow * C);
}

// A sparse 3x3x3 conv layer C -> C (bias, optional residual, ReLU), the last
// one fused with the head.  One block of 16 waves per CU, the layer's weights
// (and the head's) staged in its LDS.
//
// Against the same layers on fp32 MFMA, 14-bit scan: middle layer 68 -> 43 us,
// last layer with the 256-way head 108 -> 60 us in the encoder's launch (no
// tile order before them: 10.7 us more); 155 + 203 -> 105 + 130 us over the
// decoder's nine scales each.
enum { CONV_MID = 0, CONV_SCATTER = 1, CONV_HEAD = 2, CONV_HEAD2 = 3 };

template <int C, int KIND, bool BIG>
__global__ void __launch_bounds__(CONV_THREADS) k_conv(ConvArgs a) {
  constexpr bool LAST = KIND >= CONV_HEAD, TWO = KIND == CONV_HEAD2;
  constexpr int NCB = C / 16;
  constexpr int N = C / 4;
  constexpr int WSZ = 27 * NCB * weight_planes(C) * 64;  // 16-byte words
  constexpr int HSZ = LAST ? (TWO ? 2 : 16) * HeadOp<C>::BLOCK : 4;
  __shared__ uint4 s_w[WSZ];
  __shared__ uint4 s_h[HSZ];
  // neighbours of a wave's tile; the weights of the 256-way head leave room for
  // half of the offsets at a time
  constexpr int TBL = KIND == CONV_HEAD ? 16 : 32;
  __shared__ uint32_t s_tbl[CONV_WAVES][TBL][16];
  __shared__ int s_next;  // next dynamically handed-out tile of this block

  // the wave index through a lane read: the compiler then keeps the unit loop,
  // the offset sets and the group folds in scalar registers and branches
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int r = lane & 15, g = lane >> 4;
  const int nsc = a.b_hi - a.b_lo + 1;
  const RowMap rm{a.count, a.moff, a.cap_model, a.b_ext, a.ext_off, a.cap_rows};
  // sizes of the launch's scales: lane i of every wave holds scale b_lo + i
  // (rows n_l, first row mo_l; rows and tiles fit in 31 bits)
  static_assert(NLEV < 32, "the scale scan covers 32 lanes");
  int n_l = 0, mo_l = 0;
  if (lane < nsc) {
    int64_t mo, n;
    scale_span(rm, a.b_lo + lane, mo, n);
    n_l = (int)n;
    mo_l = (int)mo;
  }
  auto scan32 = [&](int v) {
    if (nsc > 1) {
#pragma unroll
      for (int o = 1; o < 32; o <<= 1) {
        const int y = __shfl_up(v, o);
        if (lane >= o) v += y;
      }
    }
    return v;
  };
  const int incl = scan32((n_l + 15) / 16);
  const int total = __builtin_amdgcn_readlane(incl, nsc - 1);
  const int mo_first = __builtin_amdgcn_readlane(mo_l, 0);
  // chunk size: 256 chunks per launch (32 per XCD) between 16 and 256 tiles
  const int64_t tch = total / 256 < 16 ? 16 : (total / 256 > 256 ? 256 : total / 256);
  // small launches: a quad of waves per tile
  const bool quads = total <= (int)gridDim.x * (CONV_WAVES / 4);
  static_assert(16 * NCB * 64 + 8 * 64 <= WSZ, "quad exchange area exceeds the weight area");
  if (quads ? (int)blockIdx.x >= total : conv_tile(0, tch) >= total) return;  // whole block idle: no weight staging
  // weight and head loads of the whole block in one round trip
  {
    Staged<WSZ, CONV_THREADS> stw;
    Staged<LAST ? HSZ : 1, CONV_THREADS> sth;
    stw.load(reinterpret_cast<const f4*>(a.w), tid);
    if (LAST) sth.load(reinterpret_cast<const f4*>(a.hw), tid);
    if (tid == 0) s_next = 0;
    stw.store(reinterpret_cast<f4*>(s_w), tid);
    if (LAST) sth.store(reinterpret_cast<f4*>(s_h), tid);
  }
  __syncthreads();

  // Opens tile u and sums it.
  auto open = [&](int u, int grp, TileRef& tr, f4 (&sum)[NCB]) {
    const int si = nsc > 1 ? __popcll(__ballot(lane < nsc && incl <= u)) : 0;
    const int n = __builtin_amdgcn_readlane(n_l, si), mo = __builtin_amdgcn_readlane(mo_l, si);
    const int u0 = si ? __builtin_amdgcn_readlane(incl, si - 1) : 0;
    const int row = (u - u0) * 16 + r;
    const bool valid = row < n;
    const int32_t pos = mo + (valid ? row : n - 1);  // idle lanes name a real row
    tr = TileRef{a.b_lo + si, mo, (int64_t)(a.b_lo + si - a.b0) * a.cap_pts, pos, valid};
    conv_sum<C, TBL, BIG>(a, s_w, s_tbl[w], lane, mo, n, (u - u0) * 16, grp, sum);
  };
  if (!quads) {
    // XCD-aware tile order (conv_tile); inside a block the waves take the
    // block's tiles dynamically from an LDS counter: the first CONV_WAVES
    // statically, the rest first come, first served.
    for (int64_t slot = w;;) {
      const int64_t u = conv_tile(slot, tch);
      if (u >= total) break;
      TileRef tr;
      f4 sum[NCB];
      float x[N];
      open((int)u, -1, tr, sum);
      conv_epilogue<C, KIND == CONV_SCATTER>(a, sum, g, tr, x);
      if constexpr (LAST) head_epilogue<C, TWO>(a, x, s_h, lane, g, tr, mo_first);
      int nxt = 0;
      if (lane == 0) nxt = atomicAdd(&s_next, 1);
      slot = CONV_WAVES + __builtin_amdgcn_readfirstlane(nxt);
    }
    return;
  }

  // Small launch (at most one tile per quad of waves): quad q of block x takes
  // tile x + q G, its wave i the offsets of group i, so a tile's serial chain
  // is split four ways.  The group sums meet in the weight area of LDS (free
  // once every conv loop is done) and are added by wave 0 in the same order as
  // above; the 256-way head is split by symbol group the same way.  Every wave
  // passes every barrier (no early exit below).
  {
    const int q = w >> 2, gi = w & 3;
    const int tile = (int)blockIdx.x + (int)gridDim.x * q;
    const bool has = tile < total;  // wave-uniform
    TileRef tr{};
    f4 sum[NCB];
    if (has) open(tile, gi, tr, sum);
    __syncthreads();  // every conv loop of the block is done: the weight area is free
    f4* s_x = reinterpret_cast<f4*>(s_w);                           // [quad][slot 0..3][NCB][64]: group sums 1-3, x
    float2* s_x2 = reinterpret_cast<float2*>(s_x + 16 * NCB * 64);  // [quad][group][64]: (gm, part)
    auto xs = [&](int slot, int cb) -> f4* { return s_x + ((q * 4 + slot) * NCB + cb) * 64 + lane; };
    if (has && gi > 0) {
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) *xs(gi - 1, cb) = sum[cb];
    }
    __syncthreads();
    if (has && gi == 0) {
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        f4 t = f4{0.0f, 0.0f, 0.0f, 0.0f} + sum[cb];
        t += *xs(0, cb);
        t += *xs(1, cb);
        t += *xs(2, cb);
        sum[cb] = t;
      }
      float x[N];
      conv_epilogue<C, KIND == CONV_SCATTER>(a, sum, g, tr, x);
      if constexpr (LAST && !TWO) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)  // the features for the quad's other waves
          *xs(3, cb) = f4{x[4 * cb], x[4 * cb + 1], x[4 * cb + 2], x[4 * cb + 3]};
      }
      if constexpr (LAST && TWO) head_epilogue<C, TWO>(a, x, s_h, lane, g, tr, mo_first);
    }
    if constexpr (LAST && !TWO) {
      __syncthreads();
      if (has) {
        float x[N];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
          const f4 t = *xs(3, cb);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[4 * cb + e] = t[e];
        }
        HeadOp<C> op;
        op.set(x);
        float* lo = (a.logits && tr.valid) ? a.logits + (tr.prow - mo_first) * 256 + 4 * g : nullptr;
        float gm, part;
        head_group<C>(s_h, a.hb, a.hfac, op, lo, lane, g, gi, gm, part);
        s_x2[(q * 4 + gi) * 64 + lane] = make_float2(gm, part);
      }
      __syncthreads();
      if (has && gi == 0) {
        float m = -INFINITY, ssum = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float2 v = s_x2[(q * 4 + k) * 64 + lane];
          lse_merge(m, ssum, v.x, v.y);
        }
        lse_finish(a, m, ssum, g, tr.valid, tr.prow);
      }
    }
  }
}

// Tile order of the streamed-weight layers (k_convw): inside each window of TO_W
// consecutive voxels of a scale, voxels are grouped by an 11-bit signature of
// their neighbour occupancy (the 9 offsets of their own z plane and the two
// z faces), so a 16-voxel tile gathers voxels with similar neighbourhoods and
// the union of occupied offsets a tile must issue shrinks (14-bit scan: about
// 2.4x -> 1.6x the occupied pairs).  A voxel's result does not depend on which
// voxels share its tile (absent offsets add exact zeros), so any order, even
// the arrival order inside a group, gives the same outputs.  One block per
// window: counting sort in LDS.  The first block also clears the work counters
// of the launches that follow.
constexpr int TO_W = 2048;
constexpr int TO_THREADS = 1024;
constexpr int TO_KEYS = 2048;
constexpr int CW_LAYERS = 4;  // launches of k_convw that follow

__global__ void __launch_bounds__(TO_THREADS) k_tile_order(int b_lo, int nsc, RowMap rm, int ks,
                                                           const int32_t* __restrict__ nbr, int32_t* __restrict__ perm,
                                                           uint32_t* __restrict__ next) {
  __shared__ uint32_t s_cnt[TO_KEYS];
  __shared__ uint32_t s_wsum[TO_THREADS / 64];
  __shared__ int64_t s_n[NLEV], s_mo[NLEV];
  __shared__ int64_t s_w0, s_wmo, s_wn;
  const int tid = threadIdx.x;
  if (blockIdx.x == 0 && tid < CW_LAYERS * 8) next[tid] = 0u;
  if (tid < nsc) {  // sizes of the launch's scales, loaded in parallel
    int64_t mo, n;
    scale_span(rm, b_lo + tid, mo, n);
    s_n[tid] = n;
    s_mo[tid] = mo;
  }
  for (int k = tid; k < TO_KEYS; k += TO_THREADS) s_cnt[k] = 0u;
  __syncthreads();
  if (tid == 0) {  // window blockIdx.x -> (scale, first voxel of the window)
    int64_t wacc = 0, w0 = -1;
    for (int i = 0; i < nsc; ++i) {
      const int64_t nw = (s_n[i] + TO_W - 1) / TO_W;
      if (w0 < 0 && (int64_t)blockIdx.x < wacc + nw) {
        w0 = ((int64_t)blockIdx.x - wacc) * TO_W;
        s_wmo = s_mo[i];
        s_wn = s_n[i];
      }
      wacc += nw;
    }
    s_w0 = w0;
  }
  __syncthreads();
  const int64_t w0 = s_w0;
  if (w0 < 0) return;  // beyond the last window (uniform over the block)
  const int64_t mo = s_wmo, n = s_wn;
  constexpr int PER = TO_W / TO_THREADS;
  uint32_t key[PER], rank[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int64_t i = w0 + e * TO_THREADS + tid;
    key[e] = TO_KEYS;  // absent
    if (i < n && ks == 3) {
      const int32_t* r = nbr + (mo + i) * NBR_STRIDE;
      const int4 a = *reinterpret_cast<const int4*>(r + 8), c = *reinterpret_cast<const int4*>(r + 12);
      const int4 d = *reinterpret_cast<const int4*>(r + 16);
      const int f4v = r[4], f22 = r[22];
      // offsets 9..17 (dz = 0), then 4 (dz = -1 face) and 22 (dz = +1 face)
      key[e] = (uint32_t)(a.y >= 0) | ((uint32_t)(a.z >= 0) << 1) | ((uint32_t)(a.w >= 0) << 2) |
               ((uint32_t)(c.x >= 0) << 3) | ((uint32_t)(c.y >= 0) << 4) | ((uint32_t)(c.z >= 0) << 5) |
               ((uint32_t)(c.w >= 0) << 6) | ((uint32_t)(d.x >= 0) << 7) | ((uint32_t)(d.y >= 0) << 8) |
               ((uint32_t)(f4v >= 0) << 9) | ((uint32_t)(f22 >= 0) << 10);
      rank[e] = atomicAdd(&s_cnt[key[e]], 1u);
    } else if (i < n) {
      // 5x5x5 map (stride 128): the same cells, k = (dx+2) + 5(dy+2) + 25(dz+2)
      const int32_t* r = nbr + (mo + i) * 128;
      const int32_t v[11] = {r[56], r[57], r[58], r[61], r[62], r[63], r[66], r[67], r[68], r[37], r[87]};
      uint32_t kk = 0;
#pragma unroll
      for (int j = 0; j < 11; ++j) kk |= (uint32_t)(v[j] >= 0) << j;
      key[e] = kk;
      rank[e] = atomicAdd(&s_cnt[key[e]], 1u);
    }
  }
  __syncthreads();
  // exclusive scan of the TO_KEYS counts: two per thread, wave scans, wave totals
  constexpr int KPT = TO_KEYS / TO_THREADS;
  uint32_t v[KPT], sum = 0;
#pragma unroll
  for (int e = 0; e < KPT; ++e) {
    v[e] = s_cnt[tid * KPT + e];
    sum += v[e];
  }
  uint32_t inc = sum;
  const int lane = tid & 63, w = tid >> 6;
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t t = (uint32_t)__shfl_up((int)inc, d);
    if (lane >= d) inc += t;
  }
  if (lane == 63) s_wsum[w] = inc;
  __syncthreads();
  uint32_t wbase = 0;
  for (int k = 0; k < w; ++k) wbase += s_wsum[k];
  uint32_t ex = wbase + inc - sum;
#pragma unroll
  for (int e = 0; e < KPT; ++e) {
    s_cnt[tid * KPT + e] = ex;
    ex += v[e];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int64_t i = w0 + e * TO_THREADS + tid;
    if (i < n) perm[mo + w0 + s_cnt[key[e]] + rank[e]] = (int32_t)(mo + i);
  }
}

// ---------------------------------------------------------------------------
// Inputs of the full predictor (Sec. 3.2): the neighbour maps of the scales
// it convolves on and the occupancy embeddings X_A = Emb_O[O^{d-1}] (Eq. 6),
// in one launch; one wave per tile of 16 voxels of the scales lo ..
// lo + nsc - 1, the first n_embed of which also get X_A rows.

// Last index si with pre[si] <= e (pre non-decreasing, 32 entries, pre[0] = 0
// <= e): binary lifting, si + step never exceeds 31.
__device__ __forceinline__ int scale_of(const int64_t* pre, int64_t e) {
  int si = 0;
#pragma unroll
  for (int step = 16; step; step >>= 1)
    if (pre[si + step] <= e) si += step;
  return si;
}

// Neighbour rows of a voxel of the base scale, whose parent scale is not
// stored: the 8 cells of lane group g located among the scale's n sorted
// Morton keys by 8 interleaved searches for the last key <= the cell
// (wave-uniform trip count; every probe stays below n).
__device__ __forceinline__ void base_cell_rows(uint64_t kf, int b, int g, const uint64_t* __restrict__ keys,
                                               int64_t n, int32_t (&nb)[8]) {
  const uint64_t key = morton_part(kf, b), fr = kf ^ key;  // frame id bits, in place
  const int x = (int)compact3(key), y = (int)compact3(key >> 1), z = (int)compact3(key >> 2);
  const int lim = 1 << b;
  uint64_t want[8];
  bool ok[8];
  int64_t at[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int k = 8 * g + j;
    const int ux = x + (k % 3) - 1, uy = y + (k / 3) % 3 - 1, uz = z + (k / 9) % 3 - 1;
    ok[j] = k < 27 && ux >= 0 && uy >= 0 && uz >= 0 && ux < lim && uy < lim && uz < lim;
    want[j] = ok[j] ? (fr | morton3((uint32_t)ux, (uint32_t)uy, (uint32_t)uz)) : 0ull;
    at[j] = 0;
  }
  for (int64_t len = n; len > 1;) {
    const int64_t half = len >> 1;
#pragma unroll
    for (int j = 0; j < 8; ++j) at[j] += (keys[at[j] + half] <= want[j]) ? half : 0;
    len -= half;
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) nb[j] = (ok[j] && keys[at[j]] == want[j]) ? (int32_t)at[j] : -1;
}

// Emb_O [256][C] as split rows with the balance of the conv that reads X_A (emb as
// given); 64
// lanes 4r + g per 16 rows.
template <int C>
__global__ void __launch_bounds__(64) k_split_embed(const float* __restrict__ emb, const float* __restrict__ bal,
                                                    uint32_t* __restrict__ rows, float* __restrict__ facs) {
  const int row = blockIdx.x * 16 + (threadIdx.x >> 2), g = threadIdx.x & 3;
  float x[C / 4], y[C / 4];
  load_row<C>(emb + row * C, g, x);
  mul_row<C>(x, bal, g, y);
  auto own = [&](int c0, auto& p) {
#pragma unroll
    for (int i = 0; i < at_once(C); ++i) p[i] = y[c0 + i];
  };
  store_split<C, 1>(own, g, rows + row * C, facs + row);
}

// X_A = Emb_O[code] at a row, as the split row of k_split_embed; lanes 4r + g.
struct EmbedTab {
  const uint32_t* rows;  // [256][C]
  const float* facs;     // [256]
};
template <int C>
__device__ __forceinline__ void embed_row(const EmbedTab& t, int code, int g, int64_t row, uint32_t* __restrict__ XS,
                                          float* __restrict__ XR) {
  const uint4* src = reinterpret_cast<const uint4*>(t.rows + code * C);
  uint4* dst = reinterpret_cast<uint4*>(XS + row * C);
#pragma unroll
  for (int i = g; i < C / 4; i += 4) dst[i] = src[i];
  if (g == 0) XR[row] = t.facs[code];
}

// WIDE: plain map rows, as k_convw reads them; else those of store_map (k_conv).
template <int C, bool WIDE>
__global__ void __launch_bounds__(256) k_top_prep(int lo, int nsc, int n_embed, int b0, RowMap rm,
                                                  const uint64_t* __restrict__ lv_key,
                                                  const uint8_t* __restrict__ lv_code, int64_t cap_pts,
                                                  CellArgs cells, EmbedTab emb_o, int32_t* __restrict__ nbr,
                                                  uint32_t* __restrict__ XS, float* __restrict__ XR) {
  __shared__ uint64_t s_par[4][16][9];  // rows padded: the 16 voxels' cells in different banks
  __shared__ int64_t s_n[32], s_mo[32], s_tpre[32];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int r = lane >> 2, g = lane & 3;  // 4 consecutive lanes per voxel: their accesses to its rows coalesce
  if (tid < nsc) {  // sizes of the launch's scales, loaded in parallel
    int64_t o, n;
    scale_span(rm, lo + tid, o, n);
    s_n[tid] = n;
    s_mo[tid] = o;
  }
  __syncthreads();
  if (tid == 0) {
    int64_t acc = 0;
    for (int i = 0; i < nsc; ++i) {
      s_tpre[i] = acc;
      acc += (s_n[i] + 15) / 16;
    }
    for (int i = nsc; i < 32; ++i) s_tpre[i] = acc;
  }
  __syncthreads();
  const int64_t total = s_tpre[31];
  for (int64_t tile = (int64_t)blockIdx.x * 4 + w; tile < total; tile += (int64_t)gridDim.x * 4) {
    const int si = scale_of(s_tpre, tile);
    const int b = lo + si;
    const int64_t n = s_n[si], mo = s_mo[si];
    const int64_t row = (tile - s_tpre[si]) * 16 + r;
    const bool valid = row < n;
    const int64_t vr = valid ? row : n - 1;  // idle lanes search a real voxel
    const int64_t lvb = (int64_t)(b - b0) * cap_pts;
    int32_t nb[8];
    if (b == rm.b_ext)
      base_cell_rows(lv_key[lvb + vr], b, g, lv_key + lvb, n, nb);
    else
      parent_cell_rows(lv_key[lvb + vr], b, g, cells, s_par[w][r], nb);
    if constexpr (WIDE) {
      if (valid) {
        int4* dst = reinterpret_cast<int4*>(nbr + (mo + vr) * NBR_STRIDE + 8 * g);
        dst[0] = make_int4(nb[0], nb[1], nb[2], nb[3]);
        dst[1] = make_int4(nb[4], nb[5], nb[6], nb[7]);
      }
    } else {
      store_map(nbr, mo + vr, valid, g, nb);
    }
    if (valid && si < n_embed) embed_row<C>(emb_o, lv_code[lvb + vr], g, mo + vr, XS, XR);
  }
}

// ---------------------------------------------------------------------------
// Large kernels and wide layers of the full predictor (5x5x5 kernels, C up to
// 128: the paper's large variant is c128, k5).

// Neighbour rows of a voxel for a 5x5x5 kernel.  The 125 cells around v span
// x-2 .. x+2 on each axis, i.e. the parents p-1 .. p+1: 27 cells of the
// parent scale.  Lane (r, g) probes parent cells e = g, g+4, ... (e = (ex+1) +
// 3(ey+1) + 9(ez+1)), the hits are exchanged through par (27 LDS slots of
// voxel r), and the lane ends with the rows of offsets k = 32g .. 32g+31,
// k = (dx+2) + 5(dy+2) + 25(dz+2) (125 .. 127 padding; -1: absent or
// off-grid).
__device__ __forceinline__ void parent_cell_rows5(uint64_t kf, int b, int g, const CellArgs& a,
                                                  uint64_t* par, int32_t (&nb)[32]) {
  const uint64_t key = morton_part(kf, b), fr = frame_part(kf, b) << (3 * (b - 1));
  const int x = (int)compact3(key), y = (int)compact3(key >> 1), z = (int)compact3(key >> 2);
  const int px = x >> 1, py = y >> 1, pz = z >> 1;
  const int plim = 1 << (b - 1);
  uint64_t cells[7];
  bool ok[7];
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    const int e = g + 4 * i;
    const int cx = px + e % 3 - 1, cy = py + (e / 3) % 3 - 1, cz = pz + e / 9 - 1;
    ok[i] = e < 27 && cx >= 0 && cy >= 0 && cz >= 0 && cx < plim && cy < plim && cz < plim;
    cells[i] = ok[i] ? morton3((uint32_t)cx, (uint32_t)cy, (uint32_t)cz) : 0ull;
  }
  uint2 hit[7];
  find_cells<7>(a, b - 1, fr, cells, ok, hit);
  wave_lds_fence();  // earlier reads of the slots are done
#pragma unroll
  for (int i = 0; i < 7; ++i)
    if (g + 4 * i < 27) par[g + 4 * i] = ((uint64_t)hit[i].y << 32) | hit[i].x;
  wave_lds_fence();
  const int lim = 1 << b;
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    const int k = 32 * g + j;
    const int ux = x + k % 5 - 2, uy = y + (k / 5) % 5 - 2, uz = z + k / 25 - 2;
    nb[j] = -1;
    if (k < 125 && ux >= 0 && uy >= 0 && uz >= 0 && ux < lim && uy < lim && uz < lim) {
      const int e = ((ux >> 1) - px + 1) + 3 * ((uy >> 1) - py + 1) + 9 * ((uz >> 1) - pz + 1);
      const uint64_t pc = par[e];
      const uint32_t first = (uint32_t)pc, code = (uint32_t)(pc >> 32);
      const uint32_t d = (uint32_t)((ux & 1) | ((uy & 1) << 1) | ((uz & 1) << 2));
      if ((code >> d) & 1u) nb[j] = (int32_t)first + __popc(code & ((1u << d) - 1u));
    }
  }
}

// Base-scale rows for a 5x5x5 kernel: the searches of base_cell_rows, eight
// interleaved at a time over the 32 entries of the lane.
__device__ __forceinline__ void base_cell_rows5(uint64_t kf, int b, int g, const uint64_t* __restrict__ keys,
                                                int64_t n, int32_t (&nb)[32]) {
  const uint64_t key = morton_part(kf, b), fr = kf ^ key;
  const int x = (int)compact3(key), y = (int)compact3(key >> 1), z = (int)compact3(key >> 2);
  const int lim = 1 << b;
#pragma unroll
  for (int j0 = 0; j0 < 32; j0 += 8) {
    uint64_t want[8];
    bool ok[8];
    int64_t at[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = 32 * g + j0 + j;
      const int ux = x + k % 5 - 2, uy = y + (k / 5) % 5 - 2, uz = z + k / 25 - 2;
      ok[j] = k < 125 && ux >= 0 && uy >= 0 && uz >= 0 && ux < lim && uy < lim && uz < lim;
      want[j] = ok[j] ? (fr | morton3((uint32_t)ux, (uint32_t)uy, (uint32_t)uz)) : 0ull;
      at[j] = 0;
    }
    for (int64_t len = n; len > 1;) {
      const int64_t half = len >> 1;
#pragma unroll
      for (int j = 0; j < 8; ++j) at[j] += (keys[at[j] + half] <= want[j]) ? half : 0;
      len -= half;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) nb[j0 + j] = (ok[j] && keys[at[j]] == want[j]) ? (int32_t)at[j] : -1;
  }
}

// k_top_prep for a 5x5x5 kernel: neighbour maps of stride 128 and X_A rows.
template <int C>
__global__ void __launch_bounds__(256) k_top_prep5(int lo, int nsc, int n_embed, int b0, RowMap rm,
                                                   const uint64_t* __restrict__ lv_key,
                                                   const uint8_t* __restrict__ lv_code, int64_t cap_pts,
                                                   CellArgs cells, EmbedTab emb_o, int32_t* __restrict__ nbr,
                                                   uint32_t* __restrict__ XS, float* __restrict__ XR) {
  __shared__ uint64_t s_par[4][16][27];
  __shared__ int64_t s_n[32], s_mo[32], s_tpre[32];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, r = lane >> 2, g = lane & 3;
  if (tid < nsc) {
    int64_t o, n;
    scale_span(rm, lo + tid, o, n);
    s_n[tid] = n;
    s_mo[tid] = o;
  }
  __syncthreads();
  if (tid == 0) {
    int64_t acc = 0;
    for (int i = 0; i < nsc; ++i) {
      s_tpre[i] = acc;
      acc += (s_n[i] + 15) / 16;
    }
    for (int i = nsc; i < 32; ++i) s_tpre[i] = acc;
  }
  __syncthreads();
  const int64_t total = s_tpre[31];
  for (int64_t tile = (int64_t)blockIdx.x * 4 + w; tile < total; tile += (int64_t)gridDim.x * 4) {
    const int si = scale_of(s_tpre, tile);
    const int b = lo + si;
    const int64_t n = s_n[si], mo = s_mo[si];
    const int64_t row = (tile - s_tpre[si]) * 16 + r;
    const bool valid = row < n;
    const int64_t vr = valid ? row : n - 1;
    const int64_t lvb = (int64_t)(b - b0) * cap_pts;
    int32_t nb[32];
    if (b == rm.b_ext)
      base_cell_rows5(lv_key[lvb + vr], b, g, lv_key + lvb, n, nb);
    else
      parent_cell_rows5(lv_key[lvb + vr], b, g, cells, s_par[w][r], nb);
    if (valid) {
      int4* dst = reinterpret_cast<int4*>(nbr + (mo + vr) * 128 + 32 * g);
#pragma unroll
      for (int q = 0; q < 8; ++q) dst[q] = make_int4(nb[4 * q], nb[4 * q + 1], nb[4 * q + 2], nb[4 * q + 3]);
      if (si < n_embed) embed_row<C>(emb_o, lv_code[lvb + vr], g, mo + vr, XS, XR);
    }
  }
}

// Offset set of up to 128 offsets (wave-uniform).
struct OffMask {
  uint64_t lo = 0, hi = 0;
  __device__ __forceinline__ bool has(int o) const { return o < 64 ? (lo >> o) & 1ull : (hi >> (o - 64)) & 1ull; }
  // lowest offset, removed from the set (-1 when empty)
  __device__ __forceinline__ int pop() {
    if (lo) {
      const int k = __builtin_ctzll(lo);
      lo &= lo - 1ull;
      return k;
    }
    if (hi) {
      const int k = 64 + __builtin_ctzll(hi);
      hi &= hi - 1ull;
      return k;
    }
    return -1;
  }
};

constexpr int cw_waves(int C) { return C == 128 ? 16 : 8; }         // waves of a block
constexpr unsigned cw_blocks(int C) { return C == 128 ? 256 : 512; }  // 16 waves of 128 registers on each CU
constexpr int64_t CW_SPLIT_TILES = 2048;  // column split up to this many tiles a launch

// The rows of one offset's neighbours as a lane's operands (k_conv's layout,
// one piece per 32 input channels).
template <int C>
struct WideRows {
  static constexpr int NCH = C >= 32 ? C / 32 : 1;
  uint4 hi[NCH], lo[C >= 32 ? NCH : 1];
  float fac = 0.0f;
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) hi[ch] = make_uint4(0u, 0u, 0u, 0u);
    if constexpr (C >= 32) {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) lo[ch] = make_uint4(0u, 0u, 0u, 0u);
    }
  }
  // row < 0: absent, nothing is loaded; the (finite) rows held stay, against the factor 0
  __device__ __forceinline__ void load(const ConvArgs& a, int64_t row, int g) {
    fac = 0.0f;
    if (row < 0) return;
    const uint4* src = reinterpret_cast<const uint4*>(a.h_in + row * C) + g;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      hi[ch] = src[4 * ch];
      if constexpr (C >= 32) lo[ch] = src[C / 8 + 4 * ch];
    }
    fac = a.r_in[row];
  }
};

// acc += fac W_k^T rows for N column blocks, wb their packed operands of the
// offset ([block][32-channel piece][plane][64]); a piece's smallest products first.
template <int C, int N>
__device__ __forceinline__ void wide_mma(const uint4* wb, int lane, const WideRows<C>& x, f4* acc) {
  constexpr int NCH = WideRows<C>::NCH, PL = weight_planes(C);
  f4 p[N];
#pragma unroll
  for (int q = 0; q < N; ++q) p[q] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  auto w = [&](int q, int ch, int pl) { return wb[((q * NCH + ch) * PL + pl) * 64 + lane]; };
  if constexpr (C >= 32) {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      uint4 wh[N];
#pragma unroll
      for (int q = 0; q < N; ++q) p[q] = mfma_h(w(q, ch, 1), x.hi[ch], p[q]);
#pragma unroll
      for (int q = 0; q < N; ++q) {
        wh[q] = w(q, ch, 0);
        p[q] = mfma_h(wh[q], x.lo[ch], p[q]);
      }
#pragma unroll
      for (int q = 0; q < N; ++q) p[q] = mfma_h(wh[q], x.hi[ch], p[q]);
    }
  } else {
#pragma unroll
    for (int pl = PL - 1; pl >= 0; --pl)
#pragma unroll
      for (int q = 0; q < N; ++q) p[q] = mfma_h(w(q, 0, pl), x.hi[0], p[q]);
  }
#pragma unroll
  for (int q = 0; q < N; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[q][e] = fmaf(p[q][e], x.fac, acc[q][e]);
}

// A block's view of the scales of a launch (in LDS).
struct WideScales {
  int64_t tpre[NLEV + 1];  // first tile of each scale
  int64_t nv[NLEV], mo[NLEV];
};

// Tile `tile` as lane (r, .) sees it; idle lanes name a real row.
__device__ __forceinline__ TileRef wide_tile(const ConvArgs& a, const WideScales& sc, int64_t tile, int r) {
  int si = 0;
#pragma unroll
  for (int i = 1; i < NLEV; ++i) si += (sc.tpre[i] <= tile) ? 1 : 0;
  const int64_t nvox = sc.nv[si];
  const int64_t row = (tile - sc.tpre[si]) * 16 + r;
  TileRef tr;
  tr.b = a.b_lo + si;
  tr.mo = sc.mo[si];
  tr.lvb = (int64_t)(tr.b - a.b0) * a.cap_pts;
  tr.valid = row < nvox;
  const int64_t pos = tr.mo + (tr.valid ? row : nvox - 1);
  tr.prow = a.perm ? (int64_t)a.perm[pos] : pos;  // with a tile order, slot -> row
  return tr;
}

// A lane's share of a tile's map rows (lane (r, g): entries EPL g .. of voxel r;
// -1 where `have` is false or the voxel is not valid) and the tile's occupied offsets.
template <int EPL>
__device__ __forceinline__ OffMask wide_map(const ConvArgs& a, const TileRef& tr, bool have, int g, int32_t (&nbv)[EPL]) {
#pragma unroll
  for (int q = 0; q < EPL / 4; ++q) {
    int4 t = make_int4(-1, -1, -1, -1);
    if (have && tr.valid) t = reinterpret_cast<const int4*>(a.nbr + tr.prow * (4 * EPL) + EPL * g)[q];
    nbv[4 * q] = t.x;
    nbv[4 * q + 1] = t.y;
    nbv[4 * q + 2] = t.z;
    nbv[4 * q + 3] = t.w;
  }
  uint32_t mine = 0;
#pragma unroll
  for (int j = 0; j < EPL; ++j) mine |= (nbv[j] >= 0 ? 1u : 0u) << j;
  mine = or_row16(mine);
  uint64_t q[4];
#pragma unroll
  for (int gg = 0; gg < 4; ++gg) q[gg] = (uint32_t)__builtin_amdgcn_readlane((int)mine, 16 * gg);
  OffMask own;
  if constexpr (EPL == 32) {
    own.lo = q[0] | (q[1] << 32);
    own.hi = q[2] | (q[3] << 32);
  } else {
    own.lo = q[0] | (q[1] << EPL) | (q[2] << 2 * EPL) | (q[3] << 3 * EPL);
  }
  return own;
}

// v, as a value that the compiler knows nothing of: addresses formed from it stay
// where they are used instead of in registers across the walk over the offsets.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The lane, formed anew: in the staged walk over the offsets, whose registers are
// full at C = 128, a lane index kept across an offset went through scratch.
__device__ __forceinline__ int lane_now() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// Shapes of k_convw.  Staged form: one tile per wave.  Column-split form: half
// of the waves multiply, one column block each (SG tile subgroups of NCB waves),
// the others fetch the rows of their subgroup's tiles, one of the NCB slices
// (32-channel piece, plane) of a row each; SLOTS tiles per subgroup.
template <int C, int KV>
struct WideShape {
  static constexpr int WAVES = cw_waves(C), THREADS = 64 * WAVES;
  static constexpr int NCB = C / 16, NCH = WideRows<C>::NCH, PL = weight_planes(C);
  static constexpr int NBS = KV > 27 ? 128 : NBR_STRIDE, EPL = NBS / 4;  // map row, entries per lane
  static constexpr int CBW = NCH * PL * 64;  // 16-byte words of a column block's weights of an offset
  static constexpr int WQ = NCB * CBW;       // of all of them
  static constexpr bool SPLITS = NCB > 1;
  static constexpr int SG = SPLITS ? WAVES / 2 / NCB : 1, SLOTS = SPLITS ? 4 / SG : 0, TILES = SG * SLOTS;
  static constexpr int ROWS = 2 * TILES * NCB * 64;  // 16-byte words: rows of two offsets,
  static constexpr int MAP = TILES * NBS * 16 / 4;   // the tiles' maps [offset][voxel],
  static constexpr int FAC = 2 * TILES * 16 / 4;     // the rows' factors
  static constexpr int LDS = 2 * WQ > ROWS + MAP + FAC ? 2 * WQ : ROWS + MAP + FAC;
};

// Column-split form of k_convw, for launches whose tiles would leave most CUs
// idle at one tile per wave.  A block takes up to TILES tiles and walks the union
// of their occupied offsets; at each, a multiplying wave holds its column block's
// weights in registers and reads the tiles' rows from LDS, so that the tiles
// share one read of the weights, which bounds these launches (64 KB an offset and
// block at C = 128).  Both weights (two sets of registers) and rows (two LDS
// buffers, the gathers of one more in registers) are fetched one offset ahead.
// With one tile's column block per wave, its weights and rows loaded after the
// products of the offset before, a decoder's launches at C = 128 took 447 to 690
// us with 5x5x5 kernels and 96 to 147 us with 3x3x3 ones; now 96 to 420 and 34 to
// 48 (16 to 64 beams, 11 and 12 bits).
template <int C, int KV, bool XB>
__device__ __forceinline__ void convw_split(const ConvArgs& a, const WideScales& sc, uint4* s_buf,
                                            uint64_t (*s_mask)[2], int64_t total_tiles, int tps, int w, int lane0) {
  using S = WideShape<C, KV>;
  constexpr int NCB = S::NCB, NCH = S::NCH, SLOTS = S::SLOTS, TILES = S::TILES, WR = S::CBW / 64;
  static_assert(NCB >= SLOTS && NCB == 2 * NCH, "a fetching wave per row slice, one of them per tile's factors");
  uint4* s_rows = s_buf;                                            // [2][TILES][NCB][64]
  int32_t* s_map = reinterpret_cast<int32_t*>(s_buf + S::ROWS);     // [TILES][NBS][16]
  float* s_fac = reinterpret_cast<float*>(s_buf + S::ROWS + S::MAP);  // [2][TILES][16]
  const bool mult = w < S::WAVES / 2;  // multiplying wave
  const int sg = (w % (S::WAVES / 2)) / NCB, cb = w % NCB;
  for (int64_t set = blockIdx.x; set * tps < total_tiles; set += gridDim.x) {
    __syncthreads();  // prefix visible; the previous set is done with the LDS
    const int lane = opaque(lane0), r = lane & 15, g = lane >> 4;
    const uint4* wsrc = reinterpret_cast<const uint4*>(a.w) + cb * S::CBW + lane;
    // wave w opens tile w
    const int64_t tile = set * tps + w;
    const bool have = w < tps && tile < total_tiles;
    TileRef tr{a.b_lo, 0, 0, 0, false};
    if (w < TILES) {
      if (have) tr = wide_tile(a, sc, tile, r);
      int32_t nbv[S::EPL];
      const OffMask own = wide_map<S::EPL>(a, tr, have, g, nbv);
#pragma unroll
      for (int j = 0; j < S::EPL; ++j)
        s_map[(w * S::NBS + S::EPL * g + j) * 16 + r] = nbv[j] >= 0 ? (int32_t)tr.mo + nbv[j] : -1;
      if (lane == 0) {
        s_mask[w][0] = own.lo;
        s_mask[w][1] = own.hi;
      }
    }
    __syncthreads();
    OffMask uni, m[SLOTS];  // of the set, and of the subgroup's tiles
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      uni.lo |= uniform64(s_mask[t][0]);
      uni.hi |= uniform64(s_mask[t][1]);
    }
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
      m[j].lo = uniform64(s_mask[j * S::SG + sg][0]);
      m[j].hi = uniform64(s_mask[j * S::SG + sg][1]);
    }
    // a multiplying wave's sums, a fetching wave's rows in flight
    f4 st[SLOTS];
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) st[j] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    float vf = 0.0f;  // fetching wave of slice j < SLOTS: slot j's factors in flight
    uint4 wv[2][WR];
    auto weights = [&](int k, uint4 (&v)[WR]) {
#pragma unroll
      for (int i = 0; i < WR; ++i) v[i] = wsrc[(int64_t)k * S::WQ + i * 64];
    };
    auto fetch = [&](int k) {
#pragma unroll
      for (int j = 0; j < SLOTS; ++j) {
        if (!m[j].has(k)) continue;
        const int32_t row = s_map[((j * S::SG + sg) * S::NBS + k) * 16 + r];
        if (row >= 0)
          st[j] = reinterpret_cast<const f4*>(a.h_in + (int64_t)row * C)[(cb & 1) * (C / 8) + 4 * (cb >> 1) + g];
        if (cb == j) vf = row >= 0 ? a.r_in[row] : 0.0f;
      }
    };
    auto put = [&](int k, int buf) {
#pragma unroll
      for (int j = 0; j < SLOTS; ++j) {
        if (!m[j].has(k)) continue;
        const int t = buf * TILES + j * S::SG + sg;
        s_rows[(t * NCB + cb) * 64 + lane] = __builtin_bit_cast(uint4, st[j]);
        if (cb == j && g == 0) s_fac[t * 16 + r] = vf;
      }
    };
    auto mma = [&](int k, const uint4 (&v)[WR], int buf) {
#pragma unroll
      for (int j = 0; j < SLOTS; ++j) {
        if (!m[j].has(k)) continue;
        const int t = buf * TILES + j * S::SG + sg;
        const uint4* x = s_rows + t * NCB * 64 + lane;
        const float fac = s_fac[t * 16 + r];
        f4 p = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {  // the chain of wide_mma
          const uint4 hi = x[2 * ch * 64], lo = x[(2 * ch + 1) * 64];
          p = mfma_h(v[2 * ch + 1], hi, p);
          p = mfma_h(v[2 * ch], lo, p);
          p = mfma_h(v[2 * ch], hi, p);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) st[j][e] = fmaf(p[e], fac, st[j][e]);
      }
    };
    int kc = uni.pop(), kn = uni.pop();
    if (kc >= 0) {  // block-uniform
      if (mult) {
        weights(kc, wv[0]);
        weights(kn >= 0 ? kn : kc, wv[1]);
      } else {
        fetch(kc);
        put(kc, 0);
        if (kn >= 0) fetch(kn);
      }
      __syncthreads();
      // one offset: products of kc from set BUF, rows of kn to the other buffer,
      // the loads of the offset after
      auto step = [&](auto which) {
        constexpr int BUF = decltype(which)::value;
        const int kf = uni.pop();
        if (mult) {
          mma(kc, wv[BUF], BUF);
          weights(kf >= 0 ? kf : kc, wv[BUF]);  // unconditional: exact waits
        } else {
          if (kn >= 0) put(kn, BUF ^ 1);
          if (kf >= 0) fetch(kf);
        }
        __syncthreads();
        kc = kn;
        kn = kf;
        return kc >= 0;
      };
      while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{})) {
      }
    }
    // the column blocks of a tile meet in LDS; wave t goes on with tile t
    f4* s_x = reinterpret_cast<f4*>(s_rows);  // [TILES][NCB][64]
    if (mult) {
#pragma unroll
      for (int j = 0; j < SLOTS; ++j) s_x[((j * S::SG + sg) * NCB + cb) * 64 + lane] = st[j];
    }
    __syncthreads();
    if (!have) continue;
    f4 acc[NCB];
#pragma unroll
    for (int q = 0; q < NCB; ++q) acc[q] = s_x[(w * NCB + q) * 64 + lane];
    float x[C / 4];
    const int l2 = opaque(lane);  // the tile is opened again: held across the walk it would cost registers there
    conv_epilogue<C, XB>(a, acc, l2 >> 4, wide_tile(a, sc, tile, l2 & 15), x);
  }
}

// Sparse conv C -> C (ReLU, optional residual input, child scatter and row
// store as in k_conv) with the weights streamed, for layers whose weights do
// not fit in LDS (a 5x5x5 kernel at C = 128 holds 8 MB).  Staged form: a block
// takes groups of tiles, one per wave.  For each offset in the union of the
// group's occupied offsets, in ascending order, the block stages that offset's
// weights in LDS (one offset ahead there, the one after in flight), and each wave
// whose tile has the offset adds its gathered neighbour rows on split fp16 MFMA as
// k_conv does and gathers its next rows into the same registers.  Launches with
// few tiles take the column-split form above.  A voxel adds its offsets in
// ascending order, each chained from zero, whatever its group or form, so results
// do not depend on the grouping.
//
// A 5x5x5 layer at C = 128 is bound by the weights' way from memory (8 MB do
// not stay in a 4 MB L2: half of the lines miss, 3.7 GB a layer of the 64-beam
// scan's encoder launch), so its groups are as large as the waves of a CU allow,
// 16 tiles on 16 waves; with 8 waves of twice the registers and the rows gathered
// ahead into a second set it took 2.0 ms instead of 1.55 (64-beam scan at 14 bits,
// mean of the layers; 4.2 ms on fp32 MFMA).  128 registers a wave hold a tile's
// sums and rows at C = 128 with little to spare: a few values of the opening and
// the epilogue go through scratch (52 to 104 bytes a lane; at C = 64 up to 12 in
// the layer that feeds the children), none of the walk: one lane index reloaded for
// each gather cost 8 % of the encoder's launch, for it waits for all loads in flight.
// Groups differ in their offsets (27 to 125), so blocks take them first come,
// first served, their own XCD's share before the others' (2.33 -> 2.0 ms in the
// 8-wave form).
//
// Staged against column-split form, us a launch by tiles (one scale of LiDAR
// scans per call, mean of the four layers):
//   tiles        137   294   555   974  1227  2027  2320  4220  6699
//   C 128 k 5  496/157 537/190 525/228 526/262 528/350 545/418 561/573 678/801 981/1152
//   C 128 k 3  147/44  156/50  160/59  159/68  163/80  169/104 176/141 219/211 296/305
//   C  64 k 5  158/71  162/72  157/87  156/100 165/117 179/139 192/196 262/268 331/371
//   C  64 k 3   49/26   50/28   52/32   55/37   59/42   67/48   73/63  103/89  119/120
//   C  32 k 5   91/61   94/68   95/64   95/66  104/79  114/84  123/123 166/161 201/217
// so launches of up to CW_SPLIT_TILES = 2048 tiles split.
template <int C, int KV, bool XB>
__global__ void __launch_bounds__(64 * cw_waves(C), 4) k_convw(ConvArgs a) {
  using S = WideShape<C, KV>;
  constexpr int CW_WAVES = S::WAVES, CW_THREADS = S::THREADS, NCB = S::NCB, CBW = S::CBW, WQ = S::WQ;
  __shared__ uint4 s_buf[S::LDS];  // staged form: the weights of two offsets
  __shared__ uint64_t s_mask[CW_WAVES][2];
  __shared__ WideScales s_sc;
  __shared__ int64_t s_next[2];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int r = lane & 15, g = lane >> 4;
  const int nsc = a.b_hi - a.b_lo + 1;
  const RowMap rm{a.count, a.moff, a.cap_model, a.b_ext, a.ext_off, a.cap_rows};
  int64_t total_tiles = 0;
  for (int i = 0; i < nsc; ++i) {
    int64_t mo, nb;
    scale_span(rm, a.b_lo + i, mo, nb);
    total_tiles += (nb + 15) / 16;
  }
  const int64_t groups = (total_tiles + CW_WAVES - 1) / CW_WAVES;
  const int64_t tch = groups / 64 < 4 ? 4 : (groups / 64 > 64 ? 64 : groups / 64);
  const bool split = S::SPLITS && total_tiles <= CW_SPLIT_TILES;  // uniform
  // tiles of a column-split block: as few per subgroup as give every block one set
  const int64_t per = (total_tiles + (int64_t)gridDim.x * S::SG - 1) / ((int64_t)gridDim.x * S::SG);
  const int tps = S::SG * (int)(per < 1 ? 1 : (per > S::SLOTS ? S::SLOTS : per));
  if (split ? (int64_t)blockIdx.x * tps >= total_tiles : conv_tile(0, tch) >= groups) return;  // whole block idle
  if (tid == 0) {
    int64_t acc = 0;
    for (int i = 0; i < nsc; ++i) {
      int64_t mo, nb;
      scale_span(rm, a.b_lo + i, mo, nb);
      s_sc.tpre[i] = acc;
      s_sc.nv[i] = nb;
      s_sc.mo[i] = mo;
      acc += (nb + 15) / 16;
    }
    for (int i = nsc; i <= NLEV; ++i) s_sc.tpre[i] = acc;
  }
  if constexpr (S::SPLITS) {
    if (split) {
      convw_split<C, KV, XB>(a, s_sc, s_buf, s_mask, total_tiles, tps, w, lane);
      return;
    }
  }
  const uint4* wsrc = reinterpret_cast<const uint4*>(a.w);
  WideRows<C> xa;
  xa.clear();
  int vic = blockIdx.x & 7;  // thread 0: the XCD whose share the block takes groups of
  for (int64_t gs = 0;; ++gs) {
    __syncthreads();  // prefix and s_next visible; the previous group is done with s_mask and s_buf
    const int64_t grp = gs == 0 ? conv_tile(0, tch) : s_next[gs & 1];  // block-uniform
    if (grp >= groups) break;
    if (tid == 0) {  // the next group, read after the next turn's barrier
      int64_t ng = groups;
      for (int t = 0; t < 8; ++t) {
        ng = xcd_tile(vic, (gridDim.x >> 3) + (int64_t)atomicAdd(a.next + vic, 1u), tch);
        if (ng < groups) break;
        vic = (vic + 1) & 7;
      }
      s_next[(gs + 1) & 1] = ng;
    }
    const int64_t tile = grp * CW_WAVES + w;
    const bool have = tile < total_tiles;
    TileRef tr{a.b_lo, 0, 0, 0, false};
    if (have) tr = wide_tile(a, s_sc, tile, r);
    OffMask own;
    {
      int32_t nbv[S::EPL];
      own = wide_map<S::EPL>(a, tr, have, g, nbv);
    }
    // each lane reads its own voxel's map entry of an offset one of the wave's
    // offsets ahead of the gather, which follows the products of the offset
    // before into the same registers
    const int32_t* maprow = a.nbr + tr.prow * S::NBS;
    auto entry = [&](int k) -> int32_t { return (k >= 0 && have) ? maprow[k] : -1; };
    auto gather = [&](int32_t nn) { xa.load(a, tr.valid && nn >= 0 ? tr.mo + nn : -1, lane_now() >> 4); };
    f4 acc[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[cb] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    if (lane == 0) {
      s_mask[w][0] = own.lo;
      s_mask[w][1] = own.hi;
    }
    int ko = own.pop();
    const int32_t eo = entry(ko);
    int kq = own.pop();
    int32_t eq = entry(kq);
    if (ko >= 0) gather(eo);
    __syncthreads();
    OffMask uni;
    for (int ww = 0; ww < CW_WAVES; ++ww) {
      uni.lo |= s_mask[ww][0];
      uni.hi |= s_mask[ww][1];
    }
    int kc = uni.pop(), kn = uni.pop();
    Staged<WQ, CW_THREADS> stw;
    auto weights = [&](int k) { stw.load(reinterpret_cast<const f4*>(wsrc + (int64_t)k * WQ), tid); };
    // a group can have no offset at all: base voxels that are not in order (an
    // error that the host learns of later) are not even found as their own neighbours
    if (kc >= 0) {
      weights(kc);
      stw.store(reinterpret_cast<f4*>(s_buf), tid);
    }
    if (kn >= 0) weights(kn);
    __syncthreads();
    int buf = 0;
    while (kc >= 0) {  // block-uniform
      const bool mine = kc == ko;
      if (mine) {
        constexpr int NB = NCB == 2 || NCB == 4 ? 2 : 1;
#pragma unroll
        for (int cb = 0; cb < NCB; cb += NB) {
          wide_mma<C, NB>(s_buf + buf * WQ + cb * CBW, lane, xa, acc + cb);
          __builtin_amdgcn_sched_barrier(0);  // operands of all blocks at once would not fit the registers
        }
      }
      kc = kn;
      if (kn >= 0) {  // weights one offset ahead in LDS, two ahead in flight
        stw.store(reinterpret_cast<f4*>(s_buf + (buf ^ 1) * WQ), tid);
        kn = uni.pop();
        if (kn >= 0) weights(kn);
      }
      if (mine) {
        ko = kq;
        if (ko >= 0) gather(eq);
        kq = own.pop();
        eq = entry(kq);
      }
      __syncthreads();
      buf ^= 1;
    }
    if (!have) continue;
    float x[C / 4];
    const int l2 = opaque(lane);  // opened again, as in the column-split form
    conv_epilogue<C, XB>(a, acc, l2 >> 4, wide_tile(a, s_sc, tile, l2 & 15), x);
  }
}

// Threads and blocks of a k_headw launch.  C >= 64 needs more registers than 16
// waves per CU allow (112 to 190 a wave), and there the blocks are no more than
// are resident at once: the grid has to cover the largest scale of the context,
// every further block would stage the head for a tile or two, or for none.  One
// stage, C = 128 (128 KB staged, one block a CU): 8 waves, 11 us at 16 beams 11
// bits, 18 at 64 beams 14 bits (decoder), 76 us in the encoder's launch; 4 waves
// 11, 20, 106; 16 waves, with scratch, 18, 24, 70 (4 waves and up to 4096 blocks,
// idle ones staging too: 11, 50, 150).  C = 64 with 4 waves 7, 11, 46, with 8 waves
// 8, 11, 44 (before: 7, 21, 66).  Two stages, C = 128: 512 blocks 8 us (decoder, 64
// beams) and 47 (encoder), 1024 8 and 49, 4096 9 and 69 (idle ones staging: 14, 62).
template <int C, bool TWO>
constexpr int headw_threads() { return C < 64 ? 1024 : (C == 128 && !TWO ? 512 : 256); }
template <int C, bool TWO>
constexpr int headw_blocks() { return C >= 64 ? (C == 128 && !TWO ? 256 : 512) : (TWO ? 4096 : 1024); }

// The head on stored last-layer features h_in (rows of the scales b_lo ..
// b_hi), for layers computed by k_convw: one wave per tile of 16 voxels, the
// head weights in LDS, the same arithmetic as the fused head of k_conv.
template <int C, bool TWO>
__global__ void __launch_bounds__((headw_threads<C, TWO>())) k_headw(ConvArgs a) {
  constexpr int HT = headw_threads<C, TWO>();
  constexpr int HWV = HT / 64;
  constexpr int HQ = (TWO ? 2 : 16) * HeadOp<C>::BLOCK;  // 16-byte words of the packed head
  __shared__ uint4 s_h[HQ];
  __shared__ int64_t s_tpre[NLEV + 1];
  __shared__ int64_t s_nv[NLEV];
  __shared__ int64_t s_mo[NLEV];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int nsc = a.b_hi - a.b_lo + 1;
  const RowMap rm{a.count, a.moff, a.cap_model, -1, 0, a.cap_model + 1};
  int64_t total = 0;
  for (int i = 0; i < nsc; ++i) {
    int64_t mo, nb;
    scale_span(rm, a.b_lo + i, mo, nb);
    total += (nb + 15) / 16;
  }
  if ((int64_t)blockIdx.x * HWV >= total) return;  // whole block idle: no staging
  Staged<HQ, HT> sth;
  sth.load(reinterpret_cast<const f4*>(a.hw), tid);
  if (tid == 0) {
    int64_t acc = 0;
    for (int i = 0; i < nsc; ++i) {
      int64_t mo, nb;
      scale_span(rm, a.b_lo + i, mo, nb);
      s_tpre[i] = acc;
      s_nv[i] = nb;
      s_mo[i] = mo;
      acc += (nb + 15) / 16;
    }
    for (int i = nsc; i <= NLEV; ++i) s_tpre[i] = acc;
  }
  sth.store(reinterpret_cast<f4*>(s_h), tid);
  __syncthreads();
  for (int64_t tile = (int64_t)blockIdx.x * HWV + w; tile < total; tile += (int64_t)gridDim.x * HWV) {
    int si = 0;
#pragma unroll
    for (int i = 1; i < NLEV; ++i) si += (s_tpre[i] <= tile) ? 1 : 0;
    const int64_t nvox = s_nv[si], mo = s_mo[si];
    const int64_t row = (tile - s_tpre[si]) * 16 + r;
    const bool valid = row < nvox;
    const TileRef tr{a.b_lo + si, mo, (int64_t)(a.b_lo + si - a.b0) * a.cap_pts, mo + (valid ? row : nvox - 1), valid};
    float x[C / 4];
    load_row<C>(a.h_in + tr.prow * C, g, x);
    head_epilogue<C, TWO>(a, x, s_h, lane, g, tr, s_mo[0]);
  }
}

template <int C>
hipError_t run_headw(Ctx& c, bool two, const ConvArgs& a) {
  auto go = [&](auto kern, int threads, int most) {
    const int64_t per = threads / 4;  // voxels of a block's waves: 16 each
    const int64_t blocks = std::min<int64_t>(most, (c.cap_model + per - 1) / per);
    if (c.ext_start) {  // timed: the events are the dispatch's own start and end
      hipExtLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(threads), 0, c.stream, c.ext_start, c.ext_stop, 0u, a);
      c.ext_start = c.ext_stop = nullptr;
    } else {
      hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(threads), 0, c.stream, a);
    }
    return hipGetLastError();
  };
  return two ? go(k_headw<C, true>, headw_threads<C, true>(), headw_blocks<C, true>())
             : go(k_headw<C, false>, headw_threads<C, false>(), headw_blocks<C, false>());
}

// ---------------------------------------------------------------------------
// First conv layer of the plain model, with the neighbour search.
//
// Its 11 input bits are the voxel's octant and its parent's code, so what the
// children of one parent-scale cell add to a voxel's sum depends only on the
// voxel's octant (8), which of the 8 cells around it the cell is (8) and the
// cell's code (256): F[oct][e][code] [C] = the sum over the cell's occupied
// children that touch the voxel of W[k]^T [delta, code].  The table is formed
// once per weight set, in double (times the balance obal of the layer's output),
// and the layer is the bias plus 8 rows of it,
// in cell order (code 0, an absent cell, has a zero row).
//
// Bound by the probe -> row latency chain and L2 reads (8 C-float rows per
// voxel; the whole table is 2 MB at C = 32 and stays in each XCD's L2).  One
// wave per 16 voxels, 4 lanes per voxel: they probe two cells each, exchange
// the hits through LDS and then sum C / 4 channels each.  Small blocks without
// staged weights, so that more waves hide the chain than the LDS-resident conv
// kernel allows.  Against the former layer (27 offsets gathered and issued as
// fp32 MFMA in the conv kernel): 14-bit scan 56 -> 34 us in the encoder's
// launch, 131 -> 84 us over the decoder's nine; 10 frames 500 -> 380 us; 16-bit
// 128-beam scan 159 -> 127 us.  8 unconditional rows per voxel instead of the
// occupied cells' only took 42 us at 14 bits.
template <int C>
__global__ void __launch_bounds__(256) k_first_table(const float* __restrict__ W, const float* __restrict__ obal,
                                                     float* __restrict__ F) {
  const int co = threadIdx.x % C;
  const int row = blockIdx.x * (256 / C) + threadIdx.x / C;  // (oct * 8 + e) * 256 + code
  const uint32_t code = row & 255u, e = (row >> 8) & 7u, oct = (uint32_t)row >> 11;
  double acc = 0.0;
  for (uint32_t d = 0; d < 8; ++d) {
    if (!((code >> d) & 1u)) continue;
    // per axis, the child's cell minus the voxel's: in v's parent d - oct; in
    // the neighbour cell on v's side 1 + d or d - 2, touching when that is +-1
    int k = 0;
    bool touch = true;
    for (int ax = 2; ax >= 0; --ax) {
      const int o = (oct >> ax) & 1, dd = (d >> ax) & 1;
      const int step = ((e >> ax) & 1u) ? (o ? 1 + dd : dd - 2) : dd - o;
      touch = touch && step >= -1 && step <= 1;
      k = 3 * k + step + 1;
    }
    if (!touch) continue;
    const float* w = W + (size_t)k * RENO_IN_FEATURES * C + co;
    for (int i = 0; i < 3; ++i)
      if ((d >> i) & 1u) acc += (double)w[i * C];
    for (int i = 0; i < 8; ++i)
      if ((code >> i) & 1u) acc += (double)w[(3 + i) * C];
  }
  F[(size_t)row * C + co] = (float)acc * obal[co];
}

struct FirstArgs {
  int b_lo, nsc;
  RowMap rm;
  CellArgs cells;
  const uint64_t* lv_key;
  const float* table;    // [8][8][256][C]
  const float* bias;     // [C]
  int32_t* nbr;          // [rows][NBR_STRIDE]
  float* out;            // fp32 output rows [rows][C], or NULL
  uint32_t* s_out;       // split output rows, or NULL
  float* r_out;          // their factors
};

constexpr int FIRST_WAVES = 4;

template <int C>
__global__ void __launch_bounds__(64 * FIRST_WAVES, 4) k_first(FirstArgs a) {
  constexpr int Q = C / 16;  // f4 words of a lane's C / 4 channels
  __shared__ uint64_t s_par[FIRST_WAVES][16][9];  // rows padded: the 16 voxels' cells in different banks
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int r = lane >> 2, g = lane & 3;  // 4 consecutive lanes per voxel: their accesses to its rows coalesce
  // lane i holds scale i of the launch: rows, first row, inclusive tile prefix
  int64_t n_l = 0, mo_l = 0;
  if (lane < a.nsc) scale_span(a.rm, a.b_lo + lane, mo_l, n_l);
  int incl = (int)((n_l + 15) / 16);
  if (a.nsc > 1) {
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
      const int y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
  }
  const int total = __builtin_amdgcn_readlane(incl, a.nsc - 1);
  // chunks of consecutive tiles are dealt to the XCDs (blockIdx % 8) in turn,
  // as conv_tile does
  const int tch = total / 256 < FIRST_WAVES ? FIRST_WAVES : (total / 256 > 256 ? 256 : total / 256);
  const int xcd = blockIdx.x & 7, step = (int)(gridDim.x >> 3) * FIRST_WAVES;
  for (int j = (int)(blockIdx.x >> 3) * FIRST_WAVES + w;; j += step) {
    const int tile = ((j / tch) * 8 + xcd) * tch + j % tch;
    if (tile >= total) break;
    const int si = __popcll(__ballot(lane < a.nsc && incl <= tile));
    const int b = a.b_lo + si;
    const int n = __builtin_amdgcn_readlane((int)n_l, si);       // voxel and model-row counts stay below 2^30
    const int64_t mo = __builtin_amdgcn_readlane((int)mo_l, si);
    const int t0 = si ? __builtin_amdgcn_readlane(incl, si - 1) : 0;
    const int row = (tile - t0) * 16 + r;
    const bool valid = row < n;
    const int vr = valid ? row : n - 1;  // idle lanes search a real voxel
    const uint64_t key = a.lv_key[(int64_t)(b - a.cells.b0) * a.cells.cap_pts + vr];
    int32_t nb[8];
    uint64_t* par = s_par[w][r];
    parent_cell_rows(key, b, g, a.cells, par, nb);
    // lane g takes channels 16 q + 4 g .. + 3: the 4 lanes of a voxel read 64
    // contiguous bytes; absent cells (code 0) load nothing
    const f4* T = reinterpret_cast<const f4*>(a.table) + (size_t)((uint32_t)key & 7u) * (8 * 256 * C / 4) + g;
    f4 v[8][Q];
    uint32_t code[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      code[e] = (uint32_t)(par[e] >> 32);
#pragma unroll
      for (int q = 0; q < Q; ++q) v[e][q] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (code[e]) {
        const f4* src = T + (size_t)(e * 256 + (code[e] & 255u)) * (C / 4);
#pragma unroll
        for (int q = 0; q < Q; ++q) v[e][q] = src[4 * q];
      }
    }
    const int64_t prow = mo + vr;
    store_map(a.nbr, prow, valid, g, nb);
    float x[C / 4];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      f4 acc = reinterpret_cast<const f4*>(a.bias)[4 * q + g];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc += v[e][q];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[4 * q + i] = fmaxf(acc[i], 0.0f);
    }
    if (!valid) continue;
    if (a.s_out) {
      uint32_t hi[C / 8], lo[C / 8];
      const float f = row_split<C / 4, 1>(x, hi, lo);
      uint32_t* orow = a.s_out + prow * C;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        *reinterpret_cast<uint2*>(orow + 8 * q + 2 * g) = make_uint2(hi[2 * q], hi[2 * q + 1]);
        *reinterpret_cast<uint2*>(orow + C / 2 + 8 * q + 2 * g) = make_uint2(lo[2 * q], lo[2 * q + 1]);
      }
      if (g == 0) a.r_out[prow] = f;
    }
    if (a.out) {
#pragma unroll
      for (int q = 0; q < Q; ++q)
        reinterpret_cast<f4*>(a.out + prow * C)[4 * q + g] = f4{x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
    }
  }
}

CellArgs cell_args(const Ctx& c) {
  return CellArgs{c.d_hash, c.hash_lg, c.hreg(), c.fbits, c.b0(), c.cap_pts, c.lv_code, c.lv_fc};
}

EmbedTab embed_tab(const Ctx& c) { return EmbedTab{c.w_embs, c.w_embr}; }

template <int C>
hipError_t run_first(Ctx& c, const FirstArgs& a) {
  // 8 blocks per CU at most; fewer when the capacity cannot fill them
  int64_t blocks = ((c.cap_model + 16 * FIRST_WAVES - 1) / (16 * FIRST_WAVES) + 7) & ~int64_t(7);
  if (blocks > 2048) blocks = 2048;
  if (c.ext_start) {  // timed: the events are the dispatch's own start and end
    hipExtLaunchKernelGGL(k_first<C>, dim3((unsigned)blocks), dim3(64 * FIRST_WAVES), 0, c.stream, c.ext_start,
                          c.ext_stop, 0u, a);
    c.ext_start = c.ext_stop = nullptr;
  } else {
    hipLaunchKernelGGL(k_first<C>, dim3((unsigned)blocks), dim3(64 * FIRST_WAVES), 0, c.stream, a);
  }
  return hipGetLastError();
}

template <int C, int KIND>
hipError_t run_conv(Ctx& c, const ConvArgs& a) {
  // one block per CU stages the weights once for its 16 waves
  auto go = [&](auto kern) {
    if (c.ext_start) {  // timed: the events are the dispatch's own start and end
      hipExtLaunchKernelGGL(kern, dim3(256), dim3(CONV_THREADS), 0, c.stream, c.ext_start, c.ext_stop, 0u, a);
      c.ext_start = c.ext_stop = nullptr;
    } else {
      hipLaunchKernelGGL(kern, dim3(256), dim3(CONV_THREADS), 0, c.stream, a);
    }
    return hipGetLastError();
  };
  return c.cap_pts > CONV_BUF_ROWS ? go(k_conv<C, KIND, true>) : go(k_conv<C, KIND, false>);
}

template <int C>
hipError_t run_layer(Ctx& c, bool last, bool two, const ConvArgs& a) {
  if (last) return two ? run_conv<C, CONV_HEAD2>(c, a) : run_conv<C, CONV_HEAD>(c, a);
  return a.xb ? run_conv<C, CONV_SCATTER>(c, a) : run_conv<C, CONV_MID>(c, a);
}

// Stage 2 of the two-stage head for one scale from the stored features of the
// last conv layer and a given S1 per voxel (decoder).  One wave per tile of
// 16 voxels, the same tile split and arithmetic as the fused path.
template <int C>
__global__ void __launch_bounds__(256) k_head2(int b, const int32_t* __restrict__ count,
                                               const int32_t* __restrict__ moff, int64_t cap_model,
                                               const float* __restrict__ hL, const uint8_t* __restrict__ s1,
                                               const uint8_t* __restrict__ code, const uint4* __restrict__ hw2,
                                               const float* __restrict__ hfac2, const float* __restrict__ hrat,
                                               const float* __restrict__ hb2,
                                               const float* __restrict__ emb, float* __restrict__ lse2,
                                               float* __restrict__ logits2, uint8_t* __restrict__ s1_out,
                                               uint32_t* err) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int64_t mo = moff[b];
  int64_t n = count[b];
  if (mo + n > cap_model) n = 0;  // overflow was latched where the size was made
  const int64_t ntiles = (n + 15) / 16;
  const int wpb = blockDim.x / 64;
  for (int64_t tile = (int64_t)blockIdx.x * wpb + (threadIdx.x >> 6); tile < ntiles;
       tile += (int64_t)gridDim.x * wpb) {
    const int64_t row = tile * 16 + r;
    const bool valid = row < n;
    const int64_t vr = valid ? row : n - 1;
    const int64_t prow = mo + vr;
    float x[C / 4], x2[C / 4];
    load_row<C>(hL + prow * C, g, x);
    int a1 = s1 ? s1[vr] : (code[vr] & 15);
    if (a1 > 15) {
      if (valid) latch(err, ERR_SYMBOL);
      a1 = 0;
    }
    add_row<C>(x, emb + a1 * C, g, x2);
    mul_row<C>(x2, hrat, g, x2);
    const f4 z2 = head16<C>(hw2, hfac2, hb2, x2, lane, g);
    const float l2 = lse16(z2);
    if (valid && g == 0) {
      lse2[prow] = l2;
      s1_out[prow] = (uint8_t)a1;
    }
    if (valid && logits2) *reinterpret_cast<f4*>(logits2 + row * 16 + 4 * g) = z2;
  }
}

}  // namespace

// 32-bit words of one 16-symbol block of the packed head (k_pack_head)
static int head_block_words(int C) { return (C >= 32 ? C / 32 : 1) * weight_planes(C) * 64 * 4; }

hipError_t launch_pack_weights(Ctx& c, const reno_weights& w) {
  ProfScope ps_(c, RENO_K_OTHER);
  const int C = c.p.channels;
  const bool top = c.top(), two = c.p.head_mode == RENO_HEAD_TWO_STAGE;
  const int L = top ? 4 : c.p.layers, kv = top ? c.kvol() : 27;
  auto conv_w = [&](int l) { return top ? w.top_w[l] : w.conv_w[l]; };
  // balance of every matrix's inputs
  for (int l = top ? 0 : 1; l < L; ++l)
    hipLaunchKernelGGL(k_balance, dim3(C), dim3(256), 0, c.stream, conv_w(l), kv, C, C, c.wbal(l));
  if (two) {
    hipLaunchKernelGGL(k_balance, dim3(C), dim3(256), 0, c.stream, w.head1_w, 1, C, 16, c.w_hbal);
    hipLaunchKernelGGL(k_balance, dim3(C), dim3(256), 0, c.stream, w.head2_w, 1, C, 16, c.w_hbal + 128);
  } else {
    hipLaunchKernelGGL(k_balance, dim3(C), dim3(256), 0, c.stream, w.head_w, 1, C, 256, c.w_hbal);
  }
  hipLaunchKernelGGL(k_feature_balance, dim3(1), dim3(128), 0, c.stream, C, c.w_hbal, two ? c.w_hbal + 128 : nullptr,
                     c.w_hrat, top ? c.wbal(2) : nullptr, c.w_xrat);
  // and of a layer's output (full predictor, conv A2: X_B, added to B2's output)
  auto obal = [&](int l) -> const float* { return l == L - 1 || (top && l == 1) ? c.w_hbal : c.wbal(l + 1); };
  auto rows = [&](const float* src, const float* bal, int n, float* dst) {
    hipLaunchKernelGGL(k_balance_rows, dim3((unsigned)(n * C + 255) / 256), dim3(256), 0, c.stream, src, bal, n, C, dst);
  };
  for (int l = 0; l < L; ++l) {
    const float* src = conv_w(l);
    if (!top && l == 0) {
      const dim3 grid(8 * 8 * 256 * C / 256);
      if (C == 32) hipLaunchKernelGGL(k_first_table<32>, grid, dim3(256), 0, c.stream, src, obal(0), c.w_conv[0]);
      else hipLaunchKernelGGL(k_first_table<16>, grid, dim3(256), 0, c.stream, src, obal(0), c.w_conv[0]);
    } else {
      uint16_t* out = reinterpret_cast<uint16_t*>(c.w_conv[l]);
      hipLaunchKernelGGL(k_weight_max, dim3(WMAX_BLOCKS), dim3(256), 0, c.stream, src, kv * C, C, c.wbal(l), c.w_part);
      const dim3 grid((unsigned)std::min<int64_t>(1024, ((int64_t)kv * C * C + 255) / 256));
      auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, c.stream, src, kv, c.w_part, c.wbal(l), obal(l), out, c.wfac(l));
      };
      switch (C) {
        case 128: go(k_pack_conv<128>); break;
        case 64: go(k_pack_conv<64>); break;
        case 32: go(k_pack_conv<32>); break;
        default: go(k_pack_conv<16>);
      }
    }
    rows(top ? w.top_b[l] : w.conv_b[l], obal(l), 1, c.w_bias[l]);
  }
  if (top) {
    rows(w.emb_o, c.w_hbal, 256, c.w_embo);
    rows(w.emb_d, c.w_hbal, 8, c.w_embd);
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(16), dim3(64), 0, c.stream, w.emb_o, c.wbal(0), c.w_embs, c.w_embr);
    };
    switch (C) {
      case 128: go(k_split_embed<128>); break;
      case 64: go(k_split_embed<64>); break;
      case 32: go(k_split_embed<32>); break;
      default: go(k_split_embed<16>);
    }
  }
  uint16_t* hw = reinterpret_cast<uint16_t*>(c.w_head);
  if (two) {
    // packed blocks [stage 1][stage 2], biases [b1 | b2], plain [C][H1 | H2]
    hipLaunchKernelGGL(k_head_max, dim3(1), dim3(64), 0, c.stream, w.head1_w, C, 16, c.w_hbal, c.w_part);
    hipLaunchKernelGGL(k_head_max, dim3(1), dim3(64), 0, c.stream, w.head2_w, C, 16, c.w_hbal + 128, c.w_part + 16);
    hipLaunchKernelGGL(k_pack_head, dim3(1), dim3(256), 0, c.stream, w.head1_w, C, 16, c.w_hbal, c.w_part, hw, c.w_hfac);
    hipLaunchKernelGGL(k_pack_head, dim3(1), dim3(256), 0, c.stream, w.head2_w, C, 16, c.w_hbal + 128, c.w_part + 16,
                       hw + head_block_words(C) * 2, c.w_hfac + 16);
    hipLaunchKernelGGL(k_copy_f32, dim3(1), dim3(64), 0, c.stream, w.head1_b, c.w_hbias, 16);
    hipLaunchKernelGGL(k_copy_f32, dim3(1), dim3(64), 0, c.stream, w.head2_b, c.w_hbias + 16, 16);
    hipLaunchKernelGGL(k_unbalance_head, dim3(2), dim3(256), 0, c.stream, w.head1_w, c.w_hbal, C, 16, 32, 0, c.w_head_plain);
    hipLaunchKernelGGL(k_unbalance_head, dim3(2), dim3(256), 0, c.stream, w.head2_w, c.w_hbal, C, 16, 32, 16, c.w_head_plain);
    rows(w.emb_s1, c.w_hbal, 16, c.w_emb);
    hipLaunchKernelGGL(k_transpose_head, dim3(2), dim3(256), 0, c.stream, w.head1_w, c.w_hbal, C, 16, 0, c.w_head_t);
    hipLaunchKernelGGL(k_transpose_head, dim3(2), dim3(256), 0, c.stream, w.head2_w, c.w_hbal, C, 16, 16, c.w_head_t);
  } else {
    hipLaunchKernelGGL(k_head_max, dim3(4), dim3(64), 0, c.stream, w.head_w, C, 256, c.w_hbal, c.w_part);
    hipLaunchKernelGGL(k_pack_head, dim3(16), dim3(256), 0, c.stream, w.head_w, C, 256, c.w_hbal, c.w_part, hw, c.w_hfac);
    hipLaunchKernelGGL(k_copy_f32, dim3(1), dim3(256), 0, c.stream, w.head_b, c.w_hbias, 256);
    hipLaunchKernelGGL(k_unbalance_head, dim3(32), dim3(256), 0, c.stream, w.head_w, c.w_hbal, C, 256, 256, 0, c.w_head_plain);
    hipLaunchKernelGGL(k_transpose_head, dim3(32), dim3(256), 0, c.stream, w.head_w, c.w_hbal, C, 256, 0, c.w_head_t);
  }
  return hipGetLastError();
}

// What every layer and head launch of a context is given.
static ConvArgs conv_args(const Ctx& c, bool second) {
  ConvArgs a{};
  a.b0 = c.b0();
  a.count = c.d_count;
  a.moff = c.d_moff;
  a.cap_pts = c.cap_pts;
  a.cap_model = c.cap_model;
  a.nbr = c.d_nbr;
  a.hb = c.w_hbias;
  a.hw = reinterpret_cast<const uint4*>(c.w_head);
  a.hfac = c.w_hfac;
  a.hrat = c.w_hrat;
  a.lse = c.d_lse;
  a.emb = c.w_emb;
  a.s1_code = second ? c.lv_code : nullptr;
  a.lse2 = c.d_lse2;
  a.s1_out = c.d_s1;
  a.b_ext = -1;
  a.cap_rows = c.cap_rows();
  if (c.top()) {  // the base scale's rows live past the zero row
    a.b_ext = c.b0();
    a.ext_off = c.cap_model + 1;
    a.emb_d = c.w_embd;
    a.emb_o = c.w_embo;
    a.code = c.lv_code;
    a.fc = c.lv_fc;
    a.xb_s = c.s_c;
    a.xb_r = c.r_c;
    a.xrat = c.w_xrat;
    a.r_out = c.r_b;
  }
  return a;
}

// Full predictor on the scales b_lo .. b_hi (Sec. 3.2, Eqs. 6-9), after its inputs:
//   neighbour maps of scales b_lo-1 .. b_hi, X_A = Emb_O[O^{d-1}] on scales
//   b_lo-1 .. b_hi-1 (split rows s_c)                             one prep launch
//   T = ReLU(conv_A1(X_A))                                        (split h_b)
//   F_A = ReLU(X_A + conv_A2(T)), scattered to the children as
//   X_B = F_A[parent] + Emb_D[delta] on scales b_lo .. b_hi       (h_d, split s_c, X_A being used up; F_A itself
//   is not stored)
//   T = ReLU(conv_B1(X_B))                                        (split h_b)
//   F_B = ReLU(X_B + conv_B2(T)), and the head                    (h_a)
// F_B of earlier calls is never overwritten (code lengths of a scale stay valid
// after the next scale's call).  layer(wi, last) launches a.
template <typename Layer>
hipError_t top_layers(Ctx& c, ConvArgs& a, int b_lo, int b_hi, Layer layer) {
  const int n_lo = b_lo - 1;  // stage A runs one scale below stage B
  hipError_t e = hipSuccess;
  auto conv = [&](int lo, int hi, int wi, const void* in, const float* r_in, float* out, float* s_out, const float* res,
                  float* xb) {
    if (e != hipSuccess) return;
    a.b_lo = lo;
    a.b_hi = hi;
    a.h_in = static_cast<const float*>(in);
    a.r_in = r_in;
    a.h_out = out;
    a.s_out = reinterpret_cast<uint32_t*>(s_out);
    a.res = res;
    a.xb = xb;
    a.w = c.w_conv[wi];
    a.wfac = c.wfac(wi);
    a.bias = c.w_bias[wi];
    e = layer(wi, wi == 3);
  };
  conv(n_lo, b_hi - 1, 0, c.s_c, c.r_c, nullptr, c.h_b, nullptr, nullptr);
  conv(n_lo, b_hi - 1, 1, c.h_b, c.r_b, nullptr, nullptr, nullptr, c.h_d);
  conv(b_lo, b_hi, 2, c.s_c, c.r_c, nullptr, c.h_b, nullptr, nullptr);
  conv(b_lo, b_hi, 3, c.h_b, c.r_b, c.h_a, nullptr, c.h_d, nullptr);
  return e;
}

hipError_t launch_top(Ctx& c, int b_lo, int b_hi, float* logits, bool second) {
  const int b0 = c.b0(), n_lo = b_lo - 1;
  ConvArgs a = conv_args(c, second);
  const RowMap rm{a.count, a.moff, a.cap_model, a.b_ext, a.ext_off, a.cap_rows};
  const bool c32 = c.p.channels == 32, two = c.p.head_mode == RENO_HEAD_TWO_STAGE;
  {
    ProfScope ps_(c, RENO_K_TOP_INPUT);
    const int blocks = (int)std::min<int64_t>(2048, (c.cap_rows() + 63) / 64);
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, c.stream, n_lo, b_hi - n_lo + 1, b_hi - n_lo, b0, rm,
                         c.lv_key, c.lv_code, (int64_t)c.cap_pts, cell_args(c), embed_tab(c), c.d_nbr, c.s_c, c.r_c);
    };
    if (c32) go(k_top_prep<32, false>);
    else go(k_top_prep<16, false>);
  }
  const hipError_t e = top_layers(c, a, b_lo, b_hi, [&](int, bool last) {  // the head fused with the last one
    a.logits = last ? logits : nullptr;
    ProfScope ps_(c, last ? RENO_K_CONV_LAST : RENO_K_CONV_MID);
    return c32 ? run_layer<32>(c, last, two, a) : run_layer<16>(c, last, two, a);
  });
  return e == hipSuccess ? hipGetLastError() : e;
}

// Full predictor with streamed weights (5x5x5 kernels or C above 32): the same
// layers on k_convw and a separate head launch.
template <int C, int KV>
hipError_t launch_top_wide(Ctx& c, int b_lo, int b_hi, float* logits, bool second) {
  const int b0 = c.b0(), n_lo = b_lo - 1;
  ConvArgs a = conv_args(c, second);
  const RowMap rm{a.count, a.moff, a.cap_model, a.b_ext, a.ext_off, a.cap_rows};
  {
    ProfScope ps_(c, RENO_K_TOP_INPUT);
    const int blocks = (int)std::min<int64_t>(2048, (c.cap_rows() + 63) / 64);
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, c.stream, n_lo, b_hi - n_lo + 1, b_hi - n_lo, b0, rm,
                         c.lv_key, c.lv_code, (int64_t)c.cap_pts, cell_args(c), embed_tab(c), c.d_nbr, c.s_c, c.r_c);
    };
    if constexpr (KV == 125) go(k_top_prep5<C>);
    else go(k_top_prep<C, true>);
  }
  {  // tiles of voxels with similar neighbourhoods: smaller offset unions per tile and group
    ProfScope pso_(c, RENO_K_OTHER);
    const int nsc = b_hi - n_lo + 1;
    const int64_t windows = (c.cap_model + c.cap_pts + TO_W - 1) / TO_W + nsc;
    hipLaunchKernelGGL(k_tile_order, dim3((unsigned)windows), dim3(TO_THREADS), 0, c.stream, n_lo, nsc, rm,
                       KV == 125 ? 5 : 3, c.d_nbr, c.d_perm, c.d_next);
    a.perm = c.d_perm;
  }
  hipError_t e = top_layers(c, a, b_lo, b_hi, [&](int wi, bool) {
    a.next = c.d_next + 8 * wi;
    ProfScope ps_(c, RENO_K_CONV_MID);
    if (a.xb)
      hipLaunchKernelGGL((k_convw<C, KV, true>), dim3(cw_blocks(C)), dim3(64 * cw_waves(C)), 0, c.stream, a);
    else
      hipLaunchKernelGGL((k_convw<C, KV, false>), dim3(cw_blocks(C)), dim3(64 * cw_waves(C)), 0, c.stream, a);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  {
    ProfScope ps_(c, RENO_K_CONV_LAST);
    a.h_in = c.h_a;
    a.logits = logits;
    e = run_headw<C>(c, c.p.head_mode == RENO_HEAD_TWO_STAGE, a);
  }
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

hipError_t launch_top_wide_any(Ctx& c, int b_lo, int b_hi, float* logits, bool second) {
  const bool k5 = c.ks() == 5;
  switch (c.p.channels) {
    case 16: return k5 ? launch_top_wide<16, 125>(c, b_lo, b_hi, logits, second)
                       : launch_top_wide<16, 27>(c, b_lo, b_hi, logits, second);
    case 32: return k5 ? launch_top_wide<32, 125>(c, b_lo, b_hi, logits, second)
                       : launch_top_wide<32, 27>(c, b_lo, b_hi, logits, second);
    case 64: return k5 ? launch_top_wide<64, 125>(c, b_lo, b_hi, logits, second)
                       : launch_top_wide<64, 27>(c, b_lo, b_hi, logits, second);
    default: return k5 ? launch_top_wide<128, 125>(c, b_lo, b_hi, logits, second)
                       : launch_top_wide<128, 27>(c, b_lo, b_hi, logits, second);
  }
}

hipError_t launch_model(Ctx& c, int b_lo, int b_hi, float* logits, bool second) {
  if (c.wide()) return launch_top_wide_any(c, b_lo, b_hi, logits, second);
  if (c.top()) return launch_top(c, b_lo, b_hi, logits, second);
  ConvArgs a = conv_args(c, second);
  a.b_lo = b_lo;
  a.b_hi = b_hi;
  const bool two = c.p.head_mode == RENO_HEAD_TWO_STAGE;
  const int L = c.p.layers;
  const RowMap rm{c.d_count, c.d_moff, (int64_t)c.cap_model, -1, 0, c.cap_rows()};
  const bool c32 = c.p.channels == 32;
  hipError_t e = hipSuccess;
  // features ping-pong between (h_a, r_a) and (h_b, r_b): split rows, and fp32
  // rows of the last layer; layer 0 writes h_a
  {
    ProfScope ps_(c, RENO_K_CONV_FIRST, true);
    FirstArgs f{b_lo, b_hi - b_lo + 1, rm, cell_args(c), c.lv_key, c.w_conv[0], c.w_bias[0], c.d_nbr,
                L == 1 ? c.h_a : nullptr, L == 1 ? nullptr : reinterpret_cast<uint32_t*>(c.h_a), c.r_a};
    e = c32 ? run_first<32>(c, f) : run_first<16>(c, f);
  }
  if (L == 1 && e == hipSuccess) {  // the head alone, on the first layer's rows
    ProfScope ps_(c, RENO_K_CONV_LAST, true);
    a.h_in = c.h_a;
    a.logits = logits;
    e = c32 ? run_headw<32>(c, two, a) : run_headw<16>(c, two, a);
  }
  for (int l = 1; l < L && e == hipSuccess; ++l) {
    const bool last = l == L - 1, odd = l & 1;
    float* out = odd ? c.h_b : c.h_a;
    a.h_in = odd ? c.h_a : c.h_b;
    a.r_in = odd ? c.r_a : c.r_b;
    a.h_out = last ? out : nullptr;
    a.s_out = last ? nullptr : reinterpret_cast<uint32_t*>(out);
    a.r_out = odd ? c.r_b : c.r_a;
    a.w = c.w_conv[l];
    a.wfac = c.wfac(l);
    a.bias = c.w_bias[l];
    a.logits = last ? logits : nullptr;
    ProfScope ps_(c, last ? RENO_K_CONV_LAST : RENO_K_CONV_MID, true);
    e = c32 ? run_layer<32>(c, last, two, a) : run_layer<16>(c, last, two, a);
  }
  return e;
}

hipError_t launch_head2(Ctx& c, int b, const uint8_t* s1, float* logits2) {
  ProfScope ps_(c, RENO_K_CONV_LAST);
  const uint4* hw2 = reinterpret_cast<const uint4*>(c.w_head + head_block_words(c.p.channels));
  const uint8_t* code = c.lv_code + c.lv(b);
  const int blocks = (int)std::min<int64_t>(1024, (c.cap_pts + 63) / 64);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, c.stream, b, c.d_count, c.d_moff, (int64_t)c.cap_model,
                       c.hlast(), s1, code, hw2, c.w_hfac + 16, c.w_hrat, c.w_hbias + 16, c.w_emb, c.d_lse2, logits2, c.d_s1,
                       c.d_err);
  };
  switch (c.p.channels) {
    case 128: go(k_head2<128>); break;
    case 64: go(k_head2<64>); break;
    case 32: go(k_head2<32>); break;
    default: go(k_head2<16>);
  }
  return hipGetLastError();
}

}  // namespace reno

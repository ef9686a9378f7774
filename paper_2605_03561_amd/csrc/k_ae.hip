// k_ae.hip -- learned pre-screen: autoencoder training and scoring kernels.
//
// Dense layers run on the matrix cores (v_mfma_f32_16x16x16_bf16): operands
// are bfloat16 (round to nearest even), accumulation is FP32.  A workgroup
// (8 waves) processes row tiles of 16 profile rows; every wave owns a fixed set
// of 16x16 output tiles per layer, so weight-gradient tiles stay in the MFMA
// accumulators across all row tiles of a training step and are written once
// per workgroup.  Partials are summed in workgroup order by the Adam kernel, so
// a step is deterministic.
#include "ta_ae.h"
#include "ta_device.h"
#include "ta_internal.h"
#include "ta_select.h"

namespace ta {
namespace {

constexpr int TR = 16;        // rows per tile

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ inline uint16_t f2bf(float f) {
  const uint32_t u = __float_as_uint(f);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// Sum of a value over the four lane groups that hold the same column.
__device__ inline float col_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}

// SplitMix64 finaliser (Steele, Lea & Flood 2014), used as a counter-based
// generator: draw = mix64(key + counter * golden gamma).
__device__ inline uint64_t mix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Standard normal draw for (key, row, feature): two 24-bit uniforms from
// SplitMix64 counter draws, then Box-Muller (Box & Muller 1958),
// sqrt(-2 ln u1) cos(2 pi u2), with u1 in (0, 1).
__device__ inline float gauss_draw(uint64_t key, uint64_t row, int c) {
  const uint64_t base = mix64(key ^ mix64(row * (uint64_t)AE_IN + (uint64_t)c));
  const uint64_t z1 = mix64(base), z2 = mix64(base ^ 0xD1B54A32D192ED03ull);
  const float u1 = ((float)(z1 >> 40) + 0.5f) * (1.0f / 16777216.0f);
  const float u2 = (float)(z2 >> 40) * (1.0f / 16777216.0f);
  return sqrtf(-2.0f * logf(u1)) * cosf(6.2831853071795864f * u2);
}

// (a * k + c) % n for a, c, k < n <= 2^31 (n_inv = 1.0 / n): the FP64 quotient
// is off by at most one.
__device__ inline int64_t perm_row(int64_t k, int64_t a, int64_t c, int64_t n, double n_inv) {
  const int64_t x = a * k + c;
  int64_t r = x - (int64_t)((double)x * n_inv) * n;
  r += r < 0 ? n : 0;
  return r - (r >= n ? n : 0);
}

// ---------------------------------------------------------------------------
// Training step: gradient partials of the mean squared error over the rows
// perm(k), k in [k0, k_end), written per workgroup to part[wg][AE_PS].
// With noise_sd > 0 the network sees x + noise_sd * N(0, 1) (drawn for the
// row's index and the feature under noise_key) and is scored against x
// (denoising training).
//
// Bound by the chain of seven dependent products of one 16-row tile per
// workgroup (4,096 rows: one tile per CU), so by latencies.  Eight waves; wave w
// owns columns 16w..16w+15 of the 128-wide layers (waves 0-1 those of the
// 32-wide one, 0-3 the outputs) and keeps its weight operands in registers,
// read from global memory once, while the rows and the noise come in.  With q =
// lane >> 4 and x = lane & 15 an operand of the 16x16x16 product is entries
// (x, k = 4q..4q+3), and a product yields rows 4q..4q+3 of column x.  So
// each tile is computed with its operands in both orders (the same products in
// the same order: the same bits): rows-in-lanes ("T": row x, columns 4q..4q+3)
// is the next product's operand, columns-in-lanes ("N": column x, rows 4q..4q+3)
// is the operand of the weight gradients, which contract over rows.  Neither is
// transposed: 8-byte LDS words by lane, without conflicts.  With the weights
// staged in LDS, four waves and operands gathered by 2-byte reads 25 us at 4,096
// rows, now 17, of which the stores of the partials (25.5 MB, past the caches: 2 us
// less than through them) are about 7 and the weights about 3.
// ---------------------------------------------------------------------------
constexpr int AT = 512;  // threads per workgroup

// The partials of the weights stand as the waves hold them, 16x16 tiles of 64
// lanes x 4 entries: a store instruction writes 1 KB in order.  (At the weights'
// own places it wrote sixteen pieces of 64 bytes: 18.4 us
// per step of 4,096 rows, now 17.)
constexpr int PT_W1 = 0, PT_W4 = 32, PT_W2 = 64, PT_W3 = 80;  // first tiles
static_assert((PT_W3 + 16) * 256 == AE_NW, "the tiles cover the weights");

// The parameter whose partials are at entry e of a workgroup's.
__device__ inline int tiled_param(int e) {
  if (e >= AE_NW) return e;
  const int t = e >> 8, lane = (e >> 2) & 63, x = lane & 15, k = 4 * (lane >> 4) + (e & 3);
  if (t < PT_W4) return AE_W1 + (16 * (t >> 2) + x) * AE_IN + 16 * (t & 3) + k;
  if (t < PT_W2) return AE_W4 + (16 * (t & 3) + x) * AE_H3 + 16 * ((t - PT_W4) >> 2) + k;
  if (t < PT_W3) return AE_W2 + (16 * (t & 1) + x) * AE_H1 + 16 * ((t - PT_W2) >> 1) + k;
  return AE_W3 + (16 * ((t - PT_W3) >> 1) + x) * AE_H2 + 16 * (t & 1) + k;
}

__device__ __forceinline__ f4 mma(s4 a, s4 b, f4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ s4 ld4(const uint16_t *p) { return *reinterpret_cast<const s4 *>(p); }

__device__ __forceinline__ s4 relu_bf(f4 a, f4 b) {
  s4 r;
#pragma unroll
  for (int j = 0; j < 4; j++) r[j] = (short)f2bf(fmaxf(a[j] + b[j], 0.f));
  return r;
}
// The gradient where the ReLU was active.
__device__ __forceinline__ f4 masked(f4 a, s4 h) {
  f4 r;
#pragma unroll
  for (int j = 0; j < 4; j++) r[j] = h[j] > 0 ? a[j] : 0.f;
  return r;
}
__device__ __forceinline__ s4 to_bf(f4 a) {
  s4 r;
#pragma unroll
  for (int j = 0; j < 4; j++) r[j] = (short)f2bf(a[j]);
  return r;
}

__global__ __launch_bounds__(AT) void ae_fwdbwd(const float *__restrict__ rows, int64_t n,
                                                 int64_t k0, int64_t k_end, int64_t pa,
                                                 int64_t pc, double n_inv, float scale, float noise_sd,
                                                 uint64_t noise_key,
                                                 const uint16_t *__restrict__ wb,
                                                 const float *__restrict__ w, float *part) {
  constexpr int XS = AE_IN + 4;  // floats per staged row
  __shared__ __align__(16) float X[TR * XS];
  __shared__ s4 XT[4][64], XN[4][64], H1T[8][64], H2T[2][64], H2N[2][64], H3T[8][64];
  __shared__ s4 D4T[4][64], D4N[4][64], D3T[8][64], D2T[2][64], D2N[2][64];
  __shared__ double redd[AT];
  const int tid = threadIdx.x, wid = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int q4 = 4 * (lane >> 4), x = lane & 15;
  const int64_t tiles = (k_end - k0 + TR - 1) / TR;
  const int64_t t_lo = tiles * blockIdx.x / gridDim.x, t_hi = tiles * (blockIdx.x + 1) / gridDim.x;

  // the rows of the first tile; two floats per thread
  const int xr = tid >> 5, xc = (tid & 31) * 2;
  int32_t row = 0;
  float2 v = {0.f, 0.f};
  auto load_rows = [&](int64_t t) {
    const int64_t k = k0 + t * TR + xr;
    v = float2{0.f, 0.f};
    if (t < t_hi && k < k_end) {
      row = (int32_t)perm_row(k, pa, pc, n, n_inv);
      v = *reinterpret_cast<const float2 *>(rows + (int64_t)row * AE_IN + xc);
    }
  };
  load_rows(t_lo);

  // this wave's weights: operand entries (x, 4q..4q+3) of 16-wide pieces
  const int c0 = 16 * wid + x;
  const uint16_t *wt = wb + AE_NW - AE_W2;
  s4 W1[4], W2[8], W3[2], W4[8], T4[4], T3[8], T2[2];
#pragma unroll
  for (int i = 0; i < 4; i++) W1[i] = ld4(wb + AE_W1 + c0 * AE_IN + 16 * i + q4);
#pragma unroll
  for (int i = 0; i < 2; i++) W3[i] = ld4(wb + AE_W3 + c0 * AE_H2 + 16 * i + q4);
#pragma unroll
  for (int i = 0; i < 4; i++) T4[i] = ld4(wt + AE_W4 + c0 * AE_IN + 16 * i + q4);
#pragma unroll
  for (int i = 0; i < 2; i++) T2[i] = ld4(wt + AE_W2 + c0 * AE_H2 + 16 * i + q4);
  const f4 z0 = {0.f, 0.f, 0.f, 0.f};
  const float b1 = w[AE_B1 + c0], b3 = w[AE_B3 + c0];
  const f4 b1n = {b1, b1, b1, b1}, b3n = {b3, b3, b3, b3};
  const f4 b1t = *reinterpret_cast<const f4 *>(w + AE_B1 + 16 * wid + q4);
  const f4 b3t = *reinterpret_cast<const f4 *>(w + AE_B3 + 16 * wid + q4);
  float b2 = 0.f, b4 = 0.f;
  f4 b2t = z0, b4t = z0;
  if (wid < 2) {
#pragma unroll
    for (int i = 0; i < 8; i++) {
      W2[i] = ld4(wb + AE_W2 + c0 * AE_H1 + 16 * i + q4);
      T3[i] = ld4(wt + AE_W3 + c0 * AE_H3 + 16 * i + q4);
    }
    b2 = w[AE_B2 + c0];
    b2t = *reinterpret_cast<const f4 *>(w + AE_B2 + 16 * wid + q4);
  }
  if (wid < 4) {
#pragma unroll
    for (int i = 0; i < 8; i++) W4[i] = ld4(wb + AE_W4 + c0 * AE_H3 + 16 * i + q4);
    b4 = w[AE_B4 + c0];
    b4t = *reinterpret_cast<const f4 *>(w + AE_B4 + 16 * wid + q4);
  }

  f4 gW1[4], gW4[4], gW2[2], gW3[2];
#pragma unroll
  for (int i = 0; i < 4; i++) gW1[i] = gW4[i] = z0;
#pragma unroll
  for (int i = 0; i < 2; i++) gW2[i] = gW3[i] = z0;
  float gb1 = 0.f, gb2 = 0.f, gb3 = 0.f, gb4 = 0.f, loss = 0.f;

  for (int64_t t = t_lo; t < t_hi; t++) {
    {
      float2 in = v;
      if (noise_sd > 0.f && k0 + t * TR + xr < k_end) {
        in.x += noise_sd * gauss_draw(noise_key, (uint64_t)row, xc);
        in.y += noise_sd * gauss_draw(noise_key, (uint64_t)row, xc + 1);
      }
      const uint16_t i0 = f2bf(in.x), i1 = f2bf(in.y);
      *reinterpret_cast<float2 *>(&X[xr * XS + xc]) = v;
      const int ft = xc >> 4, f = xc & 15;
      uint16_t *xt = reinterpret_cast<uint16_t *>(&XT[ft][(f >> 2) * 16 + xr]) + (f & 3);
      *reinterpret_cast<uint32_t *>(xt) = (uint32_t)i0 | (uint32_t)i1 << 16;
      uint16_t *xn = reinterpret_cast<uint16_t *>(&XN[ft][(xr >> 2) * 16 + f]) + (xr & 3);
      xn[0] = i0;
      xn[4] = i1;
    }
    __syncthreads();
    f4 an = z0, at = z0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const s4 xi = XT[i][lane];
      an = mma(xi, W1[i], an);
      at = mma(W1[i], xi, at);
    }
    const s4 h1n = relu_bf(an, b1n);
    H1T[wid][lane] = relu_bf(at, b1t);
    __syncthreads();
    s4 h2n, h2t;
    if (wid < 2) {
      an = at = z0;
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const s4 hi = H1T[i][lane];
        an = mma(hi, W2[i], an);
        at = mma(W2[i], hi, at);
      }
      const f4 b2n = {b2, b2, b2, b2};
      H2N[wid][lane] = h2n = relu_bf(an, b2n);
      H2T[wid][lane] = h2t = relu_bf(at, b2t);
    }
    __syncthreads();
    an = at = z0;
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const s4 hi = H2T[i][lane];
      an = mma(hi, W3[i], an);
      at = mma(W3[i], hi, at);
    }
    const s4 h3n = relu_bf(an, b3n), h3t = relu_bf(at, b3t);
    H3T[wid][lane] = h3t;
    __syncthreads();
    if (wid < 4) {  // outputs -> dL/dy, loss, db4
      an = at = z0;
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const s4 hi = H3T[i][lane];
        an = mma(hi, W4[i], an);
        at = mma(W4[i], hi, at);
      }
      const f4 xt = *reinterpret_cast<const f4 *>(&X[x * XS + 16 * wid + q4]);
      const int64_t left = k_end - (k0 + t * TR);  // rows of this tile
      f4 dn, dt;
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const float e = an[j] + b4 - X[(q4 + j) * XS + c0];
        const bool ok = q4 + j < left;
        if (ok) loss += e * e;
        dn[j] = ok ? scale * e : 0.f;
        gb4 += dn[j];
        dt[j] = x < left ? scale * (at[j] + b4t[j] - xt[j]) : 0.f;
      }
      D4N[wid][lane] = to_bf(dn);
      D4T[wid][lane] = to_bf(dt);
    }
    load_rows(t + 1);
    __syncthreads();
    // dW4 += D4^T H3; dH3 = D4 W4
    an = at = z0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const s4 di = D4T[i][lane];
      an = mma(di, T4[i], an);
      at = mma(T4[i], di, at);
      gW4[i] = mma(h3n, D4N[i][lane], gW4[i]);
    }
    an = masked(an, h3n);
#pragma unroll
    for (int j = 0; j < 4; j++) gb3 += an[j];
    const s4 d3n = to_bf(an);
    D3T[wid][lane] = to_bf(masked(at, h3t));
    __syncthreads();
    // dW3 += D3^T H2; dH2 = D3 W3
    if (wid < 2) {
      an = at = z0;
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const s4 di = D3T[i][lane];
        an = mma(di, T3[i], an);
        at = mma(T3[i], di, at);
      }
      an = masked(an, h2n);
#pragma unroll
      for (int j = 0; j < 4; j++) gb2 += an[j];
      D2N[wid][lane] = to_bf(an);
      D2T[wid][lane] = to_bf(masked(at, h2t));
    }
#pragma unroll
    for (int i = 0; i < 2; i++) gW3[i] = mma(H2N[i][lane], d3n, gW3[i]);
    __syncthreads();
    // dW2 += D2^T H1; dH1 = D2 W2; dW1 += D1^T X
    an = z0;
#pragma unroll
    for (int i = 0; i < 2; i++) {
      an = mma(D2T[i][lane], T2[i], an);
      gW2[i] = mma(h1n, D2N[i][lane], gW2[i]);
    }
    an = masked(an, h1n);
#pragma unroll
    for (int j = 0; j < 4; j++) gb1 += an[j];
    const s4 d1n = to_bf(an);
#pragma unroll
    for (int i = 0; i < 4; i++) gW1[i] = mma(XN[i][lane], d1n, gW1[i]);
    __syncthreads();
  }

  // Write this workgroup's partials (every element exactly once).
  float *P = part + (int64_t)blockIdx.x * AE_PS;
  auto put = [&](int tile, f4 g) {
    __builtin_nontemporal_store(g, reinterpret_cast<f4 *>(P + tile * 256 + lane * 4));
  };
#pragma unroll
  for (int i = 0; i < 4; i++) {
    put(PT_W1 + 4 * wid + i, gW1[i]);
    put(PT_W4 + 4 * wid + i, gW4[i]);
  }
#pragma unroll
  for (int i = 0; i < 2; i++) {
    put(PT_W2 + 2 * wid + i, gW2[i]);
    put(PT_W3 + 2 * wid + i, gW3[i]);
  }
  gb1 = col_sum(gb1);
  gb2 = col_sum(gb2);
  gb3 = col_sum(gb3);
  gb4 = col_sum(gb4);
  if (lane < 16) {
    P[AE_B1 + c0] = gb1;
    P[AE_B3 + c0] = gb3;
    if (wid < 4) P[AE_B4 + c0] = gb4;
    if (wid < 2) P[AE_B2 + c0] = gb2;
  }
  const double ls = block_sum_f64<AT>((double)loss, redd);
  if (tid == 0) P[AE_NP] = (float)ls;
}

// ---------------------------------------------------------------------------
// FP32 debug gradient: the same network, loss and input noise with every
// operation in FP32 (no bfloat16 operand rounding), for checking the gradient
// code against an FP64 reference.  A workgroup takes rows blockIdx.x,
// blockIdx.x + gridDim.x, ...; each layer's outputs are dot products in
// ascending k by single threads; thread t owns the partial entries p = t mod
// 256 (so the read-modify-writes of a row need no atomics).  Not a fast path.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void ae_grad_f32_kernel(const float *__restrict__ rows, int64_t n,
                                                          float scale, float noise_sd,
                                                          uint64_t noise_key,
                                                          const float *__restrict__ w, float *part) {
  __shared__ float x[AE_IN], xin[AE_IN], h1[AE_H1], h2[AE_H2], h3[AE_H3];
  __shared__ float d4[AE_IN], d3[AE_H3], d2[AE_H2], d1[AE_H1];
  __shared__ double red[256];
  const int t = threadIdx.x;
  float *P = part + (int64_t)blockIdx.x * AE_PS;
  for (int p = t; p < AE_NP; p += 256) P[p] = 0.f;
  double loss = 0.0;
  for (int64_t r = blockIdx.x; r < n; r += gridDim.x) {
    if (t < AE_IN) {
      x[t] = rows[r * AE_IN + t];
      xin[t] = noise_sd > 0.f ? x[t] + noise_sd * gauss_draw(noise_key, (uint64_t)r, t) : x[t];
    }
    __syncthreads();
    if (t < AE_H1) {
      float a = w[AE_B1 + t];
      for (int k = 0; k < AE_IN; k++) a = fmaf(w[AE_W1 + t * AE_IN + k], xin[k], a);
      h1[t] = a > 0.f ? a : 0.f;
    }
    __syncthreads();
    if (t < AE_H2) {
      float a = w[AE_B2 + t];
      for (int k = 0; k < AE_H1; k++) a = fmaf(w[AE_W2 + t * AE_H1 + k], h1[k], a);
      h2[t] = a > 0.f ? a : 0.f;
    }
    __syncthreads();
    if (t < AE_H3) {
      float a = w[AE_B3 + t];
      for (int k = 0; k < AE_H2; k++) a = fmaf(w[AE_W3 + t * AE_H2 + k], h2[k], a);
      h3[t] = a > 0.f ? a : 0.f;
    }
    __syncthreads();
    if (t < AE_IN) {
      float a = w[AE_B4 + t];
      for (int k = 0; k < AE_H3; k++) a = fmaf(w[AE_W4 + t * AE_H3 + k], h3[k], a);
      const float e = a - x[t];
      loss += (double)e * e;
      d4[t] = scale * e;
    }
    __syncthreads();
    if (t < AE_H3) {
      float a = 0.f;
      for (int o = 0; o < AE_IN; o++) a = fmaf(w[AE_W4 + o * AE_H3 + t], d4[o], a);
      d3[t] = h3[t] > 0.f ? a : 0.f;
    }
    __syncthreads();
    if (t < AE_H2) {
      float a = 0.f;
      for (int o = 0; o < AE_H3; o++) a = fmaf(w[AE_W3 + o * AE_H2 + t], d3[o], a);
      d2[t] = h2[t] > 0.f ? a : 0.f;
    }
    __syncthreads();
    if (t < AE_H1) {
      float a = 0.f;
      for (int o = 0; o < AE_H2; o++) a = fmaf(w[AE_W2 + o * AE_H1 + t], d2[o], a);
      d1[t] = h1[t] > 0.f ? a : 0.f;
    }
    __syncthreads();
    for (int p = t; p < AE_NP; p += 256) {
      float g;
      if (p < AE_W2) g = d1[p / AE_IN] * xin[p % AE_IN];
      else if (p < AE_W3) g = d2[(p - AE_W2) / AE_H1] * h1[(p - AE_W2) % AE_H1];
      else if (p < AE_W4) g = d3[(p - AE_W3) / AE_H2] * h2[(p - AE_W3) % AE_H2];
      else if (p < AE_NW) g = d4[(p - AE_W4) / AE_H3] * h3[(p - AE_W4) % AE_H3];
      else if (p < AE_B2) g = d1[p - AE_B1];
      else if (p < AE_B3) g = d2[p - AE_B2];
      else if (p < AE_B4) g = d3[p - AE_B3];
      else g = d4[p - AE_B4];
      P[p] += g;
    }
    __syncthreads();
  }
  const double ls = block_sum_f64<256>(loss, red);
  if (t == 0) P[AE_NP] = (float)ls;
}

// Sums the workgroup partials of every parameter (and of the loss) in workgroup
// order; optionally takes one Adam step.  With epoch_loss, also epoch_loss[0] +=
// loss * lfrac (the step's share of the epoch's rows), in the kernel rather than
// a launch of its own.
//
// Bound by reading the partials (256 of them: 25.5 MB).  A workgroup takes AP
// entries and brings their partials to LDS, 16 loads per thread in flight; one
// thread per entry then adds them in order.  With a thread per entry reading
// its own partials only 98 workgroups were in flight, 16 loads a turn each: 23
// us, now 8.
constexpr int AP = 32;          // entries per workgroup
constexpr int ADT = 512;        // threads
constexpr int ADU = 16;         // loads per thread and turn
constexpr int ADK = ADT / AP * ADU;  // partials per turn

template <bool TILED>  // partials in tiles, as ae_fwdbwd writes them, or by parameter
__global__ __launch_bounds__(ADT) void ae_adam(const float *__restrict__ part, int nwg, float *w, uint16_t *wb,
                                               float *m, float *v, float lr, float bc1, float bc2,
                                               int update, float *grad_out, float *loss_out,
                                               float loss_scale, float *epoch_loss, float lfrac) {
  __shared__ float pl[ADK][AP];
  const int e = (int)threadIdx.x % AP, k1 = (int)threadIdx.x / AP;
  const int at = blockIdx.x * AP + e, p = TILED ? tiled_param(at) : at;
  const bool mine = at <= AE_NP, sums = mine && threadIdx.x < AP;
  float w0 = 0.f, m0 = 0.f, v0 = 0.f;
  if (sums && update && p < AE_NP) {
    w0 = w[p];
    m0 = m[p];
    v0 = v[p];
  }
  float g = 0.f;
  for (int kb = 0; kb < nwg; kb += ADK) {
    float x[ADU];
#pragma unroll
    for (int u = 0; u < ADU; u++) {
      const int k = kb + u * (ADT / AP) + k1;
      x[u] = mine && k < nwg ? __builtin_nontemporal_load(&part[(int64_t)k * AE_PS + at]) : 0.f;
    }
    if (kb) __syncthreads();
#pragma unroll
    for (int u = 0; u < ADU; u++) pl[u * (ADT / AP) + k1][e] = x[u];
    __syncthreads();
    if (sums) {
      const int nk = nwg - kb < ADK ? nwg - kb : ADK;
#pragma unroll 16
      for (int k = 0; k < nk; k++) g += pl[k][e];
    }
  }
  if (!sums) return;
  if (p == AE_NP) {
    if (loss_out) {
      const float l = g * loss_scale;
      loss_out[0] = l;
      if (epoch_loss) epoch_loss[0] += l * lfrac;
    }
    return;
  }
  if (grad_out) grad_out[p] = g;
  if (update) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float mm = b1 * m0 + (1.f - b1) * g;
    const float vv = b2 * v0 + (1.f - b2) * g * g;
    m[p] = mm;
    v[p] = vv;
    const float wn = w0 - lr * (mm / bc1) / (sqrtf(vv / bc2) + eps);
    w[p] = wn;
    if (p < AE_NW) {
      const uint16_t b = f2bf(wn);
      wb[p] = b;
      if (p >= AE_W2) wb[ae_transposed(p)] = b;
    }
  }
}

// ---------------------------------------------------------------------------
// Initialisation: Xavier-uniform weights from SplitMix64 counter draws.
// ---------------------------------------------------------------------------

__global__ void ae_init_kernel(uint64_t seed, float *w, uint16_t *wb, float *m, float *v) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= AE_NP) return;
  float val = 0.f;
  if (p < AE_NW) {
    int l, base, fin, fout;
    if (p < AE_W2) { l = 0; base = AE_W1; fin = AE_IN; fout = AE_H1; }
    else if (p < AE_W3) { l = 1; base = AE_W2; fin = AE_H1; fout = AE_H2; }
    else if (p < AE_W4) { l = 2; base = AE_W3; fin = AE_H2; fout = AE_H3; }
    else { l = 3; base = AE_W4; fin = AE_H3; fout = AE_IN; }
    const uint64_t s = mix64(seed);
    const uint64_t key = s ^ mix64((uint64_t)(l + 1));
    const uint64_t idx = (uint64_t)(p - base);
    const uint64_t z = mix64(key + idx * 0x9E3779B97F4A7C15ull);
    const double u = ((double)(z >> 11) + 0.5) / 9007199254740992.0;
    const double a = sqrt(6.0 / (double)(fin + fout));
    val = (float)((2.0 * u - 1.0) * a);
    wb[p] = f2bf(val);
    if (p >= AE_W2) wb[ae_transposed(p)] = wb[p];
  }
  w[p] = val;
  m[p] = 0.f;
  v[p] = 0.f;
}

// ---------------------------------------------------------------------------
// Normalisation fit: exact per-region sums over the valid cells.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void ae_norm_partial(const int64_t *__restrict__ T, int64_t R,
                                                       int I, const int32_t *it, int64_t rpb,
                                                       int64_t *ps, uint64_t *pq, int64_t *pc) {
  const int g = threadIdx.x & 63, rs = threadIdx.x >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * rpb, r1 = r0 + rpb < R ? r0 + rpb : R;
  int64_t s = 0, cnt = 0;
  u128 q = 0;
  for (int64_t r = r0 + rs; r < r1; r += 4) {
    int ni = it ? it[r] : I;
    if (ni > I) ni = I;
    if (ni < 0) ni = 0;
    const int64_t *row = T + r * (int64_t)I * AE_IN + g;
    for (int i = 0; i < ni; i++) {
      const int64_t x = row[(int64_t)i * AE_IN];
      s += x;
      q += (u128)((i128)x * x);
    }
    cnt += ni;
  }
  __shared__ int64_t ss[256], sc[256];
  __shared__ uint64_t sl[256], sh[256];
  ss[threadIdx.x] = s;
  sc[threadIdx.x] = cnt;
  sl[threadIdx.x] = (uint64_t)q;
  sh[threadIdx.x] = (uint64_t)(q >> 64);
  __syncthreads();
  if (threadIdx.x < 64) {
    int64_t a = 0, c = 0;
    u128 b = 0;
    for (int k = 0; k < 4; k++) {
      const int t = k * 64 + threadIdx.x;
      a += ss[t];
      c += sc[t];
      b += ((u128)sh[t] << 64) | sl[t];
    }
    ps[(int64_t)blockIdx.x * 64 + g] = a;
    pq[((int64_t)blockIdx.x * 64 + g) * 2] = (uint64_t)b;
    pq[((int64_t)blockIdx.x * 64 + g) * 2 + 1] = (uint64_t)(b >> 64);
    if (g == 0) pc[blockIdx.x] = c;
  }
}

__global__ void ae_norm_final(int nb, const int64_t *ps, const uint64_t *pq, const int64_t *pc,
                              int reset, int64_t *nsum, uint64_t *nsq, int64_t *ncnt, float *mu,
                              float *isd) {
  const int g = threadIdx.x;
  if (g >= 64) return;
  int64_t s = reset ? 0 : nsum[g];
  u128 q = reset ? 0 : (((u128)nsq[2 * g + 1] << 64) | nsq[2 * g]);
  int64_t n = reset ? 0 : ncnt[0];
  int64_t add = 0;
  for (int b = 0; b < nb; b++) {
    s += ps[(int64_t)b * 64 + g];
    q += ((u128)pq[((int64_t)b * 64 + g) * 2 + 1] << 64) | pq[((int64_t)b * 64 + g) * 2];
    add += pc[b];
  }
  n += add;
  nsum[g] = s;
  nsq[2 * g] = (uint64_t)q;
  nsq[2 * g + 1] = (uint64_t)(q >> 64);
  if (g == 0) ncnt[0] = n;
  double m = 0.0, sd = 1.0;
  if (n > 0) {
    m = i64_to_f64(s) / (double)n;
    const i128 num = (i128)((u128)n * q) - (i128)s * s;
    sd = sqrt(i128_to_f64(num) / ((double)n * (double)n));
    if (!(sd > 0.0)) sd = 1.0;
  }
  const float sd32 = (float)sd;
  mu[g] = (float)m;
  isd[g] = 1.0f / sd32;
}

// ---------------------------------------------------------------------------
// Training rows: normalised profile rows of every valid (rank, iteration).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void ae_rows_scan(const int32_t *it, int64_t R, int I,
                                                     int64_t *off) {
  __shared__ int64_t buf[1024];
  const int t = threadIdx.x;
  const int64_t per = (R + 1023) / 1024;
  const int64_t a = t * per, b = a + per < R ? a + per : R;
  int64_t s = 0;
  for (int64_t r = a; r < b; r++) {
    int ni = it ? it[r] : I;
    s += ni > I ? I : (ni < 0 ? 0 : ni);
  }
  buf[t] = s;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {  // inclusive Hillis-Steele scan
    const int64_t x = t >= d ? buf[t - d] : 0;
    __syncthreads();
    buf[t] += x;
    __syncthreads();
  }
  int64_t run = buf[t] - s;
  for (int64_t r = a; r < b; r++) {
    off[r] = run;
    int ni = it ? it[r] : I;
    run += ni > I ? I : (ni < 0 ? 0 : ni);
  }
  if (t == 1023) off[R] = buf[1023];
}

__global__ __launch_bounds__(256) void ae_rows_fill(const int64_t *__restrict__ T, int64_t R, int I,
                                                    const int64_t *off, const float *mu,
                                                    const float *isd, float *rows) {
  const int64_t r = blockIdx.x;
  const int64_t o = off[r], n = off[r + 1] - o;
  const int g = threadIdx.x & 63;
  const float m = mu[g], s = isd[g];
  const int64_t *src = T + r * (int64_t)I * AE_IN;
  for (int64_t k = threadIdx.x; k < n * AE_IN; k += 256)
    rows[(o + k / AE_IN) * AE_IN + (k % AE_IN)] = ((float)src[k] - m) * s;
}

// ---------------------------------------------------------------------------
// Scoring.  One wave per rank (8 waves per workgroup share the weights in
// LDS).  The rank's profile rows go through the network 32 at a time, as two
// 16-row tiles of v_mfma_f32_16x16x32_bf16: every weight fragment read from
// LDS feeds both tiles.  The FP32 input tile goes through LDS (the inputs the
// residual needs are held in registers in the output layout), and the next 32
// rows are loaded from HBM into registers while the current ones are in the
// network.  No workgroup barrier after the weights are staged.  The weights are
// the product's left operand: a lane then holds four consecutive features of
// one row, two packed conversions (with the rows on the left, four conversions
// by hand of six instructions and four 2-byte LDS writes bound the kernel), and
// row swaps turn them into the next layer's operand, so the hidden layers stay
// in registers.  10,000 ranks x 300 rows (1.54 GB): 394 us with the rows on the
// left, 327 us with the hidden layers through LDS, 306 with them in registers,
// 299 with the weights staged by 16-byte loads and a rank's length read during
// the rank before.
//   kind 0: score = max_g mean_i (y - x)^2     kind 1: max_g |mean_i (y - x)|
// ---------------------------------------------------------------------------
constexpr int SW = 8;                  // waves per workgroup
constexpr int SR = 32;                 // rows per wave step (two MFMA tiles)
constexpr int P_W1 = 72, P_W2 = 136, P_W3 = 40, P_W4 = 136;   // padded row strides (bf16)
constexpr int P_X = 68;                // FP32 row stride of the input tile

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

struct ScoreLds {
  uint16_t W1[AE_H1 * P_W1], W2[AE_H2 * P_W2], W3[AE_H3 * P_W3], W4[AE_IN * P_W4];
  float b[AE_NP - AE_NW];
  float mu[AE_IN], isd[AE_IN];
  float X[SW][SR * P_X];  // a wave's normalised inputs (FP32)
};

__device__ inline bf8 ld_bf8(const uint16_t *p) {
  return __builtin_bit_cast(bf8, *reinterpret_cast<const u4v *>(p));
}

// Two floats to bfloat16, to nearest even (one v_cvt_pk_bf16_f32).
__device__ inline uint32_t pack_bf2(float a, float b) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  const f2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf2));
}

__device__ inline bf8 ld_bf8_from_f32(const float *p) {
  const float4 a = *reinterpret_cast<const float4 *>(p);
  const float4 b = *reinterpret_cast<const float4 *>(p + 4);
  const u4v u = {pack_bf2(a.x, a.y), pack_bf2(a.z, a.w), pack_bf2(b.x, b.y), pack_bf2(b.z, b.w)};
  return __builtin_bit_cast(bf8, u);
}

// Orders this wave's LDS accesses: every earlier LDS read and write of the
// wave has completed before any later one is issued.
__device__ inline void lds_wave_sync() {
  __builtin_amdgcn_wave_barrier();
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

__device__ inline f4 mfma32(bf8 a, bf8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Four features of a hidden layer after bias and ReLU, as bfloat16.
__device__ inline void hidden(uint32_t *h, f4 acc, const float *bias) {
  const float4 b = *reinterpret_cast<const float4 *>(bias);
  h[0] = pack_bf2(fmaxf(acc[0] + b.x, 0.f), fmaxf(acc[1] + b.y, 0.f));
  h[1] = pack_bf2(fmaxf(acc[2] + b.z, 0.f), fmaxf(acc[3] + b.w, 0.f));
}

// From the output layout of two feature tiles (h[0], h[1]: features 4 * g + 0..3
// of the first, h[2], h[3]: of the second, g = lane / 16) to the operand layout
// of the next product, features 8 * g + 0..7 of the 32: the lane groups are
// exchanged by two row swaps per register, with no LDS.
__device__ inline bf8 next_operand(const uint32_t *h) {
  u4v u;
#pragma unroll
  for (int j = 0; j < 2; j++) {
    const auto x = __builtin_amdgcn_permlane32_swap(h[j], h[j + 2], false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(x[0], x[1], false, false);
    u[j] = y[0];
    u[j + 2] = y[1];
  }
  return __builtin_bit_cast(bf8, u);
}

// Sums v[0..16) over the 16 lanes that share lane / 16; lane l is left with
// the sum of v[l mod 16].
template <int B, typename F>
__device__ inline void rows_sum_step(F (&v)[16]) {
  const bool up = (threadIdx.x & B) != 0;
#pragma unroll
  for (int k = 0; k < B; k++) {
    const F send = up ? v[k] : v[k + B];
    v[k] = (up ? v[k + B] : v[k]) + __shfl_xor(send, B, 64);
  }
}
template <typename F>
__device__ inline F rows_sum(F (&v)[16]) {
  rows_sum_step<8>(v);
  rows_sum_step<4>(v);
  rows_sum_step<2>(v);
  rows_sum_step<1>(v);
  return v[0];
}

// SQ: squared errors (kind 0), else residuals (kinds 1 and 2).
template <bool SQ>
__global__ __launch_bounds__(SW * 64) void ae_score_kernel(const int64_t *__restrict__ T, int64_t R,
                                                           int I, const int32_t *it,
                                                           const uint16_t *__restrict__ wb,
                                                           const float *__restrict__ w,
                                                           const float *mu, const float *isd,
                                                           int kind, float *score, float *v_t) {
  extern __shared__ __align__(16) unsigned char smem[];
  ScoreLds &L = *reinterpret_cast<ScoreLds *>(smem);
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  {  // the weights, eight of a row at a time, all loads in flight
    constexpr int PER = AE_NW / 8 / (SW * 64);
    static_assert(AE_NW % (8 * SW * 64) == 0 && (P_W1 | P_W2 | P_W3 | P_W4) % 8 == 0, "whole 16-byte words");
    uint4 v[PER];
#pragma unroll
    for (int u = 0; u < PER; u++) v[u] = reinterpret_cast<const uint4 *>(wb)[u * (SW * 64) + tid];
#pragma unroll
    for (int u = 0; u < PER; u++) {
      const int k = 8 * (u * (SW * 64) + tid);
      uint16_t *d;
      if (k < AE_W2) d = &L.W1[(k / AE_IN) * P_W1 + k % AE_IN];
      else if (k < AE_W3) d = &L.W2[((k - AE_W2) / AE_H1) * P_W2 + (k - AE_W2) % AE_H1];
      else if (k < AE_W4) d = &L.W3[((k - AE_W3) / AE_H2) * P_W3 + (k - AE_W3) % AE_H2];
      else d = &L.W4[((k - AE_W4) / AE_H3) * P_W4 + (k - AE_W4) % AE_H3];
      *reinterpret_cast<uint4 *>(d) = v[u];
    }
  }
  for (int k = tid; k < AE_NP - AE_NW; k += SW * 64) L.b[k] = w[AE_NW + k];
  for (int k = tid; k < AE_IN; k += SW * 64) {
    L.mu[k] = mu[k];
    L.isd[k] = isd[k];
  }
  __syncthreads();
  float *X = L.X[wid];
  // MFMA operand layout: A/B lane -> row lane & 15, k = 8 * (lane >> 4) + 0..7;
  // D lane -> rows 4 * (lane >> 4) + 0..3, column lane & 15.  A: 16 features of
  // the weights, B: 16 profile rows.
  const int row = lane & 15, kq = 8 * (lane >> 4), fq = 4 * (lane >> 4);
  // Loader: load h of a step reads rows 2h, 2h+1 (1 KB contiguous); lane ->
  // row 2h + lane / 32, columns lc, lc + 1.
  const int lh = lane >> 5, lc = 2 * (lane & 31);
  const float m0 = L.mu[lc], m1 = L.mu[lc + 1], s0 = L.isd[lc], s1 = L.isd[lc + 1];
  const float *bias = L.b;
  const int64_t nw = (int64_t)gridDim.x * SW;
  int n_next = 0;
  {
    const int64_t r = (int64_t)blockIdx.x * SW + wid;
    if (r < R) n_next = it ? it[r] : I;
  }
  for (int64_t r = (int64_t)blockIdx.x * SW + wid; r < R; r += nw) {
    int n = n_next;
    if (r + nw < R) n_next = it ? it[r + nw] : I;  // arrives during this rank
    if (n > I) n = I;
    if (n < 0) n = 0;
    const int64_t *src = T + r * (int64_t)I * AE_IN;
    // FP64 sums of the FP32 residuals: rows with equal residuals give exactly
    // equal means whatever the number of iterations (the robust z of kind 2
    // must see exact ties); squared errors are summed in FP32.  Entry
    // 4 * nt + j: feature 16 * nt + fq + j over this lane's rows.
    float e2[16];
    double rs[16];
#pragma unroll
    for (int k = 0; k < 16; k++) {
      e2[k] = 0.f;
      rs[k] = 0.0;
    }
    u4v buf[16];
    // Rows past the rank's last one are clamped to it (loaded, then ignored),
    // so every load is in bounds and unconditional.
    auto load = [&](int i0) {
#pragma unroll
      for (int h = 0; h < 16; h++) {
        int i = i0 + 2 * h + lh;
        i = i < n ? i : n - 1;
        buf[h] = __builtin_nontemporal_load(reinterpret_cast<const u4v *>(src + (int64_t)i * AE_IN + lc));
      }
    };
    if (n > 0) load(0);
    for (int i0 = 0; i0 < n; i0 += SR) {
      // int64 -> FP32 (correctly rounded): cells in [0, 2^32) take one
      // unsigned conversion; a lane holding any wider cell converts all 32 in full.
      float cv[32];
      uint32_t wide = 0;
#pragma unroll
      for (int h = 0; h < 16; h++) {
        wide |= buf[h][1] | buf[h][3];
        cv[2 * h] = (float)buf[h][0];
        cv[2 * h + 1] = (float)buf[h][2];
      }
      if (wide) {
#pragma unroll
        for (int h = 0; h < 16; h++) {
          cv[2 * h] = (float)(int64_t)(((uint64_t)buf[h][1] << 32) | buf[h][0]);
          cv[2 * h + 1] = (float)(int64_t)(((uint64_t)buf[h][3] << 32) | buf[h][2]);
        }
      }
#pragma unroll
      for (int h = 0; h < 16; h++) {  // normalised inputs of this step (rows past n are zero)
        const int i = 2 * h + lh;
        const bool ok = i0 + i < n;
        float2 x;
        x.x = ok ? (cv[2 * h] - m0) * s0 : 0.f;
        x.y = ok ? (cv[2 * h + 1] - m1) * s1 : 0.f;
        *reinterpret_cast<float2 *>(&X[i * P_X + lc]) = x;
      }
      if (i0 + SR < n) load(i0 + SR);  // next step's rows, in flight during the network
      lds_wave_sync();
      bf8 a1[2][2];
      float4 xr[2][4];
#pragma unroll
      for (int t = 0; t < 2; t++) {
#pragma unroll
        for (int k = 0; k < 2; k++) a1[t][k] = ld_bf8_from_f32(&X[(16 * t + row) * P_X + 32 * k + kq]);
#pragma unroll
        for (int nt = 0; nt < 4; nt++)
          xr[t][nt] = *reinterpret_cast<const float4 *>(&X[(16 * t + row) * P_X + 16 * nt + fq]);
      }
      lds_wave_sync();
      // L1: [32 x 64] -> [32 x 128]; h[t][2 * nt ..]: feature tile nt of row tile t
      uint32_t h[2][AE_H1 / 8];
#pragma unroll
      for (int nt = 0; nt < AE_H1 / 16; nt++) {
        const bf8 w0 = ld_bf8(&L.W1[(16 * nt + row) * P_W1 + kq]);
        const bf8 w1 = ld_bf8(&L.W1[(16 * nt + row) * P_W1 + 32 + kq]);
#pragma unroll
        for (int t = 0; t < 2; t++) {
          f4 acc = {0.f, 0.f, 0.f, 0.f};
          acc = mfma32(w0, a1[t][0], acc);
          acc = mfma32(w1, a1[t][1], acc);
          hidden(&h[t][2 * nt], acc, bias + 16 * nt + fq);
        }
      }
      // L2: [32 x 128] -> [32 x 32]
      uint32_t h2[2][AE_H2 / 8];
      {
        bf8 a2[2][4];
#pragma unroll
        for (int t = 0; t < 2; t++)
#pragma unroll
          for (int k = 0; k < 4; k++) a2[t][k] = next_operand(&h[t][4 * k]);
#pragma unroll
        for (int nt = 0; nt < AE_H2 / 16; nt++) {
          bf8 bw[4];
#pragma unroll
          for (int k = 0; k < 4; k++) bw[k] = ld_bf8(&L.W2[(16 * nt + row) * P_W2 + 32 * k + kq]);
#pragma unroll
          for (int t = 0; t < 2; t++) {
            f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 4; k++) acc = mfma32(bw[k], a2[t][k], acc);
            hidden(&h2[t][2 * nt], acc, bias + AE_B2 - AE_B1 + 16 * nt + fq);
          }
        }
      }
      // L3: [32 x 32] -> [32 x 128]
      {
        bf8 a3[2];
#pragma unroll
        for (int t = 0; t < 2; t++) a3[t] = next_operand(h2[t]);
#pragma unroll
        for (int nt = 0; nt < AE_H3 / 16; nt++) {
          const bf8 bw = ld_bf8(&L.W3[(16 * nt + row) * P_W3 + kq]);
#pragma unroll
          for (int t = 0; t < 2; t++) {
            f4 acc = {0.f, 0.f, 0.f, 0.f};
            acc = mfma32(bw, a3[t], acc);
            hidden(&h[t][2 * nt], acc, bias + AE_B3 - AE_B1 + 16 * nt + fq);
          }
        }
      }
      // L4: [32 x 128] -> [32 x 64], residuals of the valid rows
      {
        bf8 a4[2][4];
#pragma unroll
        for (int t = 0; t < 2; t++)
#pragma unroll
          for (int k = 0; k < 4; k++) a4[t][k] = next_operand(&h[t][4 * k]);
#pragma unroll
        for (int nt = 0; nt < AE_IN / 16; nt++) {
          bf8 bw[4];
#pragma unroll
          for (int k = 0; k < 4; k++) bw[k] = ld_bf8(&L.W4[(16 * nt + row) * P_W4 + 32 * k + kq]);
          const float4 bc = *reinterpret_cast<const float4 *>(bias + AE_B4 - AE_B1 + 16 * nt + fq);
          const float b4[4] = {bc.x, bc.y, bc.z, bc.w};
#pragma unroll
          for (int t = 0; t < 2; t++) {
            f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 4; k++) acc = mfma32(bw[k], a4[t][k], acc);
            const float x4[4] = {xr[t][nt].x, xr[t][nt].y, xr[t][nt].z, xr[t][nt].w};
            const bool ok = i0 + 16 * t + row < n;  // rows past n add 0
#pragma unroll
            for (int j = 0; j < 4; j++) {
              const float r0 = acc[j] + b4[j] - x4[j];
              const float res = ok ? r0 : 0.f;
              if (SQ) e2[4 * nt + j] += res * res;
              else rs[4 * nt + j] += (double)res;
            }
          }
        }
      }
    }
    // lane l is left with feature 16 * ((l mod 16) / 4) + fq + l mod 4
    float best = 0.f;
    if (SQ) {
      const float a = rows_sum(e2);
      best = n > 0 ? fmaxf(best, a / (float)n) : 0.f;
    } else {
      const double b = rows_sum(rs);
      if (kind == 2) v_t[(int64_t)(16 * (row >> 2) + fq + (row & 3)) * R + r] = n > 0 ? (float)(b / (double)n) : 0.f;
      else best = n > 0 ? fmaxf(best, (float)(fabs(b) / (double)n)) : 0.f;
    }
    for (int d = 32; d >= 1; d >>= 1) best = fmaxf(best, __shfl_xor(best, d, 64));
    if (kind != 2 && lane == 0) score[r] = best;
  }
}

// ---------------------------------------------------------------------------
// Second stage of score kind 2, in FP32: per region g over the ranks with
// iterations, med = median of m(., g), MAD = median of |m - med|, z = (m - med)
// / (1.4826 MAD); when MAD is 0, 1.253314 * mean |m - med| (summed in FP64)
// replaces 1.4826 MAD; when that is 0 too, z = 0.  Medians of an even count
// are (a + b) * 0.5.  Every step is one IEEE FP32 operation in this order.
// Exact selection: radix select with 11-bit digits on order-preserving keys.
// ---------------------------------------------------------------------------
constexpr int RS = 1024;            // threads per region workgroup
constexpr int RSW = RS / 64;
constexpr int RNB = 2048;           // bins of an 11-bit digit
constexpr int RBPT = RNB / RS;

__device__ inline uint32_t fkey(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float fdec(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

struct RegLds {
  uint32_t hist[RNB];
  int64_t wtot[RSW];
  uint32_t wmin[RSW];
  double wsum[RSW];
  uint32_t state[4];
};

__device__ inline bool region_active(const int32_t *it, int I, int64_t r) {
  return it ? it[r] > 0 : I > 0;
}

// k-th smallest of keyf(r) over active ranks (32-bit keys), and with
// want_next the (k+1)-th.
template <class KeyF>
__device__ void select32(int64_t R, const int32_t *it, int I, KeyF keyf, int64_t k, bool want_next,
                         RegLds &L, uint32_t &v1, uint32_t &v2) {
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  uint32_t pref = 0;
  v1 = v2 = 0;
  for (int hi = 32; hi > 0;) {
    const int w = hi >= 11 ? 11 : hi;
    const int lo = hi - w;
    const bool last = lo == 0;
    uint32_t mgt = 0xffffffffu;
    for (int64_t r = t; r < R; r += RS) {
      if (!region_active(it, I, r)) continue;
      const uint32_t key = keyf(r);
      const uint32_t top = hi >= 32 ? 0u : key >> hi;
      if (top == pref) atomicAdd(&L.hist[(key >> lo) & ((1u << w) - 1)], 1u);
      else if (last && top > pref && key < mgt) mgt = key;
    }
    for (int d = 32; d >= 1; d >>= 1) {
      const uint32_t o = __shfl_xor(mgt, d, 64);
      mgt = o < mgt ? o : mgt;
    }
    if (lane == 0) L.wmin[wid] = mgt;
    __syncthreads();
    uint32_t cnt[RBPT];
    int64_t own = 0;
#pragma unroll
    for (int j = 0; j < RBPT; j++) {
      cnt[j] = L.hist[t * RBPT + j];
      own += cnt[j];
    }
    int64_t incl = own;
    for (int d = 1; d < 64; d <<= 1) {
      const int64_t o = __shfl_up(incl, d, 64);
      if (lane >= d) incl += o;
    }
    if (lane == 63) L.wtot[wid] = incl;
    __syncthreads();
    int64_t excl = incl - own;
    for (int q = 0; q < wid; q++) excl += L.wtot[q];
    uint32_t mg = L.wmin[0];
    for (int q = 1; q < RSW; q++) mg = L.wmin[q] < mg ? L.wmin[q] : mg;
    __syncthreads();  // all histogram reads are done
    for (int j = t; j < RNB; j += RS) L.hist[j] = 0;
    if (excl <= k && k < excl + own) {
      int64_t cum = excl;
      int j = 0;
      for (; j < RBPT; j++) {
        if (cum + (int64_t)cnt[j] > k) break;
        cum += cnt[j];
      }
      L.state[0] = (pref << w) | (uint32_t)(t * RBPT + j);
      L.state[1] = (uint32_t)(k - cum);
      L.state[2] = (k - cum + 1 < (int64_t)cnt[j]) ? 1u : 0u;
      // next non-empty bin above the selected one (only meaningful on the last digit)
      uint32_t nb = 0xffffffffu;
      for (int jj = j + 1; jj < RBPT && nb == 0xffffffffu; jj++)
        if (cnt[jj]) nb = (uint32_t)(t * RBPT + jj);
      L.state[3] = nb;
    }
    __syncthreads();
    const uint32_t np = L.state[0];
    const int64_t kk = (int64_t)L.state[1];
    if (last && want_next && L.state[2] == 0 && L.state[3] == 0xffffffffu) {
      // the next non-empty bin lies in a later thread's range: scan the merged
      // counts again (read before the clear by the owners, kept in cnt)
      uint32_t nb = 0xffffffffu;
      const uint32_t bsel = np & ((1u << w) - 1);
#pragma unroll
      for (int j = RBPT - 1; j >= 0; j--)
        if ((uint32_t)(t * RBPT + j) > bsel && cnt[j]) nb = (uint32_t)(t * RBPT + j);
      for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t o = __shfl_xor(nb, d, 64);
        nb = o < nb ? o : nb;
      }
      if (lane == 0) L.wmin[wid] = nb;
      __syncthreads();
      nb = L.wmin[0];
      for (int q = 1; q < RSW; q++) nb = L.wmin[q] < nb ? L.wmin[q] : nb;
      __syncthreads();
      if (t == 0) L.state[3] = nb;
      __syncthreads();
    }
    if (last) {
      v1 = np;
      if (!want_next || L.state[2]) v2 = np;
      else if (L.state[3] != 0xffffffffu) v2 = (pref << w) | L.state[3];
      else v2 = mg;
    }
    __syncthreads();
    pref = np;
    k = kk;
    hi = lo;
  }
  if (!want_next) v2 = v1;
}

__global__ __launch_bounds__(RS) void region_robust_f32(const float *__restrict__ v_t, int64_t R,
                                                        const int32_t *it, int I, float *z_t) {
  __shared__ RegLds L;
  const int g = blockIdx.x, t = threadIdx.x, lane = t & 63, wid = t >> 6;
  const float *v = v_t + (int64_t)g * R;
  float *z = z_t + (int64_t)g * R;
  for (int j = t; j < RNB; j += RS) L.hist[j] = 0;
  int64_t nl = 0;
  for (int64_t r = t; r < R; r += RS) nl += region_active(it, I, r) ? 1 : 0;
  for (int d = 32; d >= 1; d >>= 1) nl += __shfl_xor(nl, d, 64);
  if (lane == 0) L.wtot[wid] = nl;
  __syncthreads();
  int64_t n = 0;
  for (int q = 0; q < RSW; q++) n += L.wtot[q];
  __syncthreads();
  float med = 0.f, scale = 0.f;
  if (n > 0) {
    const int64_t k = (n - 1) / 2;
    const bool even = (n & 1) == 0;
    uint32_t a, b;
    select32(R, it, I, [&](int64_t r) { return fkey(v[r]); }, k, even, L, a, b);
    med = even ? (fdec(a) + fdec(b)) * 0.5f : fdec(a);
    // |m - med| >= 0: its bit pattern orders like the value
    select32(R, it, I, [&](int64_t r) { return __float_as_uint(fabsf(v[r] - med)); }, k, even, L, a,
             b);
    const float mad = even ? (__uint_as_float(a) + __uint_as_float(b)) * 0.5f : __uint_as_float(a);
    if (mad > 0.f) {
      scale = 1.4826f * mad;
    } else {
      double sl = 0.0;
      for (int64_t r = t; r < R; r += RS)
        if (region_active(it, I, r)) sl += (double)fabsf(v[r] - med);
      for (int d = 32; d >= 1; d >>= 1) sl += __shfl_xor(sl, d, 64);
      if (lane == 0) L.wsum[wid] = sl;
      __syncthreads();
      double s = 0.0;
      for (int q = 0; q < RSW; q++) s += L.wsum[q];
      const double mean_ad = s / (double)n;
      if (mean_ad > 0.0) scale = (float)(1.253314 * mean_ad);
    }
  }
  for (int64_t r = t; r < R; r += RS)
    z[r] = (scale > 0.f && region_active(it, I, r)) ? (v[r] - med) / scale : 0.f;
}

// The same for at most 1,024 * V ranks with the region's values in registers
// (ta_select.h) instead of three passes over memory per order statistic:
// 64 regions of 10,000 ranks 42 -> 21 us.
template <int V>
__global__ __launch_bounds__(RS) void region_robust_reg(const float *__restrict__ v_t, int64_t R,
                                                        const int32_t *it, int I, float *z_t) {
  __shared__ SelGroup<RSW, 2048, uint32_t> L;
  __shared__ uint32_t wmn[RSW], wmx[RSW], wn[RSW];
  __shared__ double wsum[RSW];
  const int g = blockIdx.x, t = threadIdx.x, lane = t & 63, wid = t >> 6;
  const float *v = v_t + (int64_t)g * R;
  float *z = z_t + (int64_t)g * R;
  float x[V];
  uint32_t ok = 0;
#pragma unroll
  for (int j = 0; j < V; j++) {
    const int64_t r = (int64_t)j * RS + t;
    x[j] = r < R ? v[r] : 0.f;
    if (r < R && region_active(it, I, r)) ok |= 1u << j;
  }
  sel_clear(L);
  uint32_t n = 0;
  // the two middle keys of key(x) over the active ranks
  auto middle = [&](auto key, uint32_t &a, uint32_t &b) {
    uint32_t u[V], lo = 0xffffffffu, hi = 0, c = (uint32_t)__popc(ok);
#pragma unroll
    for (int j = 0; j < V; j++) {
      u[j] = key(x[j]);
      if (ok >> j & 1) {
        lo = u[j] < lo ? u[j] : lo;
        hi = u[j] > hi ? u[j] : hi;
      }
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    c = wave_sum(c);
    if (lane == 0) {
      wmn[wid] = lo;
      wmx[wid] = hi;
      wn[wid] = c;
    }
    __syncthreads();
    n = 0;
    for (int q = 0; q < RSW; q++) {
      lo = wmn[q] < lo ? wmn[q] : lo;
      hi = wmx[q] > hi ? wmx[q] : hi;
      n += wn[q];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < V; j++) u[j] = ok >> j & 1 ? u[j] - lo : 0xffffffffu;
    const uint32_t last = n > 0 ? hi - lo : 0;
    reg_select<false>(L, u, 0u, 0u, last, last ? 32 - __clz((int)last) : 0, n, n > 0 ? (n - 1) / 2 : 0u,
                      n > 0 && (n & 1) == 0, a, b);
    a += lo;
    b += lo;
  };
  float med = 0.f, scale = 0.f;
  uint32_t a, b;
  middle([&](float f) { return fkey(f); }, a, b);
  if (n > 0) {
    const bool even = (n & 1) == 0;
    med = even ? (fdec(a) + fdec(b)) * 0.5f : fdec(a);
    // |m - med| >= 0: its bit pattern orders like the value
    middle([&](float f) { return __float_as_uint(fabsf(f - med)); }, a, b);
    const float mad = even ? (__uint_as_float(a) + __uint_as_float(b)) * 0.5f : __uint_as_float(a);
    if (mad > 0.f) {
      scale = 1.4826f * mad;
    } else {  // summed as in region_robust_f32
      double sl = 0.0;
#pragma unroll
      for (int j = 0; j < V; j++)
        if (ok >> j & 1) sl += (double)fabsf(x[j] - med);
      for (int d = 32; d >= 1; d >>= 1) sl += __shfl_xor(sl, d, 64);
      if (lane == 0) wsum[wid] = sl;
      __syncthreads();
      double s = 0.0;
      for (int q = 0; q < RSW; q++) s += wsum[q];
      const double mean_ad = s / (double)n;
      if (mean_ad > 0.0) scale = (float)(1.253314 * mean_ad);
    }
  }
#pragma unroll
  for (int j = 0; j < V; j++) {
    const int64_t r = (int64_t)j * RS + t;
    if (r < R) z[r] = (scale > 0.f && (ok >> j & 1)) ? (x[j] - med) / scale : 0.f;
  }
}

// score[r] = max_g |z(r, g)| (0 for ranks without iterations).
__global__ __launch_bounds__(256) void rank_max_z32(const float *z_t, int64_t R, int G, float *score) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= R) return;
  float best = 0.f;
#pragma unroll 16
  for (int g = 0; g < G; g++)  // 16 loads in flight: 16 -> 5 us at 10,000 ranks
    best = fmaxf(best, fabsf(z_t[(int64_t)g * R + r]));
  score[r] = best;
}

// ---------------------------------------------------------------------------
// Top-k: the k largest scores (ties toward the lower rank id), listed in
// ascending rank id; also counts scores above a threshold.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void topk_kernel(const float *score, int64_t R, int64_t k,
                                                    int32_t *idx, int32_t *n_above, float thr) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t sh[4];
  __shared__ int64_t sc[1024];
  const int t = threadIdx.x;
  // Threshold key K*: the (R-k)-th smallest key (0-based); keys > K* all
  // selected, keys == K* taken in rank order until k are chosen.
  uint32_t pref = 0;
  int64_t want = R - k;  // rank of K* among ascending keys
  for (int sh_ = 24; sh_ >= 0; sh_ -= 8) {
    for (int b = t; b < 256; b += 1024) hist[b] = 0;
    __syncthreads();
    for (int64_t r = t; r < R; r += 1024) {
      const uint32_t key = fkey(score[r]);
      if (sh_ == 24 || (key >> (sh_ + 8)) == pref) atomicAdd(&hist[(key >> sh_) & 255], 1u);
    }
    __syncthreads();
    if (t == 0) {
      int64_t cum = 0;
      int b = 0;
      for (; b < 256; b++) {
        if (cum + (int64_t)hist[b] > want) break;
        cum += hist[b];
      }
      sh[0] = (pref << 8) | (uint32_t)b;
      sh[1] = (uint32_t)(want - cum);
    }
    __syncthreads();
    pref = sh[0];
    want = sh[1];
    __syncthreads();
  }
  const uint32_t kstar = pref;
  // count keys strictly greater than K*
  int64_t gt = 0, above = 0;
  for (int64_t r = t; r < R; r += 1024) {
    gt += fkey(score[r]) > kstar;
    above += score[r] > thr;
  }
  sc[t] = gt;
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if (t < s) sc[t] += sc[t + s];
    __syncthreads();
  }
  const int64_t n_gt = sc[0];
  __syncthreads();
  sc[t] = above;
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if (t < s) sc[t] += sc[t + s];
    __syncthreads();
  }
  if (t == 0 && n_above) n_above[0] = (int32_t)sc[0];
  __syncthreads();
  const int64_t ties = k - n_gt;  // how many keys equal to K* to take
  // Ordered compaction in chunks of 1024 ranks.
  int64_t base_gt = 0, base_tie = 0;
  for (int64_t c0 = 0; c0 < R; c0 += 1024) {
    const int64_t r = c0 + t;
    const uint32_t key = r < R ? fkey(score[r]) : 0u;
    const int is_gt = r < R && key > kstar;
    const int is_eq = r < R && key == kstar;
    sc[t] = ((int64_t)is_eq << 32) | is_gt;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
      const int64_t x = t >= d ? sc[t - d] : 0;
      __syncthreads();
      sc[t] += x;
      __syncthreads();
    }
    const int64_t incl = sc[t];
    const int64_t gt_before = base_gt + (incl & 0xffffffffll) - is_gt;
    const int64_t tie_before = base_tie + (incl >> 32) - is_eq;
    if (is_gt || (is_eq && tie_before < ties))
      idx[gt_before + (tie_before < ties ? tie_before : ties)] = (int32_t)r;
    const int64_t tot = sc[1023];
    __syncthreads();
    base_gt += tot & 0xffffffffll;
    base_tie += tot >> 32;
  }
}

// The same for at most 1,024 * V ranks, V consecutive ranks per thread: the
// keys stay in registers (ta_select.h), and one scan over the threads places
// what is selected in rank order.  topk_kernel walks each histogram with one
// thread and scans every 1,024 ranks with twenty barriers: 10,000 ranks 54 ->
// 15 us.
template <int V>
__global__ __launch_bounds__(1024) void topk_reg(const float *__restrict__ score, int64_t R, int64_t k,
                                                 int32_t *idx, int32_t *n_above, float thr) {
  __shared__ SelGroup<16, 2048, uint64_t> L;
  __shared__ uint32_t wgt[16], weq[16], wab[16];
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  uint64_t u[V];
  uint32_t ab = 0;
  float f[V];
#pragma unroll
  for (int j = 0; j < V; j += 4) {
    const int64_t r = (int64_t)t * V + j;
    if (r + 4 <= R) {
      const float4 q = *reinterpret_cast<const float4 *>(score + r);
      f[j] = q.x;
      f[j + 1] = q.y;
      f[j + 2] = q.z;
      f[j + 3] = q.w;
    } else {
#pragma unroll
      for (int q = 0; q < 4; q++) f[j + q] = r + q < R ? score[r + q] : 0.f;
    }
  }
#pragma unroll
  for (int j = 0; j < V; j++) {
    const bool in = (int64_t)t * V + j < R;
    u[j] = in ? (uint64_t)fkey(f[j]) : ~0ull;
    ab += in && f[j] > thr ? 1u : 0u;
  }
  sel_clear(L);
  // K*: the (R - k)-th smallest key; greater keys are all selected, keys equal
  // to it in rank order until k are chosen
  uint64_t kstar, next;
  reg_select<false>(L, u, (uint64_t)0, 0u, (uint64_t)0xffffffffu, 32, (uint32_t)R, (uint32_t)(R - k), false,
                    kstar, next);
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int j = 0; j < V; j++) {
    gt += u[j] > kstar && u[j] != ~0ull ? 1u : 0u;
    eq += u[j] == kstar ? 1u : 0u;
  }
  const uint32_t gi = wave_scan_u32(gt), ei = wave_scan_u32(eq), ai = wave_scan_u32(ab);
  if (lane == 63) {
    wgt[wid] = gi;
    weq[wid] = ei;
    wab[wid] = ai;
  }
  __syncthreads();
  uint32_t gb = gi - gt, eb = ei - eq, n_gt = 0, above = 0;
  for (int q = 0; q < 16; q++) {
    gb += q < wid ? wgt[q] : 0;
    eb += q < wid ? weq[q] : 0;
    n_gt += wgt[q];
    above += wab[q];
  }
  if (t == 0 && n_above) n_above[0] = (int32_t)above;
  const uint32_t ties = (uint32_t)k - n_gt;  // how many keys equal to K* to take
#pragma unroll
  for (int j = 0; j < V; j++) {
    const bool is_gt = u[j] > kstar && u[j] != ~0ull, is_eq = u[j] == kstar;
    if (is_gt || (is_eq && eb < ties)) idx[gb + (eb < ties ? eb : ties)] = (int32_t)((int64_t)t * V + j);
    gb += is_gt ? 1u : 0u;
    eb += is_eq ? 1u : 0u;
  }
}

}  // namespace

hipError_t ae_alloc(AeState &s) {
  hipError_t e = hipSuccess;
  auto A = [&](void **p, size_t b) {
    if (e == hipSuccess) e = hipMalloc(p, b);
  };
  A((void **)&s.w, AE_NP * 4);
  A((void **)&s.wb, AE_NB16 * 2);
  A((void **)&s.m, AE_NP * 4);
  A((void **)&s.v, AE_NP * 4);
  A((void **)&s.mu, 64 * 4);
  A((void **)&s.isd, 64 * 4);
  A((void **)&s.nsum, 64 * 8);
  A((void **)&s.nsq, 128 * 8);
  A((void **)&s.ncnt, 8 * 8);
  A((void **)&s.part, (size_t)AE_WG * AE_PS * 4);
  A((void **)&s.loss, 16);
  return e;
}

void ae_free(AeState &s) {
  void *ps[] = {s.w, s.wb, s.m, s.v, s.mu, s.isd, s.nsum, s.nsq, s.ncnt, s.part, s.loss};
  for (void *p : ps)
    if (p) (void)hipFree(p);
  s = AeState{};
}

hipError_t launch_ae_init(AeState &s, uint64_t seed, hipStream_t st) {
  hipLaunchKernelGGL(ae_init_kernel, dim3((AE_NP + 255) / 256), dim3(256), 0, st, seed, s.w, s.wb,
                     s.m, s.v);
  s.step = 0;
  return hipGetLastError();
}

size_t ae_norm_ws_bytes(int64_t R) {
  const int64_t nb = (R + 63) / 64 < 1024 ? (R + 63) / 64 + 1 : 1025;
  return (size_t)nb * (64 * 8 + 128 * 8 + 8) + 1024;
}

hipError_t launch_ae_norm(AeState &s, const int64_t *T, int64_t R, int I, const int32_t *it,
                          bool reset, void *ws, size_t ws_bytes, hipStream_t st) {
  int64_t nb = (R + 63) / 64;
  if (nb > 1024) nb = 1024;
  if (nb < 1) nb = 1;
  const int64_t rpb = (R + nb - 1) / nb;
  char *p = (char *)ws;
  int64_t *ps = (int64_t *)p;
  uint64_t *pq = (uint64_t *)(p + nb * 64 * 8);
  int64_t *pc = (int64_t *)(p + nb * 64 * 8 + nb * 128 * 8);
  if ((size_t)(nb * (64 * 8 + 128 * 8 + 8)) > ws_bytes) return hipErrorInvalidValue;
  hipLaunchKernelGGL(ae_norm_partial, dim3((unsigned)nb), dim3(256), 0, st, T, R, I, it, rpb, ps, pq, pc);
  hipLaunchKernelGGL(ae_norm_final, dim3(1), dim3(64), 0, st, (int)nb, ps, pq, pc, reset ? 1 : 0,
                     s.nsum, s.nsq, s.ncnt, s.mu, s.isd);
  return hipGetLastError();
}

size_t ae_rows_ws_bytes(int64_t R) { return (size_t)(R + 1) * 8 + 256; }

hipError_t launch_ae_rows(const AeState &s, const int64_t *T, int64_t R, int I, const int32_t *it,
                          float *rows, int64_t *n_rows, void *ws, size_t ws_bytes, hipStream_t st) {
  if ((size_t)(R + 1) * 8 > ws_bytes) return hipErrorInvalidValue;
  int64_t *off = (int64_t *)ws;
  hipLaunchKernelGGL(ae_rows_scan, dim3(1), dim3(1024), 0, st, it, R, I, off);
  if (rows && R > 0)
    hipLaunchKernelGGL(ae_rows_fill, dim3((unsigned)R), dim3(256), 0, st, T, R, I, off, s.mu, s.isd, rows);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && n_rows) e = hipMemcpyAsync(n_rows, off + R, 8, hipMemcpyDeviceToHost, st);
  return e;
}

hipError_t launch_ae_step(AeState &s, const float *rows, int64_t n, int64_t k0, int batch,
                          uint64_t a, uint64_t c, float lr, bool update, float noise_sd,
                          uint64_t noise_key, hipStream_t st, float *grad_out, float *loss_out,
                          float *epoch_loss, float lfrac) {
  const int64_t k_end = k0 + batch < n ? k0 + batch : n;
  const int64_t bv = k_end - k0;
  if (bv <= 0) return hipErrorInvalidValue;
  const float scale = 2.0f / (float)(bv * AE_IN);
  hipLaunchKernelGGL(ae_fwdbwd, dim3(AE_WG), dim3(AT), 0, st, rows, n, k0, k_end, (int64_t)a, (int64_t)c,
                     1.0 / (double)n, scale, noise_sd, noise_key, s.wb, s.w, s.part);
  float bc1 = 1.f, bc2 = 1.f;
  if (update) {
    s.step++;
    bc1 = (float)(1.0 - pow(0.9, (double)s.step));
    bc2 = (float)(1.0 - pow(0.999, (double)s.step));
  }
  hipLaunchKernelGGL(ae_adam<true>, dim3(AE_NP / AP + 1), dim3(ADT), 0, st, s.part, AE_WG, s.w, s.wb,
                     s.m, s.v, lr, bc1, bc2, update ? 1 : 0, grad_out, loss_out ? loss_out : s.loss,
                     1.0f / (float)(bv * AE_IN), epoch_loss, lfrac);
  return hipGetLastError();
}

hipError_t launch_ae_grad_f32(AeState &s, const float *rows, int64_t n, float noise_sd,
                              uint64_t noise_key, hipStream_t st, float *grad_out, float *loss_out) {
  if (n <= 0) return hipErrorInvalidValue;
  const float scale = 2.0f / (float)(n * AE_IN);
  hipLaunchKernelGGL(ae_grad_f32_kernel, dim3(AE_WG), dim3(256), 0, st, rows, n, scale, noise_sd,
                     noise_key, s.w, s.part);
  hipLaunchKernelGGL(ae_adam<false>, dim3(AE_NP / AP + 1), dim3(ADT), 0, st, s.part, AE_WG, s.w, s.wb,
                     s.m, s.v, 0.f, 1.f, 1.f, 0, grad_out, loss_out ? loss_out : s.loss,
                     1.0f / (float)(n * AE_IN), (float *)nullptr, 0.f);
  return hipGetLastError();
}

size_t ae_score_ws_bytes(int64_t R) { return 2 * (((size_t)R * AE_IN * 4 + 255) & ~(size_t)255); }

hipError_t launch_ae_score(const AeState &s, const int64_t *T, int64_t R, int I, const int32_t *it,
                           float *score, void *ws, size_t ws_bytes, hipStream_t st) {
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&ae_score_kernel<true>),
                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(ScoreLds));
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&ae_score_kernel<false>),
                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(ScoreLds));
    attr = true;
  }
  if (R <= 0) return hipSuccess;
  const bool stage2 = s.score_kind == 2;
  const size_t half = ae_score_ws_bytes(R) / 2;
  if (stage2 && (ws == nullptr || ws_bytes < 2 * half)) return hipErrorInvalidValue;
  float *v_t = stage2 ? (float *)ws : nullptr;
  float *z_t = stage2 ? (float *)((char *)ws + half) : nullptr;
  int cus = 256, dev = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  int64_t grid = (R + SW - 1) / SW;
  if (grid > cus) grid = cus;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(SW * 64), sizeof(ScoreLds), st, T, R, I, it, s.wb, s.w,
                       s.mu, s.isd, s.score_kind, score, v_t);
  };
  if (s.score_kind == 0) go(ae_score_kernel<true>);
  else go(ae_score_kernel<false>);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && stage2) {
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(AE_IN), dim3(RS), 0, st, (const float *)v_t, R, it, I, z_t);
    };
    // the fewest keys per lane that hold a region, in half octaves (20,000 ranks, the
    // whole pre-screen: 165 us with 32, 147 with 24; 10,000 with 16 100, with 12 98)
    if (R <= 1024) go(region_robust_reg<1>);
    else if (R <= 4096) go(region_robust_reg<4>);
    else if (R <= 8192) go(region_robust_reg<8>);
    else if (R <= 12288) go(region_robust_reg<12>);
    else if (R <= 16384) go(region_robust_reg<16>);
    else if (R <= 24576) go(region_robust_reg<24>);
    else if (R <= 32768) go(region_robust_reg<32>);
    else go(region_robust_f32);
    hipLaunchKernelGGL(rank_max_z32, dim3((unsigned)((R + 255) / 256)), dim3(256), 0, st, z_t, R, AE_IN,
                       score);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_topk(const float *score, int64_t R, int64_t k, int32_t *idx, int32_t *n_above,
                       float thr, hipStream_t st) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(1), dim3(1024), 0, st, score, R, k, idx, n_above, thr);
  };
  if (R <= 4096) go(topk_reg<4>);
  else if (R <= 8192) go(topk_reg<8>);
  else if (R <= 12288) go(topk_reg<12>);
  else if (R <= 16384) go(topk_reg<16>);
  else if (R <= 24576) go(topk_reg<24>);
  else if (R <= 32768) go(topk_reg<32>);
  else go(topk_kernel);
  return hipGetLastError();
}

}  // namespace ta

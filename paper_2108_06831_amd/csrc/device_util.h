// Device helpers shared by the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace tnq {
namespace {

constexpr int kThreads = 256;

__device__ inline float2 f2(float x, float y) { return make_float2(x, y); }

// round-to-nearest-even to bfloat16, returned as float
__device__ inline float bf16_round(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return __uint_as_float(u & 0xffff0000u);
}

// a*b (real) in the requested precision: FP32, or the three-term bf16 split
template <int PREC>
__device__ inline float rmul(float a, float b) {
  if constexpr (PREC == TN_PREC_C64) {
    return a * b;
  } else {
    const float ah = bf16_round(a), al = bf16_round(a - ah);
    const float bh = bf16_round(b), bl = bf16_round(b - bh);
    return fmaf(ah, bh, fmaf(ah, bl, al * bh));
  }
}

// acc + a b.  In FP32 as two fused multiply-adds per component (a separate
// product, difference and sum would take three instructions each).
template <int PREC>
__device__ inline float2 cmac(float2 acc, float2 a, float2 b) {
  if constexpr (PREC == TN_PREC_C64) {
    acc.x = fmaf(a.x, b.x, fmaf(-a.y, b.y, acc.x));
    acc.y = fmaf(a.x, b.y, fmaf(a.y, b.x, acc.y));
  } else {
    acc.x += rmul<PREC>(a.x, b.x) - rmul<PREC>(a.y, b.y);
    acc.y += rmul<PREC>(a.x, b.y) + rmul<PREC>(a.y, b.x);
  }
  return acc;
}

// a b (no accumulator): one product and one fused multiply-add per component
template <int PREC>
__device__ inline float2 cmul(float2 a, float2 b) {
  if constexpr (PREC == TN_PREC_C64)
    return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
  else
    return make_float2(rmul<PREC>(a.x, b.x) - rmul<PREC>(a.y, b.y), rmul<PREC>(a.x, b.y) + rmul<PREC>(a.y, b.x));
}

__device__ inline double block_sum(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) red[w] = v;
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
  __syncthreads();
  return t;
}

// deposit(x, pos, nbits): bit j of x (j < nbits) placed at address position
// pos[j]; the address maps of the permute and matrix-product kernels.
// The positions are read four at a time as 32-bit words (each map starts at
// a multiple of 4 bytes of the argument block): word loads of the argument
// block are scalar loads, while a byte-wise read becomes one vector memory
// load per bit that the loop waits for.
static_assert(kGemmMaxBits % 4 == 0, "position maps of whole 32-bit words");
__device__ inline int64_t deposit(int64_t x, const int8_t* pos, int nbits) {
  const int32_t* w = reinterpret_cast<const int32_t*>(pos);
  int64_t r = 0;
  for (int j = 0; j < nbits; j += 4) {
    const int32_t p4 = w[j >> 2];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (j + q < nbits) r |= ((x >> (j + q)) & 1) << ((p4 >> (8 * q)) & 63);
  }
  return r;
}
// Streaming (non-temporal) loads and stores.  The matrix products store their
// results this way: a large product writes far more result than it reads
// operands, and ordinary stores would evict the operand tiles that later
// tiles of the same XCD still read from its L2.  The fused passes move each
// chunk through once.
typedef float float2_nt __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_stream(float2* p, float re, float im) {
  float2_nt v;
  v.x = re;
  v.y = im;
  __builtin_nontemporal_store(v, reinterpret_cast<float2_nt*>(p));
}
__device__ __forceinline__ float2 load_stream(const float2* p) {
  const float2_nt v = __builtin_nontemporal_load(reinterpret_cast<const float2_nt*>(p));
  return f2(v.x, v.y);
}

// w[j] <- sum over mu of w[mu] (-1)^popc(j & mu)
__device__ inline void walsh16(double (&w)[16]) {
#pragma unroll
  for (int h = 1; h < 16; h <<= 1)
#pragma unroll
    for (int a = 0; a < 16; a += 2 * h)
#pragma unroll
      for (int b = a; b < a + h; ++b) {
        const double u = w[b], v = w[b + h];
        w[b] = u + v;
        w[b + h] = u - v;
      }
}

// D at sixteen addresses: A with none of four bits set, and every combination
// of them, the terms sorted by their pattern mu of those bits.  Each term's
// sign at A is taken once, the sums per pattern go into w[mu], and a 16-point
// Walsh-Hadamard transform gives D at combination j = sum_mu w[mu] (-1)^popc(j & mu).
__device__ inline void sum_terms16(uint64_t A, const ZTerms& t, double (&w)[16]) {
#pragma unroll
  for (int mu = 0; mu < 16; ++mu) {
    double acc = 0;
    for (int i = t.mu_start[mu]; i < t.mu_start[mu + 1]; ++i)
      acc += (__popcll(A & t.mask[i]) & 1) ? -t.coeff[i] : t.coeff[i];
    w[mu] = acc;
  }
  walsh16(w);
}

}  // namespace
}  // namespace tnq

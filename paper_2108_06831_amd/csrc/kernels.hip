// gfx950 kernels of the contraction path.
//
//  * k_materialize / k_projectors: gate tensors from angles (FP64, rounded once
//    to complex64), |0> vectors and one-hot bitstring projectors.
//  * k_skinny: a pairwise contraction whose smaller operand is gate-sized.  It
//    streams the large operand once from HBM (HBM-bound) through strided
//    addresses, so no permute is needed before it.
//  * k_permute: bit-permutation transpose staged through LDS so that both the
//    reads and the writes are coalesced.
//  * k_gemm: complex matrix product on the FP32 matrix cores (4M form through
//    a real embedding, below), batched over the batch modes.
//  * k_expect_* / k_adjoint_*: FP64-accumulated reductions for expectations
//    and the adjoint gradient.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "device_util.h"
#include "kernels.h"

namespace tnq {

// ---------------------------------------------------------------------------
// Materialisation of the network's input tensors
// ---------------------------------------------------------------------------
// One block per tensor: the elementary matrices of the tensor's ops (the FP64
// trigonometry) are evaluated in parallel, one op per thread, into LDS; one
// thread then multiplies them in order, with the block matrices in registers
// (every array below is indexed by constants).  Rounded once to complex64.
constexpr int kRecipeThreads = 64;

// The nearest Q3.28 value (raw int32 = value * 2^28), ties to even, saturated.
__device__ inline int32_t q328_from_double(double x) {
  const double r = rint(x * 268435456.0);
  return r >= 2147483647.0 ? 2147483647 : r <= -2147483648.0 ? (int32_t)0x80000000 : (int32_t)r;
}

// One FP64 complex value stored rounded once: to complex64 (Q = false) or to
// a Q3.28 (re, im) pair in the same 8 bytes (Q = true).
template <bool Q>
__device__ inline void store_c(float2* o, int i, const c128& v) {
  if constexpr (Q)
    reinterpret_cast<int2*>(o)[i] = make_int2(q328_from_double(v.re), q328_from_double(v.im));
  else
    o[i] = f2((float)v.re, (float)v.im);
}

template <bool Q, class GetU>
__device__ void write_recipe(const Recipe& r, const RecipeOp* ops, GetU get_u, float2* o) {
  if (r.split_side >= 0) {
    c128 H[8];
    recipe_split_half_g(r, ops, get_u, H);
#pragma unroll
    for (int i = 0; i < 8; ++i) store_c<Q>(o, i, H[i]);
  } else if (r.nq == 2) {
    c128 M[16];
    recipe_matrix_dg<4>(r, ops, get_u, M);
    if (r.diag) {
#pragma unroll
      for (int i = 0; i < 4; ++i) store_c<Q>(o, i, M[5 * i]);
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) store_c<Q>(o, i, M[i]);
    }
  } else {
    c128 M[4];
    recipe_matrix_dg<2>(r, ops, get_u, M);
    if (r.diag) {
      store_c<Q>(o, 0, M[0]);
      store_c<Q>(o, 1, M[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) store_c<Q>(o, i, M[i]);
    }
  }
}

// tensor d of one parameter vector (p) into o
template <bool Q>
__device__ __forceinline__ void materialize_tensor(const DevTensor& d, const Recipe* rs, const RecipeOp* ops,
                                                   const double* mats, const double* p, float2* o) {
  __shared__ c128 U[kRecipeThreads][16];
  if (d.kind == TK_KET0) {
    if (threadIdx.x == 0) {
      store_c<Q>(o, 0, c128{1.0, 0.0});
      store_c<Q>(o, 1, c128{0.0, 0.0});
    }
  } else if (d.kind == TK_GATE) {
    const Recipe r = rs[d.recipe];
    const int n = r.op_end - r.op_begin;
    if (n <= kRecipeThreads) {
      if ((int)threadIdx.x < n) {
        c128 u[16];
        op_matrix(ops[r.op_begin + threadIdx.x], mats, p, u);
#pragma unroll
        for (int i = 0; i < 16; ++i) U[threadIdx.x][i] = u[i];
      }
      __syncthreads();
      if (threadIdx.x == 0)
        write_recipe<Q>(r, ops, [&](int op, c128* u) {
#pragma unroll
          for (int i = 0; i < 16; ++i) u[i] = U[op - r.op_begin][i];
        }, o);
    } else if (threadIdx.x == 0) {
      write_recipe<Q>(r, ops, [&](int op, c128* u) { op_matrix(ops[op], mats, p, u); }, o);
    }
  }
}

template <bool Q>
__global__ __launch_bounds__(kRecipeThreads) void k_materialize(const DevTensor* ts, int nt, const Recipe* rs,
                                                                const RecipeOp* ops, const double* mats,
                                                                const double* params, int64_t pstride, float2* in,
                                                                int64_t in_bs) {
  const int t = blockIdx.x;
  const int z = blockIdx.y;
  if (t >= nt) return;
  const DevTensor d = ts[t];
  materialize_tensor<Q>(d, rs, ops, mats, params ? params + (int64_t)z * pstride : nullptr,
                        in + (int64_t)z * in_bs + d.offset);
}

__global__ __launch_bounds__(kRecipeThreads) void k_materialize_many(MatArgs a) {
  const int z = blockIdx.y;
  int i = 0;
  while (i + 1 < a.n && (int)blockIdx.x >= a.net[i + 1].block0) ++i;
  const MatNet& m = a.net[i];
  const DevTensor d = m.ts[(int)blockIdx.x - m.block0];
  materialize_tensor<false>(d, m.recipes, m.ops, m.mats,
                            m.params ? m.params + (int64_t)z * m.params_stride : nullptr,
                            m.in + (int64_t)z * m.in_bs + d.offset);
}

hipError_t launch_materialize_many(hipStream_t s, MatArgs& a, int batch) {
  if (a.n < 1 || a.n > kMatMax) return hipErrorInvalidValue;
  int blocks = 0;
  for (int i = 0; i < a.n; ++i) {
    if (a.net[i].n_tensors < 1) return hipErrorInvalidValue;
    a.net[i].block0 = blocks;
    blocks += a.net[i].n_tensors;
  }
  hipLaunchKernelGGL(k_materialize_many, dim3(blocks, batch), dim3(kRecipeThreads), 0, s, a);
  return hipGetLastError();
}

// one_bits: the 32-bit pattern of the value 1 (1.0f, or 2^28 in Q3.28)
__global__ void k_projectors(const uint64_t* bits, int64_t count, int n, int blog2, int64_t first, float2* in,
                             int64_t in_bs, uint32_t one_bits) {
  const int64_t per = (int64_t)1 << blog2;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int z = blockIdx.y;
  if (i >= per * n) return;
  const int q = (int)(i / per);
  const int64_t s = i % per;
  const int bit = s < count ? (int)((bits[s] >> (n - 1 - q)) & 1) : 0;
  uint2* o = reinterpret_cast<uint2*>(in + (int64_t)z * in_bs + first + (int64_t)q * per * 2 + 2 * s);
  o[0] = make_uint2(bit == 0 ? one_bits : 0u, 0u);
  o[1] = make_uint2(bit == 1 ? one_bits : 0u, 0u);
}

hipError_t launch_materialize(hipStream_t s, const DevTensor* ts, int nt, const Recipe* recipes, const RecipeOp* ops,
                              const double* mats, const double* params, int64_t params_stride, int batch,
                              float2* in, int64_t in_bs, bool q328) {
  if (nt == 0) return hipSuccess;
  if (q328)
    hipLaunchKernelGGL(k_materialize<true>, dim3(nt, batch), dim3(kRecipeThreads), 0, s, ts, nt, recipes, ops, mats,
                       params, params_stride, in, in_bs);
  else
    hipLaunchKernelGGL(k_materialize<false>, dim3(nt, batch), dim3(kRecipeThreads), 0, s, ts, nt, recipes, ops, mats,
                       params, params_stride, in, in_bs);
  return hipGetLastError();
}

hipError_t launch_projectors(hipStream_t s, const uint64_t* bits, int64_t count, int n_qubits, int blog2,
                             int64_t first_offset, int batch, float2* in, int64_t in_bs, bool q328) {
  const int64_t total = ((int64_t)1 << blog2) * n_qubits;
  dim3 grid((unsigned)((total + kThreads - 1) / kThreads), batch);
  const uint32_t one = q328 ? (1u << 28) : 0x3f800000u;
  hipLaunchKernelGGL(k_projectors, grid, dim3(kThreads), 0, s, bits, count, n_qubits, blog2, first_offset, in, in_bs,
                     one);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Q3.28 fixed point: one step of a path as a per-output product over raw int32
// (re, im) pairs (value = raw / 2^28).  Every real product is the exact 64-bit
// product shifted back by 28 bits, rounded to nearest with ties to even and
// saturated; every sum saturates at the int32 range.
// ---------------------------------------------------------------------------
__device__ inline int32_t q_sat(int64_t v) {
  return v > 2147483647ll ? 2147483647 : v < -2147483648ll ? (int32_t)0x80000000 : (int32_t)v;
}
__device__ inline int64_t q_mul(int32_t a, int32_t b) {
  const int64_t p = (int64_t)a * (int64_t)b;
  int64_t q = p >> 28;
  const int64_t rem = p & (((int64_t)1 << 28) - 1);
  q += (rem > ((int64_t)1 << 27)) | ((rem == ((int64_t)1 << 27)) & (q & 1));
  return q_sat(q);
}

constexpr int kQChunks = (kQMaxOutBits + 7) / 8;  // 8-bit chunks of a result index
constexpr int kQKTable = 1024;                    // summed indices resolved through an LDS table

struct QStepArgs {
  const int2* a;
  const int2* b;
  int2* c;
  int64_t a_bs, b_bs, c_bs;
  QStep st;
};

__global__ __launch_bounds__(kThreads) void k_q328_step(QStepArgs g) {
  __shared__ int64_t ta[kQChunks][256], tb[kQChunks][256];
  __shared__ int64_t ka[kQKTable], kb[kQKTable];
  const QStep& q = g.st;
  const int nc = (q.n_out + 7) / 8;
  const int nkl = q.n_k < 10 ? q.n_k : 10;  // low summed bits through the table
  for (int i = threadIdx.x; i < nc * 256; i += kThreads) {
    const int c = i >> 8, v = i & 255;
    int64_t da = 0, db = 0;
    for (int j = 0; j < 8; ++j) {
      const int bit = 8 * c + j;
      if (bit >= q.n_out || !((v >> j) & 1)) continue;
      if (q.a_o[bit] >= 0) da |= (int64_t)1 << q.a_o[bit];
      if (q.b_o[bit] >= 0) db |= (int64_t)1 << q.b_o[bit];
    }
    ta[c][v] = da;
    tb[c][v] = db;
  }
  for (int k = threadIdx.x; k < (1 << nkl); k += kThreads) {
    int64_t da = 0, db = 0;
    for (int j = 0; j < nkl; ++j)
      if ((k >> j) & 1) {
        da |= (int64_t)1 << q.a_k[j];
        db |= (int64_t)1 << q.b_k[j];
      }
    ka[k] = da;
    kb[k] = db;
  }
  __syncthreads();
  const int z = blockIdx.y;
  const int2* A = g.a + (int64_t)z * g.a_bs;
  const int2* B = g.b + (int64_t)z * g.b_bs;
  int2* C = g.c + (int64_t)z * g.c_bs;
  const int64_t n_out = (int64_t)1 << q.n_out;
  const int64_t n_hi = (int64_t)1 << (q.n_k - nkl);
  for (int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x; o < n_out; o += (int64_t)gridDim.x * kThreads) {
    int64_t a0 = 0, b0 = 0;
    for (int c = 0; c < nc; ++c) {
      const int v = (int)((o >> (8 * c)) & 255);
      a0 |= ta[c][v];
      b0 |= tb[c][v];
    }
    int32_t re = 0, im = 0;
    for (int64_t h = 0; h < n_hi; ++h) {
      int64_t ah = a0, bh = b0;
      for (int j = nkl; j < q.n_k; ++j)
        if ((h >> (j - nkl)) & 1) {
          ah |= (int64_t)1 << q.a_k[j];
          bh |= (int64_t)1 << q.b_k[j];
        }
      for (int k = 0; k < (1 << nkl); ++k) {
        const int2 x = A[ah | ka[k]], y = B[bh | kb[k]];
        const int32_t pr = q_sat(q_mul(x.x, y.x) - q_mul(x.y, y.y));
        const int32_t pi = q_sat(q_mul(x.x, y.y) + q_mul(x.y, y.x));
        re = q_sat((int64_t)re + pr);
        im = q_sat((int64_t)im + pi);
      }
    }
    C[o] = make_int2(re, im);
  }
}

hipError_t launch_q328_step(hipStream_t s, const QStep& q, const void* a, int64_t a_bs, const void* b, int64_t b_bs,
                            void* c, int64_t c_bs, int batch) {
  if (q.n_out < 0 || q.n_out > kQMaxOutBits || q.n_k < 0 || q.n_k > kQMaxKBits) return hipErrorInvalidValue;
  QStepArgs g;
  g.a = (const int2*)a; g.b = (const int2*)b; g.c = (int2*)c;
  g.a_bs = a_bs; g.b_bs = b_bs; g.c_bs = c_bs;
  g.st = q;
  int64_t blocks = (((int64_t)1 << q.n_out) + kThreads - 1) / kThreads;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_q328_step, dim3((unsigned)blocks, batch), dim3(kThreads), 0, s, g);
  return hipGetLastError();
}

// out[z][o] (complex64) = the Q3.28 value at F[z][deposit(o)], where bit j of o
// sits at bit pos[j] of F's address
__global__ __launch_bounds__(kThreads) void k_q328_finish(const int2* F, int64_t f_bs, float2* out, int64_t out_bs,
                                                          int64_t count, QStep map) {
  __shared__ int64_t ta[kQChunks][256];
  const int nc = (map.n_out + 7) / 8;
  for (int i = threadIdx.x; i < nc * 256; i += kThreads) {
    const int c = i >> 8, v = i & 255;
    int64_t d = 0;
    for (int j = 0; j < 8; ++j) {
      const int bit = 8 * c + j;
      if (bit < map.n_out && ((v >> j) & 1)) d |= (int64_t)1 << map.a_o[bit];
    }
    ta[c][v] = d;
  }
  __syncthreads();
  const int z = blockIdx.y;
  for (int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x; o < count; o += (int64_t)gridDim.x * kThreads) {
    int64_t a = 0;
    for (int c = 0; c < nc; ++c) a |= ta[c][(o >> (8 * c)) & 255];
    const int2 v = F[(int64_t)z * f_bs + a];
    out[(int64_t)z * out_bs + o] = f2((float)((double)v.x * (1.0 / 268435456.0)), (float)((double)v.y * (1.0 / 268435456.0)));
  }
}

hipError_t launch_q328_finish(hipStream_t s, const void* f, int64_t f_bs, float2* out, int64_t out_bs, int64_t count,
                              const QStep& map, int batch) {
  if (map.n_out < 0 || map.n_out > kQMaxOutBits) return hipErrorInvalidValue;
  int64_t blocks = (count + kThreads - 1) / kThreads;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_q328_finish, dim3((unsigned)std::max<int64_t>(blocks, 1), batch), dim3(kThreads), 0, s,
                     (const int2*)f, f_bs, out, out_bs, count, map);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Small-operand contraction
// ---------------------------------------------------------------------------
struct SkinnyArgs {
  const float2* g;
  const float2* t;
  float2* c;
  int64_t g_bs, t_bs, c_bs;
  int64_t n_outer;
  int32_t nb, c_mode, g_elems, pad;
  int32_t k_pos[kSkinnyMaxK];
  int32_t b_pos[kSkinnyMaxG];
  int64_t kofs[1 << kSkinnyMaxK];
  int64_t mofs[1 << kSkinnyMaxM];
  int32_t gidx[1 << kSkinnyMaxG];
};

template <int NK, int NM, int PREC>
__global__ __launch_bounds__(kThreads) void k_skinny(SkinnyArgs a) {
  __shared__ float2 gs[1 << kSkinnyMaxG];
  const int z = blockIdx.y;
  const float2* G = a.g + (int64_t)z * a.g_bs;
  const float2* Tp = a.t + (int64_t)z * a.t_bs;
  float2* Cp = a.c + (int64_t)z * a.c_bs;
  for (int i = threadIdx.x; i < a.g_elems; i += kThreads) gs[i] = G[a.gidx[i]];
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x; o < a.n_outer; o += stride) {
    int64_t tb = o;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
      const int p = a.k_pos[j];
      tb = ((tb >> p) << (p + 1)) | (tb & (((int64_t)1 << p) - 1));
    }
    int b = 0;
    for (int j = 0; j < a.nb; ++j) b |= (int)((o >> a.b_pos[j]) & 1) << j;
    float2 x[1 << NK];
#pragma unroll
    for (int k = 0; k < (1 << NK); ++k) x[k] = Tp[tb | a.kofs[k]];
    const int64_t cb = a.c_mode ? o : tb;
    const float2* gb = gs + (b << (NM + NK));
#pragma unroll
    for (int m = 0; m < (1 << NM); ++m) {
      float2 acc = f2(0.f, 0.f);
#pragma unroll
      for (int k = 0; k < (1 << NK); ++k) acc = cmac<PREC>(acc, gb[(m << NK) + k], x[k]);
      Cp[cb | a.mofs[m]] = acc;
    }
  }
}

// A run of outer products (see OuterChain): block (h, z) writes the 2^t_bits
// elements of C whose vector bits are h, T times the block's factor
// g_1[h_1] .. g_k[h_k].  The factor is formed in FP32 whatever the precision
// of the products (each step has a single term: there is nothing to sum).
struct OuterArgs {
  const float2* t;
  float2* c;
  const float2* in;
  const float2* ws;
  int64_t t_bs, c_bs, in_bs, ws_bs;
  int32_t t_bits, k;
  int64_t vsrc[kOuterMax][2];
};

__global__ __launch_bounds__(kThreads) void k_outer_chain(OuterArgs a) {
  const int z = blockIdx.y;
  const int64_t h = blockIdx.x;
  float2 f = f2(1.f, 0.f);
  for (int i = 0; i < a.k; ++i) {
    const int64_t v = a.vsrc[i][(h >> i) & 1];
    const float2* b = ((v >> 56) & 0x3f) == BUF_IN ? a.in + (int64_t)z * a.in_bs : a.ws + (int64_t)z * a.ws_bs;
    f = cmul<TN_PREC_C64>(f, b[v & (((int64_t)1 << 56) - 1)]);
  }
  // two elements per access (t_bits >= 8)
  const float4* T = reinterpret_cast<const float4*>(a.t + (int64_t)z * a.t_bs);
  float4* C = reinterpret_cast<float4*>(a.c + (int64_t)z * a.c_bs + (h << a.t_bits));
  const int64_t n = (int64_t)1 << (a.t_bits - 1);
  for (int64_t o = threadIdx.x; o < n; o += blockDim.x) {
    const float4 x = T[o];
    const float2 y0 = cmul<TN_PREC_C64>(f, f2(x.x, x.y)), y1 = cmul<TN_PREC_C64>(f, f2(x.z, x.w));
    C[o] = make_float4(y0.x, y0.y, y1.x, y1.y);
  }
}

hipError_t launch_outer_chain(hipStream_t s, const OuterChain& oc, const float2* t, int64_t t_bs, float2* c,
                              int64_t c_bs, const float2* in, int64_t in_bs, const float2* ws, int64_t ws_bs,
                              int batch) {
  if (oc.k < 1 || oc.k > kOuterMax || oc.k > 24 || oc.t_bits < 8 || oc.t_bits > 40) return hipErrorInvalidValue;
  if ((reinterpret_cast<uintptr_t>(t) | reinterpret_cast<uintptr_t>(c)) & 15) return hipErrorInvalidValue;
  if (((t_bs | c_bs) & 1) != 0) return hipErrorInvalidValue;  // float4 accesses in every batch item
  OuterArgs a;
  a.t = t; a.c = c; a.in = in; a.ws = ws;
  a.t_bs = t_bs; a.c_bs = c_bs; a.in_bs = in_bs; a.ws_bs = ws_bs;
  a.t_bits = oc.t_bits;
  a.k = oc.k;
  for (int i = 0; i < kOuterMax; ++i)
    for (int m = 0; m < 2; ++m) a.vsrc[i][m] = i < oc.k ? oc.vsrc[i][m] : 0;
  hipLaunchKernelGGL(k_outer_chain, dim3(1u << oc.k, batch), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

template <int NK, int NM>
static void* skinny_fn(int prec) {
  return prec == TN_PREC_BF16X3 ? (void*)k_skinny<NK, NM, TN_PREC_BF16X3> : (void*)k_skinny<NK, NM, TN_PREC_C64>;
}

template <int NK>
static void* skinny_fn_m(int nm, int prec) {
  switch (nm) {
    case 0: return skinny_fn<NK, 0>(prec);
    case 1: return skinny_fn<NK, 1>(prec);
    case 2: return skinny_fn<NK, 2>(prec);
    case 3: return skinny_fn<NK, 3>(prec);
    default: return skinny_fn<NK, 4>(prec);
  }
}

hipError_t launch_skinny(hipStream_t s, const SkinnyDesc& d, const float2* g, int64_t g_bs, const float2* t,
                         int64_t t_bs, float2* c, int64_t c_bs, int batch, int precision) {
  SkinnyArgs a;
  a.g = g; a.t = t; a.c = c;
  a.g_bs = g_bs; a.t_bs = t_bs; a.c_bs = c_bs;
  a.n_outer = (int64_t)1 << (d.t_bits - d.nk);
  a.nb = d.nb;
  a.c_mode = d.c_mode;
  a.g_elems = 1 << (d.nb + d.nm + d.nk);
  a.pad = 0;
  for (int j = 0; j < kSkinnyMaxK; ++j) a.k_pos[j] = d.k_pos[j];
  for (int j = 0; j < kSkinnyMaxG; ++j) a.b_pos[j] = d.b_pos[j];
  for (int j = 0; j < (1 << kSkinnyMaxK); ++j) a.kofs[j] = d.kofs[j];
  for (int j = 0; j < (1 << kSkinnyMaxM); ++j) a.mofs[j] = d.mofs[j];
  for (int j = 0; j < (1 << kSkinnyMaxG); ++j) a.gidx[j] = d.gidx[j];
  void* fn;
  switch (d.nk) {
    case 0: fn = skinny_fn_m<0>(d.nm, precision); break;
    case 1: fn = skinny_fn_m<1>(d.nm, precision); break;
    case 2: fn = skinny_fn_m<2>(d.nm, precision); break;
    case 3: fn = skinny_fn_m<3>(d.nm, precision); break;
    default: fn = skinny_fn_m<4>(d.nm, precision); break;
  }
  int64_t blocks = (a.n_outer + kThreads - 1) / kThreads;
  if (blocks > 16384) blocks = 16384;
  void* args[] = {&a};
  return hipLaunchKernel(fn, dim3((unsigned)blocks, batch), dim3(kThreads), args, 0, s);
}

// ---------------------------------------------------------------------------
// Interpreter of small steps (one launch for all the tiny contractions that
// only depend on inputs): each workgroup walks one independent work list.
// A step is computed into registers, then written after a barrier, so a step
// may overwrite one of its own operands.
// ---------------------------------------------------------------------------

// byte j (0..11) of three packed words, sign-extended
__device__ inline int packed_byte(uint32_t w0, uint32_t w1, uint32_t w2, int j) {
  const uint32_t x = j < 4 ? w0 : j < 8 ? w1 : w2;
  return (int)(int8_t)(x >> (8 * (j & 3)));
}

constexpr int kStageInFlight = 8;  // operand loads each interpreter thread issues before it waits

template <int PREC>
__global__ __launch_bounds__(kSmallThreads) void k_small_steps(const SmallStep* steps, const int32_t* list_off,
                                                          const int32_t* level_off, const uint32_t* items,
                                                          float2* in, int64_t in_bs, float2* ws, int64_t ws_bs) {
  __shared__ __attribute__((aligned(16))) SmallStep desc[kSmallDescCache];
  __shared__ __attribute__((aligned(16))) float2 stage[kSmallStage];
  const int w = blockIdx.x, z = blockIdx.y;
  float2* IN = in + (int64_t)z * in_bs;
  float2* WS = ws + (int64_t)z * ws_bs;
  int win0 = -1, win1 = -1;  // steps whose descriptors are in LDS
  for (int lv = list_off[w]; lv < list_off[w + 1]; ++lv) {
    const int l0 = level_off[lv], l1 = level_off[lv + 1];
    for (int cb = l0; cb < l1; cb += kSmallDescCache) {
      const int ce = min(l1, cb + kSmallDescCache), ns = ce - cb;
      if (cb < win0 || ce > win1) {
        // load the descriptors of as many whole following levels as fit (at
        // least this chunk): one global round trip for several levels
        int end = ce;
        if (cb == l0 && l1 - l0 <= kSmallDescCache) {
          int nl = lv + 1;
          while (nl < list_off[w + 1] && level_off[nl + 1] - cb <= kSmallDescCache) ++nl;
          end = level_off[nl];
        }
        const int words = (end - cb) * (int)(sizeof(SmallStep) / 16);
        const uint4* src = reinterpret_cast<const uint4*>(steps + cb);
        uint4* dst = reinterpret_cast<uint4*>(desc);
        __syncthreads();  // the previous window is no longer read
        for (int i = threadIdx.x; i < words; i += kSmallThreads) dst[i] = src[i];
        win0 = cb;
        win1 = end;
        __syncthreads();
      }
      const SmallStep* desc_c = desc + (cb - win0);  // this chunk's descriptors
      // rounds (planned on the host): steps of the level whose operands fit in LDS together
      for (int r0 = 0; r0 < ns;) {
        const int r1 = desc_c[r0].round_end;
        const SmallStep& last = desc_c[r1 - 1];
        const int stage_end = last.stage_b + (1 << last.b_bits);
        // this thread's work items, fetched while the operands are staged
        const int it0 = desc_c[r0].item0, nit = desc_c[r0].n_items;
        const uint32_t my0 = (int)threadIdx.x < nit ? items[it0 + threadIdx.x] : 0u;
        const uint32_t my1 = (int)threadIdx.x + kSmallThreads < nit ? items[it0 + threadIdx.x + kSmallThreads] : 0u;
        // stage the operands: one flat loop over the round's operand elements,
        // every thread keeping kStageInFlight independent loads in flight
        for (int e0 = threadIdx.x; e0 < stage_end; e0 += kStageInFlight * kSmallThreads) {
          float2 v[kStageInFlight];
#pragma unroll
          for (int u = 0; u < kStageInFlight; ++u) {
            const int e = e0 + u * kSmallThreads;
            if (e >= stage_end) break;
            int lo = r0, hi = r1 - 1;  // the step owning staged element e
            while (lo < hi) {
              const int mid = (lo + hi + 1) >> 1;
              if (desc_c[mid].stage_a <= e) lo = mid; else hi = mid - 1;
            }
            const SmallStep& st = desc_c[lo];
            const bool is_a = e < st.stage_b;
            const float2* src = is_a ? (st.a_buf == BUF_IN ? IN : WS) + st.a_off + (e - st.stage_a)
                                     : (st.b_buf == BUF_IN ? IN : WS) + st.b_off + (e - st.stage_b);
            v[u] = *src;
          }
#pragma unroll
          for (int u = 0; u < kStageInFlight; ++u) {
            const int e = e0 + u * kSmallThreads;
            if (e >= stage_end) break;
            stage[e] = v[u];
          }
        }
        __syncthreads();
        // each item: the outputs j + t 2^qb of one step; the operand addresses
        // of the first come from the step's index maps (packed in registers),
        // the next ones by flipping the address bits of the output bits that change
        for (int q = 0; q < 2; ++q) {
          if ((int)threadIdx.x + q * kSmallThreads >= nit) break;
          const uint32_t wd = q == 0 ? my0 : my1;
          const SmallStep& st = desc_c[wd & 255u];
          const int o0 = (int)((wd >> 8) & 4095u), qb = (int)(wd >> 20), nt_ = 1 << (st.c_bits - qb);
          const uint32_t* ap = reinterpret_cast<const uint32_t*>(st.apos);
          const uint32_t* bp = reinterpret_cast<const uint32_t*>(st.bpos);
          const uint32_t* ka = reinterpret_cast<const uint32_t*>(st.ka);
          const uint32_t* kb = reinterpret_cast<const uint32_t*>(st.kb);
          const uint32_t ap0 = ap[0], ap1 = ap[1], ap2 = ap[2], bp0 = bp[0], bp1 = bp[1], bp2 = bp[2];
          const uint32_t ka0 = ka[0], ka1 = ka[1], ka2 = ka[2], kb0 = kb[0], kb1 = kb[1], kb2 = kb[2];
          const int nk = 1 << st.k_bits;
          const float2* As = stage + st.stage_a;
          const float2* Bs = stage + st.stage_b;
          float2* C = (st.c_buf == BUF_IN ? IN : WS) + st.c_off;
          int ab = 0, bb = 0;
          for (uint32_t m = (uint32_t)o0; m; m &= m - 1) {
            const int p = __builtin_ctz(m);
            const int pa = packed_byte(ap0, ap1, ap2, p), pb = packed_byte(bp0, bp1, bp2, p);
            if (pa >= 0) ab |= 1 << pa;
            if (pb >= 0) bb |= 1 << pb;
          }
          for (int t = 0; t < nt_; ++t) {
            const int o = o0 | (t << qb);
            if (t != 0)
              for (uint32_t f = (uint32_t)((t ^ (t - 1)) << qb); f; f &= f - 1) {
                const int p = __builtin_ctz(f);
                const int pa = packed_byte(ap0, ap1, ap2, p), pb = packed_byte(bp0, bp1, bp2, p);
                if (pa >= 0) ab ^= 1 << pa;
                if (pb >= 0) bb ^= 1 << pb;
              }
            // summed index in Gray-code order: one address bit flips per term
            int a = ab, b = bb;
            float2 acc = cmul<PREC>(As[a], Bs[b]);
            for (int k = 1; k < nk; ++k) {
              const int j = __builtin_ctz(k);
              a ^= 1 << packed_byte(ka0, ka1, ka2, j);
              b ^= 1 << packed_byte(kb0, kb1, kb2, j);
              acc = cmac<PREC>(acc, As[a], Bs[b]);
            }
            C[o] = acc;
          }
        }
        __syncthreads();
        r0 = r1;
      }
    }
  }
}

hipError_t launch_small_steps(hipStream_t s, const SmallStep* steps, const int32_t* list_off,
                              const int32_t* level_off, const uint32_t* items, int n_lists, float2* in,
                              int64_t in_bs, float2* ws, int64_t ws_bs, int batch, int precision) {
  if (n_lists == 0) return hipSuccess;
  if (precision == TN_PREC_BF16X3)
    hipLaunchKernelGGL(k_small_steps<TN_PREC_BF16X3>, dim3(n_lists, batch), dim3(kSmallThreads), 0, s, steps, list_off,
                       level_off, items, in, in_bs, ws, ws_bs);
  else
    hipLaunchKernelGGL(k_small_steps<TN_PREC_C64>, dim3(n_lists, batch), dim3(kSmallThreads), 0, s, steps, list_off,
                       level_off, items, in, in_bs, ws, ws_bs);
  return hipGetLastError();
}

// The interpreter for lists that stay in LDS: inputs are staged once, then a
// level is its items' arithmetic and a barrier.  A level is bound by its chain
// of LDS reads (descriptor, operands); items and their operand places are
// planned on the host and fetched a level ahead.  The arithmetic is
// k_small_steps', term by term.  (The 125 products of a 10-qubit state, 9
// levels: 38 us in k_small_steps, 13 so.)
struct ResArgs {
  float2* out;
  int64_t out_bs;
  int32_t final_list;
  int8_t out_pos[kSmallMaxBits];
};

template <int PREC>
__global__ __launch_bounds__(kSmallThreads) void k_small_resident(ResTables tb, const float2* in, int64_t in_bs,
                                                                  float2* ws, int64_t ws_bs, ResArgs fin) {
  __shared__ __attribute__((aligned(16))) float2 T[kResElems];
  __shared__ __attribute__((aligned(16))) ResStep desc[kResSteps];
  __shared__ ResLevel lev[kResLevels];
  const int w = blockIdx.x, z = blockIdx.y, tid = threadIdx.x;
  const ResList L = tb.lists[w];
  const float2* IN = in + (int64_t)z * in_bs;
  const ResItem* items = tb.items;
  const ResLevel l0 = tb.levels[L.level0];
  ResItem it0, it1, nx0 = {}, nx1 = {};
  if (tid < l0.n_items) nx0 = items[l0.item0 + tid];
  if (tid + kSmallThreads < l0.n_items) nx1 = items[l0.item0 + tid + kSmallThreads];
  for (int i = tid; i < L.n_levels; i += kSmallThreads) lev[i] = tb.levels[L.level0 + i];
  {
    const uint4* src = reinterpret_cast<const uint4*>(tb.steps + L.step0);
    uint4* dst = reinterpret_cast<uint4*>(desc);
    for (int i = tid; i < L.n_steps * (int)(sizeof(ResStep) / 16); i += kSmallThreads) dst[i] = src[i];
  }
  for (int e0 = tid; e0 < L.n_copy; e0 += 4 * kSmallThreads) {
    uint32_t from[4];
    float2 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (e0 + u * kSmallThreads < L.n_copy) from[u] = tb.copy[L.copy0 + e0 + u * kSmallThreads];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (e0 + u * kSmallThreads < L.n_copy) v[u] = IN[from[u]];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (e0 + u * kSmallThreads < L.n_copy) T[e0 + u * kSmallThreads] = v[u];
  }
  __syncthreads();
  const bool to_out = w == fin.final_list;
  float2* C = to_out ? fin.out + (int64_t)z * fin.out_bs : ws + (int64_t)z * ws_bs + L.c_off;
  for (int lv = 0; lv < L.n_levels; ++lv) {
    const int nit = lev[lv].n_items;
    it0 = nx0;
    it1 = nx1;
    if (lv + 1 < L.n_levels) {  // the next level's items
      const ResLevel n = lev[lv + 1];
      if (tid < n.n_items) nx0 = items[n.item0 + tid];
      if (tid + kSmallThreads < n.n_items) nx1 = items[n.item0 + tid + kSmallThreads];
    }
    for (int q = 0; q < 2; ++q) {
      if (tid + q * kSmallThreads >= nit) break;
      const ResItem it = q == 0 ? it0 : it1;
      const ResStep& st = desc[it.what & 255u];
      const int o0 = (int)((it.what >> 8) & 4095u), qb = (int)(it.what >> 20), nt = 1 << (st.c_bits - qb);
      const uint32_t* ap = reinterpret_cast<const uint32_t*>(st.apos);
      const uint32_t* bp = reinterpret_cast<const uint32_t*>(st.bpos);
      const uint32_t* ka = reinterpret_cast<const uint32_t*>(st.ka);
      const uint32_t* kb = reinterpret_cast<const uint32_t*>(st.kb);
      const uint32_t ap0 = ap[0], ap1 = ap[1], ap2 = ap[2], bp0 = bp[0], bp1 = bp[1], bp2 = bp[2];
      const uint32_t ka0 = ka[0], ka1 = ka[1], ka2 = ka[2], kb0 = kb[0], kb1 = kb[1], kb2 = kb[2];
      const int nk = 1 << st.k_bits, c = st.c;
      int ab = it.a, bb = it.b;  // (a tensor's place is a multiple of its size)
      for (int t = 0; t < nt; ++t) {
        const int o = o0 | (t << qb);
        if (t != 0)
          for (uint32_t f = (uint32_t)((t ^ (t - 1)) << qb); f; f &= f - 1) {
            const int p = __builtin_ctz(f);
            const int pa = packed_byte(ap0, ap1, ap2, p), pb = packed_byte(bp0, bp1, bp2, p);
            if (pa >= 0) ab ^= 1 << pa;
            if (pb >= 0) bb ^= 1 << pb;
          }
        // summed index in Gray-code order: one address bit flips per term
        int a = ab, b = bb;
        float2 acc = cmul<PREC>(T[a], T[b]);
        for (int k = 1; k < nk; ++k) {
          const int j = __builtin_ctz(k);
          a ^= 1 << packed_byte(ka0, ka1, ka2, j);
          b ^= 1 << packed_byte(kb0, kb1, kb2, j);
          acc = cmac<PREC>(acc, T[a], T[b]);
        }
        if (c != kResOut) {
          T[c + o] = acc;
        } else {
          int at = o;
          if (to_out) {
            at = 0;
#pragma unroll
            for (int j = 0; j < kSmallMaxBits; ++j) at |= ((o >> j) & 1) << fin.out_pos[j];
          }
          C[at] = acc;
        }
      }
    }
    __syncthreads();
  }
}

hipError_t launch_small_resident(hipStream_t s, const ResTables& t, int n_lists, const float2* in, int64_t in_bs,
                                 float2* ws, int64_t ws_bs, int final_list, float2* out, int64_t out_bs,
                                 const int8_t (&out_pos)[kSmallMaxBits], int batch, int precision) {
  if (n_lists == 0) return hipSuccess;
  ResArgs a;
  a.out = out;
  a.out_bs = out_bs;
  a.final_list = final_list;
  for (int j = 0; j < kSmallMaxBits; ++j) a.out_pos[j] = out_pos[j];
  const dim3 grid(n_lists, batch), block(kSmallThreads);
  if (precision == TN_PREC_BF16X3)
    hipLaunchKernelGGL(k_small_resident<TN_PREC_BF16X3>, grid, block, 0, s, t, in, in_bs, ws, ws_bs, a);
  else
    hipLaunchKernelGGL(k_small_resident<TN_PREC_C64>, grid, block, 0, s, t, in, in_bs, ws, ws_bs, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Index slicing: the input tensors of one slice gathered from the full ones,
// and the slices' results summed.
// ---------------------------------------------------------------------------
__global__ void k_slice_gather(const SliceTensor* ts, int nt, const float2* full, int64_t full_bs, float2* sl,
                               int64_t sl_bs, int64_t slice) {
  const int t = blockIdx.x, z = blockIdx.y;
  if (t >= nt) return;
  const SliceTensor st = ts[t];
  int64_t cut = 0;  // the fixed bits of this slice, at their places in the full tensor
  for (int k = 0; k < st.n_cut; ++k) cut |= ((slice >> st.cut_src[k]) & 1) << st.cut_pos[k];
  const float2* src = full + (int64_t)z * full_bs + st.src_off;
  float2* dst = sl + (int64_t)z * sl_bs + st.dst_off;
  const int64_t n = (int64_t)1 << st.n_keep;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
    int64_t a = cut;
    for (int j = 0; j < st.n_keep; ++j) a |= ((i >> j) & 1) << st.keep_pos[j];
    dst[i] = src[a];
  }
}

hipError_t launch_slice_gather(hipStream_t s, const SliceTensor* ts, int nt, const float2* full, int64_t full_bs,
                               float2* sl, int64_t sl_bs, int64_t slice, int batch) {
  if (nt == 0) return hipSuccess;
  hipLaunchKernelGGL(k_slice_gather, dim3(nt, batch), dim3(64), 0, s, ts, nt, full, full_bs, sl, sl_bs, slice);
  return hipGetLastError();
}

// acc = src (first) or acc += src
__global__ void k_accumulate(const float2* src, int64_t src_bs, float2* acc, int64_t acc_bs, int64_t n, int first) {
  const int z = blockIdx.y;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
    const float2 v = src[(int64_t)z * src_bs + i];
    float2& a = acc[(int64_t)z * acc_bs + i];
    a = first ? v : f2(a.x + v.x, a.y + v.y);
  }
}

hipError_t launch_accumulate(hipStream_t s, const float2* src, int64_t src_bs, float2* acc, int64_t acc_bs, int64_t n,
                             int first, int batch) {
  int64_t blocks = (n + kThreads - 1) / kThreads;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(k_accumulate, dim3((unsigned)std::max<int64_t>(blocks, 1), batch), dim3(kThreads), 0, s, src,
                     src_bs, acc, acc_bs, n, first);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Bit-permutation transpose through LDS
// ---------------------------------------------------------------------------
constexpr int kMaxTileBits = 10;

// (every map starts at a multiple of 4 bytes: deposit() reads them as 32-bit words)
struct PermArgs {
  const float2* in;
  float2* out;
  int64_t in_bs, out_bs;
  int64_t n_blocks;
  int32_t tile_bits, rest_bits;
  int8_t rest_in[64];
  int8_t rest_out[64];
  int8_t tin[kMaxTileBits + 2];   // input position of tile-index bit j (load order)
  int8_t tsrc[kMaxTileBits + 2];  // store order: bit j of the store index = load-index bit tsrc[j]
  int8_t tout[kMaxTileBits + 2];  // output position of store-index bit j
};
static_assert(offsetof(PermArgs, rest_in) % 4 == 0 && offsetof(PermArgs, tin) % 4 == 0 &&
                  offsetof(PermArgs, tsrc) % 4 == 0 && offsetof(PermArgs, tout) % 4 == 0,
              "position maps aligned to 32-bit words");

__global__ __launch_bounds__(kThreads) void k_permute(PermArgs a) {
  __shared__ float2 buf[(1 << kMaxTileBits) + (1 << (kMaxTileBits - 5))];
  const int z = blockIdx.y;
  const float2* in = a.in + (int64_t)z * a.in_bs;
  float2* out = a.out + (int64_t)z * a.out_bs;
  const int tile = 1 << a.tile_bits;
  constexpr int kPer = (1 << kMaxTileBits) / kThreads;
  int64_t in_off[kPer], out_off[kPer];
  int lds_src[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int l = threadIdx.x + e * kThreads;
    in_off[e] = deposit(l, a.tin, a.tile_bits);
    out_off[e] = deposit(l, a.tout, a.tile_bits);
    const int src = (int)deposit(l, a.tsrc, a.tile_bits);
    lds_src[e] = src + (src >> 5);
  }
  for (int64_t blk = blockIdx.x; blk < a.n_blocks; blk += gridDim.x) {
    const int64_t ib = deposit(blk, a.rest_in, a.rest_bits), ob = deposit(blk, a.rest_out, a.rest_bits);
    for (int e = 0; e < kPer; ++e) {
      const int l = threadIdx.x + e * kThreads;
      if (l < tile) buf[l + (l >> 5)] = in[ib | in_off[e]];
    }
    __syncthreads();
    for (int e = 0; e < kPer; ++e) {
      const int l = threadIdx.x + e * kThreads;
      if (l < tile) out[ob | out_off[e]] = buf[lds_src[e]];
    }
    __syncthreads();
  }
}

hipError_t launch_permute(hipStream_t s, const PermuteDesc& d, const float2* in, int64_t in_bs, float2* out,
                          int64_t out_bs, int batch) {
  const int R = d.bits;
  // tile: the low input bits plus the input bits that land on the low output bits,
  // grown while it fits in kMaxTileBits
  std::vector<int> best;
  for (int a = 1; a <= R; ++a) {
    std::vector<char> in_tile(R, 0);
    for (int p = 0; p < a; ++p) in_tile[p] = 1;
    for (int p = 0; p < R; ++p)
      if (d.dst[p] < a) in_tile[p] = 1;
    std::vector<int> t;
    for (int p = 0; p < R; ++p)
      if (in_tile[p]) t.push_back(p);
    if ((int)t.size() > kMaxTileBits) break;
    best = t;
  }
  PermArgs a;
  a.in = in; a.out = out; a.in_bs = in_bs; a.out_bs = out_bs;
  a.tile_bits = (int)best.size();
  for (int j = 0; j < a.tile_bits; ++j) a.tin[j] = (int8_t)best[j];
  // store order: tile bits by ascending output position
  std::vector<int> order(a.tile_bits);
  for (int j = 0; j < a.tile_bits; ++j) order[j] = j;
  std::sort(order.begin(), order.end(), [&](int x, int y) { return d.dst[best[x]] < d.dst[best[y]]; });
  for (int j = 0; j < a.tile_bits; ++j) {
    a.tsrc[j] = (int8_t)order[j];
    a.tout[j] = (int8_t)d.dst[best[order[j]]];
  }
  int nr = 0;
  for (int p = 0; p < R; ++p) {
    if (std::find(best.begin(), best.end(), p) != best.end()) continue;
    a.rest_in[nr] = (int8_t)p;
    a.rest_out[nr] = (int8_t)d.dst[p];
    ++nr;
  }
  a.rest_bits = nr;
  a.n_blocks = (int64_t)1 << nr;
  int64_t blocks = a.n_blocks;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_permute, dim3((unsigned)blocks, batch), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Complex GEMM on the FP32 matrix cores
//
// With complex64 stored as interleaved (re, im), A (M x K complex) is read as
// the real M x 2K matrix A_r, and B (K x N complex) is expanded on the fly
// into the real 2K x 2N matrix B' whose 2x2 block (k, n) is
// [[Re b, Im b], [-Im b, Re b]].  Then A_r B' is the interleaved real view of
// A B (4M form: 4 real multiply-adds per complex one).  One
// v_mfma_f32_32x32x2f32 consumes exactly one complex k: lanes 0-31 carry
// Re A / the first row of the block of B', lanes 32-63 Im A / the second row,
// and produces a 32 x 16 complex tile.
// ---------------------------------------------------------------------------
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kBK = kGemmBK;          // complex k per staged K tile
constexpr int kB3Row = 2 * kBK + 8;   // bf16 per LDS row of a split-precision K tile (16-byte pad)

// Operands and result are read and written through bit-deposit maps: the
// address of logical index x of an operand is the OR of x's bits moved to
// their positions in that operand's layout.  A tile's base address is the
// deposit of its (multiple-of-tile) origin; the offsets inside a tile come
// from small LDS tables, so no separate permute pass is needed.
struct GemmArgs {
  const float2* A;
  const float2* B;
  float2* C;
  int64_t a_bs, b_bs, c_bs;
  int64_t batch, M, N, K;
  int32_t nbb, nbm, nbn, nbk;
  int8_t a_b[kGemmMaxBits], a_m[kGemmMaxBits], a_k[kGemmMaxBits];
  int8_t b_b[kGemmMaxBits], b_k[kGemmMaxBits], b_n[kGemmMaxBits];
  int8_t c_b[kGemmMaxBits], c_m[kGemmMaxBits], c_n[kGemmMaxBits];
};

// The matrix-core tiles' view of a product.  Every size is a power of two.
constexpr int kTileBits = 12;
struct TileArgs {
  const float2* A;
  const float2* B;
  float2* C;
  int64_t a_bs, b_bs, c_bs;
  int64_t M, N, K;
  int64_t c_elems;  // elements of C per parameter vector (split-K partial stride)
  int32_t xcd;
  int32_t lg_tm, lg_tn, lg_band, lg_split, lg_batch;  // tile rows, tile columns, columns per band, ranges of K, batch groups
  // the bits of a block's result tile (64 x 64, or 64 x 32, at a time), ascending by their
  // address in C: address bit, place in LDS (linear over XOR), m (low byte) and n (high byte)
  int32_t st_pos[kTileBits], st_lds[kTileBits], st_mn[kTileBits];
  int32_t lines;   // a tile holds whole 128-byte lines of C (else several blocks write to a line, which may meet in L2)
  int32_t c_next;  // address bit of C between the rounds of a 128-row tile
  // address bits of a tile's rows of A, columns of B, and of the low 10 bits of k (a K tile's, then the tile's number)
  int32_t a_row[7], b_col[7], a_k[10], b_k[10];
  // which index bit each address bit of an operand is: source (1 the batch; A: 2 m, 3 k; B: 2 n, 3 k; C: 2 m, 3 n)
  // times 64, plus the bit
  uint8_t from_a[64], from_b[64], from_c[64];
};

// An address from its indices: lane p decides address bit p, and the wave's vote is the address.  (A loop over the
// index's bits waits for each four positions in turn; with those, and 64-bit divisions by the tile counts, the kernels'
// first load came after some 2000 scalar instructions: a launch of small products took 9.2 us, now 5.6; 8192 x 32768 x
// 16 for a 28-qubit state, 65536 blocks of one K tile, 700 us, now 490.)
__device__ __forceinline__ int64_t gather_bits(unsigned from, int64_t x1, int64_t x2, int64_t x3) {
  const unsigned src = from >> 6;
  const int64_t x = src == 1 ? x1 : src == 2 ? x2 : x3;
  return (int64_t)__ballot(src != 0 && ((x >> (from & 63)) & 1));
}

// the low n bits of x to the given places
template <int N>
__device__ __forceinline__ int64_t place_bits(int x, const int32_t* pos) {
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const uint64_t at = (uint64_t)1 << pos[j];
    const uint32_t on = 0u - ((unsigned)(x >> j) & 1u);
    lo |= on & (uint32_t)at;
    hi |= on & (uint32_t)(at >> 32);
  }
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Tile order of the matrix-product kernels.  The GPU hands consecutive
// workgroup ids to its eight XCDs in turn, and each XCD has its own L2.  With
// xcd set (the grid is a multiple of 8), workgroup h takes logical id
// (h mod 8) * (grid / 8) + h / 8, so each XCD runs one contiguous range of
// logical ids, in order.  Logical ids walk the tile grid in bands of
// 2^lg_band tile columns, n fastest inside a band: an XCD's range then covers a
// block of rows of one band, whose B column tiles stay in its L2 while the rows
// pass and whose A row tiles are used 2^lg_band times in a row.
struct TileCoord {
  int64_t tm, tn;
  uint32_t ks, gb, z;  // range of K, batch group, parameter vector
};

__device__ inline TileCoord tile_coord(const TileArgs& g) {
  uint32_t bid = blockIdx.x;
  if (g.xcd) bid = (bid & 7) * (gridDim.x >> 3) + (bid >> 3);
  const uint32_t r = bid & ((1u << (g.lg_tm + g.lg_tn)) - 1), rest = bid >> (g.lg_tm + g.lg_tn);
  const uint32_t band = r >> (g.lg_tm + g.lg_band), q = r & ((1u << (g.lg_tm + g.lg_band)) - 1);
  return {(int64_t)(q >> g.lg_band), (int64_t)((band << g.lg_band) + (q & ((1u << g.lg_band) - 1))),
          rest & ((1u << g.lg_split) - 1), (rest >> g.lg_split) & ((1u << g.lg_batch) - 1),
          rest >> (g.lg_split + g.lg_batch)};
}

// BF16x3 split precision: x_hi = bf16(x), x_lo = bf16(x - x_hi), both round
// to nearest even; the product keeps a_hi b_hi + a_hi b_lo + a_lo b_hi.
__device__ inline void split_bf16(float2 v, uint32_t* hi, uint32_t* lo) {
  const __bf16 h0 = (__bf16)v.x, h1 = (__bf16)v.y;
  const __bf16 l0 = (__bf16)(v.x - (float)h0), l1 = (__bf16)(v.y - (float)h1);
  const bf16x2 H = {h0, h1}, L = {l0, l1};
  *hi = __builtin_bit_cast(uint32_t, H);
  *lo = __builtin_bit_cast(uint32_t, L);
}

// (re, im) bf16 pairs of B -> the B' column entries of real column parity d:
// (re, -im) for even real columns, (im, re) for odd ones
__device__ inline bf16x8 b_embed(uint4 w, int d) {
  uint4 r;
  r.x = d ? ((w.x >> 16) | (w.x << 16)) : (w.x ^ 0x80000000u);
  r.y = d ? ((w.y >> 16) | (w.y << 16)) : (w.y ^ 0x80000000u);
  r.z = d ? ((w.z >> 16) | (w.z << 16)) : (w.z ^ 0x80000000u);
  r.w = d ? ((w.w >> 16) | (w.w << 16)) : (w.w ^ 0x80000000u);
  return __builtin_bit_cast(bf16x8, r);
}

// Result tiles go through LDS so that a wave stores along C's lowest address
// bits, whichever of m and n they are: a matrix-core result holds 32 columns
// of one row per half-wave, and stored from there a line of C is written in up
// to 16 pieces (complex64, 8 x 1024 x 1024 x 4 with C's bits alternating
// between m and n: 87 us, 30 through LDS; a line's pieces do not meet in L2
// again before they are written).  Element (r, c) of the 64 x 64 (64 x 32) elements
// is at place r BN + (c ^ reversed low bits of r): C's lowest five tile bits
// are the lowest a of n and b of m, so 32 lanes read 32 distinct bank pairs.
__host__ __device__ __forceinline__ int tile_place(int r, int c, int bn) {
  return r * bn + (c ^ ((r & 1) << 4 | (r & 2) << 2 | (r & 4) | (r & 8) >> 2 | (r & 16) >> 4));
}

// Elements of T (2^nb of them) to C: thread t and round e hold element e 256 + t
// in the order of the tile's bits; limits: m and n that exist beyond the tile's
// origin (whole: no guards).
template <int NB>
__device__ __forceinline__ void store_tile(const TileArgs& g, const float2* T, float2* C, bool whole, int64_t m_left,
                                           int64_t n_left) {
  const int t = threadIdx.x;
  const int64_t at = place_bits<8>(t, g.st_pos);
  int lt = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) lt ^= (0 - ((t >> j) & 1)) & g.st_lds[j];
  constexpr int kRounds = 1 << (NB - 8);
  int64_t ae[kRounds];
  int le[kRounds];
  float2 v[kRounds];
  ae[0] = 0;
  le[0] = 0;
#pragma unroll
  for (int e = 1; e < kRounds; ++e) {
    const int j = 8 + __builtin_ctz(e), e1 = e & (e - 1);
    ae[e] = ae[e1] | (int64_t)1 << g.st_pos[j];
    le[e] = le[e1] ^ g.st_lds[j];
  }
#pragma unroll
  for (int e = 0; e < kRounds; ++e) v[e] = T[lt ^ le[e]];
  if (whole && g.lines) {
#pragma unroll
    for (int e = 0; e < kRounds; ++e) store_stream(C + ae[e] + at, v[e].x, v[e].y);
    return;
  }
  int mt = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) mt |= (0 - ((t >> j) & 1)) & g.st_mn[j];
#pragma unroll
  for (int e = 0; e < kRounds; ++e) {
    int mn = mt;
#pragma unroll
    for (int j = 8; j < NB; ++j) mn |= (e >> (j - 8)) & 1 ? g.st_mn[j] : 0;
    if ((mn & 255) < m_left && (mn >> 8) < n_left) C[ae[e] + at] = v[e];
  }
}

// Complex GEMM on the matrix cores.
//
// With complex64 stored as interleaved (re, im), A (M x K complex) is read as
// the real M x 2K matrix A_r, and B (K x N complex) is expanded on the fly
// into the real 2K x 2N matrix B' whose 2x2 block (k, n) is
// [[Re b, Im b], [-Im b, Re b]].  Then A_r B' is the interleaved real view of
// A B (4M form: 4 real multiply-adds per complex one).
//
// Four waves in a 2 x 2 arrangement; each wave owns TM x TN result tiles of
// 32 x 16 complex, so a block computes (64 TM) x (32 TN).  Form F = 0: FP32,
// one v_mfma_f32_32x32x2f32 per complex k (lanes 0-31 carry Re A / the first
// row of B's 2x2 block, lanes 32-63 Im A / the second row).  Form F = 1:
// BF16x3 on the bf16 matrix cores, v_mfma_f32_32x32x16_bf16 covering 8
// complex k: lane l holds the eight consecutive k' = 8*(l/32) .. +7 of row
// (A) or column (B) l%32, i.e. four complex values of one A row as stored,
// or four complex values of one B column turned into B' entries (b_embed).
// Operands are split into hi/lo once, while a tile is staged into LDS.
template <int AK, int BNF, int TM, int TN, int F>
__global__ __launch_bounds__(kThreads) void k_gemm(TileArgs g) {
  constexpr int BM = 64 * TM, BN = 32 * TN;
  constexpr int kPA = (BM * kBK) / kThreads, kPB = (BN * kBK) / kThreads;
  constexpr int kF32Bytes = 2 * kBK * (BM + 1) * 4 + kBK * (BN + 1) * 8;
  constexpr int kB3Bytes = 2 * BM * kB3Row * 2 + 2 * BN * kB3Row * 2;
  constexpr int kSmem = std::max(F == 0 ? kF32Bytes : kB3Bytes, 64 * BN * 8);
  __shared__ __attribute__((aligned(16))) char smem[kSmem];
  constexpr int kKt = 64;  // K tiles whose origin deposits are tabulated (the rest computed on the fly)
  __shared__ int64_t TAt[kKt], TBt[kKt];
  float (*As_re)[BM + 1] = reinterpret_cast<float (*)[BM + 1]>(smem);
  float (*As_im)[BM + 1] = reinterpret_cast<float (*)[BM + 1]>(smem + kBK * (BM + 1) * 4);
  float2 (*Bs)[BN + 1] = reinterpret_cast<float2 (*)[BN + 1]>(smem + 2 * kBK * (BM + 1) * 4);
  __bf16 (*Ah)[kB3Row] = reinterpret_cast<__bf16 (*)[kB3Row]>(smem);
  __bf16 (*Al)[kB3Row] = reinterpret_cast<__bf16 (*)[kB3Row]>(smem + BM * kB3Row * 2);
  __bf16 (*Bh)[kB3Row] = reinterpret_cast<__bf16 (*)[kB3Row]>(smem + 2 * BM * kB3Row * 2);
  __bf16 (*Bl)[kB3Row] = reinterpret_cast<__bf16 (*)[kB3Row]>(smem + 2 * BM * kB3Row * 2 + BN * kB3Row * 2);

  const TileCoord tc = tile_coord(g);
  const int64_t tn = tc.tn, tm = tc.tm;
  const int64_t ks = tc.ks, z = tc.z;
  const int64_t gb = tc.gb;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const unsigned from_a = g.from_a[lane], from_b = g.from_b[lane], from_c = g.from_c[lane];
  const float2* A = g.A + z * g.a_bs;
  const float2* B = g.B + z * g.b_bs;
  float2* C = g.C + z * g.c_bs + ks * g.c_elems;
  const int64_t m0 = tm * BM, n0 = tn * BN;
  const int64_t kchunk = g.K >> g.lg_split;
  const int64_t kbeg = ks * kchunk, kend = kbeg + kchunk;
  const int wm = w >> 1, wn = w & 1;
  const int64_t base_a = gather_bits(from_a, gb, m0, 0);
  const int64_t base_b = gather_bits(from_b, gb, n0, 0);
  const int64_t base_c = gather_bits(from_c, gb, m0, n0);
  const int64_t beg_a = gather_bits(from_a, 0, 0, kbeg), beg_b = gather_bits(from_b, 0, 0, kbeg);
  if (tid < kKt) {
    TAt[tid] = beg_a | place_bits<6>(tid, g.a_k + 4);
    TBt[tid] = beg_b | place_bits<6>(tid, g.b_k + 4);
  }
  constexpr int kLogBN = 5 + (TN == 2);
  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  __syncthreads();

  // tile element e of this thread: (row or column, k) inside the tile
  auto a_elem = [&](int e, int& mm, int& kk) {
    const int idx = tid + e * kThreads;
    if (AK) { mm = idx / kBK; kk = idx % kBK; } else { mm = idx % BM; kk = idx / BM; }
  };
  auto b_elem = [&](int e, int& nn, int& kk) {
    const int idx = tid + e * kThreads;
    if (BNF) { nn = idx % BN; kk = idx / BN; } else { nn = idx / kBK; kk = idx % kBK; }
  };
  // software pipeline: the next K tile is fetched into registers while the
  // current one is multiplied out of LDS
  // per-thread element addresses without the K tile's origin, fixed for the block
  const float2* pa[kPA];
  const float2* pb[kPB];
  bool va[kPA], vb[kPB];
  int ka_e[kPA], kb_e[kPB];
  int a_m0, a_k0, b_n0, b_k0;  // element 0's; the others' differ by bits of their own
  a_elem(0, a_m0, a_k0);
  b_elem(0, b_n0, b_k0);
  const int64_t at_a = base_a | place_bits<7>(a_m0, g.a_row) | place_bits<4>(a_k0, g.a_k);
  const int64_t at_b = base_b | place_bits<6>(b_n0, g.b_col) | place_bits<4>(b_k0, g.b_k);
#pragma unroll
  for (int e = 0; e < kPA; ++e) {
    int mm, kk;
    a_elem(e, mm, kk);
    pa[e] = A + (at_a | place_bits<7>(mm ^ a_m0, g.a_row) | place_bits<4>(kk ^ a_k0, g.a_k));
    va[e] = m0 + mm < g.M;
    ka_e[e] = kk;
  }
#pragma unroll
  for (int e = 0; e < kPB; ++e) {
    int nn, kk;
    b_elem(e, nn, kk);
    pb[e] = B + (at_b | place_bits<6>(nn ^ b_n0, g.b_col) | place_bits<4>(kk ^ b_k0, g.b_k));
    vb[e] = n0 + nn < g.N;
    kb_e[e] = kk;
  }
  const bool interior = m0 + BM <= g.M && n0 + BN <= g.N;
  float2 ra[kPA], rb[kPB];
  auto fetch = [&](int64_t k0) {
    const int64_t t = (k0 - kbeg) / kBK;
    const int64_t ka = t < kKt ? TAt[t] : gather_bits(from_a, 0, 0, k0);
    const int64_t kb = t < kKt ? TBt[t] : gather_bits(from_b, 0, 0, k0);
    const int64_t rem = kend - k0;
    const int kleft = rem < kBK ? (int)rem : kBK;  // valid k of this tile
    if (interior && kleft == kBK) {  // whole tile inside the operands: no guards
#pragma unroll
      for (int e = 0; e < kPA; ++e) ra[e] = pa[e][ka];
#pragma unroll
      for (int e = 0; e < kPB; ++e) rb[e] = pb[e][kb];
    } else {
#pragma unroll
      for (int e = 0; e < kPA; ++e) ra[e] = (va[e] && ka_e[e] < kleft) ? pa[e][ka] : f2(0.f, 0.f);
#pragma unroll
      for (int e = 0; e < kPB; ++e) rb[e] = (vb[e] && kb_e[e] < kleft) ? pb[e][kb] : f2(0.f, 0.f);
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int e = 0; e < kPA; ++e) {
      int mm, kk;
      a_elem(e, mm, kk);
      if constexpr (F == 0) {
        As_re[kk][mm] = ra[e].x;
        As_im[kk][mm] = ra[e].y;
      } else {
        uint32_t h, l;
        split_bf16(ra[e], &h, &l);
        *reinterpret_cast<uint32_t*>(&Ah[mm][2 * kk]) = h;
        *reinterpret_cast<uint32_t*>(&Al[mm][2 * kk]) = l;
      }
    }
#pragma unroll
    for (int e = 0; e < kPB; ++e) {
      int nn, kk;
      b_elem(e, nn, kk);
      if constexpr (F == 0) {
        Bs[kk][nn] = rb[e];
      } else {
        uint32_t h, l;
        split_bf16(rb[e], &h, &l);
        *reinterpret_cast<uint32_t*>(&Bh[nn][2 * kk]) = h;
        *reinterpret_cast<uint32_t*>(&Bl[nn][2 * kk]) = l;
      }
    }
  };
  fetch(kbeg);
  for (int64_t k0 = kbeg; k0 < kend; k0 += kBK) {
    stage();
    __syncthreads();
    if (k0 + kBK < kend) fetch(k0 + kBK);
    if constexpr (F == 0) {
#pragma unroll 4
      for (int kk = 0; kk < kBK; ++kk) {
        float av[TM], bv[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int row = wm * 32 * TM + i * 32 + (lane & 31);
          av[i] = lane < 32 ? As_re[kk][row] : As_im[kk][row];
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const float2 bb = Bs[kk][wn * 16 * TN + j * 16 + ((lane & 31) >> 1)];
          const bool odd = lane & 1;
          bv[j] = lane < 32 ? (odd ? bb.y : bb.x) : (odd ? bb.x : -bb.y);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], acc[i][j], 0, 0, 0);
      }
    } else {
      const int half = lane >> 5, d = lane & 1;
#pragma unroll
      for (int kq = 0; kq < kBK / 8; ++kq) {
        const int col = kq * 16 + half * 8;  // first bf16 of this lane's eight
        bf16x8 ah[TM], al[TM], bh[TN], bl[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int row = wm * 32 * TM + i * 32 + (lane & 31);
          ah[i] = *reinterpret_cast<const bf16x8*>(&Ah[row][col]);
          al[i] = *reinterpret_cast<const bf16x8*>(&Al[row][col]);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int nn = wn * 16 * TN + j * 16 + ((lane & 31) >> 1);
          bh[j] = b_embed(*reinterpret_cast<const uint4*>(&Bh[nn][col]), d);
          bl[j] = b_embed(*reinterpret_cast<const uint4*>(&Bl[nn][col]), d);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  const bool whole = m0 + BM <= g.M && n0 + BN <= g.N;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if (i > 0) __syncthreads();
    const int own = tile_place(wm * 32 + 4 * (lane >> 5), wn * 16 * TN + ((lane & 31) >> 1), BN);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        reinterpret_cast<float*>(smem)[2 * (own ^ tile_place(8 * (v >> 2) + (v & 3), j * 16, BN)) + (lane & 1)] =
            acc[i][j][v];
    __syncthreads();
    store_tile<6 + kLogBN>(g, reinterpret_cast<const float2*>(smem), C + (base_c | (i ? (int64_t)1 << g.c_next : 0)),
                           whole, g.M - m0 - 32 * i, g.N - n0);
  }
}

// 3M form on the FP32 matrix cores: with A = Ar + i Ai and B = Br + i Bi,
//   Re C = Ar Br - Ai Bi,   Im C = (Ar + Ai)(Br + Bi) - Ar Br - Ai Bi,
// three real products instead of the four of the real embedding.  Operands
// are staged as interleaved complex and split into real and imaginary parts
// as a lane reads them; one v_mfma_f32_32x32x2f32 takes
// two complex k (lanes 0-31 the first, 32-63 the second) and a 32 x 32
// complex tile keeps three accumulators (P1 = Ar Br, P2 = Ai Bi,
// P3 = (Ar + Ai)(Br + Bi)).  Four waves in a 2 x 2 arrangement, each owning
// TM tiles of 32 x 32 complex: the block computes (64 TM) x 64.
//
// FOUR = 1: the same staging with the four real products of the real embedding
// (two accumulators), whose error the imaginary part's differences do not
// enlarge (4096 products of 32 x 32 x 32: 1.44e-7 against 1.55e-7, and where
// imaginary parts are 2^-12 of the real ones, theirs 2^12 times as good).  It is
// the 64 x 64 tile of 4M and both packed tiles: 4 x 1024 x 512 x 256 43.2 us
// (35.5 in 3M), the 4096 products 25.2 (23.1).
template <int AK, int BNF, int TM, int BK, int NW, int BP, int FOUR>
__global__ __launch_bounds__(kThreads, TM == 1 && !BP ? 4 : 2) void k_gemm3m(TileArgs g) {
  // BP = 1 (batch-packed): four batch items of at most 32 x 32 per block, wave
  // w computing item w; operand "rows" are (item, m) for A and (item, n) for
  // B.  BP = 2 (column-packed): M <= 32 and four 32-column slices of N per
  // block, wave w computing slice w; A's rows repeat per slice, B's rows are
  // n - n0.
  static_assert(!BP || TM == 1, "packed blocks hold one 32 x 32 tile per wave");
  constexpr int BM = BP ? 128 : 64 * TM, BN = BP ? 128 : 64;
  constexpr int kPA = (BM * BK) / kThreads, kPB = (BN * BK) / kThreads;
  constexpr int kLogBK = BK == 32 ? 5 : 4;
  // operands staged as interleaved complex with k contiguous per row of A and
  // per column of B, rows kRow = 2 BK + 4 words apart: a lane reads four
  // consecutive complex k of its row as two 16-byte loads, and 16 consecutive
  // rows start on distinct multiples of 4 banks (36 r mod 64)
  static_assert(BK % 8 == 0, "whole 16-byte operand reads");
  constexpr int kRow = 2 * BK + 4;
  constexpr int kStage = (BM + BN) * kRow, kTile = 64 * 64 * 2;
  __shared__ __attribute__((aligned(16))) float smem[kStage > kTile ? kStage : kTile];
  float* const As = smem;
  float* const Bs = smem + BM * kRow;
  constexpr int kKt = 64;  // K tiles whose origin deposits are tabulated (the rest computed on the fly)
  __shared__ int64_t TAt[kKt], TBt[kKt];
  const TileCoord tc = tile_coord(g);
  const int64_t tn = tc.tn, tm = tc.tm;
  const int64_t ks = tc.ks, z = tc.z;
  const int64_t gb = (int64_t)tc.gb << (BP == 1 ? 2 : 0);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const unsigned from_a = g.from_a[lane], from_b = g.from_b[lane], from_c = g.from_c[lane];
  const float2* A = g.A + z * g.a_bs;
  const float2* B = g.B + z * g.b_bs;
  float2* C = g.C + z * g.c_bs + ks * g.c_elems;
  const int64_t m0 = tm * BM, n0 = tn * BN;
  const int64_t kchunk = g.K >> g.lg_split;
  const int64_t kbeg = ks * kchunk, kend = kbeg + kchunk;
  const int wm = w >> 1, wn = w & 1;
  const int64_t base_a = gather_bits(from_a, gb, m0, 0);
  const int64_t base_b = gather_bits(from_b, gb, n0, 0);
  const int64_t base_c = gather_bits(from_c, gb, m0, n0);
  const int64_t beg_a = gather_bits(from_a, 0, 0, kbeg), beg_b = gather_bits(from_b, 0, 0, kbeg);
  if (tid < kKt) {
    TAt[tid] = beg_a | place_bits<6>(tid, g.a_k + 4);
    TBt[tid] = beg_b | place_bits<6>(tid, g.b_k + 4);
  }
  floatx16 p1[TM], p2[TM], p3[FOUR ? 1 : TM];  // FOUR: real and imaginary part in p1 and p2
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      p1[i][v] = p2[i][v] = 0.f;
      if constexpr (!FOUR) p3[i][v] = 0.f;
    }
  __syncthreads();

  // Staging order (16-wide K tiles, four waves), element e of a thread at row
  // rt + row_e(e), complex k kt + k_e(e) of its operand tile:
  //  - k fastest in the operand: a quarter-wave loads 16 consecutive k of one
  //    row (a 128-byte run) and writes them as 8-byte words; the two rows of
  //    a half-wave are 8 apart (36 * 8 = 32 mod 64 banks), so its 64 words
  //    fall on distinct banks;
  //  - m or n fastest: a wave loads 64 consecutive rows at one k per load and
  //    each thread writes its four consecutive k of a row as two 16-byte
  //    words (16 consecutive rows per LDS cycle, distinct banks).
  static_assert(BK == 16 && kThreads == 256 && (BN == 64 || BN == 128), "staging order assumes 16-wide K tiles");
  auto slot_t = [&](bool k_fast, int& r, int& kk) {
    if (k_fast) {
      r = w + 4 * ((lane >> 5) & 1) + 8 * ((lane >> 4) & 1);
      kk = lane & 15;
    } else {
      r = lane;
      kk = 4 * w;
    }
  };
  auto row_e = [](bool k_fast, int e) { return k_fast ? 16 * e : 64 * (e >> 2); };
  auto k_e = [](bool k_fast, int e) { return k_fast ? 0 : (e & 3); };
  constexpr bool kfa = AK != 0, kfb = BNF == 0;
  int a_rt, a_kt, b_rt, b_kt;
  slot_t(kfa, a_rt, a_kt);
  slot_t(kfb, b_rt, b_kt);
  // element offsets within a K tile, without the tile's origin: 32-bit byte
  // offsets from a block-uniform base when every offset of the tile stays
  // below 2^32 bytes (NW), else full pointers
  const float2* pa[NW ? 1 : kPA];
  const float2* pb[NW ? 1 : kPB];
  uint32_t oa[NW ? kPA : 1], ob[NW ? kPB : 1];
  // (column-packed: A's rows repeat per slice)
  const int64_t thr_a = place_bits<7>(BP == 2 ? a_rt & 31 : a_rt, g.a_row) | place_bits<4>(a_kt, g.a_k);
  const int64_t thr_b = place_bits<7>(b_rt, g.b_col) | place_bits<4>(b_kt, g.b_k);
#pragma unroll
  for (int e = 0; e < kPA; ++e) {
    const int re = row_e(kfa, e);
    const int64_t off = thr_a | place_bits<7>(BP == 2 ? re & 31 : re, g.a_row) | place_bits<4>(k_e(kfa, e), g.a_k);
    if constexpr (NW) oa[e] = (uint32_t)off * (uint32_t)sizeof(float2);
    else pa[e] = A + (base_a | off);
  }
#pragma unroll
  for (int e = 0; e < kPB; ++e) {
    const int64_t off = thr_b | place_bits<7>(row_e(kfb, e), g.b_col) | place_bits<4>(k_e(kfb, e), g.b_k);
    if constexpr (NW) ob[e] = (uint32_t)off * (uint32_t)sizeof(float2);
    else pb[e] = B + (base_b | off);
  }
  const bool interior = BP == 1   ? g.M == 32 && g.N == 32
                        : BP == 2 ? g.M == 32 && n0 + BN <= g.N
                                  : m0 + BM <= g.M && n0 + BN <= g.N;
  // whether tile row r of A (of B) lies inside the operand
  auto a_in = [&](int r) { return BP ? (r & 31) < g.M : m0 + r < g.M; };
  auto b_in = [&](int r) { return BP == 1 ? (r & 31) < g.N : n0 + r < g.N; };
  float2 ra[kPA], rb[kPB];
  auto fetch = [&](int64_t k0) {
    const int64_t t = (k0 - kbeg) / BK;
    int64_t ka = t < kKt ? TAt[t] : gather_bits(from_a, 0, 0, k0);
    int64_t kb = t < kKt ? TBt[t] : gather_bits(from_b, 0, 0, k0);
    // the same value in every lane: keep it in scalar registers
    ka = ((int64_t)__builtin_amdgcn_readfirstlane((int)(ka >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)ka);
    kb = ((int64_t)__builtin_amdgcn_readfirstlane((int)(kb >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)kb);
    const char* a_org = reinterpret_cast<const char*>(A + (base_a | ka));
    const char* b_org = reinterpret_cast<const char*>(B + (base_b | kb));
    auto lda = [&](int e) -> float2 {
      if constexpr (NW) return *reinterpret_cast<const float2*>(a_org + oa[e]);
      else return pa[e][ka];
    };
    auto ldb = [&](int e) -> float2 {
      if constexpr (NW) return *reinterpret_cast<const float2*>(b_org + ob[e]);
      else return pb[e][kb];
    };
    const int64_t rem = kend - k0;
    const int kleft = rem < BK ? (int)rem : BK;  // valid k of this tile
    if (interior && kleft == BK) {  // whole tile inside the operands: no guards
#pragma unroll
      for (int e = 0; e < kPA; ++e) ra[e] = lda(e);
#pragma unroll
      for (int e = 0; e < kPB; ++e) rb[e] = ldb(e);
    } else {
#pragma unroll
      for (int e = 0; e < kPA; ++e)
        ra[e] = (a_in(a_rt + row_e(kfa, e)) && a_kt + k_e(kfa, e) < kleft) ? lda(e) : f2(0.f, 0.f);
#pragma unroll
      for (int e = 0; e < kPB; ++e)
        rb[e] = (b_in(b_rt + row_e(kfb, e)) && b_kt + k_e(kfb, e) < kleft) ? ldb(e) : f2(0.f, 0.f);
    }
  };
  float* const as_t = As + a_rt * kRow + 2 * a_kt;
  float* const bs_t = Bs + b_rt * kRow + 2 * b_kt;
  auto put = [&](float* dst, bool k_fast, const float2* r, int n) {
    if (k_fast) {
#pragma unroll
      for (int e = 0; e < n; ++e) *reinterpret_cast<float2*>(dst + row_e(true, e) * kRow) = r[e];
    } else {
#pragma unroll
      for (int e = 0; e < n; e += 4) {
        float* d = dst + row_e(false, e) * kRow;
        *reinterpret_cast<float4*>(d) = make_float4(r[e].x, r[e].y, r[e + 1].x, r[e + 1].y);
        *reinterpret_cast<float4*>(d + 4) = make_float4(r[e + 2].x, r[e + 2].y, r[e + 3].x, r[e + 3].y);
      }
    }
  };
  auto stage = [&]() {
    put(as_t, kfa, ra, kPA);
    put(bs_t, kfb, rb, kPB);
  };
  const int h = lane >> 5, r32 = lane & 31;
  const int col = BP ? 32 * w + r32 : wn * 32 + r32;
  fetch(kbeg);
  for (int64_t k0 = kbeg; k0 < kend; k0 += BK) {
    stage();
    __syncthreads();
    if (k0 + BK < kend) fetch(k0 + BK);
    // MFMA step s takes k = s on lanes 0-31 and k = BK/2 + s on lanes 32-63
    // (the same order for A and B), so a lane's operands for the whole tile are
    // the BK/2 contiguous k values of its row or column starting at h BK/2
    constexpr int kHalf = BK / 2;
#pragma unroll
    for (int hh = 0; hh < kHalf / 4; ++hh) {  // groups of four steps: four k values per lane and plane
      const int kw = 2 * (kHalf * h + 4 * hh);  // word offset of the lane's four complex k
      const float4 b0 = *reinterpret_cast<const float4*>(&Bs[col * kRow + kw]);
      const float4 b1 = *reinterpret_cast<const float4*>(&Bs[col * kRow + kw + 4]);
      const float br[4] = {b0.x, b0.z, b1.x, b1.z}, bi[4] = {b0.y, b0.w, b1.y, b1.w};
      float ar[TM][4], ai[TM][4];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = BP ? 32 * w + r32 : wm * 32 * TM + i * 32 + r32;
        const float4 a0 = *reinterpret_cast<const float4*>(&As[row * kRow + kw]);
        const float4 a1 = *reinterpret_cast<const float4*>(&As[row * kRow + kw + 4]);
        ar[i][0] = a0.x; ar[i][1] = a0.z; ar[i][2] = a1.x; ar[i][3] = a1.z;
        ai[i][0] = a0.y; ai[i][1] = a0.w; ai[i][2] = a1.y; ai[i][3] = a1.w;
      }
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        const float bs = FOUR ? -bi[st] : br[st] + bi[st];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          if constexpr (FOUR) {
            p1[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar[i][st], br[st], p1[i], 0, 0, 0);
            p2[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar[i][st], bi[st], p2[i], 0, 0, 0);
            p1[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(ai[i][st], bs, p1[i], 0, 0, 0);
            p2[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(ai[i][st], br[st], p2[i], 0, 0, 0);
            continue;
          }
          p1[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar[i][st], br[st], p1[i], 0, 0, 0);
          p2[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(ai[i][st], bi[st], p2[i], 0, 0, 0);
          if constexpr (!FOUR)
            p3[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar[i][st] + ai[i][st], bs, p3[i], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if (i > 0) __syncthreads();
    const int own = tile_place(wm * 32 + 4 * h, wn * 32 + r32, 64);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float a = p1[i][v], b = p2[i][v];
      float2 c = f2(a, b);
      if constexpr (!FOUR) c = f2(a - b, p3[i][v] - a - b);
      reinterpret_cast<float2*>(smem)[own ^ tile_place(8 * (v >> 2) + (v & 3), 0, 64)] = c;
    }
    __syncthreads();
    store_tile<12>(g, reinterpret_cast<const float2*>(smem), C + (base_c | (i ? (int64_t)1 << g.c_next : 0)), interior,
                   g.M - m0 - 32 * i, BP == 1 ? g.N : g.N - n0);
  }
}

// Products too narrow for the matrix-core tiles (M < 64 or N < 32, e.g. a
// 4096-way batch of 2x2 outer products): one thread per output element, the
// same deposit-map addressing, K loop on the vector ALUs.
template <int PREC>
__global__ __launch_bounds__(kThreads) void k_contract_elem(GemmArgs g) {
  __shared__ int64_t TKa[kElemMaxK], TKb[kElemMaxK];
  const int z = blockIdx.y;
  const float2* A = g.A + (int64_t)z * g.a_bs;
  const float2* B = g.B + (int64_t)z * g.b_bs;
  float2* C = g.C + (int64_t)z * g.c_bs;
  const int K = (int)g.K;
  for (int k = threadIdx.x; k < K; k += kThreads) {
    TKa[k] = deposit(k, g.a_k, g.nbk);
    TKb[k] = deposit(k, g.b_k, g.nbk);
  }
  __syncthreads();
  const int64_t total = g.batch * g.M * g.N;
  for (int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x; o < total; o += (int64_t)gridDim.x * kThreads) {
    const int64_t n = o & (g.N - 1);
    const int64_t m = (o >> g.nbn) & (g.M - 1);
    const int64_t b = o >> (g.nbn + g.nbm);
    const int64_t db_a = deposit(b, g.a_b, g.nbb), db_b = deposit(b, g.b_b, g.nbb);
    const int64_t ab = db_a | deposit(m, g.a_m, g.nbm);
    const int64_t bb = db_b | deposit(n, g.b_n, g.nbn);
    float2 acc = f2(0.f, 0.f);
    int k = 0;
    // eight operand pairs in flight at a time (the loads do not wait on the sum)
    for (; k + 8 <= K; k += 8) {
      float2 av[8], bv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        av[u] = A[ab | TKa[k + u]];
        bv[u] = B[bb | TKb[k + u]];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) acc = cmac<PREC>(acc, av[u], bv[u]);
    }
    for (; k < K; ++k) acc = cmac<PREC>(acc, A[ab | TKa[k]], B[bb | TKb[k]]);
    C[deposit(b, g.c_b, g.nbb) | deposit(m, g.c_m, g.nbm) | deposit(n, g.c_n, g.nbn)] = acc;
  }
}

constexpr int kElemChunks = (kElemGroupOutBits + 5) / 6;

// A grouped member with long sums: thread t takes result o = t >> lane_bits
// and the terms k = s, s + L, s + 2L, ... (s = t mod L, L = 2^lane_bits); the
// L lanes of a result are adjacent lanes of one wave, leave the loop together
// (2^(out_bits + lane_bits) is a multiple of L) and combine their partial sums
// with cross-lane adds.
template <int PREC>
__device__ void elem_sum_lanes(const ElemMember& e, const int64_t* TO, const int64_t* TKa, const int64_t* TKb,
                               const float2* A, const float2* B, float2* C, int blk, int nblk) {
  const int lb = e.lane_bits, L = 1 << lb, s = threadIdx.x & (L - 1);
  const int KL = (1 << e.k_bits) >> lb;  // terms per lane, at least 4
  const int n_thr = 1 << (e.out_bits + lb);
  for (int t = blk * kThreads + threadIdx.x; t < n_thr; t += nblk * kThreads) {
    const int o = t >> lb;
    int64_t ab = 0, bb = 0, cc = 0;
#pragma unroll
    for (int ch = 0; ch < kElemChunks; ++ch) {
      const int i = ch * 64 + ((o >> (6 * ch)) & 63);
      ab |= TO[i];
      bb |= TO[kElemChunks * 64 + i];
      cc |= TO[2 * kElemChunks * 64 + i];
    }
    float2 acc = f2(0.f, 0.f);
    for (int j = 0; j < KL; j += 4) {  // four operand pairs in flight at a time
      float2 av[4], bv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = s + ((j + u) << lb);
        av[u] = A[ab | TKa[k]];
        bv[u] = B[bb | TKb[k]];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = cmac<PREC>(acc, av[u], bv[u]);
    }
    for (int off = L >> 1; off > 0; off >>= 1) {
      acc.x += __shfl_xor(acc.x, off);
      acc.y += __shfl_xor(acc.y, off);
    }
    if (s == 0) C[cc] = acc;
  }
}

// Grouped form of the per-output products: every member's address maps are
// turned into LDS tables (four 6-bit chunks of the result index, one table of
// summed offsets per operand), so an output costs twelve table reads before
// its sum.
static_assert(offsetof(ElemMember, bo) == offsetof(ElemMember, ao) + kElemGroupOutBits &&
                  offsetof(ElemMember, co) == offsetof(ElemMember, bo) + kElemGroupOutBits &&
                  offsetof(ElemMember, ak) == offsetof(ElemMember, co) + kElemGroupOutBits &&
                  offsetof(ElemMember, bk) == offsetof(ElemMember, ak) + kElemKBits,
              "the position maps of a member are consecutive bytes");

template <int PREC>
__global__ __launch_bounds__(kThreads) void k_elem_group(ElemGroupArgs g) {
  __shared__ int64_t TO[3 * kElemChunks * 64];  // [operand A, B, C][chunk][chunk value]
  __shared__ int64_t TKa[kElemMaxK], TKb[kElemMaxK];
  const int bx = blockIdx.x, z = blockIdx.y;
  int mi = 0;
  for (int i = 1; i < g.n; ++i)
    if (bx >= g.m[i].block0) mi = i;
  const ElemMember& e = g.m[mi];
  const int nblk = (mi + 1 < g.n ? g.m[mi + 1].block0 : g.total_blocks) - e.block0;
  const int ob = e.out_bits, kb = e.k_bits;
  // the member's position maps (ao, bo, co, ak, bk: consecutive bytes) staged in LDS with one
  // load per thread: read from the argument block at a run-time member index, each byte
  // would be a vector memory load that the table loops below wait for
  constexpr int kPosBytes = 3 * kElemGroupOutBits + 2 * kElemKBits;
  __shared__ int8_t PM[kPosBytes];
  for (int t = threadIdx.x; t < kPosBytes; t += kThreads) PM[t] = e.ao[t];
  __syncthreads();
  const int8_t* pak = PM + 3 * kElemGroupOutBits;
  const int8_t* pbk = pak + kElemKBits;
  for (int t = threadIdx.x; t < 3 * kElemChunks * 64; t += kThreads) {
    const int map = t / (kElemChunks * 64), ch = (t >> 6) % kElemChunks, x = t & 63;
    const int8_t* pos = PM + map * kElemGroupOutBits;
    int64_t r = 0;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const int bit = ch * 6 + j;
      if (bit < ob && ((x >> j) & 1)) {
        const int p = pos[bit];
        if (p >= 0) r |= (int64_t)1 << p;
      }
    }
    TO[t] = r;
  }
  const int K = 1 << kb;
  for (int k = threadIdx.x; k < K; k += kThreads) {
    int64_t ra = 0, rb = 0;
#pragma unroll
    for (int j = 0; j < kElemKBits; ++j)
      if (j < kb && ((k >> j) & 1)) {
        ra |= (int64_t)1 << pak[j];
        rb |= (int64_t)1 << pbk[j];
      }
    TKa[k] = ra;
    TKb[k] = rb;
  }
  __syncthreads();
  const float2* A = e.A + (int64_t)z * e.a_bs;
  const float2* B = e.B + (int64_t)z * e.b_bs;
  float2* C = e.C + (int64_t)z * e.c_bs;
  if (e.lane_bits > 0) {
    elem_sum_lanes<PREC>(e, TO, TKa, TKb, A, B, C, bx - e.block0, nblk);
    return;
  }
  const int n_out = 1 << ob;
  for (int o = (bx - e.block0) * kThreads + threadIdx.x; o < n_out; o += nblk * kThreads) {
    int64_t ab = 0, bb = 0, cc = 0;
#pragma unroll
    for (int ch = 0; ch < kElemChunks; ++ch) {
      const int i = ch * 64 + ((o >> (6 * ch)) & 63);
      ab |= TO[i];
      bb |= TO[kElemChunks * 64 + i];
      cc |= TO[2 * kElemChunks * 64 + i];
    }
    float2 acc = f2(0.f, 0.f);
    int k = 0;
    for (; k + 8 <= K; k += 8) {
      float2 av[8], bv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        av[u] = A[ab | TKa[k + u]];
        bv[u] = B[bb | TKb[k + u]];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) acc = cmac<PREC>(acc, av[u], bv[u]);
    }
    for (; k < K; ++k) acc = cmac<PREC>(acc, A[ab | TKa[k]], B[bb | TKb[k]]);
    C[cc] = acc;
  }
}

ElemMember elem_member(const GemmDesc& d, const float2* a, int64_t a_bs, const float2* b, int64_t b_bs, float2* c,
                       int64_t c_bs) {
  ElemMember m;
  m.A = a;
  m.B = b;
  m.C = c;
  m.a_bs = a_bs;
  m.b_bs = b_bs;
  m.c_bs = c_bs;
  m.block0 = 0;  // laid out by the launcher
  m.out_bits = d.nbb + d.nbm + d.nbn;
  m.k_bits = d.nbk;
  m.lane_bits = 0;  // laid out by the launcher
  // result index bits: n lowest, then m, then batch
  for (int j = 0; j < kElemGroupOutBits; ++j) {
    m.ao[j] = m.bo[j] = m.co[j] = -1;
    if (j < d.nbn) {
      m.bo[j] = d.b_n[j];
      m.co[j] = d.c_n[j];
    } else if (j < d.nbn + d.nbm) {
      m.ao[j] = d.a_m[j - d.nbn];
      m.co[j] = d.c_m[j - d.nbn];
    } else if (j < m.out_bits) {
      m.ao[j] = d.a_b[j - d.nbn - d.nbm];
      m.bo[j] = d.b_b[j - d.nbn - d.nbm];
      m.co[j] = d.c_b[j - d.nbn - d.nbm];
    }
  }
  for (int j = 0; j < kElemKBits; ++j) {
    m.ak[j] = j < d.nbk ? d.a_k[j] : 0;
    m.bk[j] = j < d.nbk ? d.b_k[j] : 0;
  }
  return m;
}

hipError_t launch_elem_group(hipStream_t s, const ElemGroupArgs& a, int batch, int precision) {
  if (a.n < 1 || a.n > kElemGroupMax || batch < 1) return hipErrorInvalidValue;
  ElemGroupArgs g = a;
  int32_t blocks = 0;
  for (int i = 0; i < g.n; ++i) {
    ElemMember& m = g.m[i];
    if (m.out_bits < 0 || m.out_bits > kElemGroupOutBits || m.k_bits < 0 || m.k_bits > kElemKBits)
      return hipErrorInvalidValue;
    // one thread per result, or 2^lane_bits lanes for a long sum
    const int lb = elem_lane_bits(m.out_bits, m.k_bits);
    m.lane_bits = lb;
    m.block0 = blocks;
    blocks += (int32_t)((((int64_t)1 << (m.out_bits + lb)) + kThreads - 1) / kThreads);
  }
  g.total_blocks = blocks;
  const void* fn = precision == TN_PREC_BF16X3 ? (const void*)k_elem_group<TN_PREC_BF16X3>
                                               : (const void*)k_elem_group<TN_PREC_C64>;
  void* args[] = {&g};
  return hipLaunchKernel(fn, dim3((unsigned)blocks, batch), dim3(kThreads), args, 0, s);
}

// C[i] = sum over s of partial[s][i] (split-K), contiguous per parameter vector: in pairs (PAIRS), which rounds an
// element log2 SPLIT times instead of SPLIT - 1, or in turn where BF16x3 results keep their order of sums.
template <int SPLIT, bool PAIRS>
__global__ void k_sum_partials(const float2* part, int64_t part_bs, int64_t n, float2* C, int64_t c_bs) {
  const int z = blockIdx.y;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
    float2 v[SPLIT];
#pragma unroll
    for (int s = 0; s < SPLIT; ++s) v[s] = part[(int64_t)z * part_bs + (int64_t)s * n + i];
#pragma unroll
    for (int h = 1; h < SPLIT; h *= 2)
#pragma unroll
      for (int s = 0; s < SPLIT; s += 2 * h)
        if (PAIRS) v[s] = f2(v[s].x + v[s + h].x, v[s].y + v[s + h].y);
    float2 acc = f2(0.f, 0.f);
#pragma unroll
    for (int s = 0; s < (PAIRS ? 1 : SPLIT); ++s) acc = f2(acc.x + v[s].x, acc.y + v[s].y);
    C[(int64_t)z * c_bs + i] = acc;
  }
}

template <bool PAIRS>
static void* sum_fn(int split) {
  return split == 2 ? (void*)k_sum_partials<2, PAIRS> : split == 4 ? (void*)k_sum_partials<4, PAIRS> : (void*)k_sum_partials<8, PAIRS>;
}

template <int TM, int TN, int F>
static void* gemm_fn(int ak, int bnf) {
  if (ak && bnf) return (void*)k_gemm<1, 1, TM, TN, F>;
  if (ak) return (void*)k_gemm<1, 0, TM, TN, F>;
  if (bnf) return (void*)k_gemm<0, 1, TM, TN, F>;
  return (void*)k_gemm<0, 0, TM, TN, F>;
}

template <int TM, int BK, int NW, int BP, int FOUR>
static void* gemm3m_fn_nw(int ak, int bnf) {
  if (ak && bnf) return (void*)k_gemm3m<1, 1, TM, BK, NW, BP, FOUR>;
  if (ak) return (void*)k_gemm3m<1, 0, TM, BK, NW, BP, FOUR>;
  if (bnf) return (void*)k_gemm3m<0, 1, TM, BK, NW, BP, FOUR>;
  return (void*)k_gemm3m<0, 0, TM, BK, NW, BP, FOUR>;
}

template <int TM, int BK, int FOUR = 0>
static void* gemm3m_fn(int ak, int bnf, bool narrow) {
  return narrow ? gemm3m_fn_nw<TM, BK, 1, 0, FOUR>(ak, bnf) : gemm3m_fn_nw<TM, BK, 0, 0, FOUR>(ak, bnf);
}

template <int F>
static void* gemm_fn_tile(int tile, int ak, int bnf, bool narrow) {
  switch (tile) {
    case 0: return gemm_fn<2, 2, F>(ak, bnf);
    case 1: return gemm_fn<2, 1, F>(ak, bnf);
    case 2:
      if constexpr (F == 0) return gemm3m_fn<1, 16, 1>(ak, bnf, narrow);
      else return gemm_fn<1, 2, F>(ak, bnf);
    case 3: return gemm_fn<1, 1, F>(ak, bnf);
    case 5: return gemm3m_fn<2, 16>(ak, bnf, narrow);
    case 7: return narrow ? gemm3m_fn_nw<1, 16, 1, 1, 1>(ak, bnf) : nullptr;
    case 8: return narrow ? gemm3m_fn_nw<1, 16, 1, 2, 1>(ak, bnf) : nullptr;
    default: return gemm3m_fn<1, 16>(ak, bnf, narrow);
  }
}

// Whether every element offset inside one operand tile (its tile-local m or n
// bits, k bits and, batch-packed, batch bits, without the tile's origin) is
// below 2^32 bytes.
static bool tile_offsets_narrow(const int8_t* pos_mn, int n_mn, const int8_t* pos_k, int n_k,
                                const int8_t* pos_b = nullptr, int n_b = 0) {
  int top = -1;
  for (int j = 0; j < n_mn; ++j) top = pos_mn[j] > top ? pos_mn[j] : top;
  for (int j = 0; j < n_k; ++j) top = pos_k[j] > top ? pos_k[j] : top;
  for (int j = 0; j < n_b; ++j) top = pos_b[j] > top ? pos_b[j] : top;
  return top + 1 + 3 <= 32;  // 8-byte elements
}

static bool tile_narrow(const GemmDesc& d, int tile) {
  const int lbk = std::min(d.nbk, 4);
  if (tile == kGemmBatchPacked)
    return tile_offsets_narrow(d.a_m, std::min(d.nbm, 5), d.a_k, lbk, d.a_b, std::min(d.nbb, 2)) &&
           tile_offsets_narrow(d.b_n, std::min(d.nbn, 5), d.b_k, lbk, d.b_b, std::min(d.nbb, 2));
  if (tile == kGemmColumnPacked)
    return tile_offsets_narrow(d.a_m, std::min(d.nbm, 5), d.a_k, lbk) &&
           tile_offsets_narrow(d.b_n, std::min(d.nbn, 7), d.b_k, lbk);
  const int lbm = kGemmTileM[tile] == 128 ? 7 : 6, lbn = kGemmTileN[tile] == 64 ? 6 : 5;
  return tile_offsets_narrow(d.a_m, std::min(d.nbm, lbm), d.a_k, lbk) &&
         tile_offsets_narrow(d.b_n, std::min(d.nbn, lbn), d.b_k, lbk);
}

bool gemm_tile_supported(const GemmDesc& d, int tile) {
  if (tile < 0 || tile >= kGemmTiles) return false;
  if (tile == kGemmBatchPacked)  // four whole batch items of at most 32 x 32 per block
    return d.M <= 32 && d.N <= 32 && d.nbb >= 2 && tile_narrow(d, tile);
  if (tile == kGemmColumnPacked)  // M <= 32, four 32-column slices per block
    return d.M <= 32 && d.N >= 64 && tile_narrow(d, tile);
  return true;
}

// The order in which store_tile walks a result tile: its bits by ascending address in C, bits beyond the product's
// sizes (whose elements are not stored) last.  Row bit 5 and column bit 5 of the 64 x 64 elements at a time are wave
// bits: m and n of a plain tile (m bit 6 of the 128-row ones, whose bit 5 is the round), batch items or columns of the
// packed ones.
static void tile_args(const GemmDesc& d, int tile, TileArgs& g) {
  const bool batch_packed = tile == kGemmBatchPacked, col_packed = tile == kGemmColumnPacked;
  const bool packed = batch_packed || col_packed;
  const int bn = packed ? 64 : kGemmTileN[tile], n_col = bn == 64 ? 6 : 5;
  struct Bit {
    int pos, lds, mn;
  };
  std::vector<Bit> bits;
  auto add = [&](bool row, int j) {
    Bit b;
    const int place = row ? tile_place(1 << j, 0, bn) : 1 << j;
    b.lds = place;
    auto m_bit = [&](int i) { b.pos = i < d.nbm ? d.c_m[i] : 64; b.mn = 1 << i; };
    auto n_bit = [&](int i) { b.pos = i < d.nbn ? d.c_n[i] : 64; b.mn = 1 << (i + 8); };
    if (packed && j == 5) {
      if (col_packed) n_bit(row ? 6 : 5);
      else { b.pos = d.c_b[row ? 1 : 0]; b.mn = 0; }
    } else if (row) {
      m_bit(j == 5 && kGemmTileM[tile] == 128 ? 6 : j);
    } else {
      n_bit(j);
    }
    bits.push_back(b);
  };
  for (int j = 0; j < 6; ++j) add(true, j);
  for (int j = 0; j < n_col; ++j) add(false, j);
  std::stable_sort(bits.begin(), bits.end(), [](const Bit& a, const Bit& b) { return a.pos < b.pos; });
  g.lines = 1;
  for (int j = 0; j < 4; ++j) g.lines &= bits[j].pos == j;
  for (int j = 0; j < kTileBits; ++j) {
    g.st_pos[j] = j < (int)bits.size() && bits[j].pos < 64 ? bits[j].pos : 0;
    g.st_lds[j] = j < (int)bits.size() ? bits[j].lds : 0;
    g.st_mn[j] = j < (int)bits.size() ? bits[j].mn : 0;
  }
  g.c_next = d.c_m[5];
  for (int j = 0; j < 7; ++j) {
    g.a_row[j] = batch_packed && j >= 5 ? d.a_b[j - 5] : packed && j >= 5 ? 0 : d.a_m[j];
    g.b_col[j] = batch_packed && j >= 5 ? d.b_b[j - 5] : d.b_n[j];
  }
  for (int j = 0; j < 10; ++j) {
    g.a_k[j] = d.a_k[j];
    g.b_k[j] = d.b_k[j];
  }
  for (int j = 0; j < 64; ++j) g.from_a[j] = g.from_b[j] = g.from_c[j] = 0;
  auto from = [](uint8_t* of, const int8_t* pos, int n, int src) {
    for (int j = 0; j < n; ++j) of[pos[j]] = (uint8_t)(src * 64 + j);
  };
  from(g.from_a, d.a_b, d.nbb, 1);
  from(g.from_a, d.a_m, d.nbm, 2);
  from(g.from_a, d.a_k, d.nbk, 3);
  from(g.from_b, d.b_b, d.nbb, 1);
  from(g.from_b, d.b_n, d.nbn, 2);
  from(g.from_b, d.b_k, d.nbk, 3);
  from(g.from_c, d.c_b, d.nbb, 1);
  from(g.from_c, d.c_m, d.nbm, 2);
  from(g.from_c, d.c_n, d.nbn, 3);
}

// The product with the low bits of its m, n and k indices (those that a tile spans) first the ones that lie in a
// 128-byte line of an operand or of C (its 4 lowest address bits), the rest as they were: a line is then used whole by
// one block.  (The descriptor orders m and n by C and k by A alone; with B's lowest three bits above k's low four,
// complex64 1024 x 4096 x 512 loaded each line of B 8 times over: 349 us, 135 so.)  Short sums store more than they
// load, and keep C's order in m and n: their tiles are then longer runs of C.
static GemmDesc line_order(const GemmDesc& d, int precision) {
  GemmDesc r = d;
  auto order = [](int n, const int8_t* x, const int8_t* y, int8_t* rx, int8_t* ry) {
    std::vector<int> v(n);
    for (int j = 0; j < n; ++j) v[j] = j;
    auto key = [&](int j) { return std::min<int>(std::min(x[j], y[j]), 4); };
    std::stable_sort(v.begin(), v.end(), [&](int a, int b) { return key(a) < key(b); });
    for (int j = 0; j < n; ++j) {
      rx[j] = x[v[j]];
      ry[j] = y[v[j]];
    }
  };
  if (d.K >= 64) {
    order(d.nbm, d.a_m, d.c_m, r.a_m, r.c_m);
    order(d.nbn, d.b_n, d.c_n, r.b_n, r.c_n);
  }
  if (precision != TN_PREC_BF16X3 || !d.fixed_sum) order(d.nbk, d.a_k, d.b_k, r.a_k, r.b_k);
  return r;
}

hipError_t launch_gemm(hipStream_t s, const GemmDesc& desc, int tile, int split, const float2* a, int64_t a_bs,
                       const float2* b, int64_t b_bs, float2* c, int64_t c_bs, float2* tmp, int64_t tmp_bs, int batch,
                       int precision) {
  if (!gemm_tile_supported(desc, tile)) return hipErrorInvalidValue;
  const bool reorder = tile != kGemmVector && tile != kGemmBatchPacked && tile != kGemmColumnPacked;
  const GemmDesc d = reorder ? line_order(desc, precision) : desc;
  if (tile > kGemmVector && precision != TN_PREC_C64) return hipErrorInvalidValue;  // 3M: FP32 only
  const int64_t c_elems = d.batch * d.M * d.N;
  if (tile == kGemmVector) {
    if (d.K > kElemMaxK) return hipErrorInvalidValue;
    if (d.nbb + d.nbm + d.nbn <= kElemGroupOutBits && d.nbk <= kElemKBits) {  // the table-driven kernel
      ElemGroupArgs ga;
      ga.n = 1;
      ga.total_blocks = 0;
      ga.m[0] = elem_member(d, a, a_bs, b, b_bs, c, c_bs);
      return launch_elem_group(s, ga, batch, precision);
    }
    GemmArgs g;
    g.A = a; g.B = b; g.C = c;
    g.batch = d.batch; g.M = d.M; g.N = d.N; g.K = d.K;
    g.a_bs = a_bs; g.b_bs = b_bs; g.c_bs = c_bs;
    g.nbb = d.nbb; g.nbm = d.nbm; g.nbn = d.nbn; g.nbk = d.nbk;
    for (int j = 0; j < kGemmMaxBits; ++j) {
      g.a_b[j] = d.a_b[j]; g.a_m[j] = d.a_m[j]; g.a_k[j] = d.a_k[j];
      g.b_b[j] = d.b_b[j]; g.b_k[j] = d.b_k[j]; g.b_n[j] = d.b_n[j];
      g.c_b[j] = d.c_b[j]; g.c_m[j] = d.c_m[j]; g.c_n[j] = d.c_n[j];
    }
    int64_t eb = (c_elems + kThreads - 1) / kThreads;
    if (eb > 65535) eb = 65535;
    if (precision == TN_PREC_BF16X3)
      hipLaunchKernelGGL(k_contract_elem<TN_PREC_BF16X3>, dim3((unsigned)eb, batch), dim3(kThreads), 0, s, g);
    else
      hipLaunchKernelGGL(k_contract_elem<TN_PREC_C64>, dim3((unsigned)eb, batch), dim3(kThreads), 0, s, g);
    return hipGetLastError();
  }
  TileArgs g;
  split = split > 1 ? split : 1;
  if (split > 1 && (d.K % split != 0 || split > d.max_split || !tmp || (split != 2 && split != 4 && split != kGemmMaxSplit)))
    return hipErrorInvalidValue;
  g.A = a; g.B = b;
  g.C = split > 1 ? tmp : c;
  g.a_bs = a_bs; g.b_bs = b_bs;
  g.c_bs = split > 1 ? tmp_bs : c_bs;
  g.M = d.M; g.N = d.N; g.K = d.K;
  g.c_elems = c_elems;
  tile_args(d, tile, g);
  auto log2_of = [](int64_t x) {
    int l = 0;
    while (((int64_t)1 << l) < x) ++l;
    return l;
  };
  const int64_t tiles_m = (d.M + kGemmTileM[tile] - 1) / kGemmTileM[tile];
  const int64_t tiles_n = (d.N + kGemmTileN[tile] - 1) / kGemmTileN[tile];
  const int64_t batch_blocks = tile == kGemmBatchPacked ? d.batch / 4 : d.batch;
  const int64_t blocks = tiles_m * tiles_n * split * batch_blocks * batch;
  if (blocks > ((int64_t)1 << 24)) return hipErrorInvalidValue;  // grid of < 2^32 work-items
  g.lg_tm = log2_of(tiles_m);
  g.lg_tn = log2_of(tiles_n);
  // bands of a quarter of the tile columns on large grids (two XCDs per band), whole rows otherwise
  g.lg_band = tiles_n >= 16 && tiles_m >= 16 ? g.lg_tn - 2 : g.lg_tn;
  g.lg_split = log2_of(split);
  g.lg_batch = log2_of(batch_blocks);
  g.xcd = blocks % 8 == 0 ? 1 : 0;
  const bool narrow = tile_narrow(d, tile);
  void* fn = precision == TN_PREC_BF16X3 ? gemm_fn_tile<1>(tile, d.a_kfast, d.b_nfast, narrow)
                                         : gemm_fn_tile<0>(tile, d.a_kfast, d.b_nfast, narrow);
  void* args[] = {&g};
  hipError_t e = hipLaunchKernel(fn, dim3((unsigned)blocks), dim3(kThreads), args, 0, s);
  if (e != hipSuccess || split == 1) return e;
  int64_t rb = (c_elems + kThreads - 1) / kThreads;
  if (rb > 16384) rb = 16384;
  const float2* part = tmp;
  void* sum_args[] = {&part, &tmp_bs, (void*)&c_elems, &c, &c_bs};
  return hipLaunchKernel(precision == TN_PREC_BF16X3 ? sum_fn<false>(split) : sum_fn<true>(split),
                         dim3((unsigned)rb, batch), dim3(kThreads), sum_args, 0, s);
}

// ---------------------------------------------------------------------------
// Reductions (FP64 accumulation)
// ---------------------------------------------------------------------------
__device__ inline double zdiag(uint64_t x, const ZTerms& t) {
  double d = 0;
  for (int i = 0; i < t.n; ++i) d += (__popcll(x & t.mask[i]) & 1) ? -t.coeff[i] : t.coeff[i];
  return d;
}

__global__ __launch_bounds__(kThreads) void k_expect_partial(const float2* psi, int64_t bs, int64_t n, ZTerms t,
                                                             double* partial) {
  __shared__ double red[kThreads / 64];
  const int z = blockIdx.y;
  const float2* p = psi + (int64_t)z * bs;
  double acc = 0;
  for (int64_t x = (int64_t)blockIdx.x * kThreads + threadIdx.x; x < n; x += (int64_t)gridDim.x * kThreads) {
    const float2 v = p[x];
    const double pr = (double)v.x * v.x + (double)v.y * v.y;
    acc += pr * zdiag((uint64_t)x, t);
  }
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0) partial[(int64_t)z * kExpectBlocks + blockIdx.x] = s;
}

// one block per parameter vector; fixed summation order (deterministic)
__global__ __launch_bounds__(kThreads) void k_reduce_rows(const double* partial, int nb, double* out,
                                                          int64_t out_stride) {
  __shared__ double red[kThreads / 64];
  const int z = blockIdx.x;
  double s = 0;
  for (int i = threadIdx.x; i < nb; i += kThreads) s += partial[(int64_t)z * kExpectBlocks + i];
  s = block_sum(s, red);
  if (threadIdx.x == 0) out[(int64_t)z * out_stride] = s;
}

// blocks of 4096 consecutive elements: thread t takes base + t + 256 j
__global__ __launch_bounds__(kThreads) void k_expect_partial16(const float2* psi, int64_t bs, int64_t n, ZTerms t,
                                                               double* partial) {
  __shared__ double red[kThreads / 64];
  const int z = blockIdx.y;
  const float2* p = psi + (int64_t)z * bs;
  double acc = 0;
  for (int64_t c = blockIdx.x; c < (n >> 12); c += gridDim.x) {
    const int64_t base = (c << 12) | threadIdx.x;
    double w[16];
    sum_terms16((uint64_t)base, t, w);  // at base + 256 j
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const float2 v = p[base + 256 * j];
      acc += ((double)v.x * v.x + (double)v.y * v.y) * w[j];
    }
  }
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0) partial[(int64_t)z * kExpectBlocks + blockIdx.x] = s;
}

hipError_t launch_reduce_rows(hipStream_t s, const double* partial, int n, int batch, double* out,
                              int64_t out_stride) {
  hipLaunchKernelGGL(k_reduce_rows, dim3(batch), dim3(kThreads), 0, s, partial, n, out, out_stride);
  return hipGetLastError();
}

hipError_t launch_expectation(hipStream_t s, const float2* psi, int64_t psi_bs, int64_t n_elems, const ZTerms& terms,
                              int batch, double* partial, double* out, int64_t out_stride) {
  int64_t blocks;
  if (n_elems >= 4096) {
    blocks = std::min<int64_t>(n_elems >> 12, kExpectBlocks);
    hipLaunchKernelGGL(k_expect_partial16, dim3((unsigned)blocks, batch), dim3(kThreads), 0, s, psi, psi_bs, n_elems,
                       terms, partial);
  } else {
    blocks = std::min<int64_t>((n_elems + kThreads - 1) / kThreads, kExpectBlocks);
    hipLaunchKernelGGL(k_expect_partial, dim3((unsigned)blocks, batch), dim3(kThreads), 0, s, psi, psi_bs, n_elems,
                       terms, partial);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_reduce_rows(s, partial, (int)blocks, batch, out, out_stride);
}

__global__ void k_copy(const float2* in, int64_t in_bs, float2* out, int64_t out_bs, int64_t n) {
  const int z = blockIdx.y;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads)
    out[(int64_t)z * out_bs + i] = in[(int64_t)z * in_bs + i];
}

hipError_t launch_copy(hipStream_t s, const float2* in, int64_t in_bs, float2* out, int64_t out_bs, int64_t n,
                       int batch) {
  int64_t blocks = (n + kThreads - 1) / kThreads;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(k_copy, dim3((unsigned)blocks, batch), dim3(kThreads), 0, s, in, in_bs, out, out_bs, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Adjoint sweep
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_apply_diag_obs(const float2* psi, int64_t psi_bs, float2* lam,
                                                             int64_t lam_bs, int64_t n, ZTerms t) {
  const int z = blockIdx.y;
  for (int64_t x = (int64_t)blockIdx.x * kThreads + threadIdx.x; x < n; x += (int64_t)gridDim.x * kThreads) {
    const float2 v = psi[(int64_t)z * psi_bs + x];
    const double d = zdiag((uint64_t)x, t);
    lam[(int64_t)z * lam_bs + x] = f2((float)(d * v.x), (float)(d * v.y));
  }
}

__global__ __launch_bounds__(kThreads) void k_apply_diag_obs16(const float2* psi, int64_t psi_bs, float2* lam,
                                                               int64_t lam_bs, int64_t n, ZTerms t) {
  const int z = blockIdx.y;
  for (int64_t c = blockIdx.x; c < (n >> 12); c += gridDim.x) {
    const int64_t base = (c << 12) | threadIdx.x;
    double w[16];
    sum_terms16((uint64_t)base, t, w);  // at base + 256 j
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const float2 v = psi[(int64_t)z * psi_bs + base + 256 * j];
      lam[(int64_t)z * lam_bs + base + 256 * j] = f2((float)(w[j] * v.x), (float)(w[j] * v.y));
    }
  }
}

hipError_t launch_apply_diag_obs(hipStream_t s, const float2* psi, int64_t psi_bs, float2* lam, int64_t lam_bs,
                                 int64_t n_elems, const ZTerms& terms, int batch) {
  if (n_elems >= 4096) {
    const int64_t blocks = std::min<int64_t>(n_elems >> 12, 16384);
    hipLaunchKernelGGL(k_apply_diag_obs16, dim3((unsigned)blocks, batch), dim3(kThreads), 0, s, psi, psi_bs, lam,
                       lam_bs, n_elems, terms);
    return hipGetLastError();
  }
  int64_t blocks = (n_elems + kThreads - 1) / kThreads;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(k_apply_diag_obs, dim3((unsigned)blocks, batch), dim3(kThreads), 0, s, psi, psi_bs, lam, lam_bs,
                     n_elems, terms);
  return hipGetLastError();
}

// Im(conj(l) * p)
__device__ inline double im_cl_p(float2 l, float2 p) { return (double)l.x * p.y - (double)l.y * p.x; }
// Re(conj(l) * p)
__device__ inline double re_cl_p(float2 l, float2 p) { return (double)l.x * p.x + (double)l.y * p.y; }

template <int NQ, int PREC>
__global__ __launch_bounds__(kThreads) void k_adjoint_step(SweepArgs a, const float2* U, int64_t u_bs, float2* psi,
                                                           int64_t psi_bs, float2* lam, int64_t lam_bs,
                                                           int64_t n_groups, double* partials, int64_t pstride) {
  __shared__ double red[kThreads / 64];
  constexpr int D = 1 << NQ;
  const int z = blockIdx.y;
  float2* P = psi + (int64_t)z * psi_bs;
  float2* L = lam + (int64_t)z * lam_bs;
  float2 u[D * D];
  for (int i = 0; i < D * D; ++i) u[i] = U[(int64_t)z * u_bs + i];
  int lo = a.pos[0], hi = a.pos[0];
  if (NQ == 2) { lo = min(a.pos[0], a.pos[1]); hi = max(a.pos[0], a.pos[1]); }
  double g = 0;
  for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < n_groups; j += (int64_t)gridDim.x * kThreads) {
    int64_t base = ((j >> lo) << (lo + 1)) | (j & (((int64_t)1 << lo) - 1));
    if (NQ == 2) base = ((base >> hi) << (hi + 1)) | (base & (((int64_t)1 << hi) - 1));
    int64_t idx[D];
    if (NQ == 1) {
      idx[0] = base;
      idx[1] = base | ((int64_t)1 << a.pos[0]);
    } else {
      for (int v = 0; v < 4; ++v)
        idx[v] = base | ((int64_t)(v >> 1) << a.pos[0]) | ((int64_t)(v & 1) << a.pos[1]);
    }
    float2 p[D], l[D];
    for (int v = 0; v < D; ++v) { p[v] = P[idx[v]]; l[v] = L[idx[v]]; }
    switch (a.gen) {
      case GEN_X_HALF: g += im_cl_p(l[0], p[1]) + im_cl_p(l[1], p[0]); break;
      case GEN_X: g += 2.0 * (im_cl_p(l[0], p[1]) + im_cl_p(l[1], p[0])); break;
      case GEN_Y_HALF:  // Y p = (-i p1, i p0);  Im(conj(l) (-i p)) = -Re(conj(l) p)
        g += -re_cl_p(l[0], p[1]) + re_cl_p(l[1], p[0]); break;
      case GEN_Z_HALF: g += im_cl_p(l[0], p[0]) - im_cl_p(l[1], p[1]); break;
      case GEN_ZZ_PHASE: if (NQ == 2) g += 2.0 * (im_cl_p(l[1], p[1]) + im_cl_p(l[2], p[2])); break;
      case GEN_CPHASE: if (NQ == 2) g += -2.0 * im_cl_p(l[3], p[3]); break;
      default: break;
    }
    // psi <- U^dagger psi, lam <- U^dagger lam (products in the requested precision)
    for (int r = 0; r < D; ++r) {
      float2 ap = f2(0.f, 0.f), al = f2(0.f, 0.f);
      for (int c = 0; c < D; ++c) {
        const float2 uc = f2(u[c * D + r].x, -u[c * D + r].y);  // conj(U[c][r])
        ap = cmac<PREC>(ap, uc, p[c]);
        al = cmac<PREC>(al, uc, l[c]);
      }
      P[idx[r]] = ap;
      L[idx[r]] = al;
    }
  }
  if (a.slot >= 0) {
    const double s = block_sum(g, red);
    if (threadIdx.x == 0) partials[(int64_t)z * pstride + (int64_t)a.slot * kReduceBlocks + blockIdx.x] = s;
  }
}

hipError_t launch_adjoint_step(hipStream_t s, const SweepArgs& a, const float2* u, int64_t u_bs, float2* psi,
                               int64_t psi_bs, float2* lam, int64_t lam_bs, int64_t n_elems, int batch,
                               double* partials, int64_t partial_stride, int precision) {
  const int64_t groups = n_elems >> a.nq;
  // a fixed grid so that every partial slot is written
  const int blocks = kReduceBlocks;
  const bool bf = precision == TN_PREC_BF16X3;
  void* fn = a.nq == 2 ? (bf ? (void*)k_adjoint_step<2, TN_PREC_BF16X3> : (void*)k_adjoint_step<2, TN_PREC_C64>)
                       : (bf ? (void*)k_adjoint_step<1, TN_PREC_BF16X3> : (void*)k_adjoint_step<1, TN_PREC_C64>);
  SweepArgs aa = a;
  void* args[] = {&aa, (void*)&u, (void*)&u_bs, (void*)&psi, (void*)&psi_bs, (void*)&lam, (void*)&lam_bs,
                  (void*)&groups, (void*)&partials, (void*)&partial_stride};
  return hipLaunchKernel(fn, dim3(blocks, batch), dim3(kThreads), args, 0, s);
}

// One wave per parameter and parameter vector: its slots in turn, the lanes
// over a slot's columns.  (One thread per slot and then one per parameter
// over all slots took 20 + 17 us on a 13-qubit ansatz and 21 + 47 us on the
// 20-qubit one; this takes 5 and 9.)
__global__ __launch_bounds__(kThreads) void k_gradient_sums(const double* partials, int64_t pstride, int n_cols,
                                                            const int32_t* __restrict__ param_slots, int n_params,
                                                            const double* grad_out, double* grad) {
  const int p = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6), z = blockIdx.y, lane = threadIdx.x & 63;
  if (p >= n_params) return;
  double s = 0;
  for (int i = param_slots[p]; i < param_slots[p + 1]; ++i) {
    const double* row = partials + (int64_t)z * pstride + (int64_t)param_slots[i] * kReduceBlocks;
    for (int c = lane; c < n_cols; c += 64) s += row[c];
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) grad[(int64_t)z * n_params + p] = (grad_out ? grad_out[z] : 1.0) * s;
}

hipError_t launch_gradient_reduce(hipStream_t s, const double* partials, int64_t partial_stride, int n_cols,
                                  const int32_t* param_slots, int n_params, const double* grad_out, int batch,
                                  double* grad) {
  if (n_params == 0) return hipSuccess;
  const int per = kThreads / 64;
  hipLaunchKernelGGL(k_gradient_sums, dim3((n_params + per - 1) / per, batch), dim3(kThreads), 0, s, partials,
                     partial_stride, n_cols, param_slots, n_params, grad_out, grad);
  return hipGetLastError();
}

__global__ __launch_bounds__(kRecipeThreads) void k_sweep_matrices(const Recipe* rs, int n, const RecipeOp* ops,
                                                                    const double* mats,
                                 const double* params, int64_t pstride, float2* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int z = blockIdx.y;
  if (i >= n) return;
  const double* p = params ? params + (int64_t)z * pstride : nullptr;
  float2* o = out + ((int64_t)z * n + i) * 16;
  if (rs[i].nq == 2) {
    c128 M[16];
    recipe_matrix_d<4>(rs[i], ops, mats, p, M);
#pragma unroll
    for (int k = 0; k < 16; ++k) o[k] = f2((float)M[k].re, (float)M[k].im);
  } else {
    c128 M[4];
    recipe_matrix_d<2>(rs[i], ops, mats, p, M);
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = f2((float)M[k].re, (float)M[k].im);
  }
}

hipError_t launch_sweep_matrices(hipStream_t s, const Recipe* recipes, int n, const RecipeOp* ops, const double* mats,
                                 const double* params, int64_t params_stride, int batch, float2* out) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_sweep_matrices, dim3((n + kRecipeThreads - 1) / kRecipeThreads, batch), dim3(kRecipeThreads),
                     0, s, recipes, n, ops, mats, params, params_stride, out);
  return hipGetLastError();
}

}  // namespace tnq

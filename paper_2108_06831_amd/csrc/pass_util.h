// Device helpers of the gate passes: gates on sixteen register elements, chunk
// moves between HBM and LDS, gradient terms and wave sums.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "device_util.h"
#include "kernels.h"

namespace tnq {

// ---------------------------------------------------------------------------
// Fused streaming pass: a chunk of 2^l elements (address bits lpos, the five
// lowest always among them so that loads and stores move 256-byte runs) is
// staged in LDS and every gate of the pass is applied to it before it is
// written back: one HBM read and one write for the whole pass.  Gates run in
// segments: each thread holds the 16 elements that differ in the segment's
// four register bits, applies the segment's gates in registers, and the chunk
// goes through LDS only between segments.
// ---------------------------------------------------------------------------
// (lpos and rest start at multiples of 4 bytes: deposit() reads them as 32-bit words)
struct SweepPassArgs {
  const float2* in;
  float2* out;
  int64_t in_bs, out_bs;
  const float2* vals;  // the chain's gathered gate values
  int64_t vals_bs;
  const SweepGateDesc* gates;
  const SweepSegment* segs;
  int32_t n_segs, l, n_rest, pad;
  int32_t ctab_off;          // the pass's power tables in vals
  int32_t lds_off, lds_n;    // the range of vals staged in LDS: the pass's gate values and power
                             // tables when they fit (gates_in_lds), else the power tables only
  int32_t gates_in_lds, pad2;
  int8_t lpos[kSweepMaxLocal];
  int8_t rest[64];
};
static_assert(offsetof(SweepPassArgs, lpos) % 4 == 0 && offsetof(SweepPassArgs, rest) % 4 == 0 &&
                  kSweepMaxLocal % 4 == 0, "position maps aligned to 32-bit words");

__device__ inline int64_t ins0(int64_t x, int p) { return ((x >> p) << (p + 1)) | (x & (((int64_t)1 << p) - 1)); }
__device__ inline int lds_phys(int i) { return i + (i >> 5); }

// Moving a chunk of 2^l = 16 nt elements between HBM and LDS: thread tid
// takes elements tid + k nt, k = 0..15 (consecutive threads on consecutive
// addresses).  The loads are issued eight at a time before their LDS writes,
// so a thread waits for HBM twice per chunk instead of once per element,
// without holding all sixteen in registers (which would lower the occupancy
// of the pass kernels); the empty asm keeps the compiler from merging the two
// halves.
__device__ __forceinline__ void chunk_to_lds(float2* buf, const float2* src, int64_t base, const int64_t* dep_hi,
                                             int tid, int nt) {
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    float2 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int i = tid + (8 * h + k) * nt;
      v[k] = load_stream(&src[base | (i & 31) | dep_hi[i >> 5]]);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) buf[lds_phys(tid + (8 * h + k) * nt)] = v[k];
    asm volatile("" ::: "memory");
  }
}
// The same for two tensors at once (eight elements of each in flight).
__device__ __forceinline__ void chunk2_to_lds(float2* buf0, float2* buf1, const float2* src0, const float2* src1,
                                              int64_t base, const int64_t* dep_hi, int tid, int nt) {
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    float2 v[8], w[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int i = tid + (8 * h + k) * nt;
      const int64_t x = base | (i & 31) | dep_hi[i >> 5];
      v[k] = load_stream(&src0[x]);
      w[k] = load_stream(&src1[x]);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      buf0[lds_phys(tid + (8 * h + k) * nt)] = v[k];
      buf1[lds_phys(tid + (8 * h + k) * nt)] = w[k];
    }
    asm volatile("" ::: "memory");
  }
}
__device__ __forceinline__ void chunk_from_lds(float2* dst, const float2* buf, int64_t base, const int64_t* dep_hi,
                                               int tid, int nt) {
  // the addresses are computed again here rather than kept in registers since the load
  asm volatile("" ::: "memory");
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    float2 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = buf[lds_phys(tid + (8 * h + k) * nt)];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int i = tid + (8 * h + k) * nt;
      store_stream(&dst[base | (i & 31) | dep_hi[i >> 5]], v[k].x, v[k].y);
    }
    asm volatile("" ::: "memory");
  }
}

// -v of a uniform value, as an integer operation (which stays on the scalar unit)
__device__ __forceinline__ float neg_s(float v) { return __uint_as_float(__float_as_uint(v) ^ 0x80000000u); }
// v with the sign bits of s flipped
__device__ __forceinline__ float2 flip_s(float2 v, uint32_t s) {
  return f2(__uint_as_float(__float_as_uint(v.x) ^ s), __uint_as_float(__float_as_uint(v.y) ^ s));
}

// Shapes of a one-qubit matrix that take half the multiplies (known from the
// gate kinds, see GateForm): every entry real (RY, H, X, ...), or a real
// diagonal and an imaginary off-diagonal (RX, Y, the QAOA mixer exp(-i b X)).
enum { kDenseGeneric = 0, kDenseReal = 1, kDenseRxLike = 2 };

// The register-position variants of a helper below are the same code apart
// from which elements they touch, and in reduced precision they are long
// enough that the compiler merges their common tails, selecting the elements
// through pointers, which puts all of them in scratch memory.  A distinct
// (empty) marker at the end of each variant keeps the tails apart.
template <int PREC, int ID>
__device__ __forceinline__ void variant_end() {
  if constexpr (PREC != TN_PREC_C64) asm volatile("; variant %0" ::"n"(ID));
}

template <int PREC, int U, int FORM>
__device__ __forceinline__ void reg_apply1(float2 (&x)[16], const float2* g) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r & (1 << U)) continue;
    const int r1 = r | (1 << U);
    const float2 a = x[r], b = x[r1];
    if (PREC == TN_PREC_C64 && FORM == kDenseReal) {
      x[r] = f2(fmaf(g[0].x, a.x, g[1].x * b.x), fmaf(g[0].x, a.y, g[1].x * b.y));
      x[r1] = f2(fmaf(g[2].x, a.x, g[3].x * b.x), fmaf(g[2].x, a.y, g[3].x * b.y));
    } else if (PREC == TN_PREC_C64 && FORM == kDenseRxLike) {
      // g1 = i g1.y, g2 = i g2.y: i t (u + i v) = -t v + i t u
      x[r] = f2(fmaf(g[0].x, a.x, -g[1].y * b.y), fmaf(g[0].x, a.y, g[1].y * b.x));
      x[r1] = f2(fmaf(g[3].x, b.x, -g[2].y * a.y), fmaf(g[3].x, b.y, g[2].y * a.x));
    } else {
      x[r] = cmac<PREC>(cmul<PREC>(g[0], a), g[1], b);
      x[r1] = cmac<PREC>(cmul<PREC>(g[2], a), g[3], b);
    }
  }
  variant_end<PREC, U * 3 + FORM>();
}

// A dense one-qubit gate on register bit rb, its values in the given form, on
// one state (NS = 1) or on x and y (NS = 2).  Bit and form are compile-time
// constants in every case: a form tested inside the unrolled element loop
// would be turned into per-element selects between the variants.
template <int PREC, int NS>
__device__ __forceinline__ void apply_dense1(float2 (&x)[16], float2 (&y)[16], const float2* g, int rb, int form) {
#define TNQ_DENSE1(U, F)                   \
  reg_apply1<PREC, U, F>(x, g);            \
  if (NS == 2) reg_apply1<PREC, U, F>(y, g); \
  break;
  // (the reduced-precision products take one form for all: identical cases would be merged
  // into code that indexes the elements through pointers, which keeps them out of registers)
  switch (rb * 3 + (PREC == TN_PREC_C64 ? form : kDenseGeneric)) {
    case 0: TNQ_DENSE1(0, 0)
    case 1: TNQ_DENSE1(0, 1)
    case 2: TNQ_DENSE1(0, 2)
    case 3: TNQ_DENSE1(1, 0)
    case 4: TNQ_DENSE1(1, 1)
    case 5: TNQ_DENSE1(1, 2)
    case 6: TNQ_DENSE1(2, 0)
    case 7: TNQ_DENSE1(2, 1)
    case 8: TNQ_DENSE1(2, 2)
    case 9: TNQ_DENSE1(3, 0)
    case 10: TNQ_DENSE1(3, 1)
    default: TNQ_DENSE1(3, 2)
  }
#undef TNQ_DENSE1
}

// A run of two to four dense one-qubit gates of one form on the register bits
// of mask M, in increasing bit order (the k-th gate's values at gp[k]), on x
// (NS = 1) or on x and y (NS = 2): straight-line code, where gate-by-gate
// dispatch would end every gate with a copy of the elements back into the
// registers the loop carries them in.
template <int PREC, int NS, int M, int F>
__device__ __forceinline__ void run_apply(float2 (&x)[16], float2 (&y)[16], const float2* const (&gp)[4]) {
  int k = 0;
  if constexpr ((M & 1) != 0) {
    reg_apply1<PREC, 0, F>(x, gp[k]);
    if (NS == 2) reg_apply1<PREC, 0, F>(y, gp[k]);
    ++k;
  }
  if constexpr ((M & 2) != 0) {
    reg_apply1<PREC, 1, F>(x, gp[k]);
    if (NS == 2) reg_apply1<PREC, 1, F>(y, gp[k]);
    ++k;
  }
  if constexpr ((M & 4) != 0) {
    reg_apply1<PREC, 2, F>(x, gp[k]);
    if (NS == 2) reg_apply1<PREC, 2, F>(y, gp[k]);
    ++k;
  }
  if constexpr ((M & 8) != 0) {
    reg_apply1<PREC, 3, F>(x, gp[k]);
    if (NS == 2) reg_apply1<PREC, 3, F>(y, gp[k]);
  }
  variant_end<PREC, 200 + M * 8 + NS * 4 + F>();
}

template <int PREC, int NS>
__device__ __forceinline__ void apply_dense1_run(float2 (&x)[16], float2 (&y)[16], const float2* const (&g)[4],
                                                 int mask, int form) {
#define TNQ_RUN(M)                                                   \
  case M * 3 + kDenseGeneric: run_apply<PREC, NS, M, kDenseGeneric>(x, y, g); break; \
  case M * 3 + kDenseReal: run_apply<PREC, NS, M, kDenseReal>(x, y, g); break;       \
  case M * 3 + kDenseRxLike: run_apply<PREC, NS, M, kDenseRxLike>(x, y, g); break;
  switch (mask * 3 + (PREC == TN_PREC_C64 ? form : kDenseGeneric)) {
    TNQ_RUN(3) TNQ_RUN(5) TNQ_RUN(6) TNQ_RUN(7) TNQ_RUN(9) TNQ_RUN(10) TNQ_RUN(11) TNQ_RUN(12) TNQ_RUN(13)
    TNQ_RUN(14)
    default: run_apply<PREC, NS, 15, kDenseGeneric>(x, y, g); break;  // mask 15, generic form
    case 15 * 3 + kDenseReal: run_apply<PREC, NS, 15, kDenseReal>(x, y, g); break;
    case 15 * 3 + kDenseRxLike: run_apply<PREC, NS, 15, kDenseRxLike>(x, y, g); break;
  }
#undef TNQ_RUN
}

template <int PREC, int U0, int U1>
__device__ __forceinline__ void reg_apply2(float2 (&x)[16], const float2* g) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r & ((1 << U0) | (1 << U1))) continue;
    const int id[4] = {r, r | (1 << U0), r | (1 << U1), r | (1 << U0) | (1 << U1)};
    float2 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = x[id[k]];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      float2 acc = f2(0.f, 0.f);
#pragma unroll
      for (int k = 0; k < 4; ++k) acc = cmac<PREC>(acc, g[4 * m + k], v[k]);
      x[id[m]] = acc;
    }
  }
  variant_end<PREC, 16 + U0 * 4 + U1>();
}

// Diagonal factor on the 16 register elements, with the bits of the factor's
// index resolved at compile time: e_{bit U of r} ...
template <int PREC, int U>
__device__ __forceinline__ void diag_reg1(float2 (&x)[16], float2 e0, float2 e1) {
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = cmul<PREC>((r >> U) & 1 ? e1 : e0, x[r]);
  variant_end<PREC, 32 + U>();
}
// ... or d_{bit U0 of r + 2 bit U1 of r}
template <int PREC, int U0, int U1>
__device__ __forceinline__ void diag_reg2(float2 (&x)[16], float2 d0, float2 d1, float2 d2, float2 d3) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int b = ((r >> U0) & 1) | (((r >> U1) & 1) << 1);
    x[r] = cmul<PREC>(b == 0 ? d0 : b == 1 ? d1 : b == 2 ? d2 : d3, x[r]);
  }
  variant_end<PREC, 48 + U0 * 4 + U1>();
}

// x[r] *= d_b, b = bit0 + 2 bit1 of the diagonal's index.  Bit j is register
// bit k_j of r (k_j in 0..3), or, for k_j < 0, the constant bit j of c.  All
// selections are per gate and thread, none per element.
template <int PREC>
__device__ __forceinline__ void apply_diag(float2 (&x)[16], int n, int k0, int k1, int c, float2 d0, float2 d1, float2 d2,
                                  float2 d3) {
  if (n == 2 && k0 >= 0 && k1 >= 0) {
    switch (k0 * 4 + k1) {
      case 1: diag_reg2<PREC, 0, 1>(x, d0, d1, d2, d3); break;
      case 2: diag_reg2<PREC, 0, 2>(x, d0, d1, d2, d3); break;
      case 3: diag_reg2<PREC, 0, 3>(x, d0, d1, d2, d3); break;
      case 4: diag_reg2<PREC, 1, 0>(x, d0, d1, d2, d3); break;
      case 6: diag_reg2<PREC, 1, 2>(x, d0, d1, d2, d3); break;
      case 7: diag_reg2<PREC, 1, 3>(x, d0, d1, d2, d3); break;
      case 8: diag_reg2<PREC, 2, 0>(x, d0, d1, d2, d3); break;
      case 9: diag_reg2<PREC, 2, 1>(x, d0, d1, d2, d3); break;
      case 11: diag_reg2<PREC, 2, 3>(x, d0, d1, d2, d3); break;
      case 12: diag_reg2<PREC, 3, 0>(x, d0, d1, d2, d3); break;
      case 13: diag_reg2<PREC, 3, 1>(x, d0, d1, d2, d3); break;
      default: diag_reg2<PREC, 3, 2>(x, d0, d1, d2, d3); break;
    }
    return;
  }
  int k = -1;
  float2 e0, e1;
  if (n == 2 && k0 >= 0) {  // bit 1 constant
    k = k0;
    e0 = (c & 2) ? d2 : d0;
    e1 = (c & 2) ? d3 : d1;
  } else if (n == 2 && k1 >= 0) {  // bit 0 constant
    k = k1;
    e0 = (c & 1) ? d1 : d0;
    e1 = (c & 1) ? d3 : d2;
  } else if (n == 1 && k0 >= 0) {
    k = k0;
    e0 = d0;
    e1 = d1;
  }
  if (k < 0) {  // constant over the thread's elements
    const float2 f = c == 0 ? d0 : c == 1 ? d1 : c == 2 ? d2 : d3;
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = cmul<PREC>(f, x[r]);
    return;
  }
  switch (k) {
    case 0: diag_reg1<PREC, 0>(x, e0, e1); break;
    case 1: diag_reg1<PREC, 1>(x, e0, e1); break;
    case 2: diag_reg1<PREC, 2>(x, e0, e1); break;
    default: diag_reg1<PREC, 3>(x, e0, e1); break;
  }
}

// Unit-modulus diagonals with the entry of index 0 factored out: the caller
// multiplies d0 into the thread's deferred phase, and only the elements whose
// index is not 0 are multiplied, by d_b conj(d0); an entry whose ratio is
// exactly 1 (the ZZ phase diag(1, e, e, 1) has d3 = d0) is skipped.
// (NS = 2: the same factors on a second state y)
template <int PREC, int NS, int U0, int U1>
__device__ __forceinline__ void diag_reg2_rel(float2 (&x)[16], float2 (&y)[16], float2 q1, float2 q2, float2 q3,
                                              int skip) {
  const bool s1 = (skip >> 1) & 1, s2 = (skip >> 2) & 1, s3 = (skip >> 3) & 1;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int b = ((r >> U0) & 1) | (((r >> U1) & 1) << 1);  // compile-time per r
    if (b == 0 || (b == 1 && s1) || (b == 2 && s2) || (b == 3 && s3)) continue;
    const float2 q = b == 1 ? q1 : b == 2 ? q2 : q3;
    x[r] = cmul<PREC>(q, x[r]);
    if (NS == 2) y[r] = cmul<PREC>(q, y[r]);
  }
  variant_end<PREC, 64 + NS * 16 + U0 * 4 + U1>();
}
template <int PREC, int NS, int U>
__device__ __forceinline__ void diag_reg1_rel(float2 (&x)[16], float2 (&y)[16], float2 q1) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if ((r >> U) & 1) {
      x[r] = cmul<PREC>(q1, x[r]);
      if (NS == 2) y[r] = cmul<PREC>(q1, y[r]);
    }
  variant_end<PREC, 112 + NS * 4 + U>();
}
__device__ inline bool is_one(float2 v) { return v.x == 1.f && v.y == 0.f; }

// x[r] *= d_b (unit-modulus entries) as ph *= d_{b0} and x[r] *= d_b conj(d_{b0}),
// b0 the index value of r = 0 (bits as in apply_diag: register bits k_j, else
// bit j of c).  Returns with nothing done to x when no bit is a register bit.
template <int PREC, int NS>
__device__ __forceinline__ void apply_diag_unit(float2 (&x)[16], float2 (&y)[16], float2& ph, int n, int k0, int k1,
                                                int c, float2 d0, float2 d1, float2 d2, float2 d3) {
  auto rel = [](float2 d, float2 base) { return cmul<TN_PREC_C64>(d, f2(base.x, -base.y)); };
  auto mulph = [&](float2 f) { ph = cmul<TN_PREC_C64>(ph, f); };
  if (n == 2 && k0 >= 0 && k1 >= 0) {
    mulph(d0);
    const float2 q1 = rel(d1, d0), q2 = rel(d2, d0), q3 = rel(d3, d0);
    const int skip = (is_one(q1) << 1) | (is_one(q2) << 2) | (is_one(q3) << 3);
    switch (k0 * 4 + k1) {
      case 1: diag_reg2_rel<PREC, NS, 0, 1>(x, y, q1, q2, q3, skip); break;
      case 2: diag_reg2_rel<PREC, NS, 0, 2>(x, y, q1, q2, q3, skip); break;
      case 3: diag_reg2_rel<PREC, NS, 0, 3>(x, y, q1, q2, q3, skip); break;
      case 4: diag_reg2_rel<PREC, NS, 1, 0>(x, y, q1, q2, q3, skip); break;
      case 6: diag_reg2_rel<PREC, NS, 1, 2>(x, y, q1, q2, q3, skip); break;
      case 7: diag_reg2_rel<PREC, NS, 1, 3>(x, y, q1, q2, q3, skip); break;
      case 8: diag_reg2_rel<PREC, NS, 2, 0>(x, y, q1, q2, q3, skip); break;
      case 9: diag_reg2_rel<PREC, NS, 2, 1>(x, y, q1, q2, q3, skip); break;
      case 11: diag_reg2_rel<PREC, NS, 2, 3>(x, y, q1, q2, q3, skip); break;
      case 12: diag_reg2_rel<PREC, NS, 3, 0>(x, y, q1, q2, q3, skip); break;
      case 13: diag_reg2_rel<PREC, NS, 3, 1>(x, y, q1, q2, q3, skip); break;
      default: diag_reg2_rel<PREC, NS, 3, 2>(x, y, q1, q2, q3, skip); break;
    }
    return;
  }
  int k = -1;
  float2 e0, e1;
  if (n == 2 && k0 >= 0) {  // bit 1 constant
    k = k0;
    e0 = (c & 2) ? d2 : d0;
    e1 = (c & 2) ? d3 : d1;
  } else if (n == 2 && k1 >= 0) {  // bit 0 constant
    k = k1;
    e0 = (c & 1) ? d1 : d0;
    e1 = (c & 1) ? d3 : d2;
  } else if (n == 1 && k0 >= 0) {
    k = k0;
    e0 = d0;
    e1 = d1;
  }
  if (k < 0) return;
  mulph(e0);
  const float2 q1 = rel(e1, e0);
  switch (k) {
    case 0: diag_reg1_rel<PREC, NS, 0>(x, y, q1); break;
    case 1: diag_reg1_rel<PREC, NS, 1>(x, y, q1); break;
    case 2: diag_reg1_rel<PREC, NS, 2>(x, y, q1); break;
    default: diag_reg1_rel<PREC, NS, 3>(x, y, q1); break;
  }
}

// A run of one-bit unit diagonal gates on the register bits of mask M, in
// increasing bit order, each already split as in apply_diag_unit (its first
// entry joined the deferred phase; q[k]: the k-th gate's second entry relative
// to its first): straight-line code, without the gate loop's copy per gate.
template <int PREC, int NS, int M>
__device__ __forceinline__ void diag_run_m(float2 (&x)[16], float2 (&y)[16], const float2 (&q)[4]) {
  int k = 0;
  if constexpr ((M & 1) != 0) diag_reg1_rel<PREC, NS, 0>(x, y, q[k++]);
  if constexpr ((M & 2) != 0) diag_reg1_rel<PREC, NS, 1>(x, y, q[k++]);
  if constexpr ((M & 4) != 0) diag_reg1_rel<PREC, NS, 2>(x, y, q[k++]);
  if constexpr ((M & 8) != 0) diag_reg1_rel<PREC, NS, 3>(x, y, q[k]);
  variant_end<PREC, 500 + NS * 16 + M>();
}

template <int PREC, int NS>
__device__ __forceinline__ void diag_run(float2 (&x)[16], float2 (&y)[16], const float2 (&q)[4], int mask) {
  switch (mask) {
    case 3: diag_run_m<PREC, NS, 3>(x, y, q); break;
    case 5: diag_run_m<PREC, NS, 5>(x, y, q); break;
    case 6: diag_run_m<PREC, NS, 6>(x, y, q); break;
    case 7: diag_run_m<PREC, NS, 7>(x, y, q); break;
    case 9: diag_run_m<PREC, NS, 9>(x, y, q); break;
    case 10: diag_run_m<PREC, NS, 10>(x, y, q); break;
    case 11: diag_run_m<PREC, NS, 11>(x, y, q); break;
    case 12: diag_run_m<PREC, NS, 12>(x, y, q); break;
    case 13: diag_run_m<PREC, NS, 13>(x, y, q); break;
    case 14: diag_run_m<PREC, NS, 14>(x, y, q); break;
    default: diag_run_m<PREC, NS, 15>(x, y, q); break;
  }
}

// The thread's elements that a diagonal with entries +-1 negates, as a 16-bit
// mask over the register combinations r: entry b (bit 0 from register bit k0
// or constant bit 0 of c, bit 1 likewise from k1 or c) is -1 where bit b of
// `signs` is set, as in apply_signs.
__device__ __forceinline__ int sign_pattern(int n, int k0, int k1, int c, int signs) {
  auto ones = [](int k) { return k == 0 ? 0xAAAA : k == 1 ? 0xCCCC : k == 2 ? 0xF0F0 : 0xFF00; };
  const int A = k0 >= 0 ? ones(k0) : ((c & 1) ? 0xFFFF : 0);
  const int B = n == 2 ? (k1 >= 0 ? ones(k1) : ((c & 2) ? 0xFFFF : 0)) : 0;
  int m = 0;
  if (signs & 1) m |= ~A & ~B;
  if (signs & 2) m |= A & ~B;
  if (signs & 4) m |= ~A & B;
  if (signs & 8) m |= A & B;
  return m & 0xFFFF;
}

// x[r] = -x[r] where bit r of m is set (sign-bit flips, no multiplies)
__device__ __forceinline__ void flip_signs(float2 (&x)[16], int m) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const unsigned s = (unsigned)((m >> r) & 1) << 31;
    x[r] = f2(__uint_as_float(__float_as_uint(x[r].x) ^ s), __uint_as_float(__float_as_uint(x[r].y) ^ s));
  }
}

// Sign mask of a diagonal whose used entries are all +1 or -1 (CZ, Z), or -1.
__device__ __forceinline__ int sign_mask(int n, float2 d0, float2 d1, float2 d2, float2 d3) {
  auto pm1 = [](float2 d) { return d.y == 0.f && fabsf(d.x) == 1.f; };
  const bool two = n == 2;
  if (!pm1(d0) || !pm1(d1) || (two && (!pm1(d2) || !pm1(d3)))) return -1;
  return (d0.x < 0.f) | ((d1.x < 0.f) << 1) | (two ? ((d2.x < 0.f) << 2) | ((d3.x < 0.f) << 3) : 0);
}

// x[r] = -x[r] where the diagonal's entry b is -1 (bit b of mask), b resolved as in apply_diag
template <int U>
__device__ __forceinline__ void signs_reg1(float2 (&x)[16], int m01) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if ((m01 >> ((r >> U) & 1)) & 1) x[r] = f2(-x[r].x, -x[r].y);
}
template <int U0, int U1>
__device__ __forceinline__ void signs_reg2(float2 (&x)[16], int mask) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int b = ((r >> U0) & 1) | (((r >> U1) & 1) << 1);
    if ((mask >> b) & 1) x[r] = f2(-x[r].x, -x[r].y);
  }
}
__device__ __forceinline__ void apply_signs(float2 (&x)[16], int n, int k0, int k1, int c, int mask) {
  if (n == 2 && k0 >= 0 && k1 >= 0) {
    switch (k0 * 4 + k1) {
      case 1: signs_reg2<0, 1>(x, mask); break;
      case 2: signs_reg2<0, 2>(x, mask); break;
      case 3: signs_reg2<0, 3>(x, mask); break;
      case 4: signs_reg2<1, 0>(x, mask); break;
      case 6: signs_reg2<1, 2>(x, mask); break;
      case 7: signs_reg2<1, 3>(x, mask); break;
      case 8: signs_reg2<2, 0>(x, mask); break;
      case 9: signs_reg2<2, 1>(x, mask); break;
      case 11: signs_reg2<2, 3>(x, mask); break;
      case 12: signs_reg2<3, 0>(x, mask); break;
      case 13: signs_reg2<3, 1>(x, mask); break;
      default: signs_reg2<3, 2>(x, mask); break;
    }
    return;
  }
  int k = -1, m01 = 0;  // signs of the register bit's two values
  if (n == 2 && k0 >= 0) {
    k = k0;
    m01 = (c & 2) ? (mask >> 2) & 3 : mask & 3;
  } else if (n == 2 && k1 >= 0) {
    k = k1;
    m01 = (c & 1) ? ((mask >> 1) & 1) | (((mask >> 3) & 1) << 1) : (mask & 1) | (((mask >> 2) & 1) << 1);
  } else if (n == 1 && k0 >= 0) {
    k = k0;
    m01 = mask & 3;
  }
  if (k < 0) {
    if ((mask >> c) & 1)
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = f2(-x[r].x, -x[r].y);
    return;
  }
  switch (k) {
    case 0: signs_reg1<0>(x, m01); break;
    case 1: signs_reg1<1>(x, m01); break;
    case 2: signs_reg1<2>(x, m01); break;
    default: signs_reg1<3>(x, m01); break;
  }
}


// A count group: x[r] *= w^cut(r), cut(r) the number of the group's E member
// edges whose two bits differ at the thread's element r.  An edge between
// two bits outside the registers adds a per-thread constant; an edge from
// register bit j to a constant bit b adds 1 where bit j of r differs from b;
// an edge between register bits j and k (the same for every thread) adds 1
// where they differ.  The powers come from the pass's LDS table tab.
__device__ __forceinline__ int count_pair(int j, int k) {  // 0..5 for the unordered pairs of 0..3
  const int lo = j < k ? j : k, hi = j < k ? k : j;
  return lo == 0 ? hi - 1 : lo == 1 ? hi + 1 : 5;
}
template <int PREC>
__device__ __forceinline__ void apply_count_group(float2 (&x)[16], const SweepGateDesc* __restrict__ m, int E, int ob,
                                                  int64_t base, const float2* tab) {
  int K = 0;                  // constant edges that differ
  uint32_t to0 = 0, to1 = 0;  // per register bit j (8-bit fields): edges to a constant 0 / 1
  uint64_t pr = 0;            // per register-bit pair (8-bit fields): edges between two register bits
  for (int e = 0; e < E; ++e) {
    const int k0 = m[e].kreg[0], k1 = m[e].kreg[1];
    auto cbit = [&](int j) {
      const int cs = m[e].csrc[j];
      return cs >= 64 ? (int)((base >> (cs - 64)) & 1) : ((ob >> cs) & 1);
    };
    if (k0 < 0 && k1 < 0) {
      K += cbit(0) ^ cbit(1);
    } else if (k0 >= 0 && k1 >= 0) {
      pr += (uint64_t)1 << (8 * count_pair(k0, k1));
    } else {
      const int j = k0 >= 0 ? k0 : k1;
      if (cbit(k0 >= 0 ? 1 : 0)) to1 += 1u << (8 * j);
      else to0 += 1u << (8 * j);
    }
  }
  // partial sums over register bits {0, 1} and {2, 3}: where bit j is set the edges to a
  // constant 0 differ, where it is clear those to a constant 1
  int s01[4], s23[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    s01[b] = K + (int)(((b & 1 ? to0 : to1) >> 0) & 255) + (int)(((b & 2 ? to0 : to1) >> 8) & 255);
    s23[b] = (int)(((b & 1 ? to0 : to1) >> 16) & 255) + (int)(((b & 2 ? to0 : to1) >> 24) & 255);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    int pc = 0;  // register-register edges that differ at r (the same for every thread)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = j + 1; k < 4; ++k)
        if (((r >> j) ^ (r >> k)) & 1) pc += (int)((pr >> (8 * count_pair(j, k))) & 255);
    x[r] = cmul<PREC>(tab[s01[r & 3] + s23[r >> 2] + pc], x[r]);
  }
}

// Fused adjoint pass (see AdjGateDesc).  Two chunks (psi and lambda) in LDS;
// per segment each thread holds 16 elements of each in registers.
struct AdjPassArgs {
  float2* psi;
  float2* lam;
  int64_t psi_bs, lam_bs;
  const float2* U;
  int64_t u_bs;
  const AdjGateDesc* gates;
  const SweepSegment* segs;
  double* partials;
  int64_t pstride;
  int64_t n_chunks;
  int32_t n_segs, l, n_rest, n_red;
  int32_t first_gate, n_gates;
  int8_t lpos[kSweepMaxLocal];
  int8_t rest[64];
};
static_assert(offsetof(AdjPassArgs, lpos) % 4 == 0 && offsetof(AdjPassArgs, rest) % 4 == 0,
              "position maps aligned to 32-bit words");

__device__ inline float im_conj_mul(float2 l, float2 q) { return l.x * q.y - l.y * q.x; }
__device__ inline float2 cmulf(float2 a, float2 b) { return f2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }

// sum over the register pairs along bit U of Im(conj(l_m) (G p)_m)
template <int U>
__device__ __forceinline__ float reg_grad1(const float2 (&p)[16], const float2 (&l)[16], const float2* G) {
  float g = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r & (1 << U)) continue;
    const int r1 = r | (1 << U);
    const float2 q0 = f2(G[0].x * p[r].x - G[0].y * p[r].y + G[1].x * p[r1].x - G[1].y * p[r1].y,
                         G[0].x * p[r].y + G[0].y * p[r].x + G[1].x * p[r1].y + G[1].y * p[r1].x);
    const float2 q1 = f2(G[2].x * p[r].x - G[2].y * p[r].y + G[3].x * p[r1].x - G[3].y * p[r1].y,
                         G[2].x * p[r].y + G[2].y * p[r].x + G[3].x * p[r1].y + G[3].y * p[r1].x);
    g += im_conj_mul(l[r], q0) + im_conj_mul(l[r1], q1);
  }
  return g;
}

// Sum over the 16 register elements of q_b Im(conj(l) p), b resolved as in
// apply_diag (the diagonal generators Z, 1 - ZZ and |11><11| are real)
template <int U>
__device__ __forceinline__ float dgrad_reg1(const float2 (&p)[16], const float2 (&l)[16], float e0, float e1) {
  float g = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) g += ((r >> U) & 1 ? e1 : e0) * im_conj_mul(l[r], p[r]);
  return g;
}
template <int U0, int U1>
__device__ __forceinline__ float dgrad_reg2(const float2 (&p)[16], const float2 (&l)[16], float q0, float q1, float q2,
                                   float q3) {
  float g = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int b = ((r >> U0) & 1) | (((r >> U1) & 1) << 1);
    g += (b == 0 ? q0 : b == 1 ? q1 : b == 2 ? q2 : q3) * im_conj_mul(l[r], p[r]);
  }
  return g;
}
__device__ __forceinline__ float diag_grad(const float2 (&p)[16], const float2 (&l)[16], int n, int k0, int k1, int c,
                                  float q0, float q1, float q2, float q3) {
  if (n == 2 && k0 >= 0 && k1 >= 0) {
    switch (k0 * 4 + k1) {
      case 1: return dgrad_reg2<0, 1>(p, l, q0, q1, q2, q3);
      case 2: return dgrad_reg2<0, 2>(p, l, q0, q1, q2, q3);
      case 3: return dgrad_reg2<0, 3>(p, l, q0, q1, q2, q3);
      case 4: return dgrad_reg2<1, 0>(p, l, q0, q1, q2, q3);
      case 6: return dgrad_reg2<1, 2>(p, l, q0, q1, q2, q3);
      case 7: return dgrad_reg2<1, 3>(p, l, q0, q1, q2, q3);
      case 8: return dgrad_reg2<2, 0>(p, l, q0, q1, q2, q3);
      case 9: return dgrad_reg2<2, 1>(p, l, q0, q1, q2, q3);
      case 11: return dgrad_reg2<2, 3>(p, l, q0, q1, q2, q3);
      case 12: return dgrad_reg2<3, 0>(p, l, q0, q1, q2, q3);
      case 13: return dgrad_reg2<3, 1>(p, l, q0, q1, q2, q3);
      default: return dgrad_reg2<3, 2>(p, l, q0, q1, q2, q3);
    }
  }
  int k = -1;
  float e0 = 0.f, e1 = 0.f;
  if (n == 2 && k0 >= 0) {
    k = k0;
    e0 = (c & 2) ? q2 : q0;
    e1 = (c & 2) ? q3 : q1;
  } else if (n == 2 && k1 >= 0) {
    k = k1;
    e0 = (c & 1) ? q1 : q0;
    e1 = (c & 1) ? q3 : q2;
  } else if (n == 1 && k0 >= 0) {
    k = k0;
    e0 = q0;
    e1 = q1;
  }
  if (k < 0) {
    const float f = c == 0 ? q0 : c == 1 ? q1 : c == 2 ? q2 : q3;
    float g = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) g += im_conj_mul(l[r], p[r]);
    return f * g;
  }
  switch (k) {
    case 0: return dgrad_reg1<0>(p, l, e0, e1);
    case 1: return dgrad_reg1<1>(p, l, e0, e1);
    case 2: return dgrad_reg1<2>(p, l, e0, e1);
    default: return dgrad_reg1<3>(p, l, e0, e1);
  }
}

// dense generators: c X (gradient c [Im(conj(l0) p1) + Im(conj(l1) p0)]) and Y
template <int U>
__device__ __forceinline__ float reg_grad_x(const float2 (&p)[16], const float2 (&l)[16], float c) {
  float g = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r & (1 << U)) continue;
    const int r1 = r | (1 << U);
    g += im_conj_mul(l[r], p[r1]) + im_conj_mul(l[r1], p[r]);
  }
  return c * g;
}
template <int U>
__device__ __forceinline__ float reg_grad_y(const float2 (&p)[16], const float2 (&l)[16]) {
  float g = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r & (1 << U)) continue;
    const int r1 = r | (1 << U);
    // Y p = (-i p1, i p0): Im(conj(l0)(-i p1)) + Im(conj(l1)(i p0)) = -Re(conj(l0) p1) + Re(conj(l1) p0)
    g += (l[r1].x * p[r].x + l[r1].y * p[r].y) - (l[r].x * p[r1].x + l[r].y * p[r1].y);
  }
  return g;
}

// Sum over the 64 lanes of a wave, the result in lane 63: DPP moves within
// quads, half rows and rows, then the row broadcasts of lane 15 and lane 31
// (six dependent VALU operations; a shuffle network would wait on LDS at each
// of its six steps).
__device__ __forceinline__ float wave_sum_to_63(float v) {
  auto dpp = [](float x, int ctrl, int row_mask) -> float {
    switch (ctrl) {  // the control word must be a compile-time constant
      case 0xb1: return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xb1, 0xf, 0xf, false));
      case 0x4e: return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4e, 0xf, 0xf, false));
      case 0x141: return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xf, 0xf, false));
      case 0x140: return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xf, 0xf, false));
      case 0x142: return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x142, 0xa, 0xf, false));
      default: return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x143, 0xc, 0xf, false));
    }
  };
  v += dpp(v, 0xb1, 0xf);   // quad_perm [1, 0, 3, 2]
  v += dpp(v, 0x4e, 0xf);   // quad_perm [2, 3, 0, 1]
  v += dpp(v, 0x141, 0xf);  // row_half_mirror
  v += dpp(v, 0x140, 0xf);  // row_mirror: every lane of a row holds the row's sum
  v += dpp(v, 0x142, 0xa);  // row_bcast:15 into rows 1 and 3
  v += dpp(v, 0x143, 0xc);  // row_bcast:31 into rows 2 and 3: lane 63 holds the total
  return v;
}

// One gate of a run of dense one-qubit gates in the reverse sweep (see
// run_apply): its gradient term from the states as they stand, then
// U^dagger on register bit R of both states, R and U's form F fixed.
template <int PREC, int R, int F, class AddGrad>
__device__ __forceinline__ void adj_run_slot(float2 (&xp)[16], float2 (&xl)[16], const AdjGateDesc& gd,
                                             const float2* Up, AddGrad& add_grad) {
  if (gd.red >= 0) {
    const float2* G = reinterpret_cast<const float2*>(gd.gen);
    const float g = gd.form == ADJ_GEN_X ? reg_grad_x<R>(xp, xl, G[2].x)
                    : gd.form == ADJ_GEN_Y ? reg_grad_y<R>(xp, xl)
                                           : reg_grad1<R>(xp, xl, G);
    add_grad(gd.red, g);
  }
  // U^dagger[m][k] = conj(U[k][m])
  const float2 ud[4] = {f2(Up[0].x, -Up[0].y), f2(Up[2].x, -Up[2].y), f2(Up[1].x, -Up[1].y), f2(Up[3].x, -Up[3].y)};
  reg_apply1<PREC, R, F>(xp, ud);
  reg_apply1<PREC, R, F>(xl, ud);
}

// The run of mask M: its k-th gate (descriptor gd[k], U entries Up[k]) on the k-th bit of M.
template <int PREC, int M, int F, class AddGrad>
__device__ __forceinline__ void adj_run(float2 (&xp)[16], float2 (&xl)[16], const AdjGateDesc* gd,
                                        const float2 (*Up)[4], AddGrad& add_grad) {
  int k = 0;
  if constexpr ((M & 1) != 0) { adj_run_slot<PREC, 0, F>(xp, xl, gd[k], Up[k], add_grad); ++k; }
  if constexpr ((M & 2) != 0) { adj_run_slot<PREC, 1, F>(xp, xl, gd[k], Up[k], add_grad); ++k; }
  if constexpr ((M & 4) != 0) { adj_run_slot<PREC, 2, F>(xp, xl, gd[k], Up[k], add_grad); ++k; }
  if constexpr ((M & 8) != 0) adj_run_slot<PREC, 3, F>(xp, xl, gd[k], Up[k], add_grad);
  variant_end<PREC, 400 + M * 4 + F>();
}

template <int PREC, class AddGrad>
__device__ __forceinline__ void adj_apply_run(float2 (&xp)[16], float2 (&xl)[16], const AdjGateDesc* gd,
                                              const float2 (*Up)[4], AddGrad& add_grad, int mask, int form) {
#define TNQ_ADJ_RUN(M)                                                                              \
  case M * 3 + kDenseGeneric: adj_run<PREC, M, kDenseGeneric>(xp, xl, gd, Up, add_grad); break; \
  case M * 3 + kDenseReal: adj_run<PREC, M, kDenseReal>(xp, xl, gd, Up, add_grad); break;       \
  case M * 3 + kDenseRxLike: adj_run<PREC, M, kDenseRxLike>(xp, xl, gd, Up, add_grad); break;
  switch (mask * 3 + (PREC == TN_PREC_C64 ? form : kDenseGeneric)) {
    TNQ_ADJ_RUN(3) TNQ_ADJ_RUN(5) TNQ_ADJ_RUN(6) TNQ_ADJ_RUN(7) TNQ_ADJ_RUN(9) TNQ_ADJ_RUN(10) TNQ_ADJ_RUN(11)
    TNQ_ADJ_RUN(12) TNQ_ADJ_RUN(13) TNQ_ADJ_RUN(14)
    default: adj_run<PREC, 15, kDenseGeneric>(xp, xl, gd, Up, add_grad); break;  // mask 15, generic form
    case 15 * 3 + kDenseReal: adj_run<PREC, 15, kDenseReal>(xp, xl, gd, Up, add_grad); break;
    case 15 * 3 + kDenseRxLike: adj_run<PREC, 15, kDenseRxLike>(xp, xl, gd, Up, add_grad); break;
  }
#undef TNQ_ADJ_RUN
}

}  // namespace tnq

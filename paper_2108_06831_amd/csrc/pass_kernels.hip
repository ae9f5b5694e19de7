// Fused gate passes over a state (forward and adjoint).
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

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

// The descriptor and value tables come as separate __restrict__ arguments: the
// compiler may then read them with scalar loads (nothing the kernel writes can
// alias them) instead of vector memory loads on every gate.  VL: the gate
// values are read from their LDS copy (a compile-time choice: a pointer that
// may point to LDS or to global memory would be read with flat loads, whose
// latency every gate would wait on).
template <int PREC, bool VL>
__global__ __launch_bounds__(kThreads) void k_sweep_pass(SweepPassArgs a, const SweepGateDesc* __restrict__ gates,
                                                          const SweepSegment* __restrict__ segs,
                                                          const float2* __restrict__ vals) {
  __shared__ float2 buf[(1 << kSweepMaxLocal) + (1 << (kSweepMaxLocal - 5))];
  __shared__ int64_t dep_hi[1 << (kSweepMaxLocal - 5)];
  __shared__ float2 vtab[kPassValMax];  // see SweepPassArgs::lds_off
  const int z = blockIdx.y;
  const int64_t c = blockIdx.x;
  const int L = 1 << a.l;
  const int nt = blockDim.x, tid = threadIdx.x;
  const int64_t base = deposit(c, a.rest, a.n_rest);
  // address bits of local index bits 5.. (the five lowest local bits are address bits 0..4)
  for (int h = tid; h < (L >> 5); h += nt) dep_hi[h] = deposit((int64_t)h << 5, a.lpos, a.l);
  __syncthreads();
  const float2* in = a.in + (int64_t)z * a.in_bs;
  float2* out = a.out + (int64_t)z * a.out_bs;
  const float2* V0 = vals + (int64_t)z * a.vals_bs;
  for (int t = tid; t < a.lds_n; t += nt) vtab[t] = V0[a.lds_off + t];
  const float2* ctab = vtab + (a.ctab_off - a.lds_off);
  chunk_to_lds(buf, in, base, dep_hi, tid, nt);
  __syncthreads();
  for (int sg = 0; sg < a.n_segs; ++sg) {
    const SweepSegment& seg = segs[sg];
    // the thread's local bits outside the registers, and its slots (see SweepSegment)
    int ob = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t) ob |= ((tid >> t) & 1) << seg.tpos[t];
    const int pob = ob + (ob >> 5);
    float2 x[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = buf[pob + seg.physoff[r]];
    // diagonal factors that are the same for all of a thread's elements (every
    // bit of the gate outside the register set) commute with every gate of the
    // segment: they are multiplied into one per-thread factor, applied once
    float2 ph = f2(1.f, 0.f);
    bool ph_used = false;  // the same for the whole block: set where a gate's descriptor sends it to ph
    const int g_end = seg.first_gate + seg.n_gates;
    int gi = seg.first_gate;
    // the segment's leading diagonal gates with no bit in the registers (the
    // planner puts them first): only the per-thread factor changes, so this
    // loop carries no register elements (the main loop below copies them back
    // into place on every gate)
    for (; gi < g_end; ++gi) {
      const SweepGateDesc& gd = gates[gi];
      if (!gd.diag || gd.form == kFormCount || gd.form == kFormCountMember || gd.kreg[0] >= 0 ||
          (gd.n == 2 && gd.kreg[1] >= 0))
        break;
      const float2* V = VL ? vtab + (gd.voff - a.lds_off) : V0 + gd.voff;
      int cb = 0;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j >= gd.n) continue;
        const int cs = gd.csrc[j];
        cb |= (cs >= 64 ? (int)((base >> (cs - 64)) & 1) : ((ob >> cs) & 1)) << j;
      }
      const bool two = gd.n == 2;
      const float2 d0 = V[0], d1 = V[1], d2 = two ? V[2] : d0, d3 = two ? V[3] : d0;
      const float2 f = cb == 0 ? d0 : cb == 1 ? d1 : cb == 2 ? d2 : d3;
      ph_used = true;
      if (gd.form == kFormSigns) {
        if (f.x < 0.f) ph = f2(-ph.x, -ph.y);
      } else {
        ph = cmul<TN_PREC_C64>(ph, f);
      }
    }
    for (; gi < g_end; ++gi) {
      const SweepGateDesc& gd = gates[gi];
      const float2* V = VL ? vtab + (gd.voff - a.lds_off) : V0 + gd.voff;
      if (gd.form == kFormCount) {
        apply_count_group<PREC>(x, gates + gi + 1, gd.n, ob, base, ctab + gd.voff);
        gi += gd.n;
        continue;
      }
      if (gd.diag && gd.run_mask && gd.form == kFormSigns) {  // run_mask gates with entries +-1
        int m = 0;
        for (int j = 0; j < gd.run_mask; ++j) {
          const SweepGateDesc& gj = gates[gi + j];
          const float2* Vj = VL ? vtab + (gj.voff - a.lds_off) : V0 + gj.voff;
          const bool two = gj.n == 2;
          const int sm = (Vj[0].x < 0.f) | ((Vj[1].x < 0.f) << 1) | (two ? ((Vj[2].x < 0.f) << 2) | ((Vj[3].x < 0.f) << 3) : 0);
          int cb = 0;
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            if (t >= gj.n || gj.kreg[t] >= 0) continue;
            const int cs = gj.csrc[t];
            cb |= (cs >= 64 ? (int)((base >> (cs - 64)) & 1) : ((ob >> cs) & 1)) << t;
          }
          m ^= sign_pattern(gj.n, gj.kreg[0], two ? gj.kreg[1] : -1, cb, sm);
        }
        flip_signs(x, m);
        gi += gd.run_mask - 1;
        continue;
      }
      if (gd.diag && gd.run_mask) {  // one-bit unit diagonals on the mask's register bits, in bit order
        const int cnt = __builtin_popcount(gd.run_mask);
        float2 q[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int vo = j < cnt ? gates[gi + j].voff : gd.voff;
          const float2* Vj = VL ? vtab + (vo - a.lds_off) : V0 + vo;
          const float2 e0 = Vj[0], e1 = Vj[1];
          if (j < cnt) ph = cmul<TN_PREC_C64>(ph, e0);
          q[j] = cmul<TN_PREC_C64>(e1, f2(e0.x, -e0.y));
        }
        ph_used = true;
        diag_run<PREC, 1>(x, x, q, gd.run_mask);
        gi += cnt - 1;
        continue;
      }
      if (gd.diag) {
        const bool two = gd.n == 2;
        const float2 d0 = V[0], d1 = V[1];
        const float2 d2 = two ? V[2] : f2(1.f, 0.f), d3 = two ? V[3] : f2(1.f, 0.f);
        const int k0 = gd.kreg[0], k1 = two ? gd.kreg[1] : -1;
        int cb = 0;  // the index bits that are constant over the thread's elements
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (j >= gd.n || gd.kreg[j] >= 0) continue;
          const int cs = gd.csrc[j];
          cb |= (cs >= 64 ? (int)((base >> (cs - 64)) & 1) : ((ob >> cs) & 1)) << j;
        }
        if (gd.form == kFormSigns) {  // entries +-1: sign flips, no multiplies
          const int sm = (d0.x < 0.f) | ((d1.x < 0.f) << 1) | ((d2.x < 0.f) << 2) | ((d3.x < 0.f) << 3);
          if (k0 < 0 && k1 < 0) {
            ph_used = true;
            if ((sm >> cb) & 1) ph = f2(-ph.x, -ph.y);
          } else {
            apply_signs(x, gd.n, k0, k1, cb, sm);
          }
        } else if (k0 < 0 && k1 < 0) {
          const float2 f = cb == 0 ? d0 : cb == 1 ? d1 : cb == 2 ? d2 : d3;
          ph = cmul<TN_PREC_C64>(ph, f);
          ph_used = true;
        } else if (gd.form == kFormUnit) {
          apply_diag_unit<PREC, 1>(x, x, ph, gd.n, k0, k1, cb, d0, d1, d2, d3);
          ph_used = true;
        } else {
          apply_diag<PREC>(x, gd.n, k0, k1, cb, d0, d1, d2, d3);
        }
      } else if (gd.n == 1) {
        const int form = gd.form == kFormReal ? kDenseReal : gd.form == kFormRxLike ? kDenseRxLike : kDenseGeneric;
        if (gd.run_mask) {  // this gate and the next ones: one per bit of the mask, one form
          const int cnt = __builtin_popcount(gd.run_mask);
          const float2* gp[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int vo = j < cnt ? gates[gi + j].voff : gd.voff;
            gp[j] = VL ? vtab + (vo - a.lds_off) : V0 + vo;
          }
          apply_dense1_run<PREC, 1>(x, x, gp, gd.run_mask, form);
          gi += cnt - 1;
          continue;
        }
        const float2 g[4] = {V[0], V[1], V[2], V[3]};
        apply_dense1<PREC, 1>(x, x, g, gd.rb[0], form);
      } else {
        float2 g[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) g[e] = V[e];
        switch (gd.rb[0] * 4 + gd.rb[1]) {
          case 1: reg_apply2<PREC, 0, 1>(x, g); break;
          case 2: reg_apply2<PREC, 0, 2>(x, g); break;
          case 3: reg_apply2<PREC, 0, 3>(x, g); break;
          case 6: reg_apply2<PREC, 1, 2>(x, g); break;
          case 7: reg_apply2<PREC, 1, 3>(x, g); break;
          default: reg_apply2<PREC, 2, 3>(x, g); break;
        }
      }
    }
    if (ph_used) {
#pragma unroll
      for (int r = 0; r < 16; ++r) buf[pob + seg.physoff[r]] = cmul<TN_PREC_C64>(ph, x[r]);
    } else {  // no gate of the segment touched the factor (it is 1)
#pragma unroll
      for (int r = 0; r < 16; ++r) buf[pob + seg.physoff[r]] = x[r];
    }
    __syncthreads();
  }
  chunk_from_lds(out, buf, base, dep_hi, tid, nt);
}

// The gate values of a chain's passes in one table (see SweepChain).
__global__ void k_gather_vals(const int64_t* src, int n, const float2* IN, int64_t in_bs, const float2* WS,
                              int64_t ws_bs, float2* out, int64_t out_bs) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int z = blockIdx.y;
  if (i >= n) return;
  const int64_t v = src[i];
  const int64_t off = v & (((int64_t)1 << kValExpShift) - 1);
  const float2* b = ((v >> 56) & 0x3f) == BUF_IN ? IN + (int64_t)z * in_bs : WS + (int64_t)z * ws_bs;
  float2 r = b[off];
  if (v & kValPow) {  // w^e by repeated multiplication in FP64, rounded once
    const int e = (int)((v >> kValExpShift) & 0xff);
    double pr = 1.0, pi = 0.0;
    for (int k = 0; k < e; ++k) {
      const double t = pr * r.x - pi * r.y;
      pi = pr * r.y + pi * r.x;
      pr = t;
    }
    r = f2((float)pr, (float)pi);
  }
  out[(int64_t)z * out_bs + i] = r;
}

hipError_t launch_gather_vals(hipStream_t s, const int64_t* src, int n, const float2* IN, int64_t in_bs,
                              const float2* WS, int64_t ws_bs, float2* out, int64_t out_bs, int batch) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_vals, dim3((unsigned)((n + kThreads - 1) / kThreads), batch), dim3(kThreads), 0, s,
                     src, n, IN, in_bs, WS, ws_bs, out, out_bs);
  return hipGetLastError();
}

hipError_t launch_sweep_pass(hipStream_t s, const SweepPass& ps, int bits, const SweepGateDesc* gates_dev,
                             const SweepSegment* segs_dev, const float2* in, int64_t in_bs, float2* out,
                             int64_t out_bs, const float2* vals, int64_t vals_bs, int batch, int precision) {
  SweepPassArgs a;
  a.in = in; a.out = out; a.in_bs = in_bs; a.out_bs = out_bs;
  a.vals = vals; a.vals_bs = vals_bs;
  a.gates = gates_dev;
  a.segs = segs_dev + ps.first_seg;
  a.n_segs = ps.n_segs;
  a.l = ps.l;
  a.pad = 0;
  a.ctab_off = ps.ctab_off;
  const int n_all = ps.ctab_off + ps.ctab_n - ps.val_off;  // the pass's values and tables
  a.gates_in_lds = n_all <= kPassValMax ? 1 : 0;
  a.lds_off = a.gates_in_lds ? ps.val_off : ps.ctab_off;
  a.lds_n = a.gates_in_lds ? n_all : ps.ctab_n;
  a.pad2 = 0;
  if (ps.l < kSweepMinLocal || ps.l > kSweepMaxLocal) return hipErrorInvalidValue;
  if (ps.ctab_n < 0 || ps.ctab_n > kCountTabMax || n_all < 0 || (a.lds_n > 0 && !vals)) return hipErrorInvalidValue;
  static_assert(kCountTabMax <= kPassValMax, "the power tables alone always fit");
  std::vector<char> local(bits, 0);
  for (int j = 0; j < ps.l; ++j) {
    a.lpos[j] = ps.lpos[j];
    if (ps.lpos[j] < 0 || ps.lpos[j] >= bits || (j < 5 && ps.lpos[j] != j)) return hipErrorInvalidValue;
    local[ps.lpos[j]] = 1;
  }
  int nr = 0;
  for (int p = 0; p < bits; ++p)
    if (!local[p]) a.rest[nr++] = (int8_t)p;
  a.n_rest = nr;
  const int64_t chunks = (int64_t)1 << nr;
  if (chunks > ((int64_t)1 << 24)) return hipErrorInvalidValue;
  const int threads = 1 << (ps.l - 4);
  const dim3 grid((unsigned)chunks, batch);
  if (precision == TN_PREC_BF16X3) {
    if (a.gates_in_lds)
      hipLaunchKernelGGL((k_sweep_pass<TN_PREC_BF16X3, true>), grid, dim3(threads), 0, s, a, a.gates, a.segs, a.vals);
    else
      hipLaunchKernelGGL((k_sweep_pass<TN_PREC_BF16X3, false>), grid, dim3(threads), 0, s, a, a.gates, a.segs, a.vals);
  } else {
    if (a.gates_in_lds)
      hipLaunchKernelGGL((k_sweep_pass<TN_PREC_C64, true>), grid, dim3(threads), 0, s, a, a.gates, a.segs, a.vals);
    else
      hipLaunchKernelGGL((k_sweep_pass<TN_PREC_C64, false>), grid, dim3(threads), 0, s, a, a.gates, a.segs, a.vals);
  }
  return hipGetLastError();
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

template <int PREC>
__global__ __launch_bounds__(kThreads) void k_adjoint_pass(AdjPassArgs a, const AdjGateDesc* __restrict__ gates,
                                                            const SweepSegment* __restrict__ segs,
                                                            const float2* __restrict__ Uall) {
  constexpr int kBuf = (1 << kSweepMaxLocal) + (1 << (kSweepMaxLocal - 5));
  __shared__ float2 bp[kBuf], bl[kBuf];
  __shared__ int64_t dep_hi[1 << (kSweepMaxLocal - 5)];
  __shared__ double red[kAdjMaxRed][kThreads / 64];
  __shared__ float2 upre[kAdjPreGates][4];  // the entries of U the pass's first gates use (see below)
  const int z = blockIdx.y;
  const int L = 1 << a.l;
  const int nt = blockDim.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nw = nt >> 6;
  if (blockIdx.x >= a.n_chunks) {  // no chunk for this block: its partial of every gradient term is zero
    for (int gi = a.first_gate + tid; gi < a.first_gate + a.n_gates; gi += nt) {
      const AdjGateDesc& gd = gates[gi];
      if (gd.red >= 0 && gd.slot >= 0)
        a.partials[(int64_t)z * a.pstride + (int64_t)gd.slot * kReduceBlocks + blockIdx.x] = 0.0;
    }
    return;
  }
  const float2* Uz = Uall + (int64_t)z * a.u_bs;
  // U of the pass's gates (at most kAdjPreGates) staged in LDS, one load per thread, all in flight
  // together: diagonal U[0], U[3] (one bit) or U[0], U[5], U[10], U[15] (two bits); one-qubit dense
  // U[0..3]; two-qubit dense gates read U from memory
  for (int i = tid; i < a.n_gates * 4; i += nt) {
    const int g = i >> 2, e = i & 3;
    const AdjGateDesc& gd = gates[a.first_gate + g];
    const int idx = gd.diag ? (gd.n == 2 ? 5 * e : (e == 1 ? 3 : 0)) : e;
    upre[g][e] = Uz[(int64_t)gd.gate * 16 + idx];
  }
  for (int h = tid; h < (L >> 5); h += nt) dep_hi[h] = deposit((int64_t)h << 5, a.lpos, a.l);
  __syncthreads();
  float2* P = a.psi + (int64_t)z * a.psi_bs;
  float2* Lm = a.lam + (int64_t)z * a.lam_bs;
  // gradient sums of this wave in registers: lane j holds slot j (accA) and slot 64 + j (accB)
  double accA = 0.0, accB = 0.0;
  auto add_grad = [&](int slot, float v) {
    v = wave_sum_to_63(v);
    const double sv = (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
    const double add = lane == (slot & 63) ? sv : 0.0;  // selects only: no run-time choice of a register
    accA += slot < 64 ? add : 0.0;
    accB += slot < 64 ? 0.0 : add;
  };
  for (int64_t c = blockIdx.x; c < a.n_chunks; c += gridDim.x) {
    const int64_t base = deposit(c, a.rest, a.n_rest);
    chunk2_to_lds(bp, bl, P, Lm, base, dep_hi, tid, nt);
    __syncthreads();
    for (int sg = 0; sg < a.n_segs; ++sg) {
      const SweepSegment& seg = segs[sg];
      int ob = 0;
#pragma unroll
      for (int t = 0; t < 8; ++t) ob |= ((tid >> t) & 1) << seg.tpos[t];
      const int pob = ob + (ob >> 5);
      float2 xp[16], xl[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        xp[r] = bp[pob + seg.physoff[r]];
        xl[r] = bl[pob + seg.physoff[r]];
      }
      // unit-modulus diagonal factors that are the same for all of a thread's
      // elements go into one per-thread factor, applied to both states at the
      // segment's end; they commute with the segment's gates and leave every
      // gradient term Im<lambda|G|psi> unchanged (|factor|^2 = 1)
      float2 ph = f2(1.f, 0.f);
      bool ph_used = false;  // the same for the whole block (set by gates' descriptors)
      // Im(conj(lambda) psi) at each element is unchanged by unit-modulus diagonal gates, so
      // along a run of diagonal gates its sums are formed once: over the thread's elements
      // (tT) and over those whose register bit j is 1 (tS[j]); a one-bit diagonal generator's
      // term is then q0 (tT - s1) + q1 s1, s1 the sum where the gate's bit is 1
      bool have_t = false;
      float tT = 0.f, tS0 = 0.f, tS1 = 0.f, tS2 = 0.f, tS3 = 0.f;
      const int g_end = seg.first_gate + seg.n_gates;
      int gi = seg.first_gate;
      // the segment's leading diagonal gates with no bit in the registers (the planner puts
      // them first; they commute with the rest of the segment): their gradient terms need only
      // tT, and they change only ph, so this loop carries no register elements
      for (; gi < g_end; ++gi) {
        const AdjGateDesc& gd = gates[gi];
        if (!gd.diag || gd.kreg[0] >= 0 || (gd.n == 2 && gd.kreg[1] >= 0)) break;
        int c = 0;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (j >= gd.n) continue;
          const int cs = gd.csrc[j];
          c |= (cs >= 64 ? (int)((base >> (cs - 64)) & 1) : ((ob >> cs) & 1)) << j;
        }
        ph_used = true;
        if (gd.form & ADJ_DIAG_SIGNS) {
          if (((gd.form >> 8) >> c) & 1) ph = f2(-ph.x, -ph.y);
          continue;
        }
        const float2* Up = upre[gi - a.first_gate];
        if (gd.red >= 0) {
          if (!have_t) {
            tT = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) tT += im_conj_mul(xl[r], xp[r]);
            have_t = true;
          }
          const float* G = gd.gen;  // diagonal generator entries, re/im interleaved
          const float q = c == 0 ? G[0] : c == 1 ? G[2] : c == 2 ? G[4] : G[6];
          add_grad(gd.red, q * tT);
        }
        const bool two = gd.n == 2;
        const float2 u0 = Up[0], u1 = Up[1], u2 = two ? Up[2] : u0, u3 = two ? Up[3] : u0;
        const float2 u = c == 0 ? u0 : c == 1 ? u1 : c == 2 ? u2 : u3;  // U^dagger: conj(U[b][b])
        ph = cmul<TN_PREC_C64>(ph, f2(u.x, -u.y));
      }
      have_t = false;  // the main loop's sums also split tT by register bit
      for (; gi < g_end; ++gi) {
        const AdjGateDesc& gd = gates[gi];
        const float2* U = Uz + (int64_t)gd.gate * 16;
        const float2* G = reinterpret_cast<const float2*>(gd.gen);
        const float2* Up = upre[gi - a.first_gate];
        if (!gd.diag) have_t = false;
        if (gd.diag && gd.run_mask && (gd.form & ADJ_DIAG_SIGNS)) {  // run_mask gates with entries +-1
          // (U^dagger = U; no gradient terms; sign flips of both states leave Im(conj(l) p) as it was)
          int m = 0;
          for (int j = 0; j < gd.run_mask; ++j) {
            const AdjGateDesc& gj = gates[gi + j];
            const bool two = gj.n == 2;
            int cj = 0;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              if (t >= gj.n || gj.kreg[t] >= 0) continue;
              const int cs = gj.csrc[t];
              cj |= (cs >= 64 ? (int)((base >> (cs - 64)) & 1) : ((ob >> cs) & 1)) << t;
            }
            m ^= sign_pattern(gj.n, gj.kreg[0], two ? gj.kreg[1] : -1, cj, gj.form >> 8);
          }
          flip_signs(xp, m);
          flip_signs(xl, m);
          gi += gd.run_mask - 1;
          continue;
        }
        if (gd.diag && gd.run_mask) {  // one-bit unit diagonals on the mask's register bits, in bit order
          const int cnt = __builtin_popcount(gd.run_mask);
          // their gradient terms: a unit diagonal applied to both states leaves Im(conj(l) p)
          // unchanged, so the whole run shares one set of sums
          bool any_red = false;
#pragma unroll
          for (int j = 0; j < 4; ++j) any_red |= j < cnt && gates[gi + j].red >= 0;
          if (any_red && !have_t) {
            tT = tS0 = tS1 = tS2 = tS3 = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const float t = im_conj_mul(xl[r], xp[r]);
              tT += t;
              if (r & 1) tS0 += t;
              if (r & 2) tS1 += t;
              if (r & 4) tS2 += t;
              if (r & 8) tS3 += t;
            }
            have_t = true;
          }
          float2 q[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            q[j] = f2(1.f, 0.f);
            if (j >= cnt) continue;
            const AdjGateDesc& gj = gates[gi + j];  // the run's gates are in register-bit order
            if (gj.red >= 0) {
              const float2* Gj = reinterpret_cast<const float2*>(gj.gen);
              const int b = gj.kreg[0];
              const float s1 = b == 0 ? tS0 : b == 1 ? tS1 : b == 2 ? tS2 : tS3;
              add_grad(gj.red, Gj[0].x * (tT - s1) + Gj[1].x * s1);
            }
            // U^dagger: conj of the entries; the first joins the deferred phase
            const float2* Uj = upre[gi + j - a.first_gate];
            const float2 e0 = f2(Uj[0].x, -Uj[0].y), e1 = f2(Uj[1].x, -Uj[1].y);
            ph = cmul<TN_PREC_C64>(ph, e0);
            q[j] = cmul<TN_PREC_C64>(e1, f2(e0.x, -e0.y));
          }
          ph_used = true;
          diag_run<PREC, 2>(xp, xl, q, gd.run_mask);
          gi += cnt - 1;
          continue;
        }
        if (gd.diag) {
          const int k[2] = {gd.kreg[0], gd.n == 2 ? gd.kreg[1] : -1};
          int c = 0;  // the index bits that are constant over the thread's elements
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            if (j >= gd.n || gd.kreg[j] >= 0) continue;
            const int cs = gd.csrc[j];
            c |= (cs >= 64 ? (int)((base >> (cs - 64)) & 1) : ((ob >> cs) & 1)) << j;
          }
          const bool two = gd.n == 2;
          const bool uniform = k[0] < 0 && k[1] < 0;  // the same entry for every element of the thread
          if (gd.form & ADJ_DIAG_SIGNS) {  // Z, CZ: U^dagger = U, entries +-1
            if (uniform) {
              ph_used = true;
              if (((gd.form >> 8) >> c) & 1) ph = f2(-ph.x, -ph.y);
              continue;
            }
            apply_signs(xp, gd.n, k[0], k[1], c, gd.form >> 8);
            apply_signs(xl, gd.n, k[0], k[1], c, gd.form >> 8);
            continue;
          }
          // U^dagger diagonal: conj(U[b][b])
          const float2 u0 = Up[0], u1 = Up[1], u2 = two ? Up[2] : f2(1.f, 0.f), u3 = two ? Up[3] : f2(1.f, 0.f);
          if (gd.red >= 0) {
            float v;
            if (!two) {
              if (!have_t) {
                tT = tS0 = tS1 = tS2 = tS3 = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                  const float t = im_conj_mul(xl[r], xp[r]);
                  tT += t;
                  if (r & 1) tS0 += t;
                  if (r & 2) tS1 += t;
                  if (r & 4) tS2 += t;
                  if (r & 8) tS3 += t;
                }
                have_t = true;
              }
              const float s1 = k[0] >= 0 ? (k[0] == 0 ? tS0 : k[0] == 1 ? tS1 : k[0] == 2 ? tS2 : tS3) : (c ? tT : 0.f);
              v = G[0].x * (tT - s1) + G[1].x * s1;
            } else {
              v = diag_grad(xp, xl, gd.n, k[0], k[1], c, G[0].x, G[1].x, G[2].x, G[3].x);
            }
            add_grad(gd.red, v);
          }
          const float2 d0 = f2(u0.x, -u0.y), d1 = f2(u1.x, -u1.y), d2 = f2(u2.x, -u2.y), d3 = f2(u3.x, -u3.y);
          ph_used = true;
          if (uniform) {
            const float2 f = c == 0 ? d0 : c == 1 ? d1 : c == 2 ? d2 : d3;
            ph = cmul<TN_PREC_C64>(ph, f);
            continue;
          }
          // unitary gates: the entries have unit modulus, so the first one joins the deferred phase
          apply_diag_unit<PREC, 2>(xp, xl, ph, gd.n, k[0], k[1], c, d0, d1, d2, d3);
        } else if (gd.n == 1) {
          if (gd.run_mask) {  // this gate and the next ones: one per bit of the mask, one form of U
            const int f = gd.uform == kFormReal ? kDenseReal : gd.uform == kFormRxLike ? kDenseRxLike : kDenseGeneric;
            adj_apply_run<PREC>(xp, xl, gates + gi, upre + (gi - a.first_gate), add_grad, gd.run_mask, f);
            gi += __builtin_popcount(gd.run_mask) - 1;
            continue;
          }
          if (gd.red >= 0) {
            float g;
            if (gd.form == ADJ_GEN_X) {
              const float cx = G[2].x;
              switch (gd.rb[0]) {
                case 0: g = reg_grad_x<0>(xp, xl, cx); break;
                case 1: g = reg_grad_x<1>(xp, xl, cx); break;
                case 2: g = reg_grad_x<2>(xp, xl, cx); break;
                default: g = reg_grad_x<3>(xp, xl, cx); break;
              }
            } else if (gd.form == ADJ_GEN_Y) {
              switch (gd.rb[0]) {
                case 0: g = reg_grad_y<0>(xp, xl); break;
                case 1: g = reg_grad_y<1>(xp, xl); break;
                case 2: g = reg_grad_y<2>(xp, xl); break;
                default: g = reg_grad_y<3>(xp, xl); break;
              }
            } else {
              switch (gd.rb[0]) {
                case 0: g = reg_grad1<0>(xp, xl, G); break;
                case 1: g = reg_grad1<1>(xp, xl, G); break;
                case 2: g = reg_grad1<2>(xp, xl, G); break;
                default: g = reg_grad1<3>(xp, xl, G); break;
              }
            }
            add_grad(gd.red, g);
          }
          // U^dagger[m][k] = conj(U[k][m])
          const float2 w0 = Up[0], w1 = Up[1], w2 = Up[2], w3 = Up[3];
          float2 ud[4];
          ud[0] = f2(w0.x, -w0.y);
          ud[1] = f2(w2.x, -w2.y);
          ud[2] = f2(w1.x, -w1.y);
          ud[3] = f2(w3.x, -w3.y);
          const int form = gd.uform == kFormReal ? kDenseReal : gd.uform == kFormRxLike ? kDenseRxLike : kDenseGeneric;
          apply_dense1<PREC, 2>(xp, xl, ud, gd.rb[0], form);
        } else {
          // dense two-qubit gates carry no gradient term (the planner checks)
          float2 ud[16];
#pragma unroll
          for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int k = 0; k < 4; ++k) ud[4 * m + k] = f2(U[4 * k + m].x, -U[4 * k + m].y);
          switch (gd.rb[0] * 4 + gd.rb[1]) {
            case 1: reg_apply2<PREC, 0, 1>(xp, ud); reg_apply2<PREC, 0, 1>(xl, ud); break;
            case 4: reg_apply2<PREC, 1, 0>(xp, ud); reg_apply2<PREC, 1, 0>(xl, ud); break;
            case 2: reg_apply2<PREC, 0, 2>(xp, ud); reg_apply2<PREC, 0, 2>(xl, ud); break;
            case 8: reg_apply2<PREC, 2, 0>(xp, ud); reg_apply2<PREC, 2, 0>(xl, ud); break;
            case 3: reg_apply2<PREC, 0, 3>(xp, ud); reg_apply2<PREC, 0, 3>(xl, ud); break;
            case 12: reg_apply2<PREC, 3, 0>(xp, ud); reg_apply2<PREC, 3, 0>(xl, ud); break;
            case 6: reg_apply2<PREC, 1, 2>(xp, ud); reg_apply2<PREC, 1, 2>(xl, ud); break;
            case 9: reg_apply2<PREC, 2, 1>(xp, ud); reg_apply2<PREC, 2, 1>(xl, ud); break;
            case 7: reg_apply2<PREC, 1, 3>(xp, ud); reg_apply2<PREC, 1, 3>(xl, ud); break;
            case 13: reg_apply2<PREC, 3, 1>(xp, ud); reg_apply2<PREC, 3, 1>(xl, ud); break;
            case 11: reg_apply2<PREC, 2, 3>(xp, ud); reg_apply2<PREC, 2, 3>(xl, ud); break;
            default: reg_apply2<PREC, 3, 2>(xp, ud); reg_apply2<PREC, 3, 2>(xl, ud); break;
          }
        }
      }
      if (ph_used) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          bp[pob + seg.physoff[r]] = cmul<TN_PREC_C64>(ph, xp[r]);
          bl[pob + seg.physoff[r]] = cmul<TN_PREC_C64>(ph, xl[r]);
        }
      } else {  // no gate of the segment touched the factor (it is 1)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          bp[pob + seg.physoff[r]] = xp[r];
          bl[pob + seg.physoff[r]] = xl[r];
        }
      }
      __syncthreads();
    }
    chunk_from_lds(P, bp, base, dep_hi, tid, nt);
    chunk_from_lds(Lm, bl, base, dep_hi, tid, nt);
    __syncthreads();
  }
  red[lane][wv] = accA;
  red[64 + lane][wv] = accB;
  __syncthreads();
  // every (slot, block) entry of the pass's gates is written
  for (int gi = a.first_gate + tid; gi < a.first_gate + a.n_gates; gi += nt) {
    const AdjGateDesc& gd = gates[gi];
    if (gd.red < 0 || gd.slot < 0) continue;
    double v = 0;
    for (int w = 0; w < nw; ++w) v += red[gd.red][w];
    a.partials[(int64_t)z * a.pstride + (int64_t)gd.slot * kReduceBlocks + blockIdx.x] = v;
  }
}

hipError_t launch_adjoint_pass(hipStream_t s, const SweepPass& ps, int bits, const AdjGateDesc* gates_dev,
                               const SweepSegment* segs_dev, const float2* u, int64_t u_bs, float2* psi,
                               int64_t psi_bs, float2* lam, int64_t lam_bs, int batch, double* partials,
                               int64_t partial_stride, int precision) {
  AdjPassArgs a;
  a.psi = psi; a.lam = lam; a.psi_bs = psi_bs; a.lam_bs = lam_bs;
  a.U = u; a.u_bs = u_bs;
  a.gates = gates_dev;
  a.segs = segs_dev + ps.first_seg;
  a.partials = partials;
  a.pstride = partial_stride;
  a.n_segs = ps.n_segs;
  a.l = ps.l;
  a.n_red = ps.n_red;
  a.first_gate = ps.first_gate;
  a.n_gates = ps.n_gates;
  // 64 threads at least (whole waves for the gradient reductions), 256 at most
  if (ps.l < 10 || ps.l > kSweepMaxLocal || ps.n_red < 0 || ps.n_red > kAdjMaxRed || ps.n_gates < 0 ||
      ps.n_gates > kAdjPreGates)
    return hipErrorInvalidValue;
  std::vector<char> local(bits, 0);
  for (int j = 0; j < ps.l; ++j) {
    a.lpos[j] = ps.lpos[j];
    if (ps.lpos[j] < 0 || ps.lpos[j] >= bits || (j < 5 && ps.lpos[j] != j)) return hipErrorInvalidValue;
    local[ps.lpos[j]] = 1;
  }
  int nr = 0;
  for (int p = 0; p < bits; ++p)
    if (!local[p]) a.rest[nr++] = (int8_t)p;
  a.n_rest = nr;
  a.n_chunks = (int64_t)1 << nr;
  const int threads = 1 << (ps.l - 4);
  if (precision == TN_PREC_BF16X3)
    hipLaunchKernelGGL(k_adjoint_pass<TN_PREC_BF16X3>, dim3(kReduceBlocks, batch), dim3(threads), 0, s, a, a.gates,
                       a.segs, a.U);
  else
    hipLaunchKernelGGL(k_adjoint_pass<TN_PREC_C64>, dim3(kReduceBlocks, batch), dim3(threads), 0, s, a, a.gates, a.segs,
                       a.U);
  return hipGetLastError();
}

}  // namespace tnq

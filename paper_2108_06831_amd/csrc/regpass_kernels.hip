// Gate passes in register form (see RegSeg): complex64.
//
// A block of 256 threads takes a chunk of 2^12 elements of the state (or of
// psi and lambda), sixteen per thread and state in registers, through every
// segment of the pass.  LDS only carries the chunk from one segment's layout
// to the next, one state at a time, so a block of the reverse sweep needs
// 33.8 KB and one of the forward pass, with the count groups' power tables, 37.9.
// Three things bound such a pass: the instructions per gate, the latency of
// the scalar loads that feed them, and the registers and LDS that limit the
// waves hiding it.  So
//  - every gate is a body per register bit behind a test that is the same for
//    the whole launch, with no selection of registers at run time; the dense
//    gates are written in place (four instructions per pair and component on
//    the registers they started in), since the compiler otherwise ends each
//    such body with copies of all elements back into the registers the code
//    after the branch expects them in;
//  - gate values and descriptors come through scalar loads, a whole run's
//    together;
//  - address bits are read from the thread's element index, and sign flips
//    are one XOR mask per run.
// The arithmetic is that of the gate-by-gate kernels, operation by operation.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "kernels.h"
#include "pass_util.h"

namespace tnq {

namespace {

constexpr int kRegBuf = (1 << kSweepMaxLocal) + (1 << (kSweepMaxLocal - 5));

struct RegPassArgs {
  const float2* in;   // forward: the pass reads in and writes out; adjoint: psi and lambda in place
  float2* out;
  int64_t in_bs, out_bs;
  int64_t vals_bs;    // forward: between the value tables of parameter vectors; adjoint: between their U
  int64_t n_chunks;
  double* partials;
  int64_t pstride;
  int32_t n_segs, n_rest, ctab_off, ctab_n;
  int32_t first_gate, n_gates;
  int8_t rest[64];
};
static_assert(offsetof(RegPassArgs, rest) % 4 == 0, "position map aligned to 32-bit words");

// t -> t's bits at the positions of a segment's thread bits
__device__ __forceinline__ int thread_bits(int tid, const int32_t* pos) {
  int o = 0;
#pragma unroll
  for (int t = 0; t < 8; ++t) o |= ((tid >> t) & 1) << pos[t];
  return o;
}

// x[] from the layout whose slots are sa + offa[r] to the one whose slots are sb + offb[r]
__device__ __forceinline__ void relayout(float2 (&x)[16], float2* buf, int sa, const int32_t* offa, int sb,
                                         const int32_t* offb) {
#pragma unroll
  for (int r = 0; r < 16; ++r) buf[sa + offa[r]] = x[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = buf[sb + offb[r]];
  __syncthreads();
}

// A dense one-qubit gate's pair, in place: a <- fma(g0, a, g1 b), b <- fma(g2, a, g3 b), real entries.
__device__ __forceinline__ void pair_real(float& a, float& b, float g0, float g1, float g2, float g3) {
  float p, q;
  asm("v_mul_f32 %2, %5, %1\n\t"
      "v_mul_f32 %3, %7, %1\n\t"
      "v_fma_f32 %1, %6, %0, %3\n\t"
      "v_fma_f32 %0, %4, %0, %2"
      : "+v"(a), "+v"(b), "=&v"(p), "=&v"(q)
      : "s"(g0), "s"(g1), "s"(g2), "s"(g3));
}
// Real diagonal g0, g3 and imaginary off-diagonal i g1, i g2:
// a <- (fma(g0, a.x, -g1 b.y), fma(g0, a.y, g1 b.x)), b <- (fma(g3, b.x, -g2 a.y), fma(g3, b.y, g2 a.x)).
__device__ __forceinline__ void pair_rxlike(float2& a, float2& b, float g0, float g1, float g2, float g3) {
  float t0, t1, t2, t3;
  asm("v_mul_f32 %4, -%9, %3\n\t"
      "v_mul_f32 %5, %9, %2\n\t"
      "v_mul_f32 %6, -%10, %1\n\t"
      "v_mul_f32 %7, %10, %0\n\t"
      "v_fma_f32 %0, %8, %0, %4\n\t"
      "v_fma_f32 %1, %8, %1, %5\n\t"
      "v_fma_f32 %2, %11, %2, %6\n\t"
      "v_fma_f32 %3, %11, %3, %7"
      : "+v"(a.x), "+v"(a.y), "+v"(b.x), "+v"(b.y), "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3)
      : "s"(g0), "s"(g1), "s"(g2), "s"(g3));
}

// x <- q x, in place: (fma(q.x, x.x, -(q.y x.y)), fma(q.x, x.y, q.y x.x)), as cmul
__device__ __forceinline__ void mul_in_place(float2& x, float2 q) {
  float t0, t1;
  asm("v_mul_f32 %2, %5, %1\n\t"
      "v_mul_f32 %3, %5, %0\n\t"
      "v_fma_f32 %0, %4, %0, -%2\n\t"
      "v_fma_f32 %1, %4, %1, %3"
      : "+v"(x.x), "+v"(x.y), "=&v"(t0), "=&v"(t1)
      : "v"(q.x), "v"(q.y));
}

// Complex entries: a <- g0 a + g1 b, b <- g2 a + g3 b, each component as cmac(cmul(g0, a), g1, b).
__device__ __forceinline__ void pair_generic(float2& a, float2& b, float2 g0, float2 g1, float2 g2, float2 g3) {
  float t0, t1, t2;
  asm("v_mul_f32 %4, -%8, %1\n\t"
      "v_fma_f32 %4, %7, %0, %4\n\t"
      "v_fma_f32 %4, -%10, %3, %4\n\t"
      "v_fma_f32 %4, %9, %2, %4\n\t"
      "v_mul_f32 %5, %8, %0\n\t"
      "v_fma_f32 %5, %7, %1, %5\n\t"
      "v_fma_f32 %5, %10, %2, %5\n\t"
      "v_fma_f32 %5, %9, %3, %5\n\t"
      "v_mul_f32 %6, -%12, %1\n\t"
      "v_fma_f32 %6, %11, %0, %6\n\t"
      "v_fma_f32 %6, -%14, %3, %6\n\t"
      "v_fma_f32 %6, %13, %2, %6\n\t"
      "v_mul_f32 %0, %12, %0\n\t"
      "v_fma_f32 %0, %11, %1, %0\n\t"
      "v_fma_f32 %0, %14, %2, %0\n\t"
      "v_fma_f32 %3, %13, %3, %0\n\t"
      "v_mov_b32 %0, %4\n\t"
      "v_mov_b32 %1, %5\n\t"
      "v_mov_b32 %2, %6"
      : "+v"(a.x), "+v"(a.y), "+v"(b.x), "+v"(b.y), "=&v"(t0), "=&v"(t1), "=&v"(t2)
      : "s"(g0.x), "s"(g0.y), "s"(g1.x), "s"(g1.y), "s"(g2.x), "s"(g2.y), "s"(g3.x), "s"(g3.y));
}

template <int R>
__device__ __forceinline__ void dense_generic(float2 (&x)[16], float2 g0, float2 g1, float2 g2, float2 g3) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r & (1 << R)) continue;
    pair_generic(x[r], x[r | (1 << R)], g0, g1, g2, g3);
  }
}
template <int R>
__device__ __forceinline__ void dense_real(float2 (&x)[16], float g0, float g1, float g2, float g3) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r & (1 << R)) continue;
    pair_real(x[r].x, x[r | (1 << R)].x, g0, g1, g2, g3);
    pair_real(x[r].y, x[r | (1 << R)].y, g0, g1, g2, g3);
  }
}
template <int R>
__device__ __forceinline__ void dense_rxlike(float2 (&x)[16], float g0, float g1, float g2, float g3) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r & (1 << R)) continue;
    pair_rxlike(x[r], x[r | (1 << R)], g0, g1, g2, g3);
  }
}

// the segment's leading sign flips as bit 31 of the result
__device__ __forceinline__ uint32_t lead_signs(const RegSeg& seg, const uint32_t* __restrict__ words, uint32_t A) {
  uint32_t s = 0;
  int i = seg.sign_off;
  const int end = seg.sign_off + seg.n_sign;
  for (; i + 4 <= end; i += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t w = words[i + u];
      s ^= (A >> (w & 31)) & (A >> ((w >> 8) & 31));
    }
  }
  for (; i < end; ++i) {
    const uint32_t w = words[i];
    s ^= (A >> (w & 31)) & (A >> ((w >> 8) & 31));
  }
  return s << 31;
}

// a run of sign flips: the register combinations (16-bit mask) this thread negates
__device__ __forceinline__ uint32_t sign_mask16(const RegOp& op, const uint32_t* __restrict__ words, uint32_t A) {
  uint32_t m = (uint32_t)op.mask;
  for (int i = op.off; i < op.off + op.n; ++i) {
    const uint32_t w = words[i];
    m ^= (0u - ((A >> (w & 31)) & 1u)) & (w >> 16);
  }
  return m;
}

// x[r] *= q for the combinations whose bit R is 1
template <int R>
__device__ __forceinline__ void mul_half(float2 (&x)[16], float2 q) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if ((r >> R) & 1) mul_in_place(x[r], q);
}

// see apply_count_group: the edges come packed, sorted by how many of their bits are in the registers
__device__ __forceinline__ void count_op(float2 (&x)[16], const RegOp& op, const uint32_t* __restrict__ words,
                                         uint32_t A, const float2* tab) {
  uint32_t K = 0, to1 = 0;
  int i = op.off;
  for (; i + 4 <= op.off + op.n; i += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t w = words[i + u];
      K += ((A >> (w & 31)) ^ (A >> ((w >> 8) & 31))) & 1u;
    }
  }
  for (; i < op.off + op.n; ++i) {
    const uint32_t w = words[i];
    K += ((A >> (w & 31)) ^ (A >> ((w >> 8) & 31))) & 1u;
  }
  for (; i < op.off + op.n + op.n2; ++i) {
    const uint32_t w = words[i];
    to1 += ((A >> (w & 31)) & 1u) << (8 * ((w >> 8) & 3));
  }
  const uint32_t to0 = (uint32_t)op.tot - to1;  // no byte borrows: each field of to1 is at most tot's
  const uint32_t p0 = (uint32_t)op.pc[0], p1 = (uint32_t)op.pc[1];
  auto pair = [&](int j, int k) {  // j < k
    const int f = j == 0 ? k - 1 : j == 1 ? k + 1 : 5;
    return f < 4 ? (p0 >> (8 * f)) & 255u : (p1 >> (8 * (f - 4))) & 255u;
  };
  uint32_t s01[4], s23[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    s01[b] = K + ((b & 1 ? to0 : to1) & 255u) + (((b & 2 ? to0 : to1) >> 8) & 255u);
    s23[b] = (((b & 1 ? to0 : to1) >> 16) & 255u) + ((b & 2 ? to0 : to1) >> 24);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    uint32_t pc = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = j + 1; k < 4; ++k)
        if (((r >> j) ^ (r >> k)) & 1) pc += pair(j, k);
    mul_in_place(x[r], tab[s01[r & 3] + s23[r >> 2] + pc]);
  }
}

// F for every register bit R of `mask`, lowest first
#define TNQ_DENSE_BITS(...)                             \
  if (mask & 1) { constexpr int R = 0; __VA_ARGS__; } \
  if (mask & 2) { constexpr int R = 1; __VA_ARGS__; } \
  if (mask & 4) { constexpr int R = 2; __VA_ARGS__; } \
  if (mask & 8) { constexpr int R = 3; __VA_ARGS__; }

// The observable of a last pass that ends in an expectation (empty otherwise).
template <bool EXPECT>
struct PassTerms {};
template <>
struct PassTerms<true> {
  ZTerms t;  // sorted by their bits at the last segment's register positions
};

// Forward pass.  (Value and descriptor tables as separate __restrict__
// arguments, so that they are read with scalar loads.)  A NULL input is the
// state |0...0>: the first pass of a contraction from the qubits' |0> vectors
// then reads nothing.  EXPECT: the last pass of an expectation sums |x|^2 D(x)
// in FP64 (as k_expect_partial16) into partials[blockIdx.x] and stores no
// state.  (On a 26-qubit state each saves 1 GiB of the 1 GiB + 1 GiB that the
// product state's launch and the pass, or the pass and the reduction, moved.)
template <bool EXPECT>
__global__ __launch_bounds__(kThreads, 4) void k_sweep_regs(RegPassArgs a, const RegSeg* __restrict__ segs,
                                                            const RegOp* __restrict__ ops,
                                                            const RegPhase* __restrict__ phases,
                                                            const uint32_t* __restrict__ words,
                                                            const float2* __restrict__ vals, PassTerms<EXPECT> obs) {
  __shared__ float2 buf[kRegBuf];
  __shared__ float2 ctab[kCountTabMax];
  const int z = blockIdx.y, tid = threadIdx.x;
  const float2* V0 = vals + (int64_t)z * a.vals_bs;
  for (int t = tid; t < a.ctab_n; t += kThreads) ctab[t] = V0[a.ctab_off + t];
  double esum = 0.0;
  for (int64_t c = blockIdx.x; c < (EXPECT ? a.n_chunks : (int64_t)blockIdx.x + 1); c += gridDim.x) {
  const int64_t base = deposit(c, a.rest, a.n_rest);
  float2 x[16];
  const RegSeg& ld = segs[a.n_segs];
  int slot = thread_bits(tid, ld.tpos);
  slot += slot >> 5;
  const int32_t* off = ld.physoff;
  bool same = true;  // the first segment's registers are the load's
#pragma unroll
  for (int j = 0; j < 4; ++j) same &= ld.rbits[j] == segs[0].rbits[j];
  if (!a.in) {
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = f2(r == 0 && base == 0 && tid == 0 ? 1.f : 0.f, 0.f);
  } else {
    const float2* src = a.in + (int64_t)z * a.in_bs + (base | (uint32_t)thread_bits(tid, ld.gpos));
    const int64_t g0 = 1ll << ld.rgpos[0], g1 = 1ll << ld.rgpos[1], g2 = 1ll << ld.rgpos[2], g3 = 1ll << ld.rgpos[3];
#pragma unroll
    for (int r = 0; r < 16; ++r)
      x[r] = load_stream(src + ((r & 1 ? g0 : 0) + (r & 2 ? g1 : 0) + (r & 4 ? g2 : 0) + (r & 8 ? g3 : 0)));
  }
  __syncthreads();  // ctab
  for (int sg = 0; sg < a.n_segs; ++sg) {
    const RegSeg& seg = segs[sg];
    int ob = thread_bits(tid, seg.tpos);
    ob += ob >> 5;
    if (sg > 0 || !same) relayout(x, buf, slot, off, ob, seg.physoff);
    slot = ob;
    off = seg.physoff;
    const uint32_t A = (uint32_t)base | (uint32_t)thread_bits(tid, seg.gpos);
    // diagonal factors that are the same for all of the thread's elements, applied once at the end
    float2 ph = f2(1.f, 0.f);
    for (int i = seg.phase_off; i < seg.phase_off + seg.n_phase; ++i) {
      const RegPhase& p = phases[i];
      const float2* V = V0 + p.src;
      const bool b0 = (A >> (p.p[0] & 31)) & 1;
      float2 f;
      if (p.p[1] < 0) {
        const float2 d0 = V[0], d1 = V[1];
        f = b0 ? d1 : d0;
      } else {
        const bool b1 = (A >> (p.p[1] & 31)) & 1;
        const float2 d0 = V[0], d1 = V[1], d2 = V[2], d3 = V[3];
        const float2 lo = b0 ? d1 : d0, hi = b0 ? d3 : d2;
        f = b1 ? hi : lo;
      }
      ph = cmul<TN_PREC_C64>(ph, f);
    }
    if (seg.n_sign) ph = flip_s(ph, lead_signs(seg, words, A));
    for (int oi = seg.op_off; oi < seg.op_off + seg.n_op; ++oi) {
      const RegOp& op = ops[oi];
      const int mask = op.mask;
      if (op.type & (REG_REAL | REG_RXLIKE | REG_DENSE)) {
        float2 v[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[j][e] = V0[op.src[j] + e];
        if (op.type & REG_REAL) {
          TNQ_DENSE_BITS(dense_real<R>(x, v[R][0].x, v[R][1].x, v[R][2].x, v[R][3].x))
        }
        if (op.type & REG_RXLIKE) {
          TNQ_DENSE_BITS(dense_rxlike<R>(x, v[R][0].x, v[R][1].y, v[R][2].y, v[R][3].x))
        }
        if (op.type & REG_DENSE) {
          TNQ_DENSE_BITS(dense_generic<R>(x, v[R][0], v[R][1], v[R][2], v[R][3]))
        }
      }
      if (op.type & REG_COUNT) count_op(x, op, words, A, ctab + op.src[0]);
      if (op.type & REG_SIGNS) {
        const uint32_t m = sign_mask16(op, words, A);
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = flip_s(x[r], (m << (31 - r)) & 0x80000000u);
      }
      if (op.type & REG_DIAG) {  // one-bit unit diagonals: the first entry joins the factor
#define TNQ_DIAG_BIT(R)                                                                         \
  if (mask & (1 << R)) {                                                                        \
    const float2 e0 = V0[op.src[R]], e1 = V0[op.src[R] + 1];                                    \
    ph = cmul<TN_PREC_C64>(ph, e0);                                                             \
    mul_half<R>(x, cmul<TN_PREC_C64>(e1, f2(e0.x, -e0.y)));                                     \
  }
        TNQ_DIAG_BIT(0) TNQ_DIAG_BIT(1) TNQ_DIAG_BIT(2) TNQ_DIAG_BIT(3)
#undef TNQ_DIAG_BIT
      }
      if (op.type & REG_DIAG2) {  // a two-bit unit diagonal, one or both bits in the registers
        const float2 d0 = V0[op.src[0]], d1 = V0[op.src[0] + 1], d2 = V0[op.src[0] + 2], d3 = V0[op.src[0] + 3];
        if (op.other >= 0) {
          const bool c = (A >> (op.other & 31)) & 1;
          const bool c1 = op.other >> 8;  // the address bit is the index's bit 1
          const float2 e0 = c ? (c1 ? d2 : d1) : d0, e1 = c ? d3 : (c1 ? d1 : d2);
          ph = cmul<TN_PREC_C64>(ph, e0);
          const float2 q = cmul<TN_PREC_C64>(e1, f2(e0.x, -e0.y));
          if (mask & 1) mul_half<0>(x, q);
          if (mask & 2) mul_half<1>(x, q);
          if (mask & 4) mul_half<2>(x, q);
          if (mask & 8) mul_half<3>(x, q);
        } else {  // (a factor of exactly 1 leaves an element as it is)
          const int k0 = op.form & 255, k1 = op.form >> 8;
          ph = cmul<TN_PREC_C64>(ph, d0);
          const float2 c0 = f2(d0.x, -d0.y);
          const float2 q1 = cmul<TN_PREC_C64>(d1, c0), q2 = cmul<TN_PREC_C64>(d2, c0), q3 = cmul<TN_PREC_C64>(d3, c0);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const bool b0 = (r >> k0) & 1, b1 = (r >> k1) & 1;
            const float2 q = b0 ? (b1 ? q3 : q1) : (b1 ? q2 : f2(1.f, 0.f));
            mul_in_place(x[r], q);
          }
        }
      }
    }
    if (seg.ph_used)
#pragma unroll
      for (int r = 0; r < 16; ++r) mul_in_place(x[r], ph);
  }
  if constexpr (EXPECT) {
    const RegSeg& seg = segs[a.n_segs - 1];
    const uint32_t A = (uint32_t)base | (uint32_t)thread_bits(tid, seg.gpos);
    double w[16];  // D at the thread's elements: per pattern of the register bits, then a Walsh-Hadamard transform
    sum_terms16(A, obs.t, w);
#pragma unroll
    for (int r = 0; r < 16; ++r) esum += ((double)x[r].x * x[r].x + (double)x[r].y * x[r].y) * w[r];
  } else {
    const RegSeg& st = segs[a.n_segs + 1];
    bool keep = true;
#pragma unroll
    for (int j = 0; j < 4; ++j) keep &= st.rbits[j] == segs[a.n_segs - 1].rbits[j];
    if (!keep) {
      int ob = thread_bits(tid, st.tpos);
      ob += ob >> 5;
      relayout(x, buf, slot, off, ob, st.physoff);
    }
    float2* dst = a.out + (int64_t)z * a.out_bs + (base | (uint32_t)thread_bits(tid, st.gpos));
    const int64_t g0 = 1ll << st.rgpos[0], g1 = 1ll << st.rgpos[1], g2 = 1ll << st.rgpos[2], g3 = 1ll << st.rgpos[3];
#pragma unroll
    for (int r = 0; r < 16; ++r)
      store_stream(dst + ((r & 1 ? g0 : 0) + (r & 2 ? g1 : 0) + (r & 4 ? g2 : 0) + (r & 8 ? g3 : 0)), x[r].x, x[r].y);
  }
  }
  if constexpr (EXPECT) {
    __syncthreads();
    esum = block_sum(esum, reinterpret_cast<double*>(buf));
    if (tid == 0) a.partials[(int64_t)z * a.pstride + blockIdx.x] = esum;
  }
}

// Reverse sweep over psi and lambda (see k_adjoint_pass).
__global__ __launch_bounds__(kThreads, 4) void k_adjoint_regs(RegPassArgs a, const RegSeg* __restrict__ segs,
                                                              const RegOp* __restrict__ ops,
                                                              const RegPhase* __restrict__ phases,
                                                              const uint32_t* __restrict__ words,
                                                              const float2* __restrict__ Uall,
                                                              const AdjGateDesc* __restrict__ gates) {
  __shared__ __attribute__((aligned(16))) float2 buf[kRegBuf];
  const int z = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const float2* Uz = Uall + (int64_t)z * a.vals_bs;
  float2* P = const_cast<float2*>(a.in) + (int64_t)z * a.in_bs;
  float2* L = a.out + (int64_t)z * a.out_bs;
  // gradient sums of this wave: lane j holds accumulators j (accA) and 64 + j (accB)
  double accA = 0.0, accB = 0.0;
  const RegSeg& ld = segs[a.n_segs];
  const RegSeg& st = segs[a.n_segs + 1];
  bool same = true, keep = true;  // the first and last segments' registers are the load's and the store's
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    same &= ld.rbits[j] == segs[0].rbits[j];
    keep &= st.rbits[j] == segs[a.n_segs - 1].rbits[j];
  }
  for (int64_t c = blockIdx.x; c < a.n_chunks; c += gridDim.x) {
    const int64_t base = deposit(c, a.rest, a.n_rest);
    int accF0 = 0, accF1 = 0;  // this chunk's terms (float bits), placed as accA and accB
    auto add_grad = [&](int red, float v) {
      const int t = __builtin_amdgcn_readlane(__float_as_int(wave_sum_to_63(v)), 63);
      if (red < 64) accF0 = lane == red ? t : accF0;
      else accF1 = lane == red - 64 ? t : accF1;
    };
    float2 xp[16], xl[16];
    int slot = thread_bits(tid, ld.tpos);
    slot += slot >> 5;
    const int32_t* off = ld.physoff;
    {
      const int64_t o = base | (uint32_t)thread_bits(tid, ld.gpos);
      const int64_t g0 = 1ll << ld.rgpos[0], g1 = 1ll << ld.rgpos[1], g2 = 1ll << ld.rgpos[2], g3 = 1ll << ld.rgpos[3];
#pragma unroll
      for (int r = 0; r < 16; ++r)
        xp[r] = load_stream(P + o + ((r & 1 ? g0 : 0) + (r & 2 ? g1 : 0) + (r & 4 ? g2 : 0) + (r & 8 ? g3 : 0)));
#pragma unroll
      for (int r = 0; r < 16; ++r)
        xl[r] = load_stream(L + o + ((r & 1 ? g0 : 0) + (r & 2 ? g1 : 0) + (r & 4 ? g2 : 0) + (r & 8 ? g3 : 0)));
    }
    for (int sg = 0; sg < a.n_segs; ++sg) {
      const RegSeg& seg = segs[sg];
      int ob = thread_bits(tid, seg.tpos);
      ob += ob >> 5;
      if (sg > 0 || !same) {
        relayout(xp, buf, slot, off, ob, seg.physoff);
        relayout(xl, buf, slot, off, ob, seg.physoff);
      }
      slot = ob;
      off = seg.physoff;
      const uint32_t A = (uint32_t)base | (uint32_t)thread_bits(tid, seg.gpos);
      // unit factors that are the same for all of the thread's elements: applied to both states at
      // the end (they leave every gradient term as it is)
      float2 ph = f2(1.f, 0.f);
      float tT = 0.f;  // Im(conj(lambda) psi) over the thread's elements
      if (seg.lead_sums)
#pragma unroll
        for (int r = 0; r < 16; ++r) tT += im_conj_mul(xl[r], xp[r]);
      for (int i = seg.phase_off; i < seg.phase_off + seg.n_phase; ++i) {
        const RegPhase& p = phases[i];
        const float2* U = Uz + p.src;
        const bool b0 = (A >> (p.p[0] & 31)) & 1;
        float2 u;
        float q;
        if (p.p[1] < 0) {
          const float2 u0 = U[0], u1 = U[3];
          u = b0 ? u1 : u0;
          q = b0 ? p.q[1] : p.q[0];
        } else {
          const bool b1 = (A >> (p.p[1] & 31)) & 1;
          const float2 u0 = U[0], u1 = U[5], u2 = U[10], u3 = U[15];
          const float2 lo = b0 ? u1 : u0, hi = b0 ? u3 : u2;
          u = b1 ? hi : lo;
          const float ql = b0 ? p.q[1] : p.q[0], qh = b0 ? p.q[3] : p.q[2];
          q = b1 ? qh : ql;
        }
        if (p.red >= 0) add_grad(p.red, q * tT);
        ph = cmul<TN_PREC_C64>(ph, f2(u.x, -u.y));
      }
      if (seg.n_sign) ph = flip_s(ph, lead_signs(seg, words, A));
      float tS0 = 0.f, tS1 = 0.f, tS2 = 0.f, tS3 = 0.f;
      for (int oi = seg.op_off; oi < seg.op_off + seg.n_op; ++oi) {
        const RegOp& op = ops[oi];
        const int mask = op.mask;
        if (op.type & (REG_REAL | REG_RXLIKE | REG_DENSE)) {
          float2 u[4][4];  // U of the run's gates; U^dagger[m][k] = conj(U[k][m])
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) u[j][e] = Uz[op.src[j] + e];
#define TNQ_GRAD                                                          \
  if (op.red[R] >= 0) {                                                   \
    float g = 0.f;                                                        \
    if (op.gform[R] == ADJ_GEN_X) g = reg_grad_x<R>(xp, xl, op.g0[R]);    \
    else g = reg_grad_y<R>(xp, xl);                                       \
    add_grad(op.red[R], g);                                               \
  }
          if (op.type & REG_REAL) {
            TNQ_DENSE_BITS(TNQ_GRAD dense_real<R>(xp, u[R][0].x, u[R][2].x, u[R][1].x, u[R][3].x);
                           dense_real<R>(xl, u[R][0].x, u[R][2].x, u[R][1].x, u[R][3].x))
          }
          if (op.type & REG_RXLIKE) {
            TNQ_DENSE_BITS(TNQ_GRAD dense_rxlike<R>(xp, u[R][0].x, neg_s(u[R][2].y), neg_s(u[R][1].y), u[R][3].x);
                           dense_rxlike<R>(xl, u[R][0].x, neg_s(u[R][2].y), neg_s(u[R][1].y), u[R][3].x))
          }
          if (op.type & REG_DENSE) {
            TNQ_DENSE_BITS(TNQ_GRAD const float2 w0 = f2(u[R][0].x, neg_s(u[R][0].y)), w1 = f2(u[R][2].x, neg_s(u[R][2].y)),
                           w2 = f2(u[R][1].x, neg_s(u[R][1].y)), w3 = f2(u[R][3].x, neg_s(u[R][3].y));
                           dense_generic<R>(xp, w0, w1, w2, w3); dense_generic<R>(xl, w0, w1, w2, w3))
          }
#undef TNQ_GRAD
        }
        if (op.type & REG_SIGNS) {
          const uint32_t m = sign_mask16(op, words, A);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const uint32_t s = (m << (31 - r)) & 0x80000000u;
            xp[r] = flip_s(xp[r], s);
            xl[r] = flip_s(xl[r], s);
          }
        }
        if (op.type & REG_DIAG) {  // one-bit unit diagonals
          if (op.sums) {  // the sums, over all elements and over those with register bit j set
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
          }
#define TNQ_DIAG_BIT(R, S)                                                                  \
  if (mask & (1 << R)) {                                                                    \
    if (op.red[R] >= 0) add_grad(op.red[R], op.g0[R] * (tT - S) + op.g1[R] * S);            \
    const float2 u0 = Uz[op.src[R]], u1 = Uz[op.src[R] + 3];                                \
    const float2 e0 = f2(u0.x, -u0.y), e1 = f2(u1.x, -u1.y);                                \
    ph = cmul<TN_PREC_C64>(ph, e0);                                                         \
    const float2 q = cmul<TN_PREC_C64>(e1, f2(e0.x, -e0.y));                                \
    mul_half<R>(xp, q);                                                                     \
    mul_half<R>(xl, q);                                                                     \
  }
          TNQ_DIAG_BIT(0, tS0) TNQ_DIAG_BIT(1, tS1) TNQ_DIAG_BIT(2, tS2) TNQ_DIAG_BIT(3, tS3)
#undef TNQ_DIAG_BIT
        }
      }
      if (seg.ph_used)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          mul_in_place(xp[r], ph);
          mul_in_place(xl[r], ph);
        }
    }
    if (!keep) {
      int ob = thread_bits(tid, st.tpos);
      ob += ob >> 5;
      relayout(xp, buf, slot, off, ob, st.physoff);
      relayout(xl, buf, slot, off, ob, st.physoff);
    }
    {
      const int64_t o = base | (uint32_t)thread_bits(tid, st.gpos);
      const int64_t g0 = 1ll << st.rgpos[0], g1 = 1ll << st.rgpos[1], g2 = 1ll << st.rgpos[2], g3 = 1ll << st.rgpos[3];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t g = o + ((r & 1 ? g0 : 0) + (r & 2 ? g1 : 0) + (r & 4 ? g2 : 0) + (r & 8 ? g3 : 0));
        store_stream(P + g, xp[r].x, xp[r].y);
        store_stream(L + g, xl[r].x, xl[r].y);
      }
    }
    accA += (double)__int_as_float(accF0);
    accB += (double)__int_as_float(accF1);
  }
  __syncthreads();
  double* red = reinterpret_cast<double*>(buf);  // [accumulator][wave]
  red[lane * 4 + wv] = accA;
  red[(64 + lane) * 4 + wv] = accB;
  __syncthreads();
  for (int gi = a.first_gate + tid; gi < a.first_gate + a.n_gates; gi += kThreads) {
    const AdjGateDesc& gd = gates[gi];
    if (gd.red < 0 || gd.slot < 0) continue;
    double v = 0;
    for (int w = 0; w < 4; ++w) v += red[gd.red * 4 + w];
    a.partials[(int64_t)z * a.pstride + (int64_t)gd.slot * kReduceBlocks + blockIdx.x] = v;
  }
}
#undef TNQ_DENSE_BITS

// the address bits outside the pass's chunk; false: the chunk is not one the kernels take
bool rest_bits(const SweepPass& ps, int bits, RegPassArgs* a) {
  if (ps.l != kSweepMaxLocal || bits > 32 || ps.n_segs < 1) return false;
  std::vector<char> local(bits, 0);
  for (int j = 0; j < ps.l; ++j) {
    if (ps.lpos[j] < 0 || ps.lpos[j] >= bits || (j < 5 && ps.lpos[j] != j)) return false;
    local[ps.lpos[j]] = 1;
  }
  a->n_rest = 0;
  for (int p = 0; p < bits; ++p)
    if (!local[p]) a->rest[a->n_rest++] = (int8_t)p;
  a->n_chunks = (int64_t)1 << a->n_rest;
  a->n_segs = ps.n_segs;
  return a->n_chunks <= ((int64_t)1 << 24);
}

}  // namespace

hipError_t launch_sweep_regs(hipStream_t s, const SweepPass& ps, int bits, const RegTables& t, const float2* in,
                             int64_t in_bs, float2* out, int64_t out_bs, const float2* vals, int64_t vals_bs,
                             int batch, const ZTerms* terms, double* partial) {
  RegPassArgs a{};
  a.in = in; a.out = out; a.in_bs = in_bs; a.out_bs = out_bs;
  a.vals_bs = vals_bs;
  a.ctab_off = ps.ctab_off;
  a.ctab_n = ps.ctab_n;
  if (!rest_bits(ps, bits, &a) || ps.ctab_n < 0 || ps.ctab_n > kCountTabMax || !vals) return hipErrorInvalidValue;
  if (terms) {
    a.partials = partial;
    a.pstride = kExpectBlocks;
    PassTerms<true> p;
    p.t = *terms;
    hipLaunchKernelGGL(k_sweep_regs<true>, dim3(sweep_expect_blocks(ps, bits), batch), dim3(kThreads), 0, s, a,
                       t.segs + ps.reg_seg, t.ops, t.phases, t.words, vals, p);
  } else {
    hipLaunchKernelGGL(k_sweep_regs<false>, dim3((unsigned)a.n_chunks, batch), dim3(kThreads), 0, s, a,
                       t.segs + ps.reg_seg, t.ops, t.phases, t.words, vals, PassTerms<false>{});
  }
  return hipGetLastError();
}

hipError_t launch_adjoint_regs(hipStream_t s, const SweepPass& ps, int bits, const RegTables& t,
                               const AdjGateDesc* gates_dev, const float2* u, int64_t u_bs, float2* psi,
                               int64_t psi_bs, float2* lam, int64_t lam_bs, int batch, double* partials,
                               int64_t partial_stride) {
  RegPassArgs a{};
  a.in = psi; a.out = lam; a.in_bs = psi_bs; a.out_bs = lam_bs;
  a.vals_bs = u_bs;
  a.partials = partials;
  a.pstride = partial_stride;
  a.first_gate = ps.first_gate;
  a.n_gates = ps.n_gates;
  if (!rest_bits(ps, bits, &a) || ps.n_red < 0 || ps.n_red > kAdjMaxRed || ps.n_gates < 0)
    return hipErrorInvalidValue;
  static_assert(kAdjMaxRed * 4 * sizeof(double) <= kRegBuf * sizeof(float2), "accumulators fit the exchange buffer");
  hipLaunchKernelGGL(k_adjoint_regs, dim3(adjoint_blocks(ps, bits), batch), dim3(kThreads), 0, s, a, t.segs + ps.reg_seg, t.ops,
                     t.phases, t.words, u, gates_dev);
  return hipGetLastError();
}

}  // namespace tnq

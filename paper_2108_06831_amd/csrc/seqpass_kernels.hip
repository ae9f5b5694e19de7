// Ordered gate passes over small states (see SeqPass in internal.h).
//
// A contraction of a circuit on few qubits along the sequential order, or the
// reverse sweep of its gradient, is a chain of gates on one small state: as
// one launch per gate it costs about 6 us per gate, all of it launch latency.
// Here one block carries a chunk of up to 2^14 elements (2^13 of psi and
// lambda) through the gates, sixteen elements per thread in registers, LDS
// only between segments; a state of up to that size is one launch, larger ones
// one per pass.  What bounds it is the instructions of one compute unit (or of
// a few): about 0.3 us per gate at 2^13 elements.  Every gate is applied by
// itself and in order, with the products, sums and roundings of the
// step-by-step kernels (k_small_steps, k_elem_group, k_adjoint_step), so the
// state is bit for bit theirs; gradient terms are formed and summed in FP64 as
// in k_adjoint_step.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "kernels.h"
#include "pass_util.h"

namespace tnq {

namespace {

struct SeqArgs {
  const float2* in;  // forward: the state; adjoint: psi
  float2* out;       // forward: the result; adjoint: lambda (both states in place)
  int64_t in_bs, out_bs, vals_bs;
  double* partials;
  int64_t pstride;
  int32_t l, n_rest, n_segs, from_zero;  // from_zero: the state is |0...0>
  int32_t out_t[10], out_r[4];           // forward: positions in the result of the last segment's thread and register bits
  int8_t rest[32], rest_out[32];
};
static_assert(offsetof(SeqArgs, rest) % 4 == 0 && offsetof(SeqArgs, rest_out) % 4 == 0,
              "position maps aligned to 32-bit words");

__device__ __forceinline__ int bits10(int t, const int32_t* pos) {
  int o = 0;
#pragma unroll
  for (int j = 0; j < 10; ++j) o |= ((t >> j) & 1) << pos[j];
  return o;
}

// a <- g0 a + g1 b, b <- g2 a + g3 b (the term of index 0 first, as a sum over the gate's input index)
template <int PREC, int R>
__device__ __forceinline__ void dense_seq(float2 (&x)[16], float2 g0, float2 g1, float2 g2, float2 g3, int form,
                                          bool gate_first) {
  if (PREC == TN_PREC_C64 && form == kFormReal) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (r & (1 << R)) continue;
      float t;
      float2 &a = x[r], &b = x[r | (1 << R)];
#define TNQ_PAIR(A, B)                                                                  \
  asm("v_mul_f32 %2, %5, %0\n\t"                                                        \
      "v_mul_f32 %0, %3, %0\n\t"                                                        \
      "v_fma_f32 %0, %4, %1, %0\n\t"                                                    \
      "v_fma_f32 %1, %6, %1, %2"                                                        \
      : "+v"(A), "+v"(B), "=&v"(t)                                                      \
      : "v"(g0.x), "v"(g1.x), "v"(g2.x), "v"(g3.x));
      TNQ_PAIR(a.x, b.x)
      TNQ_PAIR(a.y, b.y)
#undef TNQ_PAIR
    }
  } else if (PREC == TN_PREC_C64 && form == kFormRxLike) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (r & (1 << R)) continue;
      float t0, t1;
      float2 &a = x[r], &b = x[r | (1 << R)];
      asm("v_mul_f32 %4, -%8, %1\n\t"
          "v_mul_f32 %5, %8, %0\n\t"
          "v_mul_f32 %0, %6, %0\n\t"
          "v_mul_f32 %1, %6, %1\n\t"
          "v_fma_f32 %0, -%7, %3, %0\n\t"
          "v_fma_f32 %1, %7, %2, %1\n\t"
          "v_fma_f32 %2, %9, %2, %4\n\t"
          "v_fma_f32 %3, %9, %3, %5"
          : "+v"(a.x), "+v"(a.y), "+v"(b.x), "+v"(b.y), "=&v"(t0), "=&v"(t1)
          : "v"(g0.x), "v"(g1.y), "v"(g2.y), "v"(g3.x));
    }
  } else if (gate_first) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (r & (1 << R)) continue;
      const float2 a = x[r], b = x[r | (1 << R)];
      x[r] = cmac<PREC>(cmul<PREC>(g0, a), g1, b);
      x[r | (1 << R)] = cmac<PREC>(cmul<PREC>(g2, a), g3, b);
    }
    variant_end<PREC, 600 + R>();
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (r & (1 << R)) continue;
      const float2 a = x[r], b = x[r | (1 << R)];
      x[r] = cmac<PREC>(cmul<PREC>(a, g0), b, g1);
      x[r | (1 << R)] = cmac<PREC>(cmul<PREC>(a, g2), b, g3);
    }
    variant_end<PREC, 604 + R>();
  }
}

// A two-qubit gate on register bits 2 H (index bit 0) and 2 H + 1 (bit 1); get(e): entry e = 4 m + k, the columns in
// the order of the sum: 0, 1, 2, 3 or (gray) 0, 1, 3, 2.
template <int PREC, int H, class Get>
__device__ __forceinline__ void dense2_seq(float2 (&x)[16], Get get, bool gate_first, bool gray) {
  constexpr int s0 = 1 << (2 * H), s1 = 2 << (2 * H);
  float2 y[16];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const float2 g[4] = {get(4 * m), get(4 * m + 1), get(4 * m + 2), get(4 * m + 3)};
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (r & (s0 | s1)) continue;
      const float2 v0 = x[r], v1 = x[r | s0];
      const float2 v2 = gray ? x[r | s0 | s1] : x[r | s1], v3 = gray ? x[r | s1] : x[r | s0 | s1];
      float2 acc;
      if (gate_first) {
        acc = cmac<PREC>(cmac<PREC>(cmac<PREC>(cmul<PREC>(g[0], v0), g[1], v1), g[2], v2), g[3], v3);
      } else {
        acc = cmac<PREC>(cmac<PREC>(cmac<PREC>(cmul<PREC>(v0, g[0]), v1, g[1]), v2, g[2]), v3, g[3]);
      }
      y[r | (m & 1 ? s0 : 0) | (m & 2 ? s1 : 0)] = acc;
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = y[r];
  variant_end<PREC, 610 + H>();
}

// x <- g x (the gate the first operand) or x g
template <int PREC>
__device__ __forceinline__ void mul_gate(float2& x, float2 g, bool gate_first) {
  x = gate_first ? cmul<PREC>(g, x) : cmul<PREC>(x, g);
}
// x[r] times e1 where bit R of r is 1, else e0
template <int PREC, int R>
__device__ __forceinline__ void diag_seq(float2 (&x)[16], float2 e0, float2 e1, bool gate_first) {
  if (gate_first) {
#pragma unroll
    for (int r = 0; r < 16; ++r) mul_gate<PREC>(x[r], (r >> R) & 1 ? e1 : e0, true);
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) mul_gate<PREC>(x[r], (r >> R) & 1 ? e1 : e0, false);
  }
  variant_end<PREC, 620 + R>();
}

// What a split-precision product leaves of a component times an exact 1: the sum of its two bfloat16 parts.
template <int PREC>
__device__ __forceinline__ float2 times_one(float2 v) {
  if constexpr (PREC == TN_PREC_C64) return v;
  else return f2(rmul<PREC>(1.f, v.x), rmul<PREC>(1.f, v.y));
}

__device__ __forceinline__ double im_d(float2 l, float2 p) { return (double)l.x * p.y - (double)l.y * p.x; }
__device__ __forceinline__ double re_d(float2 l, float2 p) { return (double)l.x * p.x + (double)l.y * p.y; }

// Im(conj(lambda) G psi) over the thread's elements for a generator on register bit R
template <int R>
__device__ __forceinline__ double grad_bit(const float2 (&p)[16], const float2 (&l)[16], int gen) {
  double g = 0.0;
  if (gen == GEN_Y_HALF) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (!(r & (1 << R))) g += re_d(l[r | (1 << R)], p[r]) - re_d(l[r], p[r | (1 << R)]);
  } else if (gen == GEN_Z_HALF) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (!(r & (1 << R))) g += im_d(l[r], p[r]) - im_d(l[r | (1 << R)], p[r | (1 << R)]);
  } else {  // X
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (!(r & (1 << R))) g += im_d(l[r], p[r | (1 << R)]) + im_d(l[r | (1 << R)], p[r]);
    if (gen == GEN_X) g *= 2.0;
  }
  return g;
}

// sum over the 64 lanes, the result in lane 63 (as wave_sum_to_63, on both halves of the doubles)
__device__ __forceinline__ double wave_sum_d(double v) {
#define TNQ_STEP(CTRL, ROWS)                                                             \
  {                                                                                      \
    const long long b = __double_as_longlong(v);                                         \
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false);       \
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false); \
    v += __longlong_as_double(((long long)hi << 32) | (unsigned)lo);                     \
  }
  TNQ_STEP(0xb1, 0xf)
  TNQ_STEP(0x4e, 0xf)
  TNQ_STEP(0x141, 0xf)
  TNQ_STEP(0x140, 0xf)
  TNQ_STEP(0x142, 0xa)
  TNQ_STEP(0x143, 0xc)
#undef TNQ_STEP
  return v;
}

// The gates of a pass on the thread's sixteen elements of the state x (and of y
// where NS = 2).  load(seg, A) fills them in the first segment's layout, A the
// address of the thread's combination 0; they are left in the last one's.
template <int PREC, int NS, class Load, class Grad>
__device__ __forceinline__ void seq_run(float2 (&x)[16], float2 (&y)[16], float2* bx, float2* by, float2* vwin,
                                        uint32_t* wwin, int n_segs, const SeqSeg* __restrict__ segs,
                                        const SeqWindow* __restrict__ wins, const uint32_t* __restrict__ words,
                                        const int32_t* __restrict__ vsrc, const float2* V, uint32_t base, int tid,
                                        Load load, Grad add_grad) {
  int slot = 0;
  const int32_t* off = nullptr;
  int win = 0, win_end = 0;  // the window's number and the end of its segments
  int wi = 0, vi = 0;        // the next operation's word and value
  auto word = [&](int i) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)wwin[i]); };
  for (int sg = 0; sg < n_segs; ++sg) {
    if (sg == win_end) {
      const SeqWindow w = wins[win++];
      __syncthreads();  // the window before is no longer read
      for (int i = threadIdx.x; i < w.n_words; i += blockDim.x) wwin[i] = words[w.word_off + i];
      for (int i = threadIdx.x; i < w.n_vals; i += blockDim.x) {
        const float2 v = V[vsrc[w.val_off + i]];
        vwin[i] = NS == 2 ? f2(v.x, -v.y) : v;
      }
      __syncthreads();
      win_end = sg + w.n_segs;
      wi = vi = 0;
    }
    const SeqSeg& seg = segs[sg];
    const int ob = bits10(tid, seg.tpos), ns = ob + (ob >> 5);
    const uint32_t A = base | (uint32_t)bits10(tid, seg.gpos);
    if (sg == 0) {
      load(seg, A);
    } else {
      // each thread writes the slots it read last, so one barrier separates the layouts
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        bx[slot + off[r]] = x[r];
        if (NS == 2) by[slot + off[r]] = y[r];
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        x[r] = bx[ns + seg.physoff[r]];
        if (NS == 2) y[r] = by[ns + seg.physoff[r]];
      }
    }
    slot = ns;
    off = seg.physoff;
    for (int oi = 0; oi < seg.n_op; ++oi) {
      const uint32_t head = word(wi++);
      if (head & SEQ_BITS) {
#define TNQ_SEQ_BIT(R)                                                                                        \
  if ((head >> (4 + R)) & 1) {                                                                                \
    if (NS == 2) {                                                                                            \
      const uint32_t w = word(wi++);                                                                          \
      if (w >> 8) add_grad((int)(w >> 8) - 1, grad_bit<R>(x, y, (int)(w & 255)));                             \
    }                                                                                                         \
    const float2 g0 = vwin[vi], g1 = vwin[vi + 1], g2 = vwin[vi + 2], g3 = vwin[vi + 3];                      \
    vi += 4;                                                                                                  \
    const int form = (head >> (20 + 2 * R)) & 3;                                                              \
    dense_seq<PREC, R>(x, g0, g1, g2, g3, form, NS == 2 || ((head >> (12 + R)) & 1));                         \
    if (NS == 2) dense_seq<PREC, R>(y, g0, g1, g2, g3, form, true);                                           \
  }                                                                                                           \
  if ((head >> (8 + R)) & 1) {                                                                                \
    if (NS == 2) {                                                                                            \
      const uint32_t w = word(wi++);                                                                          \
      if (w >> 8) add_grad((int)(w >> 8) - 1, grad_bit<R>(x, y, GEN_Z_HALF));                                 \
    }                                                                                                         \
    const float2 e0 = vwin[vi], e1 = vwin[vi + 1];                                                            \
    vi += 2;                                                                                                  \
    diag_seq<PREC, R>(x, e0, e1, NS == 2 || ((head >> (16 + R)) & 1));                                        \
    if (NS == 2) diag_seq<PREC, R>(y, e0, e1, true);                                                          \
  }
        TNQ_SEQ_BIT(0)
        TNQ_SEQ_BIT(1)
        TNQ_SEQ_BIT(2)
        TNQ_SEQ_BIT(3)
#undef TNQ_SEQ_BIT
      }
      if (head & SEQ_SIGNS) {
        uint32_t m = head >> 16;
        const int n = (int)word(wi++);
        for (int i = wi; i < wi + n; ++i) {
          const uint32_t w = wwin[i];
          m ^= (0u - ((A >> (w & 31)) & (A >> ((w >> 8) & 31)) & 1u)) & (w >> 16);
        }
        wi += n;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const uint32_t s = (m << (31 - r)) & 0x80000000u;
          x[r] = flip_s(times_one<PREC>(x[r]), s);
          if (NS == 2) y[r] = flip_s(times_one<PREC>(y[r]), s);
        }
      }
      if (head & SEQ_DIAG) {
        const uint32_t w1 = word(wi), w2 = word(wi + 1);
        wi += 2;
        const int k0 = (int)(w1 & 15) - 1, k1 = (int)((w1 >> 4) & 15) - 1;
        const bool two = ((head >> 4) & 15) == 2, gf = NS == 2 || ((head >> 12) & 1);
        const int c0 = (A >> ((w1 >> 8) & 31)) & 1, c1 = two ? (A >> ((w1 >> 16) & 31)) & 1 : 0;
        const float2 d0 = vwin[vi], d1 = vwin[vi + 1];
        float2 d2 = d0, d3 = d0;
        if (two) {
          d2 = vwin[vi + 2];
          d3 = vwin[vi + 3];
        }
        vi += two ? 4 : 2;
        if (NS == 2 && (w2 >> 8)) {
          const int gen = (int)((w2 >> 4) & 15);
          double g = 0.0;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int b0 = k0 >= 0 ? (r >> k0) & 1 : c0, b1 = k1 >= 0 ? (r >> k1) & 1 : c1;
            const double w = gen == GEN_ZZ_PHASE ? (b0 != b1 ? 2.0 : 0.0)
                             : gen == GEN_CPHASE ? (b0 && b1 ? -2.0 : 0.0)
                                                 : (b0 ? -1.0 : 1.0);
            g += w * im_d(y[r], x[r]);
          }
          add_grad((int)(w2 >> 8) - 1, g);
        }
        if (two && k0 >= 0 && k1 >= 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int b = ((r >> k0) & 1) | (((r >> k1) & 1) << 1);
            if (PREC == TN_PREC_C64 && ((w2 >> b) & 1)) continue;
            const float2 q = b == 0 ? d0 : b == 1 ? d1 : b == 2 ? d2 : d3;
            if (gf) mul_gate<PREC>(x[r], q, true);
            else mul_gate<PREC>(x[r], q, false);
            if (NS == 2) mul_gate<PREC>(y[r], q, true);
          }
        } else if (two && (k0 >= 0 || k1 >= 0)) {
          const int k = k0 >= 0 ? k0 : k1;
          const float2 e0 = k0 >= 0 ? (c1 ? d2 : d0) : (c0 ? d1 : d0), e1 = k0 >= 0 ? (c1 ? d3 : d1) : (c0 ? d3 : d2);
          if (k == 0) { diag_seq<PREC, 0>(x, e0, e1, gf); if (NS == 2) diag_seq<PREC, 0>(y, e0, e1, true); }
          if (k == 1) { diag_seq<PREC, 1>(x, e0, e1, gf); if (NS == 2) diag_seq<PREC, 1>(y, e0, e1, true); }
          if (k == 2) { diag_seq<PREC, 2>(x, e0, e1, gf); if (NS == 2) diag_seq<PREC, 2>(y, e0, e1, true); }
          if (k == 3) { diag_seq<PREC, 3>(x, e0, e1, gf); if (NS == 2) diag_seq<PREC, 3>(y, e0, e1, true); }
        } else {
          const float2 lo = c0 ? d1 : d0, hi = c0 ? d3 : d2;
          const float2 q = two && c1 ? hi : lo;
          diag_seq<PREC, 0>(x, q, q, gf);
          if (NS == 2) diag_seq<PREC, 0>(y, q, q, true);
        }
      }
      if (head & SEQ_DENSE2) {
        auto get = [&](int e) { return vwin[vi + e]; };
        const bool gf = NS == 2 || ((head >> 12) & 1), gray = NS == 1 && ((head >> 13) & 1);
        if (((head >> 4) & 15) == 0) {
          dense2_seq<PREC, 0>(x, get, gf, gray);
          if (NS == 2) dense2_seq<PREC, 0>(y, get, true, false);
        } else {
          dense2_seq<PREC, 1>(x, get, gf, gray);
          if (NS == 2) dense2_seq<PREC, 1>(y, get, true, false);
        }
        vi += 16;
      }
    }
  }
}

// address of register combination r of a segment, from its combination 0
__device__ __forceinline__ uint32_t seg_addr(const SeqSeg& seg, uint32_t A, int r) {
  return A | (r & 1 ? 1u << seg.rgpos[0] : 0) | (r & 2 ? 1u << seg.rgpos[1] : 0) | (r & 4 ? 1u << seg.rgpos[2] : 0) |
         (r & 8 ? 1u << seg.rgpos[3] : 0);
}

// NS = 1: forward, from the state `in` (or |0...0>) to `out`; vals: the network's
// input tensors.  NS = 2: reverse sweep over psi and lambda; vals: U of every
// gate; gradient slot s of wave w of chunk c into partials[s][c * waves + w].
template <int PREC, int NS, int LMAX>
__global__ __launch_bounds__(1 << (LMAX - 4)) void k_seq_pass(SeqArgs a, const SeqSeg* __restrict__ segs,
                                                              const SeqWindow* __restrict__ wins,
                                                              const uint32_t* __restrict__ words,
                                                              const int32_t* __restrict__ vsrc,
                                                              const float2* __restrict__ vals) {
  constexpr int kBuf = (1 << LMAX) + (1 << (LMAX - 5));
  __shared__ float2 bx[kBuf];
  __shared__ float2 by[NS == 2 ? kBuf : 1];
  __shared__ __attribute__((aligned(16))) float2 vwin[kSeqWinVals];  // the window's values (a reverse sweep's conjugated)
  __shared__ uint32_t wwin[kSeqWinWords];
  const int z = blockIdx.y, lane = threadIdx.x & 63;
  // chunks of fewer than 2^10 elements (forward) leave threads of the wave without elements: they repeat others
  const int n_thr = 1 << (a.l - 4), tid = threadIdx.x & (n_thr - 1);
  const uint32_t base = (uint32_t)deposit(blockIdx.x, a.rest, a.n_rest);
  const float2* V = vals + (int64_t)z * a.vals_bs;
  float2* P = const_cast<float2*>(a.in) + (int64_t)z * a.in_bs;
  float2* O = a.out + (int64_t)z * a.out_bs;
  const int col = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  double* part = a.partials + (int64_t)z * a.pstride + col;
  auto add_grad = [&](int slot, double v) {
    v = wave_sum_d(v);
    if (lane == 63) part[(int64_t)slot * kReduceBlocks] = v;
  };
  float2 x[16], y[16];  // psi (or the state), lambda
  seq_run<PREC, NS>(x, y, bx, by, vwin, wwin, a.n_segs, segs, wins, words, vsrc, V, base, tid,
                    [&](const SeqSeg& seg, uint32_t A) {
#pragma unroll
                      for (int r = 0; r < 16; ++r) {
                        const uint32_t e = seg_addr(seg, A, r);
                        if (NS == 1 && a.from_zero) {
                          x[r] = f2(e == 0 ? 1.f : 0.f, 0.f);
                        } else {
                          x[r] = P[e];
                          if (NS == 2) y[r] = O[e];
                        }
                      }
                    },
                    add_grad);
  if (NS == 1) {
    const uint32_t e0 = (uint32_t)deposit(blockIdx.x, a.rest_out, a.n_rest) | (uint32_t)bits10(tid, a.out_t);
    const uint32_t g0 = 1u << a.out_r[0], g1 = 1u << a.out_r[1], g2 = 1u << a.out_r[2], g3 = 1u << a.out_r[3];
#pragma unroll
    for (int r = 0; r < 16; ++r)
      O[e0 | (r & 1 ? g0 : 0) | (r & 2 ? g1 : 0) | (r & 4 ? g2 : 0) | (r & 8 ? g3 : 0)] = x[r];
  } else {
    const SeqSeg& seg = segs[a.n_segs - 1];
    const uint32_t A = base | (uint32_t)bits10(tid, seg.gpos);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      P[seg_addr(seg, A, r)] = x[r];
      O[seg_addr(seg, A, r)] = y[r];
    }
  }
}

// Value and gradient of a state of one chunk: the forward pass (fwd.n_segs = 0:
// psi is there already), E = sum |psi|^2 D in FP64, lambda = D psi and the
// reverse sweep, a block per parameter vector.  psi goes through memory once,
// from the forward pass's layout to the reverse sweep's; lambda never does.
// (13 qubits, 6 layers, 9 parameter vectors: 385 us with launches of their own
// for the forward pass, the value, its sum and lambda, 362 so.)
template <int PREC, int LMAX>
__global__ __launch_bounds__(1 << (LMAX - 4)) void k_seq_gradient(
    SeqArgs fwd, const SeqSeg* __restrict__ fsegs, const SeqWindow* __restrict__ fwins,
    const uint32_t* __restrict__ fwords, const int32_t* __restrict__ fvsrc, const float2* __restrict__ in_vals,
    SeqArgs a, const SeqSeg* __restrict__ segs, const SeqWindow* __restrict__ wins,
    const uint32_t* __restrict__ words, const int32_t* __restrict__ vsrc, const float2* __restrict__ u, ZTerms terms,
    double* value) {
  constexpr int kBuf = (1 << LMAX) + (1 << (LMAX - 5));
  __shared__ float2 bx[kBuf], by[kBuf];
  __shared__ __attribute__((aligned(16))) float2 vwin[kSeqWinVals];
  __shared__ uint32_t wwin[kSeqWinWords];
  __shared__ double red[(1 << (LMAX - 4)) / 64];
  const int z = blockIdx.y, lane = threadIdx.x & 63;
  const int n_thr = 1 << (a.l - 4), tid = threadIdx.x & (n_thr - 1);
  const bool active = (int)threadIdx.x < n_thr;
  float2* P = const_cast<float2*>(a.in) + (int64_t)z * a.in_bs;
  float2 x[16], y[16];
  if (fwd.n_segs > 0) {
    seq_run<PREC, 1>(x, y, bx, nullptr, vwin, wwin, fwd.n_segs, fsegs, fwins, fwords, fvsrc,
                     in_vals + (int64_t)z * fwd.vals_bs, 0, tid,
                     [&](const SeqSeg& seg, uint32_t A) {
#pragma unroll
                       for (int r = 0; r < 16; ++r) x[r] = f2(seg_addr(seg, A, r) == 0 ? 1.f : 0.f, 0.f);
                     },
                     [](int, double) {});
    const uint32_t e0 = (uint32_t)bits10(tid, fwd.out_t);
    const uint32_t g0 = 1u << fwd.out_r[0], g1 = 1u << fwd.out_r[1], g2 = 1u << fwd.out_r[2], g3 = 1u << fwd.out_r[3];
#pragma unroll
    for (int r = 0; r < 16; ++r)
      P[e0 | (r & 1 ? g0 : 0) | (r & 2 ? g1 : 0) | (r & 4 ? g2 : 0) | (r & 8 ? g3 : 0)] = x[r];
    __syncthreads();
  }
  double* part = a.partials + (int64_t)z * a.pstride + (threadIdx.x >> 6);
  auto add_grad = [&](int slot, double v) {
    v = wave_sum_d(active ? v : 0.0);
    if (lane == 63) part[(int64_t)slot * kReduceBlocks] = v;
  };
  seq_run<PREC, 2>(x, y, bx, by, vwin, wwin, a.n_segs, segs, wins, words, vsrc,
                   u + (int64_t)z * a.vals_bs, 0, tid,
                   [&](const SeqSeg& seg, uint32_t A) {
                     double w[16], e = 0;
                     sum_terms16(A, terms, w);
#pragma unroll
                     for (int r = 0; r < 16; ++r) {
                       const float2 v = P[seg_addr(seg, A, r)];
                       x[r] = v;
                       y[r] = f2((float)(w[r] * v.x), (float)(w[r] * v.y));
                       e += ((double)v.x * v.x + (double)v.y * v.y) * w[r];
                     }
                     e = block_sum(active ? e : 0.0, red);
                     if (threadIdx.x == 0) value[z] = e;
                   },
                   add_grad);
}

// Expectations of several circuits, one block per circuit and parameter vector:
// each state from |0...0> through its gates, then sum |x|^2 D(x) in FP64.  (16
// circuits of 8 to 14 qubits as launches of their own took 493 us, 172 here, most of it
// four blocks at a time on the runtime's four queues.)
template <int PREC, int LMAX>
__global__ __launch_bounds__(1 << (LMAX - 4)) void k_seq_expect(SeqExpectArgs a) {
  constexpr int kBuf = (1 << LMAX) + (1 << (LMAX - 5));
  __shared__ float2 bx[kBuf];
  __shared__ __attribute__((aligned(16))) float2 vwin[kSeqWinVals];
  __shared__ uint32_t wwin[kSeqWinWords];
  const SeqCirc& c = a.c[blockIdx.x];
  const int z = blockIdx.y;
  const int n_thr = 1 << (c.l - 4), tid = threadIdx.x & (n_thr - 1);
  float2 x[16], y[16];
  seq_run<PREC, 1>(x, y, bx, nullptr, vwin, wwin, c.n_segs, c.segs, c.wins, c.words, c.vsrc,
                   c.vals + (int64_t)z * c.vals_bs, 0, tid,
                   [&](const SeqSeg& seg, uint32_t A) {
#pragma unroll
                     for (int r = 0; r < 16; ++r) x[r] = f2(seg_addr(seg, A, r) == 0 ? 1.f : 0.f, 0.f);
                   },
                   [](int, double) {});
  const uint32_t A = (uint32_t)bits10(tid, c.segs[c.n_segs - 1].gpos);
  double w[16];
#pragma unroll
  for (int mu = 0; mu < 16; ++mu) {
    double acc = 0;
    for (int i = c.term0 + c.mu_start[mu]; i < c.term0 + c.mu_start[mu + 1]; ++i)
      acc += (__popc(A & a.mask[i]) & 1) ? -a.coeff[i] : a.coeff[i];
    w[mu] = acc;
  }
  walsh16(w);
  double s = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) s += ((double)x[r].x * x[r].x + (double)x[r].y * x[r].y) * w[r];
  __syncthreads();  // vwin is no longer read
  s = block_sum((int)threadIdx.x < n_thr ? s : 0.0, reinterpret_cast<double*>(vwin));
  if (threadIdx.x == 0) c.out[z] = s;
}

template <int PREC, int NS>
void seq_launch(hipStream_t s, const SeqArgs& a, const SeqTables& t, const SeqPass& ps, const float2* vals, int chunks,
                int batch) {
  const dim3 grid(chunks, batch), block(std::max(64, 1 << (ps.l - 4)));
  if constexpr (NS == 1)
    if (ps.l <= 12) {
      hipLaunchKernelGGL((k_seq_pass<PREC, NS, 12>), grid, block, 0, s, a, t.segs + ps.first_seg, t.wins + ps.first_win,
                         t.words, t.vals, vals);
      return;
    }
  hipLaunchKernelGGL((k_seq_pass<PREC, NS, NS == 2 ? kSeqAdjMaxLocal : kSeqMaxLocal>), grid, block, 0, s, a,
                     t.segs + ps.first_seg, t.wins + ps.first_win, t.words, t.vals, vals);
}

// the pass's chunk and the bits outside it (out_pos[p]: position of address bit p in the result, NULL: p)
bool seq_args(const SeqPass& ps, int bits, int lmax, const int8_t* out_pos, SeqArgs* a) {
  if (ps.l < kSeqMinBits || ps.l > lmax || ps.l > bits || bits > 31 || ps.n_segs < 1) return false;
  std::vector<char> local(bits, 0);
  for (int j = 0; j < ps.l; ++j) {
    if (ps.lpos[j] < 0 || ps.lpos[j] >= bits || local[ps.lpos[j]]) return false;
    local[ps.lpos[j]] = 1;
  }
  a->n_rest = 0;
  for (int p = 0; p < bits; ++p)
    if (!local[p]) {
      a->rest_out[a->n_rest] = out_pos ? out_pos[p] : (int8_t)p;
      a->rest[a->n_rest++] = (int8_t)p;
    }
  a->l = ps.l;
  a->n_segs = ps.n_segs;
  return true;
}

}  // namespace

hipError_t launch_seq_expect(hipStream_t s, const SeqExpectArgs& a, int batch, int precision) {
  if (a.n < 1 || a.n > kSeqExpectMax) return hipErrorInvalidValue;
  const int l = a.c[0].l, threads = std::max(64, 1 << (l - 4));
  for (int i = 0; i < a.n; ++i) {
    const SeqCirc& c = a.c[i];
    if (c.l < kSeqMinBits || c.l > kSeqMaxLocal || std::max(64, 1 << (c.l - 4)) != threads || c.n_segs < 1 ||
        c.term0 < 0 || c.term0 + c.mu_start[16] > kSeqExpectTerms)
      return hipErrorInvalidValue;
  }
  const dim3 grid(a.n, batch), block(threads);
  if (precision == TN_PREC_BF16X3) {
    if (l <= 12) hipLaunchKernelGGL((k_seq_expect<TN_PREC_BF16X3, 12>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_seq_expect<TN_PREC_BF16X3, kSeqMaxLocal>), grid, block, 0, s, a);
  } else {
    if (l <= 12) hipLaunchKernelGGL((k_seq_expect<TN_PREC_C64, 12>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_seq_expect<TN_PREC_C64, kSeqMaxLocal>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_seq_forward(hipStream_t s, const SeqPass& ps, int bits, const SeqTables& t, const SeqSeg& last,
                              const float2* in, int64_t in_bs, float2* out, int64_t out_bs, const int8_t* out_pos,
                              const float2* vals, int64_t vals_bs, int batch, int precision) {
  SeqArgs a{};
  a.in = in; a.out = out; a.in_bs = in_bs; a.out_bs = out_bs;
  a.vals_bs = vals_bs;
  a.from_zero = in == nullptr;
  if (!seq_args(ps, bits, kSeqMaxLocal, out_pos, &a)) return hipErrorInvalidValue;
  for (int j = 0; j < 10; ++j) a.out_t[j] = out_pos ? out_pos[last.gpos[j]] : last.gpos[j];
  for (int j = 0; j < 4; ++j) a.out_r[j] = out_pos ? out_pos[last.rgpos[j]] : last.rgpos[j];
  if (precision == TN_PREC_BF16X3) seq_launch<TN_PREC_BF16X3, 1>(s, a, t, ps, vals, 1 << a.n_rest, batch);
  else seq_launch<TN_PREC_C64, 1>(s, a, t, ps, vals, 1 << a.n_rest, batch);
  return hipGetLastError();
}

int seq_adjoint_columns(const SeqPass& ps, int bits) {
  return (1 << (bits - ps.l)) * std::max(1, (1 << (ps.l - 4)) / 64);
}

hipError_t launch_seq_gradient(hipStream_t s, const SeqPass* fwd, const SeqSeg* last, const int8_t* out_pos,
                               const SeqTables& ft, const float2* in, int64_t in_bs, const SeqPass& ps, int bits,
                               const SeqTables& t, const float2* u, int64_t u_bs, float2* psi, int64_t psi_bs,
                               const ZTerms& terms, double* value, int batch, double* partials, int64_t partial_stride,
                               int precision) {
  SeqArgs f{}, a{};
  a.in = psi; a.in_bs = psi_bs;
  a.vals_bs = u_bs;
  a.partials = partials;
  a.pstride = partial_stride;
  if (!seq_args(ps, bits, kSeqAdjMaxLocal, nullptr, &a) || ps.l != bits) return hipErrorInvalidValue;
  const SeqSeg* fsegs = nullptr;
  const SeqWindow* fwins = nullptr;
  if (fwd) {
    f.vals_bs = in_bs;
    if (!seq_args(*fwd, bits, kSeqAdjMaxLocal, out_pos, &f) || fwd->l != bits) return hipErrorInvalidValue;
    for (int j = 0; j < 10; ++j) f.out_t[j] = out_pos[last->gpos[j]];
    for (int j = 0; j < 4; ++j) f.out_r[j] = out_pos[last->rgpos[j]];
    fsegs = ft.segs + fwd->first_seg;
    fwins = ft.wins + fwd->first_win;
  }
  const dim3 grid(1, batch), block(std::max(64, 1 << (bits - 4)));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, s, f, fsegs, fwins, ft.words, ft.vals, in, a, t.segs + ps.first_seg,
                       t.wins + ps.first_win, t.words, t.vals, u, terms, value);
  };
  if (precision == TN_PREC_BF16X3) {
    if (bits <= 12) go(k_seq_gradient<TN_PREC_BF16X3, 12>);
    else go(k_seq_gradient<TN_PREC_BF16X3, kSeqAdjMaxLocal>);
  } else {
    if (bits <= 12) go(k_seq_gradient<TN_PREC_C64, 12>);
    else go(k_seq_gradient<TN_PREC_C64, kSeqAdjMaxLocal>);
  }
  return hipGetLastError();
}

hipError_t launch_seq_adjoint(hipStream_t s, const SeqPass& ps, int bits, const SeqTables& t, const float2* u,
                              int64_t u_bs, float2* psi, int64_t psi_bs, float2* lam, int64_t lam_bs, int batch,
                              double* partials, int64_t partial_stride, int precision) {
  SeqArgs a{};
  a.in = psi; a.out = lam; a.in_bs = psi_bs; a.out_bs = lam_bs;
  a.vals_bs = u_bs;
  a.partials = partials;
  a.pstride = partial_stride;
  // (a state of one chunk is launch_seq_gradient's, so a chunk here is never less than the widest)
  if (!seq_args(ps, bits, kSeqAdjMaxLocal, nullptr, &a) || ps.l != kSeqAdjMaxLocal ||
      seq_adjoint_columns(ps, bits) > kReduceBlocks)
    return hipErrorInvalidValue;
  if (precision == TN_PREC_BF16X3) seq_launch<TN_PREC_BF16X3, 2>(s, a, t, ps, u, 1 << a.n_rest, batch);
  else seq_launch<TN_PREC_C64, 2>(s, a, t, ps, u, 1 << a.n_rest, batch);
  return hipGetLastError();
}

}  // namespace tnq

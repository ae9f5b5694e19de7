// Fused gate passes over a state (forward and adjoint).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "kernels.h"
#include "pass_util.h"

namespace tnq {

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
  if (a.in) {
    chunk_to_lds(buf, in, base, dep_hi, tid, nt);
  } else {  // the state |0...0>
    for (int k = 0; k < 16; ++k) buf[lds_phys(tid + k * nt)] = f2(base == 0 && tid + k * nt == 0 ? 1.f : 0.f, 0.f);
  }
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
  if (ps.l < kSweepMinLocal || ps.l > kSweepMaxLocal || ps.l > bits) return hipErrorInvalidValue;
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
    hipLaunchKernelGGL(k_adjoint_pass<TN_PREC_BF16X3>, dim3(adjoint_blocks(ps, bits), batch), dim3(threads), 0, s, a, a.gates,
                       a.segs, a.U);
  else
    hipLaunchKernelGGL(k_adjoint_pass<TN_PREC_C64>, dim3(adjoint_blocks(ps, bits), batch), dim3(threads), 0, s, a, a.gates, a.segs,
                       a.U);
  return hipGetLastError();
}

}  // namespace tnq

// The register form of a planned gate pass (see RegSeg): the pass's segments
// and gate descriptors rewritten as the operations k_sweep_regs and
// k_adjoint_regs run.  The operations keep every product, sum and rounding of
// the gate-by-gate kernels: gates are applied in the planned order, and only
// exact rewrites are made (sign flips move, runs of one gate join the runs).
#include <algorithm>
#include <vector>

#include "internal.h"

namespace tnq {

namespace {

struct Builder {
  std::vector<RegSeg>& segs;
  std::vector<RegOp>& ops;
  std::vector<RegPhase>& phases;
  std::vector<uint32_t>& words;
  const SweepPass& ps;
  int R;
  size_t s0, o0, p0, w0;
  Builder(std::vector<RegSeg>& s, std::vector<RegOp>& o, std::vector<RegPhase>& p, std::vector<uint32_t>& w,
          const SweepPass& pass, int bits)
      : segs(s), ops(o), phases(p), words(w), ps(pass), R(bits), s0(s.size()), o0(o.size()), p0(p.size()),
        w0(w.size()) {}
  void undo() {
    segs.resize(s0);
    ops.resize(o0);
    phases.resize(p0);
    words.resize(w0);
  }
  RegSeg layout(const int32_t (&rbits)[4]) const {
    RegSeg g{};
    int t = 0;
    for (int b = 0; b < ps.l; ++b) {
      bool reg = false;
      for (int j = 0; j < 4; ++j) reg |= rbits[j] == b;
      if (reg) continue;
      g.tpos[t] = b;
      g.gpos[t++] = ps.lpos[b];
    }
    for (int j = 0; j < 4; ++j) {
      g.rbits[j] = rbits[j];
      g.rgpos[j] = ps.lpos[rbits[j]];
    }
    for (int r = 0; r < 16; ++r) {
      int off = 0;
      for (int j = 0; j < 4; ++j)
        if ((r >> j) & 1) off |= 1 << rbits[j];
      g.physoff[r] = off + (off >> 5);
    }
    return g;
  }
  // the layout of the pass's loads and stores: the neighbouring segment's own when its register
  // bits leave runs of 16 elements (128 bytes) to consecutive lanes, else the top four local bits
  RegSeg io_layout(const int32_t (&rbits)[4]) const {
    const int32_t top[4] = {ps.l - 4, ps.l - 3, ps.l - 2, ps.l - 1};
    return *std::min_element(rbits, rbits + 4) >= 4 ? layout(rbits) : layout(top);
  }
  static RegOp new_op(int type) {
    RegOp o{};
    o.type = type;
    o.other = -1;
    for (int j = 0; j < 4; ++j) o.red[j] = -1;
    return o;
  }
  // address position of index bit j of a diagonal gate (not in the registers)
  template <class Desc>
  int addr(const Desc& d, int j) const {
    return d.csrc[j] >= 64 ? d.csrc[j] - 64 : ps.lpos[d.csrc[j]];
  }
  template <class Desc>
  static bool off_register(const Desc& d) {
    return d.diag && d.kreg[0] < 0 && (d.n == 1 || d.kreg[1] < 0);
  }
  // one gate of entries +-1 (Z: pattern 2, CZ: pattern 8) with a bit in the registers
  template <class Desc>
  void add_sign(RegOp& o, const Desc& d) {
    static const int ones[4] = {0xAAAA, 0xCCCC, 0xF0F0, 0xFF00};
    const int k0 = d.kreg[0], k1 = d.n == 2 ? d.kreg[1] : -1;
    if (d.n == 1) o.mask ^= ones[k0];
    else if (k0 >= 0 && k1 >= 0) o.mask ^= ones[k0] & ones[k1];
    else {
      words.push_back((uint32_t)addr(d, k0 >= 0 ? 1 : 0) | ((uint32_t)ones[k0 >= 0 ? k0 : k1] << 16));
      o.n++;
    }
  }
  template <class Desc>
  void lead_sign(RegSeg& g, const Desc& d) {
    const int p = addr(d, 0), q = d.n == 2 ? addr(d, 1) : p;
    words.push_back((uint32_t)p | ((uint32_t)q << 8));
    g.n_sign++;
  }
};

int dense_type(int form) { return form == kFormReal ? REG_REAL : form == kFormRxLike ? REG_RXLIKE : REG_DENSE; }

bool fits(const SweepPass& ps, int R) { return ps.l == kSweepMaxLocal && R <= 32 && ps.n_segs > 0; }

}  // namespace

void build_reg_pass(tn_path* path, SweepPass& ps, int R) {
  ps.reg_seg = -1;
  if (!fits(ps, R)) return;
  Builder B(path->reg_segs, path->reg_ops, path->reg_phases, path->reg_words, ps, R);
  for (int s = 0; s < ps.n_segs; ++s) {
    const SweepSegment& seg = path->segments[ps.first_seg + s];
    RegSeg g = B.layout(seg.rbits);
    const SweepGateDesc* G = path->sweep_gates.data();
    int gi = seg.first_gate;
    const int end = seg.first_gate + seg.n_gates;
    auto plain_diag = [](const SweepGateDesc& d) {
      return d.diag && d.form != kFormCount && d.form != kFormCountMember;
    };
    g.sign_off = (int32_t)B.words.size();
    for (int i = gi; i < end && plain_diag(G[i]) && Builder::off_register(G[i]); ++i)
      if (G[i].form == kFormSigns) {
        if (G[i].signs != (G[i].n == 2 ? 8 : 2)) return B.undo();
        B.lead_sign(g, G[i]);
        g.ph_used = 1;
      }
    g.phase_off = (int32_t)B.phases.size();
    for (; gi < end && plain_diag(G[gi]) && Builder::off_register(G[gi]); ++gi) {
      const SweepGateDesc& d = G[gi];
      if (d.form == kFormSigns) continue;
      RegPhase p{};
      p.p[0] = B.addr(d, 0);
      p.p[1] = d.n == 2 ? B.addr(d, 1) : -1;
      p.src = d.voff;
      p.red = -1;
      B.phases.push_back(p);
      g.n_phase++;
      g.ph_used = 1;
    }
    g.op_off = (int32_t)B.ops.size();
    for (; gi < end; ++gi) {
      const SweepGateDesc& d = G[gi];
      if (d.diag && d.form == kFormCount) {
        RegOp o = Builder::new_op(REG_COUNT);
        o.src[0] = d.voff;
        o.off = (int32_t)B.words.size();
        uint32_t tot = 0;
        uint8_t pr[6] = {0, 0, 0, 0, 0, 0};
        std::vector<uint32_t> rc;
        for (int e = 1; e <= d.n; ++e) {
          const SweepGateDesc& m = G[gi + e];
          const int k0 = m.kreg[0], k1 = m.kreg[1];
          if (k0 < 0 && k1 < 0) {
            B.words.push_back((uint32_t)B.addr(m, 0) | ((uint32_t)B.addr(m, 1) << 8));
            o.n++;
          } else if (k0 >= 0 && k1 >= 0) {
            const int lo = std::min(k0, k1), hi = std::max(k0, k1);
            pr[lo == 0 ? hi - 1 : lo == 1 ? hi + 1 : 5]++;
          } else {
            const int j = k0 >= 0 ? k0 : k1;
            rc.push_back((uint32_t)B.addr(m, k0 >= 0 ? 1 : 0) | ((uint32_t)j << 8));
            tot += 1u << (8 * j);
          }
        }
        o.n2 = (int32_t)rc.size();
        B.words.insert(B.words.end(), rc.begin(), rc.end());
        o.tot = (int32_t)tot;
        o.pc[0] = (int32_t)(pr[0] | (pr[1] << 8) | (pr[2] << 16) | ((uint32_t)pr[3] << 24));
        o.pc[1] = (int32_t)(pr[4] | (pr[5] << 8));
        B.ops.push_back(o);
        gi += d.n;
      } else if (d.diag) {
        if (Builder::off_register(d)) return B.undo();
        const int cnt = d.run_mask == 0 ? 1 : d.form == kFormSigns ? d.run_mask : __builtin_popcount(d.run_mask);
        if (d.form == kFormSigns) {
          RegOp o = Builder::new_op(REG_SIGNS);
          o.off = (int32_t)B.words.size();
          for (int j = 0; j < cnt; ++j) {
            if (G[gi + j].signs != (G[gi + j].n == 2 ? 8 : 2)) return B.undo();
            B.add_sign(o, G[gi + j]);
          }
          B.ops.push_back(o);
        } else if (d.form != kFormUnit) {
          return B.undo();
        } else if (d.n == 2) {
          RegOp o = Builder::new_op(REG_DIAG2);
          o.src[0] = d.voff;
          if (d.kreg[0] >= 0 && d.kreg[1] >= 0) {
            o.form = d.kreg[0] | (d.kreg[1] << 8);
          } else {
            const int which = d.kreg[0] >= 0 ? 1 : 0;  // the index bit outside the registers
            o.other = B.addr(d, which) | (which << 8);
            o.mask = 1 << d.kreg[1 - which];
          }
          B.ops.push_back(o);
        } else {
          RegOp o = Builder::new_op(REG_DIAG);
          for (int j = 0; j < 4; ++j) o.src[j] = d.voff;
          for (int j = 0; j < cnt; ++j) {
            o.mask |= 1 << G[gi + j].kreg[0];
            o.src[G[gi + j].kreg[0]] = G[gi + j].voff;
          }
          B.ops.push_back(o);
        }
        gi += cnt - 1;
      } else {
        if (d.n != 1) return B.undo();
        const int cnt = d.run_mask == 0 ? 1 : __builtin_popcount(d.run_mask);
        RegOp o = Builder::new_op(dense_type(d.form));
        for (int j = 0; j < 4; ++j) o.src[j] = d.voff;
        for (int j = 0; j < cnt; ++j) {
          o.mask |= 1 << G[gi + j].rb[0];
          o.src[G[gi + j].rb[0]] = G[gi + j].voff;
        }
        B.ops.push_back(o);
        gi += cnt - 1;
      }
    }
    g.n_op = (int32_t)B.ops.size() - g.op_off;
    for (int i = g.op_off; i < (int)B.ops.size(); ++i) g.ph_used |= B.ops[i].type == REG_DIAG || B.ops[i].type == REG_DIAG2;
    B.segs.push_back(g);
  }
  const RegSeg ld = B.io_layout(path->segments[ps.first_seg].rbits);
  const RegSeg st = B.io_layout(path->segments[ps.first_seg + ps.n_segs - 1].rbits);
  B.segs.push_back(ld);
  B.segs.push_back(st);
  ps.reg_seg = (int32_t)B.s0;
}

void build_adj_reg_pass(tn_path* path, SweepPass& ps, int R) {
  ps.reg_seg = -1;
  if (!fits(ps, R)) return;
  Builder B(path->adj_reg_segs, path->adj_reg_ops, path->adj_reg_phases, path->adj_reg_words, ps, R);
  for (int s = 0; s < ps.n_segs; ++s) {
    const SweepSegment& seg = path->adj_segments[ps.first_seg + s];
    RegSeg g = B.layout(seg.rbits);
    const AdjGateDesc* G = path->adj_gates.data();
    int gi = seg.first_gate;
    const int end = seg.first_gate + seg.n_gates;
    auto sign_ok = [](const AdjGateDesc& d) { return (d.form >> 8) == (d.n == 2 ? 8 : 2); };
    g.sign_off = (int32_t)B.words.size();
    for (int i = gi; i < end && Builder::off_register(G[i]); ++i)
      if (G[i].form & ADJ_DIAG_SIGNS) {
        if (!sign_ok(G[i])) return B.undo();
        B.lead_sign(g, G[i]);
        g.ph_used = 1;
      }
    g.phase_off = (int32_t)B.phases.size();
    for (; gi < end && Builder::off_register(G[gi]); ++gi) {
      const AdjGateDesc& d = G[gi];
      if (d.form & ADJ_DIAG_SIGNS) continue;
      RegPhase p{};
      p.p[0] = B.addr(d, 0);
      p.p[1] = d.n == 2 ? B.addr(d, 1) : -1;
      p.src = 16 * d.gate;
      p.red = d.red;
      for (int j = 0; j < 4; ++j) p.q[j] = d.gen[2 * j];
      g.lead_sums |= d.red >= 0;
      B.phases.push_back(p);
      g.n_phase++;
      g.ph_used = 1;
    }
    g.op_off = (int32_t)B.ops.size();
    bool have_sums = false;  // the gradient sums stay good along diagonal gates
    for (; gi < end; ++gi) {
      const AdjGateDesc& d = G[gi];
      if (d.diag) {
        if (Builder::off_register(d)) return B.undo();
        const int cnt = d.run_mask == 0                ? 1
                        : (d.form & ADJ_DIAG_SIGNS) ? d.run_mask
                                                       : __builtin_popcount(d.run_mask);
        if (d.form & ADJ_DIAG_SIGNS) {
          RegOp o = Builder::new_op(REG_SIGNS);
          o.off = (int32_t)B.words.size();
          for (int j = 0; j < cnt; ++j) {
            if (!sign_ok(G[gi + j])) return B.undo();
            B.add_sign(o, G[gi + j]);
          }
          B.ops.push_back(o);
        } else {
          RegOp o = Builder::new_op(REG_DIAG);
          for (int j = 0; j < 4; ++j) o.src[j] = 16 * d.gate;
          for (int j = 0; j < cnt; ++j) {
            const AdjGateDesc& m = G[gi + j];
            if (m.n != 1) return B.undo();
            const int k = m.kreg[0];
            o.mask |= 1 << k;
            o.src[k] = 16 * m.gate;
            o.red[k] = m.red;
            o.g0[k] = m.gen[0];
            o.g1[k] = m.gen[2];
            if (m.red >= 0 && !have_sums) {
              o.sums = 1;
              have_sums = true;
            }
          }
          B.ops.push_back(o);
          g.ph_used = 1;
        }
        gi += cnt - 1;
      } else {
        if (d.n != 1) return B.undo();
        have_sums = false;
        const int cnt = d.run_mask == 0 ? 1 : __builtin_popcount(d.run_mask);
        RegOp o = Builder::new_op(dense_type(d.uform));
        for (int j = 0; j < 4; ++j) o.src[j] = 16 * d.gate;
        for (int j = 0; j < cnt; ++j) {
          const AdjGateDesc& m = G[gi + j];
          const int k = m.rb[0];
          if (m.red >= 0 && m.form != ADJ_GEN_X && m.form != ADJ_GEN_Y) return B.undo();
          o.mask |= 1 << k;
          o.src[k] = 16 * m.gate;
          o.red[k] = m.red;
          o.gform[k] = m.form;
          o.g0[k] = m.gen[4];
        }
        B.ops.push_back(o);
        gi += cnt - 1;
      }
    }
    g.n_op = (int32_t)B.ops.size() - g.op_off;
    B.segs.push_back(g);
  }
  const RegSeg ld = B.io_layout(path->adj_segments[ps.first_seg].rbits);
  const RegSeg st = B.io_layout(path->adj_segments[ps.first_seg + ps.n_segs - 1].rbits);
  B.segs.push_back(ld);
  B.segs.push_back(st);
  ps.reg_seg = (int32_t)B.s0;
}

}  // namespace tnq

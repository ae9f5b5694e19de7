// Planning of ordered passes (see SeqPass): every gate is applied in its place
// in the given order, so results do not depend on how the state is cut.
// A pass takes gates while the bits its dense gates use fit its chunk; a
// segment takes gates while its dense gates' bits fit four register bits, the
// register bits in the order of their first gate, so that gates on successive
// register bits make one operation.  Sign flips are exact and join their
// neighbours in one mask.
#include <algorithm>
#include <vector>

#include "internal.h"

namespace tnq {

namespace {

struct SegBuild {
  std::vector<int> bits;       // address positions in the registers, by register bit
  std::vector<int> items;
};

int find(const std::vector<int>& v, int x) {
  const auto it = std::find(v.begin(), v.end(), x);
  return it == v.end() ? -1 : (int)(it - v.begin());
}

// whether the item fits the segment's registers; adds the bits it needs
bool join(SegBuild& s, const SeqItem& it) {
  if (it.diag) return true;
  if (it.n == 1) {
    if (find(s.bits, it.pos[0]) >= 0) return true;
    if (s.bits.size() >= 4) return false;
    s.bits.push_back(it.pos[0]);
    return true;
  }
  // a two-qubit gate sits on register bits (0, 1) or (2, 3)
  const int a = find(s.bits, it.pos[0]), b = find(s.bits, it.pos[1]);
  if (a >= 0 && b >= 0) return (a == 0 && b == 1) || (a == 2 && b == 3);
  if (a >= 0 || b >= 0 || (s.bits.size() != 0 && s.bits.size() != 2)) return false;
  s.bits.push_back(it.pos[0]);
  s.bits.push_back(it.pos[1]);
  return true;
}

SeqOp new_op(int type) {
  SeqOp o{};
  o.type = type;
  for (int j = 0; j < 4; ++j) o.red[j] = o.dred[j] = -1;
  return o;
}

}  // namespace

bool build_seq_program(int R, const std::vector<SeqItem>& items, int lmax, SeqProgram* out) {
  *out = SeqProgram();
  if (R < kSeqMinBits || R > 31) return false;
  const int l = std::min(R, lmax), low = std::min(5, l);
  for (size_t i = 0; i < items.size();) {
    // the pass's gates: a prefix of what is left
    std::vector<char> local(R, 0);
    int nl = 0;
    auto take = [&](int p) {
      if (!local[p]) {
        local[p] = 1;
        ++nl;
      }
    };
    for (int p = 0; p < low; ++p) take(p);
    size_t e = i;
    for (; e < items.size(); ++e) {
      const SeqItem& it = items[e];
      if (it.n < 1 || it.n > 2) return false;
      for (int j = 0; j < it.n; ++j)
        if (it.pos[j] < 0 || it.pos[j] >= R) return false;
      if (it.diag) continue;
      int extra = 0;
      for (int j = 0; j < it.n; ++j) extra += !local[it.pos[j]];
      if (nl + extra > l) break;
      for (int j = 0; j < it.n; ++j) take(it.pos[j]);
    }
    if (e == i) return false;
    for (int p = 0; p < R && nl < l; ++p) take(p);
    SeqPass ps;
    ps.l = l;
    int n = 0;
    for (int p = 0; p < R; ++p)
      if (local[p]) ps.lpos[n++] = (int8_t)p;
    for (; n < kSeqMaxLocal; ++n) ps.lpos[n] = 0;
    ps.first_seg = (int32_t)out->segs.size();
    // segments
    std::vector<SegBuild> sb(1);
    for (size_t k = i; k < e; ++k) {
      if (!join(sb.back(), items[k])) {
        sb.emplace_back();
        if (!join(sb.back(), items[k])) return false;
      }
      sb.back().items.push_back((int)k);
    }
    for (SegBuild& s : sb) {
      // unused register bits: the highest local ones, which leave the lanes consecutive addresses
      for (int j = l - 1; j >= 0 && s.bits.size() < 4; --j)
        if (find(s.bits, ps.lpos[j]) < 0) s.bits.push_back(ps.lpos[j]);
      SeqSeg g{};
      int t = 0;
      for (int j = 0; j < l; ++j) {
        const int r = find(s.bits, ps.lpos[j]);
        if (r < 0) {
          g.tpos[t] = j;
          g.gpos[t++] = ps.lpos[j];
        } else {
          g.rgpos[r] = ps.lpos[j];
          for (int c = 0; c < 16; ++c)
            if ((c >> r) & 1) g.physoff[c] |= 1 << j;
        }
      }
      for (int c = 0; c < 16; ++c) g.physoff[c] += g.physoff[c] >> 5;
      g.op_off = (int32_t)out->ops.size();
      // the operation the next item may join (-1: none), and the register bit it has reached
      int cur = -1, reached = -1;
      for (int k : s.items) {
        const SeqItem& it = items[k];
        const int k0 = find(s.bits, it.pos[0]), k1 = it.n == 2 ? find(s.bits, it.pos[1]) : -1;
        if (it.diag && it.signs >= 0 && it.red < 0) {
          static const int half[4] = {0xAAAA, 0xCCCC, 0xF0F0, 0xFF00};
          if (cur < 0 || out->ops[cur].type != SEQ_SIGNS) {
            cur = (int)out->ops.size();
            out->ops.push_back(new_op(SEQ_SIGNS));
            out->ops[cur].off = (int32_t)out->words.size();
          }
          SeqOp& o = out->ops[cur];
          const int p0 = it.pos[0], p1 = it.n == 2 ? it.pos[1] : it.pos[0];
          const int r1 = it.n == 2 ? k1 : k0;
          if (k0 >= 0 && r1 >= 0) {
            o.mask ^= half[k0] & half[r1];
          } else {
            const int ones = k0 >= 0 ? half[k0] : r1 >= 0 ? half[r1] : 0xFFFF;
            const int p = k0 >= 0 ? p1 : p0, q = r1 >= 0 ? p0 : p1;
            out->words.push_back((uint32_t)p | ((uint32_t)q << 8) | ((uint32_t)ones << 16));
            o.n++;
          }
          continue;
        }
        if (it.n == 1 && k0 >= 0) {  // a dense gate, or a diagonal on a register bit
          const bool joins = cur >= 0 && out->ops[cur].type == SEQ_BITS &&
                             (k0 > reached || (k0 == reached && it.diag && !((out->ops[cur].dmask >> k0) & 1)));
          if (!joins) {
            cur = (int)out->ops.size();
            out->ops.push_back(new_op(SEQ_BITS));
          }
          reached = k0;
          SeqOp& o = out->ops[cur];
          if (it.diag) {
            o.dmask |= 1 << k0;
            o.gfirst |= it.gate_first ? 16 << k0 : 0;
            o.dsrc[k0] = it.src;
            o.dred[k0] = it.red;
          } else {
            o.mask |= 1 << k0;
            o.gfirst |= it.gate_first ? 1 << k0 : 0;
            o.src[k0] = it.src;
            o.form[k0] = it.form;
            o.red[k0] = it.red;
            o.gform[k0] = it.gen;
          }
          continue;
        }
        cur = -1;
        SeqOp o = new_op(it.diag ? SEQ_DIAG : SEQ_DENSE2);
        o.gfirst = it.gate_first ? 1 : 0;
        o.src[0] = it.src;
        o.red[0] = it.red;
        o.gen = it.gen;
        if (it.diag) {
          o.mask = it.n;
          o.ones = it.ones;
          o.dsrc[0] = k0;
          o.dsrc[1] = k1;
          o.dsrc[2] = it.pos[0];
          o.dsrc[3] = it.pos[1];
        } else {
          if (it.red >= 0 || !((k0 == 0 && k1 == 1) || (k0 == 2 && k1 == 3))) return false;
          o.mask = k0 / 2;
          o.perm[0] = (uint32_t)it.perm;
          o.perm[1] = (uint32_t)(it.perm >> 32);
        }
        out->ops.push_back(o);
      }
      g.n_op = (int32_t)out->ops.size() - g.op_off;
      out->segs.push_back(g);
    }
    ps.n_segs = (int32_t)out->segs.size() - ps.first_seg;
    out->passes.push_back(ps);
    i = e;
  }
  return !out->passes.empty();
}

}  // namespace tnq

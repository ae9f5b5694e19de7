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
  int words = 0, vals = 0;     // upper bounds
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

// words and values an item may need at most
int words_of(const SeqItem&) { return 3; }
int vals_of(const SeqItem& it) { return it.diag ? 1 << it.n : 1 << (2 * it.n); }

}  // namespace

bool build_seq_program(int R, const std::vector<SeqItem>& items, int lmax, bool adjoint, SeqProgram* out) {
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
    ps.first_win = (int32_t)out->wins.size();
    // segments
    std::vector<SegBuild> sb(1);
    for (size_t k = i; k < e; ++k) {
      if (sb.back().words + words_of(items[k]) > kSeqWinWords || sb.back().vals + vals_of(items[k]) > kSeqWinVals ||
          !join(sb.back(), items[k])) {
        sb.emplace_back();
        if (!join(sb.back(), items[k])) return false;
      }
      sb.back().items.push_back((int)k);
      sb.back().words += words_of(items[k]);
      sb.back().vals += vals_of(items[k]);
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
      const size_t w0 = out->words.size(), v0 = out->vals.size();
      auto emit = [&](uint32_t w) { out->words.push_back(w); };
      auto values = [&](const SeqItem& it) {
        for (int j = 0; j < vals_of(it); ++j)  // (columns 2 and 3 in the order they are summed)
          out->vals.push_back(it.val[it.gray && (j & 2) ? j ^ 1 : j]);
      };
      auto slot_word = [](const SeqItem& it) { return (uint32_t)it.gen | ((uint32_t)(it.red + 1) << 8); };
      for (size_t x = 0; x < s.items.size();) {
        const SeqItem& it = items[s.items[x]];
        const int k0 = find(s.bits, it.pos[0]), k1 = it.n == 2 ? find(s.bits, it.pos[1]) : -1;
        g.n_op++;
        if (it.diag && it.signs >= 0 && it.red < 0) {  // a run of sign flips
          static const int half[4] = {0xAAAA, 0xCCCC, 0xF0F0, 0xFF00};
          int mask = 0;
          std::vector<uint32_t> w;
          for (; x < s.items.size(); ++x) {
            const SeqItem& d = items[s.items[x]];
            if (!d.diag || d.signs < 0 || d.red >= 0) break;
            const int p0 = d.pos[0], p1 = d.n == 2 ? d.pos[1] : d.pos[0];
            const int r0 = find(s.bits, p0), r1 = find(s.bits, p1);
            if (r0 >= 0 && r1 >= 0) {
              mask ^= half[r0] & half[r1];
            } else {
              const int ones = r0 >= 0 ? half[r0] : r1 >= 0 ? half[r1] : 0xFFFF;
              w.push_back((uint32_t)(r0 >= 0 ? p1 : p0) | ((uint32_t)(r1 >= 0 ? p0 : p1) << 8) | ((uint32_t)ones << 16));
            }
          }
          emit(SEQ_SIGNS | ((uint32_t)mask << 16));
          emit((uint32_t)w.size());
          out->words.insert(out->words.end(), w.begin(), w.end());
        } else if (it.n == 1 && k0 >= 0) {  // dense gates and diagonals on ascending register bits
          uint32_t head = SEQ_BITS;
          std::vector<uint32_t> w;
          int reached = -1;
          for (; x < s.items.size(); ++x) {
            const SeqItem& d = items[s.items[x]];
            const int r = find(s.bits, d.pos[0]);
            if (d.n != 1 || r < 0 || (d.diag && d.signs >= 0 && d.red < 0)) break;
            if (!(r > reached || (r == reached && d.diag && !((head >> (8 + r)) & 1)))) break;
            reached = r;
            if (d.diag) {
              head |= (1u << (8 + r)) | (d.gate_first ? 1u << (16 + r) : 0);
            } else {
              head |= (1u << (4 + r)) | (d.gate_first ? 1u << (12 + r) : 0) | ((uint32_t)(d.form & 3) << (20 + 2 * r));
            }
            w.push_back(slot_word(d));
            values(d);
          }
          emit(head);
          if (adjoint) out->words.insert(out->words.end(), w.begin(), w.end());
        } else if (it.diag) {
          emit(SEQ_DIAG | ((uint32_t)it.n << 4) | (it.gate_first ? 1u << 12 : 0));
          emit((uint32_t)(k0 + 1) | ((uint32_t)(k1 + 1) << 4) | ((uint32_t)it.pos[0] << 8) | ((uint32_t)it.pos[1] << 16));
          emit((uint32_t)it.ones | ((uint32_t)it.gen << 4) | ((uint32_t)(it.red + 1) << 8));
          values(it);
          ++x;
        } else {
          if (it.red >= 0 || !((k0 == 0 && k1 == 1) || (k0 == 2 && k1 == 3))) return false;
          emit(SEQ_DENSE2 | ((uint32_t)(k0 / 2) << 4) | (it.gate_first ? 1u << 12 : 0) | (it.gray ? 1u << 13 : 0));
          values(it);
          ++x;
        }
      }
      const int nw = (int)(out->words.size() - w0), nv = (int)(out->vals.size() - v0);
      if (nw > kSeqWinWords || nv > kSeqWinVals) return false;
      SeqWindow* win = (int)out->wins.size() > ps.first_win ? &out->wins.back() : nullptr;
      if (!win || win->n_words + nw > kSeqWinWords || win->n_vals + nv > kSeqWinVals) {
        out->wins.push_back(SeqWindow{0, (int32_t)w0, 0, (int32_t)v0, 0, {0, 0, 0}});
        win = &out->wins.back();
      }
      win->n_segs++;
      win->n_words += nw;
      win->n_vals += nv;
      out->segs.push_back(g);
    }
    ps.n_wins = (int32_t)out->wins.size() - ps.first_win;
    ps.n_segs = (int32_t)out->segs.size() - ps.first_seg;
    out->passes.push_back(ps);
    i = e;
  }
  return !out->passes.empty();
}

}  // namespace tnq

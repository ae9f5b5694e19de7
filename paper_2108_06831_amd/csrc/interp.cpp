// Plans the interpreter's work lists that stay in LDS.
//
// A list is a tree of small contractions (SmallStep).  With a place in LDS for
// every operand and result, a level costs a barrier and its arithmetic; with
// results in memory it costs a store, a load of the next level's operands and
// descriptors, and the waits between them (4 us a level against 1).
#include <algorithm>
#include <map>
#include <vector>

#include "internal.h"

namespace tnq {
namespace {

// Places of power-of-two sizes at multiples of their size, first fit; a bit per element.
struct Places {
  static_assert(kResElems % 64 == 0, "whole words");
  uint64_t used[kResElems / 64] = {};

  int take(int n) {
    if (n < 64) {
      const uint64_t mask = ((uint64_t)1 << n) - 1;
      for (int w = 0; w < kResElems / 64; ++w) {
        if (used[w] == ~(uint64_t)0) continue;
        for (int at = 0; at < 64; at += n)
          if (!(used[w] & (mask << at))) {
            used[w] |= mask << at;
            return 64 * w + at;
          }
      }
      return -1;
    }
    for (int at = 0; at + n <= kResElems; at += n)
      if (std::find_if(used + at / 64, used + (at + n) / 64, [](uint64_t u) { return u != 0; }) == used + (at + n) / 64) {
        set(at, n, true);
        return at;
      }
    return -1;
  }
  void set(int at, int n, bool on) {  // (at: a multiple of n)
    if (n < 64) {
      const uint64_t mask = (((uint64_t)1 << n) - 1) << (at & 63);
      used[at / 64] = on ? used[at / 64] | mask : used[at / 64] & ~mask;
    } else {
      std::fill(used + at / 64, used + (at + n) / 64, on ? ~(uint64_t)0 : 0);
    }
  }
};

}  // namespace

// Whether the list's steps, levels and inputs are within the kernel's tables and LDS.
bool resident_list_fits(const std::vector<SmallStep>& steps, const std::vector<int>& level) {
  const int S = (int)steps.size();
  if (S < 1 || S > kResSteps) return false;
  int levels = 0;
  int64_t inputs = 0;
  for (int s = 0; s < S; ++s) {
    const SmallStep& d = steps[s];
    if (d.c_bits > kSmallMaxBits || d.a_bits > kSmallMaxBits || d.b_bits > kSmallMaxBits) return false;
    levels += s == 0 || level[s] != level[s - 1];
    if (d.a_buf == BUF_IN) inputs += (int64_t)1 << d.a_bits;
    if (d.b_buf == BUF_IN) inputs += (int64_t)1 << d.b_bits;
  }
  return levels <= kResLevels && inputs <= kResElems;
}

bool add_resident_list(const std::vector<SmallStep>& steps, const std::vector<int>& level, ResProgram* prog) {
  const int S = (int)steps.size();
  if (!resident_list_fits(steps, level)) return false;
  ResList L;
  L.level0 = (int32_t)prog->levels.size();
  L.step0 = (int32_t)prog->steps.size();
  L.copy0 = (int32_t)prog->copy.size();
  L.n_steps = S;
  L.n_levels = 0;
  L.c_off = steps[S - 1].c_off;
  std::vector<ResLevel> levels;
  std::vector<ResStep> out(S);
  std::vector<ResItem> items;
  std::vector<uint32_t> copy;
  Places places;
  // inputs first, the largest first, so that they lie from 0 without gaps
  struct Input {
    int step, side, bits;
    int64_t off;
  };
  std::vector<Input> inputs;
  for (int s = 0; s < S; ++s) {
    const SmallStep& d = steps[s];
    if (d.a_buf == BUF_IN) inputs.push_back({s, 0, d.a_bits, d.a_off});
    if (d.b_buf == BUF_IN) inputs.push_back({s, 1, d.b_bits, d.b_off});
  }
  std::stable_sort(inputs.begin(), inputs.end(), [](const Input& x, const Input& y) { return x.bits > y.bits; });
  for (const Input& in : inputs) {
    const int n = 1 << in.bits, at = (int)copy.size();
    if (in.off < 0 || in.off + n > ((int64_t)1 << 32)) return false;
    (in.side ? out[in.step].b : out[in.step].a) = (uint16_t)at;
    places.set(at, n, true);
    for (int e = 0; e < n; ++e) copy.push_back((uint32_t)(in.off + e));
  }
  std::map<int64_t, int> result_at;  // workspace offset -> place
  for (int s0 = 0; s0 < S;) {
    int s1 = s0;
    while (s1 < S && level[s1] == level[s0]) ++s1;
    ++L.n_levels;
    int64_t total = 0;
    for (int s = s0; s < s1; ++s) {
      const SmallStep& d = steps[s];
      ResStep& r = out[s];
      for (int side = 0; side < 2; ++side) {
        if ((side ? d.b_buf : d.a_buf) == BUF_IN) continue;
        auto it = result_at.find(side ? d.b_off : d.a_off);
        if (it == result_at.end()) return false;
        (side ? r.b : r.a) = (uint16_t)it->second;
      }
      r.c_bits = (uint8_t)d.c_bits;
      r.k_bits = (uint8_t)d.k_bits;
      for (int j = 0; j < kSmallMaxBits; ++j) {
        r.apos[j] = d.apos[j];
        r.bpos[j] = d.bpos[j];
        r.ka[j] = d.ka[j];
        r.kb[j] = d.kb[j];
      }
      r.pad[0] = r.pad[1] = 0;
      if (s == S - 1) {
        r.c = kResOut;
      } else {
        const int at = places.take(1 << d.c_bits);
        if (at < 0) return false;
        r.c = (uint16_t)at;
        result_at[d.c_off] = at;
      }
      total += ((int64_t)1 << d.c_bits) * (((int64_t)1 << d.k_bits) + 4);
    }
    // work items: about equal work (outputs times summed terms, plus the store) per thread
    const size_t first = items.size();
    int64_t target = std::max<int64_t>(1, (total + kSmallThreads - 1) / kSmallThreads);
    auto item_bits = [&](const SmallStep& d) {  // the step has 2^item_bits items
      const int64_t per = ((int64_t)1 << d.k_bits) + 4;
      int lc = 0;  // log2 of the outputs per item
      while (lc < d.c_bits && ((int64_t)2 << lc) * per <= target) ++lc;
      return d.c_bits - lc;
    };
    for (;; target *= 2) {
      int64_t n = 0;
      for (int s = s0; s < s1; ++s) n += (int64_t)1 << item_bits(steps[s]);
      if (n <= kSmallMaxItems) break;
    }
    for (int s = s0; s < s1; ++s) {
      const SmallStep& d = steps[s];
      const int qb = item_bits(d);
      const size_t i0 = items.size();
      for (int j = 0; j < (1 << qb); ++j) {
        ResItem it;
        it.a = out[s].a;
        it.b = out[s].b;
        if (j) {  // the operands of j without its lowest bit, and that bit's places
          const int p = __builtin_ctz(j);
          it.a = items[i0 + (j & (j - 1))].a | (uint16_t)(d.apos[p] >= 0 ? 1 << d.apos[p] : 0);
          it.b = items[i0 + (j & (j - 1))].b | (uint16_t)(d.bpos[p] >= 0 ? 1 << d.bpos[p] : 0);
        }
        it.what = (uint32_t)s | (uint32_t)j << 8 | (uint32_t)qb << 20;
        items.push_back(it);
      }
    }
    levels.push_back({(int32_t)(prog->items.size() + first), (int32_t)(items.size() - first)});
    // the level's operands are no longer read
    for (int s = s0; s < s1; ++s) {
      places.set(out[s].a, 1 << steps[s].a_bits, false);
      places.set(out[s].b, 1 << steps[s].b_bits, false);
    }
    s0 = s1;
  }
  L.n_copy = (int32_t)copy.size();
  prog->lists.push_back(L);
  prog->levels.insert(prog->levels.end(), levels.begin(), levels.end());
  prog->steps.insert(prog->steps.end(), out.begin(), out.end());
  prog->items.insert(prog->items.end(), items.begin(), items.end());
  prog->copy.insert(prog->copy.end(), copy.begin(), copy.end());
  return true;
}

}  // namespace tnq

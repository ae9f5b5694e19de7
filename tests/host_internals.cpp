// Reads of the library's host data structures that its C interface does not show
// (built and called by test_host_planning.py).
#include <algorithm>
#include <chrono>
#include <vector>

#include "internal.h"

using namespace tnq;

namespace {
int64_t table_entries(const tn_path& p) {
  return (int64_t)(p.res.lists.size() + p.res.items.size() + p.small_items.size() + p.outers.size() + p.reg_segs.size() +
                   p.reg_ops.size() + p.seq.prog.segs.size() + p.q_steps.size());
}
}  // namespace

// The order of `full` compiled for the run-time model alone: its modelled time, and how many entries the tables
// that only a launch reads have; entries_full: those of `full`.
extern "C" int priced_program(const tn_network* net, const tn_path* full, double* seconds, int64_t* entries,
                              int64_t* entries_full) {
  tn_path p;
  p.pairs = full->pairs;
  p.n_small = full->n_small;
  p.small_region = full->small_region;
  const std::vector<int32_t> layout = output_layout(net);
  const tn_status st = compile_program(net, &p, &layout, true);
  *seconds = modeled_seconds(&p);
  *entries = table_entries(p);
  *entries_full = table_entries(*full);
  return st;
}

// Least seconds of `runs` compilations of the order of `full`: whole, and for the run-time model alone.
extern "C" void compile_seconds(const tn_network* net, const tn_path* full, int runs, double* whole, double* priced) {
  const std::vector<int32_t> layout = output_layout(net);
  for (int price = 0; price < 2; ++price) {
    double best = 1e9;
    for (int r = 0; r < runs; ++r) {
      tn_path p;
      p.pairs = full->pairs;
      p.n_small = full->n_small;
      p.small_region = full->small_region;
      const auto t0 = std::chrono::steady_clock::now();
      (void)compile_program(net, &p, &layout, price != 0);
      best = std::min(best, std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count());
    }
    *(price ? priced : whole) = best;
  }
}

// The lists that stay in LDS, run on the host: every tensor's elements carry the id of the tensor that was written
// last.  Returns -1 if the path has no such lists, else the number of operand reads or writes that find another
// tensor's elements, or lie outside LDS.
extern "C" int64_t resident_overlaps(const tn_path* p) {
  const ResProgram& R = p->res;
  if (R.lists.empty()) return -1;
  int64_t bad = 0;
  for (const ResList& L : R.lists) {
    std::vector<int64_t> owner(kResElems, -1);  // >= 0: result of that step; -2: an input element
    std::vector<int> last_level(L.n_steps, 0);
    for (int e = 0; e < L.n_copy; ++e) owner[e] = -2;
    for (int lv = 0; lv < L.n_levels; ++lv) {
      const ResLevel& V = R.levels[L.level0 + lv];
      std::vector<int64_t> next = owner;  // a level's results are read from the next one on
      std::vector<char> written(kResElems, 0), read(kResElems, 0);
      for (int i = V.item0; i < V.item0 + V.n_items; ++i) {
        const ResItem& it = R.items[i];
        const int s = it.what & 255, j0 = (it.what >> 8) & 4095, qb = it.what >> 20;
        const ResStep& st = R.steps[L.step0 + s];
        for (int t = 0; t < (1 << (st.c_bits - qb)); ++t) {
          const int o = j0 | (t << qb);
          int a = st.a, b = st.b, a0 = it.a, b0 = it.b;
          for (int q = 0; q < st.c_bits; ++q)
            if ((o >> q) & 1) {
              if (st.apos[q] >= 0) a |= 1 << st.apos[q];
              if (st.bpos[q] >= 0) b |= 1 << st.bpos[q];
            }
          if (t == 0 && (a != a0 || b != b0)) ++bad;  // the item's own addresses
          for (int k = 0; k < (1 << st.k_bits); ++k) {
            int ak = a, bk = b;
            for (int q = 0; q < st.k_bits; ++q)
              if ((k >> q) & 1) {
                ak |= 1 << st.ka[q];
                bk |= 1 << st.kb[q];
              }
            for (int x : {ak, bk}) {
              if (x < 0 || x >= kResElems || owner[x] == -1) ++bad;
              else read[x] = 1;
            }
            // one owner per operand: that of its first element
            if (ak < kResElems && owner[ak] != owner[st.a]) ++bad;
            if (bk < kResElems && owner[bk] != owner[st.b]) ++bad;
          }
          if (st.c != kResOut) {
            if (st.c + o >= kResElems || written[st.c + o]) ++bad;
            else {
              written[st.c + o] = 1;
              next[st.c + o] = s;
            }
          }
        }
      }
      for (int e = 0; e < kResElems; ++e) bad += written[e] && read[e];
      owner = next;
    }
  }
  return bad;
}

// The gradient slots of a network; table: room for n_params + 1 + slots entries (may be NULL); returns the slots.
extern "C" int slot_table(const tn_network* net, int32_t* table, double* seconds) {
  std::vector<int32_t> of_gate, t;
  const auto t0 = std::chrono::steady_clock::now();
  const int n = gradient_slots(*net, &of_gate, &t);
  *seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  if (table) std::copy(t.begin(), t.end(), table);
  return n;
}

// Default launch shape of a product whose indices lie in blocks (bit counts of its batch, m, n and k), and the shape
// that follows from the sizes alone, in the orientation that runs.
extern "C" void default_shape(int b, int m, int n, int k, int prec, int32_t* tile, int32_t* split, int32_t* by_blocks) {
  GemmDesc g{};
  g.batch = (int64_t)1 << b;
  g.M = (int64_t)1 << m;
  g.N = (int64_t)1 << n;
  g.K = (int64_t)1 << k;
  g.nbb = b;
  g.nbm = m;
  g.nbn = n;
  g.nbk = k;
  auto put = [](int8_t* pos, int count, int at) {
    for (int j = 0; j < count; ++j) pos[j] = (int8_t)(at + j);
  };
  put(g.a_k, k, 0);
  put(g.a_m, m, k);
  put(g.a_b, b, k + m);
  put(g.b_n, n, 0);
  put(g.b_k, k, n);
  put(g.b_b, b, n + k);
  put(g.c_n, n, 0);
  put(g.c_m, m, n);
  put(g.c_b, b, n + m);
  GemmDesc t = g;  // B^T A^T
  std::swap(t.M, t.N);
  std::swap(t.nbm, t.nbn);
  std::copy(g.b_b, g.b_b + kGemmMaxBits, t.a_b);
  std::copy(g.b_n, g.b_n + kGemmMaxBits, t.a_m);
  std::copy(g.b_k, g.b_k + kGemmMaxBits, t.a_k);
  std::copy(g.a_b, g.a_b + kGemmMaxBits, t.b_b);
  std::copy(g.a_m, g.a_m + kGemmMaxBits, t.b_n);
  std::copy(g.a_k, g.a_k + kGemmMaxBits, t.b_k);
  std::swap_ranges(t.c_m, t.c_m + kGemmMaxBits, t.c_n);
  GemmDesc gm[2] = {g, t};
  for (GemmDesc& x : gm) {
    int by, sp;
    gemm_tile_by_blocks(x, &by, &sp);
    x.max_split = sp;
    if ((by != kGemmVector || x.K >= 256) && b + m + n + 3 <= 22 && k >= 6) x.max_split = kGemmMaxSplit;
  }
  const int o = gemm_default_launch(gm, prec);
  int sp;
  gemm_tile_by_blocks(gm[o], by_blocks, &sp);
  *tile = gm[o].tile[prec];
  *split = gm[o].split[prec];
}

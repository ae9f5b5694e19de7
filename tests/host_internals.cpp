// Reads of the library's host data structures that its C interface does not show
// (built and called by test_host_planning.py).
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

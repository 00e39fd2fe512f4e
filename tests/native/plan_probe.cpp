// Test helper (a shared library loaded with ctypes beside libxg.so): what
// the planner and the emitters made of a loaded program, without a GPU.
#include <fstream>
#include <string>
#include <vector>

#include "xg_program.h"

extern "C" {

// The source of the persistent kernel over k programs, written to `path`.
int probe_batch_source(xg_program** ps, int k, const char* path) {
  std::string src;
  const xg_status st = xg::batch_source(std::vector<xg_program*>(ps, ps + k), src);
  if (st == XG_OK) std::ofstream(path) << src;
  return (int)st;
}

// Whether n instances of `mode` run the plan for few tiles.
int probe_few(xg_program* p, int mode, long long n) {
  std::lock_guard<std::mutex> lk(p->mu);
  return xg::pick_few(p, mode, n);
}

// Devices that hold the code of a plan of `mode`.
int probe_loaded(xg_program* p, int mode, int few) { return (int)mode_state(p, mode, few != 0).devs.size(); }

// Whether the code objects of a plan of `mode` are compiled.
int probe_compiled(xg_program* p, int mode, int few) { return mode_state(p, mode, few != 0).compiled; }

// A hash of the sources of the plan that n instances of `mode` run, and its phases.
unsigned long long probe_code(xg_program* p, int mode, long long n, int* phases) {
  std::lock_guard<std::mutex> lk(p->mu);
  std::string err;
  if (!xg::plan_mode(p, mode, err)) return 0;
  const xg::ModeState& M = mode_state(p, mode, xg::pick_few(p, mode, n));
  *phases = M.plan.n_phases;
  uint64_t h = 1469598103934665603ull;
  for (const std::string& s : M.srcs) h = xg::fnv1a(s, h);
  return h;
}

// Sources (hashes) of the tuning candidates of `mode` for n instances, and
// whether each is one of the library's plans.  Returns their number.
int probe_candidates(xg_program* p, int mode, long long n, unsigned long long* hash, int* library, int most) {
  std::vector<xg::Candidate> cands;
  std::vector<std::unique_ptr<xg_program>> trials;
  std::string err;
  if (!xg::plan_candidates(p, n, mode, cands, trials, err)) return -1;
  for (size_t i = 0; i < cands.size() && (int)i < most; ++i) {
    library[i] = cands[i].library;
    hash[i] = 1469598103934665603ull;
    for (const std::string& s : trials[i]->m[mode].srcs) hash[i] = xg::fnv1a(s, hash[i]);
  }
  return (int)cands.size();
}

// Workgroup sizes and sources (hashes) of the batch autotuner's candidates.
int probe_batch_candidates(xg_program** ps, int k, const int64_t* n, int* block, unsigned long long* hash) {
  int i = 0;
  for (auto& c : xg::batch_candidate_sources(ps, k, n)) {
    block[i] = c.first;
    hash[i++] = xg::fnv1a(c.second, 1469598103934665603ull);
  }
  return i;
}

// Workgroups of a batch launch.
long long probe_batch_grid(int k, const int64_t* tiles, const int64_t* cost, long long resident, long long cus) {
  return xg::batch_grid({tiles, tiles + k}, {cost, cost + k}, resident, cus);
}

// Gives the plan for few tiles a source that does not compile.
void probe_spoil_few(xg_program* p, int mode) {
  std::lock_guard<std::mutex> lk(p->mu);
  (void)xg::pick_few(p, mode, 1);
  p->few[mode].srcs.assign(1, "#error planted by a test\n");
}

}  // extern "C"

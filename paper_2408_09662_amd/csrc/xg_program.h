// Program object shared by the C-ABI implementation files.
#pragma once

#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>

#include "xg_internal.h"

namespace xg {

// LDS available to spill slots: 160 KiB per workgroup on gfx950 minus 512 B
// for a kernel's own shared variables (the batch kernel's job index).
constexpr int64_t kLdsSpillBytes = 160 * 1024 - 512;

struct DevMod {
  int device = -1;
  std::vector<hipModule_t> mods;
  std::vector<hipFunction_t> fns;
};

// One evaluation mode (0 forward, 1 adjoint, 2 fused forward + adjoint):
// its program, plan, generated sources and loaded code.
struct ModeState {
  bool planned = false;
  Graph g;
  Plan plan;
  EmitStats est;
  int64_t recompute_ops = 0;
  int64_t cost = 0;     // modelled time of a tile (units of one vector operation)
  int64_t n_nodes = 0, n_ops = 0;  // SSA values and operations before products join sums
  EmitOptions eo;       // what the sources were emitted with (est counts that emission)
  std::vector<std::string> srcs;
  std::vector<CodeObject> cos;
  bool compiled = false;
  bool checked = false;  // kernels checked against their launch (host only)
  double compile_ms = 0;
  int cache_hits = 0;
  std::vector<DevMod> devs;
  int32_t ws_slots() const { return plan.n_ws + est.extra_ws; }
};

// Workspace bytes for n instances: per block of block*ipt instances,
// ws_slots x block x ipt elements.
inline size_t ws_bytes_of(int64_t n, int32_t slots, int block, int ipt, size_t es) {
  const int64_t per = (int64_t)block * ipt;
  const int64_t tiles = (n + per - 1) / per;
  return (size_t)tiles * (size_t)slots * (size_t)per * es;
}

// o with the defaults filled in; `library`: the budgets are the library's
// (library_budget of the mode), else what they are beside other options
xg_options defaults(const xg_options* o, int dtype, bool library);
EmitOptions emit_options_of(const xg_options& o);
bool check_opts(const xg_options& o, int dtype, std::string& err);

}  // namespace xg

struct xg_program {
  xg::Graph g;
  xg_options opt;   // forward evaluation (mode 0)
  xg_options aopt;  // adjoint evaluations (modes 1 and 2); the load options until tuned
  xg::ModeState m[3];
  // A mode whose plan the caller left to the library (every launch option
  // 0, not tuned) has a second plan for launches with too few tiles to fill
  // the chip (pick_few).  Both plans of a mode round alike, so which one
  // runs shows in the time only.
  bool library_plan[3] = {false, false, false};
  // A mode whose register and LDS budgets are the library's: plan_mode may
  // lower them by what the program's graph holds.  Forward: the caller set
  // neither them nor the workgroup's shape.  Adjoint: library_plan, as its
  // budgets were measured with the library's chunks.
  bool library_budget[3] = {false, false, false};
  // Forward phased plans ranked by transfers (form_few chose so, or tuning did)
  bool transfers_first = false, few_transfers_first = false;
  int few_state[3] = {0, 0, 0};  // 0 not formed yet, 1 formed, -1 none
  int64_t few_most[3] = {0, 0, 0};  // most instances that run it
  xg_options few_opt[3];
  xg::ModeState few[3];
  std::mutex mu;
  // HIP graphs whose kernel nodes run this program's loaded code.  While
  // any exists the code stays loaded: re-planning (autotuning) is refused
  // and xg_program_free only marks the program, which the last graph's
  // xg_graph_free then frees.
  int live_graphs = 0;
  bool free_pending = false;
};

// Options a mode is planned and launched with (`few`: its plan for few tiles).
inline const xg_options& mode_opt(const xg_program* p, int mode, bool few = false) {
  return few ? p->few_opt[mode] : mode == 0 ? p->opt : p->aopt;
}
inline xg::ModeState& mode_state(xg_program* p, int mode, bool few) { return few ? p->few[mode] : p->m[mode]; }

namespace xg {
bool plan_mode(xg_program* p, int mode, std::string& err, bool few = false);
// hiprtc and host checks only (no device); *code as for compile_mode
bool build_code(xg_program* p, int mode, std::string& err, xg_status* code = nullptr, bool few = false);
// + load on the current device; on failure *code (if given) says why:
// XG_ECOMPILE, XG_EUNSUPPORTED (a kernel that cannot be launched as
// planned) or XG_EDEVICE
bool compile_mode(xg_program* p, int mode, std::string& err, xg_status* code = nullptr, bool few = false);
// build_code of every plan the mode has, and those plans loaded too
bool build_plans(xg_program* p, int mode, std::string& err, xg_status* code);
bool load_plans(xg_program* p, int mode, std::string& err, xg_status* code);
// Loads what n instances of `mode` run on `stream` and says which plan that is
bool load_for(xg_program* p, int mode, int64_t n, void* stream, bool& few, std::string& err, xg_status* code);
// Whether n instances of `mode` run the plan for few tiles (formed and
// planned by this call if need be; the caller holds p->mu)
bool pick_few(xg_program* p, int mode, int64_t n);
// Launch options of the library's own plans, before any rule on n: the
// values xg_autotune's candidates are spread around
constexpr int kTuneRegs64 = 112, kTuneRegs32 = 200;
// A plan that tuning may give a mode.
struct Candidate {
  xg_options o;
  // what options do not say of a plan: the library's rules lower its budgets,
  // its phases are ranked by transfers
  bool library = false, transfers_first = false;
  Candidate(const xg_options& o_, bool l = false, bool t = false) : o(o_), library(l), transfers_first(t) {}
};
// The candidates for n instances of `mode` (cooperative plans that cannot be
// formed left out) and, for each, a copy of p planned with it
bool plan_candidates(xg_program* p, int64_t n, int mode, std::vector<Candidate>& cands,
                     std::vector<std::unique_ptr<xg_program>>& trials, std::string& err);
// The source of the persistent kernel over progs (host only: nothing is compiled)
xg_status batch_source(const std::vector<xg_program*>& progs, std::string& src);
// Workgroups of a batch launch of tiles[k] tiles of cost[k] each, of which
// `resident` fit the chip's `cus` CUs at once
int64_t batch_grid(const std::vector<int64_t>& tiles, const std::vector<int64_t>& cost, int64_t resident, int64_t cus);
// The workgroup sizes xg_batch_autotune tries for n[i] instances of program i, and the sources
std::vector<std::pair<int, std::string>> batch_candidate_sources(xg_program* const* progs, int32_t k, const int64_t* n);
void reset_mode(xg_program* p, int mode);  // drain, unload, forget the plan
void destroy_program(xg_program* p);       // unload every mode and delete
// xg_eval_adjoint on the kernels already loaded on the current device, with
// a workspace of ws_cap bytes at ws; compiles, loads and allocates nothing
xg_status eval_adjoint_loaded(xg_program* p, int64_t n, const void* const* d_in, const int64_t* ld_in,
                              const void* const* d_out_bar, const int64_t* ld_out_bar,
                              void* const* d_out, const int64_t* ld_out, void* const* d_in_bar,
                              const int64_t* ld_in_bar, void* ws, size_t ws_cap, void* stream);
// device address of the fixed scratch array on the current device (looked
// up on the first call per device)
bool noalloc_scratch(void** ptr, std::string& err);
}  // namespace xg

// Persistent multi-program launch, HIP graph capture and the autotuner.
//
// The paper launches one kernel per function.  A batch here evaluates K
// distinct programs -- of uneven size, instance count and precision -- in
// ONE launch: a grid sized to the chip's resident capacity, whose
// workgroups pull (program, tile) jobs from a 64-bit counter in the
// workspace until all are taken.  Jobs are ordered longest first (by
// operations per instance), so the long tiles start early and the short ones
// fill the tail.  Each program's chunk bodies are emitted exactly as for its
// standalone kernels, as noinline device functions in a namespace of their
// own (each with its own element type); they read their pointers from the
// kernel's argument block, found at a fixed distance before the implicit
// kernel arguments, so they stay in scalar registers.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <memory>
#include <sstream>

#include <hip/hip_runtime.h>

#include "xg_internal.h"
#include "xg_program.h"

using namespace xg;

namespace {

constexpr size_t kCounterBytes = 256;

size_t align256(size_t v) { return (v + 255) / 256 * 256; }
size_t esize_of(int dtype) { return dtype == XG_F32 ? 4 : 8; }

struct BatchDev {
  int device = -1;
  hipModule_t mod = nullptr;
  hipFunction_t kern = nullptr, reset = nullptr;
  int grid = 0, cus = 0;
};

// Instances per job of program p in a batch, and the workgroup size it needs.
int64_t tile_of(const xg_program* p) {
  return p->opt.waves > 1 ? 64 : (int64_t)p->opt.block * p->opt.ipt;
}
int launch_block_of(const xg_program* p) {
  return p->opt.waves > 1 ? 64 * p->opt.waves : p->opt.block;
}

}  // namespace

struct xg_batch {
  std::vector<xg_program*> progs;
  std::vector<xg_program*> owned;  // programs the batch made (autotuned copies), freed with it
  std::vector<int> order;       // job order: program indices, longest tiles first
  int block = 64, ipt = 1;
  std::string src;
  CodeObject co;
  std::vector<BatchDev> devs;
  size_t bargs_size = 0;
  std::mutex mu;
  // HIP graphs launching this batch's kernel: while any exists,
  // xg_batch_free only marks the batch and the last graph frees it
  int live_graphs = 0;
  bool free_pending = false;
};

struct xg_graph {
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  // the program or batch whose loaded kernels the graph launches
  xg_program* prog = nullptr;
  xg_batch* batch = nullptr;
};

namespace {

std::string build_batch_source(xg_batch* b, std::string& err) {
  const int K = (int)b->progs.size();
  std::ostringstream s;
  s << "// generated by xg: persistent batch of " << K << " programs\n";
  s << contract_pragma(b->progs[0]->opt.strict != 0);
  size_t lds_bytes = 0;
  bool any_phased = false;
  // LDS need of every program (largest chunk; all waves of a cooperative
  // tile; a phased tile's exchange slots too)
  for (int k = 0; k < K; ++k) {
    ModeState& M = b->progs[k]->m[0];
    size_t need = (size_t)M.est.lds_slots * launch_block_of(b->progs[k]) * esize_of(M.g.dtype);
    if (M.plan.phased) {
      need += (size_t)M.plan.n_xch * 64 * esize_of(M.g.dtype);
      any_phased = true;
    }
    lds_bytes = std::max(lds_bytes, need);
  }
  if (lds_bytes > 160 * 1024) { err = "batch: LDS need exceeds 160 KiB"; return ""; }
  if (lds_bytes) s << "__shared__ __attribute__((aligned(16))) char xg_lds_raw[" << lds_bytes << "];\n";
  // phased tiles: every wave of the workgroup passes the same barriers in
  // each job (all of them run the job)
  if (any_phased) s << "#define xg_barrier() __syncthreads()\n";
  // per-program types and argument structs
  for (int k = 0; k < K; ++k) {
    const Graph& g = b->progs[k]->m[0].g;
    s << "namespace P" << k << " {\n" << emit_preamble(g, b->progs[k]->m[0].eo);
    s << "struct Args { long long n; T* ws;";
    for (size_t a = 0; a < g.nnz_in.size(); ++a) s << " const T* in" << a << "; long long ldi" << a << ";";
    for (size_t a = 0; a < g.nnz_out.size(); ++a) s << " T* out" << a << "; long long ldo" << a << ";";
    s << " };\n}\n";
  }
  s << "struct BArgs { unsigned long long* counter; long long total; long long cum[" << K + 1 << "];";
  for (int k = 0; k < K; ++k) s << " P" << k << "::Args a" << k << ";";
  s << " };\n";
  s << "#define XG_BARGS ((const BArgs*)((const char*)__builtin_amdgcn_implicitarg_ptr() - sizeof(BArgs)))\n";
  for (int k = 0; k < K; ++k) {
    ModeState& M = b->progs[k]->m[0];
    const Graph& g = M.g;
    // emitted as the plan was (its register budget may be below the program's
    // option): the tile's LDS and workspace are sized from M.est
    const EmitOptions& eo = M.eo;
    std::ostringstream pro;
    pro << "  const P" << k << "::Args& A = XG_BARGS->a" << k << ";\n";
    pro << "  const long long n = A.n; T* __restrict__ ws = A.ws;\n";
    for (size_t a = 0; a < g.nnz_in.size(); ++a)
      pro << "  const T* __restrict__ in" << a << " = A.in" << a << "; const long long ldi" << a
          << " = A.ldi" << a << ";\n";
    for (size_t a = 0; a < g.nnz_out.size(); ++a)
      pro << "  T* __restrict__ out" << a << " = A.out" << a << "; const long long ldo" << a
          << " = A.ldo" << a << ";\n";
    s << contract_pragma(b->progs[0]->opt.strict != 0) << contract_end(b->progs[0]->opt.strict != 0, g);
    s << "namespace P" << k << " {\n";
    if (M.plan.phased) {
      PhasedParts pp = emit_phased_parts(g, M.plan, eo, "xg_lds_raw");
      if (pp.ns != M.ws_slots() || pp.lds_bytes > (int64_t)lds_bytes) {
        err = "batch: phased plan differs from the program's";
        return "";
      }
      s << "__device__ __forceinline__ void run(long long ibase, int xg_w) {\n" << pro.str() << pp.body
        << "}\n}\n";
      continue;
    }
    if (M.plan.waves > 1) {
      WideParts wp = emit_wide_parts(g, M.plan, eo, pro.str(), "xg_lds_raw", "g");
      if (wp.ns != M.ws_slots() || wp.st.lds_slots > M.est.lds_slots) { err = "batch: cooperative plan differs from the program's"; return ""; }
      s << wp.funcs;
      s << "__device__ __forceinline__ void run(long long ibase, int xg_w) {\n" << wp.body << "}\n}\n";
      continue;
    }
    if (lds_bytes) pro << "  lT* lds = (lT*)xg_lds_raw;\n";
    for (size_t c = 0; c < M.plan.chunks.size(); ++c) {
      EmitStats st;
      s << emit_device_chunk(g, M.plan, (int)c, eo, "c" + std::to_string(c), pro.str(), &st,
                             M.plan.n_ws, M.ws_slots());
      if (st.extra_ws > M.est.extra_ws || st.lds_slots > M.est.lds_slots) {
        err = "batch: a kernel's spills differ from the program's plan";
        return "";
      }
    }
    s << "__device__ __forceinline__ void run(long long ibase, int) {";
    for (size_t c = 0; c < M.plan.chunks.size(); ++c) s << " c" << c << "(ibase);";
    s << " }\n}\n";
  }
  // the bodies locate BArgs just before the implicit arguments (the host
  // checks that layout in the code object's metadata before loading it)
  s << "extern \"C\" __global__ void __launch_bounds__(" << b->block << ") xg_batch(BArgs b) {\n"
    << "  __shared__ long long xg_job;\n"
    << "  const int xg_w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));\n"
    << "  for (;;) {\n"
    << "    __syncthreads();\n"
    << "    if (threadIdx.x == 0) xg_job = (long long)atomicAdd(b.counter, 1ull);\n"
    << "    __syncthreads();\n"
    << "    const long long j = xg_job;\n"
    << "    if (j >= b.total) return;\n";
  for (int i = 0; i < K; ++i) {
    const xg_program* p = b->progs[b->order[i]];
    const std::string lane = p->opt.waves > 1 ? "(threadIdx.x & 63)" : "threadIdx.x";
    s << "    " << (i ? "else " : "") << "if (j < b.cum[" << i + 1 << "]) P" << b->order[i]
      << "::run((j - b.cum[" << i << "]) * " << tile_of(p) << " + " << lane << ", xg_w);\n";
  }
  s << "  }\n}\n";
  s << "extern \"C\" __global__ void xg_batch_reset(unsigned long long* c) {\n"
    << "  if (threadIdx.x == 0 && blockIdx.x == 0) *c = 0ull;\n}\n";
  return s.str();
}

size_t bargs_size_of(const xg_batch* b) {
  size_t sz = 8 + 8 + 8 * (b->progs.size() + 1);
  for (auto* p : b->progs) sz += 16 + 16 * (p->g.nnz_in.size() + p->g.nnz_out.size());
  return sz;
}

bool batch_load(xg_batch* b, std::string& err) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) { err = "hipGetDevice failed"; return false; }
  for (auto& d : b->devs) if (d.device == dev) return true;
  BatchDev d;
  d.device = dev;
  if (!check_launch_fits(b->co.bin, "xg_batch", b->block, err)) return false;
  if (!check_kernel_args(b->co.bin, "xg_batch", (int64_t)b->bargs_size, err)) return false;
  hipError_t e = hipModuleLoadData(&d.mod, b->co.bin.data());
  if (e != hipSuccess) { err = std::string("hipModuleLoadData: ") + hipGetErrorString(e); return false; }
  if (hipModuleGetFunction(&d.kern, d.mod, "xg_batch") != hipSuccess ||
      hipModuleGetFunction(&d.reset, d.mod, "xg_batch_reset") != hipSuccess) {
    (void)hipModuleUnload(d.mod);
    err = "batch kernels missing from the code object";
    return false;
  }
  int ncu = 0, nb = 0;
  if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) ncu = 256;
  if (hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(&nb, d.kern, b->block, 0) != hipSuccess || nb < 1)
    nb = 1;
  d.grid = ncu * nb;
  d.cus = ncu;
  b->devs.push_back(d);
  return true;
}

const BatchDev* batch_dev(xg_batch* b) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return nullptr;
  for (auto& d : b->devs) if (d.device == dev) return &d;
  return nullptr;
}

}  // namespace

namespace xg {
// A launch whose longest tile outlasts twice all the work on one workgroup a
// CU gets no more of them: others beside that tile would take its CU's caches
// from it (three DAGs and the MPC, 65,536 / 8,192 / 512 / 2,048 instances, the
// 512 in 8 tiles of 150,000 operations, on 64 lanes: 11.4 ms with four on a
// CU, 10.9 with one).
int64_t batch_grid(const std::vector<int64_t>& tiles, const std::vector<int64_t>& cost, int64_t resident, int64_t cus) {
  int64_t total = 0, longest = 0;
  double work = 0;
  for (size_t k = 0; k < tiles.size(); ++k) {
    if (tiles[k] == 0) continue;
    total += tiles[k];
    longest = std::max(longest, cost[k]);
    work += (double)tiles[k] * (double)cost[k];
  }
  const bool alone = 2 * work <= (double)longest * (double)cus;
  return std::min(alone ? std::min(resident, cus) : resident, total);
}
}  // namespace xg

namespace {

xg_status batch_launch(xg_batch* b, const xg_batch_args* args, void* ws, void* stream) {
  std::string err;
  {
    std::lock_guard<std::mutex> lk(b->mu);
    if (!batch_load(b, err)) { set_error(err); return XG_EDEVICE; }
  }
  const BatchDev* d = batch_dev(b);
  if (!d) { set_error("batch not loaded on this device"); return XG_EDEVICE; }
  if (!ws) { set_error("a batch needs a workspace (xg_batch_workspace_bytes)"); return XG_EINVAL; }
  const int K = (int)b->progs.size();
  std::vector<uint64_t> a;
  a.reserve(b->bargs_size / 8);
  a.push_back((uint64_t)(uintptr_t)ws);  // counter at the start of the workspace
  std::vector<int64_t> tiles(K);
  int64_t total = 0;
  for (int k = 0; k < K; ++k) {
    const int64_t n = args[k].n;
    if (n < 0) { set_error("n < 0"); return XG_EINVAL; }
    const size_t es = esize_of(b->progs[k]->g.dtype);
    if ((uint64_t)n * es > 0xffffffffull) { set_error("n too large"); return XG_EINVAL; }
    const int64_t per = tile_of(b->progs[k]);
    tiles[k] = (n + per - 1) / per;
    total += tiles[k];
  }
  a.push_back((uint64_t)total);
  int64_t cum = 0;
  a.push_back(0);
  for (int i = 0; i < K; ++i) { cum += tiles[b->order[i]]; a.push_back((uint64_t)cum); }
  size_t off = kCounterBytes;
  for (int k = 0; k < K; ++k) {
    xg_program* p = b->progs[k];
    const Graph& g = p->g;
    const int64_t n = args[k].n;
    const size_t es = esize_of(g.dtype);
    a.push_back((uint64_t)n);
    a.push_back((uint64_t)((uintptr_t)ws + off));
    off += align256(ws_bytes_of(n, p->m[0].ws_slots(), p->opt.block, p->opt.ipt, es));
    for (size_t i = 0; i < g.nnz_in.size(); ++i) {
      const void* ptr = args[k].d_in ? args[k].d_in[i] : nullptr;
      int64_t ld = args[k].ld_in ? args[k].ld_in[i] : n;
      if (n > 0 && g.nnz_in[i] > 0 && (!ptr || ld < n)) { set_error("batch input pointer/pitch"); return XG_EINVAL; }
      a.push_back((uint64_t)(uintptr_t)ptr);
      a.push_back((uint64_t)ld);
    }
    for (size_t i = 0; i < g.nnz_out.size(); ++i) {
      void* ptr = args[k].d_out ? args[k].d_out[i] : nullptr;
      int64_t ld = args[k].ld_out ? args[k].ld_out[i] : n;
      if (n > 0 && g.nnz_out[i] > 0 && (!ptr || ld < n)) { set_error("batch output pointer/pitch"); return XG_EINVAL; }
      a.push_back((uint64_t)(uintptr_t)ptr);
      a.push_back((uint64_t)ld);
    }
  }
  if (a.size() * 8 != b->bargs_size) { set_error("internal: batch argument layout"); return XG_EINVAL; }
  if (total == 0) return XG_OK;
  void* counter = ws;
  void* rp[] = {&counter};
  hipError_t e = hipModuleLaunchKernel(d->reset, 1, 1, 1, 64, 1, 1, 0, (hipStream_t)stream, rp, nullptr);
  if (e != hipSuccess) { set_error(std::string("reset launch: ") + hipGetErrorString(e)); return XG_EDEVICE; }
  size_t sz = b->bargs_size;
  void* cfg[] = {HIP_LAUNCH_PARAM_BUFFER_POINTER, a.data(), HIP_LAUNCH_PARAM_BUFFER_SIZE, &sz,
                 HIP_LAUNCH_PARAM_END};
  std::vector<int64_t> cost(K);
  for (int k = 0; k < K; ++k) cost[k] = b->progs[k]->m[0].cost;
  const int64_t grid = batch_grid(tiles, cost, d->grid, d->cus);
  e = hipModuleLaunchKernel(d->kern, (unsigned)grid, 1, 1, (unsigned)b->block, 1, 1, 0,
                            (hipStream_t)stream, nullptr, cfg);
  if (e != hipSuccess) { set_error(std::string("batch launch: ") + hipGetErrorString(e)); return XG_EDEVICE; }
  return XG_OK;
}

// ------------------------------------------------------------ autotune
// Planner/emitter generation: part of every tuning-cache key, so decisions
// timed on code an earlier generator emitted are not reused.
constexpr uint64_t kTuneVersion = 6;

// Key of a program for the tuning caches: its graph (per-instruction
// binary32 tags included: a mixed-precision program is timed on its own
// candidates), the options that change the generated code of every
// candidate (strict, inline math), and the generator version.
uint64_t graph_hash(const Graph& g, const xg_options& o) {
  uint64_t h = 1469598103934665603ull;
  auto mix = [&](uint64_t v) { for (int i = 0; i < 8; ++i) { h ^= (v >> (8 * i)) & 0xff; h *= 1099511628211ull; } };
  mix(kTuneVersion);
  mix((uint64_t)g.dtype);
  mix((uint64_t)(uint32_t)o.strict);
  mix((uint64_t)(uint32_t)o.inline_math);
  for (int32_t v : g.nnz_in) mix((uint64_t)v);
  for (int32_t v : g.nnz_out) mix((uint64_t)v);
  for (double c : g.consts) { uint64_t b; std::memcpy(&b, &c, 8); mix(b); }
  for (const Node& n : g.nodes) {
    mix(n.op); mix(n.f32); mix((uint32_t)n.a); mix((uint32_t)n.b); mix((uint64_t)n.aux);
  }
  for (auto& o2 : g.out) for (int32_t v : o2) mix((uint32_t)v);
  return h;
}

// Cached decision of the forward plan (mode 0), or of the adjoint plan timed
// on mode 1 or 2.
std::string tune_path(const xg_program* p, int64_t n, int mode) {
  char buf[80];
  const unsigned long long h = (unsigned long long)graph_hash(p->g, mode_opt(p, mode));
  if (mode == 0) std::snprintf(buf, sizeof buf, "/xg-tune-%016llx-%lld.txt", h, (long long)n);
  else std::snprintf(buf, sizeof buf, "/xg-tune-adj%d-%016llx-%lld.txt", mode, h, (long long)n);
  return cache_dir() + buf;
}

// Candidate plans for n instances: register budget (3/4 ... 5/2 of the load
// setting; the top ones leave the compiler AGPRs to hold the excess) x reload prefetch x LDS
// budget, where the smaller LDS budget is the one that lets every wave of
// an n-instance launch be resident at once (n / 64 waves over 256 CUs:
// each workgroup's spill slots must fit 160 KiB / waves-per-CU); then block
// 256, two instances per thread, half-size chunks and a single chunk where
// n or the program is large enough for them to matter; for the adjoint,
// leaf lengths and fan-outs at three register budgets; for the forward,
// cooperative tiles (level-split for wide programs with few tiles, phased
// for narrow ones, 2-wave phased also at one tile per SIMD or more).
std::vector<Candidate> tune_candidates(xg_program* p, int64_t n, int mode) {
  xg_options base = mode_opt(p, mode);
  const int64_t es = p->g.dtype == XG_F32 ? 4 : 8;
  const int64_t kCUs = 256, kSIMDs = 1024;
  if (p->library_budget[mode]) {
    base.reg_budget = p->g.dtype == XG_F32 ? kTuneRegs32 : kTuneRegs64;
    base.lds_slots = (int32_t)(kLdsSpillBytes / (64 * es));
  }
  auto lds_fit = [&](int32_t block, int32_t ipt) {
    const int64_t per = (int64_t)block * ipt;
    const int64_t wgs = (n + per - 1) / per;
    const int64_t waves_per_cu = std::max<int64_t>(1, (wgs * (block / 64) + kCUs - 1) / kCUs);
    const int64_t wgs_per_cu = std::max<int64_t>(1, waves_per_cu / (block / 64));
    int64_t fit = (kLdsSpillBytes / wgs_per_cu) / ((int64_t)block * es);
    fit = std::min<int64_t>(fit, kLdsSpillBytes / ((int64_t)block * es));
    return std::max<int64_t>(ipt, fit / ipt * ipt);
  };
  const int64_t full = std::min<int64_t>(base.lds_slots, kLdsSpillBytes / ((int64_t)base.block * es));
  std::vector<int64_t> ldss = {full};
  const int64_t fit = lds_fit(base.block, base.ipt);
  if (fit < full) ldss.push_back(fit);
  std::vector<Candidate> cands;
  const int rb0 = base.reg_budget;
  {  // what runs untuned, exactly: tuning never ends on a slower plan
    std::lock_guard<std::mutex> lk(p->mu);
    if (p->library_budget[mode]) {
      cands.emplace_back(mode_opt(p, mode), true);
      if (pick_few(p, mode, n)) cands.emplace_back(mode_opt(p, mode, true), true, mode == 0 && p->few_transfers_first);
    }
  }
  for (int64_t l : ldss)
    for (int rb : {rb0 * 3 / 4, rb0, rb0 * 4 / 3, rb0 * 5 / 3, rb0 * 2, rb0 * 16 / 7, rb0 * 5 / 2})
      for (int pf : {24, 64}) {
        if (pf != 24 && rb != rb0 && rb != rb0 * 5 / 3) continue;
        if (mode != 0 && rb > rb0 * 2) continue;  // (scratch: see below)
        xg_options o = base;
        o.reg_budget = rb;
        o.prefetch = pf;
        o.lds_slots = (int32_t)l;
        cands.push_back(o);
      }
  xg_options o = base;
  o.lds_slots = (int32_t)fit;
  if (base.block == 64 && n >= 256 * kCUs) {  // one 4-wave workgroup per CU
    xg_options b = o;
    b.block = 256;
    b.lds_slots = (int32_t)lds_fit(256, b.ipt);
    cands.push_back(b);
  }
  if (base.ipt == 1 && n >= 2 * 64 * kSIMDs) {  // enough instances for two per lane
    xg_options b = o;
    b.ipt = 2;
    b.lds_slots = (int32_t)lds_fit(b.block, 2);
    cands.push_back(b);
  }
  // the adjoint programs hold about four times the forward's operations
  const int64_t size = (int64_t)p->g.nodes.size() * (mode == 0 ? 1 : 4);
  const bool one_kernel = size > base.chunk_ops && size <= 5 * (int64_t)base.chunk_ops;
  if (size > base.chunk_ops / 2) {
    xg_options b = o;
    b.chunk_ops = std::max(1000, base.chunk_ops / 2);
    cands.push_back(b);
  }
  if (one_kernel) {  // one kernel, no crossings
    xg_options b = o;
    b.chunk_ops = 5 * base.chunk_ops;
    cands.push_back(b);
    // and with twice the LDS spill budget (half of the waves resident at
    // once): one long kernel holds more values than a chunk, and spilling
    // them to LDS rather than the workspace can pay for the second round
    // (the cart-pole MPC at 65,536 instances: 0.80 ms in three chunks,
    // 0.60 ms as one kernel with 159 LDS slots per lane)
    if (fit < full && !(mode != 0 && p->g.dtype == XG_F32)) {  // (binary32 adjoints: see below)
      b.lds_slots = (int32_t)std::min<int64_t>(full, 2 * fit);
      for (int rb : {rb0, rb0 * 5 / 3}) {
        b.reg_budget = rb;
        cands.push_back(b);
      }
    }
  }
  // adjoint: the leaf length trades the values a leaf holds for its
  // reverse sweep against the number of cuts (and levels of recomputation);
  // the fan-out trades states held per level against recomputation
  if (mode != 0) {
    // (the pendulum's fused adjoint as one kernel, leaves of 150 operations at
    // 4/3 of the load setting, fan-out 2 / 4: at 65,536 instances 245 / 263 us,
    // at 16,384, where no spill leaves the LDS, 138 / 131; leaves of 250 at 5/3
    // 250 / 290 and 148 / 153; budgets past twice the setting go to scratch)
    auto leaves = [&](int rb, int sg, int fo) {
      xg_options b = o;
      b.reg_budget = rb;
      b.adj_seg_ops = std::max(50, sg);
      b.adj_fanout = fo;
      // one kernel per adjoint for binary64 programs; binary32 ones keep
      // their chunks (a single 68,000-statement binary32 kernel takes
      // hiprtc minutes; the one-kernel candidate above stays)
      if (one_kernel && p->g.dtype != XG_F32) b.chunk_ops = 5 * base.chunk_ops;
      cands.push_back(b);
    };
    for (int rb : {rb0 * 3 / 2, rb0 * 5 / 3, rb0 * 2})
      for (int sg : {base.adj_seg_ops, base.adj_seg_ops * 2}) leaves(rb, sg, base.adj_fanout);
    for (int fo : {2, 4}) leaves(rb0 * 4 / 3, base.adj_seg_ops * 3 / 5, fo);
  }
  // cooperative tiles, when few tiles leave SIMDs idle and the program is
  // wide (operations per dependency level) enough to split
  if (mode == 0 && base.waves <= 1 && base.block == 64 && base.ipt == 1 && (n + 63) / 64 < 4 * kCUs) {
    std::vector<int32_t> lvl(p->g.nodes.size(), 0);
    int32_t depth = 1;
    int64_t ops = 0;
    for (size_t v = 0; v < p->g.nodes.size(); ++v) {
      const Node& nd = p->g.nodes[v];
      if (!is_arith(nd.op)) continue;
      int32_t l = 0;
      if (nd.a >= 0) l = std::max(l, lvl[nd.a]);
      if (nd.b >= 0) l = std::max(l, lvl[nd.b]);
      lvl[v] = l + 1;
      depth = std::max(depth, l + 1);
      ++ops;
    }
    for (int w : {4, 8, 16}) {
      if (ops / depth < 32 * w) continue;
      xg_options b = base;
      b.waves = w;
      b.coop_phase = 0;
      b.lds_slots = (int32_t)(kLdsSpillBytes / ((int64_t)64 * w * es));
      if (w >= 16) b.reg_budget = p->g.dtype == XG_F32 ? 96 : 48;
      cands.push_back(b);
    }
  }
  // phased cooperative tiles for narrow programs of 2,000 to 60,000
  // operations (the waves of a tile share the CU's LDS for their exchanges)
  if (mode == 0 && base.waves <= 1 && base.block == 64 && base.ipt == 1) {
    int64_t ops = 0;
    for (const Node& nd : p->g.nodes) ops += is_arith(nd.op);
    const int rb1 = rb0 * 3 / 2;
    const int64_t tiles = (n + 63) / 64;
    if (ops >= 2000 && ops <= 60000 && tiles < 4 * kCUs) {
      // few tiles: 4 waves with phases of about 150 or 300 operation-cost
      // units per wave at two register budgets, and 2 waves
      const int cfg[5][3] = {{4, 150, rb0}, {4, 150, rb1}, {4, 300, rb0}, {4, 300, rb1}, {2, 300, rb1}};
      for (const auto& c : cfg) {
        if (tiles * c[0] > 4 * kSIMDs) continue;
        xg_options b = base;
        b.waves = c[0];
        b.coop_phase = c[1];
        b.reg_budget = c[2];
        b.lds_slots = (int32_t)(kLdsSpillBytes / ((int64_t)64 * c[0] * es));
        cands.push_back(b);
      }
    } else if (ops >= 100 && ops < 2000 && tiles < 4 * kCUs) {
      // small programs: a few short phases per wave (the 200-operation
      // random DAG at 1,000 instances: 13.4 us on one wave per tile, 5.8 us
      // on 4-wave tiles with phases of 50 or 80 units)
      const int cfg[3][2] = {{4, 50}, {4, 80}, {2, 50}};
      for (const auto& c : cfg) {
        if (tiles * c[0] > 4 * kSIMDs) continue;
        xg_options b = base;
        b.waves = c[0];
        b.coop_phase = c[1];
        b.lds_slots = (int32_t)(kLdsSpillBytes / ((int64_t)64 * c[0] * es));
        cands.push_back(b);
      }
    } else if (ops >= 2000 && ops <= 60000 && p->g.dtype != XG_F32) {
      // a tile per SIMD or more: 2-wave tiles still split a long program's
      // live values between two waves.  With the whole LDS (one tile per
      // CU at a time) and with spill regions small enough that two tiles
      // share a CU when their exchanges take up to 46 KiB (the cart-pole
      // MPC at 65,536 instances: 0.62 ms as one single-wave kernel, 0.57
      // and 0.47 ms as these two)
      for (int64_t l : {kLdsSpillBytes / ((int64_t)64 * 2 * es),
                        ((160 * 1024) / 2 - 46 * 1024) / ((int64_t)64 * 2 * es)}) {
        xg_options b = base;
        b.waves = 2;
        b.coop_phase = 300;
        b.reg_budget = rb1;
        b.lds_slots = (int32_t)l;
        cands.push_back(b);
      }
    }
  }
  return cands;
}

// A batch over `progs` up to its generated source (not compiled).
xg_status batch_make(const std::vector<xg_program*>& progs, std::unique_ptr<xg_batch>& out) {
  std::unique_ptr<xg_batch> b(new xg_batch());
  const int k = (int)progs.size();
  std::string err;
  try {
    for (int i = 0; i < k; ++i) {
      if (!progs[i]) { set_error("null program"); return XG_EINVAL; }
      b->progs.push_back(progs[i]);
    }
    // one workgroup size for the launch: a program's block, or 64 x waves
    // for a cooperative-tile program (all its waves take the same job)
    b->block = launch_block_of(progs[0]);
    b->ipt = 1;
    for (auto* p : b->progs) if (p->opt.waves <= 1) { b->ipt = p->opt.ipt; break; }
    for (auto* p : b->progs) {
      if (launch_block_of(p) != b->block || (p->opt.waves <= 1 && p->opt.ipt != b->ipt)) {
        set_error("batch: all programs need the same workgroup size (block, or 64 x waves for "
                  "cooperative tiles) and the same ipt");
        return XG_EINVAL;
      }
      std::lock_guard<std::mutex> lk(p->mu);
      if (!plan_mode(p, 0, err)) { set_error(err); return XG_EINVAL; }
    }
    // longest tiles first: operations per instance
    b->order.resize(k);
    for (int i = 0; i < k; ++i) b->order[i] = i;
    std::stable_sort(b->order.begin(), b->order.end(), [&](int x, int y) {
      return b->progs[x]->m[0].plan.n_ops > b->progs[y]->m[0].plan.n_ops;
    });
    b->bargs_size = bargs_size_of(b.get());
    if (b->bargs_size > 4000) { set_error("batch: too many arguments for one launch"); return XG_EUNSUPPORTED; }
    b->src = build_batch_source(b.get(), err);
    if (b->src.empty()) { set_error(err); return XG_EUNSUPPORTED; }
  } catch (const std::exception& e) {
    set_error(e.what());
    return XG_ENOMEM;
  }
  out = std::move(b);
  return XG_OK;
}

}  // namespace

namespace xg {
xg_status batch_source(const std::vector<xg_program*>& progs, std::string& src) {
  std::unique_ptr<xg_batch> b;
  const xg_status st = batch_make(progs, b);
  if (st == XG_OK) src = b->src;
  return st;
}
}  // namespace xg

namespace {

void reset_modes(xg_program* p) {
  for (int m = 0; m < 3; ++m) reset_mode(p, m);
}

// Makes c the plan of p's `mode` (1 and 2 share one), for every count.
void adopt(xg_program* p, int mode, const Candidate& c) {
  if (mode == 0) {
    p->opt = c.o;
    p->transfers_first = c.transfers_first;
    p->library_plan[0] = false;
    p->library_budget[0] = c.library;
  } else {
    p->aopt = c.o;
    p->library_plan[1] = p->library_plan[2] = false;
    p->library_budget[1] = p->library_budget[2] = c.library;
  }
}

// A copy of p (graph and options) whose `mode` plan is c.
std::unique_ptr<xg_program> trial_program(const xg_program* p, int mode, const Candidate& c) {
  std::unique_ptr<xg_program> q(new xg_program());
  q->g = p->g;
  q->opt = p->opt;
  q->aopt = p->aopt;
  adopt(q.get(), mode, c);
  return q;
}

}  // namespace

namespace xg {
bool plan_candidates(xg_program* p, int64_t n, int mode, std::vector<Candidate>& cands,
                     std::vector<std::unique_ptr<xg_program>>& trials, std::string& err) {
  for (const Candidate& c : tune_candidates(p, n, mode)) {
    std::unique_ptr<xg_program> q = trial_program(p, mode, c);
    if (!plan_mode(q.get(), mode, err)) {
      if (c.o.waves <= 1) return false;
      // a cooperative plan that cannot be formed (e.g. LDS): not a candidate
      if (c.o.verbose) std::fprintf(stderr, "[xg autotune] cooperative candidate skipped: %s\n", err.c_str());
      continue;
    }
    cands.push_back(c);
    trials.push_back(std::move(q));
  }
  return true;
}
}  // namespace xg

namespace {

}  // namespace

extern "C" {

xg_status xg_batch_create(xg_program* const* progs, int32_t k, const xg_options* opts, xg_batch** out) {
  if (!out) { set_error("out is null"); return XG_EINVAL; }
  *out = nullptr;
  if (!progs || k < 1) { set_error("need at least one program"); return XG_EINVAL; }
  std::unique_ptr<xg_batch> b;
  xg_status st = batch_make(std::vector<xg_program*>(progs, progs + k), b);
  if (st != XG_OK) return st;
  std::string err;
  try {
    bool verbose = opts && opts->verbose;
    if (!compile_hip(b->src, base_compile_options(progs[0]->opt.strict != 0), b->co, err, verbose)) {
      set_error(err);
      return XG_ECOMPILE;
    }
    if (!check_launch_fits(b->co.bin, "xg_batch", b->block, err) ||
        !check_kernel_args(b->co.bin, "xg_batch", (int64_t)b->bargs_size, err)) {
      set_error("batch: " + err);
      return XG_EUNSUPPORTED;
    }
  } catch (const std::exception& e) {
    set_error(e.what());
    return XG_ENOMEM;
  }
  *out = b.release();
  return XG_OK;
}

static void destroy_batch(xg_batch* b);

void xg_batch_free(xg_batch* b) {
  if (!b) return;
  {
    std::lock_guard<std::mutex> lk(b->mu);
    if (b->live_graphs > 0) {  // graphs still launch its kernel: the last one frees it
      b->free_pending = true;
      return;
    }
  }
  destroy_batch(b);
}

static void destroy_batch(xg_batch* b) {
  int cur = -1;
  bool loaded = false;
  for (auto& d : b->devs) loaded = loaded || d.mod;
  if (loaded) (void)hipGetDevice(&cur);
  for (auto& d : b->devs) {
    if (!d.mod) continue;
    // launches may still be queued or running: drain before unloading
    if (d.device >= 0 && hipSetDevice(d.device) == hipSuccess) (void)hipDeviceSynchronize();
    (void)hipModuleUnload(d.mod);
  }
  if (cur >= 0) (void)hipSetDevice(cur);
  for (auto* p : b->owned) xg_program_free(p);
  delete b;
}

xg_status xg_batch_workspace_bytes(xg_batch* b, const int64_t* n, size_t* bytes) {
  if (!b || !n || !bytes) { set_error("bad argument"); return XG_EINVAL; }
  size_t tot = kCounterBytes;
  for (size_t k = 0; k < b->progs.size(); ++k) {
    if (n[k] < 0) { set_error("n < 0"); return XG_EINVAL; }
    xg_program* p = b->progs[k];
    tot += align256(ws_bytes_of(n[k], p->m[0].ws_slots(), p->opt.block, p->opt.ipt, esize_of(p->g.dtype)));
  }
  *bytes = tot;
  return XG_OK;
}

xg_status xg_batch_eval(xg_batch* b, const xg_batch_args* args, void* d_workspace, void* stream) {
  if (!b || !args) { set_error("bad argument"); return XG_EINVAL; }
  try {
    return batch_launch(b, args, d_workspace, stream);
  } catch (const std::exception& e) { set_error(e.what()); return XG_ENOMEM; }
}

// Finish a capture; on success the graph holds a reference to the program
// or batch whose loaded code it launches (see xg_graph_free).
static xg_status end_capture(hipStream_t s, xg_status st, xg_graph** out, xg_program* prog,
                             xg_batch* batch) {
  hipGraph_t g = nullptr;
  hipError_t e = hipStreamEndCapture(s, &g);
  if (st != XG_OK) { if (g) (void)hipGraphDestroy(g); return st; }
  if (e != hipSuccess || !g) { set_error(std::string("hipStreamEndCapture: ") + hipGetErrorString(e)); return XG_EDEVICE; }
  std::unique_ptr<xg_graph> gr(new xg_graph());
  gr->graph = g;
  e = hipGraphInstantiate(&gr->exec, g, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    (void)hipGraphDestroy(g);
    set_error(std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
    return XG_EDEVICE;
  }
  if (prog) {
    std::lock_guard<std::mutex> lk(prog->mu);
    prog->live_graphs++;
    gr->prog = prog;
  }
  if (batch) {
    std::lock_guard<std::mutex> lk(batch->mu);
    batch->live_graphs++;
    gr->batch = batch;
  }
  *out = gr.release();
  return XG_OK;
}

xg_status xg_graph_capture_eval(xg_program* p, int64_t n, const void* const* d_in, const int64_t* ld_in,
                                void* const* d_out, const int64_t* ld_out, void* d_workspace,
                                void* stream, xg_graph** out) {
  if (!p || !out) { set_error("bad argument"); return XG_EINVAL; }
  *out = nullptr;
  if (!stream) { set_error("capture needs a non-default stream"); return XG_EINVAL; }
  {
    std::string err;
    std::lock_guard<std::mutex> lk(p->mu);
    xg_status code = XG_OK;
    bool few;  // no module loads while capturing
    if (!load_for(p, 0, n, stream, few, err, &code)) { set_error(err); return code; }
  }
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) { set_error(std::string("hipStreamBeginCapture: ") + hipGetErrorString(e)); return XG_EDEVICE; }
  xg_status st = xg_eval(p, n, d_in, ld_in, d_out, ld_out, d_workspace, stream);
  return end_capture(s, st, out, p, nullptr);
}

xg_status xg_graph_capture_rollout(xg_program* p, int64_t n, int32_t steps, void* d_state0, void* d_state1,
                                   int64_t ld_state, const void* const* d_in, const int64_t* ld_in,
                                   void* d_workspace, void* stream, xg_graph** out) {
  if (!p || !out || steps <= 0 || !d_state0 || !d_state1 || d_state0 == d_state1) {
    set_error("bad argument");
    return XG_EINVAL;
  }
  *out = nullptr;
  if (!stream) { set_error("capture needs a non-default stream"); return XG_EINVAL; }
  const Graph& g = p->g;
  if (g.nnz_in.empty() || g.nnz_out.empty() || g.nnz_in[0] != g.nnz_out[0] || g.nnz_out.size() != 1) {
    set_error("rollout needs a program whose only output has the shape of its first input");
    return XG_EINVAL;
  }
  const size_t nin = g.nnz_in.size();
  std::vector<const void*> in(nin);
  std::vector<int64_t> ldi(nin);
  for (size_t a = 1; a < nin; ++a) {
    in[a] = d_in ? d_in[a] : nullptr;
    ldi[a] = ld_in ? ld_in[a] : n;
  }
  ldi[0] = ld_state;
  {
    std::string err;
    std::lock_guard<std::mutex> lk(p->mu);
    xg_status code = XG_OK;
    bool few;  // no module loads while capturing
    if (!load_for(p, 0, n, stream, few, err, &code)) { set_error(err); return code; }
  }
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) { set_error(std::string("hipStreamBeginCapture: ") + hipGetErrorString(e)); return XG_EDEVICE; }
  xg_status st = XG_OK;
  void* buf[2] = {d_state0, d_state1};
  for (int32_t k = 0; k < steps && st == XG_OK; ++k) {
    in[0] = buf[k & 1];
    void* o = buf[(k + 1) & 1];
    st = xg_eval(p, n, in.data(), ldi.data(), &o, &ld_state, d_workspace, stream);
  }
  return end_capture(s, st, out, p, nullptr);
}

xg_status xg_graph_capture_batch(xg_batch* b, const xg_batch_args* args, void* d_workspace, void* stream,
                                 xg_graph** out) {
  if (!b || !args || !out) { set_error("bad argument"); return XG_EINVAL; }
  *out = nullptr;
  if (!stream) { set_error("capture needs a non-default stream"); return XG_EINVAL; }
  {
    std::string err;
    std::lock_guard<std::mutex> lk(b->mu);
    if (!batch_load(b, err)) { set_error(err); return XG_EDEVICE; }
  }
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) { set_error(std::string("hipStreamBeginCapture: ") + hipGetErrorString(e)); return XG_EDEVICE; }
  xg_status st = batch_launch(b, args, d_workspace, stream);
  return end_capture(s, st, out, nullptr, b);
}

xg_status xg_graph_launch(xg_graph* g, void* stream) {
  if (!g || !g->exec) { set_error("bad graph"); return XG_EINVAL; }
  hipError_t e = hipGraphLaunch(g->exec, (hipStream_t)stream);
  if (e != hipSuccess) { set_error(std::string("hipGraphLaunch: ") + hipGetErrorString(e)); return XG_EDEVICE; }
  return XG_OK;
}

void xg_graph_free(xg_graph* g) {
  if (!g) return;
  if (g->exec) (void)hipGraphExecDestroy(g->exec);
  if (g->graph) (void)hipGraphDestroy(g->graph);
  if (xg_program* p = g->prog) {
    bool last;
    {
      std::lock_guard<std::mutex> lk(p->mu);
      last = --p->live_graphs == 0 && p->free_pending;
    }
    if (last) destroy_program(p);  // xg_program_free was deferred until now
  }
  if (xg_batch* b = g->batch) {
    bool last;
    {
      std::lock_guard<std::mutex> lk(b->mu);
      last = --b->live_graphs == 0 && b->free_pending;
    }
    if (last) destroy_batch(b);
  }
  delete g;
}

xg_status xg_autotune_workspace_bytes(xg_program* p, int64_t n, int32_t mode, size_t* bytes) {
  if (!p || n <= 0 || !bytes || mode < 0 || mode > 2) { set_error("bad argument"); return XG_EINVAL; }
  std::string err;
  try {
    std::vector<Candidate> cands;
    std::vector<std::unique_ptr<xg_program>> trials;
    if (!plan_candidates(p, n, mode, cands, trials, err)) { set_error(err); return XG_EINVAL; }
    size_t mx = 0;
    for (size_t i = 0; i < cands.size(); ++i)
      mx = std::max(mx, ws_bytes_of(n, trials[i]->m[mode].ws_slots(), cands[i].o.block, cands[i].o.ipt,
                                    p->g.dtype == XG_F32 ? 4 : 8));
    *bytes = mx;
  } catch (const std::exception& e) {
    set_error(e.what());
    return XG_ENOMEM;
  }
  return XG_OK;
}

xg_status xg_autotune_precompile(xg_program* p, int64_t n, int32_t mode) {
  if (!p || n <= 0 || mode < 0 || mode > 2) { set_error("bad argument"); return XG_EINVAL; }
  std::string err;
  try {
    std::vector<Candidate> cands;
    std::vector<std::unique_ptr<xg_program>> trials;
    if (!plan_candidates(p, n, mode, cands, trials, err)) { set_error(err); return XG_EINVAL; }
    std::vector<std::string> srcs;
    for (auto& q : trials)
      for (auto& s : q->m[mode].srcs) srcs.push_back(s);
    std::vector<CodeObject> cos;
    if (!compile_many(srcs, base_compile_options(p->opt.strict != 0), cos, err, p->opt.verbose != 0)) {
      set_error(err);
      return XG_ECOMPILE;
    }
  } catch (const std::exception& e) {
    set_error(e.what());
    return XG_ENOMEM;
  }
  return XG_OK;
}

}  // extern "C"

namespace {

// Time every candidate plan of `mode` for n instances with `run` (one
// evaluation of a trial program on the caller's buffers), adopt the fastest
// for that mode (the adjoint modes share one set of options) and cache the
// decision on disk.
template <class Run>
xg_status tune_mode(xg_program* p, int64_t n, int mode, size_t workspace_bytes, void* stream,
                    xg_options* chosen, Run run) {
  {
    // re-planning unloads the program's kernels, which captured graphs launch
    std::lock_guard<std::mutex> lk(p->mu);
    if (p->live_graphs > 0) {
      set_error("autotune: the program has " + std::to_string(p->live_graphs) +
                " captured graph(s); free them before re-planning it");
      return XG_EINVAL;
    }
  }
  const std::string path = tune_path(p, n, mode);
  const xg_options base = mode_opt(p, mode);
  auto apply = [&](const Candidate& c) {
    std::lock_guard<std::mutex> lk(p->mu);
    if (p->live_graphs > 0) return false;  // captured meanwhile on another thread
    for (int m = 0; m < 3; ++m)
      if ((m == 0) == (mode == 0)) reset_mode(p, m);
    adopt(p, mode, c);
    return true;
  };
  auto refused = [&]() {
    set_error("autotune: the program was captured in a graph while it was being tuned");
    return XG_EINVAL;
  };
  // cached decision
  {
    std::ifstream f(path);
    xg_options o = base;
    if (f >> o.block >> o.ipt >> o.reg_budget >> o.lds_slots >> o.prefetch >> o.chunk_ops >> o.waves) {
      int32_t sg = 0, fo = 0, cp = 0, lib = 0, first = 0;
      if (f >> sg && sg > 0) o.adj_seg_ops = sg;
      if (f >> fo && fo > 0) o.adj_fanout = fo;
      if (f >> cp && cp >= 0) o.coop_phase = cp;
      f >> lib >> first;
      std::string err;
      if (check_opts(o, p->g.dtype, err)) {
        if (!apply(Candidate(o, lib == 1, first == 1))) return refused();
        if (chosen) *chosen = o;
        return XG_OK;
      }
    }
  }
  std::vector<Candidate> cands;
  // plan all candidates, then compile every source concurrently
  std::vector<std::unique_ptr<xg_program>> trial;
  std::vector<std::string> srcs;
  std::vector<size_t> first;
  std::string err;
  try {
    if (!plan_candidates(p, n, mode, cands, trial, err)) { set_error(err); return XG_EINVAL; }
    for (auto& q : trial) {
      first.push_back(srcs.size());
      for (auto& s : q->m[mode].srcs) srcs.push_back(s);
    }
    std::vector<CodeObject> cos;
    if (!compile_many(srcs, base_compile_options(base.strict != 0), cos, err, base.verbose != 0)) {
      set_error(err);
      return XG_ECOMPILE;
    }
    for (size_t i = 0; i < trial.size(); ++i) {
      ModeState& M = trial[i]->m[mode];
      M.cos.assign(cos.begin() + first[i], cos.begin() + first[i] + M.srcs.size());
      M.compiled = true;
    }
  } catch (const std::exception& e) {
    set_error(e.what());
    return XG_ENOMEM;
  }
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    set_error("hipEventCreate failed");
    return XG_EDEVICE;
  }
  // one timing of candidate i: 20 launches after a warm one (< 0: failed)
  const int reps = 20;
  auto time_one = [&](size_t i) -> float {
    xg_program* q = trial[i].get();
    if (run(q) != XG_OK) {  // warm
      if (base.verbose) std::fprintf(stderr, "[xg autotune] candidate %zu failed: %s\n", i, xg_last_error());
      return -1.0f;
    }
    (void)hipEventRecord(e0, (hipStream_t)stream);
    for (int r = 0; r < reps; ++r) (void)run(q);
    (void)hipEventRecord(e1, (hipStream_t)stream);
    if (hipEventSynchronize(e1) != hipSuccess) return -1.0f;
    float ms = 0;
    (void)hipEventElapsedTime(&ms, e0, e1);
    return ms;
  };
  std::vector<float> t(trial.size(), -1.0f);
  for (size_t i = 0; i < trial.size(); ++i) {
    size_t need = 0;
    if (xg_workspace_bytes(trial[i].get(), n, mode, &need) != XG_OK || need > workspace_bytes) {
      if (base.verbose) std::fprintf(stderr, "[xg autotune] candidate %zu skipped: workspace %zu B\n", i, need);
      continue;
    }
    t[i] = time_one(i);
    if (base.verbose && t[i] >= 0)
      std::fprintf(stderr, "[xg autotune] mode %d n=%lld block=%d ipt=%d reg=%d lds=%d prefetch=%d chunk=%d waves=%d phase=%d seg=%d fanout=%d%s%s: %.2f us\n",
                   mode, (long long)n, cands[i].o.block, cands[i].o.ipt, cands[i].o.reg_budget, cands[i].o.lds_slots,
                   cands[i].o.prefetch, cands[i].o.chunk_ops, cands[i].o.waves, cands[i].o.coop_phase,
                   cands[i].o.adj_seg_ops, cands[i].o.adj_fanout, cands[i].library ? " library" : "",
                   cands[i].transfers_first ? " transfers" : "", 1e3 * t[i] / reps);
  }
  // the three fastest are timed twice more, in turn, and each keeps its
  // best time: one pass in sequence can catch a candidate in a slow moment
  // (clocks still rising after host work, another process), and the
  // decision is cached for good
  std::vector<size_t> top;
  for (size_t i = 0; i < trial.size(); ++i)
    if (t[i] >= 0) top.push_back(i);
  std::sort(top.begin(), top.end(), [&](size_t a, size_t b) { return t[a] < t[b]; });
  if (top.size() > 3) top.resize(3);
  if (top.size() > 1)
    for (int round = 0; round < 2; ++round)
      for (size_t i : top) {
        const float ms = time_one(i);
        if (ms >= 0 && ms < t[i]) t[i] = ms;
        if (base.verbose && ms >= 0)
          std::fprintf(stderr, "[xg autotune] again: candidate %zu: %.2f us\n", i, 1e3 * ms / reps);
      }
  float best = 1e30f;
  int besti = -1;
  for (size_t i : top)
    if (t[i] < best) { best = t[i]; besti = (int)i; }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  for (auto& q : trial) reset_modes(q.get());
  if (besti < 0) { set_error("autotune: no candidate fits the workspace"); return XG_ENOMEM; }
  const xg_options& o = cands[besti].o;
  if (!apply(cands[besti])) return refused();
  {
    std::ofstream f(path);
    f << o.block << " " << o.ipt << " " << o.reg_budget << " " << o.lds_slots << " " << o.prefetch
      << " " << o.chunk_ops << " " << o.waves << " " << o.adj_seg_ops << " " << o.adj_fanout << " "
      << o.coop_phase << " " << cands[besti].library << " " << cands[besti].transfers_first << "\n";
  }
  if (chosen) *chosen = o;
  return XG_OK;
}

}  // namespace

namespace {

// Operations per dependency level of a program's graph (how wide it is).
double width_of(const Graph& g) {
  std::vector<int32_t> lvl(g.nodes.size(), 0);
  int32_t depth = 1;
  int64_t ops = 0;
  for (size_t v = 0; v < g.nodes.size(); ++v) {
    const Node& nd = g.nodes[v];
    if (!is_arith(nd.op)) continue;
    int32_t l = 0;
    if (nd.a >= 0) l = std::max(l, lvl[nd.a]);
    if (nd.b >= 0) l = std::max(l, lvl[nd.b]);
    lvl[v] = l + 1;
    depth = std::max(depth, l + 1);
    ++ops;
  }
  return (double)ops / depth;
}

// Batch candidates: one workgroup size B in {64, 256, 512, 1024} for the
// whole launch.  A program with few tiles (under 4 per CU) and at least
// 32 x W operations per dependency level runs as W = B/64-wave cooperative
// tiles, every other program on B-lane workgroups, one lane per instance.
std::vector<std::pair<int, std::vector<Candidate>>> batch_candidates(xg_program* const* progs, int32_t k,
                                                                     const int64_t* n) {
  std::vector<std::pair<int, std::vector<Candidate>>> c;
  std::vector<double> width(k);
  for (int32_t i = 0; i < k; ++i) width[i] = width_of(progs[i]->g);
  for (int B : {64, 256, 512, 1024}) {
    const int W = B / 64;
    std::vector<Candidate> os;
    for (int32_t i = 0; i < k; ++i) {
      xg_options o = progs[i]->opt;
      const int64_t es = progs[i]->g.dtype == XG_F32 ? 4 : 8;
      // The library's budgets are for one wave on a SIMD.  Two share its 512
      // registers at 512 lanes and four at 1,024 (the MPC there, 2,048
      // instances: 2,858 us with 112 values, 888 B of scratch per lane, 1,324
      // with 48; 551 and 536 at 512 lanes with 112 and 96), and the lanes need
      // the whole LDS.
      const bool library = B == 64 && progs[i]->library_budget[0];
      if (progs[i]->library_budget[0] && B > 64) {
        o.reg_budget = progs[i]->g.dtype == XG_F32 ? (B >= 1024 ? 96 : kTuneRegs32) : (B >= 1024 ? 48 : kTuneRegs64);
        o.lds_slots = (int32_t)(kLdsSpillBytes / (64 * es));
      }
      o.ipt = 1;
      o.coop_phase = 0;  // (this autotuner does not try phased tiles; a program set to them runs so)
      if (W > 1 && (n[i] + 63) / 64 < 4 * 256 && width[i] >= 32.0 * W) {
        o.waves = W;
        o.block = 64;
        o.lds_slots = (int32_t)(kLdsSpillBytes / (64 * W * es));
        if (W >= 16) o.reg_budget = progs[i]->g.dtype == XG_F32 ? 96 : 48;
      } else {
        o.waves = 1;
        o.block = B;
        o.lds_slots = (int32_t)std::min<int64_t>(o.lds_slots, kLdsSpillBytes / (B * es));
      }
      os.emplace_back(o, library);
    }
    c.push_back({B, os});
  }
  return c;
}

// Trial copies of the programs with the candidate's options, and a batch
// over them (source generated, not compiled); the batch owns the copies.
xg_status batch_trial(xg_program* const* progs, int32_t k, const std::vector<Candidate>& os,
                      std::unique_ptr<xg_batch>& out) {
  std::vector<xg_program*> qs;
  for (int32_t i = 0; i < k; ++i) {
    std::string err;
    if (!check_opts(os[i].o, progs[i]->g.dtype, err)) {
      for (auto* q : qs) xg_program_free(q);
      set_error(err);
      return XG_EINVAL;
    }
    qs.push_back(trial_program(progs[i], 0, os[i]).release());
  }
  xg_status st = batch_make(qs, out);
  if (st != XG_OK) {
    for (auto* q : qs) xg_program_free(q);
    return st;
  }
  out->owned = qs;
  return XG_OK;
}

uint64_t batch_key(xg_program* const* progs, int32_t k, const int64_t* n) {
  uint64_t h = 1469598103934665603ull;
  for (int32_t i = 0; i < k; ++i) {
    h = fnv1a(std::to_string(graph_hash(progs[i]->g, progs[i]->opt)) + "/" + std::to_string(n[i]) + ";", h);
  }
  return h;
}

}  // namespace

namespace xg {
std::vector<std::pair<int, std::string>> batch_candidate_sources(xg_program* const* progs, int32_t k, const int64_t* n) {
  std::vector<std::pair<int, std::string>> srcs;
  for (auto& c : batch_candidates(progs, k, n)) {
    std::unique_ptr<xg_batch> b;
    if (batch_trial(progs, k, c.second, b) != XG_OK) continue;  // candidate not formable
    srcs.push_back({c.first, b->src});
    for (auto* q : b->owned) xg_program_free(q);
    b->owned.clear();
  }
  return srcs;
}
}  // namespace xg

namespace {

size_t batch_ws_bytes(xg_batch* b, const int64_t* n) {
  size_t tot = kCounterBytes;
  for (size_t i = 0; i < b->progs.size(); ++i) {
    xg_program* p = b->progs[i];
    tot += align256(ws_bytes_of(n[i], p->m[0].ws_slots(), p->opt.block, p->opt.ipt, esize_of(p->g.dtype)));
  }
  return tot;
}

}  // namespace

extern "C" {

xg_status xg_batch_autotune_workspace_bytes(xg_program* const* progs, int32_t k, const int64_t* n,
                                            size_t* bytes) {
  if (!progs || k < 1 || !n || !bytes) { set_error("bad argument"); return XG_EINVAL; }
  size_t mx = 0;
  for (auto& c : batch_candidates(progs, k, n)) {
    std::unique_ptr<xg_batch> b;
    if (batch_trial(progs, k, c.second, b) != XG_OK) continue;  // candidate not formable
    mx = std::max(mx, batch_ws_bytes(b.get(), n));
    for (auto* q : b->owned) xg_program_free(q);
    b->owned.clear();
  }
  if (mx == 0) { set_error("batch autotune: no candidate"); return XG_EINVAL; }
  *bytes = mx;
  return XG_OK;
}

xg_status xg_batch_autotune_precompile(xg_program* const* progs, int32_t k, const int64_t* n) {
  if (!progs || k < 1 || !n) { set_error("bad argument"); return XG_EINVAL; }
  std::vector<std::string> srcs;
  for (auto& c : batch_candidate_sources(progs, k, n)) srcs.push_back(std::move(c.second));
  std::vector<CodeObject> cos;
  std::string err;
  if (!compile_many(srcs, base_compile_options(progs[0]->opt.strict != 0), cos, err, progs[0]->opt.verbose != 0)) {
    set_error(err);
    return XG_ECOMPILE;
  }
  return XG_OK;
}

xg_status xg_batch_autotune(xg_program* const* progs, int32_t k, const xg_batch_args* args,
                            void* d_workspace, size_t workspace_bytes, void* stream, xg_batch** out,
                            int32_t* chosen_block) {
  if (!progs || k < 1 || !args || !out) { set_error("bad argument"); return XG_EINVAL; }
  *out = nullptr;
  std::vector<int64_t> n(k);
  for (int32_t i = 0; i < k; ++i) {
    if (!progs[i]) { set_error("null program"); return XG_EINVAL; }
    n[i] = args[i].n;
  }
  auto cands = batch_candidates(progs, k, n.data());
  char name[80];
  std::snprintf(name, sizeof name, "/xg-tune-batch-%016llx.txt", (unsigned long long)batch_key(progs, k, n.data()));
  const std::string path = cache_dir() + name;
  int cached = 0;
  {
    std::ifstream f(path);
    if (!(f >> cached)) cached = 0;
  }
  // form every candidate (or the cached choice) and compile them together
  std::vector<std::unique_ptr<xg_batch>> bs;
  std::vector<int> blocks;
  std::vector<std::string> srcs;
  for (int pass = 0; pass < 2 && bs.empty(); ++pass) {
    if (pass == 1) cached = 0;  // the cached choice cannot be formed any more: time them all
    for (auto& c : cands) {
      if (cached && c.first != cached) continue;
      std::unique_ptr<xg_batch> b;
      if (batch_trial(progs, k, c.second, b) != XG_OK) continue;
      srcs.push_back(b->src);
      bs.push_back(std::move(b));
      blocks.push_back(c.first);
    }
  }
  if (bs.empty()) { set_error("batch autotune: no candidate could be formed"); return XG_EINVAL; }
  std::vector<CodeObject> cos;
  std::string err;
  if (!compile_many(srcs, base_compile_options(progs[0]->opt.strict != 0), cos, err, progs[0]->opt.verbose != 0)) {
    for (auto& b : bs) xg_batch_free(b.release());
    set_error(err);
    return XG_ECOMPILE;
  }
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    for (auto& b : bs) xg_batch_free(b.release());
    set_error("hipEventCreate failed");
    return XG_EDEVICE;
  }
  float best = 1e30f;
  int besti = -1;
  for (size_t i = 0; i < bs.size(); ++i) {
    xg_batch* b = bs[i].get();
    b->co = cos[i];
    if (!check_launch_fits(b->co.bin, "xg_batch", b->block, err) ||
        !check_kernel_args(b->co.bin, "xg_batch", (int64_t)b->bargs_size, err))
      continue;  // cannot be resident, or an argument layout the bodies cannot read
    if (batch_ws_bytes(b, n.data()) > workspace_bytes) continue;
    if (bs.size() == 1) { besti = 0; break; }  // the cached choice
    if (batch_launch(b, args, d_workspace, stream) != XG_OK) continue;  // warm
    (void)hipEventRecord(e0, (hipStream_t)stream);
    const int reps = 5;
    for (int r = 0; r < reps; ++r) (void)batch_launch(b, args, d_workspace, stream);
    (void)hipEventRecord(e1, (hipStream_t)stream);
    if (hipEventSynchronize(e1) != hipSuccess) continue;
    float ms = 0;
    (void)hipEventElapsedTime(&ms, e0, e1);
    if (progs[0]->opt.verbose)
      std::fprintf(stderr, "[xg batch autotune] block %d: %.3f ms\n", b->block, ms / reps);
    if (ms < best) { best = ms; besti = (int)i; }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (besti < 0) {
    for (auto& b : bs) xg_batch_free(b.release());
    set_error("batch autotune: no candidate fits (registers or workspace)");
    return XG_EUNSUPPORTED;
  }
  for (size_t i = 0; i < bs.size(); ++i)
    if ((int)i != besti) xg_batch_free(bs[i].release());
  if (!cached) {
    std::ofstream f(path);
    f << blocks[besti] << "\n";
  }
  if (chosen_block) *chosen_block = blocks[besti];
  *out = bs[besti].release();
  return XG_OK;
}

}  // extern "C"

extern "C" {

xg_status xg_autotune(xg_program* p, int64_t n, const void* const* d_in, const int64_t* ld_in,
                      void* const* d_out, const int64_t* ld_out, void* d_workspace,
                      size_t workspace_bytes, void* stream, xg_options* chosen) {
  if (!p || n <= 0) { set_error("bad argument"); return XG_EINVAL; }
  return tune_mode(p, n, 0, workspace_bytes, stream, chosen, [&](xg_program* q) {
    return xg_eval(q, n, d_in, ld_in, d_out, ld_out, d_workspace, stream);
  });
}

xg_status xg_autotune_adjoint(xg_program* p, int64_t n, const void* const* d_in, const int64_t* ld_in,
                              const void* const* d_out_bar, const int64_t* ld_out_bar,
                              void* const* d_out, const int64_t* ld_out, void* const* d_in_bar,
                              const int64_t* ld_in_bar, void* d_workspace, size_t workspace_bytes,
                              void* stream, xg_options* chosen) {
  if (!p || n <= 0) { set_error("bad argument"); return XG_EINVAL; }
  return tune_mode(p, n, d_out ? 2 : 1, workspace_bytes, stream, chosen, [&](xg_program* q) {
    return xg_eval_adjoint(q, n, d_in, ld_in, d_out_bar, ld_out_bar, d_out, ld_out, d_in_bar, ld_in_bar,
                           d_workspace, stream);
  });
}

}  // extern "C"

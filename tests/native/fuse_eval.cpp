// Test driver: the library's graph passes before planning (negations folded
// into sums, products joined to sums) evaluated on the CPU by a sequential
// walk, so they can be checked without a GPU.
//
//   fuse_eval <desc.txt> <inputs.bin> <outputs.bin>
//
// desc.txt and inputs.bin as for adjoint_eval (inputs only, no seeds).
// outputs.bin: per instance the outputs of the plain graph, of the graph
// with folded negations and of the fused graph, doubles; then the operation
// counts of the three graphs.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <string>
#include <vector>

#include "xg_internal.h"

namespace {

double apply(int op, double a, double b, double c) {
  switch (op) {
    case XG_OP_ADD: return a + b;
    case XG_OP_SUB: return a - b;
    case XG_OP_MUL: return a * b;
    case XG_OP_DIV: return a / b;
    case XG_OP_NEG: return -a;
    case XG_OP_SQ: return a * a;
    case XG_OP_SQRT: return std::sqrt(a);
    case XG_OP_EXP: return std::exp(a);
    case XG_OP_SIN: return std::sin(a);
    case XG_OP_COS: return std::cos(a);
    case XG_OP_TANH: return std::tanh(a);
    case XG_OP_FABS: return std::fabs(a);
    case XG_OP_FMIN: return std::fmin(a, b);
    case XG_OP_FMAX: return std::fmax(a, b);
    case XG_OP_LT: return a < b ? 1.0 : 0.0;
    case XG_OP_LE: return a <= b ? 1.0 : 0.0;
    case xg::kOpFma: return std::fma(a, b, c);
    case xg::kOpFms: return std::fma(a, b, -c);
    case xg::kOpFnma: return std::fma(-a, b, c);
  }
  std::abort();
}

void walk(const xg::Graph& g, const std::vector<long long>& off, const std::vector<double>& x, std::ofstream& fo) {
  std::vector<double> w(g.nodes.size());
  for (size_t k = 0; k < g.nodes.size(); ++k) {
    const xg::Node& nd = g.nodes[k];
    if (nd.op == XG_OP_INPUT) w[k] = x[off[nd.aux >> 32] + (nd.aux & 0xffffffff)];
    else if (nd.op == XG_OP_CONST) w[k] = g.consts[nd.aux];
    else w[k] = apply(nd.op, w[nd.a], nd.b >= 0 ? w[nd.b] : 0.0, nd.c >= 0 ? w[nd.c] : 0.0);
  }
  for (auto& arg : g.out)
    for (int32_t v : arg) fo.write((const char*)&w[v], 8);
}

double ops(const xg::Graph& g) {
  double n = 0;
  for (const xg::Node& nd : g.nodes) n += xg::is_arith(nd.op) && nd.op != XG_OP_NEG;
  return n;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 4) return 2;
  std::ifstream f(argv[1]);
  int dtype, n_work, n_in, n_out, n_const;
  long long n_instr;
  f >> dtype >> n_work >> n_in;
  std::vector<int32_t> nnz_in(n_in);
  for (auto& v : nnz_in) f >> v;
  f >> n_out;
  std::vector<int32_t> nnz_out(n_out);
  for (auto& v : nnz_out) f >> v;
  f >> n_const;
  std::vector<double> consts(n_const);
  for (auto& c : consts) { std::string s; f >> s; c = std::strtod(s.c_str(), nullptr); }
  f >> n_instr;
  std::vector<xg_instr> ins(n_instr);
  int p;
  for (auto& in : ins) f >> in.op >> in.out >> in.a >> in.b >> p;
  if (!f) return 2;
  xg_program_desc d{n_in, nnz_in.data(), n_out, nnz_out.data(), n_work, n_instr, ins.data(),
                    n_const, consts.data(), dtype, nullptr};
  xg::Graph g0;
  std::string err;
  if (!xg::build_graph(d, g0, err)) { std::fprintf(stderr, "%s\n", err.c_str()); return 3; }
  xg::Graph g1 = g0;
  xg::fold_negations(g1, true);
  xg::Graph g2 = g1;
  xg::fuse_multiply_adds(g2);
  std::ifstream fi(argv[2], std::ios::binary);
  long long N = 0;
  fi.read((char*)&N, 8);
  std::vector<long long> off(n_in + 1, 0);
  for (int a = 0; a < n_in; ++a) off[a + 1] = off[a] + nnz_in[a];
  std::vector<double> x(off.back());
  std::ofstream fo(argv[3], std::ios::binary);
  for (long long i = 0; i < N; ++i) {
    fi.read((char*)x.data(), (std::streamsize)(8 * x.size()));
    if (!fi) return 4;
    for (const xg::Graph* g : {&g0, &g1, &g2}) walk(*g, off, x, fo);
  }
  const double n[3] = {ops(g0), ops(g1), ops(g2)};
  fo.write((const char*)n, 24);
  return 0;
}

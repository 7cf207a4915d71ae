// Kernel generation for groups in which values reduced over whole tensors feed ops on whole tensors (gradient clipping
// by the global norm and its like).  No single kernel covers such a group without a wait between its workgroups, and cut
// at every reduction it is a chain of launches whose middle links work on a few numbers.  Here it is two kernels: the
// first reduces every tensor to one partial result per workgroup, the second adds the partial results in every
// workgroup (a few KB that stay in the caches), evaluates the ops on the scalars there, in registers, and goes
// through the tensors once more.  The order of stream work is the only hand-over.  Partial results are doubles and are
// added in a fixed order, so results are bit-reproducible.
#include "grid_codegen.h"
#include "ew_ir.h"
#include "launchers.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

namespace fs {

const char* ew_preamble();                                   // ew_codegen.cpp
const char* row_reduce_preamble();                           // row_codegen.cpp
std::string ew_op_text(const EwIrNode& n, bool fast);        // ew_codegen.cpp
bool ew_analyse_parts(const Graph& g, std::vector<EwIr>* parts, std::string* err);   // ew_stitch.hip

namespace {

struct Emitter {
  std::string s;
  void line(const char* fmt, ...) __attribute__((format(printf, 2, 3))) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    s += buf;
    s += '\n';
  }
};

constexpr int kThreads = 256;
// Partial results in all: one per workgroup of the first kernel, and a workgroup of the second reads every one of them.
constexpr int64_t kPartials = 4096;

struct Reduction { int node = -1; bool is_max = false; int part = -1; int64_t first = 0, count = 0; };

// One tensor's work in a kernel: its ops, and how its elements are cut into chunks.
struct Part {
  EwIr ir;
  int W = 1;                 // elements of a chunk
  int64_t n_chunks = 0;      // the last one is moved back to end with the tensor where W does not divide it
  int64_t blocks = 0;        // workgroups
  std::vector<int> scalar_of_view;    // per view: the scalar it stands for, or -1
  int n_full = 0;
};

// The rule of a chunk: one 16-byte access of the narrowest tensor; element alignment is enough for the last chunk, since
// all others start on whole chunks.
bool lay_out(Part* p) {
  // values numbered within the part, so that parts with the same ops read the same
  std::map<int, int> number;
  for (EwIrNode& n : p->ir.nodes) {
    for (int j = 0; j < n.n_operands; ++j) if (n.opnd[j].kind == EW_FROM_NODE) n.opnd[j].index = number[n.opnd[j].index];
    const int id = (int)number.size();
    n.id = number[n.id] = id;
  }
  bool any32 = false;
  for (size_t k = 0; k < p->ir.views.size(); ++k) {
    if (p->scalar_of_view[k] >= 0) continue;
    if (!p->ir.views[k].full) return false;
    ++p->n_full;
    if (p->ir.views[k].dtype == FS_F32) any32 = true;
  }
  for (const EwIrNode& n : p->ir.nodes) if (n.out_ordinal >= 0 && n.out_dtype == FS_F32) any32 = true;
  for (const EwIrNode& n : p->ir.nodes) if (n.op == FS_CAUSAL_MASK) return false;
  if (p->n_full == 0 || p->ir.n < 1) return false;
  p->W = any32 ? 4 : 8;
  while (p->W > p->ir.n) p->W /= 2;
  if (p->W == 2) p->W = 1;
  p->n_chunks = (p->ir.n + p->W - 1) / p->W;
  return true;
}

bool is_fast(const EwIr& ir) {      // as in the elementwise kernels: 16-bit groups take the short forms of tanh and exp
  for (const EwIrView& v : ir.views) if (v.dtype != FS_F32) return true;
  for (const EwIrNode& n : ir.nodes) if (n.out_ordinal >= 0 && n.out_dtype != FS_F32) return true;
  return false;
}

// the type of a chunk as it is loaded, and with the alignment of its element
const char* raw_type(int dtype, int W) { return dtype == FS_F32 ? (W == 4 ? "f32x4" : "float") : W == 8 ? "u32x4" : W == 4 ? "u32x2" : "unsigned short"; }

// requests of U chunks: raw<k>[u], addresses clamped to the tensor (`last` is the last valid chunk of the workgroup's run)
void emit_requests(Emitter& e, const Part& p, const char* last, bool nontemporal, bool declare = true) {
  for (size_t k = 0; k < p.ir.views.size(); ++k)
    if (declare && p.scalar_of_view[k] < 0) e.line("    %s raw%zu[U];", raw_type(p.ir.views[k].dtype, p.W), k);
  e.line("    UNROLL for (int u = 0; u < U; ++u) {");
  e.line("      long long c = c0 + u * %d + (int)threadIdx.x;", kThreads);
  e.line("      c = c > %s ? %s : c;", last, last);
  e.line("      const long long e0 = c == NV - 1 ? N - W : c * W;");
  int slot = 0;
  for (size_t k = 0; k < p.ir.views.size(); ++k) {
    if (p.scalar_of_view[k] >= 0) continue;
    const EwIrView& v = p.ir.views[k];
    const char* ty = v.dtype == FS_F32 ? "float" : "unsigned short";
    if (p.W == 1) e.line("      raw%zu[u] = static_cast<const %s*>(pi%d)[e0];", k, ty, slot);
    else e.line("      raw%zu[u] = %s(reinterpret_cast<const %se*>(static_cast<const %s*>(pi%d) + e0));", k, nontemporal ? "__builtin_nontemporal_load" : "*", raw_type(v.dtype, p.W), ty, slot);
    ++slot;
  }
  e.line("    }");
}

// the ops on chunk u: t<id>[W]
void emit_ops(Emitter& e, const Part& p, bool stores) {
  const bool fast = is_fast(p.ir);
  for (size_t k = 0; k < p.ir.views.size(); ++k) {
    const EwIrView& v = p.ir.views[k];
    e.line("      float v%zu[W];", k);
    if (p.scalar_of_view[k] >= 0) {
      e.line("      UNROLL for (int j = 0; j < W; ++j) v%zu[j] = sc%d;", k, p.scalar_of_view[k]);
    } else if (p.W == 1) {
      e.line("      v%zu[0] = %s(raw%zu[u]);", k, v.dtype == FS_F32 ? "" : v.dtype == FS_F16 ? "f16_lo" : "bf16_lo", k);
    } else if (v.dtype == FS_F32) {
      e.line("      UNROLL for (int j = 0; j < 4; ++j) v%zu[j] = raw%zu[u][j];", k, k);
    } else {
      const char* lo = v.dtype == FS_F16 ? "f16_lo" : "bf16_lo";
      const char* hi = v.dtype == FS_F16 ? "f16_hi" : "bf16_hi";
      e.line("      UNROLL for (int j = 0; j < W / 2; ++j) { v%zu[2 * j] = %s(raw%zu[u][j]); v%zu[2 * j + 1] = %s(raw%zu[u][j]); }", k, lo, k, k, hi, k);
    }
  }
  int slot = 0;
  for (const EwIrNode& n : p.ir.nodes) {
    e.line("      float t%d[W];", n.id);
    e.line("      UNROLL for (int j = 0; j < W; ++j) t%d[j] = %s;", n.id, ew_op_text(n, fast).c_str());
    if (!stores || n.out_ordinal < 0) continue;
    const bool f32 = n.out_dtype == FS_F32;
    const char* ty = f32 ? "float" : "unsigned short";
    const char* cv = f32 ? "" : n.out_dtype == FS_F16 ? "to_f16" : "to_bf16";
    e.line("      if (own > 0) {");
    e.line("        %s* p = static_cast<%s*>(po%d) + e0;", ty, ty, slot);
    e.line("        if (own < W || W == 1) {");
    e.line("          UNROLL for (int j = 0; j < W; ++j) if (j >= W - own) p[j] = (%s)%s(t%d[j]);", ty, cv, n.id);
    e.line("        } else {");
    if (p.W > 1 && f32) {
      e.line("          __builtin_nontemporal_store(f32x4e{t%d[0], t%d[1], t%d[2], t%d[3]}, reinterpret_cast<f32x4e*>(p));", n.id, n.id, n.id, n.id);
    } else if (p.W > 1) {
      e.line("          unsigned w[W / 2];");
      e.line("          UNROLL for (int j = 0; j < W / 2; ++j) w[j] = pack_%s(t%d[2 * j], t%d[2 * j + 1]);", cv, n.id, n.id);
      if (p.W == 8) e.line("          __builtin_nontemporal_store(u32x4e{w[0], w[1], w[2], w[3]}, reinterpret_cast<u32x4e*>(p));");
      else e.line("          __builtin_nontemporal_store(u32x2e{w[0], w[1]}, reinterpret_cast<u32x2e*>(p));");
    }
    e.line("        }");
    e.line("      }");
    ++slot;
  }
}

// Tensors with the same ops share one piece of code: which of them a workgroup works on is a choice of pointers and
// sizes, made with scalar compares (a piece per tensor is eight times the instructions to fetch).
struct Classes {
  std::vector<std::string> text;
  std::vector<std::vector<int>> members;
  void add(int part, const std::string& body) {
    for (size_t k = 0; k < text.size(); ++k) if (text[k] == body) { members[k].push_back(part); return; }
    text.push_back(body);
    members.push_back({part});
  }
};

void emit_choice(Emitter& e, const std::vector<Part>& parts, const std::vector<int>& members, int64_t first, const std::vector<int>& in_base,
                 const std::vector<std::vector<int>>& outs) {
  const Part& p0 = parts[members[0]];
  e.line("    long long N = %lldll, NV = %lldll; unsigned first = %lldu;", (long long)p0.ir.n, (long long)p0.n_chunks, (long long)first);
  for (int v = 0; v < p0.n_full; ++v) e.line("    const void* pi%d = a.in[%d];", v, in_base[members[0]] + v);
  for (size_t o = 0; o < outs[members[0]].size(); ++o) e.line("    void* po%zu = a.out[%d];", o, outs[members[0]][o]);
  int64_t at = first + p0.blocks;
  for (size_t m = 1; m < members.size(); ++m) {
    const Part& p = parts[members[m]];
    e.line("    if (blockIdx.x >= %lldu) {", (long long)at);
    e.line("      N = %lldll; NV = %lldll; first = %lldu;", (long long)p.ir.n, (long long)p.n_chunks, (long long)at);
    for (int v = 0; v < p.n_full; ++v) e.line("      pi%d = a.in[%d];", v, in_base[members[m]] + v);
    for (size_t o = 0; o < outs[members[m]].size(); ++o) e.line("      po%zu = a.out[%d];", o, outs[members[m]][o]);
    e.line("    }");
    at += p.blocks;
  }
}

}  // namespace

bool two_step_plan(const Graph& g, TwoStepLaunch* out, std::string* err) {
  auto fail = [&](const std::string& m) { *err = "two-step schedule: " + m; return false; };
  const int n = g.size();
  auto is_reduce = [&](int i) { return g[i].kind == FS_REDUCE_SUM || g[i].kind == FS_REDUCE_MAX; };
  auto canon = [&](int i) { while (g[i].kind == FS_CONVERT && g[i].dtype == FS_F32) i = g[i].operand[0]; return i; };
  auto elementwise = [&](int i) { return is_binary(g[i].kind) || is_unary(g[i].kind) || g[i].kind == FS_CONVERT; };
  std::vector<int> users(n, 0);
  for (int i = 0; i < n; ++i) {
    const Node& x = g[i];
    if (x.numel() == 0) return fail("an empty tensor");
    if (x.kind == FS_DOT || x.kind == FS_CAUSAL_MASK) return fail("an op outside its vocabulary");
    for (int j = 0; j < operand_count(x.kind); ++j) ++users[x.operand[j]];
  }
  // ---- the reductions: chains of one kind down to rank 0, each over a value that depends on no reduction
  std::vector<char> in_chain(n, 0), depends(n, 0);      // depends: on a reduced value
  std::vector<int> red_of(n, -1), source;
  std::vector<Reduction> reds;
  for (int i = 0; i < n; ++i) {
    for (int j = 0; j < operand_count(g[i].kind); ++j) if (depends[g[i].operand[j]] || red_of[g[i].operand[j]] >= 0) depends[i] = 1;
    if (!is_reduce(i) || g[i].rank != 0) continue;
    if (depends[i]) return fail("a reduction of a value that depends on another reduction");
    int cur = i;
    for (;;) {
      if (g[cur].dtype != FS_F32) return fail("a reduction in 16 bits");
      in_chain[cur] = 1;
      const int below = g[cur].operand[0];
      if (!is_reduce(below)) break;
      if (g[below].kind != g[i].kind || users[below] != 1) return fail("a reduction that does not end in one scalar");
      cur = below;
    }
    Reduction r;
    r.node = i;
    r.is_max = g[i].kind == FS_REDUCE_MAX;
    red_of[i] = (int)reds.size();
    reds.push_back(r);
    source.push_back(g[cur].operand[0]);
  }
  for (int i = 0; i < n; ++i) if (is_reduce(i) && !in_chain[i]) return fail("a reduction that does not end in one scalar");
  if (reds.empty()) return fail("no reduction over a whole tensor");
  if (reds.size() > 64) return fail("more than 64 reductions");

  // ---- first kernel: a part per reduction, its ops as an elementwise group that ends in the value to reduce
  auto copy_op = [&](int i, const std::vector<int>& to) {
    fs_op_desc d{};
    const Node& x = g[i];
    d.kind = x.kind; d.dtype = x.dtype; d.rank = x.rank; d.axis = x.axis; d.attr = x.attr;
    for (int k = 0; k < FS_MAX_RANK; ++k) d.shape[k] = k < x.rank ? x.shape[k] : 0;
    for (int k = 0; k < 3; ++k) d.operand[k] = k < operand_count(x.kind) ? to[x.operand[k]] : -1;
    return d;
  };
  auto push = [&](std::vector<fs_op_desc>* list, int kind, int dtype, const Node& shape, int a, int b, double attr) {
    fs_op_desc d{};
    d.kind = kind; d.dtype = dtype; d.rank = shape.rank; d.attr = attr;
    for (int k = 0; k < FS_MAX_RANK; ++k) d.shape[k] = k < shape.rank ? shape.shape[k] : 0;
    d.operand[0] = a; d.operand[1] = b; d.operand[2] = -1;
    list->push_back(d);
    return (int)list->size() - 1;
  };
  Node scalar;
  scalar.dtype = FS_F32;
  TwoStepLaunch l;
  std::vector<Part> first(reds.size());
  std::vector<int> in_base1(reds.size());
  for (size_t r = 0; r < reds.size(); ++r) {
    std::vector<char> need(n, 0);
    need[source[r]] = 1;
    for (int i = n - 1; i >= 0; --i) if (need[i]) for (int j = 0; j < operand_count(g[i].kind); ++j) need[g[i].operand[j]] = 1;
    std::vector<fs_op_desc> list;
    std::vector<int> to(n, -1);
    std::vector<int> ordinal;      // of the part's parameters in the group
    for (int i = 0; i < n; ++i) if (need[i]) {
      if (g[i].kind == FS_PARAMETER) ordinal.push_back(g[i].ordinal);
      list.push_back(copy_op(i, to));
      to[i] = (int)list.size() - 1;
    }
    int end = to[source[r]];
    const Node& shape = g[source[r]];
    const int src = canon(source[r]);
    if (!elementwise(src) || g[src].dtype != FS_F32) {
      // an input as it is, or a value rounded to 16 bits: one more op, whose value is the one to reduce
      const int one = push(&list, FS_CONSTANT, FS_F32, scalar, -1, -1, 1.0);
      end = push(&list, FS_MULTIPLY, FS_F32, shape, end, one, 0.0);
    }
    push(&list, FS_OUTPUT, FS_F32, shape, end, -1, 0.0);
    Graph part;
    std::vector<EwIr> irs;
    std::string why;
    if (!build_graph(list.data(), (int32_t)list.size(), &part, &why) || !ew_analyse_parts(part, &irs, &why)) return fail(why);
    if (irs.size() != 1) return fail("a reduction over several independent values");
    Part& p = first[r];
    p.ir = irs[0];
    p.scalar_of_view.assign(p.ir.views.size(), -1);
    if (!lay_out(&p)) return fail("a broadcast operand below a reduction");
    for (const EwIrNode& x : p.ir.nodes) if (x.out_ordinal >= 0 && x.out_dtype != FS_F32) return fail("a reduction in 16 bits");
    in_base1[r] = (int)l.view_param[0].size();
    for (const EwIrView& v : p.ir.views) l.view_param[0].push_back(ordinal[v.param]);
  }
  if (l.view_param[0].size() > 64) return fail("more than 64 operand views");

  // ---- the scalars: the rank-0 ops that ops on tensors read
  std::vector<char> is_scalar(n, 0);
  for (int i = 0; i < n; ++i) is_scalar[i] = elementwise(i) && g[i].rank == 0 && canon(i) == i;
  std::vector<int> wanted, scalar_at(n, -1);      // scalars that ops on tensors or outputs read
  auto want = [&](int i) { if (scalar_at[i] < 0) { scalar_at[i] = (int)wanted.size(); wanted.push_back(i); } };
  std::vector<std::pair<int, int>> scalar_outs;   // (output ordinal, scalar)
  for (int i = 0; i < n; ++i) {
    const Node& x = g[i];
    if (x.kind == FS_BROADCAST) {
      const int s = canon(x.operand[0]);
      if (is_scalar[s] || red_of[s] >= 0 || (g[s].kind == FS_PARAMETER && g[s].rank == 0 && g[s].dtype == FS_F32)) want(s);
      else if (depends[s]) return fail("a computed value that is broadcast in another way than as a scalar");
    } else if (x.kind == FS_OUTPUT && x.rank == 0) {
      const int s = canon(x.operand[0]);
      if (!is_scalar[s] && red_of[s] < 0) return fail("an output that is a plain copy of an input");
      if (x.dtype != FS_F32) return fail("a scalar output in 16 bits");
      want(s);
      scalar_outs.push_back({x.ordinal, scalar_at[s]});
    }
  }
  std::vector<EwIrNode> scalars;                  // in list order; a view is an entry of scalar_param
  std::vector<int> scalar_param;                  // reduction r, or 1000 + ordinal of a rank-0 input
  std::vector<int> scalar_id(wanted.size(), -1);  // the op that makes it, or -1 - entry of scalar_param
  {
    bool reads = false;
    for (int w : wanted) reads = reads || depends[w] || red_of[w] >= 0;
    if (!reads) return fail("no op on a whole tensor reads a reduced value");
    std::vector<char> need(n, 0);
    std::vector<int> entry(n, -1);
    for (int w : wanted) need[w] = 1;
    for (int i = n - 1; i >= 0; --i) if (need[i] && red_of[i] < 0) for (int j = 0; j < operand_count(g[i].kind); ++j) need[g[i].operand[j]] = 1;
    for (int i = 0; i < n; ++i) if (need[i]) {
      if (g[i].rank != 0 || g[i].kind == FS_BROADCAST) return fail("a scalar that is made of a tensor");
      if (g[i].kind == FS_CONSTANT) continue;
      if (g[i].dtype != FS_F32) return fail("a scalar in 16 bits");
      if (red_of[i] >= 0 || g[i].kind == FS_PARAMETER) {
        entry[i] = (int)scalar_param.size();
        scalar_param.push_back(red_of[i] >= 0 ? red_of[i] : 1000 + g[i].ordinal);
        continue;
      }
      if (canon(i) != i) continue;                // a widening convert: its operand's value
      EwIrNode x;
      x.id = i; x.op = g[i].kind;
      x.n_operands = operand_count(x.op);
      for (int j = 0; j < x.n_operands; ++j) {
        const int o = canon(g[i].operand[j]);
        if (g[o].kind == FS_CONSTANT) { x.opnd[j].kind = EW_FROM_CONST; x.opnd[j].cval = (float)g[o].attr; }
        else if (entry[o] >= 0) { x.opnd[j].kind = EW_FROM_VIEW; x.opnd[j].index = entry[o]; }
        else { x.opnd[j].kind = EW_FROM_NODE; x.opnd[j].index = o; }
      }
      scalars.push_back(x);
    }
    for (size_t w = 0; w < wanted.size(); ++w) scalar_id[w] = entry[wanted[w]] >= 0 ? -1 - entry[wanted[w]] : wanted[w];
  }

  // ---- second kernel: the ops on tensors, with the scalars they read as further rank-0 inputs
  std::vector<Part> second;
  const int n_params = (int)g.params.size();
  {
    std::vector<char> need(n, 0);
    for (int o : g.outputs) if (g[o].rank > 0) need[o] = 1;
    for (int i = n - 1; i >= 0; --i) {
      if (!need[i]) continue;
      if (scalar_at[i] >= 0) continue;
      if (is_reduce(i)) return fail("a reduced value read as a tensor");
      for (int j = 0; j < operand_count(g[i].kind); ++j) need[scalar_at[canon(g[i].operand[j])] >= 0 ? canon(g[i].operand[j]) : g[i].operand[j]] = 1;
    }
    std::vector<fs_op_desc> list;
    std::vector<int> to(n, -1);
    for (int i = 0; i < n; ++i) if (g[i].kind == FS_PARAMETER) { list.push_back(copy_op(i, to)); to[i] = (int)list.size() - 1; }
    std::vector<int> at_scalar(wanted.size());
    for (size_t w = 0; w < wanted.size(); ++w) at_scalar[w] = push(&list, FS_PARAMETER, FS_F32, scalar, -1, -1, 0.0);
    for (int i = 0; i < n; ++i) if (scalar_at[canon(i)] >= 0) to[i] = at_scalar[scalar_at[canon(i)]];
    std::vector<int> out_ordinal;
    for (int i = 0; i < n; ++i) if (need[i] && to[i] < 0) {
      list.push_back(copy_op(i, to));
      to[i] = (int)list.size() - 1;
      if (g[i].kind == FS_OUTPUT) out_ordinal.push_back(g[i].ordinal);
    }
    if (out_ordinal.empty()) return fail("no output of the shape of a tensor");
    Graph part;
    std::vector<EwIr> irs;
    std::string why;
    if (!build_graph(list.data(), (int32_t)list.size(), &part, &why) || !ew_analyse_parts(part, &irs, &why)) return fail(why);
    for (EwIr& ir : irs) {
      Part p;
      p.ir = ir;
      for (EwIrNode& x : p.ir.nodes) if (x.out_ordinal >= 0) x.out_ordinal = out_ordinal[x.out_ordinal];
      for (const EwIrView& v : ir.views) p.scalar_of_view.push_back(v.param >= n_params ? v.param - n_params : -1);
      if (!lay_out(&p)) return fail("a broadcast operand beside a reduced value");
      second.push_back(p);
    }
  }
  if (g.outputs.size() > 16) return fail("more than 16 outputs");

  // ---- geometry
  // Bound by memory.  A thread has U chunks in flight, a workgroup U * kThreads chunks of a tensor, in both kernels: eight where that leaves
  // every CU a workgroup, fewer in smaller groups and beside more operands.  A workgroup of the second kernel then works on what the
  // workgroup of the same number has read in the first (in fp32 groups; in 16-bit ones, whose reduced value is fp32, the first kernel's chunks are
  // of four elements), and workgroups of one number run on one XCD: as far as the tensors
  // fit the XCDs' caches they are read from there (4 MB each, 32 in all; the rest comes from the memory-side cache).
  // Replayed graphs, in us; clipping of eight fp32 tensors of width 1024 (42 MB; 84 read, 42 written) and of sixteen of width 1600 (164 MB):
  //   as here                                      19.4 and 76; as four launches of packed groups 26.3, with twelve single scalars 104
  //   the same runs in both kernels                19.4; of 1281 chunks in the first and 2048 in the second 23.2; four chunks a thread and eight 22.2
  //   loads, ordinary and then nontemporal         19.4 and 76; ordinary in the second too 22.3 and 84; nontemporal in the first too 23.3 and 84
  //   a workgroup on every CU                      2.6 MB: 6.1; two 6.8; as four launches 8.3
  //   up to 4096 partial results, then further runs of a workgroup behind its first: 210 MB in two tensors 95.5, up to 8192 109, up to 1024 95.1, as launches
  //                                                of their own 105.8; 335 MB in sixteen 153, 155 and 160
  // The second kernel's workgroups in reverse order: no gain (19.4 and 76).
  int64_t total = 0, total2 = 0;
  int widest = 1;
  for (const Part& p : first) { total += p.n_chunks; widest = std::max(widest, p.n_full); }
  for (const Part& p : second) { total2 += p.n_chunks; widest = std::max(widest, p.n_full); }
  // (beyond that the launches of their own are ahead: one tensor of 537 MB 249 us, 260 so)
  int64_t read = 0;
  for (const Part& p : first) for (const EwIrView& v : p.ir.views) read += p.ir.n * (v.dtype == FS_F32 ? 4 : 2);
  if (read > (400ll << 20)) return fail("tensors of more than 400 MB");
  int U = std::max(1, 8 / widest);
  while (U > 1 && std::max(total, total2) < (int64_t)U * kThreads * 256) U /= 2;
  const int64_t run = (int64_t)U * kThreads;
  const int64_t per = ((total + kPartials - 1) / kPartials + run - 1) / run * run;      // chunks of a workgroup of the first kernel
  for (Part& p : first) p.blocks = (p.n_chunks + per - 1) / per;
  for (Part& p : second) p.blocks = (p.n_chunks + per - 1) / per;

  // ---- first kernel's text
  Emitter e;
  e.s = ew_preamble();
  e.s += row_reduce_preamble();
  e.s += R"SRC(
typedef float f32x4e __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u32x2e __attribute__((ext_vector_type(2), aligned(2)));
typedef unsigned u32x4e __attribute__((ext_vector_type(4), aligned(2)));
static __device__ __forceinline__ double wave_sum(double v) { UNROLL for (int m = 1; m < 64; m <<= 1) v += shfl_xor_f64(v, m); return v; }
static __device__ __forceinline__ double wave_max(double v) { UNROLL for (int m = 1; m < 64; m <<= 1) v = fmax(v, shfl_xor_f64(v, m)); return v; }
)SRC";
  Classes cls;
  for (size_t r = 0; r < first.size(); ++r) {
    const Part& p = first[r];
    const bool mx = reds[r].is_max;
    Emitter b;
    b.line("    constexpr int W = %d, U = %d; constexpr long long per = %lld;", p.W, U, (long long)per);
    b.line("    const long long lo = (long long)(blockIdx.x - first) * per, hi = lo + per < NV ? lo + per : NV;");
    b.line("    double acc = %s;", mx ? "-__builtin_inf()" : "0.0");
    b.line("    for (long long c0 = lo; c0 < hi; c0 += U * %d) {", kThreads);
    emit_requests(b, p, "(hi - 1)", false);
    b.line("    UNROLL for (int u = 0; u < U; ++u) {");
    b.line("      const long long c = c0 + u * %d + (int)threadIdx.x;", kThreads);
    emit_ops(b, p, false);
    int id = -1;
    for (const EwIrNode& x : p.ir.nodes) if (x.out_ordinal >= 0) id = x.id;
    // (the last chunk of a tensor: its first elements are its neighbour's)
    b.line("      const int skip = c == NV - 1 ? (int)(NV * W - N) : 0;");
    b.line("      float s = %s;", mx ? "-__builtin_inff()" : "0.0f");
    b.line("      UNROLL for (int j = 0; j < W; ++j) s = j >= skip ? %s : s;", mx ? ("fmaxf(s, t" + std::to_string(id) + "[j])").c_str() : ("s + t" + std::to_string(id) + "[j]").c_str());
    b.line("      if (c < hi) acc = %s;", mx ? "fmax(acc, (double)s)" : "acc + (double)s");
    b.line("    }");
    b.line("    }");
    b.line("    acc = %s(acc);", mx ? "wave_max" : "wave_sum");
    b.line("    if ((threadIdx.x & 63) == 0) exch[threadIdx.x >> 6] = acc;");
    b.line("    __syncthreads();");
    if (mx) b.line("    if (threadIdx.x == 0) static_cast<double*>(a.ws)[blockIdx.x] = fmax(fmax(exch[0], exch[1]), fmax(exch[2], exch[3]));");
    else b.line("    if (threadIdx.x == 0) static_cast<double*>(a.ws)[blockIdx.x] = (exch[0] + exch[1]) + (exch[2] + exch[3]);");
    cls.add((int)r, b.s);
  }
  e.line("extern \"C\" __global__ __launch_bounds__(%d) void FS_GRID_REDUCE(const Args a) {", kThreads);
  e.line("  __shared__ double exch[4];");
  int64_t at = 0;
  const std::vector<std::vector<int>> no_outs(first.size());
  for (size_t k = 0; k < cls.text.size(); ++k) {
    int64_t blocks = 0;
    for (int m : cls.members[k]) { reds[m].first = at + blocks; reds[m].count = first[m].blocks; blocks += first[m].blocks; }
    e.line("  if (blockIdx.x < %lldu) {", (long long)(at + blocks));
    emit_choice(e, first, cls.members[k], at, in_base1, no_outs);
    e.s += cls.text[k];
    e.line("    return;");
    e.line("  }");
    at += blocks;
  }
  e.line("}");
  l.grid[0] = (int)at;
  l.n_partials = at;

  // ---- second kernel's text
  std::vector<int> in_base2(second.size());
  std::vector<std::vector<int>> outs2(second.size());
  for (size_t q = 0; q < second.size(); ++q) {
    in_base2[q] = (int)l.view_param[1].size();
    for (size_t k = 0; k < second[q].ir.views.size(); ++k) if (second[q].scalar_of_view[k] < 0) l.view_param[1].push_back(second[q].ir.views[k].param);
    for (const EwIrNode& x : second[q].ir.nodes) if (x.out_ordinal >= 0) outs2[q].push_back(x.out_ordinal);
  }
  std::vector<int> input_slot(scalar_param.size(), -1);
  for (size_t k = 0; k < scalar_param.size(); ++k) if (scalar_param[k] >= 1000) { input_slot[k] = (int)l.view_param[1].size(); l.view_param[1].push_back(scalar_param[k] - 1000); }
  if (l.view_param[1].size() > 64) return fail("more than 64 operand views");
  // Every workgroup adds the partial results: a wavefront takes its share of the reductions whole, so that each is one
  // straight line of loads and one butterfly; one of more than 1024 partial results (a single large tensor) is cut into four.
  struct Piece { size_t red; int64_t first, count; };
  std::vector<Piece> pieces;
  std::vector<std::vector<size_t>> pieces_of(reds.size());
  for (size_t r = 0; r < reds.size(); ++r) {
    const int64_t cuts = reds[r].count > 1024 ? 4 : 1, each = (reds[r].count + cuts - 1) / cuts;
    for (int64_t from = 0; from < reds[r].count; from += each) {
      pieces_of[r].push_back(pieces.size());
      pieces.push_back(Piece{r, reds[r].first + from, std::min(each, reds[r].count - from)});
    }
  }
  std::vector<size_t> by_count(pieces.size());
  for (size_t r = 0; r < pieces.size(); ++r) by_count[r] = r;
  std::stable_sort(by_count.begin(), by_count.end(), [&](size_t x, size_t y) { return pieces[x].count > pieces[y].count; });
  std::vector<std::vector<size_t>> share(kThreads / 64);
  std::vector<int64_t> load(kThreads / 64, 0);
  for (size_t r : by_count) {
    const size_t w = std::min_element(load.begin(), load.end()) - load.begin();
    share[w].push_back(r);
    load[w] += (pieces[r].count + 63) / 64 + 2;
  }
  Emitter pro;
  pro.line("    {");
  pro.line("      const double* const ps = static_cast<const double*>(a.ws);");
  pro.line("      const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;");
  for (size_t w = 0; w < share.size(); ++w) {
    if (share[w].empty()) continue;
    pro.line("      if (wave == %zu) {", w);
    for (size_t r : share[w]) {
      const Piece& q = pieces[r];
      const bool mx = reds[q.red].is_max;
      pro.line("        double q%zu = %s;", r, mx ? "-__builtin_inf()" : "0.0");
      // (at most sixteen loads in flight: a piece is of 1024 partial results or fewer, kPartials of them being cut into four)
      pro.line("        UNROLL for (int i = 0; i < %lld; ++i) { const int at = i * 64 + lane; if (at < %lld) q%zu = %s; }", (long long)((q.count + 63) / 64), (long long)q.count, r,
               ((mx ? "fmax(q" + std::to_string(r) + ", ps[" : "q" + std::to_string(r) + " + (ps[") + std::to_string(q.first) + " + at])").c_str());
    }
    for (size_t r : share[w]) pro.line("        q%zu = %s(q%zu);", r, reds[pieces[r].red].is_max ? "wave_max" : "wave_sum", r);
    pro.line("        if (lane == 0) {");
    for (size_t r : share[w]) pro.line("          red[%zu] = q%zu;", r, r);
    pro.line("        }");
    pro.line("      }");
  }
  pro.line("    }");
  pro.line("    __syncthreads();");
  for (size_t w = 0; w < wanted.size(); ++w) pro.line("    float sc%zu;", w);
  pro.line("    {");
  pro.line("      constexpr int j = 0;");
  auto param_text = [&](int k) {
    if (scalar_param[k] >= 1000) return "static_cast<const float*>(a.in[" + std::to_string(input_slot[k]) + "])[0]";
    std::string t;
    for (size_t q : pieces_of[scalar_param[k]]) {
      const std::string one = "red[" + std::to_string(q) + "]";
      t = t.empty() ? one : reds[scalar_param[k]].is_max ? "fmax(" + t + ", " + one + ")" : t + " + " + one;
    }
    return "(float)(" + t + ")";
  };
  for (size_t k = 0; k < scalar_param.size(); ++k) pro.line("      const float v%zu[1] = {%s};", k, param_text((int)k).c_str());
  for (const EwIrNode& x : scalars) pro.line("      const float t%d[1] = {%s};", x.id, ew_op_text(x, false).c_str());
  for (size_t w = 0; w < wanted.size(); ++w) {
    if (scalar_id[w] >= 0) pro.line("      sc%zu = t%d[j];", w, scalar_id[w]);
    else pro.line("      sc%zu = %s;", w, param_text(-1 - scalar_id[w]).c_str());
  }
  for (const auto& so : scalar_outs) pro.line("      if (blockIdx.x == 0 && threadIdx.x == 0) static_cast<float*>(a.out[%d])[0] = sc%d;", so.first, so.second);
  pro.line("    }");

  Classes cls2;
  for (size_t q = 0; q < second.size(); ++q) {
    const Part& p = second[q];
    Emitter b;
    b.line("    constexpr int W = %d, U = %d; constexpr long long per = %lld;", p.W, U, (long long)per);
    b.line("    const long long lo = (long long)(blockIdx.x - first) * per, hi = lo + per < NV ? lo + per : NV;");
    b.line("    long long c0 = lo;");
    // the tensors' first requests go out before the partial results are asked for
    emit_requests(b, p, "(hi - 1)", true);
    b.s += pro.s;
    b.line("    for (;;) {");
    b.line("    UNROLL for (int u = 0; u < U; ++u) {");
    b.line("      const long long c = c0 + u * %d + (int)threadIdx.x;", kThreads);
    b.line("      const long long e0 = c == NV - 1 ? N - W : c * W;");
    b.line("      const int own = c >= hi ? 0 : c == NV - 1 ? (int)(N - (NV - 1) * W) : W;      // elements of the chunk that are not its neighbour's");
    emit_ops(b, p, true);
    b.line("    }");
    b.line("    c0 += U * %d;", kThreads);
    b.line("    if (c0 >= hi) break;");
    emit_requests(b, p, "(hi - 1)", true, false);
    b.line("    }");
    cls2.add((int)q, b.s);
  }
  e.line("extern \"C\" __global__ __launch_bounds__(%d) void FS_GRID_APPLY(const Args a) {", kThreads);
  e.line("  __shared__ double red[%zu];", pieces.size());
  at = 0;
  for (size_t k = 0; k < cls2.text.size(); ++k) {
    int64_t blocks = 0;
    for (int m : cls2.members[k]) blocks += second[m].blocks;
    e.line("  if (blockIdx.x < %lldu) {", (long long)(at + blocks));
    emit_choice(e, second, cls2.members[k], at, in_base2, outs2);
    e.s += cls2.text[k];
    e.line("    return;");
    e.line("  }");
    at += blocks;
  }
  e.line("}");
  if (at > 0x3fffffffLL) return fail("too many workgroups for one grid");
  l.grid[1] = (int)at;

  // both kernels named after the whole text
  uint64_t h = 1469598103934665603ull;
  for (unsigned char c : e.s) { h ^= c; h *= 1099511628211ull; }
  const char* tags[2] = {"FS_GRID_REDUCE", "FS_GRID_APPLY"};
  const char* stems[2] = {"fs_grid_reduce", "fs_grid_apply"};
  for (int k = 0; k < 2; ++k) {
    char name[48];
    snprintf(name, sizeof name, "%s_%08x", stems[k], (unsigned)(h ^ (h >> 32)));
    l.kernel_name[k] = name;
    e.s.replace(e.s.find(tags[k]), strlen(tags[k]), name);
  }
  if (const char* dump = getenv("FS_DUMP_SOURCE")) {        // debugging aid: append what was generated
    if (FILE* f = fopen(dump, "a")) { fputs(e.s.c_str(), f); fputs("\n// ----\n", f); fclose(f); }
  }
  std::string cerr;
  if (!ew_compile_source(e.s, &l.code_object, &cerr)) return fail(cerr);
  l.n_reduce = (int)reds.size();
  l.n_scalar_ops = (int)scalars.size();
  l.parts = (int)second.size();
  l.wg = kThreads;
  l.lds_bytes = std::max<int64_t>(32, (int64_t)pieces.size() * 8);
  *out = l;
  return true;
}

std::string two_step_describe(const TwoStepLaunch& l) {
  char buf[512];
  snprintf(buf, sizeof buf, "reduce x%d over whole tensors[GRID,CTA-S] (%lld partial results, kernel %s, cta_num=%d), then scalars x%d and elementwise[GRID,CTA-THREAD] in %d parts "
           "(kernel %s, cta_num=%d; %zu bytes of code); cta_size=%d, lds=%lld",
           l.n_reduce, (long long)l.n_partials, l.kernel_name[0].c_str(), l.grid[0], l.n_scalar_ops, l.parts, l.kernel_name[1].c_str(), l.grid[1], l.code_object.size(), l.wg, (long long)l.lds_bytes);
  return buf;
}

int two_step_launch(TwoStepLaunch& l, const void* const* in, void* const* out, int n_out, void* partials, void* stream, std::string* err) {
  struct { const void* in[64]; void* out[16]; void* ws; } args;      // mirrors Args of the generated source
  for (int k = 0; k < 2; ++k) {
    memset(&args, 0, sizeof args);
    for (size_t v = 0; v < l.view_param[k].size(); ++v) args.in[v] = in[l.view_param[k][v]];
    for (int o = 0; k == 1 && o < n_out && o < 16; ++o) args.out[o] = out[o];
    args.ws = partials;
    const int rc = ew_module_launch(&l.loaded[k], l.code_object, l.kernel_name[k], &args, sizeof args, l.grid[k], l.wg, stream, err, k == 1 ? &l.loaded[0] : nullptr);
    if (rc != 0) return rc;
  }
  return 0;
}

void two_step_release(TwoStepLaunch& l) {
  ew_module_release(&l.loaded[1]);      // (the first kernel's module holds both)
  ew_module_release(&l.loaded[0]);
}

}  // namespace fs

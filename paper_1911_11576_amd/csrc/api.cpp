// The C ABI of fs.h: plan construction (validate -> recognise -> size), launch, destroy.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <cmath>
#include <mutex>
#include <new>
#include <set>
#include <string>
#include <vector>

#include "../../include/fs.h"
#include "ew_ir.h"
#include "graph.h"
#include "launchers.h"
#include "match.h"
#include "per_op.h"
#include "row_codegen.h"
#include "shared_plan.h"
#include "fusion_plan.h"
#include "plan.h"

struct fs_fusion {
  fs::FusionResult result;
};

namespace fs {
fs_status set_error(fs_status st, const std::string& msg);
}
using fs::set_error;

namespace {

thread_local std::string g_error = "";

// ---- tuning cache: winning options of fs_plan_tune per group key
struct TuneEntry { fs_plan_options opt; double us; };
std::mutex g_tune_mu;
std::map<uint64_t, TuneEntry> g_tune;
thread_local bool g_tuning = false;     // the tuner's own plans are built from the options it passes

uint64_t group_key(const fs_op_desc* ops, int32_t n_ops) {
  uint64_t h = 1469598103934665603ull;
  auto mix = [&](uint64_t v) { for (int b = 0; b < 8; ++b) { h ^= (v >> (8 * b)) & 0xffu; h *= 1099511628211ull; } };
  mix((uint64_t)n_ops);
  for (int i = 0; i < n_ops; ++i) {
    const fs_op_desc& d = ops[i];
    mix((uint64_t)(uint32_t)d.kind); mix((uint64_t)(uint32_t)d.dtype); mix((uint64_t)(uint32_t)d.rank); mix((uint64_t)(uint32_t)d.axis);
    const int r = d.rank < 0 ? 0 : d.rank > FS_MAX_RANK ? FS_MAX_RANK : d.rank;
    for (int k = 0; k < r; ++k) mix((uint64_t)d.shape[k]);
    for (int k = 0; k < 3; ++k) mix((uint64_t)(uint32_t)d.operand[k]);
    uint64_t a;
    memcpy(&a, &d.attr, 8);
    mix(a);
  }
  return h;
}

// The options recorded for a group, if it was tuned.
bool tuned_options(const fs_op_desc* ops, int32_t n_ops, fs_plan_options* opt) {
  if (g_tuning || !ops || n_ops < 1 || n_ops > 4096) return false;
  std::lock_guard<std::mutex> lock(g_tune_mu);
  if (g_tune.empty()) return false;
  const auto it = g_tune.find(group_key(ops, n_ops));
  if (it == g_tune.end()) return false;
  *opt = it->second.opt;
  return true;
}

fs_status plan_create_impl(const fs_op_desc* ops, int32_t n_ops, const fs_plan_options* opt, fs_plan** out);
void collapse_reductions(fs::Graph* g);

}  // namespace

fs_status fs::set_error(fs_status st, const std::string& msg) {
  g_error = msg;
  return st;
}

extern "C" {

const char* fs_last_error(void) { return g_error.c_str(); }

fs_status fs_plan_create(const fs_op_desc* ops, int32_t n_ops, const fs_plan_options* opt, fs_plan** out) {
  if (!out) return set_error(FS_ERR_INVALID, "out is NULL");
  const bool defaults = !opt || (opt->mode == FS_MODE_STITCHED && opt->wg_size == 0 && opt->rows_per_wave == 0 && opt->grid == 0);
  fs_plan_options tuned{};
  // recorded options that no longer build (another library version wrote the file): the defaults
  if (defaults && tuned_options(ops, n_ops, &tuned) && plan_create_impl(ops, n_ops, &tuned, out) == FS_OK) return FS_OK;
  return plan_create_impl(ops, n_ops, opt, out);
}

fs_status fs_plan_create_packed(const fs_op_desc* const* groups, const int32_t* n_ops, int32_t n_groups, uint8_t* taken, fs_plan** out) {
  if (!out) return set_error(FS_ERR_INVALID, "out is NULL");
  *out = nullptr;
  if (!groups || !n_ops || !taken || n_groups < 1 || n_groups > 4096) return set_error(FS_ERR_INVALID, "fs_plan_create_packed: NULL argument or n_groups out of range [1,4096]");
  try {
    std::vector<fs::Graph> graphs((size_t)n_groups);
    std::vector<char> apart((size_t)n_groups, 0);
    for (int32_t k = 0; k < n_groups; ++k) {
      taken[k] = 0;
      std::string err;
      if (!fs::build_graph(groups[k], n_ops[k], &graphs[k], &err)) return set_error(FS_ERR_INVALID, err);
      collapse_reductions(&graphs[k]);
      // a tuned group's own plan is the one that was timed
      fs_plan_options tuned{};
      apart[k] = tuned_options(groups[k], n_ops[k], &tuned);
    }
    std::unique_ptr<fs_plan> p(new fs_plan);
    std::vector<char> which;
    int st = FS_OK;
    std::string err;
    if (!fs::row_gen_plan_packed(graphs, apart, &which, &p->row_gen, &st, &err)) return set_error((fs_status)st, err);
    // the launch's own list: the lists of the groups taken, one behind the other
    std::vector<fs_op_desc> list;
    for (int32_t k = 0; k < n_groups; ++k) {
      if (!which[k]) continue;
      const int base = (int)list.size();
      for (int32_t i = 0; i < n_ops[k]; ++i) {
        fs_op_desc d = groups[k][i];
        for (int j = 0; j < 3; ++j) if (d.operand[j] >= 0) d.operand[j] += base;
        list.push_back(d);
      }
    }
    if (!fs::build_graph(list.data(), (int32_t)list.size(), &p->graph, &err)) return set_error(FS_ERR_UNSUPPORTED, err);
    for (int32_t k = 0; k < n_groups; ++k) taken[k] = (uint8_t)which[k];
    p->mode = FS_MODE_STITCHED;
    p->match.kind = fs::MATCH_NONE;
    p->schedule = FS_SCHED_ROW;
    p->row_form = 3;
    p->lds_bytes = p->row_gen.lds_bytes;
    p->moved_bytes = p->graph.algorithmic_bytes();
    p->n_kernels = 1;
    p->description = fs::row_gen_describe(p->row_gen);
    *out = p.release();
  } catch (const std::bad_alloc&) {
    return set_error(FS_ERR_NOMEM, "out of host memory");
  } catch (...) {
    return set_error(FS_ERR_INVALID, "internal error while planning");
  }
  return FS_OK;
}

fs_status fs_plan_create_two_step(const fs_op_desc* ops, int32_t n_ops, int64_t* partial_bytes, fs_plan** out) {
  if (!out) return set_error(FS_ERR_INVALID, "out is NULL");
  *out = nullptr;
  if (!partial_bytes) return set_error(FS_ERR_INVALID, "fs_plan_create_two_step: partial_bytes is NULL");
  try {
    std::unique_ptr<fs_plan> p(new fs_plan);
    std::string err;
    if (!fs::build_graph(ops, n_ops, &p->graph, &err)) return set_error(FS_ERR_INVALID, err);
    if (!fs::two_step_plan(p->graph, &p->two_step, &err)) return set_error(FS_ERR_UNSUPPORTED, err);
    p->mode = FS_MODE_STITCHED;
    p->match.kind = fs::MATCH_NONE;
    p->schedule = FS_SCHED_TWO_STEP;
    p->lds_bytes = p->two_step.lds_bytes;
    p->n_kernels = 2;
    *partial_bytes = p->two_step.n_partials * 8;
    p->moved_bytes = p->graph.algorithmic_bytes() + 2 * *partial_bytes;
    for (int v : p->two_step.view_param[0]) {         // (what the first kernel reads is read once more)
      const fs::Node& x = p->graph[p->graph.params[v]];
      p->moved_bytes += x.numel() * (x.dtype == FS_F32 ? 4 : 2);
    }
    p->description = fs::two_step_describe(p->two_step);
    *out = p.release();
  } catch (const std::bad_alloc&) {
    return set_error(FS_ERR_NOMEM, "out of host memory");
  } catch (...) {
    return set_error(FS_ERR_INVALID, "internal error while planning");
  }
  return FS_OK;
}

fs_status fs_kernel_cache_dir(const char* dir) {
  try {
    fs::codegen_cache_dir(dir);
  } catch (...) {
    return set_error(FS_ERR_NOMEM, "out of host memory");
  }
  return FS_OK;
}

fs_status fs_kernel_cache_stats(int64_t* compiled, int64_t* from_memory, int64_t* from_disk) {
  fs::codegen_cache_stats(compiled, from_memory, from_disk);
  return FS_OK;
}

fs_status fs_kernel_cache_drop_memory(void) {
  fs::codegen_cache_drop_memory();
  return FS_OK;
}

fs_status fs_group_key(const fs_op_desc* ops, int32_t n_ops, uint64_t* key) {
  if (!ops || !key || n_ops < 1 || n_ops > 4096) return set_error(FS_ERR_INVALID, "fs_group_key: NULL argument or n_ops out of range [1,4096]");
  *key = group_key(ops, n_ops);
  return FS_OK;
}

int32_t fs_tune_cache_has(uint64_t key) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  return g_tune.count(key) ? 1 : 0;
}

int32_t fs_tune_cache_size(void) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  return (int32_t)g_tune.size();
}

fs_status fs_tune_cache_clear(void) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  g_tune.clear();
  return FS_OK;
}

fs_status fs_tune_cache_save(const char* path) {
  if (!path) return set_error(FS_ERR_INVALID, "fs_tune_cache_save: path is NULL");
  FILE* f = fopen(path, "w");
  if (!f) return set_error(FS_ERR_INVALID, std::string("fs_tune_cache_save: cannot write ") + path);
  fprintf(f, "fs-tune-cache 1\n");
  {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    for (const auto& kv : g_tune)
      fprintf(f, "%016llx %d %d %d %d %.3f\n", (unsigned long long)kv.first, kv.second.opt.mode, kv.second.opt.wg_size,
              kv.second.opt.rows_per_wave, kv.second.opt.grid, kv.second.us);
  }
  if (fclose(f) != 0) return set_error(FS_ERR_INVALID, std::string("fs_tune_cache_save: write failed on ") + path);
  return FS_OK;
}

fs_status fs_tune_cache_load(const char* path) {
  if (!path) return set_error(FS_ERR_INVALID, "fs_tune_cache_load: path is NULL");
  FILE* f = fopen(path, "r");
  if (!f) return set_error(FS_ERR_INVALID, std::string("fs_tune_cache_load: cannot read ") + path);
  const std::unique_ptr<FILE, int (*)(FILE*)> closer(f, fclose);
  try {
  std::map<uint64_t, TuneEntry> read;
  char line[256];
  bool ok = fgets(line, sizeof line, f) && strncmp(line, "fs-tune-cache 1", 15) == 0;
  int lineno = 1;
  while (ok && fgets(line, sizeof line, f)) {
    ++lineno;
    if (line[0] == '\n' || line[0] == '\0') continue;
    unsigned long long key = 0;
    TuneEntry e{};
    int used = 0;
    if (sscanf(line, "%llx %d %d %d %d %lf %n", &key, &e.opt.mode, &e.opt.wg_size, &e.opt.rows_per_wave, &e.opt.grid, &e.us, &used) != 6 ||
        line[used] != '\0' || e.opt.mode < 0 || e.opt.mode > FS_MODE_STITCHED_GENERATED || e.opt.mode == FS_MODE_PER_OP ||
        e.opt.wg_size < 0 || e.opt.rows_per_wave < 0 || e.opt.grid < 0 || !(e.us >= 0.0)) {
      ok = false;
      break;
    }
    read[(uint64_t)key] = e;
  }
  if (!ok) {
    char buf[96];
    snprintf(buf, sizeof buf, ": malformed line %d", lineno);
    return set_error(FS_ERR_INVALID, std::string("fs_tune_cache_load: ") + path + buf);
  }
  std::lock_guard<std::mutex> lock(g_tune_mu);
  for (const auto& kv : read) g_tune[kv.first] = kv.second;
  } catch (...) {
    return set_error(FS_ERR_NOMEM, "out of host memory");
  }
  return FS_OK;
}

}  // extern "C"

namespace {

// The graph of a group as the generator takes it: chained reductions over the trailing dims become one reduction over a
// merged dim, reductions over the leading dim that keep the inner dims one over merged inner dims (same memory).
void collapse_reductions(fs::Graph* g) {
  std::vector<fs_op_desc> merged;
  for (int step = 0; step < FS_MAX_RANK && fs::collapse_trailing_reductions(*g, &merged); ++step) {
    fs::Graph g2;
    std::string err;
    if (!fs::build_graph(merged.data(), (int32_t)merged.size(), &g2, &err)) break;
    *g = g2;
  }
  if (fs::collapse_kept_dims_of_leading_reductions(*g, &merged)) {
    fs::Graph g2;
    std::string err;
    if (fs::build_graph(merged.data(), (int32_t)merged.size(), &g2, &err)) *g = g2;
  }
}

fs_status plan_create_impl(const fs_op_desc* ops, int32_t n_ops, const fs_plan_options* opt, fs_plan** out) {
  if (!out) return set_error(FS_ERR_INVALID, "out is NULL");
  *out = nullptr;
  fs_plan* p = new (std::nothrow) fs_plan;
  if (!p) return set_error(FS_ERR_NOMEM, "out of host memory");
  std::string err;
  try {
    if (!fs::build_graph(ops, n_ops, &p->graph, &err)) { delete p; return set_error(FS_ERR_INVALID, err); }
    fs::LaunchOpts lo;
    bool want_generated = false;
    if (opt) {
      if (opt->mode != FS_MODE_STITCHED && opt->mode != FS_MODE_PER_OP && opt->mode != FS_MODE_STITCHED_PREBUILT &&
          opt->mode != FS_MODE_STITCHED_GENERATED) {
        delete p;
        return set_error(FS_ERR_INVALID, "unknown mode");
      }
      if (opt->wg_size < 0 || opt->rows_per_wave < 0 || opt->grid < 0) { delete p; return set_error(FS_ERR_INVALID, "negative launch option"); }
      p->mode = opt->mode == FS_MODE_PER_OP ? FS_MODE_PER_OP : FS_MODE_STITCHED;
      lo.codegen = opt->mode != FS_MODE_STITCHED_PREBUILT;
      want_generated = opt->mode == FS_MODE_STITCHED_GENERATED;
      lo.wg_size = opt->wg_size; lo.rows_per_wave = opt->rows_per_wave; lo.grid = opt->grid;
    }
    if (p->mode != FS_MODE_PER_OP) {
      collapse_reductions(&p->graph);
    }
    const int64_t algo = p->graph.algorithmic_bytes();
    if (p->mode == FS_MODE_PER_OP) {
      if (!fs::per_op_plan(p->graph, &p->per_op, &err)) { delete p; return set_error(FS_ERR_UNSUPPORTED, err); }
      p->schedule = FS_SCHED_PER_OP;
      p->n_kernels = p->per_op.n_kernels;
      p->workspace_bytes = p->per_op.workspace_bytes;
      p->moved_bytes = p->per_op.moved_bytes;
      p->description = fs::per_op_describe(p->per_op);
    } else {
      p->moved_bytes = algo;
      // the plan's fields once p->row_gen holds a generated row kernel
      auto adopt_generated_row_kernel = [&]() {
        p->match.kind = fs::MATCH_NONE;
        p->schedule = p->row_gen.mma ? FS_SCHED_BLOCK_DOT : p->row_gen.n_col > 0 ? FS_SCHED_ROW_COL : FS_SCHED_ROW;
        p->row_form = 3;
        p->lds_bytes = p->row_gen.lds_bytes;
        p->workspace_bytes = p->row_gen.workspace_bytes;
        p->moved_bytes = algo + 2 * p->row_gen.workspace_bytes;
        p->n_kernels = p->row_gen.n_kernels;
        p->description = fs::row_gen_describe(p->row_gen);
      };
      const bool recognised = fs::recognise(p->graph, &p->match);
      if (!recognised || want_generated) {
        // Not one of the hand-written reduce / dot patterns (or the caller prefers generated
        // kernels): an all-elementwise group stitches as schedule 0, a group of elementwise
        // ops and row reductions as a generated row kernel.
        const std::string why = p->match.why;
        bool has_reduce = false;
        for (const fs::Node& x : p->graph.nodes) if (x.kind == FS_REDUCE_SUM || x.kind == FS_REDUCE_MAX) has_reduce = true;
        int st = FS_OK, st2 = FS_ERR_UNSUPPORTED;
        std::string err2;
        if (fs::ew_stitch_plan(p->graph, lo, &p->ew, &st, &err)) {
          p->match.kind = fs::MATCH_NONE;
          p->schedule = FS_SCHED_ELEMENTWISE;
          p->lds_bytes = p->ew.lds_bytes;
          p->description = fs::ew_stitch_describe(p->ew);
        } else if (lo.codegen && fs::row_gen_plan(p->graph, lo, &p->row_gen, &st2, &err2)) {
          adopt_generated_row_kernel();
        } else if (!recognised) {
          if (lo.codegen && (has_reduce || st2 == FS_ERR_INVALID)) { st = st2; err = err2; }
          else if (lo.codegen && st == FS_ERR_UNSUPPORTED && !err2.empty()) err += "; " + err2;
          if (st == FS_ERR_UNSUPPORTED && why != "no stitched schedule matches this group") err = why + " (" + err + ")";
          delete p;
          return set_error((fs_status)st, err);
        } else if (st2 == FS_ERR_INVALID) {
          delete p;
          return set_error(FS_ERR_INVALID, err2);
        }
      }
      // a recognised group whose hand-written kernel does not take its size: the generated row kernel
      std::string gen_err;
      auto fall_back_to_generated = [&]() {
        if (!lo.codegen) return false;
        int st2 = FS_OK;
        if (!fs::row_gen_plan(p->graph, lo, &p->row_gen, &st2, &gen_err)) return false;
        adopt_generated_row_kernel();
        return true;
      };
      switch (p->match.kind) {
        case fs::MATCH_NONE: break;   // elementwise schedule, set up above
        case fs::MATCH_ROW:
          p->schedule = FS_SCHED_ROW;
          // With the GELU prologue the generated kernel measured faster than the hand-written one
          // (18.3 against 19.0 us on config 4): the default where kernels may be generated and the
          // caller fixes no launch shape; the hand-written one serves the prebuilt mode.
          if (p->match.row.gelu && lo.codegen && lo.wg_size == 0 && lo.rows_per_wave == 0 && lo.grid == 0 && fall_back_to_generated()) break;
          if (fs::row_stitch_plan(p->match.row, lo, &p->row, &err)) {
            p->lds_bytes = p->row.lds_bytes;
            p->description = fs::row_stitch_describe(p->match.row, p->row);
          } else if (err.find("wg_size") != std::string::npos || err.find("rows_per_wave") != std::string::npos) {
            delete p;
            return set_error(FS_ERR_INVALID, err);
          } else if (fs::row_team_plan(p->match.row, lo, &p->row_team, &err)) {
            // the row does not fit one wavefront: a team of wavefronts holds it in registers
            p->row_form = 1;
            p->lds_bytes = 2 * 16 * 4;
            p->description = fs::row_team_describe(p->match.row, p->row_team);
          } else {
            // a row shorter than one vector, or too long for a team: block-composed form, row cached in LDS
            int st = FS_OK;
            fs::LaunchOpts lb = lo;
            if (!fs::row_block_plan(p->match.row, lb, &p->row_block, &st, &err)) {
              if (st != FS_ERR_INVALID && fall_back_to_generated()) break;
              delete p;
              return set_error((fs_status)st, err);
            }
            p->row_form = 2;
            p->lds_bytes = p->row_block.lds_bytes;
            p->description = fs::row_block_describe(p->match.row, p->row_block);
          }
          break;
        case fs::MATCH_LNBWD:
          // The hand-written kernel (rows requested two steps ahead, per-wavefront LDS arrays) measured
          // faster than the generated one on config 5 (69.0 against 71.2 us): it is the default where it
          // takes the shape (fp32, up to 1024 columns, with teams of wavefronts up to 4096); the generated kernel serves the other shapes and
          // FS_MODE_STITCHED_GENERATED.
          if (want_generated && fall_back_to_generated()) break;
          // Few rows: one launch.
          if (!want_generated && (lo.codegen || (p->match.lnbwd.cols % 4 == 0 && p->match.lnbwd.cols <= 1024)) && fs::lnbwd_packed_plan(p->match.lnbwd, lo, &p->lnbwd)) {
            p->schedule = FS_SCHED_ROW_COL;
            p->lds_bytes = p->lnbwd.lds_bytes;
            p->n_kernels = 1;
            p->description = fs::lnbwd_packed_describe(p->lnbwd);
            break;
          }
          if (!want_generated && fs::lnbwd_team_plan(p->match.lnbwd, lo, &p->lnbwd)) {
            p->schedule = FS_SCHED_ROW_COL;
            p->lds_bytes = p->lnbwd.lds_bytes;
            p->workspace_bytes = p->lnbwd.workspace_bytes;
            p->n_kernels = p->lnbwd.n_kernels;
            p->moved_bytes = algo + 2 * p->lnbwd.workspace_bytes;
            p->description = fs::lnbwd_team_describe(p->lnbwd);
            break;
          }
          if (!fs::lnbwd_stitch_plan(p->match.lnbwd, lo, &p->lnbwd, &err)) {
            const bool bad_opt = err.find("wg_size") != std::string::npos;
            if (!bad_opt && fall_back_to_generated()) break;
            if (!bad_opt && !gen_err.empty()) err += "; " + gen_err;
            delete p;
            return set_error(bad_opt ? FS_ERR_INVALID : FS_ERR_UNSUPPORTED, err);
          }
          p->schedule = FS_SCHED_ROW_COL;
          p->lds_bytes = p->lnbwd.lds_bytes;
          p->workspace_bytes = p->lnbwd.workspace_bytes;
          p->n_kernels = p->lnbwd.n_kernels;
          p->moved_bytes = algo + 2 * (p->lnbwd.workspace_bytes);
          p->description = fs::lnbwd_stitch_describe(p->match.lnbwd, p->lnbwd);
          break;
        case fs::MATCH_ATTN: {
          int st = FS_OK;
          if (!fs::attn_stitch_plan(p->match.attn, lo, &p->attn, &st, &err)) { delete p; return set_error((fs_status)st, err); }
          p->schedule = FS_SCHED_BDOT_SOFTMAX;
          p->lds_bytes = p->attn.lds_bytes;
          p->description = fs::attn_stitch_describe(p->match.attn, p->attn);
          break;
        }
        default:
          delete p;
          return set_error(FS_ERR_UNSUPPORTED, "no stitched schedule matches this group");
      }
    }
  } catch (const std::bad_alloc&) {
    delete p;
    return set_error(FS_ERR_NOMEM, "out of host memory");
  } catch (...) {
    delete p;
    return set_error(FS_ERR_INVALID, "internal error while planning");
  }
  *out = p;
  return FS_OK;
}

}  // namespace

extern "C" {

}  // extern "C"

// Arguments of a launch checked against the plan (counts, NULL and alignment, identical pointers).
fs_status fs::check_launch_args(fs_plan* p, const void* const* inputs, int32_t n_in, void* const* outputs, int32_t n_out) {
  if (!p) return set_error(FS_ERR_INVALID, "plan is NULL");
  const fs::Graph& g = p->graph;
  if (n_in != (int32_t)g.params.size()) return set_error(FS_ERR_INVALID, "n_in differs from the number of parameters");
  const bool two_step = p->schedule == FS_SCHED_TWO_STEP;
  if (n_out != (int32_t)g.outputs.size() + (two_step ? 1 : 0)) return set_error(FS_ERR_INVALID, "n_out differs from the number of outputs");
  if (!inputs || !outputs) return set_error(FS_ERR_INVALID, "inputs/outputs is NULL");
  for (int i = 0; i < n_in; ++i) {
    if (g[g.params[i]].numel() == 0) continue;
    if (!inputs[i] || (reinterpret_cast<uintptr_t>(inputs[i]) & 15)) return set_error(FS_ERR_INVALID, "input pointer is NULL or not 16-byte aligned");
  }
  if (two_step) {
    // the partial results: one more output, of no op
    const void* partials = outputs[--n_out];
    if (!partials || (reinterpret_cast<uintptr_t>(partials) & 15)) return set_error(FS_ERR_INVALID, "output pointer is NULL or not 16-byte aligned");
    for (int k = 0; k < n_out; ++k) if (outputs[k] == partials) return set_error(FS_ERR_INVALID, "two outputs share one buffer");
    for (int k = 0; k < n_in; ++k) if (inputs[k] == partials) return set_error(FS_ERR_INVALID, "an output shares its buffer with an input");
  }
  for (int i = 0; i < n_out; ++i) {
    if (g[g.outputs[i]].numel() == 0) continue;
    if (!outputs[i] || (reinterpret_cast<uintptr_t>(outputs[i]) & 15)) return set_error(FS_ERR_INVALID, "output pointer is NULL or not 16-byte aligned");
    for (int k = 0; k < i; ++k)
      if (outputs[k] == outputs[i] && g[g.outputs[k]].numel() != 0) return set_error(FS_ERR_INVALID, "two outputs share one buffer");
    // An output in the very buffer of a parameter (an update in place): fine where the kernel reads
    // every element of that parameter once, in the thread (or the row's lanes) that writes the same
    // element, before it writes -- the generated elementwise kernels and the generated register
    // row kernels, for parameters of the output's own shape and dtype that are read in no other way, and the
    // hand-written LayerNorm backward where its plan says so, for dx.
    for (int k = 0; k < n_in; ++k) {
      if (inputs[k] != outputs[i] || g[g.params[k]].numel() == 0) continue;
      const fs::Node& pn = g[g.params[k]];
      const fs::Node& on = g[g.outputs[i]];
      bool ok = p->mode == FS_MODE_STITCHED && pn.dtype == on.dtype && pn.same_shape(on);
      const std::vector<int>* vp = nullptr;
      const std::vector<char>* vf = nullptr;
      if (ok && p->schedule == FS_SCHED_ELEMENTWISE && p->ew.generated) { vp = &p->ew.view_param; vf = &p->ew.view_full; }
      else if (ok && p->schedule == FS_SCHED_ROW_COL && p->row_form != 3 && p->lnbwd.in_place) ok = !fs::lnbwd_broadcasts(p->match.lnbwd, pn.ordinal);      // (dy and x have dx's shape alone)
      else if (ok && p->row_form == 3 && !p->row_gen.streamed && p->row_gen.rows_read_before_written &&
               (p->schedule == FS_SCHED_ROW || p->schedule == FS_SCHED_ROW_COL)) { vp = &p->row_gen.view_param; vf = &p->row_gen.view_dense; }
      else ok = false;
      for (size_t q = 0; ok && vp && q < vp->size(); ++q) if ((*vp)[q] == pn.ordinal && !(*vf)[q]) ok = false;
      if (!ok) return set_error(FS_ERR_INVALID, "an output shares its buffer with an input that this plan may still read after writing it "
                                                "(in-place updates: generated elementwise and register row kernels, LayerNorm backward plans that say so; same shape and dtype, parameter read only as the group's own layout)");
    }
  }
  return FS_OK;
}

// The plan's kernels enqueued with `workspace` as their scratch memory (the plan's own, or the static array).
fs_status fs::enqueue_plan(fs_plan* p, const void* const* inputs, void* const* outputs, int32_t n_out, void* workspace,
                              void* hip_stream) {
  std::string err;
  try {
    int rc = 0;
    switch (p->schedule) {
      case FS_SCHED_ROW:
        rc = p->row_form == 3   ? fs::row_gen_launch(p->row_gen, inputs, outputs, n_out, workspace, hip_stream, &err)
             : p->row_form == 2 ? fs::row_block_launch(p->match.row, p->row_block, inputs, outputs, hip_stream, &err)
             : p->row_form == 1 ? fs::row_team_launch(p->match.row, p->row_team, inputs, outputs, hip_stream, &err)
                                : fs::row_stitch_launch(p->match.row, p->row, inputs, outputs, hip_stream, &err);
        break;
      case FS_SCHED_ROW_COL:
        rc = p->row_form == 3  ? fs::row_gen_launch(p->row_gen, inputs, outputs, n_out, workspace, hip_stream, &err)
             : p->lnbwd.packed ? fs::lnbwd_packed_launch(p->match.lnbwd, p->lnbwd, inputs, outputs, hip_stream, &err)
             : p->lnbwd.teams  ? fs::lnbwd_team_launch(p->match.lnbwd, p->lnbwd, inputs, outputs, workspace, hip_stream, &err)
                               : fs::lnbwd_stitch_launch(p->match.lnbwd, p->lnbwd, inputs, outputs, workspace, hip_stream, &err);
        break;
      case FS_SCHED_BLOCK_DOT: rc = fs::row_gen_launch(p->row_gen, inputs, outputs, n_out, workspace, hip_stream, &err); break;
      case FS_SCHED_BDOT_SOFTMAX: rc = fs::attn_stitch_launch(p->match.attn, p->attn, inputs, outputs, hip_stream, &err); break;
      case FS_SCHED_ELEMENTWISE: rc = fs::ew_stitch_launch(p->ew, inputs, outputs, n_out, hip_stream, &err); break;
      case FS_SCHED_TWO_STEP: rc = fs::two_step_launch(p->two_step, inputs, outputs, n_out - 1, outputs[n_out - 1], hip_stream, &err); break;
      default: rc = fs::per_op_launch(p->graph, p->per_op, inputs, outputs, workspace, hip_stream, &err); break;
    }
    if (rc != 0) return set_error(FS_ERR_HIP, err);
  } catch (...) {
    return set_error(FS_ERR_HIP, "internal error while launching");
  }
  return FS_OK;
}

extern "C" {

fs_status fs_launch(fs_plan* p, const void* const* inputs, int32_t n_in, void* const* outputs, int32_t n_out,
                    void* hip_stream) {
  const fs_status st = fs::check_launch_args(p, inputs, n_in, outputs, n_out);
  if (st != FS_OK) return st;
  if (p->workspace_bytes > 0) {
    // Nothing in the workspace needs an initial value: every kernel that reads it reads only what an
    // earlier kernel of the same launch wrote there.
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return set_error(FS_ERR_HIP, "hipGetDevice failed");
    if (!p->workspace) {
      const hipError_t e = hipMalloc(&p->workspace, (size_t)p->workspace_bytes);
      if (e != hipSuccess) { p->workspace = nullptr; return set_error(FS_ERR_NOMEM, std::string("workspace hipMalloc: ") + hipGetErrorString(e)); }
      p->device = dev;
    } else if (dev != p->device) {
      return set_error(FS_ERR_INVALID, "plan is bound to the device of its first launch");
    }
  }
  return fs::enqueue_plan(p, inputs, outputs, n_out, p->workspace, hip_stream);
}

fs_status fs_plan_tune(const fs_op_desc* ops, int32_t n_ops, const void* const* inputs, int32_t n_in,
                       void* const* outputs, int32_t n_out, void* hip_stream, int32_t trials, fs_plan** out,
                       fs_plan_options* best, double* best_us) {
  if (!out) return set_error(FS_ERR_INVALID, "out is NULL");
  *out = nullptr;
  if (trials < 1 || trials > 1000) return set_error(FS_ERR_INVALID, "trials out of range [1,1000]");
  try {
  // the default template first: it decides the schedule, and it is the fallback
  struct Tuning { Tuning() { g_tuning = true; } ~Tuning() { g_tuning = false; } } tuning_scope;
  fs_plan* base = nullptr;
  fs_status st = fs_plan_create(ops, n_ops, nullptr, &base);
  if (st != FS_OK) return st;
  // launch templates worth trying for each schedule (TemplatesGeneration, pruned by hand as
  // the paper does for JIT use)
  std::vector<fs_plan_options> cands;
  cands.push_back(fs_plan_options{FS_MODE_STITCHED, 0, 0, 0});
  if (base->schedule == FS_SCHED_ROW && base->row_form == 0) {
    for (int wg : {128, 256, 512})
      for (int u : {1, 2, 4}) cands.push_back(fs_plan_options{FS_MODE_STITCHED, wg, u, 0});
    cands.push_back(fs_plan_options{FS_MODE_STITCHED_GENERATED, 0, 0, 0});   // hand-written against generated
  } else if (base->schedule == FS_SCHED_ROW && base->row_form == 3) {
    const fs::RowGenLaunch& rg = base->row_gen;
    const int all_rows = (int)(rg.rows < (1 << 22) ? rg.rows : (1 << 22));
    if (rg.streamed || rg.L > 64) {
      // long rows: the streamed template under three workgroup sizes (against the register
      // team, if that is the default)
      for (int wg : {256, 512, 1024}) cands.push_back(fs_plan_options{FS_MODE_STITCHED, wg, 0, all_rows});
    } else {
      // lanes per row around the default (templates that do not fit the row are skipped when
      // their plan fails), two workgroup sizes
      const int rpw = 64 / rg.L;
      for (int r : {rpw / 2, rpw * 2, rpw * 4, 64})
        if (r >= 1 && r <= 64 && r != rpw) cands.push_back(fs_plan_options{FS_MODE_STITCHED, 0, r, 0});
      for (int wg : {64, 128}) cands.push_back(fs_plan_options{FS_MODE_STITCHED, wg, 0, 0});
    }
  } else if (base->schedule == FS_SCHED_ROW) {
    for (int wg : {128, 256, 512, 1024}) cands.push_back(fs_plan_options{FS_MODE_STITCHED, wg, 0, 0});
    cands.push_back(fs_plan_options{FS_MODE_STITCHED_GENERATED, 0, 0, 0});
  } else if (base->schedule == FS_SCHED_ROW_COL) {
    // the hand-written kernel (where it matches the group) and the generated one, each under a few
    // workgroup sizes and grids
    for (int wg : {128, 192, 256, 512})
      for (int grid : {256, 512}) cands.push_back(fs_plan_options{FS_MODE_STITCHED, wg, 0, grid});
    cands.push_back(fs_plan_options{FS_MODE_STITCHED_GENERATED, 0, 0, 0});
    for (int wg : {128, 256, 512})
      for (int grid : {256, 512}) cands.push_back(fs_plan_options{FS_MODE_STITCHED_GENERATED, wg, 0, grid});
  } else if (base->schedule == FS_SCHED_ELEMENTWISE) {
    // the generated kernel under two workgroup sizes, and the interpreted form
    for (int wg : {128, 256}) cands.push_back(fs_plan_options{FS_MODE_STITCHED, wg, 0, 0});
    cands.push_back(fs_plan_options{FS_MODE_STITCHED_PREBUILT, 0, 0, 0});
  }
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    if (e0) (void)hipEventDestroy(e0);
    fs_destroy(base);
    return set_error(FS_ERR_HIP, "hipEventCreate failed");
  }
  std::set<std::string> seen;
  fs_plan* best_plan = nullptr;
  fs_plan_options best_opt = cands[0];
  double best_t = 0.0;
  std::string first_launch_error;
  fs_status launch_status = FS_OK;
  for (size_t i = 0; i < cands.size(); ++i) {
    fs_plan* p = nullptr;
    if (i == 0) p = base;
    else if (fs_plan_create(ops, n_ops, &cands[i], &p) != FS_OK) continue;   // template not generable: skip
    // identical geometry to a template already timed: skip
    if (!seen.insert(p->description).second) { fs_destroy(p); continue; }
    fs_status ls = FS_OK;
    for (int w = 0; w < 2 && ls == FS_OK; ++w) ls = fs_launch(p, inputs, n_in, outputs, n_out, hip_stream);
    bool ok = ls == FS_OK && hipEventRecord(e0, stream) == hipSuccess;
    for (int t = 0; t < trials && ok; ++t) ok = (ls = fs_launch(p, inputs, n_in, outputs, n_out, hip_stream)) == FS_OK;
    if (ok) ok = hipEventRecord(e1, stream) == hipSuccess && hipEventSynchronize(e1) == hipSuccess;
    float ms = 0.f;
    if (ok) ok = hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
    if (!ok) {
      if (launch_status == FS_OK) {
        launch_status = ls != FS_OK ? ls : FS_ERR_HIP;
        first_launch_error = ls != FS_OK ? g_error : std::string("HIP event call failed while timing");
      }
      fs_destroy(p);
      if (i == 0) break;   // the default template itself fails: argument error, report it
      continue;
    }
    const double us = 1e3 * ms / trials;
    if (!best_plan || us < best_t) {
      if (best_plan) fs_destroy(best_plan);
      best_plan = p; best_t = us; best_opt = cands[i];
    } else {
      fs_destroy(p);
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (!best_plan) return set_error(launch_status == FS_OK ? FS_ERR_HIP : launch_status,
                                   first_launch_error.empty() ? "no template could be launched" : first_launch_error);
  // leave the outputs written by the returned plan
  st = fs_launch(best_plan, inputs, n_in, outputs, n_out, hip_stream);
  if (st != FS_OK) { fs_destroy(best_plan); return st; }
  *out = best_plan;
  if (best) *best = best_opt;
  if (best_us) *best_us = best_t;
  {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    g_tune[group_key(ops, n_ops)] = TuneEntry{best_opt, best_t};
  }
  } catch (const std::bad_alloc&) {
    return set_error(FS_ERR_NOMEM, "out of host memory");
  } catch (...) {
    return set_error(FS_ERR_INVALID, "internal error while tuning");
  }
  return FS_OK;
}

fs_status fs_destroy(fs_plan* p) {
  if (!p) return FS_OK;
  fs_status st = FS_OK;
  if (p->workspace) {
    const hipError_t e = hipFree(p->workspace);
    if (e != hipSuccess) st = set_error(FS_ERR_HIP, std::string("hipFree: ") + hipGetErrorString(e));
  }
  fs::ew_stitch_release(p->ew);
  fs::row_gen_release(p->row_gen);
  fs::two_step_release(p->two_step);
  delete p;
  return st;
}

fs_status fs_plan_info(const fs_plan* p, int32_t* schedule, int32_t* n_kernels, int64_t* lds_bytes,
                       int64_t* workspace_bytes, int64_t* algorithmic_bytes, int64_t* moved_bytes) {
  if (!p) return set_error(FS_ERR_INVALID, "plan is NULL");
  if (schedule) *schedule = p->schedule;
  if (n_kernels) *n_kernels = p->n_kernels;
  if (lds_bytes) *lds_bytes = p->lds_bytes;
  if (workspace_bytes) *workspace_bytes = p->workspace_bytes;
  if (algorithmic_bytes) *algorithmic_bytes = p->graph.algorithmic_bytes();
  if (moved_bytes) *moved_bytes = p->moved_bytes;
  return FS_OK;
}

const char* fs_plan_describe(const fs_plan* p) { return p ? p->description.c_str() : ""; }

fs_status fs_shared_plan(const int32_t* operands, const int64_t* req_bytes, const uint8_t* is_output, int32_t n,
                         int64_t* offset, int32_t* shares_with, int64_t* total_bytes) {
  if (n < 0 || (n > 0 && (!operands || !req_bytes || !offset)) || !total_bytes)
    return set_error(FS_ERR_INVALID, "fs_shared_plan: NULL argument");
  try {
    fs::SharedPlanInput in;
    in.operands.resize(n);
    in.req_bytes.assign(req_bytes, req_bytes + n);
    if (is_output) in.is_output.assign(is_output, is_output + n);
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < 3; ++j) {
        const int o = operands[3 * i + j];
        if (o < 0) continue;
        if (o >= i) return set_error(FS_ERR_INVALID, "fs_shared_plan: operand index not smaller than the op's own");
        in.operands[i].push_back(o);
      }
    const fs::SharedPlanResult r = fs::shared_plan(in);
    for (int i = 0; i < n; ++i) {
      offset[i] = r.offset[i];
      if (shares_with) shares_with[i] = r.shares_with[i];
    }
    *total_bytes = r.total_bytes;
  } catch (...) {
    return set_error(FS_ERR_NOMEM, "out of host memory");
  }
  return FS_OK;
}

fs_status fs_fusion_create(const fs_op_desc* ops, int32_t n_ops, const fs_fusion_options* opt, fs_fusion** out) {
  if (!out) return set_error(FS_ERR_INVALID, "out is NULL");
  *out = nullptr;
  if (!ops || n_ops < 1) return set_error(FS_ERR_INVALID, "ops is NULL or empty");
  try {
    fs::FusionConfig cfg;
    if (opt) {
      if (opt->n_extra < 0 || (opt->n_extra > 0 && (!opt->extra_sizes || !opt->extra_ops))) return set_error(FS_ERR_INVALID, "extra patterns: NULL table");
      const int32_t* next = opt->extra_ops;
      for (int k = 0; k < opt->n_extra; ++k) {
        if (opt->extra_sizes[k] < 1) return set_error(FS_ERR_INVALID, "extra patterns: empty pattern");
        std::vector<int> pat(next, next + opt->extra_sizes[k]);
        next += opt->extra_sizes[k];
        for (int o : pat) if (o < 0 || o >= n_ops) return set_error(FS_ERR_INVALID, "extra patterns: op index out of range");
        cfg.extra_patterns.push_back(pat);
        if (opt->extra_scores) {
          const double sc = opt->extra_scores[k];
          if (std::isinf(sc) || std::fabs(sc) > 1e12) return set_error(FS_ERR_INVALID, "extra patterns: a measured score must be a finite number of microseconds (or NaN for none)");
          cfg.extra_scores.push_back(sc);
        }
      }
      if (opt->max_patterns < 0 || opt->max_patterns > 256) return set_error(FS_ERR_INVALID, "max_patterns out of range [0,256]");
      if (opt->n_bw < 0 || (opt->n_bw > 0 && (!opt->bw_bytes || !opt->bw_gbs))) return set_error(FS_ERR_INVALID, "bandwidth model: NULL table");
      if (opt->launch_us > 0) cfg.launch_us = opt->launch_us;
      if (opt->max_patterns > 0) cfg.max_patterns = opt->max_patterns;
      if (opt->explore_budget != 0) cfg.explore_budget = opt->explore_budget < 0 ? 0 : opt->explore_budget;
      if (opt->seed_bytes > 0) cfg.seed_bytes = opt->seed_bytes;
      for (int k = 0; k < opt->n_bw; ++k) {
        if (opt->bw_bytes[k] <= 0 || opt->bw_gbs[k] <= 0 || (k > 0 && opt->bw_bytes[k] <= opt->bw_bytes[k - 1]))
          return set_error(FS_ERR_INVALID, "bandwidth model: bytes must increase and rates be positive");
        cfg.bandwidth.push_back({opt->bw_bytes[k], opt->bw_gbs[k]});
      }
    }
    std::unique_ptr<fs_fusion> f(new fs_fusion);
    std::string err;
    const std::vector<fs_op_desc> list(ops, ops + n_ops);
    if (!fs::fusion_plan(list, cfg, &f->result, &err)) return set_error(FS_ERR_INVALID, err);
    *out = f.release();
  } catch (const std::bad_alloc&) {
    return set_error(FS_ERR_NOMEM, "out of host memory");
  } catch (...) {
    return set_error(FS_ERR_INVALID, "internal error while planning the fusion");
  }
  return FS_OK;
}

fs_status fs_fusion_destroy(fs_fusion* f) {
  delete f;
  return FS_OK;
}

fs_status fs_fusion_info(const fs_fusion* f, int32_t* n_groups, int32_t* n_patterns, double* total, int32_t* rounds) {
  if (!f) return set_error(FS_ERR_INVALID, "fusion is NULL");
  if (n_groups) *n_groups = (int32_t)f->result.groups.size();
  if (n_patterns) *n_patterns = (int32_t)f->result.patterns.size();
  if (total) *total = f->result.total_score;
  if (rounds) *rounds = f->result.solver_rounds;
  return FS_OK;
}

fs_status fs_fusion_group_size(const fs_fusion* f, int32_t g, int32_t* n_ops, int32_t* n_in, int32_t* n_out,
                               int32_t* n_members, double* score) {
  if (!f) return set_error(FS_ERR_INVALID, "fusion is NULL");
  if (g < 0 || g >= (int32_t)f->result.groups.size()) return set_error(FS_ERR_INVALID, "group index out of range");
  const fs::FusionGroup& gr = f->result.groups[g];
  if (n_ops) *n_ops = (int32_t)gr.list.size();
  if (n_in) *n_in = (int32_t)gr.input_of.size();
  if (n_out) *n_out = (int32_t)gr.output_of.size();
  if (n_members) *n_members = (int32_t)gr.ops.size();
  if (score) *score = gr.score;
  return FS_OK;
}

fs_status fs_fusion_group(const fs_fusion* f, int32_t g, fs_op_desc* ops, int32_t* input_of, int32_t* output_of,
                          int32_t* members) {
  if (!f) return set_error(FS_ERR_INVALID, "fusion is NULL");
  if (g < 0 || g >= (int32_t)f->result.groups.size()) return set_error(FS_ERR_INVALID, "group index out of range");
  const fs::FusionGroup& gr = f->result.groups[g];
  if (ops) for (size_t k = 0; k < gr.list.size(); ++k) ops[k] = gr.list[k];
  if (input_of) for (size_t k = 0; k < gr.input_of.size(); ++k) input_of[k] = gr.input_of[k];
  if (output_of) for (size_t k = 0; k < gr.output_of.size(); ++k) output_of[k] = gr.output_of[k];
  if (members) for (size_t k = 0; k < gr.ops.size(); ++k) members[k] = gr.ops[k];
  return FS_OK;
}

fs_status fs_fusion_pattern(const fs_fusion* f, int32_t k, int32_t* n_ops, int32_t* ops, int32_t cap, int32_t* origin,
                            int64_t* saved_bytes, double* score, int32_t* chosen) {
  if (!f) return set_error(FS_ERR_INVALID, "fusion is NULL");
  if (k < 0 || k >= (int32_t)f->result.patterns.size()) return set_error(FS_ERR_INVALID, "pattern index out of range");
  const fs::FusionPattern& p = f->result.patterns[k];
  if (n_ops) *n_ops = (int32_t)p.ops.size();
  if (ops) for (int32_t j = 0; j < cap && j < (int32_t)p.ops.size(); ++j) ops[j] = p.ops[j];
  if (origin) *origin = p.origin;
  if (saved_bytes) *saved_bytes = p.saved_bytes;
  if (score) *score = p.score;
  if (chosen) *chosen = p.chosen ? 1 : 0;
  return FS_OK;
}

fs_status fs_fusion_pattern_group_size(const fs_fusion* f, int32_t k, int32_t* n_ops, int32_t* n_in, int32_t* n_out,
                                       int32_t* measured) {
  if (!f) return set_error(FS_ERR_INVALID, "fusion is NULL");
  if (k < 0 || k >= (int32_t)f->result.patterns.size()) return set_error(FS_ERR_INVALID, "pattern index out of range");
  const fs::FusionPattern& p = f->result.patterns[k];
  if (n_ops) *n_ops = (int32_t)p.list.size();
  if (n_in) *n_in = (int32_t)p.input_of.size();
  if (n_out) *n_out = (int32_t)p.output_of.size();
  if (measured) *measured = p.measured ? 1 : 0;
  return FS_OK;
}

fs_status fs_fusion_pattern_group(const fs_fusion* f, int32_t k, fs_op_desc* ops, int32_t* input_of, int32_t* output_of) {
  if (!f) return set_error(FS_ERR_INVALID, "fusion is NULL");
  if (k < 0 || k >= (int32_t)f->result.patterns.size()) return set_error(FS_ERR_INVALID, "pattern index out of range");
  const fs::FusionPattern& p = f->result.patterns[k];
  if (ops) for (size_t j = 0; j < p.list.size(); ++j) ops[j] = p.list[j];
  if (input_of) for (size_t j = 0; j < p.input_of.size(); ++j) input_of[j] = p.input_of[j];
  if (output_of) for (size_t j = 0; j < p.output_of.size(); ++j) output_of[j] = p.output_of[j];
  return FS_OK;
}

fs_status fs_stream_copy(void* dst, const void* src, int64_t bytes, void* hip_stream) {
  if (bytes < 0 || (bytes & 15)) return set_error(FS_ERR_INVALID, "bytes must be a non-negative multiple of 16");
  if (bytes == 0) return FS_OK;
  if (!dst || !src || (reinterpret_cast<uintptr_t>(dst) & 15) || (reinterpret_cast<uintptr_t>(src) & 15))
    return set_error(FS_ERR_INVALID, "pointer is NULL or not 16-byte aligned");
  std::string err;
  if (fs::stream_copy_launch(dst, src, bytes, hip_stream, &err) != 0) return set_error(FS_ERR_HIP, err);
  return FS_OK;
}

}  // extern "C"

// Groups in which values reduced over whole tensors feed ops on whole tensors, as two generated kernels.
#pragma once
#include <string>
#include <vector>

#include "ew_ir.h"
#include "graph.h"

namespace fs {

struct TwoStepLaunch {
  int n_reduce = 0, n_scalar_ops = 0, parts = 0;
  int64_t n_partials = 0;                 // doubles handed from the first kernel to the second
  int grid[2] = {0, 0}, wg = 256;
  int64_t lds_bytes = 0;
  std::vector<int> view_param[2];         // per kernel: the parameter behind each entry of Args::in
  std::vector<char> code_object;          // holds both kernels
  std::string kernel_name[2];
  EwModule loaded[2];
};

bool two_step_plan(const Graph& g, TwoStepLaunch* out, std::string* err);
std::string two_step_describe(const TwoStepLaunch&);
// `partials`: n_partials doubles, written by the first kernel and read by the second
int two_step_launch(TwoStepLaunch&, const void* const* in, void* const* out, int n_out, void* partials, void* stream, std::string* err);
void two_step_release(TwoStepLaunch&);

}  // namespace fs

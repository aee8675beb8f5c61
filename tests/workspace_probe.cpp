// Stands in for the Linear Relation launches of librelation.so, on the CPU:
// notes which bytes of the workspace the kernels would use, from the arguments
// that the C-ABI layer hands to the launch. The extents are those of the arrays
// as linear.hip and linear_bf16.hip index them.
#include "kernels.h"

#include <algorithm>
#include <cstdint>
#include <vector>

namespace {

struct Span {
  uintptr_t begin, end;
};
std::vector<Span> spans;
bool bf16_kernels;

void add(const void* p, size_t bytes) {
  if (bytes) spans.push_back({(uintptr_t)p, (uintptr_t)p + bytes});
}

void add_linear(const rel::LinearArgs& a, bool backward) {
  const size_t N = (size_t)a.B * a.H, nc = (size_t)a.nchunks, ns = (size_t)a.nseg, D = (size_t)a.D, T = (size_t)a.T;
  bf16_kernels = a.seg > 0;
  if (a.seg) {
    const size_t segments = ns > 1 ? N * ns : 0;
    if (a.seg > 1) add(a.cprev, N * nc * D * D * 4);
    add(a.segc, segments * D * D * 4);
    add(a.segg, segments * D * 4);
    if (ns > 1) add(a.gpre, N * nc * D * 4);
    if (backward) {
      if (a.seg > 1) add(a.gout, N * nc * D * D * 4);
      add(a.segp, segments * D * D * 4);
      if (ns > 1) add(a.gsuf, N * nc * D * 4);
      if (D >= 64) add(a.qn, N * T * D * 4);
    }
    if (a.rope_half) add(a.rope, (nc + 64) * (size_t)((2 * a.rope_half + 7) / 8 * 8) * 8);
  } else {
    const size_t NV = a.split ? 4 * N : N, W = a.split ? D / 2 : D;
    add(a.dstate, NV * nc * W * W * 4);
    add(a.gamma, NV * nc * W * 4);
    add(a.cprev, NV * nc * W * W * 4);
    add(a.segc, NV * ns * W * W * 4);
    add(a.segg, NV * ns * W * 4);
    if (backward) {
      add(a.pstate, NV * nc * W * W * 4);
      add(a.gout, NV * nc * W * W * 4);
      add(a.segp, NV * ns * W * W * 4);
    }
    if (a.split) {
      add(a.qn, N * T * D * 4);
      add(a.kn, N * T * D * 4);
      add(a.part, 8 * N * T * D * 4);
    }
    if (a.rope_half) add(a.rope, (nc + 64) * (size_t)a.rope_half * 8);
  }
  if (backward && a.a_log) add(a.gpart, N * nc * 2 * D * 4);
}

}  // namespace

namespace rel {

hipError_t launch_linear_fwd(const LinearArgs& a, int, hipStream_t) {
  add_linear(a, false);
  return hipSuccess;
}
hipError_t launch_linear_bwd(const LinearArgs& a, int, hipStream_t) {
  add_linear(a, true);
  return hipSuccess;
}
hipError_t launch_linear_rope_table(float2*, int, int, double, hipStream_t) { return hipSuccess; }
hipError_t launch_linear_bf16_rope_table(float2*, int, int, double, hipStream_t) { return hipSuccess; }

}  // namespace rel

extern "C" {

// Bytes from `workspace` to the end of the last array noted since the last
// call; -1 where one starts before it, -2 where two overlap.
int64_t probe_used(uintptr_t workspace) {
  std::vector<Span> s;
  s.swap(spans);
  std::sort(s.begin(), s.end(), [](const Span& x, const Span& y) { return x.begin < y.begin; });
  uintptr_t end = workspace;
  for (const Span& x : s) {
    if (x.begin < workspace) return -1;
    if (x.begin < end) return -2;
    end = x.end;
  }
  return (int64_t)(end - workspace);
}
int probe_bf16_kernels() { return bf16_kernels; }
}

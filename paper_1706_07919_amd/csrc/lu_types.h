// Matrix tables and complex helpers shared by the LU kernels' translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "common.h"

namespace bem {
namespace lud {

// Pointers into the matrices are qualified with the global address space so
// that loads and stores compile to global (not flat) memory instructions: flat
// accesses also count against the LDS wait counter and would make every LDS
// wait in the GEMM loop wait for the global prefetch as well.  (The qualifier
// only exists in the device pass; the host pass sees plain pointers.)
#if defined(__HIP_DEVICE_COMPILE__)
#define GLOBAL __attribute__((address_space(1)))
#define LDS_AS __attribute__((address_space(3)))
#else
#define GLOBAL
#define LDS_AS
#endif

template <typename R> struct Cx;
template <> struct Cx<float> { using T = float2; };
template <> struct Cx<double> { using T = double2; };

template <typename C> __device__ inline C cmk(decltype(C::x) a, decltype(C::x) b) {
  C c; c.x = a; c.y = b; return c;
}
template <typename C> __device__ inline C cmul(C a, C b) {
  return cmk<C>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
template <typename C> __device__ inline C csub(C a, C b) { return cmk<C>(a.x - b.x, a.y - b.y); }
// s + a b as four fused multiply-adds
template <typename C> __device__ inline C cfma(C s, C a, C b) {
  return cmk<C>(fma(a.x, b.x, fma(-a.y, b.y, s.x)), fma(a.x, b.y, fma(a.y, b.x, s.y)));
}
template <typename C> __device__ inline C crecip(C a) {
  // 1/a with scaling to avoid overflow (Smith's method)
  using R = decltype(C::x);
  if (fabs(a.x) >= fabs(a.y)) {
    R t = a.y / a.x, d = a.x + a.y * t;
    return cmk<C>(R(1) / d, -t / d);
  } else {
    R t = a.x / a.y, d = a.y + a.x * t;
    return cmk<C>(t / d, R(-1) / d);
  }
}

// ============================================================== matrix groups
// The matrices of one launch come in up to kMaxGroups size classes (uneven
// batches: bodies of different node counts, each with many wavenumbers).  The
// table travels by value in the kernel arguments; the flattened matrix index
// of a workgroup selects its group, and every range is clipped to the group's
// own n, so one recursion over the largest n factors every matrix.
constexpr int kMaxGroups = 8;
struct LuGroup {
  void* A;          // matrix 0 of the group (row-major, element type of the launch)
  int32_t* piv;     // [count][n]
  int32_t* info;    // [count]
  int64_t ld;       // leading dimension (elements)
  int64_t stride;   // elements between consecutive matrices
  int n;
  int count;
};
struct LuGroups {
  LuGroup g[kMaxGroups];
  int ng;
};

// q: flattened matrix index -> its group (copied out) and index li inside it.
// Both loops run over constant indices and copy field by field, so the table
// is read with uniform loads from the kernel arguments (a dynamic index or a
// whole-struct copy would place the table in scratch memory).
__device__ inline bool locate(const LuGroups& G, int q, LuGroup& out, int& li) {
  int sel = -1;
#pragma unroll
  for (int i = 0; i < kMaxGroups; ++i) {
    if (sel < 0 && i < G.ng) {
      if (q < G.g[i].count) { sel = i; li = q; }
      else q -= G.g[i].count;
    }
  }
  if (sel < 0) return false;
#pragma unroll
  for (int i = 0; i < kMaxGroups; ++i)
    if (i == sel) {
      out.A = G.g[i].A;
      out.piv = G.g[i].piv;
      out.info = G.g[i].info;
      out.ld = G.g[i].ld;
      out.stride = G.g[i].stride;
      out.n = G.g[i].n;
      out.count = G.g[i].count;
    }
  return true;
}

// matrix b of a group, as a global pointer
template <typename C> __device__ inline GLOBAL C* gmat(const LuGroup& g, int b) {
  return (GLOBAL C*)g.A + (int64_t)b * g.stride;
}

// Panels of a factorisation with `rows` rows left: their width, and the launch
// over `total` matrices factoring w columns from c0 on.
constexpr int kPanelRows = 12 * 1024;
int panel_width(bem_prec prec, int rows);
void launch_panel(bem_ctx* ctx, bem_prec prec, const LuGroups& G, int total, int rows, int c0, int w);

}  // namespace lud
}  // namespace bem

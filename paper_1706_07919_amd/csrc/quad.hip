// Quadratic-element discretisation of the non-singular boundary integral
// equation (Sec. III: quadratic interpolants within each element, integrals
// free of singularities evaluated by standard Gauss quadrature; Sec. IV A:
// 500 six-node elements and 1002 nodes on the sphere), collocated at the
// nodes:
//   4 pi phi_i + int [psi - phi_i g' - psi_i f'] G dS = int [phi - phi_i g - psi_i f] H dS
// with phi, psi and the geometry interpolated by the six shape functions of
// each element (nodes v0 v1 v2 m01 m12 m20; L_a (2 L_a - 1) at the vertices,
// 4 L_a L_b at the midpoints), f, g of Appendix A about x_i with its normal,
// and H = dG/dn with the element's normal at the quadrature point.  The
// integrands are regular at x_i, so every element takes the same rule: the
// symmetric 7-point rule of degree 5 on triangles (Radon's).  Collecting terms:
//   (M_psi)_ij =  sum_{e,q : node a of e is j} N_a(q) wJ_q G_q
//   (M_phi)_ij = -sum ...                      N_a(q) wJ_q H_q
//   (M_phi)_ii += 4 pi - sum_{all q} (g'_q G_q - g_q H_q) wJ_q
//   (M_psi)_ii += -sum_{all q} (f'_q G_q - f_q H_q) wJ_q
// All in float64.  Column j of A is column j of M_phi (hard node) or M_psi
// (soft node), b = -B y.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "phase.h"
#include "reduce.h"

namespace bem {

namespace {

constexpr int kQ = 7;          // points of the triangle rule
constexpr int kMaxInc = 12;    // element incidences kept per node
constexpr int kQT = 256;       // threads of the row kernels
constexpr int kRhsChunk = 2;   // most right-hand sides per assembly launch
constexpr int kRhsWide = 4;    // and of a row that goes one wavenumber at a time
constexpr int kKc = 8;         // wavenumbers per assembly workgroup
constexpr double kFourPiQ = 12.566370614359172953850573533118;

// Barycentric coordinates (L0, L1, L2) of the rule's points and the six shape
// functions there.
struct Shapes {
  double L[kQ][3], N[kQ][6];
};
constexpr double kS15 = 3.872983346207417;   // sqrt(15)
constexpr Shapes make_shapes() {
  Shapes S{};
  const double as[2] = {(6.0 - kS15) / 21.0, (6.0 + kS15) / 21.0};
  for (int q = 0; q < kQ; ++q) {
    for (int c = 0; c < 3; ++c) {
      const double a = q ? as[(q - 1) / 3] : 1.0 / 3.0;
      S.L[q][c] = q && (q - 1) % 3 == c ? 1.0 - 2.0 * a : a;
    }
    const double L0 = S.L[q][0], L1 = S.L[q][1], L2 = S.L[q][2];
    const double N[6] = {L0 * (2 * L0 - 1), L1 * (2 * L1 - 1), L2 * (2 * L2 - 1), 4 * L0 * L1, 4 * L1 * L2, 4 * L2 * L0};
    for (int a = 0; a < 6; ++a) S.N[q][a] = N[a];
  }
  return S;
}
// for the kernels that index them per thread
__device__ __constant__ Shapes kShapes = make_shapes();

// The rule's weights (summing to the reference area 1/2) and the shape functions with
// their derivatives at the points.
struct QuadRule {
  double N[kQ][6], dxi[kQ][6], deta[kQ][6], w[kQ];
};

QuadRule make_rule() {
  constexpr Shapes S = make_shapes();
  QuadRule R;
  for (int q = 0; q < kQ; ++q) {
    R.w[q] = 0.5 * (q == 0 ? 9.0 / 40.0 : (q < 4 ? 155.0 - kS15 : 155.0 + kS15) / 1200.0);
    // barycentric L1 = xi, L2 = eta
    const double L0 = S.L[q][0], L1 = S.L[q][1], L2 = S.L[q][2];
    // d/dxi: dL0 = -1, dL1 = +1; d/deta: dL0 = -1, dL2 = +1
    const double dx[6] = {-(4 * L0 - 1), 4 * L1 - 1, 0.0, 4 * (L0 - L1), 4 * L2, -4 * L2};
    const double de[6] = {-(4 * L0 - 1), 0.0, 4 * L2 - 1, -4 * L1, 4 * L1, 4 * (L0 - L2)};
    for (int a = 0; a < 6; ++a) {
      R.N[q][a] = S.N[q][a];
      R.dxi[q][a] = dx[a];
      R.deta[q][a] = de[a];
    }
  }
  return R;
}

// quadrature points of every element: [F*7][8] = x, y, z, nx, ny, nz (unit
// normal of the element surface), wJ (weight times area Jacobian), 0
__global__ void quad_points_kernel(int F, const double* __restrict__ x,
                                   const int32_t* __restrict__ elem, QuadRule R,
                                   double* __restrict__ qp) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= F * kQ) return;
  const int e = t / kQ, q = t % kQ;
  double p[3] = {0, 0, 0}, t1[3] = {0, 0, 0}, t2[3] = {0, 0, 0};
  for (int a = 0; a < 6; ++a) {
    const int v = elem[6 * e + a];
    for (int d = 0; d < 3; ++d) {
      const double c = x[3 * v + d];
      p[d] += R.N[q][a] * c;
      t1[d] += R.dxi[q][a] * c;
      t2[d] += R.deta[q][a] * c;
    }
  }
  const double c0 = t1[1] * t2[2] - t1[2] * t2[1];
  const double c1 = t1[2] * t2[0] - t1[0] * t2[2];
  const double c2 = t1[0] * t2[1] - t1[1] * t2[0];
  const double J = sqrt(c0 * c0 + c1 * c1 + c2 * c2);
  double* o = qp + 8 * (int64_t)t;
  o[0] = p[0];
  o[1] = p[1];
  o[2] = p[2];
  o[3] = c0 / J;
  o[4] = c1 / J;
  o[5] = c2 / J;
  o[6] = R.w[q] * J;
  o[7] = 0.0;
}

// inc[j][c] = 6 e + a for the c-th (element e, local node a) holding node j,
// in element order; -1 past the last; *overflow set when a node has more
// than kMaxInc incidences or an element refers to a node outside [0, n).  One
// wave per node scans the table 64 entries at a time (a thread per node took
// 0.23 ms for 1002 nodes; 0.01 ms).
__global__ __launch_bounds__(256) void quad_incidence_kernel(int n, int F,
                                                             const int32_t* __restrict__ elem,
                                                             int32_t* __restrict__ inc,
                                                             int32_t* __restrict__ overflow) {
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (j >= n) return;   // the whole wave
  int c = 0;
  bool bad = false;
  for (int t0 = 0; t0 < 6 * F; t0 += 64) {
    const int t = t0 + lane;
    const int v = t < 6 * F ? elem[t] : -1;
    bad |= t < 6 * F && (v < 0 || v >= n);
    const unsigned long long hit = __ballot(v == j && t < 6 * F);
    const int at = c + __popcll(hit & ((1ull << lane) - 1));
    if (((hit >> lane) & 1) && at < kMaxInc) inc[(int64_t)j * kMaxInc + at] = t;
    c += __popcll(hit);
  }
  if ((j == 0 && bad) || c > kMaxInc) overflow[0] = 1;
  if (lane >= c && lane < kMaxInc) inc[(int64_t)j * kMaxInc + lane] = -1;
}

__device__ inline double block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  for (int w = 0; w < kQT / 64; ++w) s += sh[w];
  return s;
}

// One workgroup per (row i, chunk of kKc wavenumbers): the row's diagonal
// integrals over every quadrature point, then each column's entries gathered
// from the elements that hold its node (deterministic order, no atomics).
//
// Bound by float64 instructions: 7 x (incidences of the column) kernel values
// per entry.  The pair's geometry and phases are formed once for the chunk and
// e^{ikr} / r advanced by rotation along its wavenumbers (four multiply-adds), so
// a value costs about 11 instructions and a twelfth of a sincos; a workgroup per
// wavenumber with a library sincos, square root and division per value took
// 10.1 ms for 63 wavenumbers on 1002 nodes, this form 2.2 ms (2.0 without the
// roundings that EvenChunk keeps).  A partial chunk is continued evenly (nothing
// stored past its end).  Uneven wavenumbers, or a phase past the 2^20 rad of phase.h's
// reduction, go one wavenumber at a time; their values cost the most, so a row then
// takes up to kRhsWide right-hand sides, those of the next launch among them (24
// uneven wavenumbers with four of them: 3.3 ms, with two a launch 6.5).
struct QuadRow {
  int n, npts, i, kq0, kc, n_rhs, r0, nr;
  const double *x, *nrm, *qp;
  const uint8_t* bc;
  const int32_t* inc;
  const double2* y;
};

struct QuadPair {
  double r, c, wr;   // |d|, (d.n_q) / r^2, 1 / r
  double dx, dy, dz;
};
__device__ __forceinline__ QuadPair quad_pair(const double* o, double x0, double x1, double x2) {
  QuadPair g;
  g.dx = o[0] - x0;
  g.dy = o[1] - x1;
  g.dz = o[2] - x2;
  dist_and_inverse64(g.dx * g.dx + g.dy * g.dy + g.dz * g.dz, g.r, g.wr);
  g.c = (g.dx * o[3] + g.dy * o[4] + g.dz * o[5]) * (g.wr * g.wr);
  return g;
}
template <bool NEAR>
__device__ __forceinline__ double2 quad_phase(double k, double t) {
  if (NEAR) return unit_phase(k, t);
  double s, c;
  phase_sincos(k * t, &s, &c);
  return make_double2(c, s);
}

// The row for the KC wavenumbers of kc (p.kq0 the first's index): A, b, diag64.
// red: LDS; NR: at least p.nr.  False (nothing stored) if a phase is too wide for the
// NEAR form.
template <int KC, bool NEAR, int NR, int COMPS, typename OUT>
__device__ __forceinline__ bool quad_row(const QuadRow& p, const EvenChunk<KC>& kc, OUT* __restrict__ A, int64_t ld,
                                         int64_t a_stride, double2* __restrict__ b,
                                         double2* __restrict__ diag64,
                                         double (&red)[kQT / 64][COMPS][8]) {
  static_assert(COMPS >= 2 * NR + 4, "the row's sums");
  const int i = p.i, lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const double x0 = p.x[3 * i], x1 = p.x[3 * i + 1], x2 = p.x[3 * i + 2];
  const double n0 = p.nrm[3 * i], n1 = p.nrm[3 * i + 1], n2 = p.nrm[3 * i + 2];
  bool wide = false;
  // workgroup sums of component c of the chunk into red[.][c][q]
  auto reduce = [&](int c, const double (&v)[KC]) {
    double v8[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v8[q] = q < KC ? v[q < KC ? q : 0] : 0.0;
    const double s = wave_reduce8(v8);
    if ((lane & 7) == 0) red[wid][c][lane >> 3] = s;
  };
  auto total = [&](int c, int q) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kQT / 64; ++w) s += red[w][c][q];
    return s;
  };
  {
    // diagonal integrals: d1 = sum wJ (g' G - g H), d2 k = sum wJ k (f' G - f H)
    double d[4][KC];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int q = 0; q < KC; ++q) d[c][q] = 0.0;
    for (int t = threadIdx.x; t < p.npts; t += kQT) {
      const double* o = p.qp + 8 * (int64_t)t;
      const QuadPair g = quad_pair(o, x0, x1, x2);
      const double s0 = n0 * g.dx + n1 * g.dy + n2 * g.dz;
      const double nn = n0 * o[3] + n1 * o[4] + n2 * o[5], wr = o[6] * g.wr;
      if (NEAR) wide |= !(kc.kmax * fmax(g.r, fabs(s0)) < kPhaseNear);
      const double2 E = quad_phase<NEAR>(kc.k[kc.kMid], g.r), F0 = quad_phase<NEAR>(kc.k[kc.kMid], s0);
      const double2 G0 = make_double2(wr * E.x, wr * E.y);
      double2 F = F0, G = G0, dE, dF;
      if (KC > 1) {
        dE = quad_phase<NEAR>(kc.dk, g.r);
        dF = quad_phase<NEAR>(kc.dk, s0);
      }
#pragma unroll
      for (int i = 0; i < KC; ++i) {
        const int q = kc.order(i);
        if (i > 0) {
          G = kc.advance(i, i == kc.kUp ? G0 : G, dE, g.r);
          F = kc.advance(i, i == kc.kUp ? F0 : F, dF, s0);
        }
        const double k = kc.k[q], ckr = k * (g.c * g.r), kn = k * nn;
        const double2 H = make_double2(fma(-g.c, G.x, -ckr * G.y), fma(ckr, G.x, -g.c * G.y));
        const double gp = -kn * F.y, fp = kn * F.x;
        d[0][q] += fma(gp, G.x, -F.x * H.x);
        d[1][q] += fma(gp, G.y, -F.x * H.y);
        d[2][q] += fma(fp, G.x, -F.y * H.x);
        d[3][q] += fma(fp, G.y, -F.y * H.y);
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) reduce(2 * NR + c, d[c]);
  }
  if (__syncthreads_or(wide)) return false;
  double bac[2 * NR][KC];
#pragma unroll
  for (int c = 0; c < 2 * NR; ++c)
#pragma unroll
    for (int q = 0; q < KC; ++q) bac[c][q] = 0.0;
  for (int j = threadIdx.x; j < p.n; j += kQT) {
    double2 mp[KC], mh[KC];   // M_psi and M_phi entries
#pragma unroll
    for (int q = 0; q < KC; ++q) mp[q] = mh[q] = make_double2(0.0, 0.0);
    for (int c = 0; c < kMaxInc; ++c) {
      const int v = p.inc[(int64_t)j * kMaxInc + c];
      if (v < 0) break;
      const int e = v / 6, a = v % 6;
      for (int t = 0; t < kQ; ++t) {
        const double* o = p.qp + 8 * ((int64_t)e * kQ + t);
        const QuadPair g = quad_pair(o, x0, x1, x2);
        const double wr = o[6] * g.wr * kShapes.N[t][a], cr = g.c * g.r;
        const double2 E = quad_phase<NEAR>(kc.k[kc.kMid], g.r);
        const double2 G0 = make_double2(wr * E.x, wr * E.y);
        double2 G = G0, dE;
        if (KC > 1) dE = quad_phase<NEAR>(kc.dk, g.r);
#pragma unroll
        for (int i = 0; i < KC; ++i) {
          const int q = kc.order(i);
          if (i > 0) G = kc.advance(i, i == kc.kUp ? G0 : G, dE, g.r);
          const double ckr = kc.k[q] * cr;
          mp[q].x += G.x;
          mp[q].y += G.y;
          mh[q].x = fma(g.c, G.x, fma(ckr, G.y, mh[q].x));
          mh[q].y = fma(g.c, G.y, fma(-ckr, G.x, mh[q].y));
        }
      }
    }
    const bool hard = p.bc[j] == BEM_BC_HARD;
#pragma unroll
    for (int q = 0; q < KC; ++q) {
      if (q >= p.kc) break;   // uniform
      const int64_t kq = p.kq0 + q;
      if (j == i) {
        const double ki = 1.0 / kc.k[q];
        mh[q].x += kFourPiQ - total(2 * NR, q);
        mh[q].y -= total(2 * NR + 1, q);
        mp[q].x -= total(2 * NR + 2, q) * ki;
        mp[q].y -= total(2 * NR + 3, q) * ki;
        if (p.r0 == 0 && diag64) {
          diag64[2 * (kq * p.n + i)] = mh[q];
          diag64[2 * (kq * p.n + i) + 1] = mp[q];
        }
      }
      const double2 u = hard ? mh[q] : mp[q], v = hard ? mp[q] : mh[q];
      if (p.r0 == 0 && A) {
        OUT* Ap = A + kq * a_stride + (int64_t)i * ld + j;
        Ap->x = u.x;
        Ap->y = u.y;
      }
#pragma unroll
      for (int r = 0; r < NR; ++r)
        if (r < p.nr) {
          const double2 yv = p.y[(kq * p.n_rhs + p.r0 + r) * p.n + j];
          bac[2 * r][q] -= v.x * yv.x - v.y * yv.y;
          bac[2 * r + 1][q] -= v.x * yv.y + v.y * yv.x;
        }
    }
  }
#pragma unroll
  for (int c = 0; c < 2 * NR; ++c)
    if (c < 2 * p.nr) reduce(c, bac[c]);
  __syncthreads();
  const int q = threadIdx.x & 7, r = threadIdx.x >> 3;
  if (r < p.nr && q < p.kc && q < KC)
    b[((int64_t)(p.kq0 + q) * p.n_rhs + p.r0 + r) * p.n + i] =
        make_double2(total(2 * r, q), total(2 * r + 1, q));
  __syncthreads();   // red is free again
  return true;
}

template <typename OUT, int NR>
__global__ __launch_bounds__(kQT, 2) void quad_assemble_kernel(
    int n, const double* __restrict__ x, const double* __restrict__ nrm,
    const uint8_t* __restrict__ bc, int npts, const double* __restrict__ qp,
    const int32_t* __restrict__ inc, const double* __restrict__ kv, int n_k, int n_rhs, int r0,
    int nr, const double2* __restrict__ y, OUT* __restrict__ A, int64_t ld, int64_t a_stride,
    double2* __restrict__ b, double2* __restrict__ diag64) {
  constexpr int NW = NR == 1 ? 1 : kRhsWide;
  static_assert(kRhsWide % kRhsChunk == 0, "whole launches per wide row");
  __shared__ double red[kQT / 64][2 * NW + 4][8];
  const int q0 = blockIdx.y * kKc, kc = min(kKc, n_k - q0);
  QuadRow p{n, npts, (int)blockIdx.x, q0, kc, n_rhs, r0, nr, x, nrm, qp, bc, inc, y};
  EvenChunk<kKc> chunk;
  chunk.load(kv + q0, kc);
  if (chunk.even && quad_row<kKc, true, NR>(p, chunk, A, ld, a_stride, b, diag64, red)) return;
  if (r0 % kRhsWide) return;   // (uniform) its right-hand sides are an earlier launch's
  p.kc = 1;
  p.nr = min(NW, n_rhs - r0);
  for (int q = 0; q < kc; ++q) {
    p.kq0 = q0 + q;
    EvenChunk<1> one;
    one.load(kv + p.kq0, 1);
    (void)quad_row<1, false, NW>(p, one, A, ld, a_stride, b, diag64, red);
  }
}

// r = b - A x for the stored float64 operator: one workgroup per (row, vector)
__global__ __launch_bounds__(kQT) void quad_residual_kernel(int n, const double2* __restrict__ A,
                                                            int64_t ld, int64_t stride, int nr,
                                                            const double2* __restrict__ b,
                                                            const double2* __restrict__ xv,
                                                            double2* __restrict__ r) {
  __shared__ double sh[kQT / 64];
  const int i = blockIdx.x, q = blockIdx.y, kq = q / nr;
  const double2* Ar = A + kq * stride + (int64_t)i * ld;
  const double2* xq = xv + (int64_t)q * n;
  double sr = 0, si = 0;
  for (int j = threadIdx.x; j < n; j += kQT) {
    const double2 a = Ar[j], v = xq[j];
    sr += a.x * v.x - a.y * v.y;
    si += a.x * v.y + a.y * v.x;
  }
  sr = block_sum(sr, sh);
  si = block_sum(si, sh);
  if (threadIdx.x == 0) {
    const double2 bb = b[(int64_t)q * n + i];
    r[(int64_t)q * n + i] = make_double2(bb.x - sr, bb.y - si);
  }
}

// surface data at the quadrature points: out[v][p] = sum_a N_a(q) data[v][node a of e]
__global__ void quad_interp_kernel(int n, int F, int nvec, const int32_t* __restrict__ elem,
                                   QuadRule R, const double2* __restrict__ data,
                                   double2* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t npts = (int64_t)F * kQ;
  if (t >= npts * nvec) return;
  const int v = (int)(t / npts);
  const int p = (int)(t % npts), e = p / kQ, q = p % kQ;
  double sr = 0, si = 0;
  for (int a = 0; a < 6; ++a) {
    const double2 d = data[(int64_t)v * n + elem[6 * e + a]];
    sr += R.N[q][a] * d.x;
    si += R.N[q][a] * d.y;
  }
  out[t] = make_double2(sr, si);
}

}  // namespace

size_t quad_setup_bytes(int n, int F) {
  return ((size_t)F * kQ * 8 * 8 + 255) / 256 * 256 + ((size_t)n * kMaxInc * 4 + 255) / 256 * 256 + 256;
}

// Quadrature points and node incidences of the surface into ws (at least
// quad_setup_bytes); *qp and *inc point into it.  Synchronises the stream (the
// incidence check is read back).
bem_status quad_setup(bem_ctx* ctx, const bem_quad_surface* s, void* ws, double** qp,
                      int32_t** inc) {
  char* p = (char*)ws;
  *qp = (double*)p;
  p += ((size_t)s->n_elem * kQ * 8 * 8 + 255) / 256 * 256;
  *inc = (int32_t*)p;
  p += ((size_t)s->n * kMaxInc * 4 + 255) / 256 * 256;
  int32_t* flag = (int32_t*)p;
  const QuadRule R = make_rule();
  bem_status st = fill_zero(ctx, flag, 4);
  if (st != BEM_OK) return st;
  const int npts = s->n_elem * kQ;
  hipLaunchKernelGGL(quad_points_kernel, dim3((npts + 255) / 256), dim3(256), 0, ctx->stream,
                     s->n_elem, s->x, s->elem, R, *qp);
  hipLaunchKernelGGL(quad_incidence_kernel, dim3((s->n + 3) / 4), dim3(256), 0, ctx->stream,
                     s->n, s->n_elem, s->elem, *inc, flag);
  BEM_CHECK_LAUNCH(ctx);
  int32_t hflag = 0;
  BEM_HIP_TRY(ctx, hipMemcpyAsync(&hflag, flag, 4, hipMemcpyDeviceToHost, ctx->stream));
  BEM_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  if (hflag)
    return fail(ctx, BEM_EINVAL,
                "quadratic surface: an element refers to a node outside [0, n) or a node belongs "
                "to more than %d elements",
                kMaxInc);
  return BEM_OK;
}

bem_status launch_quad_assemble(bem_ctx* ctx, const bem_quad_surface* s, const double* qp,
                                const int32_t* inc, int n_k, const double* k, int n_rhs,
                                const void* y, bem_prec prec, void* A, int64_t ld,
                                int64_t a_stride, void* b, void* diag64) {
  const int npts = s->n_elem * kQ;
  const int pi = prof_begin(ctx, "assemble_quad");
  for (int r0 = 0; r0 < n_rhs; r0 += kRhsChunk) {
    const int nr = std::min(kRhsChunk, n_rhs - r0);
    dim3 grid(s->n, (n_k + kKc - 1) / kKc);
#define BEM_QUAD_ASSEMBLE(OUT, NR)                                                                \
  hipLaunchKernelGGL((quad_assemble_kernel<OUT, NR>), grid, dim3(kQT), 0, ctx->stream, s->n, s->x, \
                     s->nrm, s->bc, npts, qp, inc, k, n_k, n_rhs, r0, nr, (const double2*)y,      \
                     (OUT*)A, ld, a_stride, (double2*)b, (double2*)diag64)
    // (one right-hand side's accumulators leave the registers for the phases)
    if (prec == BEM_C128 && nr == 1) BEM_QUAD_ASSEMBLE(double2, 1);
    else if (prec == BEM_C128) BEM_QUAD_ASSEMBLE(double2, kRhsChunk);
    else if (nr == 1) BEM_QUAD_ASSEMBLE(float2, 1);
    else BEM_QUAD_ASSEMBLE(float2, kRhsChunk);
#undef BEM_QUAD_ASSEMBLE
    BEM_CHECK_LAUNCH(ctx);
  }
  // node-pair work: every (row, quadrature point) kernel value once for the
  // diagonal integrals plus once per element node holding the column
  prof_end(ctx, "assemble_quad", pi, (double)s->n * n_k * (npts + 6.0 * npts), 0.0);
  return BEM_OK;
}

bem_status launch_quad_residual(bem_ctx* ctx, int n, const void* A64, int64_t ld, int64_t stride,
                                int n_k, int n_rhs, const void* b, const void* x, void* r) {
  hipLaunchKernelGGL(quad_residual_kernel, dim3(n, n_k * n_rhs), dim3(kQT), 0, ctx->stream, n,
                     (const double2*)A64, ld, stride, n_rhs, (const double2*)b,
                     (const double2*)x, (double2*)r);
  BEM_CHECK_LAUNCH(ctx);
  return BEM_OK;
}

bem_status launch_quad_field(bem_ctx* ctx, const bem_quad_surface* s, const double* qp,
                             int n_k, const double* k, int n_rhs, const void* phi,
                             const void* psi, void* phq, void* psq, void* sums, int32_t* list_ws,
                             int m, const double* xp, const int32_t* i0, const uint8_t* inside,
                             void* U) {
  const QuadRule R = make_rule();
  const int npts = s->n_elem * kQ;
  const int64_t tot = (int64_t)npts * n_k * n_rhs;
  hipLaunchKernelGGL(quad_interp_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0,
                     ctx->stream, s->n, s->n_elem, n_k * n_rhs, s->elem, R,
                     (const double2*)phi, (double2*)phq);
  hipLaunchKernelGGL(quad_interp_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0,
                     ctx->stream, s->n, s->n_elem, n_k * n_rhs, s->elem, R,
                     (const double2*)psi, (double2*)psq);
  // Eq. BRIEFdmn by the element quadrature, x0 the closest node a: the field sums
  // of field64_kernel over the quadrature points instead of the nodes
  const int pi = prof_begin(ctx, "field_quad");
  const bem_surface nodal{s->n, s->x, s->nrm, nullptr, s->bc};
  const FieldSources src{qp, qp + 3, qp + 6, 8, 8, npts, false, (const double2*)phq,
                         (const double2*)psq};
  const bem_status st = launch_field64(ctx, src, &nodal, n_k, k, n_rhs, phi, psi, m, xp, i0, inside,
                                       sums, list_ws, U);
  prof_end(ctx, "field_quad", pi, (double)m * n_k * n_rhs * npts, 0.0);
  return st;
}

}  // namespace bem

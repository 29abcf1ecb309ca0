// Surface-to-field evaluation by the non-singular representation (Sec. III,
// Eq. BRIEFdmn; its S_inf integrals evaluated, which leaves 4 pi P(x0) as the
// constant term when the integrals run over S only):
//   4 pi P(x_p) = 4 pi phi_a + sum_{j!=a} w_j [u_j (H^p_j - H^a_j) - u'_j (G^p_j - G^a_j)]
// with a the surface node closest to x_p, u_j = phi_j - phi_a g_aj - psi_a f_aj,
// u'_j = psi_j - phi_a g'_aj - psi_a f'_aj (f, g of Appendix A about x_a).
// The sum splits into S(x_p) - S(x_a) with
//   S(x) = A1 - phi_a A2 - psi_a A3,
//   A1 = sum w_j (phi_j H^x_j - psi_j G^x_j), A2 = sum w_j (g_aj H^x_j - g'_aj G^x_j),
//   A3 = sum w_j (f_aj H^x_j - f'_aj G^x_j)   (j != a).
// S(x_a) is computed once per node by the same kernel, so the per-point work
// is one sweep over the nodes.  A2 and A3 do not depend on the right-hand
// side: a workgroup takes NR right-hand sides at once and applies every
// generated kernel value (w G, w H for one node, point and frequency) to all
// of them, so NR right-hand sides cost one kernel generation and NR complex
// multiply-adds per term instead of NR generations.  The float32 kernel takes every phase k*r and k*s
// in float64, reduces it to [-1/2, 1/2) revolutions, and evaluates the
// trigonometric functions in float32 on the reduced argument.  Each point's
// sweep is split over kParts lanes (lane q takes every kParts-th node), whose
// partial sums are combined by a butterfly at the end: the float32 sums then
// run over n / kParts terms each, which bounds their rounding error kParts
// times tighter than one chain over all n nodes.
#include <type_traits>

#include "common.h"
#include "phase.h"

namespace bem {
namespace {

// ---------------------------------------------------------------- fixed scratch
// The node sums S(x_a) of bem_field_eval_noalloc live in this file-scope
// array (one copy per device, held until the process ends) instead of the
// context's workspace.  Host code never passes the array's name as an address
// (in host code it is only a stand-in for the device symbol): field_scratch_init
// takes the device address once per context, with the context's device
// current, and the kernels receive that pointer.
constexpr size_t kFieldScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[kFieldScratchBytes];

constexpr double kInv2Pi = 0.15915494309189533576888376337251;
constexpr double kFourPi = 12.566370614359172953850573533118;

// --------------------------------------------------------------- closest node
// i0[p] = argmin_j (dx*dx + dy*dy) + dz*dz, float64 without contraction,
// ties to the lowest j; inside[p] = n_a.(x_p - x_a) < 0.
constexpr int kCT = 256, kCChunk = 1024;

__global__ __launch_bounds__(kCT) void closest_kernel(int n, const double* __restrict__ x,
                                                      const double* __restrict__ nrm, int m,
                                                      const double* __restrict__ xp,
                                                      int32_t* __restrict__ i0,
                                                      uint8_t* __restrict__ inside) {
  __shared__ double sx[kCChunk], sy[kCChunk], sz[kCChunk];
  const int p = blockIdx.x * kCT + threadIdx.x;
  const bool valid = p < m;
  const double px = valid ? xp[3 * p] : 0.0, py = valid ? xp[3 * p + 1] : 0.0,
               pz = valid ? xp[3 * p + 2] : 0.0;
  double best = __builtin_inf();
  int bi = 0;
  for (int j0 = 0; j0 < n; j0 += kCChunk) {
    const int cnt = min(kCChunk, n - j0);
    __syncthreads();
    for (int e = threadIdx.x; e < cnt; e += kCT) {
      sx[e] = x[3 * (j0 + e)];
      sy[e] = x[3 * (j0 + e) + 1];
      sz[e] = x[3 * (j0 + e) + 2];
    }
    __syncthreads();
    for (int e = 0; e < cnt; ++e) {
      const double d0 = __dsub_rn(px, sx[e]);
      const double d1 = __dsub_rn(py, sy[e]);
      const double d2 = __dsub_rn(pz, sz[e]);
      const double dist = __dadd_rn(__dadd_rn(__dmul_rn(d0, d0), __dmul_rn(d1, d1)), __dmul_rn(d2, d2));
      if (dist < best) { best = dist; bi = j0 + e; }
    }
  }
  if (!valid) return;
  i0[p] = bi;
  const double d0 = __dsub_rn(px, x[3 * bi]), d1 = __dsub_rn(py, x[3 * bi + 1]),
               d2 = __dsub_rn(pz, x[3 * bi + 2]);
  const double nd = __dadd_rn(__dadd_rn(__dmul_rn(nrm[3 * bi], d0), __dmul_rn(nrm[3 * bi + 1], d1)),
                              __dmul_rn(nrm[3 * bi + 2], d2));
  inside[p] = nd < 0.0 ? 1 : 0;
}

__global__ void inside_kernel(const double* __restrict__ x, const double* __restrict__ nrm, int m,
                              const double* __restrict__ xp, const int32_t* __restrict__ i0,
                              uint8_t* __restrict__ inside) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= m) return;
  const int bi = i0[p];
  const double d0 = __dsub_rn(xp[3 * p], x[3 * bi]), d1 = __dsub_rn(xp[3 * p + 1], x[3 * bi + 1]),
               d2 = __dsub_rn(xp[3 * p + 2], x[3 * bi + 2]);
  const double nd = __dadd_rn(__dadd_rn(__dmul_rn(nrm[3 * bi], d0), __dmul_rn(nrm[3 * bi + 1], d1)),
                              __dmul_rn(nrm[3 * bi + 2], d2));
  inside[p] = nd < 0.0 ? 1 : 0;
}

// --------------------------------------------------------------- field sums
// sine and cosine in float32 of a float64 phase, in radians or (phase_rev) in
// revolutions, reduced in float64
__device__ inline void phase_rev(double t, float& s, float& c) {
  t -= rint(t);
  const float tf = (float)t;
  s = __builtin_amdgcn_sinf(tf);   // argument in revolutions
  c = __builtin_amdgcn_cosf(tf);
}
__device__ inline void phase_f32(double theta, float& s, float& c) {
  phase_rev(theta * kInv2Pi, s, c);
}

constexpr int kUneven = 4;
constexpr int kFT = 256, kNJ = 128, kParts = 8, kPW = kFT / kParts;   // kPW points per workgroup

// sum over the kParts consecutive lanes of one point (butterfly: every lane
// ends with the total)
template <typename R>
__device__ inline R part_sum(R v) {
#pragma unroll
  for (int o = 1; o < kParts; o <<= 1) v += __shfl_xor(v, o, kParts);
  return v;
}

// Float64 sums S(x) over the sources j of src (the surface nodes, or the
// quadrature points of the quadratic elements) for a chunk of FCH wavenumbers
// and NR right-hand sides.
// MODE 0: points = nodes; S into Snode [rhs][n_k][n].  With a node list (its
// length at *ncount) only the listed nodes.
// MODE 1: U [rhs][m][n_k] = P(x_p) = phi_a + (S(x_p) - S(x_a)) / (4 pi).
// Right-hand sides blockIdx.z * NR + r, r < min(NR, n_rhs - blockIdx.z * NR).
//
// Bound by float64 instructions: about 31 per (point, source, wavenumber) in
// the recurrence form plus 180 of geometry and phases per (point, source), and
// the LDS reads of 32 bytes of data per wavenumber.  On an even chunk (k_q =
// k_0 + q dk to a few ulp) both phases advance by rotation, so a pair takes
// four sincos instead of 2 FCH, and G carries w / r from the start; the products
// k r keep their rounding errors and every step the wavenumbers' own (EvenChunk), so
// the phases are closer than a sincos of each rounded product.  Uneven
// wavenumbers, and workgroups with a phase past the 2^20 rad for which the
// reduction of phase.h holds, go one wavenumber at a time (any other form in
// this kernel spills registers).  2304 points x 32 wavenumbers x 2562 nodes with
// the nodes' own sums take 1.29 ms (4.46 with a library sincos per value; 1.13 with
// the roundings left out).
template <int FCH, int MODE, int NR>
__global__ __launch_bounds__(kFT, 2) void field64_kernel(
    FieldSources src, int n, const double* __restrict__ x, const double* __restrict__ nrm,
    const double* __restrict__ kv, int n_k, int n_rhs, const double2* __restrict__ phi,
    const double2* __restrict__ psi, int m, const double* __restrict__ xp,
    const int32_t* __restrict__ i0, const uint8_t* __restrict__ inside,
    double2* __restrict__ Snode, double2* __restrict__ U, const int32_t* __restrict__ nlist,
    const int32_t* __restrict__ ncount) {
  if (MODE == 0 && nlist) {
    m = *ncount;
    if ((int)blockIdx.x * kPW >= m) return;   // the whole workgroup
  }
  __shared__ double sx[kNJ][3], sn[kNJ][3], sw[kNJ];
  __shared__ double2 sphi[NR][FCH][kNJ], spsi[NR][FCH][kNJ];
  const int p = blockIdx.x * kPW + threadIdx.x / kParts;
  const int part = threadIdx.x % kParts;
  const int m0 = blockIdx.y * FCH;
  const int r0 = blockIdx.z * NR;
  const int nrh = min(NR, n_rhs - r0);
  const int nf = min(FCH, n_k - m0);
  const bool valid = p < m && (MODE == 0 || !inside[p]);
  const int a = p < m ? (MODE == 0 ? (nlist ? nlist[p] : p) : i0[p]) : 0;
  const double ax = x[3 * a], ay = x[3 * a + 1], az = x[3 * a + 2];
  const double anx = nrm[3 * a], any = nrm[3 * a + 1], anz = nrm[3 * a + 2];
  const bool own = MODE == 0 || p >= m;
  const double px = own ? ax : xp[3 * p], py = own ? ay : xp[3 * p + 1],
               pz = own ? az : xp[3 * p + 2];
  // (the sums of wavenumbers past a partial chunk's end are not stored)
  EvenChunk<FCH> kc;
  kc.load(kv + m0, nf);
  // geometry of source jj of the staged tile: r, n_a.(x_j - x_a), w / r,
  // (d.n_j) / r^2, n_a.n_j
  struct Pair {
    double r, sa, wr, c, nn;
  };
  auto geometry = [&](int jj) {
    Pair g;
    const double dx = sx[jj][0] - px, dy = sx[jj][1] - py, dz = sx[jj][2] - pz;
    double rinv;
    dist_and_inverse64(dx * dx + dy * dy + dz * dz, g.r, rinv);
    g.c = (dx * sn[jj][0] + dy * sn[jj][1] + dz * sn[jj][2]) * (rinv * rinv);
    g.nn = anx * sn[jj][0] + any * sn[jj][1] + anz * sn[jj][2];
    g.sa = anx * (sx[jj][0] - ax) + any * (sx[jj][1] - ay) + anz * (sx[jj][2] - az);
    g.wr = sw[jj] * rinv;
    return g;
  };
  // sources [j0, j0 + cnt) and their data for the wavenumbers f0 .. f0 + nfs - 1
  // of the chunk into LDS
  auto stage = [&](int j0, int cnt, int f0, int nfs) {
    __syncthreads();
    for (int e = threadIdx.x; e < cnt * 3; e += kFT) {
      const int64_t j = j0 + e / 3;
      sx[e / 3][e % 3] = src.x[j * src.sx + e % 3];
      sn[e / 3][e % 3] = src.nrm[j * src.sx + e % 3];
    }
    for (int e = threadIdx.x; e < cnt; e += kFT) sw[e] = src.w[(int64_t)(j0 + e) * src.sw];
    for (int e = threadIdx.x; e < NR * nfs * kNJ; e += kFT) {
      const int r = e / (nfs * kNJ), f = (e / kNJ) % nfs, jj = e % kNJ;
      double2 u = make_double2(0.0, 0.0), v = u;
      if (r < nrh && f0 + f < nf && jj < cnt) {
        const int64_t o = ((int64_t)(m0 + f0 + f) * n_rhs + r0 + r) * src.n + j0 + jj;
        u = src.phi[o];
        v = src.psi[o];
      }
      sphi[r][f][jj] = u;
      spsi[r][f][jj] = v;
    }
    __syncthreads();
  };
  // one term: w G in G, e^{i k s} in F; slot f of the staged data
  auto term = [&](int jj, int f, double k, const Pair& g, double2 G, double2 F, auto& A1, double2& A2,
                  double2& A3) {
    // w H = w G (ikr - 1) c;  g = F.x, f = F.y / k, g' = -k nn F.y, f' = nn F.x
    const double ckr = k * (g.c * g.r), kn = k * g.nn;
    const double2 H = make_double2(fma(-g.c, G.x, -ckr * G.y), fma(ckr, G.x, -g.c * G.y));
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (NR > 1 && r >= nrh) break;   // uniform (one right-hand side: nrh = 1)
      const double2 u = sphi[r][f][jj], v = spsi[r][f][jj];
      A1[r].x = fma(u.x, H.x, fma(-u.y, H.y, fma(-v.x, G.x, fma(v.y, G.y, A1[r].x))));
      A1[r].y = fma(u.x, H.y, fma(u.y, H.x, fma(-v.x, G.y, fma(-v.y, G.x, A1[r].y))));
    }
    const double gp = kn * F.y, fp = kn * F.x;
    A2.x = fma(F.x, H.x, fma(gp, G.x, A2.x));
    A2.y = fma(F.x, H.y, fma(gp, G.y, A2.y));
    A3.x = fma(F.y, H.x, fma(-fp, G.x, A3.x));
    A3.y = fma(F.y, H.y, fma(-fp, G.y, A3.y));
  };
  // result of right-hand side r and wavenumber f of the chunk
  auto store = [&](int r, int f, double2 A1, double2 A2, double2 A3) {
    const int rhs = r0 + r;
    const double k = kv[m0 + f];
    const int64_t oa = ((int64_t)(m0 + f) * n_rhs + rhs) * n + a;
    const double2 pa = phi[oa];
    double2 qa = psi[oa];
    qa.x /= k;
    qa.y /= k;
    double2 S;
    S.x = A1.x - (pa.x * A2.x - pa.y * A2.y) - (qa.x * A3.x - qa.y * A3.y);
    S.y = A1.y - (pa.x * A2.y + pa.y * A2.x) - (qa.x * A3.y + qa.y * A3.x);
    if (MODE == 0) {
      Snode[((int64_t)rhs * n_k + m0 + f) * n + a] = S;
    } else {
      double2 out = make_double2(0.0, 0.0);
      if (valid && px == ax && py == ay && pz == az) {
        out = pa;   // the point is the node
      } else if (valid) {
        const double2 s0 = Snode[((int64_t)rhs * n_k + m0 + f) * n + a];
        out.x = pa.x + (S.x - s0.x) * (1.0 / kFourPi);
        out.y = pa.y + (S.y - s0.y) * (1.0 / kFourPi);
      }
      U[((int64_t)rhs * m + p) * n_k + m0 + f] = out;
    }
  };
  bool wide = false;
  if (kc.even) {
    double2 A1[FCH][NR], A2[FCH], A3[FCH];   // A3 times k
#pragma unroll
    for (int f = 0; f < FCH; ++f) {
#pragma unroll
      for (int r = 0; r < NR; ++r) A1[f][r] = make_double2(0.0, 0.0);
      A2[f] = A3[f] = make_double2(0.0, 0.0);
    }
    for (int j0 = 0; j0 < src.n; j0 += kNJ) {
      const int cnt = min(kNJ, src.n - j0);
      stage(j0, cnt, 0, FCH);
      if (!valid) continue;
      for (int jj = part; jj < cnt; jj += kParts) {
        if (src.nodes && j0 + jj == a) continue;   // both brackets vanish there
        const Pair g = geometry(jj);
        wide |= !(kc.kmax * fmax(g.r, fabs(g.sa)) < kPhaseNear);
        const double2 E = unit_phase(kc.k[kc.kMid], g.r), dE = unit_phase(kc.dk, g.r);
        const double2 F0 = unit_phase(kc.k[kc.kMid], g.sa), dF = unit_phase(kc.dk, g.sa);
        const double2 G0 = make_double2(g.wr * E.x, g.wr * E.y);
        double2 G = G0, F = F0;
#pragma unroll
        for (int i = 0; i < FCH; ++i) {
          const int f = kc.order(i);
          if (i > 0) {
            G = kc.advance(i, i == kc.kUp ? G0 : G, dE, g.r);
            F = kc.advance(i, i == kc.kUp ? F0 : F, dF, g.sa);
          }
          term(jj, f, kc.k[f], g, G, F, A1[f], A2[f], A3[f]);
        }
      }
    }
    // (a workgroup with a wide phase stores nothing here)
    wide = __syncthreads_or(wide);
    // the point's NR * FCH outputs are shared out over its kParts lanes
#pragma unroll
    for (int f = 0; f < FCH; ++f) {
      const double2 s2 = make_double2(part_sum(A2[f].x), part_sum(A2[f].y));
      const double2 s3 = make_double2(part_sum(A3[f].x), part_sum(A3[f].y));
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const double2 s1 = make_double2(part_sum(A1[f][r].x), part_sum(A1[f][r].y));
        if (p < m && !wide && (r * FCH + f) % kParts == part && r < nrh && f < nf)
          store(r, f, s1, s2, s3);
      }
    }
    if (!wide) return;   // uniform
  }
  // uneven wavenumbers: kUneven of them share a pair's geometry, a sincos each
  if (!wide) {
    constexpr int NU = FCH < kUneven ? FCH : kUneven;
    for (int f0 = 0; f0 < nf; f0 += NU) {
      double2 A1[NU][NR], A2[NU], A3[NU];
      double k[NU];
#pragma unroll
      for (int f = 0; f < NU; ++f) {
#pragma unroll
        for (int r = 0; r < NR; ++r) A1[f][r] = make_double2(0.0, 0.0);
        A2[f] = A3[f] = make_double2(0.0, 0.0);
        k[f] = kv[m0 + min(f0 + f, nf - 1)];
      }
      for (int j0 = 0; j0 < src.n; j0 += kNJ) {
        const int cnt = min(kNJ, src.n - j0);
        stage(j0, cnt, f0, NU);
        if (!valid) continue;
        for (int jj = part; jj < cnt; jj += kParts) {
          if (src.nodes && j0 + jj == a) continue;
          const Pair g = geometry(jj);
          wide |= !(kc.kmax * fmax(g.r, fabs(g.sa)) < kPhaseNear);
#pragma unroll
          for (int f = 0; f < NU; ++f) {
            const double2 E = unit_phase(k[f], g.r), F = unit_phase(k[f], g.sa);
            term(jj, f, k[f], g, make_double2(g.wr * E.x, g.wr * E.y), F, A1[f], A2[f], A3[f]);
          }
        }
      }
      if (f0 == 0) wide = __syncthreads_or(wide);   // (kmax covers the whole chunk)
      if (wide) break;
#pragma unroll
      for (int f = 0; f < NU; ++f) {
        const double2 s2 = make_double2(part_sum(A2[f].x), part_sum(A2[f].y));
        const double2 s3 = make_double2(part_sum(A3[f].x), part_sum(A3[f].y));
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          const double2 s1 = make_double2(part_sum(A1[f][r].x), part_sum(A1[f][r].y));
          if (p < m && (r * NU + f) % kParts == part && r < nrh && f0 + f < nf) store(r, f0 + f, s1, s2, s3);
        }
      }
    }
    if (!wide) return;   // uniform
  }
  // wide phases: one wavenumber at a time, by the library past the reduction's range
  for (int f = 0; f < nf; ++f) {
    const double k = kv[m0 + f];
    double2 A1[NR], A2 = make_double2(0.0, 0.0), A3 = A2;
#pragma unroll
    for (int r = 0; r < NR; ++r) A1[r] = make_double2(0.0, 0.0);
    for (int j0 = 0; j0 < src.n; j0 += kNJ) {
      const int cnt = min(kNJ, src.n - j0);
      stage(j0, cnt, f, 1);
      if (!valid) continue;
      for (int jj = part; jj < cnt; jj += kParts) {
        if (src.nodes && j0 + jj == a) continue;
        const Pair g = geometry(jj);
        double2 E, F;
        phase_sincos(k * g.r, &E.y, &E.x);
        phase_sincos(k * g.sa, &F.y, &F.x);
        term(jj, 0, k, g, make_double2(g.wr * E.x, g.wr * E.y), F, A1, A2, A3);
      }
    }
    const double2 s2 = make_double2(part_sum(A2.x), part_sum(A2.y));
    const double2 s3 = make_double2(part_sum(A3.x), part_sum(A3.y));
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const double2 s1 = make_double2(part_sum(A1[r].x), part_sum(A1[r].y));
      if (p < m && part == r % kParts && r < nrh) store(r, f, s1, s2, s3);
    }
  }
}

// list[0 .. *count) = the nodes that are some outside point's closest node (in
// no particular order; flag and *count zeroed)
__global__ void used_nodes_kernel(int m, const int32_t* __restrict__ i0,
                                  const uint8_t* __restrict__ inside, int32_t* __restrict__ flag,
                                  int32_t* __restrict__ count, int32_t* __restrict__ list) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x, lane = threadIdx.x & 63;
  const bool valid = p < m && !inside[p];
  const int a = valid ? i0[p] : -1;
  // neighbouring points share their node: one lane of a wave asks for each (one lane a
  // point put 20000 atomics on 12 nodes: 173 us, now 4)
  unsigned long long todo = __ballot(valid);
  while (todo) {
    const int l = __ffsll(todo) - 1;
    const int node = __builtin_amdgcn_readlane(a, l);
    todo &= ~__ballot(a == node);
    if (lane == l && flag[node] == 0 && atomicExch(&flag[node], 1) == 0)
      list[atomicAdd(count, 1)] = node;
  }
}

// ---------------------------------------------------------------- grouped field
// The float32 field of points grouped by their closest node a.  For one
// node, Eq. BRIEFdmn's brackets
//   u_j = w_j (phi_j - phi_a g_aj - psi_a f_aj),  v_j = w_j (psi_j - phi_a g'_aj - psi_a f'_aj)
// depend on (a, j, k) only, so a workgroup holding points of one node forms
// them once per node tile and frequency chunk (float64, rounded to float32)
// and every point's sum becomes S(x) = sum_{j != a} (u_j H^x_j - v_j G^x_j):
// one phase and two complex multiply-adds per term.  The node sums S(x_a)
// come from the float64 node pass (they are of the size of the surface data,
// while far from the bodies S(x_p) and the field are much smaller), and
//   P(x_p) = phi_a + (S(x_p) - S(x_a)) / (4 pi)
// is formed in float64.  Points are sorted by closest node with a counting
// sort; each node's points are cut into chunks of kGP = kPW (one workgroup
// each).  Inside points are in no chunk and get 0.
constexpr int kGP = kPW;

// cnt[a] = number of outside points whose closest node is a (cnt zeroed)
__global__ void group_count_kernel(int m, const int32_t* __restrict__ i0,
                                   const uint8_t* __restrict__ inside, int32_t* __restrict__ cnt) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < m && !inside[p]) atomicAdd(&cnt[i0[p]], 1);
}

// one workgroup of 1024 threads: off = exclusive scan of cnt, choff =
// exclusive scan of ceil(cnt / kGP), uoff = exclusive scan of (cnt > 0), all
// with their totals at [n]
__global__ __launch_bounds__(1024) void group_scan_kernel(int n, const int32_t* __restrict__ cnt,
                                                          int32_t* __restrict__ off,
                                                          int32_t* __restrict__ choff,
                                                          int32_t* __restrict__ uoff) {
  __shared__ int32_t sa[1024], sb[1024], sc[1024];
  __shared__ int32_t carry[3];
  if (threadIdx.x == 0) carry[0] = carry[1] = carry[2] = 0;
  __syncthreads();
  for (int b0 = 0; b0 < n; b0 += 1024) {
    const int i = b0 + threadIdx.x;
    const int c = i < n ? cnt[i] : 0;
    const int u = c > 0;
    sa[threadIdx.x] = c;
    sb[threadIdx.x] = (c + kGP - 1) / kGP;
    sc[threadIdx.x] = u;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {   // inclusive scans (Hillis-Steele)
      const int va = threadIdx.x >= o ? sa[threadIdx.x - o] : 0;
      const int vb = threadIdx.x >= o ? sb[threadIdx.x - o] : 0;
      const int vc = threadIdx.x >= o ? sc[threadIdx.x - o] : 0;
      __syncthreads();
      sa[threadIdx.x] += va;
      sb[threadIdx.x] += vb;
      sc[threadIdx.x] += vc;
      __syncthreads();
    }
    if (i < n) {
      off[i] = carry[0] + sa[threadIdx.x] - c;
      choff[i] = carry[1] + sb[threadIdx.x] - (c + kGP - 1) / kGP;
      uoff[i] = carry[2] + sc[threadIdx.x] - u;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      carry[0] += sa[1023];
      carry[1] += sb[1023];
      carry[2] += sc[1023];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    off[n] = carry[0];
    choff[n] = carry[1];
    uoff[n] = carry[2];
  }
}

// perm: the outside points ordered by closest node (fill zeroed); the order
// inside a node's range does not matter
__global__ void group_scatter_kernel(int m, const int32_t* __restrict__ i0,
                                     const uint8_t* __restrict__ inside,
                                     const int32_t* __restrict__ off, int32_t* __restrict__ fill,
                                     int32_t* __restrict__ perm) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= m || inside[p]) return;
  const int a = i0[p];
  perm[off[a] + atomicAdd(&fill[a], 1)] = p;
}

// chunks[c] = (node, first index into perm, points), kGP points at most;
// used[uoff[a]] = a for the nodes that are some point's closest node
__global__ void group_chunks_kernel(int n, const int32_t* __restrict__ cnt,
                                    const int32_t* __restrict__ off,
                                    const int32_t* __restrict__ choff, int4* __restrict__ chunks,
                                    const int32_t* __restrict__ uoff, int32_t* __restrict__ used) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= n) return;
  if (cnt[a] > 0) used[uoff[a]] = a;
  const int c0 = choff[a], nc = choff[a + 1] - c0;
  for (int c = 0; c < nc; ++c)
    chunks[c0 + c] = make_int4(a, off[a] + c * kGP, min(kGP, cnt[a] - c * kGP), 0);
}

// U = 0 for inside points
__global__ void zero_inside_kernel(int m, int n_k, int n_rhs, const uint8_t* __restrict__ inside,
                                   float2* __restrict__ U) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)m * n_k * n_rhs) return;
  const int p = (int)((t / n_k) % m);
  if (inside[p]) U[t] = make_float2(0.f, 0.f);
}

template <int FCH, int NR>
__global__ __launch_bounds__(kFT, 3) void field_grouped_kernel(
    int n, const double* __restrict__ x, const double* __restrict__ nrm,
    const double* __restrict__ w, const double* __restrict__ kv, int n_k, int n_rhs,
    const double2* __restrict__ phi, const double2* __restrict__ psi, int m,
    const double* __restrict__ xp, const int4* __restrict__ chunks,
    const int32_t* __restrict__ nchunks, const int32_t* __restrict__ perm,
    const double2* __restrict__ Snode, float2* __restrict__ U) {
  __shared__ double sx[kNJ][3];
  __shared__ float2 su[NR][FCH][kNJ], sv[NR][FCH][kNJ];
  __shared__ float snrm[kNJ][3];
  // per chunk frequency f: k, 1/k, and phi, psi of node a per right-hand side
  // (looked up by the bracket loop, whose f varies per thread)
  __shared__ double skk[FCH], skinv[FCH];
  __shared__ double2 spa[NR][FCH], sqa[NR][FCH];
  if ((int)blockIdx.x >= *nchunks) return;   // uniform
  const int4 ch = chunks[blockIdx.x];
  const int a = ch.x, start = ch.y, len = ch.z;
  const int gi = threadIdx.x / kParts, part = threadIdx.x % kParts;
  const bool valid = gi < len;
  const int p = valid ? perm[start + gi] : -1;
  const double ax = x[3 * a], ay = x[3 * a + 1], az = x[3 * a + 2];
  const double anx = nrm[3 * a], any = nrm[3 * a + 1], anz = nrm[3 * a + 2];
  const double px = p >= 0 ? xp[3 * p] : ax, py = p >= 0 ? xp[3 * p + 1] : ay,
               pz = p >= 0 ? xp[3 * p + 2] : az;
  const int m0 = blockIdx.y * FCH;
  const int r0 = blockIdx.z * NR;
  const int nrh = min(NR, n_rhs - r0);
  const int nf = min(FCH, n_k - m0);
  double kk[FCH];
#pragma unroll
  for (int f = 0; f < FCH; ++f) kk[f] = f < nf ? kv[m0 + f] : kv[m0];
  const double dkk = nf > 1 ? (kk[nf - 1] - kk[0]) / (nf - 1) : 0.0;
  bool uni = nf > 1;
#pragma unroll
  for (int f = 1; f < FCH; ++f)
    if (f < nf && !(fabs(kk[f] - (kk[0] + f * dkk)) <= 4e-16 * fabs(kk[f]))) uni = false;
  if (threadIdx.x < FCH) {
    const double kf0 = kv[m0 + min((int)threadIdx.x, nf - 1)];
    skk[threadIdx.x] = kf0;
    skinv[threadIdx.x] = 1.0 / kf0;
  }
  if (threadIdx.x < NR * FCH) {
    const int r = threadIdx.x / FCH, f = threadIdx.x % FCH;
    double2 pa = make_double2(0.0, 0.0), qa = pa;
    if (r < nrh && f < nf) {
      const int64_t va = ((int64_t)(m0 + f) * n_rhs + r0 + r) * n;
      pa = phi[va + a];
      qa = psi[va + a];
    }
    spa[r][f] = pa;
    sqa[r][f] = qa;
  }
  // (the node loop's first barrier publishes these tables)
  const double k0rev = kk[0] * kInv2Pi, dkrev = dkk * kInv2Pi;
  float2 S[NR][FCH], S1[NR][FCH];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int f = 0; f < FCH; ++f) S[r][f] = S1[r][f] = make_float2(0.f, 0.f);
  for (int j0 = 0; j0 < n; j0 += kNJ) {
    const int cnt = min(kNJ, n - j0);
    __syncthreads();
    for (int e = threadIdx.x; e < cnt * 3; e += kFT) {
      sx[e / 3][e % 3] = x[3 * j0 + e];
      snrm[e / 3][e % 3] = (float)nrm[3 * j0 + e];
    }
    // the brackets u, v of the tile's nodes for the workgroup's node a
    for (int e = threadIdx.x; e < NR * FCH * kNJ; e += kFT) {
      const int r = e / (FCH * kNJ), f = (e / kNJ) % FCH, jj = e % kNJ;
      float2 uu = make_float2(0.f, 0.f), vv = uu;
      const int j = j0 + jj;
      if (r < nrh && f < nf && jj < cnt && j != a) {
        const double k = skk[f];
        const double njx = nrm[3 * j], njy = nrm[3 * j + 1], njz = nrm[3 * j + 2];
        const double sa = anx * (x[3 * j] - ax) + any * (x[3 * j + 1] - ay) + anz * (x[3 * j + 2] - az);
        const double nn = anx * njx + any * njy + anz * njz;
        // the phase reduced in float64, its sine and cosine in float32 (the
        // brackets are rounded to float32)
        float fsn, fcs;
        phase_f32(k * sa, fsn, fcs);
        const double sn = fsn, cs = fcs;
        const double g = cs, fv = sn * skinv[f], gp = -k * sn * nn, fp = cs * nn;
        const int64_t va = ((int64_t)(m0 + f) * n_rhs + r0 + r) * n;
        const double2 pa = spa[r][f], qa = sqa[r][f], pj = phi[va + j], qj = psi[va + j];
        const double wj = w[j];
        uu = make_float2((float)(wj * (pj.x - pa.x * g - qa.x * fv)),
                         (float)(wj * (pj.y - pa.y * g - qa.y * fv)));
        vv = make_float2((float)(wj * (qj.x - pa.x * gp - qa.x * fp)),
                         (float)(wj * (qj.y - pa.y * gp - qa.y * fp)));
      }
      su[r][f][jj] = uu;
      sv[r][f][jj] = vv;
    }
    __syncthreads();
    if (!valid) continue;
    // the lane's nodes alternate between two partial sums (halving the
    // length of each float32 chain)
    // uni_c: std::true_type / std::false_type (the test folded away) or a
    // runtime bool
    auto term = [&](int jj, float2 (&Sh)[NR][FCH], auto uni_c) {
      const bool UNI = static_cast<bool>(uni_c);
      if (j0 + jj == a) return;   // its brackets vanish (and r = 0 for a point on the node)
      const double dx = sx[jj][0] - px, dy = sx[jj][1] - py, dz = sx[jj][2] - pz;
      // r from the float32 reciprocal square root of r^2 and one Newton step in
      // float64 (relative error ~1e-14, ample for the float64 phase k r);
      // that reciprocal is also the kernel's float32 1/r
      const double r2 = dx * dx + dy * dy + dz * dz;
      const float rinv = __builtin_amdgcn_rsqf((float)r2);
      double r = r2 * (double)rinv;
      r = fma(fma(-r, r, r2), 0.5 * (double)rinv, r);
      // u H - v G = E' t with E' = -E / r (rotated like E) and
      // t = c u (1 - ikr) + v, c = (d.n_j)/r^2
      const float c = ((float)dx * snrm[jj][0] + (float)dy * snrm[jj][1] + (float)dz * snrm[jj][2]) *
                      (rinv * rinv);
      float es, ec, des = 0.f, dec = 1.f;
      // (the wavenumbers carry the 1 / 2 pi of the reduction)
      phase_rev(k0rev * r, es, ec);
      if (UNI) phase_rev(dkrev * r, des, dec);
      const float cr = c * (float)r;
      es *= -rinv;
      ec *= -rinv;
      // on an even chunk the phase advances by the three-term recurrence
      // E'_{f+1} = 2 cos(dk r) E'_f - E'_{f-1} (two multiply-adds a step; a
      // rounding at step f grows at most f-fold over the chunk)
      const float tc = 2.f * dec;
      float esp = 0.f, ecp = 0.f;
#pragma unroll
      for (int f = 0; f < FCH; ++f) {
        if (f > 0) {
          if (UNI) {
            float e1, e0;
            if (f == 1) {
              e1 = ec * des + es * dec;
              e0 = ec * dec - es * des;
            } else {
              e1 = fmaf(tc, es, -esp);
              e0 = fmaf(tc, ec, -ecp);
            }
            esp = es;
            ecp = ec;
            es = e1;
            ec = e0;
          } else {
            phase_f32(kk[f] * r, es, ec);
            es *= -rinv;
            ec *= -rinv;
          }
        }
        const float cq = (float)kk[f] * cr;   // c k r
#pragma unroll
        for (int rr = 0; rr < NR; ++rr) {
          if (NR > 1 && rr >= nrh) break;   // uniform (one right-hand side: nrh = 1)
          const float2 u = su[rr][f][jj], v = sv[rr][f][jj];
          const float tx = fmaf(c, u.x, fmaf(cq, u.y, v.x));
          const float ty = fmaf(c, u.y, fmaf(-cq, u.x, v.y));
          Sh[rr][f].x = fmaf(ec, tx, fmaf(-es, ty, Sh[rr][f].x));
          Sh[rr][f].y = fmaf(ec, ty, fmaf(es, tx, Sh[rr][f].y));
        }
      }
    };
    auto nodes = [&](auto uni_c) {
      for (int jj = part; jj < cnt; jj += 2 * kParts) {
        term(jj, S, uni_c);
        if (jj + kParts < cnt) term(jj + kParts, S1, uni_c);
      }
    };
    // one right-hand side: the even-chunk test is hoisted out of the node loop
    // (no per-frequency branch inside it); with several, the two loop bodies
    // would not fit the register budget, so the test stays inside
    if constexpr (NR == 1) {
      if (uni)
        nodes(std::true_type{});
      else
        nodes(std::false_type{});
    } else {
      nodes(uni);
    }
  }
#pragma unroll
  for (int rr = 0; rr < NR; ++rr)
#pragma unroll
    for (int f = 0; f < FCH; ++f) {
      S[rr][f].x += S1[rr][f].x;
      S[rr][f].y += S1[rr][f].y;
    }
#pragma unroll
  for (int rr = 0; rr < NR; ++rr)
#pragma unroll
    for (int f = 0; f < FCH; ++f) {
      S[rr][f].x = part_sum(S[rr][f].x);
      S[rr][f].y = part_sum(S[rr][f].y);
    }
  if (p < 0) return;
  const double inv4pi = 1.0 / kFourPi;
#pragma unroll
  for (int rr = 0; rr < NR; ++rr)
#pragma unroll
    for (int f = 0; f < FCH; ++f) {
      if ((rr * FCH + f) % kParts != part || rr >= nrh || f >= nf) continue;
      const double2 pa = phi[((int64_t)(m0 + f) * n_rhs + r0 + rr) * n + a];
      const double2 sa = Snode[((int64_t)(r0 + rr) * n_k + m0 + f) * n + a];
      U[((int64_t)(r0 + rr) * m + p) * n_k + m0 + f] =
          make_float2((float)(pa.x + ((double)S[rr][f].x - sa.x) * inv4pi),
                      (float)(pa.y + ((double)S[rr][f].y - sa.y) * inv4pi));
    }
}

size_t al256(size_t b) { return (b + 255) / 256 * 256; }

FieldSources node_sources(const bem_surface* s, const void* phi, const void* psi) {
  return FieldSources{s->x, s->nrm, s->w, 3, 1, s->n, true, (const double2*)phi, (const double2*)psi};
}

// MODE 0 over every node, or the list's
void launch_node_sums(bem_ctx* ctx, const FieldSources& src, const bem_surface* s, int n_k,
                      const double* k, int n_rhs, const void* phi, const void* psi, void* Snode,
                      const int32_t* nlist, const int32_t* ncount) {
  // one right-hand side: 8 frequencies per thread; more: 4 frequencies and up
  // to 4 right-hand sides per workgroup
#define BEM_NODE_SUMS(FCH, NR)                                                                     \
  hipLaunchKernelGGL((field64_kernel<FCH, 0, NR>),                                                 \
                     dim3((s->n + kPW - 1) / kPW, (n_k + FCH - 1) / FCH, (n_rhs + NR - 1) / NR),   \
                     dim3(kFT), 0, ctx->stream, src, s->n, s->x, s->nrm, k, n_k, n_rhs,            \
                     (const double2*)phi, (const double2*)psi, s->n, s->x, (const int32_t*)nullptr, \
                     (const uint8_t*)nullptr, (double2*)Snode, (double2*)nullptr, nlist, ncount)
  if (n_rhs == 1) BEM_NODE_SUMS(8, 1);
  else BEM_NODE_SUMS(4, 4);
#undef BEM_NODE_SUMS
}

// fixed: the fixed scratch (bem_field_eval_noalloc: no workspace, no
// profiling events), else NULL
template <int FCH, int NR>
bem_status field_grouped(bem_ctx* ctx, const bem_surface* s, int n_k, const double* k, int n_rhs,
                         const void* phi, const void* psi, int m, const double* xp,
                         const int32_t* i0, const uint8_t* inside, void* U, void* fixed) {
  const int n = s->n;
  auto al = al256;
  const size_t max_chunks = (size_t)(m + kGP - 1) / kGP + n;
  const size_t bytes = field_group_bytes(n, m, n_k, n_rhs);
  void* ws = fixed;
  bem_status st = BEM_OK;
  if (!ws && (st = workspace(ctx, bytes, &ws)) != BEM_OK) return st;
  char* q = (char*)ws;
  double2* Snode = (double2*)q; q += al(16 * (size_t)n_rhs * n_k * n);
  int32_t* cnt = (int32_t*)q;   q += al(4 * (size_t)n);
  int32_t* fill = (int32_t*)q;  q += al(4 * (size_t)n);
  int32_t* off = (int32_t*)q;   q += al(4 * (size_t)(n + 1));
  int32_t* choff = (int32_t*)q; q += al(4 * (size_t)(n + 1));
  int32_t* uoff = (int32_t*)q;  q += al(4 * (size_t)(n + 1));
  int32_t* used = (int32_t*)q;  q += al(4 * (size_t)n);
  int32_t* perm = (int32_t*)q;  q += al(4 * (size_t)m);
  int4* chunks = (int4*)q;
  if ((st = fill_zero(ctx, cnt, 2 * al(4 * (size_t)n))) != BEM_OK) return st;   // cnt and fill
  const int pi = fixed ? -1 : prof_begin(ctx, "field");
  hipLaunchKernelGGL(group_count_kernel, dim3((m + 255) / 256), dim3(256), 0, ctx->stream, m, i0,
                     inside, cnt);
  hipLaunchKernelGGL(group_scan_kernel, dim3(1), dim3(1024), 0, ctx->stream, n, cnt, off, choff,
                     uoff);
  hipLaunchKernelGGL(group_chunks_kernel, dim3((n + 255) / 256), dim3(256), 0, ctx->stream, n, cnt,
                     off, choff, chunks, uoff, used);
  // float64 node sums S(x_a) of the nodes that are some point's closest node
  // (their count uoff[n] stays on the device: the grid covers all n nodes and
  // the workgroups past the count return at once)
  launch_node_sums(ctx, node_sources(s, phi, psi), s, n_k, k, n_rhs, phi, psi, Snode, used, uoff + n);
  hipLaunchKernelGGL(group_scatter_kernel, dim3((m + 255) / 256), dim3(256), 0, ctx->stream, m, i0,
                     inside, off, fill, perm);
  const int64_t tot = (int64_t)m * n_k * n_rhs;
  hipLaunchKernelGGL(zero_inside_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0,
                     ctx->stream, m, n_k, n_rhs, inside, (float2*)U);
  dim3 grid((unsigned)max_chunks, (n_k + FCH - 1) / FCH, (n_rhs + NR - 1) / NR);
  hipLaunchKernelGGL((field_grouped_kernel<FCH, NR>), grid, dim3(kFT), 0, ctx->stream, n, s->x,
                     s->nrm, s->w, k, n_k, n_rhs, (const double2*)phi, (const double2*)psi, m, xp,
                     chunks, choff + n, perm, Snode, (float2*)U);
  // kernel terms: one per (point, frequency, node, rhs); the node pass adds
  // as many per node used as some point's closest node
  if (!fixed)
    prof_end(ctx, "field", pi, (double)m * n_k * n * n_rhs, 8.0 * (double)m * n_k * n_rhs);
  BEM_CHECK_LAUNCH(ctx);
  return BEM_OK;
}

// c128: the node sums of the points' closest nodes (of every node with the fixed
// scratch, which holds nothing else), then the points
bem_status field_c128(bem_ctx* ctx, const bem_surface* s, int n_k, const double* k, int n_rhs,
                      const void* phi, const void* psi, int m, const double* xp,
                      const int32_t* i0, const uint8_t* inside, void* U, void* fixed) {
  void* ws = fixed;
  const size_t sums = al256(16 * (size_t)n_rhs * n_k * s->n), ints = al256(4 * (size_t)(s->n + 1));
  bem_status st;
  if (!ws && (st = workspace(ctx, sums + 2 * ints, &ws)) != BEM_OK) return st;
  const int pi = fixed ? -1 : prof_begin(ctx, "field");
  st = launch_field64(ctx, node_sources(s, phi, psi), s, n_k, k, n_rhs, phi, psi, m, xp, i0, inside,
                      ws, fixed ? nullptr : (int32_t*)((char*)ws + sums), U);
  // kernel terms: one per (point, frequency, node, rhs)
  if (!fixed)
    prof_end(ctx, "field", pi, (double)m * n_k * s->n * n_rhs, 16.0 * (double)m * n_k * n_rhs);
  return st;
}

}  // namespace

bem_status launch_closest(bem_ctx* ctx, const bem_surface* s, int m, const double* xp,
                          int32_t* i0, uint8_t* inside) {
  if (m <= 0) return BEM_OK;
  hipLaunchKernelGGL(closest_kernel, dim3((m + kCT - 1) / kCT), dim3(kCT), 0, ctx->stream, s->n,
                     s->x, s->nrm, m, xp, i0, inside);
  BEM_CHECK_LAUNCH(ctx);
  return BEM_OK;
}

bem_status launch_inside(bem_ctx* ctx, const bem_surface* s, int m, const double* xp,
                         const int32_t* i0, uint8_t* inside) {
  if (m <= 0) return BEM_OK;
  hipLaunchKernelGGL(inside_kernel, dim3((m + 255) / 256), dim3(256), 0, ctx->stream, s->x, s->nrm,
                     m, xp, i0, inside);
  BEM_CHECK_LAUNCH(ctx);
  return BEM_OK;
}

bem_status launch_field64(bem_ctx* ctx, const FieldSources& src, const bem_surface* s, int n_k,
                          const double* k, int n_rhs, const void* phi, const void* psi, int m,
                          const double* xp, const int32_t* i0, const uint8_t* inside, void* Snode,
                          int32_t* list_ws, void* U) {
  int32_t *list = nullptr, *count = nullptr;
  // the list pays once the sums of every node no longer fit the chip at once (below, its
  // two launches cost 10 us of a call of 40, 12 nodes and 40 points)
  const int fch = n_rhs == 1 ? 8 : 4, nr = n_rhs == 1 ? 1 : 4;
  const int64_t all = (int64_t)((s->n + kPW - 1) / kPW) * ((n_k + fch - 1) / fch) * ((n_rhs + nr - 1) / nr);
  if (list_ws && all > ctx->num_cus) {
    // flag [n], count, then (256-byte aligned) the list
    const size_t ints = al256(4 * (size_t)(s->n + 1));
    count = list_ws + s->n;
    list = (int32_t*)((char*)list_ws + ints);
    const bem_status st = fill_zero(ctx, list_ws, 4 * (size_t)(s->n + 1));
    if (st != BEM_OK) return st;
    hipLaunchKernelGGL(used_nodes_kernel, dim3((m + 255) / 256), dim3(256), 0, ctx->stream, m, i0,
                       inside, list_ws, count, list);
  }
  launch_node_sums(ctx, src, s, n_k, k, n_rhs, phi, psi, Snode, list, count);
#define BEM_POINTS(FCH, NR)                                                                       \
  hipLaunchKernelGGL((field64_kernel<FCH, 1, NR>),                                                \
                     dim3((m + kPW - 1) / kPW, (n_k + FCH - 1) / FCH, (n_rhs + NR - 1) / NR),     \
                     dim3(kFT), 0, ctx->stream, src, s->n, s->x, s->nrm, k, n_k, n_rhs,           \
                     (const double2*)phi, (const double2*)psi, m, xp, i0, inside, (double2*)Snode, \
                     (double2*)U, (const int32_t*)nullptr, (const int32_t*)nullptr)
  if (n_rhs == 1) BEM_POINTS(8, 1);
  else BEM_POINTS(4, 4);
#undef BEM_POINTS
  BEM_CHECK_LAUNCH(ctx);
  return BEM_OK;
}

bem_status launch_field(bem_ctx* ctx, const bem_surface* s, int n_k, const double* k, int n_rhs,
                        const void* phi, const void* psi, int m, const double* xp,
                        const int32_t* i0, const uint8_t* inside, bem_prec prec, void* U,
                        bool fixed_scratch) {
  if (m <= 0) return BEM_OK;
  void* fixed = nullptr;
  if (fixed_scratch && prec == BEM_C128) {
    const size_t need = 16 * (size_t)n_rhs * n_k * s->n;
    if (!ctx->field_scratch)
      return fail(ctx, BEM_EHIP, "bem_field_eval_noalloc: no device address for the fixed scratch");
    if (need > ctx->field_scratch_bytes)
      return fail(ctx, BEM_EINVAL,
                  "bem_field_eval_noalloc: n_rhs * n_k * n = %lld node sums need %zu bytes, more "
                  "than the %zu-byte fixed scratch",
                  (long long)n_rhs * n_k * s->n, need, ctx->field_scratch_bytes);
    fixed = ctx->field_scratch;
  }
  if (prec == BEM_C128)
    return field_c128(ctx, s, n_k, k, n_rhs, phi, psi, m, xp, i0, inside, U, fixed);
  // float32: points grouped by closest node (the bookkeeping in the fixed
  // scratch for bem_field_eval_noalloc, whose caller checked its size)
  void* gfixed = fixed_scratch ? ctx->field_scratch : nullptr;
  if (fixed_scratch && field_group_bytes(s->n, m, n_k, n_rhs) > ctx->field_scratch_bytes)
    return fail(ctx, BEM_EINVAL, "bem_field_eval_noalloc: point grouping does not fit the fixed scratch");
  if (n_rhs == 1)
    return field_grouped<8, 1>(ctx, s, n_k, k, n_rhs, phi, psi, m, xp, i0, inside, U, gfixed);
  return field_grouped<4, 4>(ctx, s, n_k, k, n_rhs, phi, psi, m, xp, i0, inside, U, gfixed);
}

bem_status field_scratch_init(bem_ctx* ctx) {
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr) {
    ctx->field_scratch = nullptr;
    ctx->field_scratch_bytes = 0;
    return fail(ctx, BEM_EHIP, "hipGetSymbolAddress of the field scratch failed: %s",
                hipGetErrorString(e));
  }
  ctx->field_scratch = ptr;
  ctx->field_scratch_bytes = kFieldScratchBytes;
  return BEM_OK;
}

size_t field_group_bytes(int n, int m, int n_k, int n_rhs) {
  const size_t max_chunks = (size_t)(m + kGP - 1) / kGP + n;
  return al256(16 * (size_t)n_rhs * n_k * n) + 3 * al256(4 * (size_t)n) +
         3 * al256(4 * (size_t)(n + 1)) + al256(4 * (size_t)m) + al256(16 * max_chunks);
}

}  // namespace bem

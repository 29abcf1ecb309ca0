// Triangular solves X = U^{-1} L^{-1} P B with the factors of the batched LU
// (row-major, P A = L U, unit L) for one or more right-hand sides per matrix,
// and the permutation of the recorded interchanges.
//
// The factors are read once per solve (8 or 16 n^2 bytes), so the bound is HBM;
// what has to be avoided is the chain through the unknowns.  The unknowns are
// solved in blocks of TS_NB: one workgroup per vector solves a block's triangle
// (trsv_block), then every unknown left takes the block's contribution in a
// matrix-vector launch over all of the chip (trsv_update_kernel).  A single
// workgroup per vector doing both read its factors at 21 GB/s: 64 systems of
// n = 5124 took 9.9 ms per solve, 8 of n = 10242 12 ms, 32 of n = 2562 with 8 sets
// of factors 2.9 ms; now 5.1, about 2.5 and 1.0 ms.
//
// The blocks' contributions are taken off float64 copies of the float32 vectors (acc,
// where the caller has room for them): rounding a vector once per block of 256
// gave solves of n = 5124 a 1.2 times larger error than one sum per unknown.
#include <algorithm>

#include "lu_types.h"

namespace bem {
using namespace lud;
namespace {

// a b, fused the same way in every loop
template <typename C> __device__ inline C product(C a, C b) {
  return cmk<C>(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
// value of lane l (wave-uniform) in every lane
__device__ inline float lane_value(float v, int l) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), l));
}
__device__ inline double lane_value(double v, int l) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, l);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// ============================================================== pivots -> permutation
// perm[i] = original row that ends in position i after the interchanges; one
// wave composes them in LDS, skipping the positions that are not interchanged
// (most, for the boundary-integral systems) 64 at a time.
__global__ __launch_bounds__(64) void perm_kernel(int n, const int32_t* __restrict__ piv,
                                                  int32_t* __restrict__ perm) {
  extern __shared__ int32_t q[];
  const int32_t* pb = piv + (int64_t)blockIdx.x * n;
  int32_t* qb = perm + (int64_t)blockIdx.x * n;
  const int lane = threadIdx.x;
  for (int i = lane; i < n; i += 64) q[i] = i;
  __syncthreads();
  int p = pb[min(lane, n - 1)];
  for (int i0 = 0; i0 < n; i0 += 64) {
    const int cur = p;
    if (i0 + 64 < n) p = pb[min(i0 + 64 + lane, n - 1)];
    unsigned long long todo = __ballot(i0 + lane < n && cur != i0 + lane);
    while (todo) {
      const int l = __ffsll((unsigned long long)todo) - 1;
      todo &= todo - 1;
      const int a = i0 + l, b = __builtin_amdgcn_readlane(cur, l);
      if (lane == 0) {
        const int32_t t = q[a];
        q[a] = q[b];
        q[b] = t;
      }
    }
  }
  __syncthreads();
  for (int i = lane; i < n; i += 64) qb[i] = q[i];
}

// ============================================================== blocks of the solve
constexpr int TS_B = 64;             // tile
constexpr int TS_T = 512;            // threads of the block kernels
constexpr int TS_TILES = 5;          // tiles of the largest block
constexpr int TS_NB = 4 * TS_B;      // block; a remainder of up to a tile joins the last one
constexpr int TS_DLD = TS_B + 1;     // leading dimension of a staged diagonal tile

// LDS of trsv_block: the block's right-hand side, two diagonal tiles, the block's
// unknowns, the sums of the row tile about to be solved
template <typename C>
constexpr size_t trsv_lds() {
  return sizeof(double2) * TS_TILES * TS_B + sizeof(C) * (2 * TS_B * TS_DLD + TS_TILES * TS_B + 2 * TS_B);
}

// Solves rows [i0, i0 + rows) of L (FWD) or U: bs (LDS) holds the block's right-hand
// side, in float64 so that an unknown is rounded once when the earlier tiles' sums
// have been taken off, and xs and bs its solution on exit.  Tiles are taken
// in solving order (logical tile t is physical t, or T - 1 - t backwards).  Wave
// 2 (I - 1) + half owns row tile I and one half of the columns of each tile it
// multiplies: a lane keeps its row's 32 entries in registers, loaded while the
// tile's unknowns are still being solved, and its sum over the tiles before I.
// The unknowns of a tile come from one wave, a lane per row, the solved value
// broadcast through a scalar register; each product is formed before it is
// subtracted (one rounding of the unknown per step: fused into it, the two
// multiply-adds of a component round it twice, and the chain's error grew from
// 2.3e-7 to 3.4e-7 at n = 642).
template <typename R, bool FWD>
__device__ __forceinline__ void trsv_block(const typename Cx<R>::T* __restrict__ Lb, int64_t ld, int i0,
                                           int rows, bool vec, double2* bs, typename Cx<R>::T* D,
                                           typename Cx<R>::T* xs, typename Cx<R>::T* sums) {
  using C = typename Cx<R>::T;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = (rows + TS_B - 1) / TS_B;
  auto phys = [&](int t) { return FWD ? t : T - 1 - t; };
  const C zero = cmk<C>(R(0), R(0));
  // diagonal tile of logical tile t: loaded into registers, then stored into
  // buffer t & 1, the other triangle and rows past the end zero
  constexpr int SQ = TS_B * TS_B / TS_T;
  C nxt[SQ];
  auto stage_load = [&](int t) {
    const int r0 = phys(t) * TS_B, m = min(TS_B, rows - r0);
#pragma unroll
    for (int q = 0; q < SQ; ++q) {
      const int e = tid + q * TS_T, r = e / TS_B, c = e % TS_B;
      nxt[q] = Lb[(int64_t)(i0 + r0 + min(r, m - 1)) * ld + i0 + r0 + min(c, m - 1)];
    }
  };
  auto stage_store = [&](int t) {
    const int m = min(TS_B, rows - phys(t) * TS_B);
    C* d = D + (t & 1) * TS_B * TS_DLD;
#pragma unroll
    for (int q = 0; q < SQ; ++q) {
      const int e = tid + q * TS_T, r = e / TS_B, c = e % TS_B;
      d[r * TS_DLD + c] = r < m && c < m && (FWD ? c < r : c >= r) ? nxt[q] : zero;
    }
  };
  // this wave's half of tile (I, J)
  const int I = 1 + wid / 2, half = wid & 1;
  C l[TS_B / 2];
  auto load = [&](int J) {
    const int r = min(phys(I) * TS_B + lane, rows - 1), c0 = phys(J) * TS_B + half * (TS_B / 2);
    const C* src = Lb + (int64_t)(i0 + r) * ld + i0 + c0;
    if (c0 + TS_B / 2 <= rows && vec) {
#pragma unroll
      for (int c = 0; c < TS_B / 2; c += 16 / (int)sizeof(C)) {
        const uint4 v = *reinterpret_cast<const uint4*>(src + c);
        __builtin_memcpy(&l[c], &v, 16);
      }
    } else {
      const int left = rows - c0;   // columns past the block: zero
#pragma unroll
      for (int c = 0; c < TS_B / 2; ++c) {
        const C v = src[min(c, left - 1)];
        l[c] = c < left ? v : zero;
      }
    }
  };
  C acc = zero;
  stage_load(0);
  stage_store(0);
  for (int J = 0; J < T; ++J) {
    __syncthreads();   // the tile and the sums of row tile J are there
    const int solver = J == 0 ? TS_T / 64 - 1 : 2 * (J - 1);
    if (J + 1 < T) stage_load(J + 1);
    if (I > J && I < T && phys(J) * TS_B + half * (TS_B / 2) < rows) load(J);
    if (wid == solver) {
      const C* d = D + (J & 1) * TS_B * TS_DLD + lane * TS_DLD;
      const int r0 = phys(J) * TS_B;
      double2 b = bs[r0 + lane];   // (padded with zeros to whole tiles)
      if (J > 0) {
        b.x -= sums[lane].x + sums[TS_B + lane].x;
        b.y -= sums[lane].y + sums[TS_B + lane].y;
      }
      C v = cmk<C>((R)b.x, (R)b.y);
      if (FWD) {
#pragma unroll
        for (int c = 0; c < TS_B; ++c) {
          const C x = cmk<C>(lane_value(v.x, c), lane_value(v.y, c));
          const C p = product(d[c], x), s = cmk<C>(v.x - p.x, v.y - p.y);
          v = lane > c ? s : v;
        }
      } else {
        const C dinv = r0 + lane < rows ? crecip(d[lane]) : cmk<C>(R(1), R(0));
#pragma unroll
        for (int c = TS_B - 1; c >= 0; --c) {
          const C t = product(v, dinv);
          const C x = cmk<C>(lane_value(t.x, c), lane_value(t.y, c));
          const C p = product(d[c], x), s = cmk<C>(v.x - p.x, v.y - p.y);
          v = lane == c ? t : (lane < c ? s : v);
        }
      }
      xs[r0 + lane] = v;
      bs[r0 + lane] = make_double2(v.x, v.y);
    }
    if (J + 1 < T) stage_store(J + 1);
    __syncthreads();   // the unknowns of tile J are there
    if (I > J && I < T) {
      const int c0 = phys(J) * TS_B + half * (TS_B / 2);
      if (c0 < rows) {
        C a = zero, b = zero;
#pragma unroll
        for (int c = 0; c < TS_B / 2; c += 2) {
          a = cfma(a, l[c], xs[c0 + c]);
          b = cfma(b, l[c + 1], xs[c0 + c + 1]);
        }
        acc.x += a.x + b.x;
        acc.y += a.y + b.y;
      }
      if (I == J + 1) sums[half * TS_B + lane] = acc;
    }
  }
  __syncthreads();
}

// One workgroup per vector.  WHOLE: the whole solve of systems of one block
// (permuted right-hand side in, both triangles); else the block [i0, i0 + rows)
// of L (FWD) or U of the vectors in acc [gridDim.x][n], or NULL: in X.
template <typename R, bool WHOLE, bool FWD>
__global__ __launch_bounds__(TS_T) void trsv_block_kernel(
    int n, int64_t ld, int64_t stride, const typename Cx<R>::T* __restrict__ LU,
    const int32_t* __restrict__ perm, int n_rhs, const typename Cx<R>::T* __restrict__ Bin,
    typename Cx<R>::T* __restrict__ X, int64_t bstride, const int32_t* __restrict__ fac_index,
    const int32_t* __restrict__ vidx, int i0, int rows, bool vec, double2* __restrict__ acc) {
  using C = typename Cx<R>::T;
  extern __shared__ unsigned char smem[];
  double2* bs = reinterpret_cast<double2*>(smem);
  C* D = reinterpret_cast<C*>(bs + TS_TILES * TS_B);
  C* xs = D + 2 * TS_B * TS_DLD;
  C* sums = xs + TS_TILES * TS_B;
  // vector group: blockIdx / n_rhs, or the vidx entry when a subset is solved,
  // with factor set fac_index[mat] (identity if NULL)
  const int mat = vidx ? vidx[blockIdx.x / n_rhs] : blockIdx.x / n_rhs;
  const int fac = fac_index ? fac_index[mat] : mat;
  const int64_t off = (int64_t)mat * bstride + (int64_t)(blockIdx.x % n_rhs) * n;
  const C* Lb = LU + (int64_t)fac * stride;
  if (threadIdx.x < TS_TILES * TS_B) {
    const int i = threadIdx.x;
    double2 b = make_double2(0.0, 0.0);
    if (i < rows) {
      if (!WHOLE && acc) {
        b = acc[(int64_t)blockIdx.x * n + i0 + i];
      } else {
        const C v = WHOLE ? Bin[off + perm[(int64_t)fac * n + i]] : X[off + i0 + i];
        b = make_double2(v.x, v.y);
      }
    }
    bs[i] = b;
    xs[i] = cmk<C>(R(0), R(0));
  }
  if (WHOLE) {
    trsv_block<R, true>(Lb, ld, 0, rows, vec, bs, D, xs, sums);
    trsv_block<R, false>(Lb, ld, 0, rows, vec, bs, D, xs, sums);
  } else {
    trsv_block<R, FWD>(Lb, ld, i0, rows, vec, bs, D, xs, sums);
  }
  if ((int)threadIdx.x < rows) {
    const C v = xs[threadIdx.x];
    X[off + i0 + threadIdx.x] = v;
    // (what the solve with U starts from)
    if (!WHOLE && FWD && acc) acc[(int64_t)blockIdx.x * n + i0 + threadIdx.x] = make_double2(v.x, v.y);
  }
}

// acc = P B, or X = P B
template <typename C>
__global__ void trsv_permute_kernel(int n, const int32_t* __restrict__ perm, int n_rhs,
                                    const C* __restrict__ Bin, C* __restrict__ X, int64_t bstride,
                                    const int32_t* __restrict__ fac_index,
                                    const int32_t* __restrict__ vidx, double2* __restrict__ acc) {
  const int i = blockIdx.y * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int mat = vidx ? vidx[blockIdx.x / n_rhs] : blockIdx.x / n_rhs;
  const int fac = fac_index ? fac_index[mat] : mat;
  const int64_t off = (int64_t)mat * bstride + (int64_t)(blockIdx.x % n_rhs) * n;
  const C v = Bin[off + perm[(int64_t)fac * n + i]];
  if (acc) acc[(int64_t)blockIdx.x * n + i] = make_double2(v.x, v.y);
  else X[off + i] = v;
}

// V[rows] -= LU[rows, c0 .. c0 + cols) X[c0 .. c0 + cols) for the rows [ra, rb),
// NR right-hand sides at once; V = acc, its matrices acc_stride apart, or X.  A wave takes 16 / NR rows, its lanes the columns
// (16-byte words); the 32 sums of a wave are reduced by recursive halving (32
// shuffles).
template <typename R, int NR>
__global__ __launch_bounds__(256) void trsv_update_kernel(
    int n, int64_t ld, int64_t stride, const typename Cx<R>::T* __restrict__ LU, int n_rhs,
    typename Cx<R>::T* __restrict__ X, int64_t bstride, const int32_t* __restrict__ fac_index,
    const int32_t* __restrict__ vidx, int ra, int rb, int c0, int cols, bool vec,
    double2* __restrict__ acc, int64_t acc_stride) {
  using C = typename Cx<R>::T;
  constexpr int RPW = 16 / NR, PER = 16 / (int)sizeof(C), CW = 64 * PER;   // columns of a step
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int mat = vidx ? vidx[blockIdx.y] : blockIdx.y;
  const int fac = fac_index ? fac_index[mat] : mat;
  const int rh0 = blockIdx.z * NR, nrh = min(NR, n_rhs - rh0);
  const int r0 = ra + (blockIdx.x * 4 + wid) * RPW;
  if (r0 >= rb) return;
  const C* Lb = LU + (int64_t)fac * stride + c0;
  C* x = X + (int64_t)mat * bstride + (int64_t)rh0 * n;
  R v[RPW][NR][2];
#pragma unroll
  for (int i = 0; i < RPW; ++i)
#pragma unroll
    for (int r = 0; r < NR; ++r) v[i][r][0] = v[i][r][1] = R(0);
  for (int j0 = 0; j0 < cols; j0 += CW) {
    const int j = j0 + PER * lane;
    C xv[NR][PER];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const C t = x[(int64_t)min(r, nrh - 1) * n + c0 + min(j + u, cols - 1)];
        xv[r][u] = j + u < cols ? t : cmk<C>(R(0), R(0));
      }
    // every row's word before the first is used
    C l[RPW][PER];
    const bool whole = vec && j0 + CW <= cols;   // uniform
    if (whole) {
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        const uint4 w = *reinterpret_cast<const uint4*>(Lb + (int64_t)min(r0 + i, rb - 1) * ld + j);
        __builtin_memcpy(l[i], &w, 16);
      }
    } else {
#pragma unroll
      for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const C t = Lb[(int64_t)min(r0 + i, rb - 1) * ld + min(j + u, cols - 1)];
          l[i][u] = j + u < cols ? t : cmk<C>(R(0), R(0));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          v[i][r][0] = fma(l[i][u].x, xv[r][u].x, fma(-l[i][u].y, xv[r][u].y, v[i][r][0]));
          v[i][r][1] = fma(l[i][u].x, xv[r][u].y, fma(l[i][u].y, xv[r][u].x, v[i][r][1]));
        }
  }
  // values e = (row, rhs, part): after the halvings lanes 2 e and 2 e + 1 hold e
  R h[32];
#pragma unroll
  for (int e = 0; e < 32; ++e) h[e] = v[e / (2 * NR)][(e / 2) % NR][e % 2];
#pragma unroll
  for (int s = 32, m = 16; m >= 1; s >>= 1, m >>= 1) {
    const bool up = lane & s;
#pragma unroll
    for (int e = 0; e < m; ++e) {
      const R keep = up ? h[m + e] : h[e], give = up ? h[e] : h[m + e];
      h[e] = keep + __shfl_xor(give, s, 64);
    }
  }
  h[0] += __shfl_xor(h[0], 1, 64);
  const int e = lane >> 1, i = e / (2 * NR), r = (e / 2) % NR;
  if (!(lane & 1) && r0 + i < rb && r < nrh) {
    if (acc) {
      double2* a = acc + blockIdx.y * acc_stride + (int64_t)(rh0 + r) * n + r0 + i;
      reinterpret_cast<double*>(a)[e & 1] -= h[0];
    } else {
      R* dst = reinterpret_cast<R*>(x + (int64_t)r * n + r0 + i) + (e & 1);
      *dst -= h[0];
    }
  }
}

// One workgroup (8 waves) per (matrix, right-hand side): X = U^{-1} L^{-1} P B,
// processed in blocks of 64 rows.  For each block, the 64 x 64 diagonal block
// is staged in LDS while the waves form the off-diagonal dot products (row-major
// rows against the solved part of x, coalesced), then one wave substitutes
// through the diagonal block from LDS.  x lives in LDS.
constexpr int SW_B = 64;
constexpr int SW_T = 512;
size_t sweep_lds(size_t esz, int n) { return esz * (size_t)(SW_B * (SW_B + 1) + SW_B + n); }

template <typename R>
__global__ __launch_bounds__(SW_T) void trsv_sweep_kernel(int n, int64_t ld, int64_t stride,
                                                     const typename Cx<R>::T* LU,
                                                     const int32_t* perm, int n_rhs,
                                                     const typename Cx<R>::T* Bin,
                                                     typename Cx<R>::T* X, int64_t bstride,
                                                     const int32_t* fac_index,
                                                     const int32_t* vidx) {
  using C = typename Cx<R>::T;
  extern __shared__ unsigned char smem[];
  C* D = reinterpret_cast<C*>(smem);                 // [SW_B][SW_B + 1]
  C* part = D + SW_B * (SW_B + 1);                   // [SW_B]
  C* x = part + SW_B;                                // [n]
  // vector group: blockIdx / n_rhs, or the vidx entry when a subset is solved
  const int mat = vidx ? vidx[blockIdx.x / n_rhs] : blockIdx.x / n_rhs;
  const int rhs = blockIdx.x % n_rhs;
  // vector group `mat` is solved with factor set fac_index[mat] (identity if NULL)
  const int fac = fac_index ? fac_index[mat] : mat;
  const C* Lb = LU + (int64_t)fac * stride;
  const int32_t* pb = perm + (int64_t)fac * n;
  const C* bin = Bin + (int64_t)mat * bstride + (int64_t)rhs * n;
  C* xg = X + (int64_t)mat * bstride + (int64_t)rhs * n;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  constexpr int NW = SW_T / 64;
  for (int i = tid; i < n; i += SW_T) x[i] = bin[pb[i]];
  __syncthreads();
  const int nb = (n + SW_B - 1) / SW_B;
  // every off-diagonal range starts at an even column (0, or a multiple of 64)
  const bool vec2 = sizeof(C) == 8 && ((ld | stride) & 1) == 0 && ((uintptr_t)LU & 15) == 0;
  for (int pass = 0; pass < 2; ++pass) {
    const bool fwd = pass == 0;
    for (int step = 0; step < nb; ++step) {
      const int I = fwd ? step : nb - 1 - step;
      const int i0 = I * SW_B, rows = min(SW_B, n - i0);
      // stage the diagonal block
      for (int e = tid; e < rows * SW_B; e += SW_T) {
        const int r = e / SW_B, c = e % SW_B;
        if (c < rows) D[r * (SW_B + 1) + c] = Lb[(int64_t)(i0 + r) * ld + i0 + c];
      }
      // off-diagonal dot products: forward uses columns [0, i0), backward [i0+rows, n)
      const int jlo = fwd ? 0 : i0 + rows, jhi = fwd ? i0 : n;
      for (int rr = wid; rr < rows; rr += NW) {
        const C* Li = Lb + (int64_t)(i0 + rr) * ld;
        R sr = 0, si = 0, sr2 = 0, si2 = 0;
        if (vec2) {
          // complex float rows with even ld and start: each lane takes pairs of
          // elements as 16-byte words, two pairs per iteration
          int j = jlo + 2 * lane;
          for (; j + 129 < jhi; j += 256) {
            const float4 la = *reinterpret_cast<const float4*>(Li + j);
            const float4 lb = *reinterpret_cast<const float4*>(Li + j + 128);
            const C a0 = x[j], a1 = x[j + 1], b0 = x[j + 128], b1 = x[j + 129];
            sr += (la.x * a0.x - la.y * a0.y) + (la.z * a1.x - la.w * a1.y);
            si += (la.x * a0.y + la.y * a0.x) + (la.z * a1.y + la.w * a1.x);
            sr2 += (lb.x * b0.x - lb.y * b0.y) + (lb.z * b1.x - lb.w * b1.y);
            si2 += (lb.x * b0.y + lb.y * b0.x) + (lb.z * b1.y + lb.w * b1.x);
          }
          for (; j + 1 < jhi; j += 128) {
            const float4 la = *reinterpret_cast<const float4*>(Li + j);
            const C a0 = x[j], a1 = x[j + 1];
            sr += (la.x * a0.x - la.y * a0.y) + (la.z * a1.x - la.w * a1.y);
            si += (la.x * a0.y + la.y * a0.x) + (la.z * a1.y + la.w * a1.x);
          }
          if (j < jhi) {
            const C l0 = Li[j], v0 = x[j];
            sr += l0.x * v0.x - l0.y * v0.y;
            si += l0.x * v0.y + l0.y * v0.x;
          }
        } else {
          int j = jlo + lane;
          for (; j + 64 < jhi; j += 128) {
            const C l0 = Li[j], v0 = x[j], l1 = Li[j + 64], v1 = x[j + 64];
            sr += l0.x * v0.x - l0.y * v0.y;
            si += l0.x * v0.y + l0.y * v0.x;
            sr2 += l1.x * v1.x - l1.y * v1.y;
            si2 += l1.x * v1.y + l1.y * v1.x;
          }
          if (j < jhi) {
            const C l0 = Li[j], v0 = x[j];
            sr += l0.x * v0.x - l0.y * v0.y;
            si += l0.x * v0.y + l0.y * v0.x;
          }
        }
        sr += sr2;
        si += si2;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
          sr += __shfl_down(sr, off, 64);
          si += __shfl_down(si, off, 64);
        }
        if (lane == 0) part[rr] = cmk<C>(sr, si);
      }
      __syncthreads();
      if (wid == 0) {
        C v = cmk<C>(R(0), R(0));
        if (lane < rows) v = cmk<C>(x[i0 + lane].x - part[lane].x, x[i0 + lane].y - part[lane].y);
        if (fwd) {
          for (int c = 0; c < rows; ++c) {
            const R xr = __shfl(v.x, c, 64), xi = __shfl(v.y, c, 64);
            if (lane > c && lane < rows) v = csub(v, product(D[lane * (SW_B + 1) + c], cmk<C>(xr, xi)));
          }
        } else {
          const C dinv = lane < rows ? crecip(D[lane * (SW_B + 1) + lane]) : cmk<C>(R(1), R(0));
          for (int c = rows - 1; c >= 0; --c) {
            if (lane == c) v = product(v, dinv);
            const R xr = __shfl(v.x, c, 64), xi = __shfl(v.y, c, 64);
            if (lane < c) v = csub(v, product(D[lane * (SW_B + 1) + c], cmk<C>(xr, xi)));
          }
        }
        if (lane < rows) x[i0 + lane] = v;
      }
          __syncthreads();
    }
  }
  for (int i = tid; i < n; i += SW_T) xg[i] = x[i];
}

// Whether the sweep takes a solve.  It puts a workgroup on every vector, so it wins
// once the vectors fill the chip, whose compute units the launches by blocks leave
// between them; before that its one chain per vector costs more than their launches.
// ms by blocks against the sweep, float32, on 256 compute units:
//   n = 162    512 vectors 0.077 / 0.102    960  0.135 / 0.119   32000 3.58 / 2.83
//   n = 642    256         0.39 / 0.49      320  0.52 / 0.43     1024  0.93 / 0.51
//   n = 1284   256         0.83 / 0.92      320  1.52 / 1.20     1024  2.81 / 2.20
//   n = 5124   48          3.7 / 9.5        256  10.7 / 9.0      1024  40 / 18
// The float64 block kernels hold one workgroup per compute unit (their tiles fill the
// LDS), and win only where a vector's sweep is long:
//   n = 162    64 vectors  0.140 / 0.091                         4096  2.01 / 0.76
//   n = 642    64          0.60 / 0.57      320  1.17 / 0.63     1024  2.30 / 1.15
//   n = 1000   64          0.94 / 1.07      256  0.87 / 0.80
//   n = 1284   64          1.30 / 1.62      320  2.57 / 2.95     1024  5.05 / 5.53
// and with one right-hand side 256 matrices of 1284 take 2.2 / 1.8.
bool sweeps(const bem_ctx* ctx, bem_prec prec, int n, int batch, int n_rhs) {
  const int64_t vectors = (int64_t)batch * n_rhs, cus = ctx->num_cus;
  if (sweep_lds(prec == BEM_C128 ? 16 : 8, n) > 150 * 1024) return false;
  if (prec == BEM_C128) return n < 960 || (vectors >= cus && (n_rhs == 1 || n < 1200));
  if (n <= TS_TILES * TS_B) return vectors > (n > 2 * TS_B ? 3 * cus : cus);
  return n < 1536 ? 4 * vectors >= 5 * cus : vectors >= cus;
}

template <typename R>
void solve_go(bem_ctx* ctx, int n, int64_t ld, int64_t stride, int groups,
                    const void* LU_, const int32_t* perm, int n_rhs, const void* B_, void* X_,
                    int64_t bstride, const int32_t* fac_index, const int32_t* vidx, double2* acc) {
  using C = typename Cx<R>::T;
  const C* LU = (const C*)LU_;
  const C* B = (const C*)B_;
  C* X = (C*)X_;
  // 16-byte words: rows and blocks (starting at multiples of 64) all aligned
  const bool vec = sizeof(C) == 16 ? ((uintptr_t)LU & 15) == 0
                                   : ((ld | stride) & 1) == 0 && ((uintptr_t)LU & 15) == 0;
  const size_t lds = trsv_lds<C>();
  const dim3 bt(TS_T), vectors((unsigned)(groups * n_rhs));
  if constexpr (sizeof(R) == 4) if (n <= TS_TILES * TS_B) {   // (float64: sweeps)
    hipLaunchKernelGGL((trsv_block_kernel<R, true, true>), vectors, bt, lds, ctx->stream, n, ld,
                       stride, LU, perm, n_rhs, B, X, bstride, fac_index, vidx, 0, n, vec, acc);
    return;
  }
  hipLaunchKernelGGL(trsv_permute_kernel<C>, dim3(vectors.x, (n + 255) / 256), dim3(256), 0,
                     ctx->stream, n, perm, n_rhs, B, X, bstride, fac_index, vidx, acc);
  // blocks of TS_NB unknowns, the last with up to TS_TILES tiles
  const int nb = std::max(1, (n - TS_B + TS_NB - 1) / TS_NB);
  auto start = [&](int q) { return q * TS_NB; };
  auto rows = [&](int q) { return q + 1 < nb ? TS_NB : n - q * TS_NB; };
  auto update = [&](int ra, int rb, int q) {
    if (rb <= ra) return;
    auto go = [&](auto nr_c) {
      constexpr int NR = decltype(nr_c)::value, ZMAX = 65535 * NR;
      for (int z0 = 0; z0 < n_rhs; z0 += ZMAX) {
        const int nz = std::min(n_rhs - z0, ZMAX);
        hipLaunchKernelGGL((trsv_update_kernel<R, NR>),
                           dim3((rb - ra + 64 / NR - 1) / (64 / NR), groups, (nz + NR - 1) / NR),
                           dim3(256), 0, ctx->stream, n, ld, stride, LU, nz, X + (int64_t)z0 * n,
                           bstride, fac_index, vidx, ra, rb, start(q), rows(q), vec,
                           acc ? acc + (int64_t)z0 * n : nullptr, (int64_t)n_rhs * n);
      }
    };
    if (n_rhs == 1) go(std::integral_constant<int, 1>{});
    else if (n_rhs == 2) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 4>{});
  };
  for (int q = 0; q < nb; ++q) {
    hipLaunchKernelGGL((trsv_block_kernel<R, false, true>), vectors, bt, lds, ctx->stream, n, ld,
                       stride, LU, perm, n_rhs, B, X, bstride, fac_index, vidx, start(q), rows(q), vec, acc);
    update(start(q) + rows(q), n, q);
  }
  for (int q = nb - 1; q >= 0; --q) {
    hipLaunchKernelGGL((trsv_block_kernel<R, false, false>), vectors, bt, lds, ctx->stream, n, ld,
                       stride, LU, perm, n_rhs, B, X, bstride, fac_index, vidx, start(q), rows(q), vec, acc);
    update(0, start(q), q);
  }
}

}  // namespace

bem_status lu_perm(bem_ctx* ctx, int n, int batch, const int32_t* piv, int32_t* perm) {
  static bool attr_set = false;
  if (!attr_set) {
    hipFuncSetAttribute((const void*)perm_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                        160 * 1024);
    attr_set = true;
  }
  hipLaunchKernelGGL(perm_kernel, dim3(batch), dim3(64), sizeof(int32_t) * n, ctx->stream, n,
                     piv, perm);
  BEM_CHECK_LAUNCH(ctx);
  return BEM_OK;
}

size_t lu_solve_acc_bytes(const bem_ctx* ctx, bem_prec prec, int n, int batch, int n_rhs) {
  return prec == BEM_C64 && n > TS_TILES * TS_B && !sweeps(ctx, prec, n, batch, n_rhs)
             ? sizeof(double2) * (size_t)batch * n_rhs * n : 0;
}

bem_status lu_solve_perm(bem_ctx* ctx, bem_prec prec, int n, int64_t ld, int64_t stride,
                         int batch, const void* LU, const int32_t* perm, int n_rhs,
                         const void* Bin, void* X, int64_t bstride, double2* acc,
                         const int32_t* fac_index, const int32_t* vidx, int n_sel) {
  if (vidx) batch = n_sel;
  if (batch <= 0 || n_rhs <= 0) return BEM_OK;
  static bool attr_set = false;
  if (!attr_set) {
    auto big = [](const void* f) {
      hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    };
    big((const void*)trsv_sweep_kernel<float>);
    big((const void*)trsv_sweep_kernel<double>);
    big((const void*)trsv_block_kernel<float, true, true>);
    big((const void*)trsv_block_kernel<float, false, true>);
    big((const void*)trsv_block_kernel<float, false, false>);
    big((const void*)trsv_block_kernel<double, false, true>);
    big((const void*)trsv_block_kernel<double, false, false>);
    attr_set = true;
  }
  const size_t esz = prec == BEM_C128 ? 16 : 8;
  const int most = 65535;   // groups per launch (grid y)
  const int pi = prof_begin(ctx, "getrs");
  const double items = batch;
  const size_t lds = sweep_lds(esz, n);
  if (sweeps(ctx, prec, n, batch, n_rhs)) {
    const dim3 vectors((unsigned)(batch * n_rhs));
    if (prec == BEM_C128)
      hipLaunchKernelGGL((trsv_sweep_kernel<double>), vectors, dim3(SW_T), lds, ctx->stream, n, ld,
                         stride, (const double2*)LU, perm, n_rhs, (const double2*)Bin, (double2*)X,
                         bstride, fac_index, vidx);
    else
      hipLaunchKernelGGL((trsv_sweep_kernel<float>), vectors, dim3(SW_T), lds, ctx->stream, n, ld,
                         stride, (const float2*)LU, perm, n_rhs, (const float2*)Bin, (float2*)X,
                         bstride, fac_index, vidx);
    batch = 0;
  }
  for (int g0 = 0; g0 < batch; g0 += most) {
    const int g = std::min(most, batch - g0);
    // without an index list the slice is taken by moving the pointers
    const size_t vo = vidx ? 0 : (size_t)g0 * bstride * esz;
    const char* lu = (const char*)LU + (vidx || fac_index ? 0 : (size_t)g0 * stride * esz);
    const int32_t* pm = perm + (vidx || fac_index ? 0 : (size_t)g0 * n);
    const int32_t* fi = fac_index && !vidx ? fac_index + g0 : fac_index;
    const int32_t* vi = vidx ? vidx + g0 : nullptr;
    const char* b = (const char*)Bin + vo;
    char* x = (char*)X + vo;
    if (prec == BEM_C128)
      solve_go<double>(ctx, n, ld, stride, g, lu, pm, n_rhs, b, x, bstride, fi, vi, nullptr);
    else
      solve_go<float>(ctx, n, ld, stride, g, lu, pm, n_rhs, b, x, bstride, fi, vi,
                      acc ? acc + (size_t)g0 * n_rhs * n : nullptr);
  }
  prof_end(ctx, "getrs", pi, 8.0 * (double)n * n * n_rhs * items,
           (double)esz * ((double)n * n + 3.0 * n * n_rhs) * items);
  BEM_CHECK_LAUNCH(ctx);
  return BEM_OK;
}

}  // namespace bem

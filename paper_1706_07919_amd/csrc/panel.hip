// Panels of the batched LU: a few columns of every matrix factored by one
// workgroup per matrix with the whole panel in registers.
//
// What bounds a panel is the chain of its columns: largest entry, its row to
// everyone, reciprocal, rank-1 update, each waiting for the one before over the
// whole workgroup, on one compute unit.  Hence
//  - rows stay where they are and carry their position (an interchange is two
//    positions, and only the pivot row's active part is published);
//  - the largest entry of a wave comes from lane-permuting integer maxima (DPP)
//    of the entries' bits, and every wave publishes its candidate's row with the
//    value, so a column takes one barrier;
//  - nothing is stored to memory inside the chain;
//  - whole rows are loaded and stored as contiguous words, turned between lanes
//    in LDS (a row per lane touched every cache line once per 16 bytes: loads and
//    stores of 1000 rows of 32 columns took 44 000 cycles, now 31 000);
//  - panels are as wide as the registers allow, because every split of a block
//    of columns into narrower panels costs an interchange, a triangular solve,
//    an update and their launches;
//  - a column has one way through, also without a pivot, and the columns of a
//    partial panel run as empty ones: with branches around the update the
//    compiler copied and spilled the rows (5100 rows, 8 columns: 112 us, now 57).
// 32 columns of 256 rows take 37 us, of 1000 rows 62 us (89 with interchanged
// rows and a row per lane); the float32 panels of 21 matrices of n = 1284 take
// 2.1 ms (8 columns wide, two barriers and shuffled maxima: 3.2 ms, with 2.2
// times the launches between them), the whole solve 8.9 ms (11.9).
#include <utility>

#include "lu_types.h"

namespace bem {
namespace lud {
namespace {

// Non-negative values ordered as integers: a float's or a double's bits.
template <typename R> struct Key;
template <> struct Key<float> {
  using T = unsigned;
  static __device__ __forceinline__ T of(float v) { return __float_as_uint(v); }
};
template <> struct Key<double> {
  using T = unsigned long long;
  static __device__ __forceinline__ T of(double v) { return __builtin_bit_cast(T, v); }
};

template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned dpp_max(unsigned v) {
  return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false));
}
// largest of the first 16 lanes' values, and of a wave's (uniform)
__device__ __forceinline__ unsigned max_of_16(unsigned v) {
  v = dpp_max<0x111, 0xf>(v);   // row_shr:1, 2, 4, 8: lane 15 of a row of 16 has its largest
  v = dpp_max<0x112, 0xf>(v);
  v = dpp_max<0x114, 0xf>(v);
  v = dpp_max<0x118, 0xf>(v);
  return __builtin_amdgcn_readlane((int)v, 15);
}
__device__ __forceinline__ unsigned wave_max(unsigned v) {
  v = dpp_max<0x111, 0xf>(v);
  v = dpp_max<0x112, 0xf>(v);
  v = dpp_max<0x114, 0xf>(v);
  v = dpp_max<0x118, 0xf>(v);
  v = dpp_max<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v = dpp_max<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return __builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ unsigned long long max_of_16(unsigned long long v) {
  const unsigned hi = max_of_16((unsigned)(v >> 32));
  return (unsigned long long)hi << 32 | max_of_16((unsigned)(v >> 32) == hi ? (unsigned)v : 0u);
}
__device__ __forceinline__ unsigned long long wave_max(unsigned long long v) {
  const unsigned hi = wave_max((unsigned)(v >> 32));
  return (unsigned long long)hi << 32 | wave_max((unsigned)(v >> 32) == hi ? (unsigned)v : 0u);
}
// of the lanes in mask (not empty) the one with the smallest idx; idx of it in out
__device__ __forceinline__ int first_row(unsigned long long mask, int idx, int& out) {
  int l = __ffsll(mask) - 1;
  out = __builtin_amdgcn_readlane(idx, l);
  mask &= mask - 1;
  while (mask) {   // ties
    const int l2 = __ffsll(mask) - 1;
    const int o2 = __builtin_amdgcn_readlane(idx, l2);
    if (o2 < out) {
      out = o2;
      l = l2;
    }
    mask &= mask - 1;
  }
  return l;
}
template <typename F, int... I>
__device__ __forceinline__ void each(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
// copy by parts (struct copies of float64 rows keep the array out of registers)
template <typename C>
__device__ __forceinline__ void put(C& d, const C& v) {
  d.x = v.x;
  d.y = v.y;
}
// 1/a: float32 through float64 (no overflow, one rounding; shorter than two
// float32 divisions), float64 by Smith's method; with one infinite part 0, as
// Smith's method has it
__device__ inline float2 recip(float2 a) {
  const double x = a.x, y = a.y, d = fma(x, x, y * y);
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  const bool inf = __builtin_isinf(a.x) != __builtin_isinf(a.y);
  return make_float2(inf ? 0.f : (float)(x * r), inf ? 0.f : (float)(-y * r));
}
__device__ inline double2 recip(double2 a) { return crecip(a); }

// Factor columns [c0, c0+w) of rows [c0, n) in place; w <= W.  Thread t owns
// rows c0 + t + q*NT (q < RPT).  Pivot = max |re|+|im| (lowest row on ties).
template <typename R, int W, int RPT, int NT>
__global__ __launch_bounds__(NT) void panel_kernel(LuGroups G, int c0, int w_all) {
  using C = typename Cx<R>::T;
  using K = typename Key<R>::T;
  constexpr int NW = NT / 64;
  constexpr int PER = 16 / sizeof(C);   // complex values per 16-byte word
  constexpr int WORDS = W / PER;        // words per row; RW rows per load of a wave
  constexpr int RW = 64 / WORDS;
  constexpr int PITCH = WORDS + 1;      // of a row in LDS: odd, so rows spread over the banks
  static_assert(NW <= 16, "the waves' candidates are compared in 16 lanes");
  static_assert(64 % WORDS == 0 && RPT <= 16, "rows per load; slots are bits");
  // double-buffered by column parity: a column's readers never race the next
  // column's writers, and the barrier of the next column is behind them when
  // the buffer is written again
  __shared__ C cand[2][NW][W];
  __shared__ K rv[2][16];
  __shared__ int ri[2][16];
  __shared__ int rows_of[W];
  __shared__ C zeros[W];
  __shared__ C fin[W][W];   // finished rows: the pivot and what lies right of it
  // rows on their way between memory and their lanes, each wave's own (the LDS
  // accesses of a wave complete in order)
  __shared__ __align__(16) uint4 turn[NW][64 * PITCH];
  __shared__ int dest[NW][64];
  LuGroup grp;
  int b = 0;
  if (!locate(G, blockIdx.x, grp, b)) return;
  const int n = grp.n;
  const int64_t ld = grp.ld;
  if (c0 >= n) return;
  const int w = min(w_all, n - c0);
  GLOBAL C* Ab = gmat<C>(grp, b);
  GLOBAL int32_t* piv = (GLOBAL int32_t*)grp.piv;
  GLOBAL int32_t* info = (GLOBAL int32_t*)grp.info;
  const int t = threadIdx.x;
  const int lane = t & 63, wid = __builtin_amdgcn_readfirstlane(t >> 6);
  if (t < W) zeros[t] = cmk<C>(R(0), R(0));
  if (t < 16) {   // slots of waves that are not there
    rv[0][t] = rv[1][t] = 0;
    ri[0][t] = ri[1][t] = 0x7fffffff;
  }
  __syncthreads();
  C a[RPT][W];
  // full-width panels with 16-byte aligned rows move as words, others value by
  // value; rows past n hold a copy of the last one (they are never looked at)
  const bool vec = w == W && (sizeof(C) == 16 || ((ld | c0) & 1) == 0);
  uint4* const mine = turn[wid];
  C* const vals = (C*)mine;
  const int sub = lane / WORDS, word = lane % WORDS;
  const int first = c0 + wid * 64;
  if (vec)
#pragma unroll
    for (int q = 0; q < RPT; ++q)
#pragma unroll
      for (int m = 0; m < WORDS; ++m) {
        const int r = min(first + q * NT + m * RW + sub, n - 1);
        const uint4 x = ((const GLOBAL uint4*)(Ab + r * ld + c0))[word];
        C e[PER];
        __builtin_memcpy(e, &x, 16);
#pragma unroll
        for (int u = 0; u < PER; ++u) put(a[q][m * PER + u], e[u]);
      }
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    if (vec) {
#pragma unroll
      for (int m = 0; m < WORDS; ++m)
#pragma unroll
        for (int u = 0; u < PER; ++u)
          put(vals[((m * RW + sub) * PITCH + word) * PER + u], a[q][m * PER + u]);
    } else {
#pragma unroll
      for (int m = 0; m < W; ++m) {
        const int i = m * (64 / W) + lane / W, c = lane % W;
        const int r = min(first + q * NT + i, n - 1);
        const C e = Ab[r * ld + c0 + min(c, w - 1)];
        put(vals[i * PITCH * PER + c], c < w ? e : cmk<C>(R(0), R(0)));
      }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int c = 0; c < W; ++c) put(a[q][c], vals[lane * PITCH * PER + c]);
    __builtin_amdgcn_wave_barrier();
  }
  int pos[RPT];   // where the row now belongs; -1: no row
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int r = c0 + t + q * NT;
    pos[q] = r < n ? r : -1;
  }
  int bad = 0;   // first column without a pivot, from 1
  // The columns are instantiated one by one so that every register index is static.
  auto column = [&](auto ic) __attribute__((always_inline)) {
    constexpr int c = decltype(ic)::value;
    const int pr = c0 + c;
    constexpr int buf = c & 1;
    // candidate of this thread, then of its wave, published with its row (a
    // column of zeros or NaN has none)
    R best = R(0);
    int brow = 0x7fffffff, bslot = 0;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const R m = fabs(a[q][c].x) + fabs(a[q][c].y);
      if (pos[q] >= pr && (m > best || (m == best && m > R(0) && pos[q] < brow))) {
        best = m;
        brow = pos[q];
        bslot = 1 << q;
      }
    }
    const K key = Key<R>::of(best);
    const K wkey = wave_max(key);
    int wrow = 0x7fffffff;
    if (wkey) {   // uniform
      const int wl = first_row(__ballot(key == wkey), brow, wrow);
      const int slot = __builtin_amdgcn_readlane(bslot, wl);
#pragma unroll
      for (int q = 0; q < RPT; ++q)
        if (((slot >> q) & 1) && lane == wl)
#pragma unroll
          for (int cc = c; cc < W; ++cc) put(cand[buf][wid][cc], a[q][cc]);
    }
    if (lane == 0) {
      rv[buf][wid] = wkey;
      ri[buf][wid] = wrow;
    }
    __syncthreads();
    const K v16 = rv[buf][lane & 15];
    const int i16 = ri[buf][lane & 15];
    const K top = max_of_16(v16);
    // without a pivot (or past a partial panel): no interchange, and the update
    // runs with l = u = 0, so that the registers have one way through the column
    const bool none = !top;
    int p = pr;
    const int ws = none ? 0 : first_row(__ballot(v16 == top) & 0xffff, i16, p);
    if (t == 0) rows_of[c] = p;
    if (none) {
      if (!bad && c < w) bad = pr + 1;
#pragma unroll
      for (int q = 0; q < RPT; ++q)
        if (pos[q] == pr)
#pragma unroll
          for (int cc = c; cc < W; ++cc) put(fin[c][cc], a[q][cc]);
    } else if (wid == NW - 1 && lane >= c && lane < W) {
      put(fin[c][lane], cand[buf][ws][lane]);
    }
    const C* prow = none ? zeros : cand[buf][ws];
    C u[W];
#pragma unroll
    for (int cc = c; cc < W; ++cc) put(u[cc], prow[cc]);
    const C inv = recip(u[c]);
    // every row is updated, finished ones too: what is theirs right of their
    // pivot is in fin, what is left of it stays
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const int old = pos[q];
      pos[q] = old == p ? pr : old == pr ? p : old;
      const C m = cmul(a[q][c], inv);
      const C l = cmk<C>(none ? R(0) : m.x, none ? R(0) : m.y);
      a[q][c].x = none ? a[q][c].x : m.x;
      a[q][c].y = none ? a[q][c].y : m.y;
#pragma unroll
      for (int cc = c + 1; cc < W; ++cc) {
        // the product first, then one rounding of the entry
        const C d = cmk<C>(fma(l.x, u[cc].x, -(l.y * u[cc].y)), fma(l.x, u[cc].y, l.y * u[cc].x));
        put(a[q][cc], csub(a[q][cc], d));
      }
    }
  };
  each(column, std::make_integer_sequence<int, W>{});
  __syncthreads();
  if (t < w) piv[(int64_t)b * n + c0 + t] = rows_of[t];
  if (t == 0 && bad && info[b] == 0) info[b] = bad;
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
#pragma unroll
    for (int c = 0; c < W; ++c) put(vals[lane * PITCH * PER + c], a[q][c]);
    dest[wid][lane] = pos[q];
    __builtin_amdgcn_wave_barrier();
    if (vec) {
#pragma unroll
      for (int m = 0; m < WORDS; ++m) {
        const int r = dest[wid][m * RW + sub];
        uint4 x = mine[(m * RW + sub) * PITCH + word];
        const int f = r - c0;
        if (r >= 0 && f < W && word * PER + PER > f) {   // a finished row
          C e[PER];
          __builtin_memcpy(e, &x, 16);
#pragma unroll
          for (int u = 0; u < PER; ++u)
            if (word * PER + u >= f) put(e[u], fin[f][word * PER + u]);
          __builtin_memcpy(&x, e, 16);
        }
        if (r >= 0) ((GLOBAL uint4*)(Ab + r * ld + c0))[word] = x;
      }
    } else {
#pragma unroll
      for (int m = 0; m < W; ++m) {
        const int i = m * (64 / W) + lane / W, c = lane % W;
        const int r = dest[wid][i], f = r - c0;
        C e;
        put(e, vals[i * PITCH * PER + c]);
        if (r >= 0 && c < w) {
          if (f < w && c >= f) put(e, fin[f][c]);
          Ab[r * ld + c0 + c] = e;
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

template <typename R, int W, int RPT, int NT>
void go(bem_ctx* ctx, const LuGroups& G, int total, int c0, int w) {
  hipLaunchKernelGGL((panel_kernel<R, W, RPT, NT>), dim3(total), dim3(NT), 0, ctx->stream, G, c0, w);
}

}  // namespace

// Widest panel whose rows and pivot row (2 or 4 registers a value) fit the 256
// registers of a thread of 512, or the 128 of one of 1024, with at most a few
// spilled: 16 columns of 1284 rows take 34 us where two panels of 8 take 2 x 17
// and what lies between them; past 5632 rows 4 columns of 10242 rows take 73 us,
// 2 take 47.
int panel_width(bem_prec prec, int rows) {
  if (prec == BEM_C128) return rows <= 1024 ? 16 : rows <= 2560 ? 8 : rows <= 5120 ? 4 : 2;
  return rows <= 1024 ? 32 : rows <= 2560 ? 16 : rows <= 5632 ? 8 : 4;
}

void launch_panel(bem_ctx* ctx, bem_prec prec, const LuGroups& G, int total, int rows, int c0, int w) {
  const int rpt = (rows + 511) / 512;
  if (prec == BEM_C128) {
    if (rows <= 256) go<double, 16, 1, 256>(ctx, G, total, c0, w);
    else if (rpt <= 1) go<double, 16, 1, 512>(ctx, G, total, c0, w);
    else if (rpt <= 2) go<double, 16, 2, 512>(ctx, G, total, c0, w);
    else if (rpt <= 3) go<double, 8, 3, 512>(ctx, G, total, c0, w);
    else if (rpt <= 4) go<double, 8, 4, 512>(ctx, G, total, c0, w);
    else if (rpt <= 5) go<double, 8, 5, 512>(ctx, G, total, c0, w);
    else if (rpt <= 6) go<double, 4, 6, 512>(ctx, G, total, c0, w);
    else if (rpt <= 8) go<double, 4, 8, 512>(ctx, G, total, c0, w);
    else if (rpt <= 10) go<double, 4, 10, 512>(ctx, G, total, c0, w);
    else if (rpt <= 12) go<double, 2, 12, 512>(ctx, G, total, c0, w);
    else go<double, 2, 12, 1024>(ctx, G, total, c0, w);
  } else {
    if (rows <= 256) go<float, 32, 1, 256>(ctx, G, total, c0, w);
    else if (rows <= 512) go<float, 32, 2, 256>(ctx, G, total, c0, w);
    else if (rpt <= 2) go<float, 32, 2, 512>(ctx, G, total, c0, w);
    else if (rpt <= 3) go<float, 16, 3, 512>(ctx, G, total, c0, w);
    else if (rpt <= 4) go<float, 16, 4, 512>(ctx, G, total, c0, w);
    else if (rpt <= 5) go<float, 16, 5, 512>(ctx, G, total, c0, w);
    else if (rpt <= 6) go<float, 8, 6, 512>(ctx, G, total, c0, w);
    else if (rpt <= 8) go<float, 8, 8, 512>(ctx, G, total, c0, w);
    else if (rpt <= 10) go<float, 8, 10, 512>(ctx, G, total, c0, w);
    else if (rpt <= 11) go<float, 8, 11, 512>(ctx, G, total, c0, w);
    else if (rpt <= 12) go<float, 4, 6, 1024>(ctx, G, total, c0, w);
    else if (rpt <= 16) go<float, 4, 8, 1024>(ctx, G, total, c0, w);
    else if (rpt <= 22) go<float, 4, 11, 1024>(ctx, G, total, c0, w);
    else go<float, 4, 12, 1024>(ctx, G, total, c0, w);
  }
}

}  // namespace lud
}  // namespace bem

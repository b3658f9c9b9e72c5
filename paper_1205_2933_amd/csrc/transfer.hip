// Restrictor R, prolongator P and the block orthonormalisation of the basis.
//
// Paper, Sec. 1: R maps fine to coarse vectors, P back, with R P = 1 on the
// coarse space.  Sec. 2: the near-null vectors are cut into blocks, one per
// coarse site, and every block spans the whole fifth dimension.  With the
// basis orthonormal on every (block, chirality) panel, R = P^+ and R P = 1.
//
// Basis storage: Nv fine fields in the internal fine layout; column
// (B, chi, k) is field k restricted to block B and to the spins of chi
// (chi = 0: spins 0,1; chi = 1: spins 2,3).
#include <algorithm>
#include <type_traits>

#include "mg_internal.h"
#include "blas.h"
#include "rules.h"

namespace mgdwf {

namespace {

struct BlockArgs {
  int L[4];
  int Ls;
  int V4;
  int V5;
  int b[4];
  int Lc[4];
  int Vc;
  int bvol;
  int Nv;
  int nsplit;  // workgroups per coarse site in R
};

BlockArgs make_args(const Geometry& g, const CoarseGeometry& cg) {
  BlockArgs a;
  for (int m = 0; m < 4; ++m) { a.L[m] = g.L[m]; a.b[m] = cg.block[m]; a.Lc[m] = cg.Lc[m]; }
  a.Ls = g.Ls; a.V4 = g.V4; a.V5 = g.V5; a.Vc = cg.Vc; a.bvol = cg.bvol; a.Nv = cg.Nv;
  a.nsplit = 4;
  return a;
}

// 4D site of the j-th site (block-local lexicographic, x fastest) of coarse site B.
__device__ __forceinline__ int block_site(const BlockArgs& a, int B, int j) {
  int X = B % a.Lc[0]; int r = B / a.Lc[0];
  int Y = r % a.Lc[1]; r /= a.Lc[1];
  int Z = r % a.Lc[2]; int T = r / a.Lc[2];
  int xx = j % a.b[0]; int q = j / a.b[0];
  int yy = q % a.b[1]; q /= a.b[1];
  int zz = q % a.b[2]; int tt = q / a.b[2];
  int x = X * a.b[0] + xx, y = Y * a.b[1] + yy, z = Z * a.b[2] + zz, t = T * a.b[3] + tt;
  return ((t * a.L[2] + z) * a.L[1] + y) * a.L[0] + x;
}

__device__ __forceinline__ int coarse_of(const BlockArgs& a, int x4) {
  int x = x4 % a.L[0]; int r = x4 / a.L[0];
  int y = r % a.L[1]; r /= a.L[1];
  int z = r % a.L[2]; int t = r / a.L[2];
  return ((t / a.b[3] * a.Lc[2] + z / a.b[2]) * a.Lc[1] + y / a.b[1]) * a.Lc[0] + x / a.b[0];
}

constexpr int KC = 8;      // basis vectors per register chunk in R

// Partial restriction: workgroup (B, split) sums its share of block B for
// every (chi, k): partial[((rhs * Vc + B) * a.nsplit + split) * 2 * n2 + ...].
template <class C2>
__global__ __launch_bounds__(256) void k_restrict(const C2* __restrict__ V, const C2* __restrict__ x,
                                                  double* __restrict__ partial, BlockArgs a) {
  const int B = blockIdx.x / a.nsplit, split = blockIdx.x % a.nsplit;
  const int rhs = blockIdx.y;
  const long long V5 = a.V5;
  const long long field = 12 * V5;
  x += rhs * field;
  const int n5 = a.bvol * a.Ls;
  const int n2 = 2 * a.Nv;
  double* out = partial + (((long long)rhs * a.Vc + B) * a.nsplit + split) * 2 * n2;
  __shared__ double red[4][2 * KC * 2];
  for (int k0 = 0; k0 < a.Nv; k0 += KC) {
    double acc[2][KC][2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int kk = 0; kk < KC; ++kk) { acc[h][kk][0] = 0.0; acc[h][kk][1] = 0.0; }
    for (int j = split * 256 + threadIdx.x; j < n5; j += 256 * a.nsplit) {
      const int jl = j / a.Ls, s = j - jl * a.Ls;
      const long long i5 = (long long)block_site(a, B, jl) * a.Ls + s;
      C2 xv[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) xv[c] = x[c * V5 + i5];
#pragma unroll
      for (int kk = 0; kk < KC; ++kk) {
        const int k = k0 + kk;
        if (k < a.Nv) {
          const C2* Vk = V + (long long)k * field;
#pragma unroll
          for (int c = 0; c < 12; ++c) {
            C2 v = Vk[c * V5 + i5];
            const int h = c / 6;
            acc[h][kk][0] += (double)v.x * xv[c].x + (double)v.y * xv[c].y;
            acc[h][kk][1] += (double)v.x * xv[c].y - (double)v.y * xv[c].x;
          }
        }
      }
    }
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int kk = 0; kk < KC; ++kk)
#pragma unroll
        for (int ri = 0; ri < 2; ++ri) {
          double v = wave_sum(acc[h][kk][ri]);
          if (l == 0) red[w][(h * KC + kk) * 2 + ri] = v;
        }
    __syncthreads();
    if (threadIdx.x < 2 * KC * 2) {
      const int h = threadIdx.x / (2 * KC), kk = (threadIdx.x / 2) % KC, ri = threadIdx.x & 1;
      const int k = k0 + kk;
      double s = red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
      if (k < a.Nv) out[(h * a.Nv + k) * 2 + ri] = s;
    }
    __syncthreads();
  }
}

// Multi-RHS restriction on MFMA: the contraction conj(V_k) x_r over a block's
// rows, chirality by chirality, is a matrix product with the basis columns as
// tile rows (KT tiles of 16) and the right-hand sides as tile columns, eight to
// a tile, Re and Im next to each other: with A = Re V against (Re x | Im x)
// and A = Im V against (Im x | -Re x) the tile holds (Re | Im) of the result.
// The basis is read once per 8 NT <= 32 right-hand sides and the sums need no
// registers per lane and right-hand side, which is what held the VALU forms to
// two (FP64) or twelve (FP32) at a time.  A workgroup's four wavefronts take
// (chirality, half of the split's rows).  A lane loads 16 U bytes of consecutive
// s: with U = 2 (Ls a multiple of 2 in FP64, 4 in FP32) the four lanes of a column
// read a whole 128-byte line; with U = 1 half lines, whose other half is often
// out of the cache when its turn comes (12 FP32 right-hand sides on 16^3x32x16:
// 1.87 against 2.48 ms with FP32 tiles).  FP32 rows are widened and go through the
// same FP64 tiles: the matrix rate is spare (FP32 tiles 1.88 ms, FP64 1.97 on that
// case) and the sums are exact to the inputs' rounding (4.4e-8 against 64 bits,
// 8.6e-8 to 2.0e-7 in the VALU form).  FP64 rows are added with a compensated sum
// every 8 products (every 8 U with four column tiles or more than four tiles, whose
// registers allow one wavefront per SIMD): 1.5e-16 to 1.8e-16 against 80 bits, where
// plain chains over a row group had 2.7e-16 to 3.9e-16 in the same time and the VALU
// form has 1.7e-16 to 2.5e-16; its serial Gram pass leaves a basis 1.1e-15 to 4.6e-15
// from orthonormal, this one 2e-16.  Bound by HBM (3.8 TB/s, read once) at few
// right-hand sides, by the FP64 matrix rate at many.  Against the VALU forms, 24
// columns: 12 FP32 right-hand sides on 16^3x32x16 3.12 -> 1.97 ms, on 8^3x16x16 365 ->
// 130 us; FP64 on 8^3x16x16, nine 1071 us -> 27 in 362 us, four 430 -> 192 us.
// Same partial layout as k_restrict.
typedef double rd4 __attribute__((ext_vector_type(4)));

template <class C2, int KT, int NT, int U>
__global__ __launch_bounds__(256, sizeof(C2) == 16 && KT == 2 && NT <= 2 ? 2 : 1)
void k_restrict_mfma(const C2* __restrict__ V, const C2* __restrict__ x, double* __restrict__ partial, BlockArgs a,
                     int nrhs) {
  using T = typename real_of<C2>::type;
  constexpr bool F64 = sizeof(T) == 8;
  constexpr int W1 = F64 ? 1 : 2;  // consecutive s in 16 bytes
  constexpr int W = W1 * U;        // and per lane
  constexpr int CH = (KT + NT) * U <= 4 ? 3 : 1;  // spin-colour components per pipeline stage
  __shared__ double red[2][KT * 16][NT * 16 + 1];
  const int B = blockIdx.x / a.nsplit, split = blockIdx.x % a.nsplit;
  const int r0 = blockIdx.y * 8 * NT;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), chi = w & 1, half = w >> 1;
  const int l = threadIdx.x & 63, col = l & 15, q = l >> 4;
  const bool im = col & 1;
  const long long V5 = a.V5, field = 12 * V5;
  const int n5 = a.bvol * a.Ls;
  const int ngrp = (n5 + 4 * W - 1) / (4 * W);
  const int per = (ngrp + 2 * a.nsplit - 1) / (2 * a.nsplit);
  const int g0 = (split * 2 + half) * per, g1 = min(g0 + per, ngrp);
  const bool uni = a.Ls % (4 * W) == 0;  // a row group lies in one 4D site: its index is wave-uniform
  const C2 *Vp[KT], *xp[NT];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) Vp[kt] = V + min(kt * 16 + col, a.Nv - 1) * field + chi * 6 * V5;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) xp[nt] = x + min(r0 + nt * 8 + (col >> 1), nrhs - 1) * field + chi * 6 * V5;
  // FP64 rows: run holds 8 (8 U) products and is added to sum with the rounding
  // carried in err (Kahan).  FP32 rows, and FP64 sums that turn out not to be finite
  // (the carried rounding of an infinity is none): run holds all rows
  rd4 run[KT][NT], sum[F64 ? KT : 1][F64 ? NT : 1], err[F64 ? KT : 1][F64 ? NT : 1];
  struct Row { C2 v[W]; };
  auto load = [](const C2* p) {
    Row r;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if constexpr (F64) {
        r.v[u] = p[u];
      } else {
        const float4 f = reinterpret_cast<const float4*>(p)[u];
        r.v[2 * u] = cmk<C2>(f.x, f.y);
        r.v[2 * u + 1] = cmk<C2>(f.z, f.w);
      }
    return r;
  };
  struct Half { Row va[CH][KT], xb[CH][NT]; };
  bool valid = true;  // rows past the block count with x = 0 (the basis is finite)
  auto place = [&](int g) {  // this lane's row in group g
    if (uni) {
      const int jl = __builtin_amdgcn_readfirstlane(g * 4 * W / a.Ls);
      return (long long)block_site(a, B, jl) * a.Ls + (g * 4 * W - jl * a.Ls) + q * W;
    }
    const int j = g * 4 * W + q * W, jj = j < n5 ? j : 0, jl = jj / a.Ls;
    return (long long)block_site(a, B, jl) * a.Ls + (jj - jl * a.Ls);
  };
  auto fetch = [&](Half& f, long long i5, int c0) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) f.va[c][kt] = load(Vp[kt] + (c0 + c) * V5 + i5);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) f.xb[c][nt] = load(xp[nt] + (c0 + c) * V5 + i5);
    }
  };
  auto sweep = [&](auto compensated) {
    constexpr bool KAHAN = decltype(compensated)::value;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        run[kt][nt] = rd4{0, 0, 0, 0};
        if constexpr (KAHAN) sum[kt][nt] = err[kt][nt] = rd4{0, 0, 0, 0};
      }
    auto multiply = [&](const Half& f) {
#pragma unroll
      for (int c = 0; c < CH; ++c) {
#pragma unroll
        for (int s = 0; s < W; ++s) {
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) {
            const double ar = f.va[c][kt].v[s].x, ai = f.va[c][kt].v[s].y;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
              const C2 xv = valid ? f.xb[c][nt].v[s] : cmk<C2>(0, 0);
              const double b1 = im ? xv.y : xv.x, b2 = im ? -xv.x : xv.y;
              run[kt][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, b1, run[kt][nt], 0, 0, 0);
              run[kt][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, b2, run[kt][nt], 0, 0, 0);
            }
          }
          if constexpr (KAHAN)
            if ((KT * NT <= 4 && NT < 4) || s == W - 1) {
#pragma unroll
              for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                  const rd4 y = run[kt][nt] - err[kt][nt], t = sum[kt][nt] + y;
                  err[kt][nt] = (t - sum[kt][nt]) - y;
                  sum[kt][nt] = t;
                  run[kt][nt] = rd4{0, 0, 0, 0};
                }
            }
        }
      }
    };
    // one stage ahead: its loads are in flight during the other stage's products
    Half f0, f1;
    long long i5 = 0;
    if (g0 < g1) {
      i5 = place(g0);
      fetch(f0, i5, 0);
    }
    for (int g = g0; g < g1; ++g) {
      valid = uni || g * 4 * W + q * W < n5;
      const long long next = place(min(g + 1, g1 - 1));
#pragma unroll
      for (int c = 0; c < 6; c += 2 * CH) {
        fetch(f1, i5, c + CH);
        __builtin_amdgcn_sched_barrier(0);
        multiply(f0);
        __builtin_amdgcn_sched_barrier(0);
        if (c + 2 * CH < 6) fetch(f0, i5, c + 2 * CH);
        else fetch(f0, next, 0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(f1);
        __builtin_amdgcn_sched_barrier(0);
      }
      i5 = next;
    }
    if constexpr (KAHAN) {
      double check = 0.0;  // NaN when a sum is
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          run[kt][nt] = sum[kt][nt];
#pragma unroll
          for (int v = 0; v < 4; ++v) check += 0.0 * sum[kt][nt][v];
        }
      return __any(check != check) != 0;
    }
    return false;
  };
  if (sweep(std::integral_constant<bool, F64>{})) sweep(std::false_type{});
  auto row = [&](int v) { return q + 4 * v; };  // tile row of element v
  if (half == 1)
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[chi][kt * 16 + row(v)][nt * 16 + col] = run[kt][nt][v];
  __syncthreads();
  if (half == 0)
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int rhs = r0 + nt * 8 + (col >> 1);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int k = kt * 16 + row(v);
          if (k < a.Nv && rhs < nrhs)
            partial[(((long long)rhs * a.Vc + B) * a.nsplit + split) * 4 * a.Nv + (chi * a.Nv + k) * 2 + (im ? 1 : 0)] =
                run[kt][nt][v] + red[chi][k][nt * 16 + col];
        }
      }
}

// ---- restriction and Gram sums in the order that keep_order keeps (ctx.h)
//
// Multi-RHS restriction: as k_restrict, for RG right-hand sides per workgroup
// (blockIdx.y picks the group).  A thread keeps the rows of its RG right-hand
// sides in registers while it sweeps KR basis columns, so the basis is read
// once per group of right-hand sides and x once per KR columns.  FP32 fields
// are read two s-values per 16-byte load.  Partial sums in the field's
// precision per thread (a handful of rows), FP64 across threads; same partial
// layout as k_restrict.  k_restrict_mfma is two to three times as fast (its figures
// are there) and adds in another order.
template <class C2, int RG, int KR>
__global__ __launch_bounds__(256) void k_restrict_mr(const C2* __restrict__ V, const C2* __restrict__ x,
                                                     double* __restrict__ partial, BlockArgs a, int nrhs) {
  using T = typename real_of<C2>::type;
  constexpr int W = sizeof(T) == 4 ? 2 : 1;  // consecutive s per load
  const int B = blockIdx.x / a.nsplit, split = blockIdx.x % a.nsplit;
  const int r0 = blockIdx.y * RG;
  const int nr = min(RG, nrhs - r0);
  const long long V5 = a.V5;
  const long long field = 12 * V5;
  const int n5 = a.bvol * a.Ls;
  const int n2 = 2 * a.Nv;
  __shared__ double red[4][RG * 2 * KR * 2];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  auto load = [&](const C2* f, long long off, C2 out[W]) {
    if constexpr (W == 2) {
      const float4 q = *reinterpret_cast<const float4*>(f + off);
      out[0] = cmk<C2>(q.x, q.y);
      out[1] = cmk<C2>(q.z, q.w);
    } else {
      out[0] = f[off];
    }
  };
  for (int k0 = 0; k0 < a.Nv; k0 += KR) {
    T acc[RG][2][KR][2];
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int kk = 0; kk < KR; ++kk) { acc[r][h][kk][0] = 0; acc[r][h][kk][1] = 0; }
    for (int j = split * 256 + threadIdx.x; j * W < n5; j += 256 * a.nsplit) {
      const int jj = j * W;
      const int jl = jj / a.Ls, s = jj - jl * a.Ls;
      const long long i5 = (long long)block_site(a, B, jl) * a.Ls + s;
      C2 xv[RG][12][W];
#pragma unroll
      for (int r = 0; r < RG; ++r)
#pragma unroll
        for (int c = 0; c < 12; ++c) {
          if (r < nr) load(x + (long long)(r0 + r) * field, c * V5 + i5, xv[r][c]);
          else for (int q = 0; q < W; ++q) xv[r][c][q] = cmk<C2>(0, 0);
        }
#pragma unroll
      for (int kk = 0; kk < KR; ++kk) {
        const int k = k0 + kk;
        if (k < a.Nv) {
#pragma unroll
          for (int c = 0; c < 12; ++c) {
            C2 v[W];
            load(V + (long long)k * field, c * V5 + i5, v);
            const int h = c / 6;
#pragma unroll
            for (int r = 0; r < RG; ++r)
#pragma unroll
              for (int q = 0; q < W; ++q) {
                acc[r][h][kk][0] += v[q].x * xv[r][c][q].x + v[q].y * xv[r][c][q].y;
                acc[r][h][kk][1] += v[q].x * xv[r][c][q].y - v[q].y * xv[r][c][q].x;
              }
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int kk = 0; kk < KR; ++kk)
#pragma unroll
          for (int ri = 0; ri < 2; ++ri) {
            const double v = wave_sum((double)acc[r][h][kk][ri]);
            if (l == 0) red[w][((r * 2 + h) * KR + kk) * 2 + ri] = v;
          }
    __syncthreads();
    for (int q = threadIdx.x; q < RG * 2 * KR * 2; q += 256) {
      const int r = q / (2 * KR * 2), h = (q / (KR * 2)) % 2, kk = (q / 2) % KR, ri = q & 1;
      const int k = k0 + kk;
      const double sum = red[0][q] + red[1][q] + red[2][q] + red[3][q];
      if (k < a.Nv && r < nr)
        partial[(((long long)(r0 + r) * a.Vc + B) * a.nsplit + split) * 2 * n2 + (h * a.Nv + k) * 2 + ri] = sum;
    }
    __syncthreads();
  }
}

// Multi-RHS restriction, FP32, basis and fields each read once: a 768-thread
// workgroup owns a quarter of block B's rows.  Per chunk of 64 rows the
// workgroup stages the rows of up to RX right-hand sides in LDS (layout
// [rhs][component][row], so a wavefront reads 64 consecutive rows); wave w
// then accumulates basis columns w and w + 12 against every staged
// right-hand side, lane = row.  Sums in FP32 within the workgroup (16 chunks
// x 6 components per lane, then 64 lanes), FP64 across workgroups; same
// partial layout as k_restrict.
constexpr int RX = 12, RW = 12, RT = 64 * RW;
__global__ __launch_bounds__(RT) void k_restrict_lds(const float2* __restrict__ V, const float2* __restrict__ x,
                                                     double* __restrict__ partial, BlockArgs a, int nrhs) {
  constexpr int KW = 2;  // columns per wave: 12 waves x 2 = 24 >= Nv
  __shared__ float2 xs[RX * 12 * 64];
  const int B = blockIdx.x / a.nsplit, split = blockIdx.x % a.nsplit;
  const int r0 = blockIdx.y * RX;
  const int nr = min(RX, nrhs - r0);
  const long long V5 = a.V5;
  const long long field = 12 * V5;
  const int n5 = a.bvol * a.Ls;
  const int n2 = 2 * a.Nv;
  const int per = n5 / a.nsplit;  // rows of this workgroup (n5 divides by 256)
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  float acc[KW][RX][2][2];
#pragma unroll
  for (int j = 0; j < KW; ++j)
#pragma unroll
    for (int r = 0; r < RX; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h) { acc[j][r][h][0] = 0.f; acc[j][r][h][1] = 0.f; }
  for (int c0 = 0; c0 < per; c0 += 64) {
    __syncthreads();  // the previous chunk's rows are consumed
    for (int q = threadIdx.x; q < nr * 12 * 64; q += RT) {
      const int row = q & 63, rc = q >> 6;  // rc = r * 12 + component
      const int jj = split * per + c0 + row;
      const int jl = jj / a.Ls, s = jj - jl * a.Ls;
      const long long i5 = (long long)block_site(a, B, jl) * a.Ls + s;
      const int r = rc / 12, c = rc - r * 12;
      xs[q] = x[(long long)(r0 + r) * field + c * V5 + i5];
    }
    __syncthreads();
    const int jj = split * per + c0 + l;
    const int jl = jj / a.Ls, s = jj - jl * a.Ls;
    const long long i5 = (long long)block_site(a, B, jl) * a.Ls + s;
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      const int h = c / 6;
      float2 v[KW];
#pragma unroll
      for (int j = 0; j < KW; ++j) {
        const int k = w + RW * j;
        v[j] = k < a.Nv ? V[(long long)k * field + c * V5 + i5] : make_float2(0.f, 0.f);
      }
#pragma unroll
      for (int r = 0; r < RX; ++r) {
        if (r < nr) {
          const float2 xv = xs[(r * 12 + c) * 64 + l];
#pragma unroll
          for (int j = 0; j < KW; ++j) {
            acc[j][r][h][0] += v[j].x * xv.x + v[j].y * xv.y;
            acc[j][r][h][1] += v[j].x * xv.y - v[j].y * xv.x;
          }
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < KW; ++j) {
    const int k = w + RW * j;
#pragma unroll
    for (int r = 0; r < RX; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int ri = 0; ri < 2; ++ri) {
          const float sum = wave_sum(acc[j][r][h][ri]);
          if (l == 0 && k < a.Nv && r < nr)
            partial[(((long long)(r0 + r) * a.Vc + B) * a.nsplit + split) * 2 * n2 + (h * a.Nv + k) * 2 + ri] = sum;
        }
  }
}

// Gram matrix of every (block, chirality) panel, in k_chol_inv's layout: <v_i, v_j>
// over the block's sites, all s, the six spin-colour components of chi.
constexpr int GRAM_ROWS = 16;  // fine rows staged per LDS chunk (one row = one 5D site, 6 comps)

__global__ __launch_bounds__(256) void k_gram(const double2* __restrict__ V, double2* __restrict__ G,
                                              BlockArgs a) {
  extern __shared__ double2 lds[];  // [GRAM_ROWS * 6][Nv]
  const int B = blockIdx.x >> 1, chi = blockIdx.x & 1;
  const int Nv = a.Nv;
  const long long V5 = a.V5, field = 12 * V5;
  const int n5 = a.bvol * a.Ls;
  const int npair = Nv * Nv;
  double2 acc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = make_double2(0.0, 0.0);
  for (int j0 = 0; j0 < n5; j0 += GRAM_ROWS) {
    // stage GRAM_ROWS sites x 6 comps x Nv vectors
    for (int e = threadIdx.x; e < GRAM_ROWS * 6 * Nv; e += 256) {
      const int k = e % Nv, rc = e / Nv, c6 = rc % 6, jj = rc / 6;
      const int j = j0 + jj;
      double2 v = make_double2(0.0, 0.0);
      if (j < n5) {
        const int jl = j / a.Ls, s = j - jl * a.Ls;
        const long long i5 = (long long)block_site(a, B, jl) * a.Ls + s;
        v = V[k * field + (long long)(chi * 6 + c6) * V5 + i5];
      }
      lds[rc * Nv + k] = v;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int p = threadIdx.x + q * 256;
      if (p < npair) {
        const int i = p / Nv, jc = p % Nv;
        double2 s = acc[q];
        for (int r = 0; r < GRAM_ROWS * 6; ++r) cfmac(s, lds[r * Nv + i], lds[r * Nv + jc]);
        acc[q] = s;
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int p = threadIdx.x + q * 256;
    if (p < npair) G[((long long)(p % Nv) * a.Vc + B) * 2 * Nv + chi * Nv + p / Nv] = acc[q];
  }
}

// coarse[(rhs * Vc + B) * n2 + row] = sum over splits, in fixed order: four chains
// with their rounding carried, or one without for keep_order
template <class C2>
__global__ void k_restrict_finalize(const double* __restrict__ partial, C2* __restrict__ coarse,
                                    int Vc, int n2, int nrhs, int nsplit, int one_chain) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  long long tot = (long long)nrhs * Vc * n2;
  if (i >= tot) return;
  long long site = i / n2;
  int row = (int)(i - site * n2);
  const double2* p = reinterpret_cast<const double2*>(partial) + site * nsplit * n2 + row;
  C2 v;
  if (one_chain) {
    double re = 0.0, im = 0.0;
    for (int sp = 0; sp < nsplit; ++sp) {
      re += p[sp * n2].x;
      im += p[sp * n2].y;
    }
    v.x = re;
    v.y = im;
  } else {
    double s[4][2] = {}, err[4][2] = {};
    for (int sp = 0; sp < nsplit; sp += 4) {
      double2 a[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) a[k] = p[min(sp + k, nsplit - 1) * n2];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (sp + k < nsplit) {
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const double y = (c ? a[k].y : a[k].x) - err[k][c], t = s[k][c] + y, e = (t - s[k][c]) - y;
            err[k][c] = e == e ? e : 0.0;  // an infinite sum stays one
            s[k][c] = t;
          }
        }
    }
    v.x = ((s[0][0] + s[1][0]) + (s[2][0] + s[3][0])) - ((err[0][0] + err[1][0]) + (err[2][0] + err[3][0]));
    v.y = ((s[0][1] + s[1][1]) + (s[2][1] + s[3][1])) - ((err[0][1] + err[1][1]) + (err[2][1] + err[3][1]));
  }
  coarse[i] = v;
}

// out = P c (ACC false) or out += P c (ACC true); one thread per 5D site.
template <class C2, class CC2, bool ACC>
__global__ __launch_bounds__(256) void k_prolong(const C2* __restrict__ V, const CC2* __restrict__ cvec,
                                                 C2* __restrict__ out, BlockArgs a) {
  using T = typename real_of<C2>::type;
  const long long i5 = (long long)blockIdx.x * 256 + threadIdx.x;
  const int rhs = blockIdx.y;
  const long long V5 = a.V5;
  const long long field = 12 * V5;
  if (i5 >= V5) return;
  out += rhs * field;
  const int n2 = 2 * a.Nv;
  const int x4 = (int)(i5 / a.Ls);
  const CC2* cb = cvec + ((long long)rhs * a.Vc + coarse_of(a, x4)) * n2;
  C2 acc[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = cmk<C2>(0, 0);
  for (int k = 0; k < a.Nv; ++k) {
    const C2* Vk = V + (long long)k * field;
    CC2 c0 = cb[k], c1 = cb[a.Nv + k];
    C2 w0 = cmk<C2>((T)c0.x, (T)c0.y), w1 = cmk<C2>((T)c1.x, (T)c1.y);
#pragma unroll
    for (int c = 0; c < 12; ++c) cfma(acc[c], Vk[c * V5 + i5], c < 6 ? w0 : w1);
  }
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    if (ACC) out[c * V5 + i5] = cadd(out[c * V5 + i5], acc[c]);
    else out[c * V5 + i5] = acc[c];
  }
}

// Multi-RHS prolongation: each thread reads its site's basis rows once and
// applies them to RG right-hand sides (blockIdx.y picks the group).
template <class C2, class CC2, bool ACC, int RG>
__global__ __launch_bounds__(256) void k_prolong_mr(const C2* __restrict__ V, const CC2* __restrict__ cvec,
                                                    C2* __restrict__ out, BlockArgs a, int nrhs) {
  using T = typename real_of<C2>::type;
  const long long i5 = (long long)blockIdx.x * 256 + threadIdx.x;
  const int r0 = blockIdx.y * RG;
  const int nr = min(RG, nrhs - r0);
  const long long V5 = a.V5;
  const long long field = 12 * V5;
  if (i5 >= V5) return;
  const int n2 = 2 * a.Nv;
  const int x4 = (int)(i5 / a.Ls);
  const int cs = coarse_of(a, x4);
  C2 acc[RG][12];
#pragma unroll
  for (int r = 0; r < RG; ++r)
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[r][c] = cmk<C2>(0, 0);
  for (int k = 0; k < a.Nv; ++k) {
    C2 v[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) v[c] = V[(long long)k * field + c * V5 + i5];
#pragma unroll
    for (int r = 0; r < RG; ++r) {
      if (r < nr) {
        const CC2* cb = cvec + ((long long)(r0 + r) * a.Vc + cs) * n2;
        const CC2 c0 = cb[k], c1 = cb[a.Nv + k];
        const C2 w0 = cmk<C2>((T)c0.x, (T)c0.y), w1 = cmk<C2>((T)c1.x, (T)c1.y);
#pragma unroll
        for (int c = 0; c < 12; ++c) cfma(acc[r][c], v[c], c < 6 ? w0 : w1);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < RG; ++r) {
    if (r < nr) {
      C2* o = out + (long long)(r0 + r) * field;
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        if (ACC) o[c * V5 + i5] = cadd(o[c * V5 + i5], acc[r][c]);
        else o[c * V5 + i5] = acc[r][c];
      }
    }
  }
}

// Prolongation for up to RW right-hand sides in one pass over the basis: one
// thread per fine component (spin-colour c, 5D site), all right-hand sides
// accumulated in registers, so each basis entry is read once per launch
// (k_prolong_mr reads the basis once per group of RG right-hand sides).
// Thread i covers c = i / V5 and i5 = i % V5, the basis layout's own order,
// so the basis loads and the output stores are unit-stride.  When the
// wavefront lies in one block and one chirality (64 consecutive 5D sites of
// one spin-colour component: always so when Ls x block_x is a multiple of 64)
// its coefficients are wave-uniform and come through scalar loads; otherwise
// every lane loads its own through the cache.
template <class C2, class CC2, bool ACC, int RW>
__global__ __launch_bounds__(256) void k_prolong_wide(const C2* __restrict__ V, const CC2* __restrict__ cvec,
                                                      C2* __restrict__ out, BlockArgs a, int nrhs) {
  using T = typename real_of<C2>::type;
  const long long V5 = a.V5;
  const long long field = 12 * V5;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= field) return;
  const int c = (int)(i / V5);
  const long long i5 = i - (long long)c * V5;
  const int n2 = 2 * a.Nv;
  const int cs = coarse_of(a, (int)(i5 / a.Ls));
  const int chi_off = c < 6 ? 0 : a.Nv;  // spins 0, 1: P+ columns; spins 2, 3: P- columns
  C2 acc[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) acc[r] = cmk<C2>(0, 0);
  const long long cstride = (long long)a.Vc * n2;
  const int cs0 = __builtin_amdgcn_readfirstlane(cs), off0 = __builtin_amdgcn_readfirstlane(chi_off);
  if (__all(cs == cs0 && chi_off == off0)) {
    const CC2* cb = cvec + (long long)cs0 * n2 + off0;  // wave-uniform
    int k = 0;
    for (; k + 4 <= a.Nv; k += 4) {  // four k at a time: wider scalar loads, more loads in flight
      C2 v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = V[(long long)(k + q) * field + i];
#pragma unroll
      for (int r = 0; r < RW; ++r)
        if (r < nrhs) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const CC2 w = cb[r * cstride + k + q];
            cfma(acc[r], v[q], cmk<C2>((T)w.x, (T)w.y));
          }
        }
    }
    for (; k < a.Nv; ++k) {
      const C2 v = V[(long long)k * field + i];
#pragma unroll
      for (int r = 0; r < RW; ++r)
        if (r < nrhs) {
          const CC2 w = cb[r * cstride + k];
          cfma(acc[r], v, cmk<C2>((T)w.x, (T)w.y));
        }
    }
  } else {
    const CC2* cb = cvec + (long long)cs * n2 + chi_off;
    for (int k = 0; k < a.Nv; ++k) {
      const C2 v = V[(long long)k * field + i];
#pragma unroll
      for (int r = 0; r < RW; ++r)
        if (r < nrhs) {
          const CC2 w = cb[r * cstride + k];
          cfma(acc[r], v, cmk<C2>((T)w.x, (T)w.y));
        }
    }
  }
#pragma unroll
  for (int r = 0; r < RW; ++r)
    if (r < nrhs) {
      C2* o = out + (long long)r * field + i;
      *o = ACC ? cadd(*o, acc[r]) : acc[r];
    }
}

// ---------------------------------------------------------------- CholQR
// Cholesky G = R^+ R (R upper, positive real diagonal) and W = R^{-1}, one
// wavefront per (block, chirality) panel, the matrix in LDS, lane = column.
// G[i][j] = <v_i, v_j> is the restriction of basis field j: coarse[(j * Vc + B) *
// n2 + chi * Nv + i].  status[panel] = 1 when a pivot is not positive or a column
// keeps less than 1e-7 of its norm (numerically rank deficient).  One thread
// per panel on matrices in memory took 0.9 ms a pass, a serial chain of loads.
__global__ __launch_bounds__(64) void k_chol_inv(const double2* __restrict__ G, double2* __restrict__ W,
                                                 int* __restrict__ status, int Vc, int Nv) {
  __shared__ double2 w[32][33];  // R, then X = R^{-1}
  const int B = blockIdx.x >> 1, chi = blockIdx.x & 1, j = threadIdx.x;
  auto g = [&](int i, int c) { return G[((long long)c * Vc + B) * 2 * Nv + chi * Nv + i]; };
  int bad = 0;
  // R_ii = sqrt(G_ii - sum_k |R_ki|^2),  R_ij = (G_ij - sum_k conj(R_ki) R_kj) / R_ii
  for (int i = 0; i < Nv; ++i) {
    double2 s = make_double2(0.0, 0.0);
    if (j >= i && j < Nv) {
      s = g(i, j);
      if (j == i) s.y = 0.0;
      for (int k = 0; k < i; ++k) {
        const double2 rki = w[k][i], rkj = w[k][j];
        s.x -= rki.x * rkj.x + rki.y * rkj.y;
        if (j > i) s.y -= rki.x * rkj.y - rki.y * rkj.x;
      }
    }
    double d = __shfl(s.x, i, 64);
    const double gii = g(i, i).x;
    if (!(d > 0.0) || d < 1e-14 * gii) { bad = 1; d = 1.0; }
    const double rii = sqrt(d);
    if (j < Nv) w[i][j] = j < i ? make_double2(0.0, 0.0) : (j == i ? make_double2(rii, 0.0) : make_double2(s.x / rii, s.y / rii));
    __syncthreads();
  }
  // X_jj = 1 / R_jj, X_ij = -(sum_{k = i+1..j} R_ik X_kj) / R_ii, bottom up; lane j
  // keeps its column in registers until every lane is done with R
  double2 xc[32];
#pragma unroll
  for (int i = 31; i >= 0; --i) {
    double2 s = make_double2(0.0, 0.0);
    if (i < Nv && j < Nv) {
      const double rii = w[i][i].x;
      if (i == j) {
        s = make_double2(1.0 / rii, 0.0);
      } else if (i < j) {
#pragma unroll
        for (int k = i + 1; k < 32; ++k)
          if (k <= j && k < Nv) {
            const double2 rik = w[i][k];
            s.x += fma(rik.x, xc[k].x, -(rik.y * xc[k].y));  // contracted as written: keep_order
            s.y += fma(rik.x, xc[k].y, rik.y * xc[k].x);
          }
        s = make_double2(-s.x / rii, -s.y / rii);
      }
    }
    xc[i] = s;
  }
  if (j < Nv)
#pragma unroll
    for (int i = 0; i < 32; ++i)
      if (i < Nv) W[(long long)blockIdx.x * Nv * Nv + i * Nv + j] = xc[i];
  if (j == 0) status[blockIdx.x] = bad;
}

// V[rows of panel] <- V[rows] * W (upper-triangular, Nv x Nv), in place;
// gridDim.y workgroups share a panel's rows (few panels leave the chip idle
// otherwise: 64 panels, 1.3 ms a pass with one workgroup each).
__global__ __launch_bounds__(256) void k_apply_rinv(double2* __restrict__ V, const double2* __restrict__ W,
                                                    BlockArgs a) {
  extern __shared__ double2 w[];  // Nv * Nv
  const int B = blockIdx.x >> 1, chi = blockIdx.x & 1;
  const int Nv = a.Nv;
  const long long V5 = a.V5, field = 12 * V5;
  for (int e = threadIdx.x; e < Nv * Nv; e += 256) w[e] = W[(long long)blockIdx.x * Nv * Nv + e];
  __syncthreads();
  const int n5 = a.bvol * a.Ls;
  for (int r = blockIdx.y * 256 + threadIdx.x; r < n5 * 6; r += 256 * gridDim.y) {
    const int j = r / 6, c6 = r % 6;
    const int jl = j / a.Ls, s = j - jl * a.Ls;
    const long long i5 = (long long)block_site(a, B, jl) * a.Ls + s;
    const long long off = (long long)(chi * 6 + c6) * V5 + i5;
    // fully unrolled with predicates so that row[] stays in registers
    double2 row[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) row[k] = (k < Nv) ? V[k * field + off] : make_double2(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      if (k < Nv) {
        double2 acc = make_double2(0.0, 0.0);
#pragma unroll
        for (int i = 0; i <= k; ++i) cfma(acc, row[i], w[i * Nv + k]);
        V[k * field + off] = acc;
      }
    }
  }
}

}  // namespace

// ---------------------------------------------------------------- host API

size_t restrict_partial_doubles(const CoarseGeometry& cg, int nrhs) {
  return (size_t)nrhs * cg.Vc * restrict_splits(cg.Vc) * 2 * cg.n2;  // the most any rule gives
}

template <class C2, class CC2>
void restrict_op(const C2* V, const C2* x, CC2* coarse, double* partial, const Geometry& g,
                 const CoarseGeometry& cg, int nrhs, hipStream_t st, bool keep_order, int column_tiles) {
  BlockArgs a = make_args(g, cg);
  constexpr bool f64 = sizeof(typename real_of<C2>::type) == 8;
  // the FP32 multi-RHS kernels read s-pairs: Ls even keeps every pair inside one site
  if (keep_order && nrhs >= 2 && (f64 || g.Ls % 2 == 0)) {
    constexpr int RG = 2, KR = f64 ? 4 : 6;
    bool done = false;
    if constexpr (!f64) {
      // basis and fields read once; rows per workgroup a multiple of 64
      done = cg.Nv <= 24 && (cg.bvol * g.Ls) % (64 * a.nsplit) == 0;
      if (done)
        hipLaunchKernelGGL(k_restrict_lds, dim3(cg.Vc * a.nsplit, ceil_div(nrhs, RX)), dim3(RT), 0, st, V, x, partial, a,
                           nrhs);
    }
    if (!done)
      hipLaunchKernelGGL((k_restrict_mr<C2, RG, KR>), dim3(cg.Vc * a.nsplit, ceil_div(nrhs, RG)), dim3(256), 0, st, V, x,
                         partial, a, nrhs);
  } else if (nrhs >= 2 && cg.Nv <= 32 && (f64 || g.Ls % 2 == 0)) {
    const int nt = std::max(column_tiles, std::min(4, ceil_div(nrhs, 8)));
    a.nsplit = restrict_splits(cg.Vc);
    const dim3 grid(cg.Vc * a.nsplit, ceil_div(nrhs, 8 * nt));
    const bool wide = g.Ls % (f64 ? 2 : 4) == 0;  // 32 bytes per lane: a group of four lanes reads whole 128-byte lines
#define MG_RM(KT, NT) \
  if (wide) hipLaunchKernelGGL((k_restrict_mfma<C2, KT, NT, 2>), grid, dim3(256), 0, st, V, x, partial, a, nrhs); \
  else hipLaunchKernelGGL((k_restrict_mfma<C2, KT, NT, 1>), grid, dim3(256), 0, st, V, x, partial, a, nrhs)
#define MG_RMN(KT) \
  if (nt == 1) { MG_RM(KT, 1); } \
  else if (nt == 2) { MG_RM(KT, 2); } \
  else if (nt == 3) { MG_RM(KT, 3); } \
  else { MG_RM(KT, 4); }
    if (cg.Nv <= 16) { MG_RMN(1); }
    else { MG_RMN(2); }
#undef MG_RMN
#undef MG_RM
  } else {
    if (!keep_order) a.nsplit = restrict_splits_general(cg.Vc, cg.bvol * g.Ls, nrhs, f64);
    hipLaunchKernelGGL((k_restrict<C2>), dim3(cg.Vc * a.nsplit, nrhs), dim3(256), 0, st, V, x, partial, a);
  }
  MG_LAUNCH_CHECK();
  long long tot = (long long)nrhs * cg.Vc * cg.n2;
  hipLaunchKernelGGL((k_restrict_finalize<CC2>), dim3(ceil_div(tot, 256)), dim3(256), 0, st, partial,
                     coarse, cg.Vc, cg.n2, nrhs, a.nsplit, keep_order ? 1 : 0);
  MG_LAUNCH_CHECK();
}

template <class C2, class CC2>
void prolong_op(const C2* V, const CC2* coarse, C2* fine, bool accumulate, const Geometry& g,
                const CoarseGeometry& cg, int nrhs, hipStream_t st) {
  BlockArgs a = make_args(g, cg);
  constexpr bool f64 = sizeof(typename real_of<C2>::type) == 8;
  constexpr int RG = f64 ? 2 : 4;
  constexpr int RW = f64 ? 8 : 16;
  if (nrhs > RG && nrhs <= RW) {  // basis read once
    dim3 grid(ceil_div(12LL * g.V5, 256));
    if (accumulate)
      hipLaunchKernelGGL((k_prolong_wide<C2, CC2, true, RW>), grid, dim3(256), 0, st, V, coarse, fine, a, nrhs);
    else
      hipLaunchKernelGGL((k_prolong_wide<C2, CC2, false, RW>), grid, dim3(256), 0, st, V, coarse, fine, a, nrhs);
  } else if (nrhs >= 2) {
    dim3 grid(ceil_div(g.V5, 256), ceil_div(nrhs, RG));
    if (accumulate)
      hipLaunchKernelGGL((k_prolong_mr<C2, CC2, true, RG>), grid, dim3(256), 0, st, V, coarse, fine, a, nrhs);
    else
      hipLaunchKernelGGL((k_prolong_mr<C2, CC2, false, RG>), grid, dim3(256), 0, st, V, coarse, fine, a, nrhs);
  } else {
    dim3 grid(ceil_div(g.V5, 256), nrhs);
    if (accumulate)
      hipLaunchKernelGGL((k_prolong<C2, CC2, true>), grid, dim3(256), 0, st, V, coarse, fine, a);
    else
      hipLaunchKernelGGL((k_prolong<C2, CC2, false>), grid, dim3(256), 0, st, V, coarse, fine, a);
  }
  MG_LAUNCH_CHECK();
}

template void restrict_op<double2, double2>(const double2*, const double2*, double2*, double*,
                                            const Geometry&, const CoarseGeometry&, int, hipStream_t, bool, int);
template void restrict_op<float2, float2>(const float2*, const float2*, float2*, double*, const Geometry&,
                                          const CoarseGeometry&, int, hipStream_t, bool, int);
template void prolong_op<double2, double2>(const double2*, const double2*, double2*, bool, const Geometry&,
                                           const CoarseGeometry&, int, hipStream_t);
template void prolong_op<float2, float2>(const float2*, const float2*, float2*, bool, const Geometry&,
                                         const CoarseGeometry&, int, hipStream_t);

// Two passes of Cholesky QR on every (block, chirality) panel of the FP64 basis.
// Returns false if any panel is numerically rank deficient.
bool orthonormalise_basis(double2* V, const Geometry& g, const CoarseGeometry& cg, bool keep_order, hipStream_t st) {
  if (cg.Nv > 32) fail(MGDWF_ERR_INVALID_ARG, "nvec above 32 is not supported");
  BlockArgs a = make_args(g, cg);
  const int npanel = 2 * cg.Vc;
  const size_t nn = (size_t)cg.Nv * cg.Nv;
  DevBuf G(npanel * nn * sizeof(double2)), W(npanel * nn * sizeof(double2)), stat(npanel * sizeof(int));
  DevBuf part(restrict_partial_doubles(cg, cg.Nv) * sizeof(double));
  std::vector<int> hs(npanel);
  bool ok = true;
  for (int pass = 0; pass < 2; ++pass) {
    if (keep_order) {
      hipLaunchKernelGGL(k_gram, dim3(npanel), dim3(256), (size_t)GRAM_ROWS * 6 * cg.Nv * sizeof(double2), st, V,
                         G.as<double2>(), a);
      MG_LAUNCH_CHECK();
    } else {
      restrict_op<double2, double2>(V, V, G.as<double2>(), part.as<double>(), g, cg, cg.Nv, st, false, 1);  // Gram matrices
    }
    hipLaunchKernelGGL(k_chol_inv, dim3(npanel), dim3(64), 0, st, G.as<double2>(), W.as<double2>(), stat.as<int>(),
                       cg.Vc, cg.Nv);
    MG_LAUNCH_CHECK();
    MG_HIP(hipMemcpyAsync(hs.data(), stat.p, npanel * sizeof(int), hipMemcpyDeviceToHost, st));
    MG_HIP(hipStreamSynchronize(st));
    for (int v : hs) if (v) ok = false;
    if (!ok) return false;
    hipLaunchKernelGGL(k_apply_rinv, dim3(npanel, std::max(1, std::min(16, ceil_div(2048, npanel)))), dim3(256),
                       nn * sizeof(double2), st, V, W.as<double2>(), a);
    MG_LAUNCH_CHECK();
  }
  return ok;
}

}  // namespace mgdwf

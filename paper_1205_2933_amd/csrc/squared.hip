// Coarse operator of the squared operator, A_c = P^+ D^+ D P: construction and
// 33-point application.
//
// Paper, Sec. 3 (first paragraph): the multigrid and the CG control act on
// the squared operator D^+D; Sec. 4 (last paragraph): its coarse operator
// couples a coarse site to sites up to two hops away.  With 4D blocks of
// extent >= 2 spanning the fifth dimension, A_c couples X to X + o for 33
// offsets o: self, the eight unit neighbours +-mu and the 24 diagonal ones
// +-mu +-nu (mu < nu).  The two hops of one direction land on opposite faces
// of the block between them, so no coupling two blocks away in one
// direction exists.
//
// Construction, one basis column j = (chi, k) at a time for every block at
// once: the face-split D applied to the chirality-chi part of basis field k
// gives nine fields W_e (e = 0: the hops into each block from the block
// itself, with the diagonal and fifth-dimension terms; e = 1+2mu / 2+2mu:
// the hops into each block from its +mu / -mu neighbour).  The face-split
// D^+ of W_e gives nine fields Z_d (the hops into each block from its
// neighbour d).  Z_d restricted to block X is D^+_{X, X+d} D_{X+d, X+d+e} V_j,
// so R Z_d is column j of A_c[X][o] with o = delta_d + delta_e; pairs with
// o = +-2 mu are zero (opposite faces) and skipped.  The same assignment by
// direction keeps coarse extents 1 and 2 exact, as for the 9-point operator.
//
// A_c is Hermitian, so one stencil serves both A_c and its adjoint.  Storage:
// column-major 2Nv x 2Nv blocks [X][o], FP64 and an FP32 copy.
#include <algorithm>
#include <type_traits>

#include "mg_internal.h"
#include "blas.h"
#include "rules.h"
#include "vecops.h"

namespace mgdwf {

void dslash_split(const double2* in, double2* out9, const double2* gauge, const Geometry& g, const int block[4],
                  double M5, double mf, int chi, hipStream_t st, bool dagger);

namespace {

struct SqArgs {
  int Lc[4];
  int Vc;
  int n2;
  int off[33][4];  // offsets in (x, y, z, t)
  int nact;        // offsets whose blocks are not all zero (33; 9 on a planar lattice)
  int act[33];
};

// Offset index table: 0 self; 1 + 2 mu = +mu; 2 + 2 mu = -mu; then for mu < nu
// the four diagonals (+mu+nu, +mu-nu, -mu+nu, -mu-nu).
void offset_table(int off[33][4]) {
  int n = 0;
  for (int m = 0; m < 4; ++m) off[n][m] = 0;
  ++n;
  for (int mu = 0; mu < 4; ++mu)
    for (int sg : {1, -1}) {
      for (int m = 0; m < 4; ++m) off[n][m] = 0;
      off[n][mu] = sg;
      ++n;
    }
  for (int mu = 0; mu < 4; ++mu)
    for (int nu = mu + 1; nu < 4; ++nu)
      for (int s1 : {1, -1})
        for (int s2 : {1, -1}) {
          for (int m = 0; m < 4; ++m) off[n][m] = 0;
          off[n][mu] = s1;
          off[n][nu] = s2;
          ++n;
        }
}

// index of delta_d + delta_e in the table, -1 for +-2 mu
int pair_offset(const int off[33][4], int d, int e) {
  int v[4] = {0, 0, 0, 0};
  for (int q : {d, e})
    if (q > 0) v[(q - 1) >> 1] += (q & 1) ? 1 : -1;
  for (int i = 0; i < 33; ++i) {
    bool eq = true;
    for (int m = 0; m < 4; ++m) eq = eq && off[i][m] == v[m];
    if (eq) return i;
  }
  return -1;
}

SqArgs sq_args(const CoarseGeometry& cg) {
  SqArgs a;
  for (int m = 0; m < 4; ++m) a.Lc[m] = cg.Lc[m];
  a.Vc = cg.Vc;
  a.n2 = cg.n2;
  offset_table(a.off);
  a.nact = 0;
  for (int o = 0; o < 33; ++o)
    if (!cg.planar || (a.off[o][2] == 0 && a.off[o][3] == 0)) a.act[a.nact++] = o;
  return a;
}

__device__ __forceinline__ int sq_neighbour(const SqArgs& a, int X, int o) {
  int c[4];
  int r = X;
  c[0] = r % a.Lc[0]; r /= a.Lc[0];
  c[1] = r % a.Lc[1]; r /= a.Lc[1];
  c[2] = r % a.Lc[2]; c[3] = r / a.Lc[2];
#pragma unroll
  for (int m = 0; m < 4; ++m) c[m] = (c[m] + a.off[o][m] + a.Lc[m]) % a.Lc[m];
  return ((c[3] * a.Lc[2] + c[2]) * a.Lc[1] + c[1]) * a.Lc[0] + c[0];
}

// Ac[X][oi[d]] column j += coarse[d][X][row] for the nine d of one e
struct PairIdx {
  int oi[9];
};

__global__ void k_sq_scatter(const double2* __restrict__ coarse, double2* __restrict__ Ac, int Vc, int n2, int j,
                             PairIdx pi) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long tot = 9LL * Vc * n2;
  if (i >= tot) return;
  const int row = (int)(i % n2);
  const long long t = i / n2;
  const int X = (int)(t % Vc), d = (int)(t / Vc);
  const int o = pi.oi[d];
  if (o < 0) return;
  double2* dst = Ac + (((long long)X * 33 + o) * n2 + j) * n2 + row;
  const double2 v = coarse[i];
  *dst = make_double2(dst->x + v.x, dst->y + v.y);
}

__global__ void k_zero64(double2* __restrict__ p, long long n) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    p[i] = make_double2(0.0, 0.0);
}

__global__ void k_sq_to_f32(const double2* __restrict__ in, float2* __restrict__ out, long long n) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    out[i] = make_float2((float)in[i].x, (float)in[i].y);
}

// y[rhs](X) = sum_o A[X][o] x[rhs](X + o) for up to NR right-hand sides.
// Workgroup = one coarse site, nine wavefronts; wavefront w takes the
// offsets o = w, w + 9, w + 18, w + 27 (< 33); lane = output row.  Per offset
// the wavefront first copies the neighbour's coarse vectors of all NR
// right-hand sides into its own LDS panel ([col][rhs], zero past the last
// right-hand side), so the inner loop reads one coalesced matrix column per
// step from memory and the NR vector entries as LDS broadcasts.  The nine
// partial sums are added in a fixed order through LDS.
template <class MC2, class VC2, class O2, int NR>
__global__ __launch_bounds__(576) void k_sq_apply(const MC2* __restrict__ M, const VC2* __restrict__ x,
                                                  O2* __restrict__ y, SqArgs a, int nrhs, int rhs0) {
  using T = typename real_of<VC2>::type;
  __shared__ VC2 xs[9][64 * NR];  // per wavefront: [col][rhs]; reused for the reduction at the end
  const int X = blockIdx.x;
  const int n2 = a.n2;
  const int w = threadIdx.x >> 6, row = threadIdx.x & 63;
  const int nr = min(NR, nrhs - rhs0);
  const long long vs = (long long)a.Vc * n2;
  VC2* panel = xs[w];
  VC2 acc[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) acc[j] = cmk<VC2>(0, 0);
  for (int k = 0; k < 4; ++k) {  // every wavefront takes four turns (the barriers need them all)
    const int o = w + 9 * k;
    const bool act = o < 33;
    if (act) {
      const int Y = sq_neighbour(a, X, o);
      const VC2* xv = x + (long long)rhs0 * vs + (long long)Y * n2;
      for (int e = row; e < NR * n2; e += 64) {
        const int j = e / n2, c = e - j * n2;
        panel[c * NR + j] = j < nr ? xv[(long long)j * vs + c] : cmk<VC2>(0, 0);
      }
    }
    __syncthreads();
    if (act && row < n2) {
      const MC2* Mo = M + ((long long)X * 33 + o) * n2 * n2;
      auto column = [&](int c) {
        const MC2 m = Mo[c * n2 + row];
        const VC2 mv = cmk<VC2>((T)m.x, (T)m.y);
#pragma unroll
        for (int j = 0; j < NR; ++j) cfma(acc[j], mv, panel[c * NR + j]);
      };
      if constexpr (sizeof(T) == 4 && NR >= 8) {
        // FP32: columns in flight, measured on 512 sites x 48 dof: at 12 RHS
        // 148 us with 16, 158 with 8, 202 with 4, 262 with none; at one
        // right-hand side 57 us with 8 and 66 with 16.  FP64 runs faster
        // without (307 against 338 us with 4)
#pragma unroll 16
        for (int c = 0; c < n2; ++c) column(c);
      } else if constexpr (sizeof(T) == 4) {
#pragma unroll 8
        for (int c = 0; c < n2; ++c) column(c);
      } else {
        for (int c = 0; c < n2; ++c) column(c);
      }
    }
    __syncthreads();
  }
  T (*red)[64][2] = reinterpret_cast<T (*)[64][2]>(&xs[0][0]);  // [rhs][row][re, im]
  for (int q = 0; q < 9; ++q) {
    if (w == q)
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        if (q == 0) { red[j][row][0] = acc[j].x; red[j][row][1] = acc[j].y; }
        else { red[j][row][0] += acc[j].x; red[j][row][1] += acc[j].y; }
      }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < nr * n2; i += blockDim.x) {
    const int j = i / n2, r = i % n2;
    y[(long long)(rhs0 + j) * vs + (long long)X * n2 + r] = cmk<O2>(red[j][r][0], red[j][r][1]);
  }
}

// The same sums bit for bit (FP32, 2 Nv = N2 a multiple of 16), for keep_order:
// as above, but blockIdx.y picks NR right-hand sides, the vector entries, the same
// for a whole wavefront, come as scalar loads (no panel, no barrier before the final
// sum) and KC columns are in flight ahead of those being multiplied.  Bound by load
// latency at few sites (32 sites x 48 dof, 4 right-hand sides: 14.4 us, 25.4 in the
// kernel above), by the bytes of M at many (512, one: 51 us, 6.2 TB/s); which of the two
// runs: sq_ordered_group.
template <int N2, int NR>
__global__ __launch_bounds__(576) void k_sq_ordered(const float2* __restrict__ M, const float2* __restrict__ x,
                                                    float2* __restrict__ y, SqArgs a, int nrhs) {
  constexpr int KC = N2 == 48 ? 12 : 8;
  __shared__ float2 sum[9][NR][64];
  const int X = blockIdx.x, r0 = blockIdx.y * NR;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l = threadIdx.x & 63;
  const long long vs = (long long)a.Vc * N2;
  float2 m0[KC], m1[KC];
  const auto hold = [] { asm volatile("" ::: "memory"); };  // loads stay where they stand (registers)
  const unsigned lane_off = (unsigned)(l < N2 ? l : N2 - 1) * sizeof(float2);
  auto fetch = [&](float2* m, int o, int c0) {  // wave-uniform base, 32-bit lane offset
    const char* Mo = reinterpret_cast<const char*>(M + (((long long)X * 33 + o) * N2 + c0) * N2);
#pragma unroll
    for (int c = 0; c < KC; ++c) m[c] = *reinterpret_cast<const float2*>(Mo + c * N2 * sizeof(float2) + lane_off);
  };
  float2 acc[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) acc[j] = make_float2(0.f, 0.f);
  auto multiply = [&](const float2* m, const float2* xo) {
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const float2* xv = xo + (long long)(r0 + j < nrhs ? j : 0) * vs;
#pragma unroll
      for (int c = 0; c < KC; ++c) cfma(acc[j], m[c], xv[c]);
    }
  };
  fetch(m0, w, 0);
#pragma unroll 1
  for (int o = w; o < 33; o += 9) {
    const float2* xo = x + (long long)r0 * vs + (long long)sq_neighbour(a, X, o) * N2;
#pragma unroll 1
    for (int c = 0; c < N2; c += 2 * KC) {
      fetch(m1, o, c + KC);
      hold();
      multiply(m0, xo + c);
      hold();
      if (c + 2 * KC < N2) fetch(m0, o, c + 2 * KC);
      else if (o + 9 < 33) fetch(m0, o + 9, 0);
      hold();
      multiply(m1, xo + c + KC);
      hold();
    }
  }
#pragma unroll
  for (int j = 0; j < NR; ++j) sum[w][j][l] = acc[j];
  __syncthreads();
  for (int e = threadIdx.x; e < NR * 64; e += 576) {
    const int j = e >> 6, row = e & 63;
    float2 s = sum[0][j][row];
#pragma unroll
    for (int q = 1; q < 9; ++q) s = cadd(s, sum[q][j][row]);
    if (row < N2 && r0 + j < nrhs) y[(long long)(r0 + j) * vs + (long long)X * N2 + row] = s;
  }
}

// ---- the product on MFMA (2 Nv a multiple of 16), alone or as a CG step
//
// A workgroup of SQW wavefronts owns 16 RT rows of one coarse site (blockIdx.y picks
// the rows and the group of 8 NT right-hand sides), wavefront w the offsets w, w +
// SQW, ...: 33 offsets are three rounds.  Tile columns are (Re | Im) of eight
// right-hand sides: A = Re M against (Re x | Im x), A = Im M against (-Im x | Re x),
// 16x16x4 tiles of the operator's own precision.  The wavefronts' partial tiles are
// added in LDS in FP64, in a fixed order.  Few sites are bound by load latency and
// by what one CU can stream of a site's 33 blocks, so their rows go to different
// workgroups; many by the bytes of M.  48 dof, us, against one lane per row and a
// vector panel in LDS: 32 sites, 4 right-hand sides FP64 37 -> 13.9, FP32 25 -> 9.8,
// 12: 100 -> 14.4, 51 -> 11.2; 512 sites, 12: 290 -> 219, 145 -> 82 (3.9 TB/s), one:
// 110 -> 111, 57.6 -> 58.9 (5.4 TB/s).
constexpr int SQW = 11;
typedef double sd4 __attribute__((ext_vector_type(4)));
typedef float sf4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ sd4 sq_mfma(double a, double b, sd4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ __forceinline__ sf4 sq_mfma(float a, float b, sf4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// CG: x is r, the product is taken with p_new = r + beta p_old, formed on the fly
// at every neighbour (one launch less than a pass of its own); np partials of
// |r|^2 per right-hand side come in, <p_new, q> per (site, row tile) go out.
template <class C2>
struct SqStep {
  const C2 *x, *p_old;
  C2* p_new;
  const double* part_in;
  int np;
  double* part_out;
  double* sl;
  int cur, nxt, rr0, first;
};

template <class C2, class O2, int N2, int NT, int RT, bool CG>
__global__ __launch_bounds__(SQW * 64) void k_sq_mfma(const C2* __restrict__ M, O2* __restrict__ y, SqStep<C2> q,
                                                      SqArgs a, int nrhs) {
  using T = typename real_of<C2>::type;
  constexpr bool F64 = sizeof(T) == 8;
  using Acc = typename std::conditional<F64, sd4, sf4>::type;
  constexpr int MT = N2 / 16, KT = N2 / 4, NR = 8 * NT, ROWS = 16 * RT, PAD = ROWS + (F64 ? 1 : 4);
  // k-tiles in flight (registers: matrix RT KC, vectors NT KC, twice that in CG)
  constexpr int KC = F64 ? (RT > 2 ? KT / (KT % 3 == 0 ? 3 : 4) : (CG && N2 > 32 ? KT / 2 : KT)) : (RT > 3 ? KT / 2 : KT);
  __shared__ __align__(16) T slab[SQW][2 * NR][PAD];
  __shared__ double bsum[NR];
  const int X = blockIdx.x, rt0 = blockIdx.y % (MT / RT) * RT, r0 = blockIdx.y / (MT / RT) * NR;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l = threadIdx.x & 63;
  const int col = l & 15, kq = l >> 4;
  const bool im = col & 1;
  const long long vs = (long long)a.Vc * N2;
  // a round's matrix tile; the first is loaded before the sums below (it depends
  // on nothing the launch before wrote).  Holding further rounds costs more in
  // resident wavefronts than it hides (512 sites x 48 dof: 7 to 10 % slower).
  C2 m[RT][KC];
  auto load_tile = [&](int k, int k0) {
    const int j = w + SQW * k;
    if (j < a.nact) {
      const C2* A = M + (((long long)X * 33 + a.act[j]) * N2 + kq) * N2 + rt0 * 16 + col;
#pragma unroll
      for (int i = 0; i < KC; ++i)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) m[rt][i] = A[4 * (k0 + i) * N2 + rt * 16];
    }
  };
  load_tile(0, 0);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (CG) {
    for (int c = w; c < NR; c += SQW) {
      double s = 0.0;
      if (r0 + c < nrhs)
#pragma unroll 4
        for (int i = l; i < q.np; i += 64) s += q.part_in[(long long)(r0 + c) * q.np + i];
      s = wave_sum(s);
      if (l == 0) bsum[c] = s;
    }
    __syncthreads();
  }
  const C2* p_in = q.first ? q.x : q.p_old;  // first: read, not used
  auto beta_of = [&](int c) {  // right-hand side r0 + c
    if (q.first) return (T)0;
    const double d = q.sl[(long long)(r0 + c) * NSLOT + q.cur];
    return (T)(d > 0.0 ? bsum[c] / d : 0.0);
  };
  T beta[NT];
  long long vo[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int c = min(nt * 8 + (col >> 1), nrhs - 1 - r0);
    vo[nt] = (long long)(r0 + c) * vs + kq;
    if constexpr (CG) beta[nt] = beta_of(c);
  }
  Acc acc[RT][NT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[rt][nt] = Acc{0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int j = w + SQW * k;
    if (j < a.nact) {
      const long long Y = (long long)sq_neighbour(a, X, a.act[j]) * N2;
#pragma unroll
      for (int k0 = 0; k0 < KT; k0 += KC) {
        C2 v[NT][KC], pv[CG ? NT : 1][KC];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int i = 0; i < KC; ++i) {
            v[nt][i] = q.x[vo[nt] + Y + 4 * (k0 + i)];
            if constexpr (CG) pv[nt][i] = p_in[vo[nt] + Y + 4 * (k0 + i)];
          }
        __builtin_amdgcn_sched_barrier(0);  // every load of the round before the first product
#pragma unroll
        for (int i = 0; i < KC; ++i)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            C2 xv = v[nt][i];
            if constexpr (CG)
              if (!q.first) xv = cadd(xv, cscale(pv[nt][i], beta[nt]));
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
              acc[rt][nt] = sq_mfma(m[rt][i].x, im ? xv.y : xv.x, acc[rt][nt]);
              acc[rt][nt] = sq_mfma(m[rt][i].y, im ? xv.x : -xv.y, acc[rt][nt]);
            }
          }
        if (k0 + KC < KT) {
          load_tile(k, k0 + KC);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (k < 2) {
      load_tile(k + 1, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int v = 0; v < 4; ++v) slab[w][nt * 16 + col][rt * 16 + (F64 ? kq + 4 * v : 4 * kq + v)] = acc[rt][nt][v];
  __syncthreads();
  for (int e = threadIdx.x; e < NR * ROWS; e += SQW * 64) {  // whole groups of 16 lanes: one row tile of one rhs
    const int c = e / ROWS, row = e % ROWS;
    if (r0 + c >= nrhs) continue;
    double re = 0.0, ii = 0.0;
#pragma unroll
    for (int s = 0; s < SQW; ++s) {
      re += slab[s][2 * c][row];
      ii += slab[s][2 * c + 1][row];
    }
    const long long i = (long long)(r0 + c) * vs + (long long)X * N2 + rt0 * 16 + row;
    if constexpr (CG) {
      const C2 qv = cmk<C2>((T)re, (T)ii);
      C2 pv = q.x[i];
      if (!q.first) pv = cadd(pv, cscale(q.p_old[i], beta_of(c)));
      y[i] = qv;
      q.p_new[i] = pv;
      double pq = (double)pv.x * qv.x + (double)pv.y * qv.y;
#pragma unroll
      for (int off = 8; off > 0; off >>= 1) pq += __shfl_xor(pq, off, 16);
      if (row % 16 == 0) {
        const int rt = rt0 + row / 16;
        q.part_out[((long long)(r0 + c) * a.Vc + X) * MT + rt] = pq;
        if (X == 0 && rt == 0) {
          double* sr = q.sl + (long long)(r0 + c) * NSLOT;
          sr[q.nxt] = bsum[c];
          if (q.first) sr[q.rr0] = bsum[c];
        }
      }
    } else {
      y[i] = cmk<O2>(re, ii);
    }
  }
}

// r = b (x null) or x (+)= alpha p, r -= alpha q with alpha = slot rr / <p, q>, the
// np partials of <p, q> added by every workgroup; partial |r|^2 per workgroup
template <class C2>
__global__ __launch_bounds__(256) void k_sq_update(C2* __restrict__ x, C2* __restrict__ r, const C2* __restrict__ p,
                                                   const C2* __restrict__ q, long long n, const double* __restrict__ pq,
                                                   int np, const double* __restrict__ sl, int rr, int first,
                                                   double* __restrict__ part) {
  using T = typename real_of<C2>::type;
  const int rhs = blockIdx.y;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x, e = rhs * n + i;
  __shared__ double tot;
  T alpha = 0;
  if (x) {
    double s = 0.0;
#pragma unroll 4
    for (int k = threadIdx.x; k < np; k += 256) s += pq[(long long)rhs * np + k];
    s = block_sum<256>(s);
    if (threadIdx.x == 0) tot = s;
    __syncthreads();
    alpha = (T)(tot > 0.0 ? sl[(long long)rhs * NSLOT + rr] / tot : 0.0);
  }
  double nn = 0.0;
  if (i < n) {
    C2 rv;
    if (x) {
      const C2 xv = first ? cmk<C2>(0, 0) : x[e];
      x[e] = cadd(xv, cscale(p[e], alpha));
      rv = csub(r[e], cscale(q[e], alpha));
    } else {
      rv = p[e];
    }
    r[e] = rv;
    nn = (double)rv.x * rv.x + (double)rv.y * rv.y;
  }
  nn = block_sum<256>(nn);
  if (threadIdx.x == 0) part[(long long)rhs * gridDim.x + blockIdx.x] = nn;
}

// Canonical layout [X][o][row][col] from the internal column-major blocks.
__global__ void k_sq_canonical(const double2* __restrict__ in, double2* __restrict__ out, long long nblk, int n2) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nblk * n2 * n2) return;
  const long long blk = i / ((long long)n2 * n2);
  const int rc = (int)(i - blk * n2 * n2);
  const int row = rc / n2, col = rc % n2;
  out[i] = in[blk * n2 * n2 + (long long)col * n2 + row];
}

}  // namespace

size_t sq_coarse_entries(const CoarseGeometry& cg) { return (size_t)cg.Vc * 33 * cg.n2 * cg.n2; }

// Build A_c (FP64) into Ac; work9 and zwork9: 9 fine FP64 fields each; cwork:
// 9 Vc n2 complex; partial: restriction scratch for 9 right-hand sides.
void build_sq_coarse_op(const double2* Vhat, const double2* gauge, double2* Ac, double2* work9, double2* zwork9,
                        double2* cwork, double* partial, const Geometry& g, const CoarseGeometry& cg, double M5,
                        double mf, hipStream_t st) {
  const long long field = 12LL * g.V5;
  const long long nA = (long long)sq_coarse_entries(cg);
  hipLaunchKernelGGL(k_zero64, dim3(std::min<long long>(ceil_div(nA, 256), 8192)), dim3(256), 0, st, Ac, nA);
  MG_LAUNCH_CHECK();
  int off[33][4];
  offset_table(off);
  for (int chi = 0; chi < 2; ++chi)
    for (int k = 0; k < cg.Nv; ++k) {
      const int j = chi * cg.Nv + k;
      dslash_split(Vhat + k * field, work9, gauge, g, cg.block, M5, mf, chi, st, false);  // W_e, e = 0..8
      for (int e = 0; e < 9; ++e) {
        PairIdx pi;
        bool any = false;
        for (int d = 0; d < 9; ++d) {
          pi.oi[d] = pair_offset(off, d, e);
          any = any || pi.oi[d] >= 0;
        }
        if (!any) continue;
        dslash_split(work9 + (long long)e * field, zwork9, gauge, g, cg.block, M5, mf, -1, st, true);
        restrict_op<double2, double2>(Vhat, zwork9, cwork, partial, g, cg, 9, st, true);
        const long long tot = 9LL * cg.Vc * cg.n2;
        hipLaunchKernelGGL(k_sq_scatter, dim3(ceil_div(tot, 256)), dim3(256), 0, st, cwork, Ac, cg.Vc, cg.n2, j, pi);
        MG_LAUNCH_CHECK();
      }
    }
}

void sq_to_f32(const double2* Ac, float2* Ac32, const CoarseGeometry& cg, hipStream_t st) {
  const long long n = (long long)sq_coarse_entries(cg);
  hipLaunchKernelGGL(k_sq_to_f32, dim3(std::min<long long>(ceil_div(n, 256), 8192)), dim3(256), 0, st, Ac, Ac32, n);
  MG_LAUNCH_CHECK();
}

void sq_canonical(const double2* Ac, double2* out, const CoarseGeometry& cg, hipStream_t st) {
  const long long nblk = 33LL * cg.Vc, tot = nblk * cg.n2 * cg.n2;
  hipLaunchKernelGGL(k_sq_canonical, dim3(ceil_div(tot, 256)), dim3(256), 0, st, Ac, out, nblk, cg.n2);
  MG_LAUNCH_CHECK();
}

// MFMA kernels for 2 Nv = 16, 32, 48, 64
template <class F>
static bool with_sq_n2(int n2, F&& f) {
  switch (n2) {
    case 16: f(std::integral_constant<int, 16>{}); return true;
    case 32: f(std::integral_constant<int, 32>{}); return true;
    case 48: f(std::integral_constant<int, 48>{}); return true;
    case 64: f(std::integral_constant<int, 64>{}); return true;
    default: return false;
  }
}

template <class C2, class O2, bool CG>
static bool sq_mfma_launch(const C2* A, O2* y, const SqStep<C2>& q, const CoarseGeometry& cg, int nrhs, hipStream_t st) {
  const SqArgs a = sq_args(cg);
  const bool done = with_sq_n2(cg.n2, [&](auto N) {
    constexpr int N2 = decltype(N)::value;
    constexpr int MT = N2 / 16;
    const int groups = ceil_div(nrhs, 8);
    const dim3 blk(SQW * 64);
    // FP32 takes 16 right-hand sides per pass over the matrix on 256 sites or more (48
    // dof, 512 sites, 12: 82 us against 113; 128, 12: 31 against 22); a CG step has no
    // registers for it
    if (sq_split_rows((long long)groups * cg.Vc, MT, std::is_same<C2, double2>::value, CG)) {
      hipLaunchKernelGGL((k_sq_mfma<C2, O2, N2, 1, 1, CG>), dim3(cg.Vc, MT * groups), blk, 0, st, A, y, q, a, nrhs);
      return;
    }
    if constexpr (!CG && std::is_same<C2, float2>::value)
      if (nrhs > 8 && cg.Vc >= 256) {
        hipLaunchKernelGGL((k_sq_mfma<C2, O2, N2, 2, MT, CG>), dim3(cg.Vc, ceil_div(nrhs, 16)), blk, 0, st, A, y, q, a,
                           nrhs);
        return;
      }
    hipLaunchKernelGGL((k_sq_mfma<C2, O2, N2, 1, MT, CG>), dim3(cg.Vc, groups), blk, 0, st, A, y, q, a, nrhs);
  });
  if (done) MG_LAUNCH_CHECK();
  return done;
}

bool sq_cg_fused(const CoarseGeometry& cg) { return cg.n2 % 16 == 0 && cg.n2 <= 64; }

static int sq_update_blocks(const CoarseGeometry& cg) { return ceil_div((long long)cg.Vc * cg.n2, 256); }
static int sq_product_parts(const CoarseGeometry& cg) { return cg.Vc * (cg.n2 / 16); }

size_t sq_cg_bytes(const CoarseGeometry& cg, int nrhs) {
  return (size_t)nrhs * (sq_update_blocks(cg) + sq_product_parts(cg)) * sizeof(double);
}

template <class F2>
void sq_cg_start(const F2* b, F2* r, void* work, const CoarseGeometry& cg, int nrhs, hipStream_t st) {
  const long long n = (long long)cg.Vc * cg.n2;
  hipLaunchKernelGGL(k_sq_update<F2>, dim3(sq_update_blocks(cg), nrhs), dim3(256), 0, st, nullptr, r, b, nullptr, n,
                     nullptr, 0, nullptr, 0, 0, static_cast<double*>(work));
  MG_LAUNCH_CHECK();
}

template <class F2>
void sq_cg_product(const F2* A, const F2* r, const F2* p_old, F2* p_new, F2* q, void* work, double* sl, int cur, int nxt,
                   int rr0, bool first, const CoarseGeometry& cg, int nrhs, hipStream_t st) {
  double* rr = static_cast<double*>(work);
  SqStep<F2> s{r, p_old, p_new, rr, sq_update_blocks(cg), rr + (size_t)nrhs * sq_update_blocks(cg), sl, cur, nxt, rr0,
               first ? 1 : 0};
  sq_mfma_launch<F2, F2, true>(A, q, s, cg, nrhs, st);
}

template <class F2>
void sq_cg_update(F2* x, F2* r, const F2* p, const F2* q, void* work, double* sl, int rr, bool first,
                  const CoarseGeometry& cg, int nrhs, hipStream_t st) {
  const long long n = (long long)cg.Vc * cg.n2;
  double* part = static_cast<double*>(work);
  hipLaunchKernelGGL(k_sq_update<F2>, dim3(sq_update_blocks(cg), nrhs), dim3(256), 0, st, x, r, p, q, n,
                     part + (size_t)nrhs * sq_update_blocks(cg), sq_product_parts(cg), sl, rr, first ? 1 : 0, part);
  MG_LAUNCH_CHECK();
}

void sq_cg_residual(void* work, double* sl, int dst, const CoarseGeometry& cg, int nrhs, hipStream_t st) {
  finalize_rhs(static_cast<double*>(work), sq_update_blocks(cg), 1, sl, dst, nrhs, st);
}

#define MG_SQCG(F2)                                                                                                  \
  template void sq_cg_start<F2>(const F2*, F2*, void*, const CoarseGeometry&, int, hipStream_t);                     \
  template void sq_cg_product<F2>(const F2*, const F2*, const F2*, F2*, F2*, void*, double*, int, int, int, bool,    \
                                  const CoarseGeometry&, int, hipStream_t);                                         \
  template void sq_cg_update<F2>(F2*, F2*, const F2*, const F2*, void*, double*, int, bool, const CoarseGeometry&,  \
                                 int, hipStream_t);
MG_SQCG(double2)
MG_SQCG(float2)
#undef MG_SQCG

// Other dof counts, and keep_order: the right-hand sides go in launches of at most NRMAX; each uses the
// smallest compiled panel width that holds its count (the inner loop runs
// over the whole width).
template <class MC2, class VC2, int NR, class O2>
static void sq_launch(const MC2* A, const VC2* x, O2* y, const SqArgs& a, int Vc, int nrhs, int r0, hipStream_t st) {
  hipLaunchKernelGGL((k_sq_apply<MC2, VC2, O2, NR>), dim3(Vc), dim3(576), 0, st, A, x, y, a, nrhs, r0);
  MG_LAUNCH_CHECK();
}

void sq_apply64(const double2* Ac, const double2* x, double2* y, const CoarseGeometry& cg, int nrhs, hipStream_t st,
                bool keep_order) {
  if (cg.n2 > 64) fail(MGDWF_ERR_INVALID_ARG, "2*nvec above 64 is not supported");
  SqStep<double2> q{};
  q.x = x;
  if (!keep_order && sq_mfma_launch<double2, double2, false>(Ac, y, q, cg, nrhs, st)) return;
  const SqArgs a = sq_args(cg);
  for (int r0 = 0; r0 < nrhs; r0 += 8) {
    const int nr = std::min(8, nrhs - r0);
    if (nr == 1) sq_launch<double2, double2, 1>(Ac, x, y, a, cg.Vc, nrhs, r0, st);
    else if (nr == 2) sq_launch<double2, double2, 2>(Ac, x, y, a, cg.Vc, nrhs, r0, st);
    else if (nr <= 4) sq_launch<double2, double2, 4>(Ac, x, y, a, cg.Vc, nrhs, r0, st);
    else sq_launch<double2, double2, 8>(Ac, x, y, a, cg.Vc, nrhs, r0, st);
  }
}

static bool sq_ordered_launch(const float2* A, const float2* x, float2* y, const SqArgs& a, const CoarseGeometry& cg, int nrhs,
                              hipStream_t st) {
  const int nr = sq_ordered_group(cg.Vc, cg.n2, nrhs);
  if (nr == 0) return false;
  const bool done = with_sq_n2(cg.n2, [&](auto N) {
    constexpr int N2 = decltype(N)::value;
    const dim3 grid(cg.Vc, ceil_div(nrhs, nr)), blk(576);
#define MG_SQO(NR) hipLaunchKernelGGL((k_sq_ordered<N2, NR>), grid, blk, 0, st, A, x, y, a, nrhs)
    if (nr == 1) MG_SQO(1);
    else if (nr == 2) MG_SQO(2);
    else if (nr == 3) MG_SQO(3);
    else MG_SQO(4);
#undef MG_SQO
  });
  if (done) MG_LAUNCH_CHECK();
  return done;
}

template <class O2>
void sq_apply32(const float2* Ac32, const float2* x, O2* y, const CoarseGeometry& cg, int nrhs, hipStream_t st,
                bool keep_order) {
  if (cg.n2 > 64) fail(MGDWF_ERR_INVALID_ARG, "2*nvec above 64 is not supported");
  SqStep<float2> q{};
  q.x = x;
  if (!keep_order && sq_mfma_launch<float2, O2, false>(Ac32, y, q, cg, nrhs, st)) return;
  const SqArgs a = sq_args(cg);
  if constexpr (std::is_same<O2, float2>::value)
    if (keep_order && sq_ordered_launch(Ac32, x, y, a, cg, nrhs, st)) return;
  for (int r0 = 0; r0 < nrhs; r0 += 16) {
    const int nr = std::min(16, nrhs - r0);
    if (nr == 1) sq_launch<float2, float2, 1>(Ac32, x, y, a, cg.Vc, nrhs, r0, st);
    else if (nr == 2) sq_launch<float2, float2, 2>(Ac32, x, y, a, cg.Vc, nrhs, r0, st);
    else if (nr <= 4) sq_launch<float2, float2, 4>(Ac32, x, y, a, cg.Vc, nrhs, r0, st);
    else if (nr <= 8) sq_launch<float2, float2, 8>(Ac32, x, y, a, cg.Vc, nrhs, r0, st);
    else if (nr <= 12) sq_launch<float2, float2, 12>(Ac32, x, y, a, cg.Vc, nrhs, r0, st);
    else sq_launch<float2, float2, 16>(Ac32, x, y, a, cg.Vc, nrhs, r0, st);
  }
}

template void sq_apply32<float2>(const float2*, const float2*, float2*, const CoarseGeometry&, int, hipStream_t, bool);
template void sq_apply32<double2>(const float2*, const float2*, double2*, const CoarseGeometry&, int, hipStream_t,
                                  bool);

}  // namespace mgdwf

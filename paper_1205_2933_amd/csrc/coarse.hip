// Coarse operator D_c = R D P: construction and 9-point application.
//
// Paper, Sec. 2 (third V-cycle step): the coarse problem uses R A P.  Sec. 4:
// coarsening the unsquared operator keeps a one-hop stencil; with blocks that
// span the fifth dimension, a coarse site couples to itself and its eight 4D
// neighbours only.
//
// Construction: column j = (chi', k') of every block is obtained at once for
// all blocks: the face-split operator applied to the chirality-chi' part of
// basis field k' gives nine fields -- the self part (diagonal, fifth-dimension
// hops and block-interior hops) and the eight block-face hops; restricting
// field d gives column j of Dc[B][d] for every block B.  A hop from x to x+mu
// belongs to d = +mu exactly when x is on the upper face of its block, a hop
// to x-mu to d = -mu exactly when x is on the lower face, which keeps the
// stencil exact when a coarse extent is 1 or 2 (neighbours coincide).
//
// Internal storage of a block: column major, element (row r, col c) of
// Dc[X][d] at ((X * 9 + d) * n2 + c) * n2 + r, so that lane r of a wavefront
// reads consecutive addresses for a fixed column.
#include <algorithm>
#include <type_traits>

#include <hip/hip_runtime.h>

#include "mg_internal.h"
#include "blas.h"
#include "vecops.h"

namespace mgdwf {

// from dslash.hip
void dslash_split(const double2* in, double2* out9, const double2* gauge, const Geometry& g, const int block[4],
                  double M5, double mf, int chi, hipStream_t st, bool dagger = false);

namespace {

// Dc columns j0 .. j0 + nb - 1 for all (X, d): coarse[j - j0][d][X][row] (from the
// restriction of field d) -> Dc[((X*9 + d)*n2 + j)*n2 + row].
__global__ void k_scatter_columns(const double2* __restrict__ coarse, double2* __restrict__ Dc, int Vc,
                                  int n2, int j0, int nb) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  long long tot = 9LL * Vc * n2 * nb;
  if (i >= tot) return;
  int row = (int)(i % n2);
  long long t = i / n2;
  int X = (int)(t % Vc), dj = (int)(t / Vc);
  Dc[(((long long)X * 9 + dj % 9) * n2 + j0 + dj / 9) * n2 + row] = coarse[i];
}

struct CoarseArgs {
  int Lc[4];
  int Vc;
  int n2;
};

CoarseArgs coarse_args(const CoarseGeometry& cg) {
  CoarseArgs a;
  for (int m = 0; m < 4; ++m) a.Lc[m] = cg.Lc[m];
  a.Vc = cg.Vc;
  a.n2 = cg.n2;
  return a;
}

__device__ __forceinline__ int opposite(int d) { return d == 0 ? 0 : (((d - 1) ^ 1) + 1); }

__device__ __forceinline__ int coarse_neighbour(const CoarseArgs& a, int X, int d) {
  if (d == 0) return X;
  const int mu = (d - 1) >> 1;
  const int sgn = (d & 1) ? 1 : -1;  // d = 1 + 2 mu is +mu
  int c[4];
  int r = X;
  c[0] = r % a.Lc[0]; r /= a.Lc[0];
  c[1] = r % a.Lc[1]; r /= a.Lc[1];
  c[2] = r % a.Lc[2]; c[3] = r / a.Lc[2];
  c[mu] = (c[mu] + sgn + a.Lc[mu]) % a.Lc[mu];
  return ((c[3] * a.Lc[2] + c[2]) * a.Lc[1] + c[1]) * a.Lc[0] + c[0];
}

// Adjoint stencil in the same form as D_c: (D_c^+ y)(X) = sum_e DcH[X][e] y(X + delta_e)
// with DcH[X][e] = Dc[X + delta_e][opposite(e)]^+.  Column-major blocks on both sides.
__global__ void k_adjoint_blocks(const double2* __restrict__ Dc, double2* __restrict__ DcH, CoarseArgs a) {
  const int blk = blockIdx.x;  // X * 9 + e
  const int X = blk / 9, e = blk % 9;
  const int Y = coarse_neighbour(a, X, e);
  const int n2 = a.n2;
  const double2* src = Dc + ((long long)Y * 9 + opposite(e)) * n2 * n2;
  double2* dst = DcH + (long long)blk * n2 * n2;
  for (int i = threadIdx.x; i < n2 * n2; i += blockDim.x) {
    const int r = i % n2, c = i / n2;           // dst element (r, c), column major
    const double2 v = src[(long long)r * n2 + c]; // src element (c, r)
    dst[i] = make_double2(v.x, -v.y);
  }
}

// y[rhs] = sum_d M[X][d] x[rhs](X + delta_d) for up to NR right-hand sides, each
// block read once for all of them.  Workgroup = one coarse site, 9 wavefronts,
// one per stencil direction d; lane = output row; the nine partial sums are
// added in a fixed order through LDS.
template <class MC2, class VC2, class O2, int NR>
__global__ __launch_bounds__(576) void k_capply(const MC2* __restrict__ M, const VC2* __restrict__ x,
                                                O2* __restrict__ y, CoarseArgs a, int nrhs, int rhs0) {
  using T = typename real_of<VC2>::type;
  __shared__ T red[NR][64][2];
  const int X = blockIdx.x;
  const int n2 = a.n2;
  const int d = threadIdx.x >> 6, row = threadIdx.x & 63;  // one wavefront per stencil direction
  const int nr = min(NR, nrhs - rhs0);
  const long long vs = (long long)a.Vc * n2;  // RHS stride
  VC2 acc[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) acc[j] = cmk<VC2>(0, 0);
  if (row < n2) {
    const int Y = coarse_neighbour(a, X, d);
    const MC2* Md = M + ((long long)X * 9 + d) * n2 * n2;
    const VC2* xv = x + (long long)rhs0 * vs + (long long)Y * n2;
    for (int c = 0; c < n2; ++c) {
      const MC2 m = Md[c * n2 + row];
      const VC2 mv = cmk<VC2>((T)m.x, (T)m.y);
#pragma unroll
      for (int j = 0; j < NR; ++j)
        if (j < nr) cfma(acc[j], mv, xv[j * vs + c]);
    }
  }
  // add the nine directions in a fixed order (bitwise reproducible)
  for (int w = 0; w < 9; ++w) {
    if (d == w)
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        if (w == 0) { red[j][row][0] = acc[j].x; red[j][row][1] = acc[j].y; }
        else { red[j][row][0] += acc[j].x; red[j][row][1] += acc[j].y; }
      }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < nr * n2; i += blockDim.x) {
    const int j = i / n2, r = i % n2;
    y[(long long)(rhs0 + j) * vs + (long long)X * n2 + r] = cmk<O2>(red[j][r][0], red[j][r][1]);
  }
}

__global__ void k_dc_to_f32(const double2* __restrict__ in, float2* __restrict__ out, long long n) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    out[i] = make_float2((float)in[i].x, (float)in[i].y);
}

// ---------------------------------------------------------------- 16-bit storage
// FP16: the hardware conversion (round to nearest even).  BF16: round to
// nearest even on the upper half of the IEEE single (NaN kept quiet).
__device__ __forceinline__ uint16_t to_f16(float v) {
  _Float16 h = (_Float16)v;
  return __builtin_bit_cast(uint16_t, h);
}
__device__ __forceinline__ uint16_t to_bf16(float v) {
  uint32_t b = __builtin_bit_cast(uint32_t, v);
  if ((b & 0x7f800000u) == 0x7f800000u && (b & 0x007fffffu)) return (uint16_t)((b >> 16) | 0x40);
  b += 0x7fffu + ((b >> 16) & 1u);
  return (uint16_t)(b >> 16);
}

template <bool BF>
__device__ __forceinline__ uint16_t to16(float v) { return BF ? to_bf16(v) : to_f16(v); }

// One workgroup per block (X, d): scale = max |Re|, |Im| over the block; store
// Re/scale and Im/scale row major (row r, col c at r * n2 + c).
template <bool BF>
__global__ __launch_bounds__(256) void k_pack_blocks(const double2* __restrict__ M, uint16_t* __restrict__ re,
                                                     uint16_t* __restrict__ im, float* __restrict__ sc, int n2) {
  __shared__ double wmax[4];
  const long long blk = blockIdx.x;
  const double2* src = M + blk * n2 * n2;
  double mx = 0.0;
  for (int i = threadIdx.x; i < n2 * n2; i += 256) mx = fmax(mx, fmax(fabs(src[i].x), fabs(src[i].y)));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = mx;
  __syncthreads();
  const double s = fmax(fmax(wmax[0], wmax[1]), fmax(wmax[2], wmax[3]));
  const double inv = s > 0.0 ? 1.0 / s : 0.0;
  if (threadIdx.x == 0) sc[blk] = (float)s;
  for (int i = threadIdx.x; i < n2 * n2; i += 256) {
    const int r = i / n2, c = i % n2;
    const double2 v = src[(long long)c * n2 + r];
    re[blk * n2 * n2 + i] = to16<BF>((float)(v.x * inv));
    im[blk * n2 * n2 + i] = to16<BF>((float)(v.y * inv));
  }
}

// Coarse vectors -> 16-bit with one scale per (site, RHS):
// xp[(rhs * Vc + X) * 2 n2 + k] = Re x_k / s, [.. + n2 + k] = Im x_k / s.
// One wavefront per (RHS, site), lane k < n2 <= 64 handles component k.
template <bool BF, class I2>
__global__ __launch_bounds__(256) void k_pack_vec(const I2* __restrict__ x, uint16_t* __restrict__ xp,
                                                  float* __restrict__ xs, int Vc, int n2, int nrhs) {
  const long long i = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int k = threadIdx.x & 63;
  if (i >= (long long)nrhs * Vc) return;  // whole wavefronts leave together
  float2 v = make_float2(0.f, 0.f);
  if (k < n2) {
    const I2 q = x[i * n2 + k];
    v = make_float2((float)q.x, (float)q.y);
  }
  float mx = fmaxf(fabsf(v.x), fabsf(v.y));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  const float inv = mx > 0.f ? 1.f / mx : 0.f;
  if (k == 0) xs[i] = mx;
  if (k < n2) {
    uint16_t* o = xp + i * 2 * n2;
    o[k] = to16<BF>(v.x * inv);
    o[n2 + k] = to16<BF>(v.y * inv);
  }
}

typedef _Float16 h4v __attribute__((ext_vector_type(4)));
typedef short s4v __attribute__((ext_vector_type(4)));
typedef _Float16 h8v __attribute__((ext_vector_type(8)));
typedef __bf16 b8v __attribute__((ext_vector_type(8)));
typedef float f4v __attribute__((ext_vector_type(4)));

// One MFMA on 16x16x16 (uint2: four k per lane) or gfx950's 16x16x32 tiles
// (uint4: eight k per lane), FP16 or BF16 inputs, FP32 accumulation.
// Whatever order the hardware gives the k-slots, A's and B's slot (lane group,
// element) hold the same k, so the tile sum is the full contraction.
template <bool BF>
__device__ __forceinline__ f4v mfma16(uint2 a, uint2 b, f4v c) {
  if (BF) return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s4v, a), __builtin_bit_cast(s4v, b), c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(h4v, a), __builtin_bit_cast(h4v, b), c, 0, 0, 0);
}
template <bool BF>
__device__ __forceinline__ f4v mfma16(uint4 a, uint4 b, f4v c) {
  if (BF) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8v, a), __builtin_bit_cast(b8v, b), c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8v, a), __builtin_bit_cast(h8v, b), c, 0, 0, 0);
}
__device__ __forceinline__ uint2 negate16(uint2 v) { return make_uint2(v.x ^ 0x80008000u, v.y ^ 0x80008000u); }
__device__ __forceinline__ uint4 negate16(uint4 v) {
  return make_uint4(v.x ^ 0x80008000u, v.y ^ 0x80008000u, v.z ^ 0x80008000u, v.w ^ 0x80008000u);
}

// ---- the product at one coarse site, up to 16 right-hand sides, on MFMA
//
// y(X) = sum_d M[X][d] x(X + delta_d).  A workgroup of nine wavefronts owns the
// site, wavefront d the direction d; the tile columns are the right-hand sides.
// The rows of [Re M, Im M] (N2 x 2 N2) are loaded once and multiplied with
// [Re x; -Im x] for Re y and with [Im x; Re x] for Im y.  Bound by the latency
// of one round of loads (few sites) or by the bytes of M (many): N2 is a
// template argument, so every load of the round is issued before the first
// product waits for one.  With N2 at run time each tile's load waited for the
// one before it: at 48 dof and FP16, 12.6 us on 32 sites (12 right-hand sides)
// and 25.8 us on 512 (one), against 8.4 and 11.9 us for the CGNE steps below,
// whose vector updates and sums are included.
// Each wavefront leaves its tiles in its slab of LDS ([col][row], Re rows then
// Im rows); slab_sum adds the nine in a fixed order.
template <int N2> __host__ __device__ constexpr int slab_stride() { return 2 * N2 + 4; }
template <int N2> __host__ __device__ constexpr int slab_floats() { return 9 * 16 * slab_stride<N2>(); }

template <int N2>
__device__ __forceinline__ float2 slab_sum(const float* slab, int col, int row) {
  double re = 0.0, im = 0.0;  // FP64: the sum over directions adds no rounding of its own
#pragma unroll
  for (int d = 0; d < 9; ++d) {
    const float* q = slab + (d * 16 + col) * slab_stride<N2>() + row;
    re += q[0];
    im += q[N2];
  }
  return make_float2((float)re, (float)im);
}

template <int N2>
__device__ __forceinline__ void slab_write(float* slab, const f4v* re, const f4v* im, float s) {
  const int d = threadIdx.x >> 6, col = threadIdx.x & 15, kq = (threadIdx.x & 63) >> 4;
  float* q = slab + (d * 16 + col) * slab_stride<N2>() + 4 * kq;
#pragma unroll
  for (int mt = 0; mt < N2 / 16; ++mt) {
    *reinterpret_cast<f4v*>(q + mt * 16) = s * re[mt];
    *reinterpret_cast<f4v*>(q + N2 + mt * 16) = s * im[mt];
  }
}

// 16-bit store: 16x16x16 tiles (SHAPE 0) or 16x16x32 tiles (SHAPE 1).  Each
// direction's sum is rescaled by (block scale) x (input scale of its RHS).
template <bool BF, int N2, int SHAPE>
struct Site16 {
  static constexpr int KL = SHAPE == 1 ? 8 : 4;  // consecutive k per lane
  static constexpr int MT = N2 / 16, KT = 2 * N2 / (4 * KL);
  using V = typename std::conditional<SHAPE == 1, uint4, uint2>::type;
  V av[MT][KT], b1[KT], b2[KT];
  float sc;

  // issue the site's loads (xp: packed [rhs][site][Re, Im], xs: its scales)
  __device__ __forceinline__ void load(const uint16_t* Are, const uint16_t* Aim, const float* Asc, const uint16_t* xp,
                                       const float* xs, const CoarseArgs& a, int nrhs, int X, int rhs0) {
    const int d = threadIdx.x >> 6, l = threadIdx.x & 63, kq = l >> 4;
    const int rhs = rhs0 + (l & 15);
    const bool valid = rhs < nrhs;
    const long long blk = (long long)X * 9 + d;
    const long long base = blk * N2 * N2 + (long long)(l & 15) * N2;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const int k = (kt * 4 + kq) * KL;
      const uint16_t* src = (k >= N2 ? Aim - N2 : Are) + base + k;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) av[mt][kt] = *reinterpret_cast<const V*>(src + mt * 16 * N2);
    }
    const int Y = coarse_neighbour(a, X, d);
    const long long iv = (long long)(valid ? rhs : 0) * a.Vc + Y;
    const uint16_t* xrow = xp + iv * 2 * N2;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const int k = (kt * 4 + kq) * KL;
      b1[kt] = *reinterpret_cast<const V*>(xrow + k);
      b2[kt] = *reinterpret_cast<const V*>(xrow + (k >= N2 ? k - N2 : k + N2));
    }
    sc = Asc[blk] * (valid ? xs[iv] : 0.f);
  }
  // the products into this wavefront's slab; no barrier.  The columns past
  // the last right-hand side repeat its row 0 with scale 0.
  __device__ __forceinline__ void multiply(float* slab) {
    f4v re[MT], im[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) re[mt] = im[mt] = f4v{0.f, 0.f, 0.f, 0.f};
    const int kq = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const V bm = (kt * 4 + kq) * KL >= N2 ? negate16(b1[kt]) : b1[kt];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        re[mt] = mfma16<BF>(av[mt][kt], bm, re[mt]);
        im[mt] = mfma16<BF>(av[mt][kt], b2[kt], im[mt]);
      }
    }
    slab_write<N2>(slab, re, im, sc);
  }
};

// FP32 store (column-major float2 blocks) on 16x16x4 FP32 tiles: exact FP32
// products, FP32 accumulation.  The vectors are read as they are.
template <int N2>
struct Site32 {
  static constexpr int MT = N2 / 16, KT = N2 / 4;
  const float2* A;
  const float2* xv;
  bool valid;
  __device__ __forceinline__ void load(const float2* M, const float2* x, const CoarseArgs& a, int nrhs, int X, int rhs0) {
    const int d = threadIdx.x >> 6, l = threadIdx.x & 63, kq = l >> 4;
    const int rhs = rhs0 + (l & 15);
    valid = rhs < nrhs;
    A = M + ((long long)X * 9 + d) * N2 * N2 + kq * N2 + (l & 15);
    xv = x + ((long long)(valid ? rhs : 0) * a.Vc + coarse_neighbour(a, X, d)) * N2 + kq;
  }
  __device__ __forceinline__ void multiply(float* slab) {
    f4v re[MT], im[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) re[mt] = im[mt] = f4v{0.f, 0.f, 0.f, 0.f};
    constexpr int KC = KT < 6 ? KT : (KT % 6 == 0 ? 6 : 4);  // k-tiles in flight together
#pragma unroll
    for (int k0 = 0; k0 < KT; k0 += KC) {
      float2 m[MT][KC], v[KC];
#pragma unroll
      for (int q = 0; q < KC; ++q) {
        v[q] = xv[4 * (k0 + q)];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) m[mt][q] = A[4 * (k0 + q) * N2 + mt * 16];
      }
#pragma unroll
      for (int q = 0; q < KC; ++q) {
        const float xr = valid ? v[q].x : 0.f, xi = valid ? v[q].y : 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          re[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(m[mt][q].x, xr, re[mt], 0, 0, 0);
          im[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(m[mt][q].x, xi, im[mt], 0, 0, 0);
          re[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(m[mt][q].y, -xi, re[mt], 0, 0, 0);
          im[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(m[mt][q].y, xr, im[mt], 0, 0, 0);
        }
      }
    }
    slab_write<N2>(slab, re, im, 1.f);
  }
};

// y = D_c x from a 16-bit store; y as FP32 or FP64 complex numbers
template <bool BF, int N2, int SHAPE, class O2>
__global__ __launch_bounds__(576) void k_capply16(const uint16_t* __restrict__ Are, const uint16_t* __restrict__ Aim,
                                                  const float* __restrict__ Asc, const uint16_t* __restrict__ xp,
                                                  const float* __restrict__ xs, O2* __restrict__ y, CoarseArgs a,
                                                  int nrhs) {
  __shared__ __align__(16) float slab[slab_floats<N2>()];
  const int X = blockIdx.x, rhs0 = blockIdx.y * 16, w = threadIdx.x >> 6, l = threadIdx.x & 63;
  Site16<BF, N2, SHAPE> s;
  s.load(Are, Aim, Asc, xp, xs, a, nrhs, X, rhs0);
  s.multiply(slab);
  __syncthreads();
  for (int c = w; c < min(16, nrhs - rhs0); c += 9)
    if (l < N2) {
      const float2 v = slab_sum<N2>(slab, c, l);
      y[((long long)(rhs0 + c) * a.Vc + X) * N2 + l] = cmk<O2>(v.x, v.y);
    }
}

// y = D_c x from the FP32 store
template <int N2, class O2>
__global__ __launch_bounds__(576) void k_capply32(const float2* __restrict__ M, const float2* __restrict__ x,
                                                  O2* __restrict__ y, CoarseArgs a, int nrhs) {
  __shared__ __align__(16) float slab[slab_floats<N2>()];
  const int X = blockIdx.x, rhs0 = blockIdx.y * 16, w = threadIdx.x >> 6, l = threadIdx.x & 63;
  Site32<N2> s;
  s.load(M, x, a, nrhs, X, rhs0);
  s.multiply(slab);
  __syncthreads();
  for (int c = w; c < min(16, nrhs - rhs0); c += 9)
    if (l < N2) {
      const float2 v = slab_sum<N2>(slab, c, l);
      y[((long long)(rhs0 + c) * a.Vc + X) * N2 + l] = cmk<O2>(v.x, v.y);
    }
}

// ---- coarse CGNE, two launches per iteration
//
// The r-step applies D_c to p and, at its own site, moves x and r; the p-step
// applies D_c^+ to r and forms the new p.  A launch also needs one sum over all
// sites per right-hand side (|p|^2 for the r-step, the new |r|^2 for the
// p-step): every workgroup adds the per-site partials the launch before left,
// in the same fixed order, while its matrix loads are in flight.  Eight
// launches (two packings, two products, two updates, two sums) took 48 us per
// iteration on 32 sites with 12 right-hand sides and 81 us on 512 with one;
// the two take 17 and 24 us.
// Every workgroup reads all partials of its right-hand sides, so their traffic
// grows as sites^2: at kPartMax (8192 partials, 64 KB per workgroup) it equals
// the 16-bit matrix's own (83 KB per site at 48 dof, read from the same
// caches); above, k_finalize_rhs (4 to 6 us) adds them first (np = 1, pstride =
// NSLOT).
struct CgneStep {
  const double* part_in;  // right-hand side r: np partials at part_in + r * pstride
  int np, pstride;
  double* part_out;       // per (rhs, site), stride Vc
  double* sl;             // slot table: |r|^2 of the current r at cur
  int cur, nxt, aux;      // p-step: the sum goes to nxt (and to aux when >= 0)
  int first;              // r-step: x = alpha p; p-step: p = t
  float2 *x, *r, *p;
  uint16_t *rp, *pp;      // packed r and p (16-bit stores only)
  float *rs, *ps;
};

__device__ __forceinline__ double part_sum(const CgneStep& q, int rhs) {
  const double* s = q.part_in + (long long)rhs * q.pstride;
  double v = 0.0;
#pragma unroll 8
  for (int i = threadIdx.x & 63; i < q.np; i += 64) v += s[i];
  return wave_sum(v);
}

// one wavefront: v (lane k < N2) -> 16 bits with one scale, and |v|^2
template <bool BF, int N2>
__device__ __forceinline__ void pack_wave(float2 v, uint16_t* o, float* scale) {
  const int l = threadIdx.x & 63;
  float mx = fmaxf(fabsf(v.x), fabsf(v.y));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  const float inv = mx > 0.f ? 1.f / mx : 0.f;
  if (l == 0) *scale = mx;
  if (l < N2) {
    o[l] = to16<BF>(v.x * inv);
    o[N2 + l] = to16<BF>(v.y * inv);
  }
}

// KIND 0: FP32 store, 1: FP16, 2: BF16.  STEP 0: r-step (M = D_c), 1: p-step (M = D_c^+).
template <int KIND, int N2, int SHAPE, int STEP>
__global__ __launch_bounds__(576, N2 <= 48 ? 5 : 3) void k_cgne_step(const void* __restrict__ M0, const uint16_t* __restrict__ Aim,
                                                   const float* __restrict__ Asc, CgneStep q, CoarseArgs a, int nrhs) {
  __shared__ __align__(16) float slab[slab_floats<N2>()];
  const int X = blockIdx.x, rhs0 = blockIdx.y * 16, w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int nr = min(16, nrhs - rhs0);
  typename std::conditional<KIND == 0, Site32<N2>, Site16<KIND == 2, N2, SHAPE>>::type s;
  if constexpr (KIND == 0)
    s.load(static_cast<const float2*>(M0), STEP == 0 ? q.p : q.r, a, nrhs, X, rhs0);
  else
    s.load(static_cast<const uint16_t*>(M0), Aim, Asc, STEP == 0 ? q.pp : q.rp, STEP == 0 ? q.ps : q.rs, a, nrhs, X, rhs0);
  // this wavefront's right-hand sides, w and w + 9: their own entries and sums
  float2 pv[2], xv[2], rv[2];
  double sum[2] = {0.0, 0.0};
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int c = w + 9 * j;
    pv[j] = xv[j] = rv[j] = make_float2(0.f, 0.f);
    if (c < nr) {
      if (l < N2) {
        const long long i = ((long long)(rhs0 + c) * a.Vc + X) * N2 + l;
        if (STEP == 0 || !q.first) pv[j] = q.p[i];
        if (STEP == 0) {
          rv[j] = q.r[i];
          if (!q.first) xv[j] = q.x[i];
        }
      }
      sum[j] = part_sum(q, rhs0 + c);
    }
  }
  s.multiply(slab);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int c = w + 9 * j;
    if (c < nr) {
      const int rhs = rhs0 + c;
      const long long site = (long long)rhs * a.Vc + X, i = site * N2 + l;
      const float2 t = l < N2 ? slab_sum<N2>(slab, c, l) : make_float2(0.f, 0.f);
      double* sr = q.sl + (long long)rhs * NSLOT;
      float2 v;
      if (STEP == 0) {  // sum = |p|^2
        const float alpha = (float)(sum[j] > 0.0 ? sr[q.cur] / sum[j] : 0.0);
        v = make_float2(rv[j].x - alpha * t.x, rv[j].y - alpha * t.y);
        if (l < N2) {
          q.x[i] = make_float2(xv[j].x + alpha * pv[j].x, xv[j].y + alpha * pv[j].y);
          q.r[i] = v;
        }
      } else {  // sum = the new |r|^2
        const double rr = q.first ? 0.0 : sr[q.cur];
        const float beta = (float)(rr > 0.0 ? sum[j] / rr : 0.0);
        v = make_float2(t.x + beta * pv[j].x, t.y + beta * pv[j].y);
        if (l < N2) q.p[i] = v;
        if (X == 0 && l == 0) {
          sr[q.nxt] = sum[j];
          if (q.aux >= 0) sr[q.aux] = sum[j];
        }
      }
      if constexpr (KIND != 0)
        pack_wave<KIND == 2, N2>(v, (STEP == 0 ? q.rp : q.pp) + site * 2 * N2, (STEP == 0 ? q.rs : q.ps) + site);
      const double nn = wave_sum((double)v.x * v.x + (double)v.y * v.y);
      if (l == 0) q.part_out[site] = nn;
    }
  }
}

// r = b with its packing and per-site |r|^2; one wavefront per (rhs, site)
template <int KIND, int N2>
__global__ __launch_bounds__(256) void k_cgne_start(const float2* __restrict__ b, CgneStep q, long long nsites) {
  const long long site = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int l = threadIdx.x & 63;
  if (site >= nsites) return;  // whole wavefronts leave together
  const float2 v = l < N2 ? b[site * N2 + l] : make_float2(0.f, 0.f);
  if (l < N2) q.r[site * N2 + l] = v;
  if constexpr (KIND != 0) pack_wave<KIND == 2, N2>(v, q.rp + site * 2 * N2, q.rs + site);
  const double nn = wave_sum((double)v.x * v.x + (double)v.y * v.y);
  if (l == 0) q.part_out[site] = nn;
}

// ---------------------------------------------------------------- persistent coarse CGNE
// The coarse solve (CGNE on D_c D_c^+ y = b, x = D_c^+ y, from x = 0) as one
// cooperative launch of at most one workgroup per CU; workgroup w owns the
// coarse sites w, w + G, w + 2G, ... (G workgroups), every RHS (<= 16) at
// once.  Per iteration: q = D_c p at each own site, then x += alpha p and
// r -= alpha q there (alpha = |r|^2 / |p|^2), r packed to 16 bits with its
// per-site |r|^2; grid barrier; |r|^2 summed over all sites (each workgroup
// sums the same partials in the same order, so all take the same decision);
// t = D_c^+ r, p = t + beta p (beta = |r_new|^2 / |r|^2), p packed with its
// |p|^2; grid barrier.  The loop ends when every RHS has |r|^2 <= tol^2 |b|^2
// at one of the tests after every 8th iteration (as in the launched loop), or
// after maxiter iterations; the last iteration skips the D_c^+ apply, whose
// result nobody reads.
//
// The grid barrier is this file's own: an arrival counter and a generation
// word in device memory, agent-scope release/acquire, and a wait bounded in
// wall-clock time.  A wait that runs out sets the error word, and every
// workgroup that sees it leaves the kernel, so a barrier that can never
// complete ends the launch with an error instead of hanging it.
__global__ void k_zero_words(int* p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0;
}

struct GridSync {
  unsigned count;  // arrivals in the current generation
  unsigned gen;    // generation, bumped by the last arrival
  int err;         // set by a wait that ran out of time
  int pad;
};

struct PersistArgs {
  const uint16_t *Are, *Aim, *Hre, *Him;  // 16-bit D_c and D_c^+ (the adjoint stencil)
  const float *Asc, *Hsc;
  const float2* b;
  float2 *x, *r, *p;
  uint16_t *rp, *pp;     // packed r and p: [rhs][X][2 n2]
  float *rs, *ps;        // their per-(rhs, X) scales
  double *part_r, *part_p;  // per-(rhs, X) |.|^2
  long long* count;      // coarse applications are added here (one thread)
  GridSync* gs;          // zeroed before the launch
  long long wait_ticks;  // bound of one barrier wait, in wall-clock ticks
  double tol2;
  int maxiter, nrhs;
  CoarseArgs a;
};

// Every thread of every workgroup calls it; returns false (the same in every
// thread of the workgroup) when the barrier failed and the kernel must end.
__device__ bool grid_barrier(GridSync* gs, unsigned nblocks, long long wait_ticks, int* ok_lds) {
  __syncthreads();
  if (threadIdx.x == 0) {
    int ok = 1;
    const unsigned g = __hip_atomic_load(&gs->gen, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned arrived = __hip_atomic_fetch_add(&gs->count, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (arrived == nblocks - 1) {
      __hip_atomic_store(&gs->count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&gs->gen, g + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      const long long t0 = wall_clock64();
      while (__hip_atomic_load(&gs->gen, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == g) {
        if (__hip_atomic_load(&gs->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ||
            wall_clock64() - t0 > wait_ticks) {
          __hip_atomic_store(&gs->err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          ok = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(2);
      }
    }
    if (__hip_atomic_load(&gs->err, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) != 0) ok = 0;
    *ok_lds = ok;
  }
  __syncthreads();
  return *ok_lds != 0;
}

template <bool BF, int N2>
__global__ __launch_bounds__(576) void k_cgne_persistent(PersistArgs q) {
  __shared__ __align__(16) float slab[slab_floats<N2>()];
  __shared__ float2 v[16][64];  // the current site's new r or p, per RHS
  __shared__ double rr0[16], rr[16], pp[16], rn[16];
  __shared__ int ok_lds;
  const CoarseArgs& a = q.a;
  constexpr int n2 = N2;
  const int nrhs = q.nrhs, Vc = a.Vc;
  const int G = gridDim.x;
  // y(X) into the slabs; the site index is opaque to the optimiser, so the
  // loop recomputes the operator addresses instead of holding them in registers
  auto apply = [&](const uint16_t* Mre, const uint16_t* Mim, const float* Msc, const uint16_t* xp, const float* xs,
                   int X) {
    asm volatile("" : "+s"(X));
    Site16<BF, N2, 1> s;
    s.load(Mre, Mim, Msc, xp, xs, a, nrhs, X, 0);
    s.multiply(slab);
    __syncthreads();
  };
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int ne = nrhs * n2;
  auto at = [&](int rhs, int X, int k) { return ((long long)rhs * Vc + X) * n2 + k; };
  // v -> 16-bit (one scale per RHS) at site X and |v|^2 per RHS; wave w takes RHS w, w + 9
  auto pack_site = [&](int X, uint16_t* xp, float* xs, double* part) {
    for (int rhs = w; rhs < nrhs; rhs += 9) {
      const float2 val = l < n2 ? v[rhs][l] : make_float2(0.f, 0.f);
      float mx = fmaxf(fabsf(val.x), fabsf(val.y));
      double nn = (double)val.x * val.x + (double)val.y * val.y;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        nn += __shfl_xor(nn, off, 64);
      }
      const float inv = mx > 0.f ? 1.f / mx : 0.f;
      const long long i = (long long)rhs * Vc + X;
      if (l == 0) {
        xs[i] = mx;
        part[i] = nn;
      }
      if (l < n2) {
        xp[i * 2 * n2 + l] = to16<BF>(val.x * inv);
        xp[i * 2 * n2 + n2 + l] = to16<BF>(val.y * inv);
      }
    }
    __syncthreads();  // v is rewritten for the next site
  };
  // dst[rhs] = sum over all sites of part[rhs][.], fixed order
  auto reduce_all = [&](const double* part, double* dst) {
    for (int rhs = w; rhs < nrhs; rhs += 9) {
      double s = 0.0;
      for (int Y = l; Y < Vc; Y += 64) s += part[(long long)rhs * Vc + Y];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
      if (l == 0) dst[rhs] = s;
    }
    __syncthreads();
  };
  auto barrier = [&]() { return grid_barrier(q.gs, (unsigned)G, q.wait_ticks, &ok_lds); };
  long long napp = 0;
  // x = 0, r = b, |b|^2
  for (int X = blockIdx.x; X < Vc; X += G) {
    for (int e = threadIdx.x; e < ne; e += blockDim.x) {
      const int rhs = e / n2, k = e - rhs * n2;
      const float2 bv = q.b[at(rhs, X, k)];
      q.x[at(rhs, X, k)] = make_float2(0.f, 0.f);
      q.r[at(rhs, X, k)] = bv;
      v[rhs][k] = bv;
    }
    __syncthreads();
    pack_site(X, q.rp, q.rs, q.part_r);
  }
  if (!barrier()) return;
  reduce_all(q.part_r, rr0);
  if (threadIdx.x < nrhs) rr[threadIdx.x] = rr0[threadIdx.x];
  // p = D_c^+ r, |p|^2
  for (int X = blockIdx.x; X < Vc; X += G) {
    apply(q.Hre, q.Him, q.Hsc, q.rp, q.rs, X);
    for (int e = threadIdx.x; e < ne; e += blockDim.x) {
      const int rhs = e / n2, k = e - rhs * n2;
      const float2 t = slab_sum<N2>(slab, rhs, k);
      q.p[at(rhs, X, k)] = t;
      v[rhs][k] = t;
    }
    __syncthreads();
    pack_site(X, q.pp, q.ps, q.part_p);
  }
  ++napp;
  if (!barrier()) return;
  reduce_all(q.part_p, pp);
  for (int it = 0; it < q.maxiter; ++it) {
    // q = D_c p; x += alpha p; r -= alpha q
    for (int X = blockIdx.x; X < Vc; X += G) {
      apply(q.Are, q.Aim, q.Asc, q.pp, q.ps, X);
      for (int e = threadIdx.x; e < ne; e += blockDim.x) {
        const int rhs = e / n2, k = e - rhs * n2;
        const float alpha = (float)(pp[rhs] > 0.0 ? rr[rhs] / pp[rhs] : 0.0);
        const long long i = at(rhs, X, k);
        const float2 pv = q.p[i], xv = q.x[i], rv = q.r[i];
        const float2 qv = slab_sum<N2>(slab, rhs, k);
        q.x[i] = make_float2(xv.x + alpha * pv.x, xv.y + alpha * pv.y);
        const float2 rn2 = make_float2(rv.x - alpha * qv.x, rv.y - alpha * qv.y);
        q.r[i] = rn2;
        v[rhs][k] = rn2;
      }
      __syncthreads();
      pack_site(X, q.rp, q.rs, q.part_r);
    }
    ++napp;
    if (!barrier()) return;
    reduce_all(q.part_r, rn);
    // the launched loop's schedule: the residual is tested after every 8th
    // iteration (the same decision in every workgroup)
    const int n = it + 1;
    bool done = n % 8 == 0;
    for (int rhs = 0; rhs < nrhs && done; ++rhs)
      if (!(rn[rhs] <= q.tol2 * rr0[rhs])) done = false;
    if (done || n == q.maxiter) break;
    // t = D_c^+ r; p = t + beta p
    for (int X = blockIdx.x; X < Vc; X += G) {
      apply(q.Hre, q.Him, q.Hsc, q.rp, q.rs, X);
      for (int e = threadIdx.x; e < ne; e += blockDim.x) {
        const int rhs = e / n2, k = e - rhs * n2;
        const float beta = (float)(rr[rhs] > 0.0 ? rn[rhs] / rr[rhs] : 0.0);
        const long long i = at(rhs, X, k);
        const float2 pv = q.p[i];
        const float2 s = slab_sum<N2>(slab, rhs, k);
        const float2 t = make_float2(s.x + beta * pv.x, s.y + beta * pv.y);
        q.p[i] = t;
        v[rhs][k] = t;
      }
      __syncthreads();
      pack_site(X, q.pp, q.ps, q.part_p);
    }
    ++napp;
    if (threadIdx.x < nrhs) rr[threadIdx.x] = rn[threadIdx.x];
    if (!barrier()) return;
    reduce_all(q.part_p, pp);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *q.count += napp;
}

}  // namespace

// Build the FP64 coarse operator, nb = `columns` columns at a time (the same bits for
// any).  Vhat: orthonormal basis (Nv FP64 fields); work9: 9 nb fine FP64 fields; cwork:
// 9 nb Vc n2 complex; partial: restriction scratch for 9 nb right-hand sides.
void build_coarse_op(const double2* Vhat, const double2* gauge, double2* Dc, double2* work9, double2* cwork,
                     double* partial, const Geometry& g, const CoarseGeometry& cg, double M5, double mf,
                     int columns, hipStream_t st) {
  const long long field = 12LL * g.V5;
  for (int j0 = 0; j0 < cg.n2; j0 += columns) {
    const int nb = std::min(columns, cg.n2 - j0);
    for (int q = 0; q < nb; ++q)  // column j = chi * Nv + k
      dslash_split(Vhat + (j0 + q) % cg.Nv * field, work9 + q * 9 * field, gauge, g, cg.block, M5, mf,
                   (j0 + q) / cg.Nv, st);
    restrict_op<double2, double2>(Vhat, work9, cwork, partial, g, cg, 9 * nb, st, false, 4);
    long long tot = 9LL * cg.Vc * cg.n2 * nb;
    hipLaunchKernelGGL(k_scatter_columns, dim3(ceil_div(tot, 256)), dim3(256), 0, st, cwork, Dc, cg.Vc, cg.n2, j0, nb);
    MG_LAUNCH_CHECK();
  }
}

static void pack_store(CoarseStore& s, const CoarseGeometry& cg, hipStream_t st) {
  const long long nblk = 9LL * cg.Vc, n = nblk * cg.n2 * cg.n2;
  s.m32.alloc(n * sizeof(float2));
  hipLaunchKernelGGL(k_dc_to_f32, dim3(std::min(ceil_div(n, 256), 8192)), dim3(256), 0, st, s.m64.as<double2>(),
                     s.m32.as<float2>(), n);
  MG_LAUNCH_CHECK();
  s.re16.alloc(n * 2); s.im16.alloc(n * 2); s.sc16.alloc(nblk * sizeof(float));
  s.reb.alloc(n * 2); s.imb.alloc(n * 2); s.scb.alloc(nblk * sizeof(float));
  hipLaunchKernelGGL(k_pack_blocks<false>, dim3(nblk), dim3(256), 0, st, s.m64.as<double2>(), s.re16.as<uint16_t>(),
                     s.im16.as<uint16_t>(), s.sc16.as<float>(), cg.n2);
  MG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_pack_blocks<true>, dim3(nblk), dim3(256), 0, st, s.m64.as<double2>(), s.reb.as<uint16_t>(),
                     s.imb.as<uint16_t>(), s.scb.as<float>(), cg.n2);
  MG_LAUNCH_CHECK();
}

// From Dc.m64: the adjoint stencil and the FP32 / FP16 / BF16 copies of both.
void finish_coarse_op(CoarseStore& Dc, CoarseStore& DcH, const CoarseGeometry& cg, hipStream_t st) {
  const long long nblk = 9LL * cg.Vc, n = nblk * cg.n2 * cg.n2;
  DcH.m64.alloc(n * sizeof(double2));
  hipLaunchKernelGGL(k_adjoint_blocks, dim3(nblk), dim3(256), 0, st, Dc.m64.as<double2>(), DcH.m64.as<double2>(),
                     coarse_args(cg));
  MG_LAUNCH_CHECK();
  pack_store(Dc, cg, st);
  pack_store(DcH, cg, st);
}

void coarse_apply64(const CoarseStore& s, const double2* x, double2* y, const CoarseGeometry& cg, int nrhs,
                    hipStream_t st) {
  if (cg.n2 > 64) fail(MGDWF_ERR_INVALID_ARG, "2*nvec above 64 is not supported");
  for (int r0 = 0; r0 < nrhs; r0 += 8) {
    hipLaunchKernelGGL((k_capply<double2, double2, double2, 8>), dim3(cg.Vc), dim3(576), 0, st, s.m64.as<double2>(), x, y,
                       coarse_args(cg), nrhs, r0);
    MG_LAUNCH_CHECK();
  }
}

size_t coarse_pack_bytes(const CoarseGeometry& cg, int nrhs) {
  return (size_t)nrhs * cg.Vc * (2 * cg.n2 * sizeof(uint16_t) + sizeof(float)) + 256;
}

// f(N2) with the coarse dof count as a compile-time constant; false where the
// MFMA kernels have none (2 Nv not a multiple of 16)
template <class F>
static bool with_n2(int n2, F&& f) {
  switch (n2) {
    case 16: f(std::integral_constant<int, 16>{}); return true;
    case 32: f(std::integral_constant<int, 32>{}); return true;
    case 48: f(std::integral_constant<int, 48>{}); return true;
    case 64: f(std::integral_constant<int, 64>{}); return true;
    default: return false;
  }
}

template <class I2, class O2>
void coarse_apply32(const CoarseStore& s, mgdwf_prec prec, const I2* x, O2* y, const CoarseGeometry& cg, int nrhs,
                    void* pack, int ctile, hipStream_t st) {
  if (cg.n2 > 64) fail(MGDWF_ERR_INVALID_ARG, "2*nvec above 64 is not supported");
  const CoarseArgs a = coarse_args(cg);
  const dim3 grid(cg.Vc, ceil_div(nrhs, 16));
  if (prec == MGDWF_F32 || prec == MGDWF_F64) {
    if constexpr (std::is_same<I2, float2>::value) {
      if (!with_n2(cg.n2, [&](auto N) {
            hipLaunchKernelGGL((k_capply32<decltype(N)::value, O2>), grid, dim3(576), 0, st, s.m32.as<float2>(), x, y, a,
                               nrhs);
          }))
        for (int r0 = 0; r0 < nrhs; r0 += 16)  // other dof counts: one lane per row
          hipLaunchKernelGGL((k_capply<float2, float2, O2, 16>), dim3(cg.Vc), dim3(576), 0, st, s.m32.as<float2>(), x,
                             y, a, nrhs, r0);
      MG_LAUNCH_CHECK();
    } else {
      fail(MGDWF_ERR_INVALID_ARG, "the FP32 coarse operator takes FP32 vectors");
    }
    return;
  }
  if (cg.n2 % 16) fail(MGDWF_ERR_INVALID_ARG, "16-bit coarse operator needs nvec divisible by 8");
  const bool bf = prec == MGDWF_BF16;
  uint16_t* xp = static_cast<uint16_t*>(pack);
  float* xs = reinterpret_cast<float*>(xp + (size_t)nrhs * cg.Vc * 2 * cg.n2);
  const long long nsv = (long long)nrhs * cg.Vc;
  if (bf)
    hipLaunchKernelGGL((k_pack_vec<true, I2>), dim3(ceil_div(nsv, 4)), dim3(256), 0, st, x, xp, xs, cg.Vc, cg.n2, nrhs);
  else
    hipLaunchKernelGGL((k_pack_vec<false, I2>), dim3(ceil_div(nsv, 4)), dim3(256), 0, st, x, xp, xs, cg.Vc, cg.n2, nrhs);
  MG_LAUNCH_CHECK();
  const uint16_t* re = (bf ? s.reb : s.re16).as<uint16_t>();
  const uint16_t* im = (bf ? s.imb : s.im16).as<uint16_t>();
  const float* sc = (bf ? s.scb : s.sc16).as<float>();
  with_n2(cg.n2, [&](auto N) {
    constexpr int N2 = decltype(N)::value;
#define MG_CA(BF, SH) hipLaunchKernelGGL((k_capply16<BF, N2, SH, O2>), grid, dim3(576), 0, st, re, im, sc, xp, xs, y, a, nrhs)
    if (bf && ctile == 1) MG_CA(true, 1);
    else if (bf) MG_CA(true, 0);
    else if (ctile == 1) MG_CA(false, 1);
    else MG_CA(false, 0);
#undef MG_CA
  });
  MG_LAUNCH_CHECK();
}
template void coarse_apply32<float2, float2>(const CoarseStore&, mgdwf_prec, const float2*, float2*,
                                             const CoarseGeometry&, int, void*, int, hipStream_t);
template void coarse_apply32<float2, double2>(const CoarseStore&, mgdwf_prec, const float2*, double2*,
                                              const CoarseGeometry&, int, void*, int, hipStream_t);
template void coarse_apply32<double2, double2>(const CoarseStore&, mgdwf_prec, const double2*, double2*,
                                               const CoarseGeometry&, int, void*, int, hipStream_t);

// ---- coarse CGNE on the fused steps
// Partials per launch up to which every workgroup adds them itself.
constexpr long long kPartMax = 8192;

bool cgne_fused(const CoarseGeometry& cg, mgdwf_prec prec) {
  return (prec == MGDWF_F32 || prec == MGDWF_F16 || prec == MGDWF_BF16) && cg.n2 % 16 == 0 && cg.n2 <= 64;
}

size_t cgne_fused_bytes(const CoarseGeometry& cg, int nrhs) {
  const size_t nsv = (size_t)nrhs * cg.Vc;
  return 2 * nsv * 2 * cg.n2 * sizeof(uint16_t) + 2 * nsv * sizeof(float) + 2 * nsv * sizeof(double) + 6 * 256;
}

static CgneStep cgne_carve(void* work, const CoarseGeometry& cg, int nrhs, float2* x, float2* r, float2* p,
                           double** part_r, double** part_p) {
  const size_t nsv = (size_t)nrhs * cg.Vc;
  char* w = static_cast<char*>(work);
  auto take = [&](size_t bytes) {
    char* q = w;
    w += (bytes + 255) / 256 * 256;
    return q;
  };
  CgneStep q{};
  q.x = x;
  q.r = r;
  q.p = p;
  q.rp = reinterpret_cast<uint16_t*>(take(nsv * 2 * cg.n2 * sizeof(uint16_t)));
  q.pp = reinterpret_cast<uint16_t*>(take(nsv * 2 * cg.n2 * sizeof(uint16_t)));
  q.rs = reinterpret_cast<float*>(take(nsv * sizeof(float)));
  q.ps = reinterpret_cast<float*>(take(nsv * sizeof(float)));
  *part_r = reinterpret_cast<double*>(take(nsv * sizeof(double)));
  *part_p = reinterpret_cast<double*>(take(nsv * sizeof(double)));
  q.aux = -1;
  return q;
}

// partials of the launch before: added in the kernel, or first by k_finalize_rhs into slot `tmp`
static void cgne_partials(CgneStep& q, const double* part, const CoarseGeometry& cg, int nrhs, double* sl, int tmp,
                          hipStream_t st) {
  q.sl = sl;
  if ((long long)std::min(nrhs, 16) * cg.Vc <= kPartMax) {
    q.part_in = part;
    q.np = q.pstride = cg.Vc;
  } else {
    finalize_rhs(part, cg.Vc, 1, sl, tmp, nrhs, st);
    q.part_in = sl + tmp;
    q.np = 1;
    q.pstride = NSLOT;
  }
}

template <int STEP>
static void cgne_launch(const CoarseStore& s, mgdwf_prec prec, int ctile, const CgneStep& q, const CoarseGeometry& cg,
                        int nrhs, hipStream_t st) {
  const dim3 grid(cg.Vc, ceil_div(nrhs, 16));
  const CoarseArgs a = coarse_args(cg);
  const bool bf = prec == MGDWF_BF16;
  const uint16_t* im = (bf ? s.imb : s.im16).as<uint16_t>();
  const float* sc = (bf ? s.scb : s.sc16).as<float>();
  with_n2(cg.n2, [&](auto N) {
    constexpr int N2 = decltype(N)::value;
#define MG_CS(K, SH, M) hipLaunchKernelGGL((k_cgne_step<K, N2, SH, STEP>), grid, dim3(576), 0, st, M, im, sc, q, a, nrhs)
    if (prec == MGDWF_F32) MG_CS(0, 0, s.m32.p);
    else if (bf && ctile == 1) MG_CS(2, 1, s.reb.p);
    else if (bf) MG_CS(2, 0, s.reb.p);
    else if (ctile == 1) MG_CS(1, 1, s.re16.p);
    else MG_CS(1, 0, s.re16.p);
#undef MG_CS
  });
  MG_LAUNCH_CHECK();
}

void cgne_fused_start(const CoarseStore& DH, mgdwf_prec prec, int ctile, const float2* b, float2* r, float2* p,
                      void* work, double* sl, int rr0, int cur, int tmp, const CoarseGeometry& cg, int nrhs,
                      hipStream_t st) {
  double *part_r, *part_p;
  CgneStep q = cgne_carve(work, cg, nrhs, nullptr, r, p, &part_r, &part_p);
  q.part_out = part_r;
  const long long nsv = (long long)nrhs * cg.Vc;
  with_n2(cg.n2, [&](auto N) {
    constexpr int N2 = decltype(N)::value;
    const dim3 grid(ceil_div(nsv, 4));
    if (prec == MGDWF_F32) hipLaunchKernelGGL((k_cgne_start<0, N2>), grid, dim3(256), 0, st, b, q, nsv);
    else if (prec == MGDWF_BF16) hipLaunchKernelGGL((k_cgne_start<2, N2>), grid, dim3(256), 0, st, b, q, nsv);
    else hipLaunchKernelGGL((k_cgne_start<1, N2>), grid, dim3(256), 0, st, b, q, nsv);
  });
  MG_LAUNCH_CHECK();
  cgne_partials(q, part_r, cg, nrhs, sl, tmp, st);
  q.part_out = part_p;
  q.first = 1;
  q.cur = q.nxt = cur;  // |r|^2 -> cur and rr0
  q.aux = rr0;
  cgne_launch<1>(DH, prec, ctile, q, cg, nrhs, st);
}

void cgne_fused_rstep(const CoarseStore& D, mgdwf_prec prec, int ctile, float2* x, float2* r, float2* p, void* work,
                      double* sl, int cur, int tmp, bool first, const CoarseGeometry& cg, int nrhs, hipStream_t st) {
  double *part_r, *part_p;
  CgneStep q = cgne_carve(work, cg, nrhs, x, r, p, &part_r, &part_p);
  cgne_partials(q, part_p, cg, nrhs, sl, tmp, st);
  q.part_out = part_r;
  q.first = first ? 1 : 0;
  q.cur = q.nxt = cur;
  cgne_launch<0>(D, prec, ctile, q, cg, nrhs, st);
}

void cgne_fused_pstep(const CoarseStore& DH, mgdwf_prec prec, int ctile, float2* r, float2* p, void* work, double* sl,
                      int cur, int nxt, int tmp, const CoarseGeometry& cg, int nrhs, hipStream_t st) {
  double *part_r, *part_p;
  CgneStep q = cgne_carve(work, cg, nrhs, nullptr, r, p, &part_r, &part_p);
  cgne_partials(q, part_r, cg, nrhs, sl, tmp, st);
  q.part_out = part_p;
  q.cur = cur;
  q.nxt = nxt;
  cgne_launch<1>(DH, prec, ctile, q, cg, nrhs, st);
}

size_t persistent_cgne_bytes(const CoarseGeometry& cg, int nrhs) {
  const size_t nsv = (size_t)nrhs * cg.Vc;
  return 2 * nsv * 2 * cg.n2 * sizeof(uint16_t) + 2 * nsv * sizeof(float) + 2 * nsv * sizeof(double) +
         sizeof(GridSync) + 7 * 256;
}

// Workgroups of k_cgne_persistent that one CU can hold at once, from the
// kernel's own register and LDS use: 576 threads are 9 wavefronts spread
// over the 4 SIMDs (3 on the fullest), each SIMD holds 512 VGPRs per lane
// (granule 8) and a CU 160 KB of LDS.
static int persistent_fit_per_cu(const void* fn) {
  hipFuncAttributes at{};
  MG_HIP(hipFuncGetAttributes(&at, fn));
  const int vgpr = std::max(8, (at.numRegs + 7) / 8 * 8);
  const int waves_per_simd = 512 / vgpr;
  const int by_vgpr = waves_per_simd / 3;  // the fullest SIMD carries 3 wavefronts of each workgroup
  const int by_lds = at.sharedSizeBytes > 0 ? (int)((160 * 1024) / at.sharedSizeBytes) : 64;
  return std::min(by_vgpr, by_lds);
}

bool coarse_cgne_persistent(const CoarseStore& D, const CoarseStore& DH, mgdwf_prec prec, const float2* b, float2* x,
                            float2* r, float2* p, void* work, long long* count, const CoarseGeometry& cg, int nrhs,
                            double tol, int maxiter, double wait_seconds, int device, hipStream_t st) {
  if (!(prec == MGDWF_F16 || prec == MGDWF_BF16) || cg.n2 % 16 || cg.n2 > 64 || nrhs < 1 || nrhs > 16 ||
      maxiter < 1)
    return false;
  const bool bf = prec == MGDWF_BF16;
  const void* fn = nullptr;
  with_n2(cg.n2, [&](auto N) {
    constexpr int N2 = decltype(N)::value;
    fn = bf ? reinterpret_cast<const void*>(&k_cgne_persistent<true, N2>)
            : reinterpret_cast<const void*>(&k_cgne_persistent<false, N2>);
  });
  int coop = 0, ncu = 0, per_cu = 0, clock_khz = 0;
  MG_HIP(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, device));
  MG_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device));
  MG_HIP(hipDeviceGetAttribute(&clock_khz, hipDeviceAttributeWallClockRate, device));
  MG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 576, 0));
  // At most one workgroup per CU, whatever the occupancy query says: the
  // kernel takes about 140 VGPRs, so a SIMD holds 3 wavefronts and a CU one
  // 9-wavefront workgroup; a grid of two workgroups per CU can never be
  // resident at once and its first grid barrier would wait for ever.
  if (!coop || per_cu < 1 || persistent_fit_per_cu(fn) < 1 || clock_khz <= 0) return false;
  const int G = std::min(cg.Vc, ncu);
  const size_t nsv = (size_t)nrhs * cg.Vc;
  char* w = static_cast<char*>(work);
  auto take = [&](size_t bytes) {
    char* q = w;
    w += (bytes + 255) / 256 * 256;
    return q;
  };
  PersistArgs q;
  q.Are = (bf ? D.reb : D.re16).as<uint16_t>();
  q.Aim = (bf ? D.imb : D.im16).as<uint16_t>();
  q.Asc = (bf ? D.scb : D.sc16).as<float>();
  q.Hre = (bf ? DH.reb : DH.re16).as<uint16_t>();
  q.Him = (bf ? DH.imb : DH.im16).as<uint16_t>();
  q.Hsc = (bf ? DH.scb : DH.sc16).as<float>();
  q.b = b;
  q.x = x;
  q.r = r;
  q.p = p;
  q.rp = reinterpret_cast<uint16_t*>(take(nsv * 2 * cg.n2 * sizeof(uint16_t)));
  q.pp = reinterpret_cast<uint16_t*>(take(nsv * 2 * cg.n2 * sizeof(uint16_t)));
  q.rs = reinterpret_cast<float*>(take(nsv * sizeof(float)));
  q.ps = reinterpret_cast<float*>(take(nsv * sizeof(float)));
  q.part_r = reinterpret_cast<double*>(take(nsv * sizeof(double)));
  q.part_p = reinterpret_cast<double*>(take(nsv * sizeof(double)));
  q.gs = reinterpret_cast<GridSync*>(take(sizeof(GridSync)));
  q.count = count;
  q.wait_ticks = (long long)(std::max(0.0, wait_seconds) * 1e3 * clock_khz);
  q.tol2 = tol * tol;
  q.maxiter = maxiter;
  q.nrhs = nrhs;
  q.a = coarse_args(cg);
  // the barrier words start from zero (a fill kernel, not a memset node, so
  // the sequence stays valid inside a captured graph)
  hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, st, reinterpret_cast<int*>(q.gs),
                     (int)(sizeof(GridSync) / sizeof(int)));
  MG_LAUNCH_CHECK();
  void* args[] = {&q};
  MG_HIP(hipLaunchCooperativeKernel(fn, dim3(G), dim3(576), args, 0, st));
  return true;
}

int persistent_cgne_error(const void* work, const CoarseGeometry& cg, int nrhs, hipStream_t st) {
  const size_t nsv = (size_t)nrhs * cg.Vc;
  auto up = [](size_t b) { return (b + 255) / 256 * 256; };
  const size_t off = 2 * up(nsv * 2 * cg.n2 * sizeof(uint16_t)) + 2 * up(nsv * sizeof(float)) +
                     2 * up(nsv * sizeof(double));
  GridSync h{};
  MG_HIP(hipMemcpyAsync(&h, static_cast<const char*>(work) + off, sizeof h, hipMemcpyDeviceToHost, st));
  MG_HIP(hipStreamSynchronize(st));
  return h.err;
}

}  // namespace mgdwf

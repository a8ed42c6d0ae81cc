// kernels_diag.hpp -- turbulence diagnostics off the step's hot path:
// Eulerian structure functions (SI, eq. structure-fun-sm) and the sums of
// the SI's moment-space analysis of a collision (m_diff against m_neq with
// the MRT matrix M).  Sums are float64 block partials reduced in a fixed
// order.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels_fwd.hpp"
#include "wide.hpp"

namespace lbm {

constexpr int DIAG_BLOCKS = 64;
constexpr int SF_PMAX = 8;
constexpr int SF_THREADS = 512;
constexpr int MRT_BLOCKS = 256;  // one per compute unit

// Values a lane still holds after l steps of wave_sums.
__host__ __device__ constexpr int held(int n, int l) {
  for (; l > 0; --l) n = (n + 1) / 2;
  return n;
}
// Sums of N values per lane over the wavefront, value k's to out[k]: at each
// step of a butterfly the lanes of a pair split the values they still hold, so
// that all of them take some N exchanges (the sums pair the lanes as a
// butterfly of every value would, which takes 6 N).  On small grids that is
// most of the time: the moment sums of 16^3 (N = 95) 28.5 -> 11.9 us, the
// structure functions of 64^2 with 60 separations and 8 orders (N = 48) 58 -> 16.
template <int N>
__device__ inline void wave_sums(double (&v)[N], double* out) {
  const int lane = threadIdx.x & 63;
  static_for<6>([&](auto lc) {
    constexpr int m = 32 >> decltype(lc)::value, n = held(N, decltype(lc)::value), h = (n + 1) / 2;
    const bool up = lane & m;
#pragma unroll
    for (int i = 0; i < h; ++i) {
      const double lo = v[i], hi = i + h < n ? v[i + h] : 0.0;
      v[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, m);
    }
  });
#pragma unroll
  for (int i = 0; i < held(N, 6); ++i) {
    int k = i;  // the value's index before each step, from the last to the first
    bool valid = true;
#pragma unroll
    for (int l = 5; l >= 0; --l) {
      k += lane & (32 >> l) ? (held(N, l) + 1) / 2 : 0;
      valid = valid && k < held(N, l);
    }
    if (valid) out[k] = v[i];
  }
}

// A flat node index walked with a constant stride: its coordinates advance by
// the stride's with carries instead of divisions.
struct NodeWalk {
  int x, y, z, b;
  int sx, sy, sz, sb;
  __device__ inline void start(const Grid& G, unsigned node, unsigned stride) {
    split(G, node, x, y, z, b);
    split(G, stride, sx, sy, sz, sb);
  }
  static __device__ inline void split(const Grid& G, unsigned n, int& x, int& y, int& z, int& b) {
    unsigned r = n / (unsigned)G.nx;
    x = (int)(n - r * (unsigned)G.nx);
    unsigned t = r / (unsigned)G.ny;
    y = (int)(r - t * (unsigned)G.ny);
    b = (int)(t / (unsigned)G.nz);
    z = (int)(t - (unsigned)b * (unsigned)G.nz);
  }
  __device__ inline void next(const Grid& G) {
    x += sx;
    int c = x >= G.nx;
    x -= c ? G.nx : 0;
    y += sy + c;
    c = y >= G.ny;
    y -= c ? G.ny : 0;
    z += sz + c;
    c = z >= G.nz;
    z -= c ? G.nz : 0;
    b += sb + c;
  }
};

// Separations l0 + 1 .. l0 + LB (l0 = LB blockIdx.y); for every node, field
// and axis a < D the longitudinal increment d = u_a(x + l e_a) - u_a(x)
// (periodic, in float64); partial[(l - 1) * DIAG_BLOCKS + block][k]: sum of
// d^(k+1) for k < PM, then sum of |d|^(k+1).
//
// Bound by the float64 additions and products: 5 + 9 per increment at PM = 6
// (even powers are their own absolute values, and |d|^p is |d^p| exactly), of
// 24 in the straightforward form, for 77 us of them at 128^3 and 32
// separations.  A thread takes LB separations of a node, so that the node's
// own values and coordinates are read and formed once.  128^3, 32 separations,
// PM = 6: 155 us (620 us with one separation per thread, all eight powers and
// 64-bit divisions).
template <int D, int PM, int LB>
__global__ __launch_bounds__(SF_THREADS) void structure_kernel(const float* __restrict__ u, Grid G,
                                                               int lmax,
                                                               double* __restrict__ partial) {
  constexpr int NO = (PM + 1) / 2;  // odd powers
  double s[LB][PM], sa[LB][NO];
#pragma unroll
  for (int j = 0; j < LB; ++j) {
#pragma unroll
    for (int p = 0; p < PM; ++p) s[j][p] = 0.0;
#pragma unroll
    for (int p = 0; p < NO; ++p) sa[j][p] = 0.0;
  }
  const int l0 = blockIdx.y * LB;
  const unsigned total = (unsigned)G.plane * (unsigned)G.batch, stride = gridDim.x * SF_THREADS;
  const unsigned first = blockIdx.x * SF_THREADS + threadIdx.x;
  const int nx4 = G.nx * 4, nxy4 = G.nx * G.ny * 4, plane4 = G.plane * 4;
  const rsrc_t src = make_rsrc(u, total * (unsigned)D * 4u);
  auto at = [&](int off, int a) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(src, off, a * plane4, 0));
  };
  NodeWalk w;
  if (first < total) w.start(G, first, stride);
  for (unsigned n = first; n < total; n += stride) {
    const int here = w.b * D * plane4 + w.z * nxy4 + w.y * nx4 + w.x * 4;
    float own[D], other[LB][D];
#pragma unroll
    for (int a = 0; a < D; ++a) own[a] = at(here, a);
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      // (lmax is at most the smallest size: one wrap is enough; separations
      // past lmax repeat the last one and are not written)
      const int l = min(l0 + j + 1, lmax);
      other[j][0] = at(here + (w.x + l >= G.nx ? (l - G.nx) * 4 : l * 4), 0);
      other[j][1] = at(here + (w.y + l >= G.ny ? (l - G.ny) * nx4 : l * nx4), 1);
      if constexpr (D == 3) other[j][2] = at(here + (w.z + l >= G.nz ? (l - G.nz) * nxy4 : l * nxy4), 2);
    }
#pragma unroll
    for (int j = 0; j < LB; ++j)
#pragma unroll
      for (int a = 0; a < D; ++a) {
        const double d = (double)other[j][a] - (double)own[a];
        double v = d;
#pragma unroll
        for (int p = 0; p < PM; ++p) {
          if (p > 0) v *= d;
          s[j][p] += v;
          if (p % 2 == 0) sa[j][p / 2] += __builtin_fabs(v);
        }
      }
    w.next(G);
  }
  // wavefront sums, then the wavefronts' in order
  constexpr int NV = LB * (PM + NO), NW = SF_THREADS / 64;
  __shared__ double red[NW][NV];
  double v[NV];
#pragma unroll
  for (int j = 0; j < LB; ++j) {
#pragma unroll
    for (int p = 0; p < PM; ++p) v[j * (PM + NO) + p] = s[j][p];
#pragma unroll
    for (int p = 0; p < NO; ++p) v[j * (PM + NO) + PM + p] = sa[j][p];
  }
  wave_sums(v, red[threadIdx.x >> 6]);
  __syncthreads();
  for (int k = threadIdx.x; k < LB * 2 * PM; k += SF_THREADS) {
    const int j = k / (2 * PM), q = k % (2 * PM), p = q % PM;
    if (l0 + j >= lmax) continue;
    // |d|^p of an even p is d^p
    const int from = j * (PM + NO) + (q < PM || p % 2 == 1 ? p : PM + p / 2);
    double t = red[0][from];
#pragma unroll
    for (int i = 1; i < NW; ++i) t += red[i][from];
    partial[((size_t)(l0 + j) * gridDim.x + blockIdx.x) * 2 * PM + q] = t;
  }
}

// S[p][l] and Sabs[p][l] (row-major [pmax][lmax]) from the partials of
// separation l + 1 = blockIdx.x + 1, divided by the sample count: sixteen slices of
// the blocks per entry, summed in slice order (4 us for 32 separations; 18.7
// us with one thread walking all 64 blocks of an entry).
static __global__ __launch_bounds__(256) void structure_reduce_kernel(const double* __restrict__ partial,
                                                               int nblk, int lmax, int pmax,
                                                               double inv_count,
                                                               double* __restrict__ S,
                                                               double* __restrict__ Sabs) {
  static_assert(2 * SF_PMAX <= 16, "sixteen entries per separation");
  __shared__ double red[16][16];
  const int l = blockIdx.x, k = threadIdx.x & 15, sl = threadIdx.x >> 4;
  double acc = 0.0;
  if (k < 2 * pmax)
    for (int b = sl; b < nblk; b += 16) acc += partial[((long long)l * nblk + b) * 2 * pmax + k];
  red[sl][k] = acc;
  __syncthreads();
  if (sl != 0 || k >= 2 * pmax) return;
  for (int i = 1; i < 16; ++i) acc += red[i][k];
  if (k < pmax)
    S[k * lmax + l] = acc * inv_count;
  else
    Sabs[(k - pmax) * lmax + l] = acc * inv_count;
}

// The MRT moment matrix M of the SI (D3Q19, velocity order of Table S1;
// rows rho, e, eps, jx, qx, jy, qy, jz, qz, pxx, pixx, pww, piww, pxy, pyz,
// pxz, mx, my, mz).
static constexpr signed char kMrtM[19][19] = {
    {1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1},
    {-30, -11, -11, -11, -11, -11, -11, 8, 8, 8, 8, 8, 8, 8, 8, 8, 8, 8, 8},
    {12, -4, -4, -4, -4, -4, -4, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1},
    {0, -1, 0, 0, 0, 0, 1, -1, -1, -1, -1, 0, 0, 0, 0, 1, 1, 1, 1},
    {0, 4, 0, 0, 0, 0, -4, -1, -1, -1, -1, 0, 0, 0, 0, 1, 1, 1, 1},
    {0, 0, -1, 0, 0, 1, 0, -1, 0, 0, 1, -1, -1, 1, 1, -1, 0, 0, 1},
    {0, 0, 4, 0, 0, -4, 0, -1, 0, 0, 1, -1, -1, 1, 1, -1, 0, 0, 1},
    {0, 0, 0, -1, 1, 0, 0, 0, -1, 1, 0, -1, 1, -1, 1, 0, -1, 1, 0},
    {0, 0, 0, 4, -4, 0, 0, 0, -1, 1, 0, -1, 1, -1, 1, 0, -1, 1, 0},
    {0, 2, -1, -1, -1, -1, 2, 1, 1, 1, 1, -2, -2, -2, -2, 1, 1, 1, 1},
    {0, -4, 2, 2, 2, 2, -4, 1, 1, 1, 1, -2, -2, -2, -2, 1, 1, 1, 1},
    {0, 0, 1, -1, -1, 1, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, -1, 1},
    {0, 0, -2, 2, 2, -2, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, -1, 1},
    {0, 0, 0, 0, 0, 0, 0, 1, 0, 0, -1, 0, 0, 0, 0, -1, 0, 0, 1},
    {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0},
    {0, 0, 0, 0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 0, 0, -1, 1, 0},
    {0, 0, 0, 0, 0, 0, 0, -1, 1, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1},
    {0, 0, 0, 0, 0, 0, 0, 1, 0, 0, -1, -1, -1, 1, 1, 1, 0, 0, -1},
    {0, 0, 0, 0, 0, 0, 0, 0, -1, 1, 0, 1, -1, 1, -1, 0, -1, 1, 0},
};

// With pre = A_n gathered at x, post = A_n1(x) (the post-collision populations
// of x in the pull-shifted layout), for every moment i
//   m_diff = M_i (post - pre - f_ext),  m_neq = M_i (f_eq - pre),
// partial[block][5 i + 0..4] = sums of m_neq, m_diff, m_neq^2, m_neq m_diff,
// m_diff^2 (float64).
//
// One pass over both states: a thread keeps the 95 sums (190 registers; one
// wavefront per SIMD, with the next node's 38 loads in flight while this
// one's moments are formed; M's zeros are skipped at compile time).  128^3:
// 111 us (bound: 64 us of reading at the rate of a copy, 60 us of VALU
// issue); 1,220 us as a workgroup row per moment, which read both states and
// formed f_eq and f_ext nineteen times.
static __global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void
mrt_sums_kernel(const float* __restrict__ An, const float* __restrict__ An1, Grid G, Force Fc,
                float rho0, double* __restrict__ partial) {
  using L = D3Q19;
  double s[19][5];
#pragma unroll
  for (int i = 0; i < 19; ++i)
#pragma unroll
    for (int k = 0; k < 5; ++k) s[i][k] = 0.0;
  const unsigned total = (unsigned)G.plane * (unsigned)G.batch, stride = gridDim.x * 256u;
  const unsigned bytes = total * 19u * 4u, plane4 = (unsigned)G.plane * 4u;
  const rsrc_t r0 = make_rsrc(An, bytes), r1 = make_rsrc(An1, bytes);
  float gn[19], pn[19];
  int xn = 0, yn = 0, zn = 0;
  auto load = [&](unsigned n) {
    NodeOffsets o;
    o.start(G, 19, n < total ? n : total - 1);
    xn = o.x;
    yn = o.y;
    zn = o.z;
#pragma unroll
    for (int q = 0; q < 19; ++q)
      gn[q] = __builtin_bit_cast(
          float, __builtin_amdgcn_raw_buffer_load_b32(r0, o.pull<L>(q), (int)(q * plane4), 0));
#pragma unroll
    for (int q = 0; q < 19; ++q)
      pn[q] = __builtin_bit_cast(
          float, __builtin_amdgcn_raw_buffer_load_b32(r1, o.at(), (int)(q * plane4), 0));
  };
  unsigned n = blockIdx.x * 256u + threadIdx.x;
  load(n);
  for (; n < total; n += stride) {
    float g[19], post[19], geq[19], fe[19], F[3];
#pragma unroll
    for (int q = 0; q < 19; ++q) {
      g[q] = gn[q];
      post[q] = pn[q];
    }
    const int x = xn, y = yn, z = zn;
    load(n + stride);
    float drho, j[3];
    moments<L>(g, drho, j);
    const float rho = rho0 + drho, inv = 1.f / rho;
    const float uv[3] = {j[0] * inv, j[1] * inv, j[2] * inv};
    Unroll<L>::feq(drho, rho, uv, uv[0] * uv[0] + uv[1] * uv[1] + uv[2] * uv[2], geq);
    body_force(Fc, G, x, y, z, F);
    const float du[3] = {F[0] * inv, F[1] * inv, F[2] * inv};
    const float dd = du[0] * (2.f * uv[0] + du[0]) + du[1] * (2.f * uv[1] + du[1]) +
                     du[2] * (2.f * uv[2] + du[2]);
    Unroll<L>::fext(rho, uv, du, dd, fe);
    double df[19], ne[19];
#pragma unroll
    for (int q = 0; q < 19; ++q) {
      df[q] = (double)post[q] - (double)g[q] - (double)fe[q];
      ne[q] = (double)geq[q] - (double)g[q];
    }
    static_for<19>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      double md = 0.0, mn = 0.0;
      static_for<19>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        if constexpr (kMrtM[i][q] != 0) {
          constexpr double m = kMrtM[i][q];
          md += m * df[q];
          mn += m * ne[q];
        }
      });
      s[i][0] += mn;
      s[i][1] += md;
      s[i][2] += mn * mn;
      s[i][3] += mn * md;
      s[i][4] += md * md;
    });
  }
  __shared__ double red[4][95];
  double v[95];
#pragma unroll
  for (int i = 0; i < 19; ++i)
#pragma unroll
    for (int k = 0; k < 5; ++k) v[5 * i + k] = s[i][k];
  wave_sums(v, red[threadIdx.x >> 6]);
  __syncthreads();
  if (threadIdx.x < 95)
    partial[blockIdx.x * 95 + threadIdx.x] = ((red[0][threadIdx.x] + red[1][threadIdx.x]) +
                                              red[2][threadIdx.x]) + red[3][threadIdx.x];
}

// stats[t] = sum over the blocks of partial[block][t]: eight slices of the
// blocks per entry, summed in slice order.
static __global__ __launch_bounds__(768) void mrt_reduce_kernel(const double* __restrict__ partial,
                                                                int nblk,
                                                                double* __restrict__ stats) {
  __shared__ double red[8][95];
  const int sl = threadIdx.x / 96, t = threadIdx.x % 96;
  if (t < 95) {
    double acc = 0.0;
    for (int b = sl; b < nblk; b += 8) acc += partial[b * 95 + t];
    red[sl][t] = acc;
  }
  __syncthreads();
  if (threadIdx.x < 95) {
    double acc = red[0][threadIdx.x];
    for (int k = 1; k < 8; ++k) acc += red[k][threadIdx.x];
    stats[threadIdx.x] = acc;
  }
}

}  // namespace lbm

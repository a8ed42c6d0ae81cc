// wide_step16.hpp -- the stream-collide step with the SI's network (see
// wide.hpp) in bf16 / fp16.
//
// A workgroup of four wavefronts takes 64 nodes at a time (any 64 consecutive
// flat node indices, so that no lane idles at the end of a row), two
// workgroups per compute unit.  A wavefront computes five of a layer's
// nineteen 16-row tiles (two of layer 3's seven) for all 64 nodes; the
// activations pass from layer to layer through LDS (two buffers of 38 KB),
// the weights are streamed from the L2 straight into registers, two steps
// ahead of their use.  One barrier per layer: four per 64 nodes.
//
// Why this split.  Its unit of work is 64 nodes per workgroup, two workgroups
// per compute unit, against 512 nodes for the kernel of wide.hpp, which leaves
// three quarters of the chip idle on a 32^3 grid: 29.4 -> 12.5 us there (D3Q19
// bf16), 48^3 62.7 -> 35.0 us.  A weight fragment feeds four matrix
// instructions (64 nodes) and an activation fragment five; the kernel of
// wide.hpp feeds sixteen and two, with the weights shared through LDS, and is
// the faster one where its units fill the chip (256^3 3.93 against 5.15 ms; 128
// nodes per workgroup of eight wavefronts here measured 5.06): wide_rule.hpp.
// What bounds a block is the sum of its phases: per 64 nodes 4,900 clocks of
// matrix instructions per wavefront, about 700 VALU instructions and 430 KB
// through LDS, between four barriers that two workgroups only partly overlap.
//
// The node work of block k (gather, network input, and at the end BGK part,
// projection, force and store) is done by wavefront k % 4, one node per
// lane; the gather of block k + 1 is in flight during block k.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "wide.hpp"

namespace lbm {

template <int Q_>
struct WideStep {
  static constexpr int Q = Q_;
  using WL = WideLayout<Q_, P_BF16>;  // widths, parameter offsets and the bias region
  // layers 1-4: tiles per wavefront; contraction units (pairs of 16-feature
  // chunks, the last one a single chunk where `odd`)
  static constexpr int NL = 4;
  static constexpr int TPW[NL] = {5, 5, 2, WL::T4};
  static constexpr int KU[NL] = {(WL::K1 + 1) / 2, 10, 10, 4};
  static constexpr bool odd(int l) {
    return l == 0 ? WL::K1 % 2 == 1 : true;
  }
  // the steps of one block: every layer's units, then empty steps up to a
  // multiple of the ring's three slots
  static constexpr int NREAL = KU[0] + KU[1] + KU[2] + KU[3];
  static constexpr int NSTEP = (NREAL + 2) / 3 * 3;
  static constexpr int layer_of(int s) {
    int l = 0;
    while (l < NL && s >= KU[l]) s -= KU[l++];
    return l;
  }
  static constexpr int first_step(int l) {
    int s = 0;
    for (int i = 0; i < l; ++i) s += KU[i];
    return s;
  }
  static constexpr int frags(int s) { return layer_of(s) < NL ? TPW[layer_of(s)] : 0; }
  static constexpr int frag_of(int s) {
    int f = 0;
    for (int i = 0; i < s; ++i) f += frags(i);
    return f;
  }
  static constexpr int NFW = frag_of(NSTEP);  // fragments of a wavefront's stream
  static constexpr int NWAVE = 4;
  static constexpr int nw = NWAVE * NFW * 512;  // 16-bit entries
  static constexpr int weight_bytes = 2 * nw;
  static constexpr int packed_bytes = weight_bytes + 4 * WL::nbias;
  // A wavefront's tiles of layers 1 and 2: two pairs, then half of the pair
  // it shares with its neighbour (tile 19 does not exist: zero weights).
  __host__ __device__ static constexpr int pair0(int w) { return (5 * w + 1) / 2; }
  __host__ __device__ static constexpr int half_pair(int w) { return 2 + 5 * (w / 2); }
  static constexpr int tile(int l, int w, int j) {
    if (l >= 2) return l == 2 ? 2 * w + j : j;
    return j < 4 ? 2 * (pair0(w) + j / 2) + j % 2 : 2 * half_pair(w) + (w & 1);
  }
};

// theta index of every packed entry (-1: zero), then the biases as in
// WideLayout.  Fragment of tile t and unit c, lane (g, i): row 16 t + i,
// columns 32 c + 4 g .. + 3 and 32 c + 16 + 4 g .. + 3.
template <int Q>
std::vector<int> wide_step_index() {
  using S = WideStep<Q>;
  using WL = typename S::WL;
  std::vector<int> idx((size_t)S::nw + WL::nbias, -1);
  auto value = [](int l, int o, int k) -> int {
    switch (l) {
      case 0: return o >= WL::N1 ? -1 : (k < Q ? WL::oW1 + o * Q + k : (k == Q ? WL::ob1 + o : -1));
      case 1: return o < WL::N2 && k < WL::N1 ? WL::oW2 + o * WL::N1 + k : -1;
      case 2: return o < WL::N3 && k < WL::N2 ? WL::oW3 + o * WL::N2 + k : -1;
      default: return o < Q && k < WL::N3 ? WL::oW4 + o * WL::N3 + k : -1;
    }
  };
  for (int w = 0; w < S::NWAVE; ++w) {
    int f = 0;
    for (int l = 0; l < S::NL; ++l)
      for (int c = 0; c < S::KU[l]; ++c)
        for (int j = 0; j < S::TPW[l]; ++j, ++f)
          for (int lane = 0; lane < 64; ++lane)
            for (int e = 0; e < 8; ++e) {
              const int o = 16 * S::tile(l, w, j) + (lane & 15);
              const int k = 32 * c + 16 * (e / 4) + 4 * (lane >> 4) + e % 4;
              idx[((size_t)(w * S::NFW + f) * 64 + lane) * 8 + e] = value(l, o, k);
            }
  }
  int* b = idx.data() + S::nw;
  for (int i = 0; i < 16 * WL::T2; ++i) b[WL::fb2 + i] = i < WL::N2 ? WL::ob2 + i : -1;
  for (int i = 0; i < 16 * WL::T3; ++i) b[WL::fb3 + i] = i < WL::N3 ? WL::ob3 + i : -1;
  for (int i = 0; i < 16 * WL::T4; ++i) b[WL::fb4 + i] = i < Q ? WL::ob4 + i : -1;
  return idx;
}

template <class L, int P>
__global__ __launch_bounds__(256, 2) void wide_step16_kernel(
    const float* __restrict__ Ain, float* __restrict__ Aout,
    const unsigned char* __restrict__ packed, Grid G, Force Fc, float rho0, float omega,
    float knn, int nblocks, int nwg) {
  constexpr int Q = L::Q;
  using S = WideStep<Q>;
  using WL = typename S::WL;
  // unit c of an activation buffer: 4 node tiles of 1 KB (16 bytes per lane);
  // the tenth (layer 3's output: fourth) unit is a single chunk, 8 bytes per
  // lane, 512 bytes per node tile
  constexpr int BUF = 9 * 4096 + 2048;
  __shared__ __attribute__((aligned(16))) unsigned char bufP[BUF];  // h1, then h3
  __shared__ __attribute__((aligned(16))) unsigned char bufQ[BUF];  // h2, then y
  __shared__ __attribute__((aligned(16))) unsigned char bufX[4096];  // [g, 1, 0 ...]
  constexpr int SY = (Q + 3) / 4 * 4;  // row stride of y (floats)
  static_assert(64 * SY * 4 <= BUF, "y rows");

  // (the builtins, not threadIdx and blockIdx: under this unit's options those
  // are calls whose results the compiler takes for per-lane values)
  const int tid = (int)__builtin_amdgcn_workitem_id_x();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, lg = lane >> 4, li = lane & 15;
  const rsrc_t wsrc = make_rsrc(reinterpret_cast<const float*>(packed), (unsigned)S::packed_bytes);
  const int l16 = lane * 16, l8 = lane * 8;

  const unsigned total = (unsigned)G.plane * (unsigned)G.batch;
  const unsigned bytes = total * (unsigned)Q * 4u, plane4 = (unsigned)G.plane * 4u;
  const rsrc_t src = make_rsrc(Ain, bytes), dst = make_rsrc(Aout, bytes);

  // Blocks of this workgroup: each XCD (workgroups go round the eight) walks
  // one contiguous part of the domain, its workgroups interleaved.
  const int bid = (int)__builtin_amdgcn_workgroup_id_x();
  int first, last, stride;
  if (nwg % 8 == 0) {
    const int per = (nblocks + 7) / 8, x = bid % 8;
    first = x * per + bid / 8;
    last = min((x + 1) * per, nblocks);
    stride = nwg / 8;
  } else {
    first = bid;
    last = nblocks;
    stride = nwg;
  }
  if (first >= last) return;

  int wbase = wave * S::NFW * 1024;
  u4 ring[3][5];
  auto issue = [&](auto sc) {
    constexpr int s = decltype(sc)::value % S::NSTEP;
    constexpr int n = S::frags(s), f = S::frag_of(s);
#pragma unroll
    for (int j = 0; j < n; ++j)
      ring[s % 3][j] = __builtin_bit_cast(
          u4, __builtin_amdgcn_raw_buffer_load_b128(wsrc, l16, wbase + (f + j) * 1024, 0));
  };
  // four biases from entry i of the bias region on
  auto bias4 = [&](int i) {
    return __builtin_bit_cast(
        f4, __builtin_amdgcn_raw_buffer_load_b128(wsrc, i * 4, S::weight_bytes, 0));
  };

  float g[Q];
  auto gather_block = [&](int blk) {
    const unsigned node = (unsigned)blk * 64u + lane;
    NodeOffsets o;
    o.start(G, Q, node < total ? node : total - 1);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      g[q] = __builtin_bit_cast(
          float, __builtin_amdgcn_raw_buffer_load_b32(src, o.pull<L>(q), (int)(q * plane4), 0));
  };
  // the network input of this lane's node, as the operand of layer 1
  auto put_input = [&] {
    float v[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) v[k] = k < Q ? g[k] : (k == Q ? 1.f : 0.f);
    unsigned char* row = bufX + (lane >> 4) * 1024 + (lane & 15) * 16;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const u4 o = {pack2<P>(v[4 * q], v[4 * q + 1]), pack2<P>(v[4 * q + 2], v[4 * q + 3]),
                    pack2<P>(v[16 + 4 * q], v[17 + 4 * q]),
                    pack2<P>(v[18 + 4 * q], v[19 + 4 * q])};
      *reinterpret_cast<u4*>(row + q * 256) = o;
    }
  };
  auto read = [&](const unsigned char* buf, int c, int n, bool single) -> u4 {
    if (!single) return *reinterpret_cast<const u4*>(buf + c * 4096 + n * 1024 + l16);
    const u2 v = *reinterpret_cast<const u2*>(buf + c * 4096 + n * 512 + l8);
    return u4{v[0], v[1], 0u, 0u};
  };
  auto mma = [&](u4 a, u4 x, f4 acc, bool single) -> f4 {
    const u2 a0 = {a[0], a[1]}, a1 = {a[2], a[3]}, x0 = {x[0], x[1]}, x1 = {x[2], x[3]};
    return single ? mma_chunk<P>(acc, a0, x0) : mma_pair<P>(acc, a0, a1, x0, x1);
  };
  // One layer for the four node tiles; ep(acc, n) takes node tile n's results.
  auto layer = [&](auto lc, const unsigned char* buf, const f4 (&bv)[5], auto&& ep) {
    constexpr int l = decltype(lc)::value, T = S::TPW[l], KU = S::KU[l], s0 = S::first_step(l);
    f4 acc[T][4];
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int n = 0; n < 4; ++n) acc[j][n] = bv[j];
    u4 xb[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) xb[n] = read(buf, 0, n, l > 0 && KU == 1);
    static_for<KU>([&](auto cc) {
      constexpr int c = decltype(cc)::value, s = s0 + c;
      constexpr bool single = S::odd(l) && c == KU - 1;
      issue(std::integral_constant<int, s + 2>{});
      static_for<4>([&](auto nc) {
        constexpr int n = decltype(nc)::value;
#pragma unroll
        for (int j = 0; j < T; ++j) {
          // (the last unit accumulates on products of the other shape: the
          // barriers keep the node tiles in order, so that at least the 3 T
          // >= 6 products of the three other tiles stand between)
          static_assert(T >= 2, "distance between products of the two shapes");
          acc[j][n] = mma(ring[s % 3][j], xb[n], acc[j][n], single);
        }
        // the next unit's operand, into the registers just consumed
        if constexpr (c + 1 < KU) xb[n] = read(buf, c + 1, n, S::odd(l) && c + 1 == KU - 1);
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    static_for<4>([&](auto nc) {
      ep(acc, decltype(nc)::value);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  const int p0 = S::pair0(wave), ph = S::half_pair(wave), hh = wave & 1;
  const bool tail = wave == 3;  // its second pair is the last, single chunk
  auto put_pair = [&](unsigned char* buf, int p, int n, u2 lo, u2 hi) {
    *reinterpret_cast<u4*>(buf + p * 4096 + n * 1024 + l16) = u4{lo[0], lo[1], hi[0], hi[1]};
  };
  auto put_tail = [&](unsigned char* buf, int p, int n, u2 lo, u2 hi) {
    if (tail)
      *reinterpret_cast<u2*>(buf + p * 4096 + n * 512 + l8) = lo;
    else
      put_pair(buf, p, n, lo, hi);
  };
  auto put5 = [&](unsigned char* buf, const f4 (&acc)[5][4], int n) {
    u2 f[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) f[j] = to_frag<P>(leaky4(acc[j][n]));
    put_pair(buf, p0, n, f[0], f[1]);
    put_tail(buf, p0 + 1, n, f[2], f[3]);
    *reinterpret_cast<u2*>(buf + ph * 4096 + n * 1024 + l16 + 8 * hh) = f[4];
  };
  const f4 zero = {0.f, 0.f, 0.f, 0.f};

  issue(std::integral_constant<int, 0>{});
  issue(std::integral_constant<int, 1>{});
  if (wave == 0) {
    gather_block(first);
    put_input();
  }
  __syncthreads();
  int k = 0;
  for (int blk = first; blk < last; blk += stride, ++k) {
    const bool more = blk + stride < last;
    // (opaque per block: the stream is read again, not kept)
    asm volatile("" : "+s"(wbase));
    f4 bv[5] = {zero, zero, zero, zero, zero};
    layer(std::integral_constant<int, 0>{}, bufX, bv,
          [&](const f4 (&acc)[5][4], int n) { put5(bufP, acc, n); });
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      const int t = j < 4 ? 2 * (p0 + j / 2) + j % 2 : 2 * ph + hh;
      // (tile 19 reads past layer 2's biases; its weights feed no product)
      bv[j] = bias4(WL::fb2 + 16 * t + 4 * lg);
    }
    __syncthreads();
    // the next block's populations: in flight through layers 2 and 3
    if (more && wave == ((k + 1) & 3)) gather_block(blk + stride);
    layer(std::integral_constant<int, 1>{}, bufP, bv,
          [&](const f4 (&acc)[5][4], int n) { put5(bufQ, acc, n); });
#pragma unroll
    for (int j = 0; j < 2; ++j) bv[j] = bias4(WL::fb3 + 16 * (2 * wave + j) + 4 * lg);
    __syncthreads();
    layer(std::integral_constant<int, 2>{}, bufQ, bv, [&](const f4 (&acc)[2][4], int n) {
      put_tail(bufP, wave, n, to_frag<P>(leaky4(acc[0][n])), to_frag<P>(leaky4(acc[1][n])));
    });
    if (more && wave == ((k + 1) & 3)) put_input();
    __syncthreads();
    // layer 4: wavefront w takes node tile w
    {
      constexpr int s0 = S::first_step(3), T4 = WL::T4;
      f4 acc[T4];
#pragma unroll
      for (int j = 0; j < T4; ++j) acc[j] = bias4(WL::fb4 + 16 * j + 4 * lg);
      static_for<4>([&](auto cc) {
        constexpr int c = decltype(cc)::value, s = s0 + c;
        issue(std::integral_constant<int, s + 2>{});
        const u4 x = read(bufP, c, wave, c == 3);
        if constexpr (c == 3) {
          mma_shape_wait(acc[0]);
          if constexpr (T4 == 2) mma_shape_wait(acc[1]);
        }
#pragma unroll
        for (int j = 0; j < T4; ++j) acc[j] = mma(ring[s % 3][j], x, acc[j], c == 3);
      });
      static_for<S::NSTEP - S::NREAL>([&](auto ec) {
        issue(std::integral_constant<int, S::NREAL + decltype(ec)::value + 2>{});
      });
      float* Y = reinterpret_cast<float*>(bufQ);
#pragma unroll
      for (int j = 0; j < T4; ++j)
        if (16 * j + 4 * lg < SY)
          *reinterpret_cast<f4*>(Y + (16 * wave + li) * SY + 16 * j + 4 * lg) = acc[j];
    }
    __syncthreads();
    // block end, one node per lane: BGK, network term, projection, force, store
    if (wave == (k & 3)) {
      const unsigned node = (unsigned)blk * 64u + lane;
      NodeOffsets o;
      o.start(G, Q, node < total ? node : total - 1);
      float upd[Q], rho, u[3];
      bgk_update<L>(g, rho0, omega, upd, rho, u);
      const float* Y = reinterpret_cast<const float*>(bufQ) + lane * SY;
#pragma unroll
      for (int q = 0; q < Q; ++q) upd[q] = __builtin_fmaf(knn, Y[q], upd[q]);
      float F3[3] = {0.f, 0.f, 0.f};
      if (Fc.kind != 0) body_force(Fc, G, o.x, o.y, o.z, F3);
      float post[Q];
      finish_wide<L>(g, upd, rho, u, F3, Fc.kind != 0, post);
      if (node < total) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, post[q]), dst, o.at(),
                                                (int)(q * plane4), 0);
      }
    }
  }
}

}  // namespace lbm

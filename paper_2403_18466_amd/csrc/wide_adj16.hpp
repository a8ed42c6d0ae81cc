// wide_adj16.hpp -- adjoint of one step with the SI's network in bf16 / fp16
// (the products and the data flow are those listed in wide_bwd.hpp; the
// float32 network keeps the chain of products there).
//
// Two kernels and a reduction per step (D3Q19 bf16, one step: 32^3 262 -> 62 us,
// 60 x 64 x 52 1,330 -> 282 us against a chain of fourteen products on 64 x 64
// tiles, which wrote every activation twice and read it three times):
//
//   wide_adj_data_kernel     64 nodes per workgroup, from the gather to the
//       scatter of lam^n: the hidden layers are recomputed and differentiated
//       with the activations of the 64 nodes in LDS (two buffers of 38 KB,
//       two workgroups per compute unit) and the weights streamed from the
//       L2 into registers in the order of use.  608 matrix instructions and
//       about 750 VALU instructions of epilogue per 16 nodes (104 us at 60 x 64
//       x 52 without the records' stores); 31 us at 32^3, which is one round
//       of workgroups, about 165 us at 60 x 64 x 52 (0.61 PFLOP/s, 4 TB/s of
//       records; its parts took 167 us at 32^3 as separate products).
//   wide_adj_weight_kernel   the weight gradients, contractions over the
//       nodes, from the activations the first kernel leaves in memory once
//       (3.1 KB per node).  Bound by that read: 23 us at 32^3, 103 us at 60 x
//       64 x 52 (6.2 TB/s; a streaming read reaches 6.3, and 7.0 with the
//       non-temporal policy).
//   wide_adj_reduce_kernel   sums the node ranges' partial gradients: 7.2 us
//       for 32 ranges, 11.2 us for 64 (22.8 us at 32^3 and 57.4 us at 60 x 64
//       x 52 before, with 64 and 128 of them).
//
// The record stores.  A wavefront stores, at each chunk of a product, the
// operand of one node tile that the product reads anyway, a whole block at a
// time, so that the stores run along with the matrix instructions.  (Stored
// from the epilogues, all at once, the next weight fragments wait for them:
// the counter of outstanding accesses is one.)  With that and the
// non-temporal policy, which keeps a record larger than the last-level cache
// from filling the L2 with lines to write back: 194 -> 165 us at 60 x 64 x 52.
//
// Work split of the first kernel.  A wavefront computes five of a layer's
// twenty 16-row tiles for all 64 nodes, so a weight fragment (read from the
// L2 once per workgroup) feeds four matrix instructions and an activation
// fragment (16 bytes per lane from LDS) five: at full matrix rate that is 64
// B per clock of L2 reads and 51 of LDS reads per compute unit.  With whole
// layers per wavefront (weights through LDS, activations in registers) the
// LDS would have to deliver 128 B per clock.
//
// Fragment order.  The contraction of every product runs over chunks of 32
// features, lane group g of 16 lanes holding features 8 g .. 8 g + 7 of the
// chunk (an operand of one 16 x 16 x 32 matrix instruction).  The rows of
// the two 16-row tiles of a pair are dealt so that lane group g's results
// are features 8 g .. 8 g + 3 (first tile) and 8 g + 4 .. 8 g + 7 (second)
// of the pair's 32: packed, they are the next product's operand.
//
// Node-tile record (kept for the second kernel): 50 blocks of 1 KB, one per
// 16 nodes x 32 features, in the order X0, dY, H1 (10), H2 (10), H3 (4),
// dZ3 (4), dZ2 (10), dZ1 (10).  Within a block, the 16 bytes of lane (g, i)
// sit at slot 16 g + (i ^ 8 (g & 1)): the second kernel reads the block
// transposed (node index as the contraction) with ds_read_b64_tr_b16, and the
// exchange puts the sixteen 8-byte rows of each 16-lane group on different
// bank pairs.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "kernels_bwd.hpp"
#include "wide.hpp"
#include "wide_bwd.hpp"
#include "wide_rule.hpp"

namespace lbm {

template <int Q_>
struct WideAdj {
  static constexpr int Q = Q_;
  using W = WideBwd<Q>;
  // layers of the first kernel in order: H1, H2, H3, dZ3, dZ2, dZ1, dX0;
  // tiles per wavefront and contraction chunks of each
  static constexpr int NL = 7;
  static constexpr int TPW[NL] = {5, 5, 2, 2, 5, 5, 2};
  static constexpr int KC[NL] = {1, 10, 10, 1, 4, 10, 10};
  static constexpr int NSTEP = 46;  // chunks of all layers
  static constexpr int layer_of(int s) {
    int l = 0;
    while (s >= KC[l]) s -= KC[l++];
    return l;
  }
  static constexpr int first_step(int l) {
    int s = 0;
    for (int i = 0; i < l; ++i) s += KC[i];
    return s;
  }
  // first fragment of step s in a wavefront's weight stream
  static constexpr int frag_of(int s) {
    int f = 0;
    for (int i = 0; i < s; ++i) f += TPW[layer_of(i)];
    return f;
  }
  static constexpr int NFW = 167;  // fragments of one wavefront's stream
  static constexpr int NWAVE = 4;
  static constexpr int nw = NWAVE * NFW * 512;  // packed weights (16-bit entries)
  static constexpr int packed_bytes = 2 * nw + 4 * W::nb;
  // A wavefront's tiles of a 20-tile layer: four that form two pairs, then
  // one half of the pair it shares with its neighbour.
  __host__ __device__ static constexpr int pair0(int w) { return (5 * w + 1) / 2; }
  __host__ __device__ static constexpr int half_pair(int w) { return 2 + 5 * (w / 2); }
  static constexpr int tile5(int w, int j) {
    return j < 4 ? 2 * (pair0(w) + j / 2) + j % 2 : 2 * half_pair(w) + (w & 1);
  }
  // record blocks
  static constexpr int RX0 = 0, RDY = 1, RH1 = 2, RH2 = 12, RH3 = 22, RZ3 = 26, RZ2 = 30, RZ1 = 40,
                       NREC = 50;
  static_assert(NREC * 1024 == 16 * kWideRecordBytes, "bytes per node");
  // gradient tiles of a partial slab (256 floats each): dW2 (19 x 19), dW3 (7
  // x 19), dW1 transposed (X0 x dZ1: 2 x 19), dW4 (2 x 7)
  static constexpr int G2 = 0, G3 = G2 + 361, G1 = G3 + 133, G4 = G1 + 38, NG = G4 + 14;
  static_assert(NG * 1024 == kWideSlabBytes, "bytes of a slab");
};

// theta index of entry e of the packed weights (see WideAdj; -1 is zero),
// then the bias vectors as in WideBwd (-2 is the constant 1).
template <int Q>
std::vector<int> wide_adj_index() {
  using A = WideAdj<Q>;
  using W = WideBwd<Q>;
  std::vector<int> idx((size_t)A::nw + W::nb, -1);
  // entry (o, k) of a layer's matrix: theta[at + o so + k sk] for o < no, k < nk
  struct Matrix {
    int no, nk, at, so, sk;
  };
  const Matrix mat[A::NL] = {{W::N1, Q, W::pW1, Q, 1},         {W::N2, W::N1, W::pW2, W::N1, 1},
                             {W::N3, W::N2, W::pW3, W::N2, 1}, {W::N3, Q, W::pW4, 1, W::N3},
                             {W::N2, W::N3, W::pW3, 1, W::N2}, {W::N1, W::N2, W::pW2, 1, W::N1},
                             {Q, W::N1, W::pW1, 1, Q}};
  int* out = idx.data();
  for (int w = 0; w < A::NWAVE; ++w)
    for (int l = 0; l < A::NL; ++l) {
      const Matrix m = mat[l];
      const int tiles = A::TPW[l];
      for (int c = 0; c < A::KC[l]; ++c)
        for (int j = 0; j < tiles; ++j) {
          const int t = tiles == 5 ? A::tile5(w, j) : (l == A::NL - 1 ? j : 2 * w + j);
          for (int lane = 0; lane < 64; ++lane, out += 8) {
            const int i = lane & 15, k = 32 * c + 8 * (lane >> 4);
            const int o = l == A::NL - 1 ? 16 * t + i
                                         : 32 * (t / 2) + 8 * (i / 4) + 4 * (t % 2) + i % 4;
            const int from = m.at + o * m.so + k * m.sk;
            if (o < m.no && k + 8 <= m.nk) {
              for (int e = 0; e < 8; ++e) out[e] = from + e * m.sk;
            } else if (o < m.no) {
              for (int e = 0; k + e < m.nk; ++e) out[e] = from + e * m.sk;
              if (l == 0 && k <= Q && Q < k + 8) out[Q - k] = W::pb1 + o;
            }
          }
        }
    }
  int* v = idx.data() + A::nw;
  for (int j = 0; j < W::D1; ++j) v[W::fE1 + j] = j == W::ONE1 ? -2 : -1;
  for (int j = 0; j < W::D2; ++j) v[W::fB2 + j] = j < W::N2 ? W::pb2 + j : (j == W::ONE2 ? -2 : -1);
  for (int j = 0; j < W::D3; ++j) v[W::fB3 + j] = j < W::N3 ? W::pb3 + j : (j == W::ONE3 ? -2 : -1);
  return idx;
}

template <int P>
__device__ inline f4 mma32(u4 a, u4 b, f4 c) {
  if constexpr (P == P_BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a),
                                                   __builtin_bit_cast(b8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a),
                                                  __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

template <class L, int P, bool NT>
__global__ __launch_bounds__(256, 2) void wide_adj_data_kernel(
    const float* __restrict__ A, const float* __restrict__ lam1, float* __restrict__ lam0,
    const unsigned char* __restrict__ packed, unsigned char* __restrict__ rec, Grid G, Force Fc,
    float rho0, float omega, float knn) {
  constexpr int Q = L::Q;
  using AJ = WideAdj<Q>;
  using W = WideBwd<Q>;
  // chunk c of an activation buffer: 4 node tiles of 1 KB; a tenth (H3-sized:
  // fourth) chunk holds 16 features, 512 bytes per node tile
  constexpr int BUF = 9 * 4096 + 2048;
  __shared__ __attribute__((aligned(16))) unsigned char bufP[BUF];
  __shared__ __attribute__((aligned(16))) unsigned char bufQ[BUF];
  __shared__ __attribute__((aligned(16))) unsigned char bufE[4096];
  constexpr int SDX = 36;  // row stride of the dX0 rows (floats) in bufQ
  static_assert(64 * SDX * 4 <= BUF, "dX0 rows");

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lg = lane >> 4, li = lane & 15;
  const rsrc_t wsrc = make_rsrc(reinterpret_cast<const float*>(packed), (unsigned)AJ::packed_bytes);
  const int wbase = wave * AJ::NFW * 1024, l16 = lane * 16;
  const rsrc_t myrec = make_rsrc(
      reinterpret_cast<const float*>(rec + (size_t)blockIdx.x * 4 * (AJ::NREC * 1024)),
      4 * AJ::NREC * 1024);
  const int slot16 = 16 * (16 * lg + (li ^ (8 * (lg & 1))));

  // the weight stream: step s + 2's fragments are issued at step s
  u4 ring[3][5];
  auto issue = [&](auto sc) {
    constexpr int s = decltype(sc)::value;
    if constexpr (s < AJ::NSTEP) {
      constexpr int n = AJ::TPW[AJ::layer_of(s)], f = AJ::frag_of(s);
#pragma unroll
      for (int j = 0; j < n; ++j)
        ring[s % 3][j] = __builtin_bit_cast(
            u4, __builtin_amdgcn_raw_buffer_load_b128(wsrc, l16, wbase + (f + j) * 1024, 0));
    }
  };
  issue(std::integral_constant<int, 0>{});
  issue(std::integral_constant<int, 1>{});

  // wavefront 0, one node per lane: the gather, the network input, and
  // (while the others start the hidden layers) the non-network adjoint
  const unsigned total = (unsigned)G.plane * (unsigned)G.batch;
  const unsigned node = blockIdx.x * 64u + lane;
  const unsigned bytes = total * (unsigned)Q * 4u, plane4 = (unsigned)G.plane * 4u;
  const rsrc_t rA = make_rsrc(A, bytes), rL1 = make_rsrc(lam1, bytes), rL0 = make_rsrc(lam0, bytes);
  float lam[Q];
  // (cast, not pack2: where v is a product, fp16 rounds it once)
  auto put_row = [&](unsigned char* buf, const float (&v)[32]) {
    using T = typename OpT<P>::T;
    typedef T t2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      u4 o;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        o[k] = __builtin_bit_cast(unsigned, t2{(T)v[8 * g + 2 * k], (T)v[8 * g + 2 * k + 1]});
      *reinterpret_cast<u4*>(buf + (lane >> 4) * 1024 + (16 * g + (lane & 15)) * 16) = o;
    }
  };
  if (wave == 0) {
    float g[Q], mu[Q], v[32];
    const bool in = node < total;
    NodeOffsets o;
    if (in) {
      o.start(G, Q, node);
#pragma unroll
      for (int q = 0; q < Q; ++q)
        g[q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                             rA, o.pull<L>(q), (int)(q * plane4), 0));
#pragma unroll
      for (int q = 0; q < Q; ++q)
        mu[q] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(rL1, o.at(), (int)(q * plane4), 0));
    }
#pragma unroll
    for (int k = 0; k < 32; ++k) v[k] = in ? (k < Q ? g[k] : (k == Q ? 1.f : 0.f)) : 0.f;
    put_row(bufQ, v);
    __syncthreads();
    float nu[Q], F[3];
    if (in) {
      body_force(Fc, G, o.x, o.y, o.z, F);
      collide_adjoint<L>(g, mu, rho0, omega, F, Fc.kind != 0, nu, lam);
    }
#pragma unroll
    for (int k = 0; k < 32; ++k) v[k] = (in && k < Q) ? knn * nu[k] : 0.f;
    put_row(bufE, v);
  } else {
    __syncthreads();
  }

  // 16-byte operand of this lane: chunk c (of KCL) of node tile n
  auto read = [&](const unsigned char* buf, int c, int n, bool half) -> u4 {
    if (!half) return *reinterpret_cast<const u4*>(buf + c * 4096 + n * 1024 + l16);
    u4 v = *reinterpret_cast<const u4*>(buf + c * 4096 + n * 512 + (lane & 31) * 16);
    if (lg >= 2) v = u4{0u, 0u, 0u, 0u};
    return v;
  };

  // LeakyReLU masks of the hidden layers: bit 15 - (4 n + r) of word j is set
  // where the activation of row r of the wavefront's tile j at node tile n is
  // > 0
  unsigned m1[5] = {0, 0, 0, 0, 0}, m2[5] = {0, 0, 0, 0, 0}, m3[2] = {0, 0};
  // an activation rounds to a positive operand value above half of the
  // format's smallest positive number
  constexpr float kTiny = P == P_BF16 ? 0x1p-134f : 0x1p-25f;

  // (the whole offset in the vector part: a wide store must not be followed
  // at once by a write to its data registers, and the compiler keeps that
  // distance only where the scalar offset is no register.  With one, the first
  // dword of some lanes was the next value's.)
  auto put_rec = [&](int blk, int n, u4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(v, myrec, slot16 + (n * AJ::NREC + blk) * 1024, 0,
                                           NT ? kStoreNT : 0);
  };
  // One product of the chain: acc[j][n] over the chunks of layer l, then
  // ep(acc, n) per node tile.  rd(c, n): operand of chunk c and node tile n;
  // blk: record block of chunk 0.
  auto layer = [&](auto lc, int blk, auto&& rd, auto&& ep) {
    constexpr int l = decltype(lc)::value, T = AJ::TPW[l], KCL = AJ::KC[l],
                  s0 = AJ::first_step(l);
    f4 acc[T][4];
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int n = 0; n < 4; ++n) acc[j][n] = f4{0.f, 0.f, 0.f, 0.f};
    u4 xb[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) xb[n] = rd(0, n);
    static_for<KCL>([&](auto cc) {
      constexpr int c = decltype(cc)::value, s = s0 + c;
      issue(std::integral_constant<int, s + 2>{});
      const u4 kept = rd(c, wave);
      static_for<4>([&](auto nc) {
        constexpr int n = decltype(nc)::value;
#pragma unroll
        for (int j = 0; j < T; ++j) acc[j][n] = mma32<P>(ring[s % 3][j], xb[n], acc[j][n]);
        // the next chunk's operand, into the registers just consumed
        if constexpr (c + 1 < KCL) xb[n] = rd(c + 1, n);
        if constexpr (n == 3) put_rec(blk + c, wave, kept);
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    static_for<4>([&](auto nc) {
      ep(acc, decltype(nc)::value);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // Results as operands, to LDS: a pair of tiles, or the half hh of a shared
  // pair.  Only
  // the second pair of wavefront 3 (`tail`) is a layer's last chunk, which
  // holds 16 features: half of the lanes, 512 bytes per node tile.
  const int p0 = AJ::pair0(wave), ph = AJ::half_pair(wave), hh = wave & 1;
  const int tail = wave == 3, tstride = tail ? 512 : 1024;
  const bool tlive = !tail || lane < 32;
  auto put_pair = [&](unsigned char* buf, int p, int n, u2 lo, u2 hi) {
    const u4 o = {lo[0], lo[1], hi[0], hi[1]};
    *reinterpret_cast<u4*>(buf + p * 4096 + n * 1024 + l16) = o;
  };
  auto put_tail = [&](unsigned char* buf, int p, int n, u2 lo, u2 hi) {
    const u4 o = {lo[0], lo[1], hi[0], hi[1]};
    if (tlive) *reinterpret_cast<u4*>(buf + p * 4096 + n * tstride + l16) = o;
  };
  // node tile n of a 20-tile layer
  auto put5 = [&](unsigned char* buf, int n, const u2 (&f)[5]) {
    put_pair(buf, p0, n, f[0], f[1]);
    put_tail(buf, p0 + 1, n, f[2], f[3]);
    *reinterpret_cast<u2*>(buf + ph * 4096 + n * 1024 + l16 + 8 * hh) = f[4];
  };
  // first feature of this lane's rows of tile j
  auto feat5 = [&](int j) {
    return j < 4 ? 32 * (p0 + j / 2) + 8 * lg + 4 * (j % 2) : 32 * ph + 8 * lg + 4 * hh;
  };
  const float* vec = reinterpret_cast<const float*>(packed + 2 * (size_t)AJ::nw);
  // h = leaky(acc + bias) in the operand type; its four mask bits are
  // shifted into m, the last row in bit 0 (h rounds to a positive value where
  // kTiny - h is negative)
  auto activate = [&](f4 a, f4 bias, unsigned& m) -> u2 {
    f4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float t = a[r] + bias[r], st = kLeakySlope * t;
      // max(t, slope t), without the quieting of NaNs that fmaxf adds
      asm("v_max_f32 %0, %1, %2" : "=v"(v[r]) : "v"(t), "v"(st));
      m = __builtin_amdgcn_alignbit(m, __builtin_bit_cast(unsigned, kTiny - v[r]), 31);
    }
    asm("" : "+v"(m));  // (the compiler would keep the sixteen values instead)
    return to_frag<P>(v);
  };
  // acc times the mask's factor, 1 or the slope
  auto masked = [&](f4 a, unsigned m, int n) -> u2 {
    constexpr unsigned one = 0x3F800000u, slope = __builtin_bit_cast(unsigned, kLeakySlope);
    f4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const unsigned on = (unsigned)__builtin_amdgcn_sbfe((int)m, 15 - (4 * n + r), 1);
      v[r] = a[r] * __builtin_bit_cast(float, (on & one) | (~on & slope));
    }
    return to_frag<P>(v);
  };
  auto bias_of = [&](int base, int feat, int dim) {
    // (features past the padded width have no entry and stay zero)
    return feat < dim ? *reinterpret_cast<const f4*>(vec + base + feat) : f4{0.f, 0.f, 0.f, 0.f};
  };

  // the bias rows of the wavefront's tiles
  f4 bv[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) bv[j] = bias_of(W::fE1, feat5(j), W::D1);
  // H1 = leaky(X0 W1^T) (b1 in column Q, the constant column from the bias vector)
  layer(
      std::integral_constant<int, 0>{}, AJ::RX0,
      [&](int, int n) { return read(bufQ, 0, n, false); },
      [&](const f4 (&acc)[5][4], int n) {
        u2 f[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) f[j] = activate(acc[j][n], bv[j], m1[j]);
        put5(bufP, n, f);
      });
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 5; ++j) bv[j] = bias_of(W::fB2, feat5(j), W::D2);
  // H2 = leaky(H1 W2^T + b2)
  layer(
      std::integral_constant<int, 1>{}, AJ::RH1, [&](int c, int n) { return read(bufP, c, n, c == 9); },
      [&](const f4 (&acc)[5][4], int n) {
        u2 f[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) f[j] = activate(acc[j][n], bv[j], m2[j]);
        put5(bufQ, n, f);
      });
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) bv[j] = bias_of(W::fB3, 32 * wave + 8 * lg + 4 * j, W::D3);
  // H3 = leaky(H2 W3^T + b3): only its mask and the record are needed
  layer(
      std::integral_constant<int, 2>{}, AJ::RH2, [&](int c, int n) { return read(bufQ, c, n, c == 9); },
      [&](const f4 (&acc)[2][4], int n) {
        u2 f[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) f[j] = activate(acc[j][n], bv[j], m3[j]);
        put_rec(AJ::RH3 + wave, n, u4{f[0][0], f[0][1], f[1][0], f[1][1]});
      });
  // dZ3 = (dY W4) . leaky'(H3)
  layer(
      std::integral_constant<int, 3>{}, AJ::RDY,
      [&](int, int n) { return read(bufE, 0, n, false); },
      [&](const f4 (&acc)[2][4], int n) {
        put_tail(bufP, wave, n, masked(acc[0][n], m3[0], n), masked(acc[1][n], m3[1], n));
      });
  __syncthreads();
  // dZ2 = (dZ3 W3) . leaky'(H2)
  layer(
      std::integral_constant<int, 4>{}, AJ::RZ3, [&](int c, int n) { return read(bufP, c, n, c == 3); },
      [&](const f4 (&acc)[5][4], int n) {
        u2 f[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) f[j] = masked(acc[j][n], m2[j], n);
        put5(bufQ, n, f);
      });
  __syncthreads();
  // dZ1 = (dZ2 W2) . leaky'(H1)
  layer(
      std::integral_constant<int, 5>{}, AJ::RZ2, [&](int c, int n) { return read(bufQ, c, n, c == 9); },
      [&](const f4 (&acc)[5][4], int n) {
        u2 f[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) f[j] = masked(acc[j][n], m1[j], n);
        put5(bufP, n, f);
      });
  __syncthreads();
  // dX0 = dZ1 W1: wavefront w takes node tile w, rows of the inputs
  {
    constexpr int s0 = AJ::first_step(6);
    f4 acc[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
    static_for<10>([&](auto cc) {
      constexpr int c = decltype(cc)::value, s = s0 + c;
      issue(std::integral_constant<int, s + 2>{});
      const u4 xv = read(bufP, c, wave, c == 9);
      put_rec(AJ::RZ1 + c, wave, xv);
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[j] = mma32<P>(ring[s % 3][j], xv, acc[j]);
    });
    float* DX = reinterpret_cast<float*>(bufQ);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      *reinterpret_cast<f4*>(DX + (16 * wave + li) * SDX + 16 * j + 4 * lg) = acc[j];
  }
  __syncthreads();
  // lam^n_q(x - c_q): the non-network adjoint plus the input gradient
  if (wave == 0 && node < total) {
    const float* DX = reinterpret_cast<const float*>(bufQ) + lane * SDX;
    unsigned nd = node;
    asm("" : "+v"(nd));  // (formed again rather than kept through the layers)
    NodeOffsets e;
    e.start(G, Q, nd);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, lam[q] + DX[q]), rL0,
                                            e.pull<L>(q), (int)(q * plane4), 0);
  }
}

// ---------------------------------------------------------------------------
// Weight gradients.  Four sets of 16 x 16 gradient tiles, each a product of
// some record blocks over the nodes: dW2 in two (H1's chunks 0-4 and 5-9),
// dW3, and dW1 with dW4; 14 to 16 of the fifty blocks each, so that sixty
// are read for fifty.  A workgroup of eight wavefronts takes one set over
// one range of nodes and walks it 32 nodes at a time; the set's blocks of
// the 32 nodes come into LDS by direct loads, four steps ahead in five
// buffers of 32 KB (one workgroup per compute unit).  The four sets of a
// node range run on one XCD (workgroups go round the eight XCDs), so that
// the blocks two sets share come from its L2.
//
// Bound by the read of the records.  Ten smaller sets (84 blocks for fifty)
// with a barrier that waited for every load, one step in flight: 29 us at
// 32^3, 183 at 60 x 64 x 52; four sets and four steps in flight 23 and 175;
// with non-temporal loads 103 (see wide_adj_ranges).
// ---------------------------------------------------------------------------
constexpr int kWideSets = 4;

// record block that set S stages as its block k
template <int Q, int S>
__device__ constexpr int wide_staged(int k) {
  using A = WideAdj<Q>;
  if (S < 2) return k < 10 ? A::RZ2 + k : A::RH1 + 5 * S + (k - 10);
  if (S == 2) return k < 4 ? A::RZ3 + k : A::RH2 + (k - 4);
  return k == 0 ? A::RX0 : (k < 11 ? A::RZ1 + k - 1 : (k == 11 ? A::RDY : A::RH3 + k - 12));
}

// Waits until at most n of the wavefront's direct-to-LDS loads are in flight
// and its LDS reads are done, then for the workgroup.  (__syncthreads would
// wait for every load, and leave a single step in flight.)
template <int n>
__device__ inline void stage_barrier() {
  static_assert(n < 16, "vmcnt field");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0070 | n);  // vmcnt(n) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

constexpr int kWideStageBytes = 16 * 2048;

template <int Q, int P, bool NT, int S>
__device__ __forceinline__ void wide_adj_weights(const unsigned char* __restrict__ rec,
                                                 float* __restrict__ slab, int step0, int steps,
                                                 unsigned char* st0, unsigned char* st1,
                                                 unsigned char* st2, unsigned char* st3,
                                                 unsigned char* st4) {
  using AJ = WideAdj<Q>;
  constexpr int NB = S < 2 ? 15 : (S == 2 ? 14 : 16), NLD = 4;  // blocks; loads per wavefront
  constexpr int NR = S < 2 ? 5 : (S == 2 ? 4 : 2), NC = S < 3 ? 5 : 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)__builtin_amdgcn_workitem_id_x() >> 6);
  const int lane = __builtin_amdgcn_workitem_id_x() & 63, lg = lane >> 4, li = lane & 15;
  // the wavefront's tiles: first staged row and column unit (16 features;
  // two per block), first gradient tile, the matrix (rows x cols tiles at
  // slab tile g0)
  int ru, cu, gr, gc, rows, cols, g0;
  if constexpr (S < 2) {  // 4 x 2 wavefronts
    ru = 5 * (wave >> 1), cu = 20 + 5 * (wave & 1);
    gr = ru, gc = 10 * S + 5 * (wave & 1), rows = 19, cols = 19, g0 = AJ::G2;
  } else if constexpr (S == 2) {  // 2 x 4
    ru = 4 * (wave >> 2), cu = 8 + 5 * (wave & 3);
    gr = ru, gc = 5 * (wave & 3), rows = 7, cols = 19, g0 = AJ::G3;
  } else {  // five wavefronts on dW1, two on dW4; the eighth repeats the seventh's
    const bool w1 = wave < 5;
    const int w = w1 ? wave : (wave == 5 ? 0 : 1);
    ru = w1 ? 0 : 22, cu = (w1 ? 2 : 24) + 4 * w;
    gr = 0, gc = 4 * w, rows = wave < 7 ? 2 : 0, cols = w1 ? 19 : 7, g0 = w1 ? AJ::G1 : AJ::G4;
  }
  f4 acc[NR][NC];
#pragma unroll
  for (int i = 0; i < NR; ++i)
#pragma unroll
    for (int j = 0; j < NC; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

  // each staged block holds the two node tiles of the step, 1 KB each; every
  // wavefront issues NLD loads, the last one again where there are fewer
  const unsigned char* src = rec + (size_t)step0 * 2 * (AJ::NREC * 1024);
  int off[NLD], dst[NLD];
#pragma unroll
  for (int q = 0; q < NLD; ++q) {
    int k = wave + 8 * q;
    if (k >= 2 * NB) k = 2 * NB - 1;
    off[q] = ((k & 1) * AJ::NREC + wide_staged<Q, S>(k >> 1)) * 1024;
    dst[q] = k * 1024;
  }
  // (steps past the range load nothing, from a resource of no bytes: the count
  // of loads in flight is the same at every turn)
  auto issue = [&](int i, unsigned char* st) {
    const rsrc_t r = make_rsrc(reinterpret_cast<const float*>(src + (size_t)i * 2 * (AJ::NREC * 1024)),
                               i < steps ? 2 * AJ::NREC * 1024 : 0);
#pragma unroll
    for (int q = 0; q < NLD; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          r, (__attribute__((address_space(3))) void*)(st + dst[q]), 16, lane * 16, off[q], 0,
          NT ? kStoreNT : 0);
  };
  // transposed read: this lane addresses the 8-byte row of node 4 (lane / 16)
  // + (lane % 16) / 4, features 4 a .. 4 a + 3 (a = lane % 4) of the unit
  const int a = lane & 3, nd = 4 * lg + (li >> 2);
  const int tr = 16 * (16 * (a >> 1) + (nd ^ (8 * (a >> 1)))) + 8 * (a & 1);
  auto unit = [&](const unsigned char* st, int u) -> u4 {
    const unsigned char* p = st + (u >> 1) * 2048 + (u & 1) * 512 + tr;
    const u2 v0 = read_tr<P>(p), v1 = read_tr<P>(p + 1024);
    return u4{v0[0], v0[1], v1[0], v1[1]};
  };
  auto compute = [&](const unsigned char* st) {
    u4 ra[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) ra[i] = unit(st, ru + i);
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const u4 cb = unit(st, cu + j);
#pragma unroll
      for (int i = 0; i < NR; ++i) acc[i][j] = mma32<P>(ra[i], cb, acc[i][j]);
    }
  };
  auto turn = [&](int i, const unsigned char* cur, unsigned char* fill) {
    stage_barrier<3 * NLD>();
    issue(i + 4, fill);
    compute(cur);
  };
  issue(0, st0);
  issue(1, st1);
  issue(2, st2);
  issue(3, st3);
  // (whole rounds of the ring, then the rest: with an exit after every turn
  // the compiler loses count of the loads and waits for all of them)
  int i = 0;
  for (; i + 5 <= steps; i += 5) {
    turn(i, st0, st4);
    turn(i + 1, st1, st0);
    turn(i + 2, st2, st1);
    turn(i + 3, st3, st2);
    turn(i + 4, st4, st3);
  }
  const int rest = steps - i;
  if (rest > 0) turn(i, st0, st4);
  if (rest > 1) turn(i + 1, st1, st0);
  if (rest > 2) turn(i + 2, st2, st1);
  if (rest > 3) turn(i + 3, st3, st2);
  stage_barrier<0>();  // (the empty loads too are done before the LDS is given up)
#pragma unroll
  for (int i = 0; i < NR; ++i)
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int r = gr + i, c = gc + j;
      if (r < rows && c < cols)
        *reinterpret_cast<f4*>(slab + ((size_t)(g0 + r * cols + c) * 64 + lane) * 4) = acc[i][j];
    }
}

// grid: sets x splits; split k covers steps [k per, k per + per) of 32 nodes
// and writes slab k (zeros if there are none left for it).
template <int Q, int P, bool NT>
__global__ __launch_bounds__(512) void wide_adj_weight_kernel(
    const unsigned char* __restrict__ rec, float* __restrict__ part, int nsteps, int per, int nsplit) {
  __shared__ __attribute__((aligned(16))) unsigned char st0[kWideStageBytes];
  __shared__ __attribute__((aligned(16))) unsigned char st1[kWideStageBytes];
  __shared__ __attribute__((aligned(16))) unsigned char st2[kWideStageBytes];
  __shared__ __attribute__((aligned(16))) unsigned char st3[kWideStageBytes];
  __shared__ __attribute__((aligned(16))) unsigned char st4[kWideStageBytes];
  const int wg = (int)__builtin_amdgcn_workgroup_id_x();
  int set, split;
  if (nsplit % 8 == 0) {
    const int i = wg / 8;
    split = wg % 8 + 8 * (i / kWideSets);
    set = i % kWideSets;
  } else {
    split = wg / kWideSets;
    set = wg % kWideSets;
  }
  const int step0 = split * per, steps = min(per, nsteps - step0);
  float* slab = part + (size_t)split * (WideAdj<Q>::NG * 256);
  switch (set) {
    case 0: wide_adj_weights<Q, P, NT, 0>(rec, slab, step0, steps, st0, st1, st2, st3, st4); break;
    case 1: wide_adj_weights<Q, P, NT, 1>(rec, slab, step0, steps, st0, st1, st2, st3, st4); break;
    case 2: wide_adj_weights<Q, P, NT, 2>(rec, slab, step0, steps, st0, st1, st2, st3, st4); break;
    default: wide_adj_weights<Q, P, NT, 3>(rec, slab, step0, steps, st0, st1, st2, st3, st4); break;
  }
}

// dtheta += the sum over the slabs, in a fixed order.  One workgroup per
// gradient tile: wavefront w sums slabs w, w + 4, ..., the four sums are
// added in wave order.
template <int Q>
__global__ __launch_bounds__(256) void wide_adj_reduce_kernel(const float* __restrict__ part,
                                                              int nsplit,
                                                              float* __restrict__ dtheta) {
  using AJ = WideAdj<Q>;
  using W = WideBwd<Q>;
  __shared__ f4 red[4][64];
  const int t = blockIdx.x, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  f4 s = {0.f, 0.f, 0.f, 0.f};
  for (int k = w; k < nsplit; k += 4)
    s += *reinterpret_cast<const f4*>(part + ((size_t)k * AJ::NG + t) * 256 + lane * 4);
  red[w][lane] = s;
  __syncthreads();
  if (w != 0) return;
  s = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
  const int r0 = 4 * (lane >> 4), c0 = lane & 15;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    int p = -1;
    if (t < AJ::G3) {
      const int i = 16 * (t / 19) + r0 + r, j = 16 * (t % 19) + c0;
      if (i < W::N2) p = j < W::N1 ? W::pW2 + i * W::N1 + j : (j == W::ONE1 ? W::pb2 + i : -1);
    } else if (t < AJ::G1) {
      const int i = 16 * ((t - AJ::G3) / 19) + r0 + r, j = 16 * ((t - AJ::G3) % 19) + c0;
      if (i < W::N3) p = j < W::N2 ? W::pW3 + i * W::N2 + j : (j == W::ONE2 ? W::pb3 + i : -1);
    } else if (t < AJ::G4) {  // rows: input features, columns: layer-1 units
      const int i = 16 * ((t - AJ::G1) / 19) + r0 + r, j = 16 * ((t - AJ::G1) % 19) + c0;
      if (j < W::N1) p = i < Q ? W::pW1 + j * Q + i : (i == Q ? W::pb1 + j : -1);
    } else {
      const int i = 16 * ((t - AJ::G4) / 7) + r0 + r, j = 16 * ((t - AJ::G4) % 7) + c0;
      if (i < Q) p = j < W::N3 ? W::pW4 + i * W::N3 + j : (j == W::ONE3 ? W::pb4 + i : -1);
    }
    if (p >= 0) dtheta[p] += s[r];
  }
}

}  // namespace lbm

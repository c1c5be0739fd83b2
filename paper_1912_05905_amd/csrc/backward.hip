// Backward passes of the lattice operators on gfx950 (Implementation: the
// lattice operators have forward and backward passes on the GPU).  Every
// gradient is that of its forward operator for a scalar loss with
// dL/d(output) given; the linear operators' gradients are their adjoints:
//   splat  -> a slice of dL/dx (each vertex row scaled by 1 / sum_{J_v} b
//             when the forward normalised);
//   slice  -> a (raw) splat of dL/df over the lists J_v;
//   conv   -> dX: the convolution of dL/dY with W'[t] = W[mirror t]^T over
//             the adjoint table (1-hop: the same table; strided: the
//             Upsample table; Upsample: the Downsample table), on the
//             forward's MFMA kernel;
//             dW[t] = sum_v dL/dY_v^T X[nb(v,t)], dbias = sum_v dL/dY_v: a
//             gathered GEMM that reduces over vertices (k_conv_wgrad, split
//             over vertex chunks, partials added in chunk order).
// A ReLU in the forward masks dL/dY with Y > 0 first (derivative 0 at 0).
//   classifier fused with DeformSlice -> with f_p the DeformSlice output and
//             z_p = dL/dlogits_p: df_p = sum_j z_pj Wc[j] (then the
//             DeformSlice backward), dWc = sum_p z_p f_p^T, dbc = sum_p z_p
//             (point chunks, partials added in chunk order).
#include <algorithm>
#include <type_traits>

#include "lattice_internal.h"

namespace lat {
namespace {

constexpr int kBlock = 256;
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---- splat backward with normalisation: 1 / (vertex weight sum) ----
// One group of 16 lanes per vertex: the weight sum comes from the forward
// (wsum) or is summed over J_v by the lanes (0 where the sum is 0, as in the
// forward).  The slice that follows folds these factors into its weights:
// dividing the rows of dL/dx first wrote and read them once more (35 against
// 12 us in front of the slice, for 128 channels of a 200k-point room).  Narrow
// rows of large clouds gain nothing (16 channels of 1M points 90 against 83 us,
// of 200k 22 against 24).
constexpr int kScaleLanes = 16;

__global__ void __launch_bounds__(kBlock)
k_weight_sum_scale(const int32_t* __restrict__ offsets, const float* __restrict__ entry_w,
                   const float* __restrict__ wsum, int64_t n, float* __restrict__ scale) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (wsum) {   // one thread per vertex
    if (t < n) scale[t] = wsum[t] > 0.f ? 1.0f / wsum[t] : 0.f;
    return;
  }
  const int lane = threadIdx.x & (kScaleLanes - 1);
  const int64_t v = t / kScaleLanes;
  if (v >= n) return;   // a whole lane group
  float ws = 0.f;
  const int32_t b = offsets[v], e = offsets[v + 1];
#pragma unroll 8
  for (int32_t j = b + lane; j < e; j += kScaleLanes) ws += entry_w[j];
#pragma unroll
  for (int o = kScaleLanes / 2; o > 0; o >>= 1) ws += __shfl_xor(ws, o, kScaleLanes);
  if (lane == 0) scale[v] = ws > 0.f ? 1.0f / ws : 0.f;
}

// ---- convolution backward ----
// Taps 0 = self, 1..4 = +n_j, 5..8 = -n_j: the mirror of a tap negates its
// offset.
__device__ inline int mirror_tap(int t) { return t == 0 ? 0 : (t <= 4 ? t + 4 : t - 4); }

// Four values of a row of fp32 or bf16 elements (8-byte aligned for bf16).
template <bool BF16>
__device__ inline float4 load4(const void* base, int64_t at) {
  if constexpr (BF16) {
    const uint2 u = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(base) + at);
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                       __uint_as_float(u.y & 0xffff0000u));
  } else {
    return *reinterpret_cast<const float4*>(static_cast<const float*>(base) + at);
  }
}

// The two preparations of the convolution backward in one launch: the first
// mask_blocks workgroups write G = dY masked by Y > 0 (the forward's ReLU; 4
// channels per thread; bf16 values are masked as they are, so G stays
// exact), the rest write the adjoint convolution's weights Wt[t][i][o] =
// W[mirror t][o][i] (W laid out [tap][Cout][Cin]).  Either part may be empty.
template <bool BF16>
__global__ void __launch_bounds__(kBlock)
k_conv_bwd_prep(const void* __restrict__ dY, int64_t ld_dy, const void* __restrict__ Y, int64_t ld_y, int64_t n,
                void* __restrict__ G, int64_t ld_g, unsigned mask_blocks, const void* __restrict__ W, int Cout,
                int Cin, void* __restrict__ Wt) {
  using E = typename std::conditional<BF16, uint16_t, float>::type;
  if (blockIdx.x < mask_blocks) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const int c4 = Cout / 4;
    const int64_t v = q / c4;
    if (v >= n) return;
    const int c = 4 * static_cast<int>(q - v * c4);
    const E* d = static_cast<const E*>(dY) + v * ld_dy + c;
    const float4 y = load4<BF16>(Y, v * ld_y + c);
    E* g = static_cast<E*>(G) + v * ld_g + c;
    const bool on[4] = {y.x > 0.f, y.y > 0.f, y.z > 0.f, y.w > 0.f};
#pragma unroll
    for (int k = 0; k < 4; ++k) g[k] = on[k] ? d[k] : E(0);
    return;
  }
  const int64_t q = static_cast<int64_t>(blockIdx.x - mask_blocks) * kBlock + threadIdx.x;
  const int64_t per = static_cast<int64_t>(Cout) * Cin;
  if (q >= 9 * per) return;
  const int t = static_cast<int>(q / per);
  const int64_t r = q - t * per;
  const int i = static_cast<int>(r / Cout), o = static_cast<int>(r - static_cast<int64_t>(i) * Cout);
  static_cast<E*>(Wt)[q] = static_cast<const E*>(W)[(mirror_tap(t) * per) + static_cast<int64_t>(o) * Cin + i];
}

// dW[t][o][i] = sum_v G[v][o] X[nb(v,t)][i] as a GEMM with the vertices as
// the reduction dimension: A = G^T, B = the gathered rows.  A workgroup owns
// one tap, one 64 x 64 tile of (o, i) and one chunk of V vertices, a quarter
// of it per wave, and each wave multiplies whole 64 x 64 tiles with operands
// loaded straight into the MFMA layout: lane (i, g) loads the 4 channels 4 i
// .. 4 i + 3 of the rows its lane group g stands for, which serve four
// products whose row (or column) i stands for channel 4 i + e.
//   fp32: a step is 16 vertices, v_mfma_f32_16x16x4_f32, 16-byte loads;
//   bf16: a step is 32 vertices, v_mfma_f32_16x16x32_bf16 (bf16 products are
//         exact in fp32 and are summed in fp32); a lane's 8 rows x 4 channels
//         are turned into 8 rows per channel by byte permutes.
// Only vertices that have the tap are multiplied: a wave compacts 64 table
// entries at a time into a ring of (v, nb) pairs in LDS and takes full steps
// from it (on rooms and scans a quarter to a half of the pairs are missing).
// The four waves are added in wave order into part[chunk][tap][o][i].
// The workgroups of blockIdx.y = 0 sum the G columns (the bias gradient).
// Staging both operands in LDS, bf16 widened to fp32, the weight gradient took
// 1191 us at 128 x 128 bf16 on a 212k-vertex level and 23 us at 64 x 64 fp32 on
// the 16k vertices of a LiDAR scan; here 143 and 21 us.
constexpr int kWgTile = 64;
constexpr int kWgRing = 256;                 // (v, nb) pairs a wave can hold, a power of two
constexpr int kWgTargetBlocks = 768;         // three workgroups per compute unit over taps, tiles and chunks

template <bool BF16> struct WgRow;
template <> struct WgRow<false> {
  static constexpr int kStep = 16, kPer = 4;   // vertices per step, rows of it per lane
  float4 v;
  __device__ inline void load(const void* base, int64_t at) {
    v = *reinterpret_cast<const float4*>(static_cast<const float*>(base) + at);
  }
  __device__ inline void zero() { v = make_float4(0.f, 0.f, 0.f, 0.f); }
};
template <> struct WgRow<true> {
  static constexpr int kStep = 32, kPer = 8;
  uint2 v;
  __device__ inline void load(const void* base, int64_t at) {
    v = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(base) + at);
  }
  __device__ inline void zero() { v = make_uint2(0u, 0u); }
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The bf16 values of channel e of a lane's 8 rows, in row order.
template <int e>
__device__ inline bf16x8 wg_channel(const WgRow<true> (&r)[8]) {
  constexpr uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
  u32x4 o;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    o[q] = __builtin_amdgcn_perm(e < 2 ? r[2 * q + 1].v.x : r[2 * q + 1].v.y, e < 2 ? r[2 * q].v.x : r[2 * q].v.y, sel);
  return __builtin_bit_cast(bf16x8, o);
}

__device__ inline void wg_mma(f32x4 (&acc)[4][4], const WgRow<true> (&g)[8], const WgRow<true> (&x)[8]) {
  const bf16x8 a[4] = {wg_channel<0>(g), wg_channel<1>(g), wg_channel<2>(g), wg_channel<3>(g)};
  const bf16x8 b[4] = {wg_channel<0>(x), wg_channel<1>(x), wg_channel<2>(x), wg_channel<3>(x)};
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int f = 0; f < 4; ++f) acc[e][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[e], b[f], acc[e][f], 0, 0, 0);
}
__device__ inline void wg_mma(f32x4 (&acc)[4][4], const WgRow<false> (&g)[4], const WgRow<false> (&x)[4]) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const float a[4] = {g[s].v.x, g[s].v.y, g[s].v.z, g[s].v.w};
    const float b[4] = {x[s].v.x, x[s].v.y, x[s].v.z, x[s].v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int f = 0; f < 4; ++f) acc[e][f] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[f], acc[e][f], 0, 0, 0);
  }
}

template <bool BF16>
__global__ void __launch_bounds__(kBlock, 2)
k_conv_wgrad(const int32_t* __restrict__ nbr, int64_t ldn, int64_t n_out, int64_t V, const void* __restrict__ X,
             int64_t ld_x, int Cin, const void* __restrict__ G, int64_t ld_g, int Cout, int tiles_i,
             float* __restrict__ part, float* __restrict__ part_b) {
  using Row = WgRow<BF16>;
  constexpr int S = Row::kStep, NR = Row::kPer;
  __shared__ __align__(16) int2 ring_s[4][kWgRing];
  __shared__ __align__(16) float sum[kWgTile * kWgTile];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int64_t chunk = blockIdx.x;
  const int ti = static_cast<int>(blockIdx.z) % tiles_i, to = static_cast<int>(blockIdx.z) / tiles_i;
  const int o0 = to * kWgTile, i0 = ti * kWgTile;
  const int64_t c_begin = chunk * V, c_end = min(c_begin + V, n_out);

  if (blockIdx.y == 0) {
    // bias: the column sums of G over the chunk (16 rows side by side)
    if (part_b == nullptr || ti != 0) return;
    const int lr = t >> 4, lc = 4 * (t & 15);
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    if (o0 + lc < Cout)
#pragma unroll 8
      for (int64_t v = c_begin + lr; v < c_end; v += 16) {
        const float4 g = load4<BF16>(G, v * ld_g + o0 + lc);
        a.x += g.x; a.y += g.y; a.z += g.z; a.w += g.w;
      }
    *reinterpret_cast<float4*>(&sum[lr * kWgTile + lc]) = a;
    __syncthreads();
    if (t < kWgTile && o0 + t < Cout) {
      float s = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) s += sum[r * kWgTile + t];
      part_b[chunk * Cout + o0 + t] = s;
    }
    return;
  }
  const int tap = blockIdx.y - 1;
  const int32_t* tab = nbr + static_cast<int64_t>(tap) * ldn;
  int2* ring = ring_s[wave];
  // the wave's vertices; columns past the matrix read its last ones (their
  // products are not written)
  const int64_t sub = (V + 3) / 4;
  int64_t vb = min(c_begin + wave * sub, c_end);
  const int64_t v_end = min(vb + sub, c_end);
  const int64_t oc = min(o0 + 4 * li, Cout - 4), ic = min(i0 + 4 * li, Cin - 4);

  f32x4 acc[4][4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int f = 0; f < 4; ++f) acc[e][f] = f32x4{0.f, 0.f, 0.f, 0.f};

  uint32_t head = 0, tail = 0;   // pairs taken from and put into the ring
  int32_t un = vb + lane < v_end ? tab[vb + lane] : -1;
  // pairs of the next 64 vertices into the ring until it holds a step
  auto fill = [&]() {
    while (tail - head < static_cast<uint32_t>(S) && vb < v_end) {
      const int32_t u = un;
      const int32_t v = static_cast<int32_t>(vb) + lane;
      const uint64_t has = __ballot(u >= 0);
      vb += 64;
      un = vb + lane < v_end ? tab[vb + lane] : -1;
      const uint32_t at = __builtin_popcountll(has & ((uint64_t{1} << lane) - 1));
      if (u >= 0) ring[(tail + at) & (kWgRing - 1)] = make_int2(v, u);
      tail += __builtin_popcountll(has);
    }
    // a wave's LDS accesses take effect in order; the fences keep the
    // compiler from moving the reads above the writes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto fetch = [&](Row (&g)[NR], Row (&x)[NR], uint32_t count) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const uint32_t e = static_cast<uint32_t>(NR * lg + r);
      if (e < count) {
        const int2 p = ring[(head + e) & (kWgRing - 1)];
        g[r].load(G, static_cast<int64_t>(p.x) * ld_g + oc);
        x[r].load(X, static_cast<int64_t>(p.y) * ld_x + ic);
      } else {
        g[r].zero();
        x[r].zero();
      }
    }
  };
  Row ga[NR], xa[NR], gb[NR], xb[NR];
  fill();
  bool more = tail - head >= static_cast<uint32_t>(S);
  if (more) {
    fetch(ga, xa, S);
    head += S;
  }
  // the rows of a step are loaded while the step before is multiplied
  auto step = [&](Row (&g)[NR], Row (&x)[NR], Row (&gn)[NR], Row (&xn)[NR]) {
    fill();
    const bool next = tail - head >= static_cast<uint32_t>(S);
    if (next) {
      fetch(gn, xn, S);
      head += S;
    }
    wg_mma(acc, g, x);
    return next;
  };
  while (more) {
    more = step(ga, xa, gb, xb);
    if (!more) break;
    more = step(gb, xb, ga, xa);
  }
  if (tail != head) {
    fetch(ga, xa, tail - head);
    wg_mma(acc, ga, xa);
  }

  // lane (i, g) of product (e, f) holds o = 4 (4 g + r) + e, i = 4 i + f
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          f32x4* d = reinterpret_cast<f32x4*>(&sum[(16 * lg + 4 * r + e) * kWgTile + 4 * li]);
          f32x4 v = f32x4{acc[e][0][r], acc[e][1][r], acc[e][2][r], acc[e][3][r]};
          if (w > 0) v += *d;
          *d = v;
        }
    }
    __syncthreads();
  }
  float* P = part + (chunk * 9 + tap) * static_cast<int64_t>(Cout) * Cin;
  for (int q = t; q < kWgTile * kWgTile / 4; q += kBlock) {
    const int o = o0 + q / (kWgTile / 4), i = i0 + 4 * (q % (kWgTile / 4));
    if (o < Cout && i < Cin)
      *reinterpret_cast<f32x4*>(P + static_cast<int64_t>(o) * Cin + i) = *reinterpret_cast<const f32x4*>(&sum[4 * q]);
  }
}

// dW = sum over chunks of the partials, dbias likewise; fixed order: a
// workgroup takes 64 groups of 4 consecutive entries (count and Cout are
// multiples of 4), four slices of the chunks are summed side by side and added
// in slice order.
constexpr int kWgRedSlices = 4, kWgRedQuads = kBlock / kWgRedSlices;

__global__ void __launch_bounds__(kBlock)
k_wgrad_reduce(const float* __restrict__ part, const float* __restrict__ part_b, int64_t chunks, int64_t count,
               int Cout, float* __restrict__ dW, float* __restrict__ dbias) {
  __shared__ f32x4 sh[kWgRedSlices][kWgRedQuads];
  const int qi = threadIdx.x % kWgRedQuads, sl = threadIdx.x / kWgRedQuads;
  const int64_t q = 4 * (static_cast<int64_t>(blockIdx.x) * kWgRedQuads + qi);
  const float* src = nullptr;
  int64_t stride = 0;
  float* dst = nullptr;
  if (q < count) {
    src = part + q;
    stride = count;
    dst = dW ? dW + q : nullptr;
  } else if (q < count + Cout) {
    src = part_b + (q - count);
    stride = Cout;
    dst = dbias ? dbias + (q - count) : nullptr;
  }
  f32x4 a = {0.f, 0.f, 0.f, 0.f};
  if (dst)
#pragma unroll 8
    for (int64_t c = sl; c < chunks; c += kWgRedSlices) a += *reinterpret_cast<const f32x4*>(src + c * stride);
  sh[sl][qi] = a;
  __syncthreads();
  if (sl != 0 || !dst) return;
#pragma unroll
  for (int k = 1; k < kWgRedSlices; ++k) a += sh[k][qi];
  *reinterpret_cast<f32x4*>(dst) = a;
}

inline unsigned blocks_for(int64_t threads) { return static_cast<unsigned>((threads + kBlock - 1) / kBlock); }

// Vertex chunks of the weight gradient: three workgroups per compute unit
// over taps and tiles (more chunks would only grow the partials the reduction
// reads), in multiples of 8 so that the taps of a chunk, which gather the same
// rows, run on one XCD (workgroup b runs on XCD b % 8), and at least 64
// vertices each.  From three tiles on, a chunk's partials (150 KB a tile) cost
// more than small chunks gain, and more than 8 chunks have at least 256
// vertices: 128 x 128 fp32 on 1.3k and 3.1k vertices 18.5 and 24.5 us with 64,
// 12.7 and 20.8 here; with 8 chunks 256 x 256 on 1.3k takes 29.7, with 6 31.5.
// Wide layers have 8 chunks where 512 workgroups in all would be one (512 x 512:
// 75 MB of partials instead of 9.4): 76 and 391 us on 1.3k and 8.4k vertices, with
// one chunk and operands through LDS 101 and 653.
void wgrad_chunks(int64_t n_out, int tiles, int64_t* chunks, int64_t* V) {
  int64_t want = std::max<int64_t>(8, (kWgTargetBlocks / (9 * static_cast<int64_t>(tiles)) + 7) / 8 * 8);
  if (tiles >= 3) want = std::min<int64_t>(want, std::max<int64_t>(8, (n_out + 255) / 256));
  want = std::min<int64_t>(want, (n_out + 63) / 64);
  int64_t v = (n_out + want - 1) / want;
  v = (v + 63) / 64 * 64;
  *V = v;
  *chunks = (n_out + v - 1) / v;
}

// ---- linear layers backward (the classifier fused with DeformSlice, the
// 1x1 layers of Distribute + PointNet) ----
// For out_p = W a_p + b over m rows p (W: K x C, [out][in]) and z = dL/dout:
//   dA_p = sum_j z_pj W[j]   (k_lin_dinput),
//   dW = sum_p z_p a_p^T, db = sum_p z_p   (k_lin_wgrad over chunks of rows,
//   then k_lin_reduce adds the chunks' partials).
// Both products run on v_mfma_f32_16x16x4_f32 with operands loaded straight
// into its layout (16 bytes a lane), 64 columns of C per workgroup: rows are
// read once per column block and nothing but the weights is staged, so the
// passes are bound by the rows' memory traffic.  At 480,000 rows, K = 64, C =
// 32 (the last PointNet layer of a LiDAR scan) they took 192 (dA), 279 (dW)
// and 239 us (the partials, one thread per output over 1,000 of them) as FMA
// loops, and 63 (dA), 92 (dW) and 6 us here with the maxima's rows routed on
// the fly; at 200,000 rows, K = 20, C = 128 (the head of a room) 91, 147 and 215
// us, and 38, 38 and 6 us here.
constexpr int kLinCols = 64;        // columns of C per workgroup
constexpr int kLinMaxChunks = 1024;
constexpr int64_t kLinMaxPartial = 4 << 20;   // floats of partials aimed at
constexpr int kLinRedOut = 16, kLinRedSlices = kBlock / kLinRedOut;

// The rows z_p: given, or dL/dx of the maximum over a vertex's list routed to
// its rows: row p of vertex v = ev[p] holds dX[v][j] where p is the row of
// channel j's maximum (am), else 0.  get<N>(key(p), p, j, o) is o = z_p[j .. j
// + N - 1], j a multiple of N, entries past K being 0; the key is loaded ahead.
// V4: rows of z allow 16-byte loads.
template <bool V4>
struct GivenRows {
  const float* z;
  int64_t ld;
  int K;
  __device__ inline int32_t key(int64_t) const { return 0; }
  template <int N>
  __device__ inline void get(int32_t, int64_t p, int j, float (&o)[N]) const {
    const float* r = z + p * ld + j;
    if constexpr (V4 && N == 4) {
      const float4 v = *reinterpret_cast<const float4*>(r);
      o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    } else if constexpr (V4 && N == 2) {
      const float2 v = *reinterpret_cast<const float2*>(r);
      o[0] = v.x; o[1] = v.y;
    } else {
#pragma unroll
      for (int e = 0; e < N; ++e) o[e] = j + e < K ? r[e] : 0.f;
    }
  }
};
struct RoutedRows {
  const int32_t* ev;
  const int32_t* am;
  const float* dX;
  int64_t ld;
  int K;
  __device__ inline int32_t key(int64_t p) const { return ev[p]; }
  template <int N>
  __device__ inline void get(int32_t v, int64_t p, int j, float (&o)[N]) const {
    const int32_t* a = am + static_cast<int64_t>(v) * K + j;
    const float* d = dX + static_cast<int64_t>(v) * ld + j;
    const int32_t r = static_cast<int32_t>(p);
    if constexpr (N == 4) {
      const int4 av = *reinterpret_cast<const int4*>(a);
      const float4 dv = *reinterpret_cast<const float4*>(d);
      o[0] = av.x == r ? dv.x : 0.f;
      o[1] = av.y == r ? dv.y : 0.f;
      o[2] = av.z == r ? dv.z : 0.f;
      o[3] = av.w == r ? dv.w : 0.f;
    } else {
#pragma unroll
      for (int e = 0; e < N; ++e) o[e] = j + e < K && a[e] == r ? d[e] : 0.f;
    }
  }
};

// dA (m x C): 16 rows a step and wave.  A = W^T (LDS, fragment order), B = z^T:
// lane (i, g) holds z[p0 + i][16 jb + 4 g + s] for step s of block jb, and
// receives dA[p0 + i][c0 + 16 nb + 4 g + r].
template <int KB, class Rows>
__global__ void __launch_bounds__(kBlock)
k_lin_dinput(Rows rows, const float* __restrict__ W, int K, int C, int64_t m, float* __restrict__ df, int64_t ld_df) {
  __shared__ __align__(16) float ws[KB * 4 * 64 * 4];   // [jb][nb][lane][s]
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int c0 = blockIdx.y * kLinCols;
  for (int q = t; q < KB * 4 * 64 * 4; q += kBlock) {
    const int s = q & 3, L = (q >> 2) & 63, nb = (q >> 8) & 3, jb = q >> 10;
    const int j = 16 * jb + 4 * (L >> 4) + s, c = c0 + 16 * nb + (L & 15);
    ws[q] = (j < K && c < C) ? W[static_cast<int64_t>(j) * C + c] : 0.f;
  }
  __syncthreads();
  const int64_t groups = (m + 15) / 16;
  const f32x4* wf = reinterpret_cast<const f32x4*>(ws) + lane;
  const int64_t step = static_cast<int64_t>(gridDim.x) * 4;
  // past the last row: zeros, no access
  auto load_key = [&](int64_t grp) {
    const int64_t p = grp * 16 + li;
    return p < m ? rows.key(p) : 0;
  };
  auto load = [&](int64_t grp, int32_t key, float (&zr)[KB][4]) {
    const int64_t p = grp * 16 + li;
#pragma unroll
    for (int jb = 0; jb < KB; ++jb) {
      const int j = 16 * jb + 4 * lg;
#pragma unroll
      for (int s = 0; s < 4; ++s) zr[jb][s] = 0.f;
      if (p < m && j < K) rows.get(key, p, j, zr[jb]);
    }
  };
  float zc[KB][4], zn[KB][4];
  int64_t grp = static_cast<int64_t>(blockIdx.x) * 4 + wave;
  int32_t key = 0;
  if (grp < groups) {
    load(grp, load_key(grp), zc);
    key = load_key(grp + step);
  }
  for (; grp < groups; grp += step) {
    load(grp + step, key, zn);
    key = load_key(grp + 2 * step);
    f32x4 acc[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int jb = 0; jb < KB; ++jb) {
      f32x4 w[4];
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) w[nb] = wf[(jb * 4 + nb) * 64];
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
          acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[nb][s], zc[jb][s], acc[nb], 0, 0, 0);
    }
    const int64_t p = grp * 16 + li;
    if (p < m) {
      float* o = df + p * ld_df + c0 + 4 * lg;
#pragma unroll
      for (int nb = 0; nb < 4; ++nb)
        if (c0 + 16 * nb + 4 * lg < C) *reinterpret_cast<f32x4*>(o + 16 * nb) = acc[nb];
    }
#pragma unroll
    for (int jb = 0; jb < KB; ++jb)
#pragma unroll
      for (int s = 0; s < 4; ++s) zc[jb][s] = zn[jb][s];
  }
}

// Workgroup (w, cb): over chunk w of the rows, part[w][j C + c] = sum_p z_pj
// a_pc for the columns of block cb, and for cb = 0 part[w][K C + j] = sum_p
// z_pj.  A = z^T: lane (i, g) holds z[p + g][KB i + jb] for block jb; B = a: the
// lane's float4 a[p + g][c0 + 4 i ..] feeds four products whose column i stands
// for c0 + 4 i + nb.  The four waves take 16 rows each in turn and are added in
// wave order.
template <int KB, class Rows>
__global__ void __launch_bounds__(kBlock)
k_lin_wgrad(Rows rows, const float* __restrict__ f, int64_t ld_f, int K, int C, int64_t m, int64_t chunk,
            float* __restrict__ part) {
  __shared__ __align__(16) float sum[KB * 16 * kLinCols];   // [j][c]
  __shared__ float sb[4][KB * 16];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int c0 = blockIdx.y * kLinCols;
  const int64_t p0 = static_cast<int64_t>(blockIdx.x) * chunk;
  const int64_t p1 = min(p0 + chunk, m);
  const bool col_ok = c0 + 4 * li < C;
  constexpr int S = KB > 2 ? 4 : 8;   // rows in flight per lane
  f32x4 acc[KB][4];
  float bs[KB];
#pragma unroll
  for (int jb = 0; jb < KB; ++jb) {
    bs[jb] = 0.f;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) acc[jb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  int32_t key[S];
  auto load_keys = [&](int64_t pb) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int64_t p = pb + 4 * s + lg;
      key[s] = p < p1 ? rows.key(p) : 0;
    }
  };
  const int j0 = KB * li;   // the lane's columns of z
  load_keys(p0 + 4 * S * wave);
  for (int64_t pb = p0 + 4 * S * wave; pb < p1; pb += 16 * S) {
    float4 a[S];
    float zr[S][KB];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int64_t p = pb + 4 * s + lg;
      a[s] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (p < p1 && col_ok) a[s] = *reinterpret_cast<const float4*>(f + p * ld_f + c0 + 4 * li);
#pragma unroll
      for (int jb = 0; jb < KB; ++jb) zr[s][jb] = 0.f;
      if (p < p1 && j0 < K) rows.get(key[s], p, j0, zr[s]);
    }
    load_keys(pb + 16 * S);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const float av[4] = {a[s].x, a[s].y, a[s].z, a[s].w};
#pragma unroll
      for (int jb = 0; jb < KB; ++jb) {
        bs[jb] += zr[s][jb];
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
          acc[jb][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(zr[s][jb], av[nb], acc[jb][nb], 0, 0, 0);
      }
    }
  }
  // lane (i, g) of block (jb, nb) holds j = KB (4 g + r) + jb, c = c0 + 4 i + nb
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int jb = 0; jb < KB; ++jb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          f32x4* d = reinterpret_cast<f32x4*>(&sum[(KB * (4 * lg + r) + jb) * kLinCols + 4 * li]);
          f32x4 v = f32x4{acc[jb][0][r], acc[jb][1][r], acc[jb][2][r], acc[jb][3][r]};
          if (w > 0) v += *d;
          *d = v;
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int jb = 0; jb < KB; ++jb) {
    float v = bs[jb];
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (lg == 0) sb[wave][j0 + jb] = v;
  }
  __syncthreads();
  float* dst = part + static_cast<int64_t>(blockIdx.x) * (static_cast<int64_t>(K) * C + K);
  const int cols = min(kLinCols, C - c0);
  for (int e = t; e < K * kLinCols; e += kBlock) {
    const int j = e / kLinCols, c = e - j * kLinCols;
    if (c < cols) dst[static_cast<int64_t>(j) * C + c0 + c] = sum[e];
  }
  if (blockIdx.y == 0)
    for (int j = t; j < K; j += kBlock) dst[static_cast<int64_t>(K) * C + j] = (sb[0][j] + sb[1][j]) + (sb[2][j] + sb[3][j]);
}

// dW[j][c] (c < C_out, row stride C_out) and db[j]: sums over the chunks of
// part[w][o].  A workgroup takes 16 outputs; 16 slices of the chunks are
// summed side by side (a thread walking all chunks of its output is a chain of
// a thousand dependent adds) and then added in slice order.
__global__ void __launch_bounds__(kBlock)
k_lin_reduce(const float* __restrict__ part, int chunks, int K, int C, int C_out, float* __restrict__ dWc,
             float* __restrict__ dbc) {
  __shared__ float sh[kLinRedSlices][kLinRedOut];
  const int nout = K * C + K;
  const int t = threadIdx.x, oi = t % kLinRedOut, sl = t / kLinRedOut;
  const int o = blockIdx.x * kLinRedOut + oi;
  float a = 0.f;
  if (o < nout)
#pragma unroll 8
    for (int w = sl; w < chunks; w += kLinRedSlices) a += part[static_cast<int64_t>(w) * nout + o];
  sh[sl][oi] = a;
  __syncthreads();
  if (sl != 0 || o >= nout) return;
  a = 0.f;
#pragma unroll
  for (int s = 0; s < kLinRedSlices; ++s) a += sh[s][oi];
  if (o < K * C) {
    const int j = o / C, c = o - j * C;
    if (dWc && c < C_out) dWc[j * C_out + c] = a;
  } else if (dbc) {
    dbc[o - K * C] = a;
  }
}

// Row chunks of k_lin_wgrad: enough for every compute unit (the column blocks
// multiply them), fewer where the partials would outgrow what they are read
// back for, and a multiple of the rows the four waves take in one step.
void lin_chunks(int64_t m, int K, int C, int64_t* chunk, int* chunks) {
  const int64_t nout = static_cast<int64_t>(K) * C + K;
  const int64_t want = std::min<int64_t>(kLinMaxChunks, std::max<int64_t>(64, kLinMaxPartial / nout));
  int64_t c = std::max<int64_t>(128, (m + want - 1) / want);
  c = (c + 127) / 128 * 128;
  *chunk = c;
  *chunks = static_cast<int>(std::max<int64_t>(1, (m + c - 1) / c));
}

}  // namespace

void launch_weight_sum_scale(const int32_t* offsets, const float* entry_w, const float* wsum, int64_t n, float* scale,
                             hipStream_t s) {
  if (n <= 0) return;
  launch(k_weight_sum_scale, dim3(blocks_for(wsum ? n : n * kScaleLanes)), dim3(kBlock), 0, s, offsets, entry_w, wsum, n,
         scale);
}

void launch_conv_bwd_prep(const void* dY, int64_t ld_dy, const void* Y, int64_t ld_y, int64_t n, void* G,
                          int64_t ld_g, const void* W, int Cout, int Cin, void* Wt, int bf16, hipStream_t s) {
  const unsigned mb = (G && n > 0) ? blocks_for(n * (Cout / 4)) : 0;
  const unsigned wb = Wt ? blocks_for(9LL * Cout * Cin) : 0;
  if (mb + wb == 0) return;
  if (bf16)
    launch(k_conv_bwd_prep<true>, dim3(mb + wb), dim3(kBlock), 0, s, dY, ld_dy, Y, ld_y, n, G, ld_g, mb, W, Cout, Cin,
           Wt);
  else
    launch(k_conv_bwd_prep<false>, dim3(mb + wb), dim3(kBlock), 0, s, dY, ld_dy, Y, ld_y, n, G, ld_g, mb, W, Cout, Cin,
           Wt);
}

int64_t wgrad_partial_floats(int64_t n_out, int Cout, int Cin) {
  if (n_out <= 0) return 0;
  const int tiles = ((Cout + kWgTile - 1) / kWgTile) * ((Cin + kWgTile - 1) / kWgTile);
  int64_t chunks, V;
  wgrad_chunks(n_out, tiles, &chunks, &V);
  return chunks * (9LL * Cout * Cin + Cout);
}

void launch_conv_wgrad(const int32_t* nbr, int64_t ldn, int64_t n_out, const void* X, int64_t ld_x, int Cin,
                       const void* G, int64_t ld_g, int Cout, float* dW, float* dbias, float* partials, int bf16,
                       hipStream_t s) {
  const int tiles_o = (Cout + kWgTile - 1) / kWgTile, tiles_i = (Cin + kWgTile - 1) / kWgTile;
  const int64_t count = 9LL * Cout * Cin;
  int64_t chunks = 0, V = 0;
  if (n_out > 0) wgrad_chunks(n_out, tiles_o * tiles_i, &chunks, &V);
  float* part = partials;
  float* part_b = dbias ? partials + chunks * count : nullptr;
  if (chunks > 0) {
    // blockIdx.y: the bias, then the taps
    const dim3 grid(static_cast<unsigned>(chunks), dW ? 10 : 1, static_cast<unsigned>(tiles_o * tiles_i));
    if (bf16)
      launch(k_conv_wgrad<true>, grid, dim3(kBlock), 0, s, nbr, ldn, n_out, V, X, ld_x, Cin, G, ld_g, Cout, tiles_i,
             part, part_b);
    else
      launch(k_conv_wgrad<false>, grid, dim3(kBlock), 0, s, nbr, ldn, n_out, V, X, ld_x, Cin, G, ld_g, Cout, tiles_i,
             part, part_b);
  }
  // with no output vertex (chunks = 0) the sums below are zero
  launch(k_wgrad_reduce, dim3(static_cast<unsigned>(((count + Cout) / 4 + kWgRedQuads - 1) / kWgRedQuads)), dim3(kBlock), 0, s, static_cast<const float*>(part),
         static_cast<const float*>(part_b), chunks, count, Cout, dW, dbias);
}

}  // namespace lat

namespace lat {

int64_t classify_backward_partial_floats(int64_t m, int K, int C) {
  int64_t chunk;
  int chunks;
  lin_chunks(m, K, C, &chunk, &chunks);
  return static_cast<int64_t>(chunks) * (static_cast<int64_t>(K) * C + K);
}

namespace {
// df by rows that allow 16-byte loads or not (Rows4), dW and db by Rows
template <class Rows4, class Rows>
void linear_backward(const Rows4& rows4, const Rows& rows, const float* W, int K, int C, int64_t m, const float* f,
                     int64_t ld_f, float* df, int64_t ld_df, float* dW, int C_out, float* db, float* part,
                     hipStream_t s) {
  const unsigned col_blocks = static_cast<unsigned>((C + kLinCols - 1) / kLinCols);
  const int kb = (K + 15) / 16;   // K <= 64
  auto by_kb = [&](auto go) {
    if (kb <= 1) go(std::integral_constant<int, 1>{});
    else if (kb == 2) go(std::integral_constant<int, 2>{});
    else if (kb == 3) go(std::integral_constant<int, 3>{});
    else go(std::integral_constant<int, 4>{});
  };
  if (df && m > 0) {
    const unsigned gx = static_cast<unsigned>(std::min<int64_t>((m + 63) / 64, std::max(1u, 2048 / col_blocks)));
    by_kb([&](auto kb_c) {
      launch((k_lin_dinput<decltype(kb_c)::value, Rows4>), dim3(gx, col_blocks), dim3(kBlock), 0, s, rows4, W, K, C, m,
             df, ld_df);
    });
  }
  if (!dW && !db) return;
  const int nout = K * C + K;
  int64_t chunk;
  int chunks;
  lin_chunks(m, K, C, &chunk, &chunks);
  if (m > 0)
    by_kb([&](auto kb_c) {
      launch((k_lin_wgrad<decltype(kb_c)::value, Rows>), dim3(static_cast<unsigned>(chunks), col_blocks), dim3(kBlock), 0,
             s, rows, f, ld_f, K, C, m, chunk, part);
    });
  launch(k_lin_reduce, dim3(static_cast<unsigned>((nout + kLinRedOut - 1) / kLinRedOut)), dim3(kBlock), 0, s,
         static_cast<const float*>(part), m > 0 ? chunks : 0, K, C, C_out, dW, db);
}
}  // namespace

void launch_linear_backward(const float* z, int64_t ld_z, const float* W, int K, int C, int64_t m, const float* f,
                            int64_t ld_f, float* df, int64_t ld_df, float* dW, int C_out, float* db, float* part,
                            hipStream_t s) {
  const GivenRows<true> r4{z, ld_z, K};
  const GivenRows<false> r1{z, ld_z, K};
  if (K % 4 == 0 && ld_z % 4 == 0 && (reinterpret_cast<uintptr_t>(z) & 15u) == 0)
    linear_backward(r4, r4, W, K, C, m, f, ld_f, df, ld_df, dW, C_out, db, part, s);
  else
    linear_backward(r1, r1, W, K, C, m, f, ld_f, df, ld_df, dW, C_out, db, part, s);
}

void launch_linear_backward_routed(const int32_t* ev, const int32_t* am, const float* dX, int64_t ld_dX, const float* W,
                                   int K, int C, int64_t m, const float* f, int64_t ld_f, float* df, int64_t ld_df,
                                   float* dW, int C_out, float* db, float* part, hipStream_t s) {
  const RoutedRows r{ev, am, dX, ld_dX, K};
  linear_backward(r, r, W, K, C, m, f, ld_f, df, ld_df, dW, C_out, db, part, s);
}

void launch_classify_backward(const float* z, int64_t ld_z, const float* Wc, int K, int C, int64_t m, const float* f,
                              float* df, float* dWc, float* dbc, float* part, hipStream_t s) {
  ScopedKernelTimer tm("classify_bwd", s);
  launch_linear_backward(z, ld_z, Wc, K, C, m, f, C, df, C, dWc, C, dbc, part, s);
}

}  // namespace lat

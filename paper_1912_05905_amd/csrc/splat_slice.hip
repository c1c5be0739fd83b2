// Splat, Slice and DeformSlice on gfx950.  All three are gathers bounded by
// HBM bandwidth: a row of C channels is handled by a group of LPR lanes
// (LPR a power of two), each lane moving 16 bytes (4 fp32 or 8 bf16 channels)
// per access so that a row is one contiguous, fully used transaction.
#include <algorithm>

#include <type_traits>
#include <utility>

#include "lattice_internal.h"

namespace lat {
namespace {

constexpr int kBlock = 256;
constexpr int64_t kDeformBwdGrid = 1024;   // workgroups of the DeformSlice backward's per-point pass
constexpr unsigned kClassifyGrid = 2048;   // workgroups of the fused classifier (a multiple of 8)
constexpr int64_t kSliceWideM = 4096;         // points beyond which rows wider than 128 channels are sliced by a wave,
constexpr int64_t kSliceWideM128 = 131072;    // and bf16 rows of 65 to 128 channels
constexpr int kClassifyMaxWeights = 16384; // K x C classifier weights staged in LDS
constexpr int kClassifyTileC = 256;        // widest rows whose LDS tiles leave room for the weights
constexpr int kClassifyMaxLds = 160 * 1024;

// float -> bfloat16, round to nearest even (NaN stays NaN).
// Row / chunk index of a lane group with XCD-contiguous workgroup order:
// workgroup b runs on XCD b % 8, so consecutive work items (which share
// feature or vertex rows) are given to workgroups of the same XCD and meet in
// its L2.  Launches use xcd_grid() workgroups.
template <int LPR>
__device__ inline int64_t xcd_item(unsigned nblocks_logical) {
  const unsigned b = blockIdx.x;
  const unsigned per = (nblocks_logical + 7) / 8;
  const int64_t logical = static_cast<int64_t>(b % 8) * per + b / 8;
  return (logical * kBlock + threadIdx.x) / LPR;
}

inline unsigned xcd_grid(unsigned nblocks_logical) { return ((nblocks_logical + 7) / 8) * 8; }

// Point outputs (slice, DeformSlice) are written once and not read back by
// the kernel: non-temporal stores keep them out of the L2.
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// Store of 4 floats of a point row.  Non-temporal when a lane's part of the
// row is 16 bytes (fp32 inputs: a wave's store covers whole lines); with
// wider parts (bf16 inputs, 32 bytes a lane) one store instruction leaves
// gaps in every line, which the L2 has to merge, so those stay ordinary.
template <bool NT>
__device__ inline void store_row4(float* o, float a, float b, float c, float d) {
  if constexpr (NT)
    __builtin_nontemporal_store(f32x4_t{a, b, c, d}, reinterpret_cast<f32x4_t*>(o));
  else
    *reinterpret_cast<float4*>(o) = make_float4(a, b, c, d);
}

// f(std::integral_constant<int, i>) for i = 0 .. N-1, unrolled.
template <class F, int... I>
__device__ inline void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ inline void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Value of lane J of this lane's group of G lanes: a DPP row broadcast for
// G = 16 (a group is a row), a swizzle for G = 8 (bit mask mode: keep the
// group bits of the lane, set the low three to J).
template <int G, int J>
__device__ inline int32_t group_bcast(int32_t x) {
  static_assert(G == 16 || G == 8, "16- or 8-lane groups");
  if constexpr (G == 16) return __builtin_amdgcn_update_dpp(0, x, 0x150 + J, 0xF, 0xF, false);
  else return __builtin_amdgcn_ds_swizzle(x, 0x18 | (J << 5));
}

// Value of lane ^ OFF: DPP for partners inside a 16-lane row that DPP can
// name (xor 1 and 2 by quad permutation, xor 8 as a rotation by 8), a
// swizzle for xor 4 and 16 (within 32 lanes), a permute across halves.
template <int OFF>
__device__ inline float xor_lane(float v) {
  const int x = __float_as_int(v);
  if constexpr (OFF == 1) return __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false));
  else if constexpr (OFF == 2) return __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false));
  else if constexpr (OFF == 8) return __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, false));
  else if constexpr (OFF == 4 || OFF == 16) return __int_as_float(__builtin_amdgcn_ds_swizzle(x, 0x1F | (OFF << 10)));
  else return __shfl_xor(v, OFF);
}

// Sum over the LPR lanes of a group, every lane receiving it.
template <int LPR>
__device__ inline float group_sum(float v) {
  if constexpr (LPR > 1) v += xor_lane<1>(v);
  if constexpr (LPR > 2) v += xor_lane<2>(v);
  if constexpr (LPR > 4) v += xor_lane<4>(v);
  if constexpr (LPR > 8) v += xor_lane<8>(v);
  if constexpr (LPR > 16) v += xor_lane<16>(v);
  if constexpr (LPR > 32) v += xor_lane<32>(v);
  return v;
}


// A 16-byte chunk of a row as 8 floats (bf16) or 4 floats (fp32).
template <bool BF16> struct Chunk;
template <> struct Chunk<false> {
  static constexpr int N = 4;
  float v[4];
  __device__ inline void load(const void* base, int64_t elem) {
    const float4 x = *reinterpret_cast<const float4*>(static_cast<const float*>(base) + elem);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
  }
  __device__ inline void store(void* base, int64_t elem) const {
    *reinterpret_cast<float4*>(static_cast<float*>(base) + elem) = make_float4(v[0], v[1], v[2], v[3]);
  }
};
template <> struct Chunk<true> {
  static constexpr int N = 8;
  float v[8];
  __device__ inline void load(const void* base, int64_t elem) {
    const uint4 x = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(base) + elem);
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  __device__ inline void store(void* base, int64_t elem) const {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
    *reinterpret_cast<uint4*>(static_cast<uint16_t*>(base) + elem) = make_uint4(w[0], w[1], w[2], w[3]);
  }
};

// 4 bf16 channels, for lanes that store a whole 16 bytes of fp32 each.
struct HalfChunk {
  static constexpr int N = 4;
  float v[N];
  __device__ inline void load(const void* base, int64_t elem) {
    const uint2 u = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(base) + elem);
    v[0] = __uint_as_float(u.x << 16);
    v[1] = __uint_as_float(u.x & 0xffff0000u);
    v[2] = __uint_as_float(u.y << 16);
    v[3] = __uint_as_float(u.y & 0xffff0000u);
  }
};

// The same chunk as loaded, widened when it is used.
template <bool BF16> struct Raw {
  uint4 u;
  __device__ inline void load(const void* base, int64_t elem) {
    u = *reinterpret_cast<const uint4*>(static_cast<const char*>(base) + elem * (BF16 ? 2 : 4));
  }
  __device__ inline void widen(Chunk<BF16>& c) const {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (BF16) {
        c.v[2 * i] = __uint_as_float(w[i] << 16);
        c.v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
      } else {
        c.v[i] = __uint_as_float(w[i]);
      }
    }
  }
};

// Splat (Eq. splat) as a gather over the point lists J_v, which are stored
// back to back (entries grouped by vertex).  The entry array is cut into
// chunks of `chunk` entries and each chunk goes to one lane group, so the
// work is balanced however skewed the vertex degrees are (a LiDAR vertex next
// to the sensor can hold thousands of points).  A vertex whose list lies
// inside one chunk is finished there.  A vertex cut by chunk boundaries
// leaves pieces: a head piece in a chunk it continues into, a tail piece in
// the chunk where it starts.  The G = kBlock/LPR consecutive chunks of a
// workgroup (its span) put their pieces in LDS and the workgroup joins them
// in chunk order: a vertex that starts and ends in the span is finished
// there; the piece of the vertex the span starts inside and the piece of the
// vertex that runs past its end go to global memory as the span's head and
// tail partials, which k_splat_finish adds in span order.  No float
// atomics; the summation order is fixed.
template <bool BF16, int LPR, int Q>
__device__ inline void splat_store(int32_t v, const float (&acc)[Q][Chunk<BF16>::N], float ws, int lane,
                                   int nchunk, int normalize, void* vals, int64_t ld_vals, float* wsum) {
  using Ch = Chunk<BF16>;
  const float scale = normalize ? (ws > 0.f ? 1.0f / ws : 0.f) : 1.0f;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int ch = lane + q * LPR;
    if (ch < nchunk) {
      Ch o;
#pragma unroll
      for (int i = 0; i < Ch::N; ++i) o.v[i] = acc[q][i] * scale;
      o.store(vals, static_cast<int64_t>(v) * ld_vals + static_cast<int64_t>(ch) * Ch::N);
    }
  }
  if (wsum && lane == 0) wsum[v] = ws;
}

// row c of a C-wide partial array (global or LDS) and its weight
template <bool BF16, int LPR, int Q>
__device__ inline void splat_partial(float* part, float* part_w, int64_t c, int slot,
                                     const float (&acc)[Q][Chunk<BF16>::N], float ws, int lane, int C) {
  using Ch = Chunk<BF16>;
  const int nchunk = C / Ch::N;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int ch = lane + q * LPR;
    if (ch < nchunk) {
      float* dst = part + c * C + static_cast<int64_t>(ch) * Ch::N;
#pragma unroll
      for (int i = 0; i < Ch::N; i += 4)
        *reinterpret_cast<float4*>(dst + i) = make_float4(acc[q][i], acc[q][i + 1], acc[q][i + 2], acc[q][i + 3]);
    }
  }
  if (lane == 0) part_w[2 * c + slot] = ws;
}

template <bool BF16, int LPR, int Q>
__device__ inline void splat_add(float (&acc)[Q][Chunk<BF16>::N], const float* part, int64_t c, int lane, int C) {
  using Ch = Chunk<BF16>;
  const int nchunk = C / Ch::N;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int ch = lane + q * LPR;
    if (ch < nchunk) {
      const float* src = part + c * C + static_cast<int64_t>(ch) * Ch::N;
#pragma unroll
      for (int i = 0; i < Ch::N; i += 4) {
        const float4 x = *reinterpret_cast<const float4*>(src + i);
        acc[q][i] += x.x;
        acc[q][i + 1] += x.y;
        acc[q][i + 2] += x.z;
        acc[q][i + 3] += x.w;
      }
    }
  }
}

// What a list entry e = 4p + k adds to its vertex's row.  The splat adds
// w_e f_p (and w_e to the weight sum).
template <bool BF16, int LPR, int Q, int B>
struct WeightedRows {
  using Ch = Chunk<BF16>;
  const float* entry_w;
  const void* feat;
  int64_t ld_feat;
  struct Batch {
    float wt[B];
    Ch f[B][Q];
  };
  static constexpr bool kGivenWeights = true;   // the kernel may load entry_w itself
  __device__ inline void init(int, int) {}
  __device__ inline void load_given(Batch& bt, int j, float w, int32_t e, bool in, int lane, int nchunk) const {
    bt.wt[j] = in ? w : 0.f;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int ch = lane + q * LPR;
      if (in && ch < nchunk)
        bt.f[j][q].load(feat, static_cast<int64_t>(e >> 2) * ld_feat + static_cast<int64_t>(ch) * Ch::N);
      else
#pragma unroll
        for (int i = 0; i < Ch::N; ++i) bt.f[j][q].v[i] = 0.f;
    }
  }
  __device__ inline void load(Batch& bt, int j, int64_t s, int32_t e, bool in, int lane, int nchunk) const {
    bt.wt[j] = in ? entry_w[s] : 0.f;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int ch = lane + q * LPR;
      if (in && ch < nchunk)
        bt.f[j][q].load(feat, static_cast<int64_t>(e >> 2) * ld_feat + static_cast<int64_t>(ch) * Ch::N);
      else
#pragma unroll
        for (int i = 0; i < Ch::N; ++i) bt.f[j][q].v[i] = 0.f;
    }
  }
  __device__ inline float add(const Batch& bt, int j, float (&acc)[Q][Ch::N]) const {
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int i = 0; i < Ch::N; ++i) acc[q][i] += bt.wt[j] * bt.f[j][q].v[i];
    return bt.wt[j];
  }
};

// DeformSlice backward, what entry e = (p, k) adds to dL/dx of its vertex:
//   alpha_e g_p + wv * (beta_e - [argmax_c(p) = k] gamma_e)
// with coef[e] = (alpha_e, beta_e, gamma_e, 0) and am[p][c] the vertex slot
// holding channel c's maximum (fp32 only).
template <int LPR, int Q, int B>
struct DeformGradRows {
  using Ch = Chunk<false>;
  static constexpr bool kGivenWeights = false;
  const float* g;
  int64_t ld_g;
  const float4* coef;
  const uint8_t* am;
  const float* wv;
  int C;
  float wvc[Q][4];
  struct Batch {
    float4 cf[B];
    int k[B];
    Ch f[B][Q];
    uint32_t m[B][Q];
  };
  __device__ inline void init(int lane, int nchunk) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int ch = lane + q * LPR;
#pragma unroll
      for (int i = 0; i < 4; ++i) wvc[q][i] = ch < nchunk ? wv[4 * ch + i] : 0.f;
    }
  }
  __device__ inline void load(Batch& bt, int j, int64_t, int32_t e, bool in, int lane, int nchunk) const {
    bt.cf[j] = in ? coef[e] : make_float4(0.f, 0.f, 0.f, 0.f);
    bt.k[j] = e & 3;
    const int64_t p = e >> 2;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int ch = lane + q * LPR;
      if (in && ch < nchunk) {
        bt.f[j][q].load(g, p * ld_g + 4 * ch);
        bt.m[j][q] = *reinterpret_cast<const uint32_t*>(am + p * C + 4 * ch);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) bt.f[j][q].v[i] = 0.f;
        bt.m[j][q] = 0xffffffffu;
      }
    }
  }
  __device__ inline float add(const Batch& bt, int j, float (&acc)[Q][4]) const {
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool mx = ((bt.m[j][q] >> (8 * i)) & 0xffu) == static_cast<uint32_t>(bt.k[j]);
        acc[q][i] += bt.cf[j].x * bt.f[j][q].v[i] + wvc[q][i] * (bt.cf[j].y - (mx ? bt.cf[j].z : 0.f));
      }
    return 0.f;
  }
};

// LDS of k_splat_chunks: head and tail pieces of the G chunks, their weights
// and flags.
inline size_t splat_lds_bytes(int lpr, int C) {
  const int G = 256 / lpr;
  return sizeof(float) * (2 * static_cast<size_t>(G) * C + 2 * G) + sizeof(int32_t) * G;
}

template <bool BF16, int LPR, int Q, int B, class Rows>
__global__ void __launch_bounds__(kBlock)
k_splat_chunks(const int32_t* __restrict__ offsets, const int32_t* __restrict__ entries, Rows rows,
               const int32_t* __restrict__ chunk_first, int chunk, int64_t n, int64_t total, int C, int normalize,
               void* __restrict__ vals, int64_t ld_vals, float* __restrict__ wsum,
               float* __restrict__ part_head, float* __restrict__ part_tail, float* __restrict__ part_w,
               unsigned nblk) {
  using Ch = Chunk<BF16>;
  constexpr int G = kBlock / LPR;
  extern __shared__ __align__(16) float sm[];
  float* sh_head = sm;                 // [G][C]
  float* sh_tail = sm + G * C;         // [G][C]
  float* sh_w = sm + 2 * G * C;        // [G][2]
  int32_t* sh_flag = reinterpret_cast<int32_t*>(sh_w + 2 * G);  // bit 0 head piece, bit 1 tail piece
  const int lane = threadIdx.x & (LPR - 1);
  const int g = threadIdx.x / LPR;
  // XCD-contiguous span order (see xcd_item)
  const unsigned b = blockIdx.x;
  const int64_t span = static_cast<int64_t>(b % 8) * ((nblk + 7) / 8) + b / 8;
  const int64_t c0 = span * G;
  if (c0 * chunk >= total) return;     // whole workgroup
  const int64_t c = c0 + g;
  const int64_t s0 = c * chunk;
  const int64_t s1 = min(s0 + static_cast<int64_t>(chunk), total);
  const int64_t span_end = min((c0 + G) * static_cast<int64_t>(chunk), total);
  const int nchunk = C / Ch::N;
  rows.init(lane, nchunk);
  if (lane == 0) sh_flag[g] = 0;
  int32_t tail_v = -1, tail_ve = 0;    // vertex of this chunk's tail piece
  int32_t head_ve = 0;                 // end of the vertex the chunk starts inside
  if (s0 < total) {
    int32_t v = chunk_first[c];
    // window of list ends for the next LPR vertices
    int32_t v_win = v;
    int32_t win = offsets[min(static_cast<int64_t>(v) + 1 + lane, n)];
    int32_t vb = offsets[v];
    int32_t ve = __shfl(win, 0, LPR);
    head_ve = ve;
    float acc[Q][Ch::N];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int i = 0; i < Ch::N; ++i) acc[q][i] = 0.f;
    float ws = 0.f;
    // what entry s (and the batch slot j it sits in) adds: the vertex's
    // running sum, and at the vertex's last entry (or the chunk's) its row or
    // piece
    auto consume = [&](const typename Rows::Batch& bt, int j, int64_t s) {
      ws += rows.add(bt, j, acc);
      const int64_t nxt = s + 1;
      if (nxt == ve || nxt == s1) {
        if (vb >= s0 && ve <= s1) {
          splat_store<BF16, LPR, Q>(v, acc, ws, lane, nchunk, normalize, vals, ld_vals, wsum);
        } else if (vb < s0) {
          splat_partial<BF16, LPR, Q>(sh_head, sh_w, g, 0, acc, ws, lane, C);
          if (lane == 0) sh_flag[g] |= 1;
        } else {
          splat_partial<BF16, LPR, Q>(sh_tail, sh_w, g, 1, acc, ws, lane, C);
          if (lane == 0) sh_flag[g] |= 2;
          tail_v = v;
          tail_ve = ve;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int i = 0; i < Ch::N; ++i) acc[q][i] = 0.f;
        ws = 0.f;
        if (nxt == ve && nxt < s1) {
          v += 1;
          vb = ve;
          if (v - v_win >= LPR) {
            v_win = v;
            win = offsets[min(static_cast<int64_t>(v) + 1 + lane, n)];
          }
          ve = __shfl(win, v - v_win, LPR);
        }
      }
    };
    if constexpr ((LPR == 16 || LPR == 8) && Rows::kGivenWeights) {
      // LPR entries at a time: lane i loads the index and weight of entry i,
      // and a broadcast inside the lane group (DPP or swizzle) hands entry
      // j's to the whole group; the next LPR are loaded while this round's
      // rows arrive
      int32_t E = s0 + lane < s1 ? entries[s0 + lane] : 0;
      float Wt = s0 + lane < s1 ? rows.entry_w[s0 + lane] : 0.f;
      for (int64_t sb = s0; sb < s1; sb += LPR) {
        const int64_t nx = sb + LPR + lane;
        const int32_t En = nx < s1 ? entries[nx] : 0;
        const float Wn = nx < s1 ? rows.entry_w[nx] : 0.f;
        static_for<LPR / B>([&](auto h_c) {
          constexpr int J0 = decltype(h_c)::value * B;
          if (sb + J0 < s1) {
            typename Rows::Batch bt;
            static_for<B>([&](auto j_c) {
              constexpr int J = decltype(j_c)::value;
              const int32_t e = group_bcast<LPR, J0 + J>(E);
              const float w = __int_as_float(group_bcast<LPR, J0 + J>(__float_as_int(Wt)));
              rows.load_given(bt, J, w, e, sb + J0 + J < s1, lane, nchunk);
            });
#pragma unroll
            for (int j = 0; j < B; ++j) {
              if (sb + J0 + j >= s1) break;
              consume(bt, j, sb + J0 + j);
            }
          }
        });
        E = En;
        Wt = Wn;
      }
    } else {
      // the entries of the next batch are loaded while this batch's rows
      // arrive and are added
      int32_t e[B];
#pragma unroll
      for (int j = 0; j < B; ++j) e[j] = s0 + j < s1 ? entries[s0 + j] : 0;
      for (int64_t s = s0; s < s1; s += B) {
        typename Rows::Batch bt;
#pragma unroll
        for (int j = 0; j < B; ++j) rows.load(bt, j, s + j, e[j], s + j < s1, lane, nchunk);
#pragma unroll
        for (int j = 0; j < B; ++j) e[j] = s + B + j < s1 ? entries[s + B + j] : 0;
#pragma unroll
        for (int j = 0; j < B; ++j) {
          if (s + j >= s1) break;
          consume(bt, j, s + j);
        }
      }
    }
  }
  __syncthreads();
  // join the pieces of the span in chunk order
  float acc[Q][Ch::N];
  if (tail_v >= 0) {
    // vertex starting in chunk g: its tail piece, then the head pieces of the
    // following chunks it runs into
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int i = 0; i < Ch::N; ++i) acc[q][i] = 0.f;
    splat_add<BF16, LPR, Q>(acc, sh_tail, g, lane, C);
    float ws = sh_w[2 * g + 1];
    for (int g2 = g + 1; g2 < G && (c0 + g2) * chunk < tail_ve; ++g2) {
      splat_add<BF16, LPR, Q>(acc, sh_head, g2, lane, C);
      ws += sh_w[2 * g2];
    }
    if (tail_ve <= span_end)
      splat_store<BF16, LPR, Q>(tail_v, acc, ws, lane, nchunk, normalize, vals, ld_vals, wsum);
    else
      splat_partial<BF16, LPR, Q>(part_tail, part_w, span, 1, acc, ws, lane, C);
  }
  if (g == 0 && (sh_flag[0] & 1)) {
    // the vertex the span starts inside: head pieces of the chunks it covers
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int i = 0; i < Ch::N; ++i) acc[q][i] = 0.f;
    float ws = 0.f;
    for (int g2 = 0; g2 < G && (c0 + g2) * chunk < head_ve; ++g2) {
      splat_add<BF16, LPR, Q>(acc, sh_head, g2, lane, C);
      ws += sh_w[2 * g2];
    }
    splat_partial<BF16, LPR, Q>(part_head, part_w, span, 0, acc, ws, lane, C);
  }
}

// Vertices cut by span boundaries: the span in which a vertex's list starts
// adds its tail partial and the head partials of the following spans.
template <bool BF16, int LPR, int Q>
__global__ void __launch_bounds__(kBlock)
k_splat_finish(const int32_t* __restrict__ offsets, const int32_t* __restrict__ chunk_first, int64_t span_len,
               int chunks_per_span, int64_t nspans, int C, int normalize, void* __restrict__ vals, int64_t ld_vals,
               float* __restrict__ wsum, const float* __restrict__ part_head, const float* __restrict__ part_tail,
               const float* __restrict__ part_w) {
  using Ch = Chunk<BF16>;
  const int lane = threadIdx.x & (LPR - 1);
  const int64_t c = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) / LPR;
  if (c + 1 >= nspans) return;
  const int64_t s0 = c * span_len, s1 = s0 + span_len;
  const int32_t v = chunk_first[(c + 1) * chunks_per_span];
  const int32_t vb = offsets[v];
  if (!(vb < s1 && vb >= s0)) return;
  const int32_t ve = offsets[v + 1];
  const int64_t last = (static_cast<int64_t>(ve) - 1) / span_len;
  const int nchunk = C / Ch::N;
  float acc[Q][Ch::N];
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int i = 0; i < Ch::N; ++i) acc[q][i] = 0.f;
  splat_add<BF16, LPR, Q>(acc, part_tail, c, lane, C);
  float ws = part_w[2 * c + 1];
#pragma unroll 8
  for (int64_t c2 = c + 1; c2 <= last; ++c2) {
    splat_add<BF16, LPR, Q>(acc, part_head, c2, lane, C);
    ws += part_w[2 * c2];
  }
  splat_store<BF16, LPR, Q>(v, acc, ws, lane, nchunk, normalize, vals, ld_vals, wsum);
}

// Slice (Eq. slice): out_p = sum_k b_pk x_{idx_pk}.  A lane group takes two
// consecutive points and issues the loads of both before using them (twice
// the bytes in flight per lane).  A vertex slot without a vertex (a lattice
// the build flagged) reads row 0 with weight 0, so that the loads are issued
// without branches.
// SCALED: every vertex row is taken times vscale[vertex], which is folded into
// the weights (the gradient of a normalised splat).
// Ch: a lane's channels of a row.
template <class Ch, int LPR, bool SCALED>
__global__ void __launch_bounds__(kBlock)
k_slice(const int4* __restrict__ idx, const float4* __restrict__ w, int64_t m,
        const void* __restrict__ vals, int64_t ld_vals, int C, float* __restrict__ out,
        const float* __restrict__ vscale, unsigned nblk) {
  constexpr int PP = 2;
  const int lane = threadIdx.x & (LPR - 1);
  const int64_t p0 = PP * xcd_item<LPR>(nblk);
  if (p0 >= m) return;
  int32_t vi[PP][4];
  float bw[PP][4];
#pragma unroll
  for (int u = 0; u < PP; ++u) {
    const int64_t p = min(p0 + u, m - 1);
    const int4 iv = idx[p];
    const float4 wv = w[p];
    vi[u][0] = max(iv.x, 0); vi[u][1] = max(iv.y, 0); vi[u][2] = max(iv.z, 0); vi[u][3] = max(iv.w, 0);
    bw[u][0] = iv.x < 0 ? 0.f : wv.x;
    bw[u][1] = iv.y < 0 ? 0.f : wv.y;
    bw[u][2] = iv.z < 0 ? 0.f : wv.z;
    bw[u][3] = iv.w < 0 ? 0.f : wv.w;
    if constexpr (SCALED) {
#pragma unroll
      for (int k = 0; k < 4; ++k) bw[u][k] *= vscale[vi[u][k]];
    }
  }
  const int nchunk = C / Ch::N;
  for (int ch = lane; ch < nchunk; ch += LPR) {
    Ch x[PP][4];
#pragma unroll
    for (int u = 0; u < PP; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        x[u][k].load(vals, static_cast<int64_t>(vi[u][k]) * ld_vals + static_cast<int64_t>(ch) * Ch::N);
#pragma unroll
    for (int u = 0; u < PP; ++u) {
      if (p0 + u >= m) break;
      float acc[Ch::N];
#pragma unroll
      for (int i = 0; i < Ch::N; ++i) acc[i] = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < Ch::N; ++i) acc[i] += bw[u][k] * x[u][k].v[i];
      float* o = out + (p0 + u) * C + static_cast<int64_t>(ch) * Ch::N;
#pragma unroll
      for (int i = 0; i < Ch::N; i += 4)
        store_row4<Ch::N == 4>(o + i, acc[i], acc[i + 1], acc[i + 2], acc[i + 3]);
    }
  }
}

// Slice of wide rows: a wave takes whole points, PP consecutive ones, a lane V
// consecutive channels of each.  Indices, weights and row addresses are then the
// same for the wave and are read and computed by the scalar unit.  What bounds
// the slice of wide rows is the sum of its vector operations, its gathers through
// the L1 (195 us alone for 1M points of 256 bf16 channels) and its stores (220 us
// alone); this takes the addresses and the weights' selects off the vector unit
// and stores whole lines: 446 us with lane groups, 361 here.  More points a
// wave, a loop over points and other orders of the blocks made no difference.
// Lane groups (k_slice) take
//   fp32 rows up to 128 channels, whose 16-byte stores a wave would halve (128
//     channels of 120k points: 15 us, a wave per point 20; 72 channels of 1M: 189
//     and 219; 136 channels of 120k: 25 and 20);
//   bf16 rows of 65 to 128 channels up to kSliceWideM128 points, 4 channels a
//     lane (120k points of 128 channels: 14.5 us, a wave per point 18, 8 channels
//     a lane 27; 200k points 46, 42 and 48, but 25, 29 and 26 with rows that the
//     caches hold);
//   clouds up to kSliceWideM points, which would have too few waves (1,024
//     channels of 2,000 points: 4.8 us and 6.2).
template <bool BF16, int V, bool SCALED>
__global__ void __launch_bounds__(kBlock)
k_slice_wide(const int4* __restrict__ idx, const float4* __restrict__ w, int64_t m,
             const void* __restrict__ vals, int64_t ld_vals, int C, float* __restrict__ out,
             const float* __restrict__ vscale, unsigned nblk) {
  constexpr int PP = BF16 ? 4 : 2;
  typedef float OutV __attribute__((ext_vector_type(V)));
  using Raw = typename std::conditional<BF16, typename std::conditional<V == 4, uint2, uint32_t>::type, OutV>::type;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const unsigned per = (nblk + 7) / 8;
  const int64_t block = static_cast<int64_t>(blockIdx.x % 8) * per + blockIdx.x / 8;   // as xcd_item
  const int64_t p0 = PP * (block * (kBlock / 64) + wave);
  if (p0 >= m) return;
  int64_t row[PP][4];
  float bw[PP][4];
#pragma unroll
  for (int u = 0; u < PP; ++u) {
    const int64_t p = min(p0 + u, m - 1);
    const int4 iv = idx[p];
    const float4 wv = w[p];
    const int32_t v[4] = {iv.x, iv.y, iv.z, iv.w};
    const float b[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {   // (a slot without a vertex: row 0 with weight 0)
      row[u][k] = max(v[k], 0) * ld_vals;
      bw[u][k] = v[k] < 0 ? 0.f : b[k];
      if constexpr (SCALED) bw[u][k] *= vscale[max(v[k], 0)];
    }
  }
  using E = typename std::conditional<BF16, uint16_t, float>::type;
  for (int ch = V * lane; ch < C; ch += 64 * V) {
    Raw x[PP][4];
#pragma unroll
    for (int u = 0; u < PP; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) x[u][k] = *reinterpret_cast<const Raw*>(static_cast<const E*>(vals) + row[u][k] + ch);
#pragma unroll
    for (int u = 0; u < PP; ++u) {
      if (p0 + u >= m) break;
      OutV acc = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if constexpr (BF16) {
          uint32_t q[2];
          if constexpr (V == 4) { q[0] = x[u][k].x; q[1] = x[u][k].y; }
          else q[0] = x[u][k];
#pragma unroll
          for (int i = 0; i < V; i += 2) {
            acc[i] += bw[u][k] * __uint_as_float(q[i / 2] << 16);
            acc[i + 1] += bw[u][k] * __uint_as_float(q[i / 2] & 0xffff0000u);
          }
        } else {
#pragma unroll
          for (int i = 0; i < V; ++i) acc[i] += bw[u][k] * x[u][k][i];
        }
      }
      __builtin_nontemporal_store(acc, reinterpret_cast<OutV*>(out + (p0 + u) * C + ch));
    }
  }
}

// DeformSlice (Eq. deformSlice): q_k = b_k x_k; M = max_k q_k per channel;
// db_k = tanh(beta + (q_k - M) . wv); out = sum_k (b_k + db_k) x_k.
// Each lane keeps its channels of the d+1 gathered rows in registers; the
// dot products are reduced across the lane group with xor shuffles.
template <bool BF16, int LPR, int CPL>
__global__ void __launch_bounds__(kBlock)
k_deform_slice(const int4* __restrict__ idx, const float4* __restrict__ w, int64_t m,
               const void* __restrict__ vals, int64_t ld_vals, int C, const float* __restrict__ wvec,
               float beta, float* __restrict__ out, float4* __restrict__ delta, float* __restrict__ plain,
               unsigned nblk) {
  using Ch = Chunk<BF16>;
  const int lane = threadIdx.x & (LPR - 1);
  const int64_t p = xcd_item<LPR>(nblk);
  const bool live = p < m;
  const int nchunk = C / Ch::N;
  int4 iv = make_int4(-1, -1, -1, -1);
  float4 wq = make_float4(0.f, 0.f, 0.f, 0.f);
  if (live) { iv = idx[p]; wq = w[p]; }
  const int32_t vi[4] = {iv.x, iv.y, iv.z, iv.w};
  const float bw[4] = {wq.x, wq.y, wq.z, wq.w};
  float x[CPL][4][Ch::N];
  float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const int ch = lane + q * LPR;
    const bool on = live && ch < nchunk;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (on && vi[k] >= 0) {
        Ch c;
        c.load(vals, static_cast<int64_t>(vi[k]) * ld_vals + static_cast<int64_t>(ch) * Ch::N);
#pragma unroll
        for (int i = 0; i < Ch::N; ++i) x[q][k][i] = c.v[i];
      } else {
#pragma unroll
        for (int i = 0; i < Ch::N; ++i) x[q][k][i] = 0.f;
      }
    }
    if (on) {
#pragma unroll
      for (int i = 0; i < Ch::N; ++i) {
        const float wc = wvec[ch * Ch::N + i];
        float qk[4];
        float mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          qk[k] = bw[k] * x[q][k][i];
          mx = fmaxf(mx, qk[k]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) part[k] += (qk[k] - mx) * wc;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) part[k] = group_sum<LPR>(part[k]);
  if (!live) return;
  float coef[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float db = tanhf(beta + part[k]);
    part[k] = db;
    coef[k] = bw[k] + db;
  }
  if (delta && lane == 0) delta[p] = make_float4(part[0], part[1], part[2], part[3]);
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const int ch = lane + q * LPR;
    if (ch >= nchunk) continue;
    float* o = out + p * C + static_cast<int64_t>(ch) * Ch::N;
#pragma unroll
    for (int i = 0; i < Ch::N; i += 4) {
      float r[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        r[u] = coef[0] * x[q][0][i + u] + coef[1] * x[q][1][i + u] + coef[2] * x[q][2][i + u] +
               coef[3] * x[q][3][i + u];
      store_row4<Ch::N == 4>(o + i, r[0], r[1], r[2], r[3]);
    }
    if (plain) {
      // the plain slice of the same rows (Eq. slice), in the order of k_slice
      float* o2 = plain + p * C + static_cast<int64_t>(ch) * Ch::N;
#pragma unroll
      for (int i = 0; i < Ch::N; i += 4) {
        float r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float a = 0.f;
#pragma unroll
          for (int k = 0; k < 4; ++k) a += bw[k] * x[q][k][i + u];
          r[u] = a;
        }
        store_row4<Ch::N == 4>(o2 + i, r[0], r[1], r[2], r[3]);
      }
    }
  }
}

// DeformSlice fused with the last linear classification layer
// (Implementation): logits = Wc f + bc for the DeformSlice rows f, which are
// never stored.  The classes run on v_mfma_f32_16x16x4_f32 with Wc (LDS, in
// fragment order) as one operand and f as the other; lane (i, g) of the product
// receives the classes 4 g .. 4 g + 3 of point i, per 16 classes.
// What bounds it are the vector operations on the gathered values (22 per
// channel of a point); with every lane reading all K weight rows of its
// channels from LDS and the K partial sums exchanged over the row's lanes, the
// classes cost more than that: C = 128, 20 classes, 1M points bf16 took 532 us
// and 120k points fp32 75 us, and 218 and 42 us here (with every lane keeping 8
// channels of the four rows of one of 16 points, and no tile, 250: a wave per SIMD).
typedef float f32x4_v __attribute__((ext_vector_type(4)));

// Wc in LDS: [block of 16 channels][nb][lane][4], the class 16 nb + i and the
// channel 4 g + e of the block in lane (i, g)
__device__ inline void stage_classifier(float* wl, const float* __restrict__ Wc, int K, int C, int blocks, int NB) {
  for (int i = threadIdx.x; i < blocks * NB * 256; i += kBlock) {
    const int e = i & 3, L = (i >> 2) & 63, run = i >> 8;
    const int nb = run % NB, cb = run / NB;
    const int cls = 16 * nb + (L & 15), ch = 16 * cb + 4 * (L >> 4) + e;
    wl[i] = cls < K && ch < C ? Wc[cls * C + ch] : 0.f;
  }
}

// Sums over the channels in short chains (a single chain through the products
// doubles the rounding error): four chains, one per channel of a lane's four,
// over kClassifyRun blocks of 16 channels make a run; where there are more than
// two runs, two are added before they go to the total.  (Relative error against
// 64 bits at 128 and 256 fp32 channels 1.07e-7 and 1.09e-7, with runs added to the
// total one by one 1.08e-7 and 1.12e-7, by lane groups 1.05e-7 and 1.06e-7.  The
// wide rows below add them one by one: pairs cost 10 to 50% there.)
constexpr int kClassifyRun = 2;
constexpr int kOffsetRun = 4;
template <int NB>
struct ClassSums {
  f32x4_v run[4][NB], total[NB];
  __device__ ClassSums() {
    clear();
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) total[nb] = f32x4_v{0.f, 0.f, 0.f, 0.f};
  }
  __device__ inline void clear() {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) run[e][nb] = f32x4_v{0.f, 0.f, 0.f, 0.f};
  }
  __device__ inline void add(const f32x4_v (&w)[NB], int e, float f) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) run[e][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[nb][e], f, run[e][nb], 0, 0, 0);
  }
  // the run's sum, and on to the next run
  __device__ inline void take(f32x4_v (&t)[NB]) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) t[nb] = (run[0][nb] + run[1][nb]) + (run[2][nb] + run[3][nb]);
    clear();
  }
  __device__ inline void flush() {
    f32x4_v t[NB];
    take(t);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) total[nb] += t[nb];
  }
  __device__ inline void flush(const f32x4_v (&before)[NB]) {
    f32x4_v t[NB];
    take(t);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) total[nb] += before[nb] + t[nb];
  }
};

// the lane's 4 classes of point p
template <int NB>
__device__ inline void store_classes(float* __restrict__ out, int64_t p, int K, int lg, int vec_out,
                                     const f32x4_v (&acc)[NB]) {
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int j = 16 * nb + 4 * lg;
    float* o = out + p * K + j;
    if (vec_out) {
      if (j < K) *reinterpret_cast<f32x4_v*>(o) = acc[nb];
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (j + r < K) o[r] = acc[nb][r];
    }
  }
}

// Rows of at most kClassifyTileC channels: a point's row is gathered by LPR
// lanes as in k_deform_slice (whole rows a load), TP points (at least 16) in
// turn, and f goes through a tile in LDS into the product's operand layout.
// Every load is issued, from a valid address (a condition would make branches
// of the loads, each waiting for all in flight): a vertex slot without a vertex
// (a lattice the build flagged) reads row 0 with weight and coefficient 0,
// lanes past C zeros in place of a row (the row's last channels against zeros in
// wvec and Wc would make NaN of an infinite value, and selects on the loaded
// values took 9% at 160 to 224 fp32 channels).
__device__ const uint4 kNoChannels = {0u, 0u, 0u, 0u};
template <bool BF16, int LPR, int CPL, int NB>
__global__ void __launch_bounds__(kBlock)
k_deform_classify(const int4* __restrict__ idx, const float4* __restrict__ w, int64_t m,
                  const void* __restrict__ vals, int64_t ld_vals, int C, const float* __restrict__ wvec, float beta,
                  const float* __restrict__ Wc, const float* __restrict__ bc, int K, float* __restrict__ out,
                  int vec_out, unsigned nblk) {
  using Ch = Chunk<BF16>;
  constexpr int EPL = Ch::N;
  constexpr int PPS = 64 / LPR;                 // points per step
  constexpr int TP = PPS > 16 ? PPS : 16;       // points per tile
  constexpr int CW = LPR * CPL * EPL;           // channels of a tile, zero-padded
  constexpr int PITCH = CW + 4;
  constexpr int BLK = (CW + 15) / 16;
  extern __shared__ __align__(16) float wl[];   // Wc, then the waves' tiles [TP][PITCH]
  stage_classifier(wl, Wc, K, C, BLK, NB);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int pl = lane / LPR, cl = lane & (LPR - 1);   // point of a step, lane of its row
  float* T = wl + BLK * NB * 256 + wave * TP * PITCH;
  float wv[CPL][EPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q)
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const int ch = (cl + q * LPR) * EPL + i;
      wv[q][i] = ch < C ? wvec[ch] : 0.f;
    }
  f32x4_v bias[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = 16 * nb + 4 * lg + r;
      bias[nb][r] = bc && j < K ? bc[j] : 0.f;
    }
  __syncthreads();
  // The weights are staged once per workgroup, which then walks a
  // contiguous range of the nblk groups of 4 TP points (each XCD a contiguous
  // share of the ranges, as xcd_item).
  const unsigned G = gridDim.x;   // a multiple of 8
  const unsigned rg = (blockIdx.x % 8) * (G / 8) + blockIdx.x / 8;
  const unsigned per = (nblk + G - 1) / G;
  const unsigned lb1 = min((rg + 1) * per, nblk);
  // Steps are pipelined over the tiles: while one is computed, the rows of the
  // next are on their way and the vertices of the one after it.
  constexpr int STEPS = TP / PPS;
  const unsigned lb0 = rg * per;
  auto point = [&](unsigned step) {
    const int64_t tile = static_cast<int64_t>(lb0 + step / STEPS) * 4 + wave;
    return min(tile * TP + static_cast<int64_t>(step % STEPS) * PPS + pl, m - 1);
  };
  Raw<BF16> xn[CPL][4];
  // the lane's channels of row 0, and the rows' distance (0 where the lane is past C)
  const void* base[CPL];
  int64_t ld[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const int ch = (cl + q * LPR) * EPL;
    const bool on = (!BF16 && LPR == 8 && CPL == 2) || ch < C;   // (two chunks a lane: 64 channels, all lanes)
    base[q] = on ? static_cast<const char*>(vals) + ch * (BF16 ? 2 : 4) : static_cast<const void*>(&kNoChannels);
    ld[q] = on ? ld_vals : 0;
  }
  auto gather = [&](const int4& v) {
    const int32_t vi[4] = {max(v.x, 0), max(v.y, 0), max(v.z, 0), max(v.w, 0)};
#pragma unroll
    for (int q = 0; q < CPL; ++q)
#pragma unroll
      for (int k = 0; k < 4; ++k) xn[q][k].load(base[q], static_cast<int64_t>(vi[k]) * ld[q]);
  };
  int4 iv = idx[point(0)], iv_next = idx[point(1)];
  float4 wq = w[point(0)], wq_next = w[point(1)];
  if (lb0 < lb1) gather(iv);
  unsigned step = 0;
  for (unsigned lb = lb0; lb < lb1; ++lb) {
    const int64_t p0 = (static_cast<int64_t>(lb) * 4 + wave) * TP;
#pragma unroll 1
    for (int st = 0; st < STEPS; ++st, ++step) {
      const bool have[4] = {iv.x >= 0, iv.y >= 0, iv.z >= 0, iv.w >= 0};
      const float bw[4] = {have[0] ? wq.x : 0.f, have[1] ? wq.y : 0.f, have[2] ? wq.z : 0.f, have[3] ? wq.w : 0.f};
      Ch x[CPL][4];
#pragma unroll
      for (int q = 0; q < CPL; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) xn[q][k].widen(x[q][k]);
      iv = iv_next;
      wq = wq_next;
      gather(iv);
      iv_next = idx[point(step + 2)];
      wq_next = w[point(step + 2)];
      float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < CPL; ++q)
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          float qk[4];
          float mx = -INFINITY;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            qk[k] = bw[k] * x[q][k].v[i];
            mx = fmaxf(mx, qk[k]);
          }
#pragma unroll
          for (int k = 0; k < 4; ++k) part[k] += (qk[k] - mx) * wv[q][i];
        }
#pragma unroll
      for (int k = 0; k < 4; ++k) part[k] = group_sum<LPR>(part[k]);
      float coef[4];
      if constexpr (LPR >= 4) {
        // lane 4 j + k of the row takes the k-th offset, the quad exchanges them
        const int k = lane & 3;
        const float mine = tanhf(beta + (k == 0 ? part[0] : (k == 1 ? part[1] : (k == 2 ? part[2] : part[3]))));
        const int x4 = __float_as_int(mine);
        coef[0] = __int_as_float(__builtin_amdgcn_update_dpp(0, x4, 0x00, 0xF, 0xF, false));
        coef[1] = __int_as_float(__builtin_amdgcn_update_dpp(0, x4, 0x55, 0xF, 0xF, false));
        coef[2] = __int_as_float(__builtin_amdgcn_update_dpp(0, x4, 0xAA, 0xF, 0xF, false));
        coef[3] = __int_as_float(__builtin_amdgcn_update_dpp(0, x4, 0xFF, 0xF, 0xF, false));
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) coef[k] = tanhf(beta + part[k]);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) coef[k] = have[k] ? bw[k] + coef[k] : 0.f;
      float* row = T + (st * PPS + pl) * PITCH;
#pragma unroll
      for (int q = 0; q < CPL; ++q)
#pragma unroll
        for (int i = 0; i < EPL; i += 4) {
          f32x4_v f;
#pragma unroll
          for (int u = 0; u < 4; ++u)
            f[u] = coef[0] * x[q][0].v[i + u] + coef[1] * x[q][1].v[i + u] + coef[2] * x[q][2].v[i + u] +
                   coef[3] * x[q][3].v[i + u];
          *reinterpret_cast<f32x4_v*>(row + (cl + q * LPR) * EPL + i) = f;
        }
    }
    // a wave's LDS accesses take effect in order; the fences keep the compiler
    // from moving the reads above the writes, and the next tile's writes above
    // the reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int mg = 0; mg < TP / 16; ++mg) {
      ClassSums<NB> sums;
      const float* f = T + (mg * 16 + li) * PITCH + 4 * lg;
      const f32x4_v* wf = reinterpret_cast<const f32x4_v*>(wl) + lane;
      auto add_run = [&](int c0) {
#pragma unroll
        for (int cb = c0; cb < c0 + kClassifyRun; ++cb) {
          if (BLK % kClassifyRun != 0 && cb >= BLK) break;
          f32x4_v x = {0.f, 0.f, 0.f, 0.f};
          if (CW % 16 == 0 || 16 * cb + 4 * lg < CW) x = *reinterpret_cast<const f32x4_v*>(f + 16 * cb);
          f32x4_v wr[NB];
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) wr[nb] = wf[(cb * NB + nb) * 64];
#pragma unroll
          for (int e = 0; e < 4; ++e) sums.add(wr, e, x[e]);
        }
      };
      if constexpr (BLK > 2 * kClassifyRun) {
        static_assert(BLK % (2 * kClassifyRun) == 0, "pairs of runs");
#pragma unroll 1
        for (int c0 = 0; c0 < BLK; c0 += 2 * kClassifyRun) {
          f32x4_v first[NB];
          add_run(c0);
          sums.take(first);
          add_run(c0 + kClassifyRun);
          sums.flush(first);
        }
      } else {
#pragma unroll 1
        for (int c0 = 0; c0 < BLK; c0 += kClassifyRun) {
          add_run(c0);
          sums.flush();
        }
      }
      f32x4_v acc[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[nb] = sums.total[nb] + bias[nb];
      const int64_t p = p0 + mg * 16 + li;
      if (p < m) store_classes<NB>(out, p, K, lg, vec_out, acc);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// Wider rows: lane (i, g) holds, of the gathered rows of point i, the channels
// 4 g .. 4 g + 3 of 16 channels at a time, which are the product's operand as
// they are; the rows are gathered once for the offsets and again for f.
template <bool BF16, int NB>
__global__ void __launch_bounds__(kBlock)
k_deform_classify_wide(const int4* __restrict__ idx, const float4* __restrict__ w, int64_t m,
                       const void* __restrict__ vals, int64_t ld_vals, int C, const float* __restrict__ wvec,
                       float beta, const float* __restrict__ Wc, const float* __restrict__ bc, int K,
                       float* __restrict__ out, int vec_out, unsigned nblk) {
  extern __shared__ __align__(16) float wl[];   // Wc, then wvec
  const int blocks = (C + 15) / 16;
  float* const wvl = wl + blocks * NB * 256;
  stage_classifier(wl, Wc, K, C, blocks, NB);
  for (int i = threadIdx.x; i < blocks * 16; i += kBlock) wvl[i] = i < C ? wvec[i] : 0.f;
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lg = lane >> 4;
  f32x4_v bias[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = 16 * nb + 4 * lg + r;
      bias[nb][r] = bc && j < K ? bc[j] : 0.f;
    }
  const unsigned G = gridDim.x;   // a multiple of 8
  const unsigned rg = (blockIdx.x % 8) * (G / 8) + blockIdx.x / 8;
  const unsigned per = (nblk + G - 1) / G;
  const unsigned lb1 = min((rg + 1) * per, nblk);
  for (unsigned lb = rg * per; lb < lb1; ++lb) {
    const int64_t p = (static_cast<int64_t>(lb) * 4 + wave) * 16 + li;
    const int4 iv = idx[min(p, m - 1)];
    const float4 wq = w[min(p, m - 1)];
    const int32_t vi[4] = {max(iv.x, 0), max(iv.y, 0), max(iv.z, 0), max(iv.w, 0)};
    const bool have[4] = {iv.x >= 0, iv.y >= 0, iv.z >= 0, iv.w >= 0};
    const float bw[4] = {have[0] ? wq.x : 0.f, have[1] ? wq.y : 0.f, have[2] ? wq.z : 0.f, have[3] ? wq.w : 0.f};
    // TAIL: the last block of channels where it is not full: lanes past C hold
    // zeros, not the row's last channels.  (Apart from the others: a select in
    // the loop keeps the compiler from overlapping its loads, 35 and 57 us at
    // 512 fp32 channels of 8,000 points.)
    auto gather = [&](int cb, f32x4_v (&x)[4], auto tail_c) {
      constexpr bool TAIL = decltype(tail_c)::value;
      const int c = 16 * cb + 4 * lg, ch = TAIL ? min(c, C - 4) : c;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int64_t at = static_cast<int64_t>(vi[k]) * ld_vals + ch;
        if constexpr (BF16) {
          const uint2 u = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(vals) + at);
          x[k] = f32x4_v{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                         __uint_as_float(u.y & 0xffff0000u)};
        } else {
          x[k] = *reinterpret_cast<const f32x4_v*>(static_cast<const float*>(vals) + at);
        }
        if (TAIL && c >= C) x[k] = f32x4_v{0.f, 0.f, 0.f, 0.f};
      }
    };
    // the offsets' sums in short chains too: kOffsetRun blocks, then the total
    const int full = C / 16;
    float part[4] = {0.f, 0.f, 0.f, 0.f}, run[4] = {0.f, 0.f, 0.f, 0.f};
    auto flush = [&]() {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        part[k] += run[k];
        run[k] = 0.f;
      }
    };
    auto offsets = [&](int cb, auto tail_c) {
      f32x4_v x[4];
      gather(cb, x, tail_c);
      const f32x4_v wv = *reinterpret_cast<const f32x4_v*>(wvl + 16 * cb + 4 * lg);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float qk[4];
        float mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          qk[k] = bw[k] * x[k][e];
          mx = fmaxf(mx, qk[k]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) run[k] += (qk[k] - mx) * wv[e];
      }
    };
    for (int cb = 0; cb < full; ++cb) {
      offsets(cb, std::false_type{});
      if (cb % kOffsetRun == kOffsetRun - 1) flush();
    }
    if (full < blocks) offsets(full, std::true_type{});
    flush();
    float coef[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      part[k] += xor_lane<16>(part[k]);
      part[k] += xor_lane<32>(part[k]);
      coef[k] = have[k] ? bw[k] + tanhf(beta + part[k]) : 0.f;
    }
    ClassSums<NB> sums;
    const f32x4_v* wf = reinterpret_cast<const f32x4_v*>(wl) + lane;
    auto classes = [&](int cb, auto tail_c) {
      f32x4_v x[4], wr[NB];
      gather(cb, x, tail_c);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) wr[nb] = wf[(cb * NB + nb) * 64];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        sums.add(wr, e, coef[0] * x[0][e] + coef[1] * x[1][e] + coef[2] * x[2][e] + coef[3] * x[3][e]);
    };
    for (int cb = 0; cb < full; ++cb) {
      classes(cb, std::false_type{});
      if (cb % kClassifyRun == kClassifyRun - 1) sums.flush();
    }
    if (full < blocks) classes(full, std::true_type{});
    sums.flush();
    f32x4_v acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = sums.total[nb] + bias[nb];
    if (p < m) store_classes<NB>(out, p, K, lg, vec_out, acc);
  }
}

// The same by lane groups: a point's row is formed in the registers of LPR lanes
// as in k_deform_slice and multiplied by Wc (K x C in LDS) there; the KP >= K
// logit partials of a lane group are summed by a reduce-scatter, after which
// each lane holds KP / LPR finished classes (the block its exchange bits
// name).  It spreads a small cloud over the chip, where the 16 points of a wave
// above are a chain of dependent steps, and it has no work for padded channels
// and classes (classify_by_rows has the figures).
// One exchange of the reduce-scatter: lanes whose bit OFF is set keep the upper
// LEN values, the others the lower LEN, and each adds the half its partner
// gives away; blk gathers the kept halves' bits.
template <int OFF, int LEN, int KP>
__device__ inline void reduce_scatter_step(float (&lg)[KP], int lane, int& blk) {
  const bool up = (lane & OFF) != 0;
#pragma unroll
  for (int i = 0; i < LEN; ++i) {
    const float give = up ? lg[i] : lg[i + LEN];
    const float keep = up ? lg[i + LEN] : lg[i];
    lg[i] = keep + xor_lane<OFF>(give);
  }
  blk = 2 * blk + (up ? 1 : 0);
}

template <bool BF16, int LPR, int CPL, int KP>
__global__ void __launch_bounds__(kBlock)
k_deform_classify_rows(const int4* __restrict__ idx, const float4* __restrict__ w, int64_t m,
                       const void* __restrict__ vals, int64_t ld_vals, int C, const float* __restrict__ wvec, float beta,
                       const float* __restrict__ Wc, const float* __restrict__ bc, int K, float* __restrict__ out,
                       unsigned nblk) {
  using Ch = Chunk<BF16>;
  extern __shared__ __align__(16) float wl[];   // [K][C]
  for (int i = threadIdx.x; i < K * C; i += kBlock) wl[i] = Wc[i];
  __syncthreads();
  const int lane = threadIdx.x & (LPR - 1);
  const int nchunk = C / Ch::N;
  // The weights are staged once per workgroup, which then walks a
  // contiguous range of the nblk logical blocks (each XCD a contiguous
  // share of the ranges, as xcd_item).
  const unsigned G = gridDim.x;   // a multiple of 8
  const unsigned r = (blockIdx.x % 8) * (G / 8) + blockIdx.x / 8;
  const unsigned per = (nblk + G - 1) / G;
  const unsigned lb1 = min((r + 1) * per, nblk);
  for (unsigned lb = r * per; lb < lb1; ++lb) {
    const int64_t p = (static_cast<int64_t>(lb) * kBlock + threadIdx.x) / LPR;
    const bool live = p < m;
    int4 iv = make_int4(-1, -1, -1, -1);
    float4 wq = make_float4(0.f, 0.f, 0.f, 0.f);
    if (live) { iv = idx[p]; wq = w[p]; }
    const int32_t vi[4] = {iv.x, iv.y, iv.z, iv.w};
    const float bw[4] = {wq.x, wq.y, wq.z, wq.w};
    float x[CPL][4][Ch::N];
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const int ch = lane + q * LPR;
      const bool on = live && ch < nchunk;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (on && vi[k] >= 0) {
          Ch c;
          c.load(vals, static_cast<int64_t>(vi[k]) * ld_vals + static_cast<int64_t>(ch) * Ch::N);
#pragma unroll
          for (int i = 0; i < Ch::N; ++i) x[q][k][i] = c.v[i];
        } else {
#pragma unroll
          for (int i = 0; i < Ch::N; ++i) x[q][k][i] = 0.f;
        }
      }
      if (on) {
#pragma unroll
        for (int i = 0; i < Ch::N; ++i) {
          const float wc = wvec[ch * Ch::N + i];
          float qk[4];
          float mx = -INFINITY;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            qk[k] = bw[k] * x[q][k][i];
            mx = fmaxf(mx, qk[k]);
          }
#pragma unroll
          for (int k = 0; k < 4; ++k) part[k] += (qk[k] - mx) * wc;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) part[k] = group_sum<LPR>(part[k]);
    float coef[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) coef[k] = bw[k] + tanhf(beta + part[k]);
    float lg[KP];
#pragma unroll
    for (int j = 0; j < KP; ++j) lg[j] = 0.f;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const int ch = lane + q * LPR;
      if (!(live && ch < nchunk)) continue;
#pragma unroll
      for (int i = 0; i < Ch::N; i += 4) {
        float f[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          f[u] = coef[0] * x[q][0][i + u] + coef[1] * x[q][1][i + u] + coef[2] * x[q][2][i + u] +
                 coef[3] * x[q][3][i + u];
#pragma unroll
        for (int j = 0; j < KP; ++j) {
          if (j >= K) break;
          const float4 wv4 = *reinterpret_cast<const float4*>(wl + j * C + ch * Ch::N + i);
          lg[j] += wv4.x * f[0] + wv4.y * f[1] + wv4.z * f[2] + wv4.w * f[3];
        }
      }
    }
    // the exchanges in the order of their cost (cheap ones move the most
    // values); blk = the class block this lane keeps
    int blk = 0;
    constexpr int S = (LPR >= 2) + (LPR >= 4) + (LPR >= 8) + (LPR >= 16) + (LPR >= 32) + (LPR >= 64);
    static_assert((KP >> S) >= 1, "at least one class per lane");
    if constexpr (LPR >= 2) reduce_scatter_step<1, (KP >> 1)>(lg, lane, blk);
    if constexpr (LPR >= 4) reduce_scatter_step<2, (KP >> 2)>(lg, lane, blk);
    if constexpr (LPR >= 16) reduce_scatter_step<8, (KP >> 3)>(lg, lane, blk);
    if constexpr (LPR >= 8) reduce_scatter_step<4, (KP >> (LPR >= 16 ? 4 : 3))>(lg, lane, blk);
    if constexpr (LPR >= 32) reduce_scatter_step<16, (KP >> 5)>(lg, lane, blk);
    if constexpr (LPR >= 64) reduce_scatter_step<32, (KP >> 6)>(lg, lane, blk);
    if (live) {
      constexpr int OWN = KP / LPR;
#pragma unroll
      for (int i = 0; i < OWN; ++i) {
        const int j = blk * OWN + i;
        if (j < K) out[p * K + j] = lg[i] + (bc ? bc[j] : 0.f);
      }
    }
  }
}

// DeformSlice backward, per point (C channels over LPR lanes, CPL 16-byte
// chunks per lane, as in the forward), with g = dL/dout_p:
//   q_k = b_k x_k; am_c = the first slot k whose float32 q_k is maximal,
//   M_c = q_{am_c}; s_k = beta + (q_k - M) . wv; db_k = tanh(s_k);
//   a_k = g . x_k; e_k = a_k (1 - db_k^2) (= dL/ds_k).
// It writes coef[4p + k] = (b_k + db_k, e_k b_k, (sum_j e_j) b_k, 0) and
// am[p][c] for the gather over J_v, and adds sum_k e_k (q_k - M) (dL/dwv) and
// sum_k e_k (dL/dbeta) into per-workgroup partials: the workgroups stride
// over the points, sum in registers, then over their lane groups in a fixed
// order.
template <int LPR, int CPL>
__global__ void __launch_bounds__(kBlock)
k_deform_bwd_point(const int4* __restrict__ idx, const float4* __restrict__ w, int64_t m,
                   const float* __restrict__ vals, int64_t ld_vals, int C, const float* __restrict__ wvec, float beta,
                   const float* __restrict__ dout, int64_t ld_dout, float4* __restrict__ coef,
                   uint8_t* __restrict__ am, float* __restrict__ part_wv, float* __restrict__ part_beta) {
  constexpr int G = kBlock / LPR;
  __shared__ float red[kBlock * CPL * 4];   // [group][channel], G * C <= this
  __shared__ float red_b[G];
  const int lane = threadIdx.x & (LPR - 1), grp = threadIdx.x / LPR;
  const int nchunk = C / 4;
  float wacc[CPL][4];
#pragma unroll
  for (int q = 0; q < CPL; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) wacc[q][i] = 0.f;
  float bacc = 0.f;
  const int64_t groups = (m + G - 1) / G;
  for (int64_t it = blockIdx.x; it < groups; it += gridDim.x) {
    const int64_t p = it * G + grp;
    const bool live = p < m;
    int4 iv = make_int4(0, 0, 0, 0);
    float4 wq = make_float4(0.f, 0.f, 0.f, 0.f);
    if (live) { iv = idx[p]; wq = w[p]; }
    const int32_t vi[4] = {iv.x, iv.y, iv.z, iv.w};
    const float bw[4] = {wq.x, wq.y, wq.z, wq.w};
    float x[CPL][4][4], gv[CPL][4], mx[CPL][4];
    float sp[4] = {0.f, 0.f, 0.f, 0.f}, ap[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const int ch = lane + q * LPR;
      const bool on = live && ch < nchunk;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (on) v = *reinterpret_cast<const float4*>(vals + static_cast<int64_t>(vi[k]) * ld_vals + 4 * ch);
        x[q][k][0] = v.x; x[q][k][1] = v.y; x[q][k][2] = v.z; x[q][k][3] = v.w;
      }
      float4 gg = make_float4(0.f, 0.f, 0.f, 0.f);
      if (on) gg = *reinterpret_cast<const float4*>(dout + p * ld_dout + 4 * ch);
      gv[q][0] = gg.x; gv[q][1] = gg.y; gv[q][2] = gg.z; gv[q][3] = gg.w;
      uint32_t word = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float wc = on ? wvec[4 * ch + i] : 0.f;
        float qk[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) qk[k] = bw[k] * x[q][k][i];
        float best = qk[0];
        uint32_t a = 0;
#pragma unroll
        for (int k = 1; k < 4; ++k)
          if (qk[k] > best) {
            best = qk[k];
            a = static_cast<uint32_t>(k);
          }
        mx[q][i] = best;
        word |= a << (8 * i);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          sp[k] += (qk[k] - best) * wc;
          ap[k] += gv[q][i] * x[q][k][i];
        }
      }
      if (on) *reinterpret_cast<uint32_t*>(am + p * C + 4 * ch) = word;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      sp[k] = group_sum<LPR>(sp[k]);
      ap[k] = group_sum<LPR>(ap[k]);
    }
    float e[4], esum = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float db = tanhf(beta + sp[k]);
      e[k] = ap[k] * (1.f - db * db);
      esum += e[k];
      sp[k] = db;
    }
    if (!live) continue;
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) coef[4 * p + k] = make_float4(bw[k] + sp[k], e[k] * bw[k], esum * bw[k], 0.f);
      bacc += esum;
    }
#pragma unroll
    for (int q = 0; q < CPL; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float a = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) a += e[k] * (bw[k] * x[q][k][i] - mx[q][i]);
        wacc[q][i] += a;
      }
  }
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const int ch = lane + q * LPR;
    if (ch < nchunk)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[grp * C + 4 * ch + i] = wacc[q][i];
  }
  if (lane == 0) red_b[grp] = bacc;
  __syncthreads();
  for (int c = threadIdx.x; c < C; c += kBlock) {
    float a = 0.f;
    for (int g2 = 0; g2 < G; ++g2) a += red[g2 * C + c];
    part_wv[static_cast<int64_t>(blockIdx.x) * C + c] = a;
  }
  if (threadIdx.x == 0) {
    float a = 0.f;
    for (int g2 = 0; g2 < G; ++g2) a += red_b[g2];
    part_beta[blockIdx.x] = a;
  }
}

// dL/dwv[c] (workgroup c < C) and dL/dbeta (workgroup C): the per-workgroup
// partials added by a fixed tree.
__global__ void __launch_bounds__(kBlock)
k_deform_bwd_reduce(const float* __restrict__ part_wv, const float* __restrict__ part_beta, int64_t nparts, int C,
                    float* __restrict__ dwv, float* __restrict__ dbeta) {
  __shared__ float sh[kBlock];
  const int c = blockIdx.x;
  float a = 0.f;
  for (int64_t b = threadIdx.x; b < nparts; b += kBlock) a += c < C ? part_wv[b * C + c] : part_beta[b];
  sh[threadIdx.x] = a;
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if (static_cast<int>(threadIdx.x) < off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (c < C) dwv[c] = sh[0];
    else *dbeta = sh[0];
  }
}

inline int lanes_per_row(int C, bool bf16) {
  const int chunks = C / (bf16 ? 8 : 4);
  int l = 1;
  while (l < chunks && l < 64) l <<= 1;
  return l;
}

// Lane group of one row (one vertex list entry or one point) for the splat,
// DeformSlice, the fused classifier and the DeformSlice gradient's point
// pass: 64 fp32 channels take 8 lanes of two 16-byte chunks each (half the
// per-entry bookkeeping per channel), every other width one chunk per lane.
// DeformSlice and its gradient must agree: the gradient recomputes the
// offsets, and the same lane groups sum the dot products in the same order.
// (The classifier sums them in this order too, except on the matrix cores for
// rows over kClassifyTileC channels, where its offsets may differ from the
// gradient's by the rounding of the order; the argmax is taken before the sum.)
inline int point_lanes_per_row(int C, bool bf16) {
  return !bf16 && C / 4 == 16 ? 8 : lanes_per_row(C, bf16);
}

inline unsigned grid_for(int64_t rows, int lpr) {
  return static_cast<unsigned>((rows * lpr + kBlock - 1) / kBlock);
}

template <bool BF16, int LPR, int Q>
void splat_launch(const int32_t* off, const int32_t* ent, const float* ew, const int32_t* cf, int chunk, int64_t n, int64_t total,
                  const void* feat, int64_t ldf, int C, int norm, void* vals, int64_t ldv, float* wsum,
                  float* ph, float* pt, float* pw, hipStream_t s) {
  constexpr int B = 8 / Q;   // entries in flight per lane group (more would cost occupancy)
  constexpr int G = kBlock / LPR;
  const int64_t span_len = static_cast<int64_t>(G) * chunk;
  const int64_t nspans = (total + span_len - 1) / span_len;
  const unsigned nblk = static_cast<unsigned>(nspans);
  const size_t lds = splat_lds_bytes(LPR, C);
  using Rows = WeightedRows<BF16, LPR, Q, B>;
  static bool lds_limit_set = false;
  if (!lds_limit_set) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_splat_chunks<BF16, LPR, Q, B, Rows>),
                              hipFuncAttributeMaxDynamicSharedMemorySize,
                              static_cast<int>(splat_lds_bytes(LPR, LPR * Q * Chunk<BF16>::N)));
    lds_limit_set = true;
  }
  const Rows rows{ew, feat, ldf};
  launch((k_splat_chunks<BF16, LPR, Q, B, Rows>), dim3(xcd_grid(nblk)), dim3(kBlock), lds, s, off, ent, rows, cf,
         chunk, n, total, C, norm, vals, ldv, wsum, ph, pt, pw, nblk);
  if (nspans > 1)
    launch((k_splat_finish<BF16, LPR, Q>), dim3(grid_for(nspans, LPR)), dim3(kBlock), 0, s, off, cf,
                       span_len, G, nspans, C, norm, vals, ldv, wsum, ph, pt, pw);
}

template <bool BF16>
void splat_dispatch(int lpr, int q, const int32_t* off, const int32_t* ent, const float* ew,
                    const int32_t* cf, int chunk, int64_t n, int64_t total, const void* feat, int64_t ldf, int C, int norm,
                    void* vals, int64_t ldv, float* wsum, float* ph, float* pt, float* pw, hipStream_t s) {
#define SPLAT_CASE(L, QQ) \
  if (lpr == L && q == QQ) return splat_launch<BF16, L, QQ>(off, ent, ew, cf, chunk, n, total, feat, ldf, C, norm, vals, ldv, wsum, ph, pt, pw, s);
  SPLAT_CASE(1, 1) SPLAT_CASE(2, 1) SPLAT_CASE(4, 1) SPLAT_CASE(8, 1) SPLAT_CASE(16, 1)
  SPLAT_CASE(32, 1) SPLAT_CASE(64, 1) SPLAT_CASE(64, 2) SPLAT_CASE(64, 4) SPLAT_CASE(8, 2)
#undef SPLAT_CASE
}

template <int LPR, int Q>
void deform_grad_gather(const int32_t* off, const int32_t* ent, const int32_t* cf, int chunk, int64_t n,
                        int64_t total, const float* g, int64_t ldg, const float4* coef, const uint8_t* am,
                        const float* wv, int C, float* dx, int64_t ldx, float* ph, float* pt, float* pw,
                        hipStream_t s) {
  constexpr int B = 8 / Q;
  constexpr int G = kBlock / LPR;
  using Rows = DeformGradRows<LPR, Q, B>;
  const int64_t span_len = static_cast<int64_t>(G) * chunk;
  const int64_t nspans = (total + span_len - 1) / span_len;
  const unsigned nblk = static_cast<unsigned>(nspans);
  const size_t lds = splat_lds_bytes(LPR, C);
  static bool lds_limit_set = false;
  if (!lds_limit_set) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_splat_chunks<false, LPR, Q, B, Rows>),
                              hipFuncAttributeMaxDynamicSharedMemorySize,
                              static_cast<int>(splat_lds_bytes(LPR, LPR * Q * 4)));
    lds_limit_set = true;
  }
  Rows rows{g, ldg, coef, am, wv, C, {}};
  launch((k_splat_chunks<false, LPR, Q, B, Rows>), dim3(xcd_grid(nblk)), dim3(kBlock), lds, s, off, ent, rows, cf,
         chunk, n, total, C, 0, static_cast<void*>(dx), ldx, static_cast<float*>(nullptr), ph, pt, pw, nblk);
  if (nspans > 1)
    launch((k_splat_finish<false, LPR, Q>), dim3(grid_for(nspans, LPR)), dim3(kBlock), 0, s, off, cf, span_len, G,
           nspans, C, 0, static_cast<void*>(dx), ldx, static_cast<float*>(nullptr), static_cast<const float*>(ph),
           static_cast<const float*>(pt), static_cast<const float*>(pw));
}

void deform_grad_dispatch(int lpr, int q, const int32_t* off, const int32_t* ent, const int32_t* cf, int chunk,
                          int64_t n, int64_t total, const float* g, int64_t ldg, const float4* coef,
                          const uint8_t* am, const float* wv, int C, float* dx, int64_t ldx, float* ph, float* pt,
                          float* pw, hipStream_t s) {
#define DGRAD_CASE(L, QQ) \
  if (lpr == L && q == QQ) return deform_grad_gather<L, QQ>(off, ent, cf, chunk, n, total, g, ldg, coef, am, wv, C, dx, ldx, ph, pt, pw, s);
  DGRAD_CASE(1, 1) DGRAD_CASE(2, 1) DGRAD_CASE(4, 1) DGRAD_CASE(8, 1) DGRAD_CASE(16, 1)
  DGRAD_CASE(32, 1) DGRAD_CASE(64, 1) DGRAD_CASE(64, 2)
#undef DGRAD_CASE
}

template <int CPL>
void deform_bwd_point_dispatch(int lpr, unsigned grid, const int32_t* idx, const float* w, int64_t m,
                               const float* vals, int64_t ldv, int C, const float* wv, float beta, const float* dout,
                               int64_t ldo, float4* coef, uint8_t* am, float* pwv, float* pb, hipStream_t s) {
  const int4* i4 = reinterpret_cast<const int4*>(idx);
  const float4* w4 = reinterpret_cast<const float4*>(w);
#define DPT_CASE(L) \
  if (lpr == L) return launch((k_deform_bwd_point<L, CPL>), dim3(grid), dim3(kBlock), 0, s, i4, w4, m, vals, ldv, C, wv, beta, dout, ldo, coef, am, pwv, pb);
  DPT_CASE(1) DPT_CASE(2) DPT_CASE(4) DPT_CASE(8) DPT_CASE(16) DPT_CASE(32) DPT_CASE(64)
#undef DPT_CASE
}

template <bool BF16, bool SCALED>
void slice_dispatch(int lpr, const int32_t* idx, const float* w, int64_t m, const void* vals,
                    int64_t ldv, int C, float* out, const float* vscale, hipStream_t s) {
  const int4* i4 = reinterpret_cast<const int4*>(idx);
  const float4* w4 = reinterpret_cast<const float4*>(w);
  const dim3 b(kBlock);
  auto go = [&](auto kernel, int lanes) {
    const unsigned nblk = grid_for((m + 1) / 2, lanes);   // two points per lane group
    launch(kernel, dim3(xcd_grid(nblk)), b, 0, s, i4, w4, m, vals, ldv, C, out, vscale, nblk);
  };
  auto wide = [&](auto kernel) {   // a wave per point
    const int64_t per_block = (kBlock / 64) * (BF16 ? 4 : 2);
    const unsigned nblk = static_cast<unsigned>((m + per_block - 1) / per_block);
    launch(kernel, dim3(xcd_grid(nblk)), b, 0, s, i4, w4, m, vals, ldv, C, out, vscale, nblk);
  };
  if (C > 128 && m > kSliceWideM) return wide(k_slice_wide<BF16, 4, SCALED>);
  if constexpr (BF16)
    if (C > 64 && C <= 128)
      return m > kSliceWideM128 ? wide(k_slice_wide<true, 2, SCALED>) : go(k_slice<HalfChunk, 32, SCALED>, 32);
  switch (lpr) {
    case 1: return go(k_slice<Chunk<BF16>, 1, SCALED>, 1);
    case 2: return go(k_slice<Chunk<BF16>, 2, SCALED>, 2);
    case 4: return go(k_slice<Chunk<BF16>, 4, SCALED>, 4);
    case 8: return go(k_slice<Chunk<BF16>, 8, SCALED>, 8);
    case 16: return go(k_slice<Chunk<BF16>, 16, SCALED>, 16);
    case 32: return go(k_slice<Chunk<BF16>, 32, SCALED>, 32);
    default: return go(k_slice<Chunk<BF16>, 64, SCALED>, 64);
  }
}

template <bool BF16, int CPL>
void deform_dispatch(int lpr, const int32_t* idx, const float* w, int64_t m, const void* vals,
                     int64_t ldv, int C, const float* wv, float beta, float* out, float* delta, float* plain,
                     hipStream_t s) {
  const unsigned nblk = grid_for(m, lpr);
  const dim3 g(xcd_grid(nblk)), b(kBlock);
  const int4* i4 = reinterpret_cast<const int4*>(idx);
  const float4* w4 = reinterpret_cast<const float4*>(w);
  float4* d4 = reinterpret_cast<float4*>(delta);
  switch (lpr) {
    case 1: launch((k_deform_slice<BF16, 1, CPL>), g, b, 0, s, i4, w4, m, vals, ldv, C, wv, beta, out, d4, plain, nblk); break;
    case 2: launch((k_deform_slice<BF16, 2, CPL>), g, b, 0, s, i4, w4, m, vals, ldv, C, wv, beta, out, d4, plain, nblk); break;
    case 4: launch((k_deform_slice<BF16, 4, CPL>), g, b, 0, s, i4, w4, m, vals, ldv, C, wv, beta, out, d4, plain, nblk); break;
    case 8: launch((k_deform_slice<BF16, 8, CPL>), g, b, 0, s, i4, w4, m, vals, ldv, C, wv, beta, out, d4, plain, nblk); break;
    case 16: launch((k_deform_slice<BF16, 16, CPL>), g, b, 0, s, i4, w4, m, vals, ldv, C, wv, beta, out, d4, plain, nblk); break;
    case 32: launch((k_deform_slice<BF16, 32, CPL>), g, b, 0, s, i4, w4, m, vals, ldv, C, wv, beta, out, d4, plain, nblk); break;
    default: launch((k_deform_slice<BF16, 64, CPL>), g, b, 0, s, i4, w4, m, vals, ldv, C, wv, beta, out, d4, plain, nblk); break;
  }
}

}  // namespace

// Largest channel count the gather kernels handle: 4 chunks per lane of a
// full wavefront for splat, 2 for DeformSlice; slice loops without limit.
int splat_max_channels(bool bf16) { return (bf16 ? 8 : 4) * 64 * 4; }
int deform_max_channels(bool bf16) { return (bf16 ? 8 : 4) * 64 * 2; }

// Partials of k_splat_chunks: a head and a tail row of C floats and two
// weights per span of kBlock/LPR chunks (sized for the smallest span, LPR =
// 64, whatever the channel count).
int64_t splat_partial_floats(int64_t total, int chunk, int C) {
  const int64_t span_len = static_cast<int64_t>(kBlock / 64) * chunk;
  const int64_t nspans = (total + span_len - 1) / span_len;
  return nspans * (2 * static_cast<int64_t>(C) + 2);
}

void launch_splat(const int32_t* offsets, const int32_t* entries, const float* entry_w,
                  const int32_t* chunk_first, int chunk, int64_t n, int64_t total, const void* feat, int64_t ld_feat, int C,
                  int bf16, int normalize, void* vals, int64_t ld_vals, float* wsum, float* partials,
                  hipStream_t s) {
  if (total <= 0) return;
  const int chunks = C / (bf16 ? 8 : 4);
  const int lpr = point_lanes_per_row(C, bf16 != 0);
  const int q = chunks <= lpr ? 1 : (chunks <= 2 * lpr ? 2 : 4);
  const int64_t span_len = static_cast<int64_t>(kBlock / lpr) * chunk;
  const int64_t nspans = (total + span_len - 1) / span_len;
  float* ph = partials;
  float* pt = partials + nspans * C;
  float* pw = partials + 2 * nspans * C;
  ScopedKernelTimer tm("splat", s);
  if (bf16) splat_dispatch<true>(lpr, q, offsets, entries, entry_w, chunk_first, chunk, n, total, feat, ld_feat, C, normalize, vals, ld_vals, wsum, ph, pt, pw, s);
  else splat_dispatch<false>(lpr, q, offsets, entries, entry_w, chunk_first, chunk, n, total, feat, ld_feat, C, normalize, vals, ld_vals, wsum, ph, pt, pw, s);
}

void launch_slice(const int32_t* idx, const float* w, int64_t m, const void* vals, int64_t ld_vals,
                  int C, int bf16, float* out, hipStream_t s, const float* vscale) {
  if (m <= 0) return;
  const int lpr = lanes_per_row(C, bf16 != 0);
  ScopedKernelTimer tm("slice", s);
  if (bf16) slice_dispatch<true, false>(lpr, idx, w, m, vals, ld_vals, C, out, nullptr, s);
  else if (vscale) slice_dispatch<false, true>(lpr, idx, w, m, vals, ld_vals, C, out, vscale, s);
  else slice_dispatch<false, false>(lpr, idx, w, m, vals, ld_vals, C, out, nullptr, s);
}

template <class Kernel>
void classify_launch(Kernel kernel, bool* limit_set, size_t lds, int points_per_group, const int32_t* idx,
                     const float* w, int64_t m, const void* vals, int64_t ldv, int C, const float* wv, float beta,
                     const float* Wc, const float* bc, int K, float* out, hipStream_t s) {
  if (!*limit_set) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                              kClassifyMaxLds);
    *limit_set = true;
  }
  const unsigned nblk = static_cast<unsigned>((m + points_per_group - 1) / points_per_group);
  const int vec_out = K % 4 == 0 && (reinterpret_cast<uintptr_t>(out) & 15u) == 0;
  launch(kernel, dim3(std::min(xcd_grid(nblk), kClassifyGrid)), dim3(kBlock), static_cast<uint32_t>(lds), s,
         reinterpret_cast<const int4*>(idx), reinterpret_cast<const float4*>(w), m, vals, ldv, C, wv, beta, Wc, bc, K,
         out, vec_out, nblk);
}

// Whether the classifier runs by lane groups (k_deform_classify_rows) rather
// than on the matrix cores.  Lines from sweeps over 250 to 200,000 points, 16 to
// 512 channels and 3 to 50 classes (us by lane groups and on the matrix cores):
// the latter take 3 to 50 us however few the points are, the time of the former
// grows with points, channels and classes.
//   48 fp32 channels, 5 classes: 3.9 and 5.4 at 2,000 points, 6.2 and 6.8 at 24,000, 12 and 8.4 at 40,000
//   64 fp32, 3 classes: 4.5 and 5.0 at 2,000, 5.6 and 6.0 at 24,000, 8.3 and 7.5 at 40,000; 10: 5.4 and 5.0 at 2,000
//   128 fp32, 20 classes: 5.5 and 11 at 2,000, 7.8 and 11 at 8,000, 20.7 and 13.8 at 24,000
//   128 bf16, 5 classes: 5.0 and 7.5 at 2,000, 9.5 and 10.4 at 24,000; 20: 7.4 and 9.6, 17.9 and 13.1
//   224 fp32, 20 classes: 13.2 and 19.1 at 1,000, 23.5 and 19.2 at 2,000
//   160 bf16, 5 classes: 5.1 and 11.4 at 1,000, 10.5 and 11.8 at 12,000, 27.5 and 31.8 at 40,000, 109 and 156 at
//   200,000 (its tiles are padded to 256 channels and 16 classes); 20: 13.2 and 15.4 at 8,000, 39.8 and 29.3 at 24,000
//   512 fp32, 20 classes: 31.6 and 43.1 at 2,000, 47.9 and 37.9 at 4,000
bool classify_by_rows(int64_t m, int C, int K, bool bf16) {
  if (C <= 32) return false;
  if (C <= 64 && (bf16 || C == 64)) return K <= 4 && m <= (bf16 ? 40000 : 32768);
  if (C <= 64) return K <= 32 && m * (K + 8) <= 360000;
  if (C <= 128 && bf16) return K <= 32 && m * (K + 2) <= 185000;
  if (C <= 128) return K <= 32 ? m * (K + 32) <= 560000 : m <= 1500;
  if (C <= 256 && bf16)
    return K <= 3 || (K <= 32 ? m * (K + 10) * C <= 46000000 : m <= 2000) ||
           (K * C <= 1920 && m >= (K * C <= 1000 ? 18000 : 100000));
  if (C <= 256) return m <= 1500;
  return m <= (K <= 20 ? (bf16 ? 14 : 13) * C / 2 : (bf16 ? 2100 : 1800));
}

template <bool BF16, int LPR, int CPL, int KP>
void classify_rows_launch(const int32_t* idx, const float* w, int64_t m, const void* vals, int64_t ldv, int C,
                          const float* wv, float beta, const float* Wc, const float* bc, int K, float* out,
                          hipStream_t s) {
  static bool set = false;
  if (!set) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_deform_classify_rows<BF16, LPR, CPL, KP>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, 4 * kClassifyMaxWeights);
    set = true;
  }
  const unsigned nblk = grid_for(m, LPR);
  launch((k_deform_classify_rows<BF16, LPR, CPL, KP>), dim3(std::min(xcd_grid(nblk), kClassifyGrid)), dim3(kBlock),
         static_cast<uint32_t>(4 * K * C), s, reinterpret_cast<const int4*>(idx), reinterpret_cast<const float4*>(w), m,
         vals, ldv, C, wv, beta, Wc, bc, K, out, nblk);
}

// the lane groups of the widths and class counts that classify_by_rows takes
template <bool BF16>
void classify_rows_dispatch(const int32_t* idx, const float* w, int64_t m, const void* vals, int64_t ldv, int C,
                            const float* wv, float beta, const float* Wc, const float* bc, int K, float* out,
                            hipStream_t s) {
  auto go = [&](auto kernel) { kernel(idx, w, m, vals, ldv, C, wv, beta, Wc, bc, K, out, s); };
  const bool two = C / Chunk<BF16>::N > 64;   // two chunks per lane of a wave
  if constexpr (BF16) {
    if (C <= 64) return go(classify_rows_launch<true, 8, 1, 32>);
    if (C <= 128) return go(classify_rows_launch<true, 16, 1, 32>);
    if (C <= 256) return K <= 32 ? go(classify_rows_launch<true, 32, 1, 32>) : go(classify_rows_launch<true, 32, 1, 64>);
  } else {
    if (C < 64) return go(classify_rows_launch<false, 16, 1, 32>);
    if (C == 64) return go(classify_rows_launch<false, 8, 2, 32>);
    if (C <= 128) return K <= 32 ? go(classify_rows_launch<false, 32, 1, 32>) : go(classify_rows_launch<false, 32, 1, 64>);
  }
  return two ? go(classify_rows_launch<BF16, 64, 2, 64>) : go(classify_rows_launch<BF16, 64, 1, 64>);
}

template <bool BF16, int NB>
void deform_classify_dispatch(const int32_t* idx, const float* w, int64_t m, const void* vals, int64_t ldv, int C,
                              const float* wv, float beta, const float* Wc, const float* bc, int K, float* out,
                              hipStream_t s) {
  const int lpr = point_lanes_per_row(C, BF16);
  const bool two = C / Chunk<BF16>::N > lpr;
  if (C > kClassifyTileC) {
    static bool set = false;
    const size_t blocks = (C + 15) / 16;
    return classify_launch(&k_deform_classify_wide<BF16, NB>, &set, 4 * (blocks * NB * 256 + blocks * 16), 64, idx, w, m,
                           vals, ldv, C, wv, beta, Wc, bc, K, out, s);
  }
#define DCL_CASE(L, CPL)                                                                                              \
  if (lpr == L && two == (CPL == 2)) {                                                                                \
    static bool set = false;                                                                                          \
    constexpr int TP = 64 / L > 16 ? 64 / L : 16, CW = L * CPL * Chunk<BF16>::N;                                      \
    return classify_launch(&k_deform_classify<BF16, L, CPL, NB>, &set,                                                \
                           4 * static_cast<size_t>((CW + 15) / 16 * NB * 256 + 4 * TP * (CW + 4)), 4 * TP, idx, w, m, vals, \
                           ldv, C, wv, beta, Wc, bc, K, out, s);                                                      \
  }
  DCL_CASE(1, 1) DCL_CASE(2, 1) DCL_CASE(4, 1) DCL_CASE(8, 1) DCL_CASE(16, 1) DCL_CASE(32, 1)
  if constexpr (!BF16) { DCL_CASE(8, 2) DCL_CASE(64, 1) }
#undef DCL_CASE
}

int deform_classify_max_classes() { return 64; }
int deform_classify_max_weights() { return kClassifyMaxWeights; }

void launch_deform_classify(const int32_t* idx, const float* w, int64_t m, const void* vals, int64_t ld_vals, int C,
                            int bf16, const float* wv, float beta, const float* Wc, const float* bc, int K, float* out,
                            hipStream_t s) {
  if (m <= 0) return;
  ScopedKernelTimer tm("deform_slice", s);
  if (classify_by_rows(m, C, K, bf16 != 0)) {
    if (bf16) classify_rows_dispatch<true>(idx, w, m, vals, ld_vals, C, wv, beta, Wc, bc, K, out, s);
    else classify_rows_dispatch<false>(idx, w, m, vals, ld_vals, C, wv, beta, Wc, bc, K, out, s);
    return;
  }
  const int nb = (K + 15) / 16;   // K <= 64
#define DCL_GO(BFV, NBV) return deform_classify_dispatch<BFV, NBV>(idx, w, m, vals, ld_vals, C, wv, beta, Wc, bc, K, out, s)
#define DCL_NB(BFV)              \
  switch (nb) {                  \
    case 1: DCL_GO(BFV, 1);      \
    case 2: DCL_GO(BFV, 2);      \
    case 3: DCL_GO(BFV, 3);      \
    default: DCL_GO(BFV, 4);     \
  }
  if (bf16) DCL_NB(true)
  else DCL_NB(false)
#undef DCL_NB
#undef DCL_GO
}

// Work space of launch_deform_slice_backward, in bytes.
int64_t deform_backward_workspace_bytes(int64_t m, int C, int64_t total, int chunk) {
  return 16 * 4 * m + m * C + 4 * (kDeformBwdGrid * (static_cast<int64_t>(C) + 1)) +
         4 * splat_partial_floats(total, chunk, C) + 64;
}

void launch_deform_slice_backward(const int32_t* idx, const float* w, int64_t m, const int32_t* offsets,
                                  const int32_t* entries, const int32_t* chunk_first, int chunk, int64_t n,
                                  int64_t total, const float* vals, int64_t ld_vals, int C, const float* wv,
                                  float beta, const float* dout, int64_t ld_dout, float* dvals, int64_t ld_dvals,
                                  float* dwv, float* dbeta, void* work, hipStream_t s) {
  ScopedKernelTimer tm("deform_bwd", s);
  if (m <= 0 || n <= 0) {
    // no point: dL/dwv and dL/dbeta are empty sums
    launch(k_deform_bwd_reduce, dim3(static_cast<unsigned>(C + 1)), dim3(kBlock), 0, s,
           static_cast<const float*>(nullptr), static_cast<const float*>(nullptr), static_cast<int64_t>(0), C, dwv,
           dbeta);
    return;
  }
  char* wp = static_cast<char*>(work);
  float4* coef = reinterpret_cast<float4*>(wp);
  wp += 16 * 4 * m;
  float* pwv = reinterpret_cast<float*>(wp);
  wp += 4 * kDeformBwdGrid * static_cast<int64_t>(C);
  float* pb = reinterpret_cast<float*>(wp);
  wp += 4 * kDeformBwdGrid;
  float* parts = reinterpret_cast<float*>(wp);
  wp += 4 * splat_partial_floats(total, chunk, C);
  uint8_t* am = reinterpret_cast<uint8_t*>(wp);
  // the point pass on the forward's lane groups (the same offsets); the
  // gather over the vertex lists on one chunk per lane
  const int plpr = point_lanes_per_row(C, false);
  const int lpr = lanes_per_row(C, false);
  const int chunks = C / 4;
  const int G = kBlock / plpr;
  const int64_t groups = (m + G - 1) / G;
  const unsigned grid = static_cast<unsigned>(std::min<int64_t>(groups, kDeformBwdGrid));
  if (chunks > plpr)
    deform_bwd_point_dispatch<2>(plpr, grid, idx, w, m, vals, ld_vals, C, wv, beta, dout, ld_dout, coef, am, pwv, pb, s);
  else
    deform_bwd_point_dispatch<1>(plpr, grid, idx, w, m, vals, ld_vals, C, wv, beta, dout, ld_dout, coef, am, pwv, pb, s);
  launch(k_deform_bwd_reduce, dim3(static_cast<unsigned>(C + 1)), dim3(kBlock), 0, s, static_cast<const float*>(pwv),
         static_cast<const float*>(pb), static_cast<int64_t>(grid), C, dwv, dbeta);
  const int q = chunks <= lpr ? 1 : 2;
  const int64_t span_len = static_cast<int64_t>(kBlock / lpr) * chunk;
  const int64_t nspans = (total + span_len - 1) / span_len;
  deform_grad_dispatch(lpr, q, offsets, entries, chunk_first, chunk, n, total, dout, ld_dout, coef, am, wv, C, dvals,
                       ld_dvals, parts, parts + nspans * C, parts + 2 * nspans * C, s);
}

void launch_deform_slice(const int32_t* idx, const float* w, int64_t m, const void* vals,
                         int64_t ld_vals, int C, int bf16, const float* wv, float beta, float* out,
                         float* delta, float* plain, hipStream_t s) {
  if (m <= 0) return;
  const int chunks = C / (bf16 ? 8 : 4);
  const int lpr = point_lanes_per_row(C, bf16 != 0);
  ScopedKernelTimer tm("deform_slice", s);
  const bool two = chunks > lpr;
  if (bf16) {
    if (two) deform_dispatch<true, 2>(lpr, idx, w, m, vals, ld_vals, C, wv, beta, out, delta, plain, s);
    else deform_dispatch<true, 1>(lpr, idx, w, m, vals, ld_vals, C, wv, beta, out, delta, plain, s);
  } else {
    if (two) deform_dispatch<false, 2>(lpr, idx, w, m, vals, ld_vals, C, wv, beta, out, delta, plain, s);
    else deform_dispatch<false, 1>(lpr, idx, w, m, vals, ld_vals, C, wv, beta, out, delta, plain, s);
  }
}

}  // namespace lat

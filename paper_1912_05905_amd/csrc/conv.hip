// Lattice convolution on gfx950 matrix cores.
//
// out[v] = bias + sum_t in[nb(v,t)] W[t]^T is a GEMM whose A operand is
// gathered: row v of A is the concatenation over the 9 taps of the input
// rows of v's neighbours (a zero row where the neighbour is missing).  The
// neighbour table is tap-major (nb[t][v]) so a wave reads the indices of its
// rows with one coalesced load per tap.  The same kernel runs the 1-hop
// convolution, the strided convolution of Downsample and the transposed
// convolution of Upsample; only the table differs.
//
// Each wave owns a (16 RM) x (16 RN) output tile in MFMA accumulators and
// walks K = 9 * Cin.  Operands go straight from global memory (L2) into
// registers in the MFMA operand layout: every lane loads 16 contiguous bytes
// of one input row (A) and of one weight row (B, weights stored
// [tap][Cout][Cin] so that the K dimension is contiguous for both).
//   fp32: v_mfma_f32_16x16x4_f32, a float4 per lane feeds 4 MFMAs (K = 16
//         per step: lane group g holds channels 4g..4g+3).
//   bf16: v_mfma_f32_16x16x32_bf16, 8 bf16 per lane feed one MFMA (K = 32
//         per step: lane group g holds channels 8g..8g+7).
// Any assignment of K indices to (lane group, element) works as long as A
// and B use the same one; the accumulator layout is fixed by the hardware:
// lane l holds rows 4*(l/16) + r, r = 0..3, of column l%16.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "lattice_internal.h"

namespace lat {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kWaves = 4;
constexpr int kBlock = 64 * kWaves;

// Buffer resource word 3 for raw (untyped) buffer loads on CDNA, and an
// offset beyond any buffer the kernels build (at most kMaxBufferBytes), for
// which a buffer load returns zeros without a memory access.
constexpr int kRsrcWord3 = 0x00020000;
constexpr int kMaxPreChannels = 1024;   // widest input of a pre-activated convolution
constexpr int kOutOfRange = static_cast<int>(0x80000000u);
constexpr int64_t kMaxBufferBytes = (int64_t{1} << 31) - 64;

// f(std::integral_constant<int, i>) for i = 0 .. N-1, unrolled.
template <class F, int... I>
__device__ inline void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ inline void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Operand fragment of one lane: 16 bytes of one row (A) or weight row (B).
template <bool BF16> struct Frag;
template <> struct Frag<false> {
  float4 v;
  __device__ inline void zero() { v = make_float4(0.f, 0.f, 0.f, 0.f); }
  __device__ inline void load(const void* base, int64_t elem) {
    v = *reinterpret_cast<const float4*>(static_cast<const float*>(base) + elem);
  }
};
template <> struct Frag<true> {
  u32x4 v;
  __device__ inline void zero() { v = u32x4{0u, 0u, 0u, 0u}; }
  __device__ inline void load(const void* base, int64_t elem) {
    v = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(base) + elem);
  }
};

__device__ inline void mma(f32x4& acc, const Frag<false>& a, const Frag<false>& b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.x, b.v.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.y, b.v.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.z, b.v.z, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.w, b.v.w, acc, 0, 0, 0);
}
__device__ inline void mma(f32x4& acc, const Frag<true>& a, const Frag<true>& b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.v), __builtin_bit_cast(bf16x8, b.v),
                                                 acc, 0, 0, 0);
}

// Workgroup of WM x WN waves; each wave owns (16 RM) x (16 RN) outputs.
template <bool BF16, int RM, int RN, int WM, int WN>
__global__ void __launch_bounds__(kBlock)
k_conv(const int32_t* __restrict__ nbr, int64_t ldn, int64_t n_out, const void* __restrict__ in,
       int64_t ld_in, int Cin, const void* __restrict__ W, const float* __restrict__ bias, int Cout,
       int relu, void* __restrict__ out, int64_t ld_out, const int32_t* __restrict__ rows) {
  static_assert(WM * WN == kWaves, "four waves per workgroup");
  constexpr int KS = BF16 ? 32 : 16;          // channels per K step
  constexpr int EPL = BF16 ? 8 : 4;           // elements per lane per step
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int li = lane & 15;                   // row (A) / column (B) within a 16-block
  const int lg = lane >> 4;                   // K group
  const int64_t row0 = (static_cast<int64_t>(blockIdx.x) * WM + wave % WM) * (16 * RM);
  const int col0 = (blockIdx.y * WN + wave / WM) * (16 * RN);

  f32x4 acc[RM][RN];
#pragma unroll
  for (int a = 0; a < RM; ++a)
#pragma unroll
    for (int b = 0; b < RN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  // neighbour rows of every tap, loaded once
  int32_t nb[kTaps][RM];
#pragma unroll
  for (int t = 0; t < kTaps; ++t)
#pragma unroll
    for (int a = 0; a < RM; ++a) {
      const int64_t r = row0 + a * 16 + li;
      nb[t][a] = r < n_out ? nbr[t * ldn + (rows ? rows[r] : r)] : -1;
    }
  int64_t wrow[RN];
  bool col_ok[RN];
#pragma unroll
  for (int b = 0; b < RN; ++b) {
    const int col = col0 + b * 16 + li;
    col_ok[b] = col < Cout;
    wrow[b] = static_cast<int64_t>(col) * Cin;
  }
  const int64_t wtap = static_cast<int64_t>(Cout) * Cin;

  Frag<BF16> A[RM], B[RN], An[RM], Bn[RN];
  auto load = [&](int t, int c0, Frag<BF16>(&fa)[RM], Frag<BF16>(&fb)[RN]) {
    const int ch = c0 + lg * EPL;
    const bool k_ok = ch < Cin;
#pragma unroll
    for (int a = 0; a < RM; ++a) {
      if (k_ok && nb[t][a] >= 0) fa[a].load(in, static_cast<int64_t>(nb[t][a]) * ld_in + ch);
      else fa[a].zero();
    }
#pragma unroll
    for (int b = 0; b < RN; ++b) {
      if (k_ok && col_ok[b]) fb[b].load(W, t * wtap + wrow[b] + ch);
      else fb[b].zero();
    }
  };

  load(0, 0, A, B);
#pragma unroll
  for (int t = 0; t < kTaps; ++t) {
    for (int c0 = 0; c0 < Cin; c0 += KS) {
      // prefetch the next K step (next channels of this tap, or the next tap)
      if (c0 + KS < Cin) load(t, c0 + KS, An, Bn);
      else if (t + 1 < kTaps) load(t + 1, 0, An, Bn);
#pragma unroll
      for (int a = 0; a < RM; ++a)
#pragma unroll
        for (int b = 0; b < RN; ++b) mma(acc[a][b], A[a], B[b]);
#pragma unroll
      for (int a = 0; a < RM; ++a) A[a] = An[a];
#pragma unroll
      for (int b = 0; b < RN; ++b) B[b] = Bn[b];
    }
  }

  // epilogue: bias, ReLU, convert, store
#pragma unroll
  for (int b = 0; b < RN; ++b) {
    const int col = col0 + b * 16 + li;
    if (col >= Cout) continue;
    const float bb = bias ? bias[col] : 0.f;
#pragma unroll
    for (int a = 0; a < RM; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t r0 = row0 + a * 16 + lg * 4 + r;
        if (r0 >= n_out) continue;
        const int64_t row = rows ? rows[r0] : r0;
        float v = acc[a][b][r] + bb;
        if (relu) v = fmaxf(v, 0.f);
        if constexpr (BF16)
          static_cast<uint16_t*>(out)[row * ld_out + col] = f32_to_bf16(v);
        else
          static_cast<float*>(out)[row * ld_out + col] = v;
      }
  }
}

template <bool BF16, int RM, int RN, int WM, int WN>
void conv_launch(const int32_t* nbr, int64_t ldn, int64_t n_out, const void* in, int64_t ld_in,
                 int Cin, const void* W, const float* bias, int Cout, int relu, void* out,
                 int64_t ld_out, const int32_t* rows, hipStream_t s) {
  const int64_t rows_per_block = static_cast<int64_t>(WM) * 16 * RM;
  const int cols_per_block = WN * 16 * RN;
  const dim3 grid(static_cast<unsigned>((n_out + rows_per_block - 1) / rows_per_block),
                  static_cast<unsigned>((Cout + cols_per_block - 1) / cols_per_block));
  launch((k_conv<BF16, RM, RN, WM, WN>), grid, dim3(kBlock), 0, s, nbr, ldn, n_out, in,
                     ld_in, Cin, W, bias, Cout, relu, out, ld_out, rows);
}

// ---------------------------------------------------------------------------
// LDS-staged pipeline.  A stage is one tap and KC channels.  The whole
// workgroup gathers the stage's A tile (BM neighbour rows, KC channels) and
// B tile (BN weight rows, KC channels) into LDS with 16-byte loads, 4 to 16
// lanes per row segment.  The 16-byte chunks of an LDS row are stored in an
// order permuted by the row (chunk c of row r at c ^ swz(r)), so that the 16
// rows an MFMA fragment reads, and the chunks a copy writes, fall in different
// banks: measured on gfx950 with rocprofv3 (SQ_LDS_BANK_CONFLICT), rows padded
// by 16 bytes cost about 3 conflict cycles per ds_read_b128, these
// permutations none.
// Workgroups are numbered so that each XCD gets a contiguous range of row
// tiles: neighbouring rows (the gather's halo) then stay in that XCD's L2.
//
// What bounds it is how early a stage's loads are issued: left to itself the
// compiler sinks them to the end of the step, right before the barrier that
// precedes their copy to LDS.  Scheduling groups therefore order the step (see
// there).  To issue the loads early they have to be cheap and free of
// branches: the table of a tile holds byte offsets, a load's address is that
// offset plus a scalar, and the tap and channel are stepped rather than divided
// out of the stage number.  With the loads sunk (and a wait for every load in
// flight in front of each) the fp32 convolutions of a LiDAR scan's network took
// 950 us, and 760 us here; a layer 128->128 on 6.4k vertices 30 and 26 us; bf16
// 256->256 on 239k vertices 513 and 420 us.
// ---------------------------------------------------------------------------
template <bool BF16, int BM, int BN, int WM, int WN, int KCB>
struct LdsConv {
  static constexpr int U = BF16 ? 2 : 4;            // bytes per element
  static constexpr int EPC = 16 / U;                // elements per 16-byte chunk
  static constexpr int KC = KCB / U;                // channels per stage
  static constexpr int CPR = KCB / 16;              // chunks per row per stage
  static constexpr int LDR = KC;                    // LDS row (elements), chunks permuted by swz
  // chunk permutation of row r: 4 chunks by (r / 2) mod 4, 8 or 16 chunks by r
  __device__ static inline int swz(int r) { return CPR == 4 ? (r >> 1) & 3 : r & (CPR - 1); }
  // element offset of channel chunk c of row r
  __device__ static inline int at(int r, int c) { return r * LDR + ((c ^ swz(r)) & (CPR - 1)) * EPC; }
  static constexpr int RM = BM / (16 * WM);
  static constexpr int RN = BN / (16 * WN);
  static constexpr int KS = BF16 ? 32 : 16;         // channels per MFMA step
  static constexpr int A_PER_T = BM * CPR / kBlock; // A chunks copied per thread
  static constexpr int B_PER_T = BN * CPR / kBlock;
  static constexpr int A_BYTES = BM * LDR * U;
  static constexpr int B_BYTES = BN * LDR * U;
  static constexpr int LDS_BYTES = 2 * (A_BYTES + B_BYTES) + kTaps * BM * 4 + 16;
  static_assert(WM * WN == kWaves, "four waves");
  static_assert(RM >= 1 && RN >= 1, "wave tile");
  static_assert(BM * CPR % kBlock == 0 && BN * CPR % kBlock == 0, "copy split");
  static_assert(kBlock % BM == 0 || BM % kBlock == 0, "table rows per thread");
  static_assert(CPR == 4 || CPR == 8 || CPR == 16, "chunk permutation");
  static_assert(KC % KS == 0 && KS * U == 64, "an MFMA step reads 4 chunks of a row");
};

// PRE: the pre-activation of the input (Group Normalization folded into a
// per-channel scale and shift, then a ReLU) is applied to every gathered
// input value of a neighbour that exists, as the stage is copied to LDS;
// pre holds Cin scales then Cin shifts.
// BUF: loads through buffer resources; else (operands beyond their reach)
// plain loads from valid addresses, replaced by zeros.
template <bool BF16, int BM, int BN, int WM, int WN, int KCB, int NS, bool BUF, bool PRE>
__global__ void __launch_bounds__(kBlock)
k_conv_lds(const int32_t* __restrict__ nbr, int64_t ldn, int64_t n_out, const void* __restrict__ in,
           int64_t ld_in, int Cin, const void* __restrict__ W, const float* __restrict__ bias, int Cout,
           int relu, void* __restrict__ out, int64_t ld_out, const int32_t* __restrict__ rows,
           unsigned row_tiles, uint32_t in_bytes, uint32_t w_bytes, const float* __restrict__ pre,
           const void* __restrict__ res, int64_t ld_res) {
  using P = LdsConv<BF16, BM, BN, WM, WN, KCB>;
  using E = typename std::conditional<BF16, uint16_t, float>::type;
  extern __shared__ __align__(16) unsigned char smem[];
  E* As = reinterpret_cast<E*>(smem);
  E* Bs = reinterpret_cast<E*>(smem + 2 * P::A_BYTES);
  // [tap][row]: byte offset of the neighbour's input row (BUF; kOutOfRange when
  // missing) or its number (-1 when missing)
  int32_t* nbt = reinterpret_cast<int32_t*>(smem + 2 * (P::A_BYTES + P::B_BYTES));
  uint32_t* used_s = reinterpret_cast<uint32_t*>(nbt + kTaps * BM);
  float* pre_s = reinterpret_cast<float*>(smem + P::LDS_BYTES);   // PRE: [Cin] scales, [Cin] shifts

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int li = lane & 15;
  const int lg = lane >> 4;
  // XCD-aware tile order: workgroup b runs on XCD b % 8; give each XCD a
  // contiguous range of (row tile, column tile) items, column tiles of a row
  // tile adjacent, so that the workgroups gathering the same input rows run
  // at the same time on one XCD and share its L2.
  const unsigned b = blockIdx.x;
  const unsigned col_tiles = (Cout + BN - 1) / BN;
  const unsigned items = row_tiles * col_tiles;
  const unsigned per_xcd = (items + 7) / 8;
  const unsigned item = (b % 8) * per_xcd + b / 8;
  if (item >= items) return;
  const unsigned tile = item / col_tiles;
  const int64_t row0 = static_cast<int64_t>(tile) * BM;
  const int col0 = static_cast<int>(item - tile * col_tiles) * BN;
  const int wm = wave % WM, wn = wave / WM;

  // The tile's neighbours.  Taps that no row of the tile uses are skipped:
  // their A rows are all zero.  Rows are multiplied independently, so the
  // result of a row does not depend on which other rows share its tile.
  if (tid == 0) *used_s = 0;
  if constexpr (PRE)
    for (int i = tid; i < 2 * Cin; i += kBlock) pre_s[i] = pre[i];
  constexpr int kTapStep = kBlock / BM > 0 ? kBlock / BM : 1;   // taps looked up side by side
  constexpr int kLook = (kTaps + kTapStep - 1) / kTapStep;
  {
    const int r = tid % BM, t0 = tid / BM;
    const bool in_tile = row0 + r < n_out;
    const int64_t v = in_tile ? (rows ? rows[row0 + r] : row0 + r) : 0;
    int32_t nb[kLook];
#pragma unroll
    for (int q = 0; q < kLook; ++q) {
      const int t = t0 + q * kTapStep;
      nb[q] = t < kTaps && in_tile ? nbr[t * ldn + v] : -1;
    }
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < kLook; ++q) {
      const int t = t0 + q * kTapStep;
      if (nb[q] >= 0) mine |= 1u << t;
      if (t < kTaps) {
        if constexpr (BUF)
          nbt[t * BM + r] = nb[q] >= 0 ? static_cast<int32_t>(nb[q] * ld_in * static_cast<int64_t>(sizeof(E))) : kOutOfRange;
        else
          nbt[t * BM + r] = nb[q];
      }
    }
    // the wave's taps, one lane each
    uint32_t wave_used = 0;
#pragma unroll
    for (int t = 0; t < kTaps; ++t)
      if (__ballot((mine >> t) & 1u)) wave_used |= 1u << t;
    __syncthreads();
    if (lane == 0 && wave_used) atomicOr(used_s, wave_used);
  }
  __syncthreads();
  // taps still to be fetched, in order (the same for every thread: scalar)
  uint32_t todo = __builtin_amdgcn_readfirstlane(*used_s);
  const int kc_steps = (Cin + P::KC - 1) / P::KC;
  const int stages = __builtin_popcount(todo) * kc_steps;

  // global -> register copies of one stage.  Every load is issued, also for
  // a missing neighbour, a channel past Cin or a stage past the last: with
  // buffer loads such a load gets an offset beyond the buffer and reads zeros
  // without touching memory.  With no load skipped, the number of loads in
  // flight is known, and the wait before a stage is copied to LDS covers that
  // stage's loads only, not the ones issued after it.
  using V = uint4;
  struct Stage {
    V a[P::A_PER_T], b[P::B_PER_T];
    int32_t nb[PRE ? P::A_PER_T : 1];   // PRE: the rows' table entries (negative: missing)
    int kc;
  };
  const __amdgpu_buffer_rsrc_t rin =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(in), 0, static_cast<int>(in_bytes), kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rw =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(W), 0, static_cast<int>(w_bytes), kRsrcWord3);
  // chunk cc of rows r0, r0 + kBlock / CPR, ... is this thread's
  const int cc = tid % P::CPR, cr = tid / P::CPR;
  constexpr int kRowStep = kBlock / P::CPR;
  const int cch = cc * P::EPC;
  int32_t boff[P::B_PER_T];   // byte offset of the weight rows' chunk (BUF), or the row times Cin
#pragma unroll
  for (int j = 0; j < P::B_PER_T; ++j) {
    const int col = col0 + cr + j * kRowStep;
    if constexpr (BUF) boff[j] = col < Cout ? (col * Cin + cch) * P::U : kOutOfRange;
    else boff[j] = col < Cout ? col : -1;
  }
  int32_t arow[P::A_PER_T];   // table entries of the next stage to fetch,
  int ft = 0, fkc = 0;        // its tap and first channel
  auto look = [&]() {
    ft = todo ? __builtin_ctz(todo) : 0;
#pragma unroll
    for (int j = 0; j < P::A_PER_T; ++j) arow[j] = nbt[ft * BM + cr + j * kRowStep];
  };
  look();
  auto fetch = [&](Stage& s) {
    // sign bit set where nothing is to be read.  (Opaque to the compiler: as a
    // condition it makes branches of the loads, and each branch waits for every
    // load in flight.)
    int32_t off_bit = todo != 0 && fkc + cch < Cin ? 0 : kOutOfRange;
    asm volatile("" : "+v"(off_bit));
    s.kc = fkc;
#pragma unroll
    for (int j = 0; j < P::A_PER_T; ++j) {
      if constexpr (BUF) {
        s.a[j] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rin, (arow[j] + cch * P::U) | off_bit,
                                                                              fkc * P::U, 0));
      } else {
        const bool on = (arow[j] | off_bit) >= 0;
        const V x = *reinterpret_cast<const V*>(static_cast<const E*>(in) + (on ? arow[j] * ld_in + fkc + cch : 0));
        s.a[j] = on ? x : make_uint4(0u, 0u, 0u, 0u);
      }
      if constexpr (PRE) s.nb[j] = arow[j] | off_bit;
    }
#pragma unroll
    for (int j = 0; j < P::B_PER_T; ++j) {
      if constexpr (BUF) {
        s.b[j] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rw, boff[j] | off_bit,
                                                                              (ft * Cout * Cin + fkc) * P::U, 0));
      } else {
        const bool on = (boff[j] | off_bit) >= 0;
        const V x = *reinterpret_cast<const V*>(static_cast<const E*>(W) +
                                                (on ? (static_cast<int64_t>(ft) * Cout + boff[j]) * Cin + fkc + cch : 0));
        s.b[j] = on ? x : make_uint4(0u, 0u, 0u, 0u);
      }
    }
    // the next stage: further channels of the tap, or the next tap
    fkc += P::KC;
    const bool wrap = fkc >= Cin;
    fkc = wrap ? 0 : fkc;
    todo = wrap ? todo & (todo - 1) : todo;
    look();
  };
  // a stage's copy from its registers to LDS buffer buf
  auto stash = [&](const Stage& s, int buf) {
    E* a = As + buf * (BM * P::LDR);
    E* bb = Bs + buf * (BN * P::LDR);
    float sc[P::EPC], sh[P::EPC];
    if constexpr (PRE) {
      const int ch = min(s.kc + cch, Cin - P::EPC);   // (past Cin: not used)
#pragma unroll
      for (int i = 0; i < P::EPC; i += 4) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(pre_s + ch + i), y = *reinterpret_cast<const f32x4*>(pre_s + Cin + ch + i);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          sc[i + q] = x[q];
          sh[i + q] = y[q];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < P::A_PER_T; ++j) {
      V v = s.a[j];
      if constexpr (PRE) {
        uint32_t w[4] = {v.x, v.y, v.z, v.w};
        const bool on = s.nb[j] >= 0;
        if constexpr (BF16) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float lo = fmaxf(fmaf(__uint_as_float(w[i] << 16), sc[2 * i], sh[2 * i]), 0.f);
            const float hi = fmaxf(fmaf(__uint_as_float(w[i] & 0xffff0000u), sc[2 * i + 1], sh[2 * i + 1]), 0.f);
            w[i] = on ? pack_bf16x2(lo, hi) : 0u;
          }
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            w[i] = on ? __float_as_uint(fmaxf(fmaf(__uint_as_float(w[i]), sc[i], sh[i]), 0.f)) : 0u;
        }
        v = make_uint4(w[0], w[1], w[2], w[3]);
      }
      *reinterpret_cast<V*>(a + P::at(cr + j * kRowStep, cc)) = v;
    }
#pragma unroll
    for (int j = 0; j < P::B_PER_T; ++j) *reinterpret_cast<V*>(bb + P::at(cr + j * kRowStep, cc)) = s.b[j];
  };

  // the lane's output rows
  int32_t out_row[P::RM];
#pragma unroll
  for (int i = 0; i < P::RM; ++i) {
    const int64_t r = row0 + (wm * P::RM + i) * 16 + li;
    out_row[i] = r < n_out ? (rows ? rows[r] : static_cast<int32_t>(r)) : -1;
  }

  // The products take the weights as their first operand, so that lane (i, g)
  // receives the 4 consecutive output channels 4 g .. 4 g + 3 of row i.
  f32x4 acc[P::RM][P::RN];
#pragma unroll
  for (int a = 0; a < P::RM; ++a)
#pragma unroll
    for (int c = 0; c < P::RN; ++c) acc[a][c] = f32x4{0.f, 0.f, 0.f, 0.f};

  // rows of a fragment are 16-aligned blocks plus li, so the permutation
  // of the lane's row is that of li: MFMA step k reads chunk 4 k + lg
  const E* a_base = As + (wm * P::RM * 16 + li) * P::LDR;
  const E* b_base = Bs + (wn * P::RN * 16 + li) * P::LDR;
  const int sw = P::swz(li);
  constexpr int NK = P::KC / P::KS;
  constexpr int N0 = (NK + 1) / 2, N1 = NK - N0;   // MFMA steps in the two halves of a stage
  struct Half {
    Frag<BF16> a[N0][P::RM], b[N0][P::RN];
  };
  // fragments of MFMA steps [K0, K0 + N) of LDS buffer buf
  auto read = [&](Half& h, int buf, auto k0_c, auto n_c) {
    constexpr int K0 = decltype(k0_c)::value, N = decltype(n_c)::value;
    const E* a = a_base + buf * (BM * P::LDR);
    const E* bb = b_base + buf * (BN * P::LDR);
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const int ck = (((4 * (K0 + k) + lg) ^ sw) & (P::CPR - 1)) * P::EPC;
#pragma unroll
      for (int i = 0; i < P::RM; ++i) h.a[k][i].load(a, i * 16 * P::LDR + ck);
#pragma unroll
      for (int j = 0; j < P::RN; ++j) h.b[k][j].load(bb, j * 16 * P::LDR + ck);
    }
  };
  auto multiply = [&](const Half& h, auto n_c) {
    constexpr int N = decltype(n_c)::value;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      if constexpr (BF16) {
#pragma unroll
        for (int i = 0; i < P::RM; ++i)
#pragma unroll
          for (int j = 0; j < P::RN; ++j) mma(acc[i][j], h.b[k][j], h.a[k][i]);
      } else {
        // interleave independent accumulators between dependent MFMAs
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < P::RM; ++i)
#pragma unroll
            for (int j = 0; j < P::RN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(h.b[k][j].v[e], h.a[k][i].v[e], acc[i][j], 0, 0, 0);
      }
    }
  };
  // One step of the pipeline: stage st is multiplied from LDS buffer st & 1 in
  // two halves whose fragments are read one half ahead, stage st + 2 is
  // requested, and stage st + 1 (requested a step ago) goes to the other
  // buffer.  Between the multiplications of a half, which keep the matrix core
  // busy for 32 (fp32) or 16 cycles each, the wave issues the half's other
  // instructions; the scheduling groups below ask for that order.
  Stage ss[NS];
  Half h0, h1;
  using C0 = std::integral_constant<int, 0>;
  using CN0 = std::integral_constant<int, N0>;
  using CN1 = std::integral_constant<int, N1>;
  static_for<NS>([&](auto i_c) { fetch(ss[decltype(i_c)::value]); });
  stash(ss[0], 0);
  __syncthreads();
  read(h0, 0, C0{}, CN0{});
  constexpr int kMfma0 = N0 * P::RM * P::RN * (BF16 ? 1 : 4);
  constexpr int kReads1 = N1 * (P::RM + P::RN);
  constexpr int kLoads = P::A_PER_T + P::B_PER_T;
  auto step = [&](Stage& mine, Stage& next, int buf) {
    fetch(mine);
    if constexpr (N1 > 0) read(h1, buf, CN0{}, CN1{});
    stash(next, buf ^ 1);
    multiply(h0, CN0{});
    if constexpr (BUF) {
      // per MFMA: one load or fragment read, then the copy to LDS
      constexpr int kSlots = kLoads + kReads1 + kLoads;
      static_for<kMfma0>([&](auto m_c) {
        constexpr int m = decltype(m_c)::value;
        constexpr int q0 = m * kSlots / kMfma0, q1 = (m + 1) * kSlots / kMfma0;
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        static_for<q1 - q0>([&](auto q_c) {
          constexpr int q = q0 + decltype(q_c)::value;
          if constexpr (q < kLoads) {
            __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
          } else if constexpr (q < kLoads + kReads1) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          } else {
            __builtin_amdgcn_sched_group_barrier(0x2, PRE ? 12 : 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
          }
        });
      });
    }
    __syncthreads();
    read(h0, buf ^ 1, C0{}, CN0{});
    if constexpr (N1 > 0) multiply(h1, CN1{});
  };
  // whole groups of NS steps without branches, then the remaining stages
  static_assert(NS % 2 == 0, "a group of steps leaves the LDS buffers as it found them");
  int st = 0;
  for (; st + NS <= stages; st += NS)
    static_for<NS>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      step(ss[i], ss[(i + 1) % NS], i & 1);
    });
  static_for<NS - 1>([&](auto i_c) {
    constexpr int i = decltype(i_c)::value;
    if (st + i < stages) step(ss[i], ss[(i + 1) % NS], i & 1);
  });

#pragma unroll
  for (int i = 0; i < P::RM; ++i) {
    if (out_row[i] < 0) continue;
    const int64_t row = out_row[i];
#pragma unroll
    for (int j = 0; j < P::RN; ++j) {
      const int col = col0 + (wn * P::RN + j) * 16 + 4 * lg;
      if (col >= Cout) continue;
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        v[r] = acc[i][j][r] + (bias ? bias[col + r] : 0.f);
        if (relu) v[r] = fmaxf(v[r], 0.f);
      }
      if constexpr (BF16) {
        if (res) {
          const uint2 x = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(res) + row * ld_res + col);
          v[0] += __uint_as_float(x.x << 16);
          v[1] += __uint_as_float(x.x & 0xffff0000u);
          v[2] += __uint_as_float(x.y << 16);
          v[3] += __uint_as_float(x.y & 0xffff0000u);
        }
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(out) + row * ld_out + col) =
            make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
      } else {
        if (res) {
          const float4 x = *reinterpret_cast<const float4*>(static_cast<const float*>(res) + row * ld_res + col);
          v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
        }
        *reinterpret_cast<float4*>(static_cast<float*>(out) + row * ld_out + col) = make_float4(v[0], v[1], v[2], v[3]);
      }
    }
  }
}

// Byte extents of the gathered operands, for the buffer resources.
struct ConvExtent {
  int64_t in_bytes, w_bytes;
  bool buffer_ok() const { return in_bytes <= kMaxBufferBytes && w_bytes <= kMaxBufferBytes; }
};

template <bool BF16, int BM, int BN, int WM, int WN, int KCB, int NS, bool PRE, bool BUF = true>
void conv_lds_launch(const int32_t* nbr, int64_t ldn, int64_t n_out, const void* in, int64_t ld_in,
                     int Cin, const void* W, const float* bias, int Cout, int relu, void* out,
                     int64_t ld_out, const int32_t* rows, ConvExtent ext, hipStream_t s, const float* pre,
                     const void* res, int64_t ld_res) {
  using P = LdsConv<BF16, BM, BN, WM, WN, KCB>;
  const int lds = P::LDS_BYTES + (PRE ? 8 * Cin : 0);
  static bool lds_limit_set = false;
  if (!lds_limit_set) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_conv_lds<BF16, BM, BN, WM, WN, KCB, NS, BUF, PRE>),
                              hipFuncAttributeMaxDynamicSharedMemorySize,
                              P::LDS_BYTES + (PRE ? 8 * kMaxPreChannels : 0));
    lds_limit_set = true;
  }
  const int64_t tiles = (n_out + BM - 1) / BM;
  const int64_t items = tiles * ((Cout + BN - 1) / BN);
  const unsigned per_xcd = static_cast<unsigned>((items + 7) / 8);
  launch((k_conv_lds<BF16, BM, BN, WM, WN, KCB, NS, BUF, PRE>), dim3(per_xcd * 8), dim3(kBlock), static_cast<uint32_t>(lds),
         s, nbr, ldn, n_out, in, ld_in, Cin, W, bias, Cout, relu, out, ld_out, rows, static_cast<unsigned>(tiles),
         static_cast<uint32_t>(BUF ? ext.in_bytes : 0), static_cast<uint32_t>(BUF ? ext.w_bytes : 0), pre, res, ld_res);
}

int64_t blocks_of(int64_t n_out, int Cout, int rows, int cols) {
  return ((n_out + rows - 1) / rows) * ((Cout + cols - 1) / cols);
}

// Tile choice, from sweeps over the lattices of LiDAR scans and of rooms on
// MI355X (us per convolution; tile rows x columns / bytes of channels a stage).
// fp32: at 900 tiles of 32 x 64 and more, stages of 32 channels (128->128 on 16k
// vertices: 48 against 53 for 64-channel stages and for 32 x 32; 128->64 Upsample
// into 212k: 60 against 75 and 63); from 500 tiles 64-channel stages: at 500 to
// 800 tiles pre-activated convolutions are 1 to 6% faster with them and plain ones
// 2 to 7% slower (256->256 on 6.4k vertices, 800 tiles: pre-activated 95 and 101,
// plain 79 and 78); below that, 32 x 32 tiles, as more workgroups matter more than
// the operand bytes per product (128->128 on 6.4k, 400 tiles: 26 against 27, on
// 4.4k, 274 tiles: 20 against 23; 256->256 on 2.3k: 37 against 46).  64 x 64 tiles
// were slower everywhere (down to one workgroup per compute unit, nothing hides a
// wave's own waits).  bf16: 128 x 128 tiles halve the gathered bytes per product
// and win once there are enough of them, with four stages in flight: from 400
// tiles for wide inputs (256->128 on 52k vertices, 410 tiles: 55 against 59 for 64
// x 64; 256->256 there 96 against 102, on 23k, 356 tiles, 49 against 47, on 2.3k,
// 36 tiles, 34 against 15; the ResNet block of 256 channels on 239k 1137 against
// 1226), from 1,500 for others; 128 x 64 for 64 output channels on large levels
// (half the weight rows per output row); 64 x 64 otherwise, with two stages in
// flight at any size (64->96 on 819k vertices: 325 with three stages of the former
// pipeline, 225 here).
// PRE (the pre-activated convolution) uses the same tiles, apart from the
// register kernel for narrow outputs, which has no pre-activation.
template <bool BF16, bool PRE>
void conv_dispatch(const int32_t* nbr, int64_t ldn, int64_t n_out, const void* in, int64_t ld_in,
                   int Cin, const void* W, const float* bias, int Cout, int relu, void* out,
                   int64_t ld_out, const int32_t* rows, ConvExtent ext, hipStream_t s, const float* pre,
                   const void* res, int64_t ld_res) {
  if (!PRE && !res && Cout <= 16)
    return conv_launch<BF16, 1, 1, 4, 1>(nbr, ldn, n_out, in, ld_in, Cin, W, bias, Cout, relu, out, ld_out, rows, s);
  auto go = [&](auto bm, auto bn, auto wm, auto wn, auto kcb, auto ns) {
    conv_lds_launch<BF16, decltype(bm)::value, decltype(bn)::value, decltype(wm)::value, decltype(wn)::value,
                    decltype(kcb)::value, decltype(ns)::value, PRE>(nbr, ldn, n_out, in, ld_in, Cin, W, bias, Cout, relu, out, ld_out, rows,
                                               ext, s, pre, res, ld_res);
  };
#define CONV_GO(BM, BN, WM, WN, KCB, NS)                                                                               \
  return go(std::integral_constant<int, BM>{}, std::integral_constant<int, BN>{}, std::integral_constant<int, WM>{},  \
            std::integral_constant<int, WN>{}, std::integral_constant<int, KCB>{}, std::integral_constant<int, NS>{})
  if (!ext.buffer_ok())  // operands beyond the reach of a buffer resource
    return conv_lds_launch<BF16, 64, 64, 2, 2, 128, 2, PRE, false>(nbr, ldn, n_out, in, ld_in, Cin, W, bias, Cout, relu, out,
                                                                ld_out, rows, ext, s, pre, res, ld_res);
  if constexpr (BF16) {
    const int64_t b128 = blocks_of(n_out, Cout, 128, 128);
    const int64_t b64 = blocks_of(n_out, Cout, 64, 64);
    if (Cout >= 128 && (b128 >= 1500 || (Cin >= 256 && Cout % 128 == 0 && b128 >= 400))) CONV_GO(128, 128, 2, 2, 64, 4);
    if (Cout == 64 && b64 >= 8192) CONV_GO(128, 64, 2, 2, 64, 2);
    if (Cout > 32 && b64 >= 256) CONV_GO(64, 64, 2, 2, 128, 2);
    CONV_GO(32, 32, 2, 2, 128, 2);
  } else {
    const int64_t b32x64 = blocks_of(n_out, Cout, 32, 64);
    if (Cout > 32 && b32x64 >= 900) CONV_GO(32, 64, 2, 2, 128, 2);
    if (Cout > 32 && b32x64 >= 500) CONV_GO(32, 64, 2, 2, 256, 2);
    if (blocks_of(n_out, Cout, 32, 32) >= 1024) CONV_GO(32, 32, 2, 2, 128, 2);
    CONV_GO(32, 32, 2, 2, 256, 2);
  }
#undef CONV_GO
}

}  // namespace

int conv_max_pre_channels() { return kMaxPreChannels; }

void launch_conv(const int32_t* nbr, int64_t ldn, int64_t n_out, int64_t n_in, const void* in, int64_t ld_in,
                 int Cin, const void* W, const float* bias, int Cout, int bf16, int relu, void* out,
                 int64_t ld_out, const int32_t* rows, hipStream_t s, const float* pre, const void* res,
                 int64_t ld_res) {
  if (n_out <= 0) return;
  ScopedKernelTimer tm("conv", s);
  const int64_t u = bf16 ? 2 : 4;
  const ConvExtent ext{n_in > 0 ? ((n_in - 1) * ld_in + Cin) * u : 0, int64_t{kTaps} * Cout * Cin * u};
  auto go = [&](auto bf_c, auto pre_c) {
    conv_dispatch<decltype(bf_c)::value, decltype(pre_c)::value>(nbr, ldn, n_out, in, ld_in, Cin, W, bias, Cout,
                                                                  relu, out, ld_out, rows, ext, s, pre, res, ld_res);
  };
  using T = std::true_type;
  using F = std::false_type;
  if (pre) bf16 ? go(T{}, T{}) : go(F{}, T{});
  else bf16 ? go(T{}, F{}) : go(F{}, F{});
}

}  // namespace lat

// The predictor on a tile of MT windows as device code (gfx950), shared by
// the step, forward and training-forward kernels: precision forms, LDS
// layout, conv levels as MFMA GEMMs, the hidden FC, the heads, and a window
// row's way from memory to LDS.
#pragma once
#include <type_traits>

#include "simnet_internal.h"

namespace simnet {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// ------------------------------------------------------ precision forms ---
// Each form stores activations and weights as T and multiplies one 16-byte
// fragment per lane per call of mma(): lane group g = lane/16 holds KG/4
// consecutive k of its row (A) or column (B); A and B use the same
// assignment, so every call adds the full KG-long partial dot products.

// Acc: the accumulator of one MFMA tile; TILE: its side; col4(g, lane):
// the first of the 4 consecutive output columns (weight-first operand
// order: the weights' N) that accumulator elements 4g .. 4g+3 of the lane
// hold, for the activation row lane % TILE.
struct PF32 {
  using T = float;
  using Acc = v4f;
  static constexpr int ID = 0, KG = 16, TILE = 16;
  __device__ static int col4(int, int lane) { return 4 * (lane >> 4); }
  static constexpr bool SCALED = false;
  __device__ static v4f mma(v4f c, uint4 a, uint4 b) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    return c;
  }
  __device__ static T cvt(float x) { return x; }
  __device__ static float val(T x) { return x; }
};

struct PBF16 {
  using T = uint16_t;  // bfloat16 bits
  using Acc = v4f;
  static constexpr int ID = 1, KG = 32, TILE = 16;
  __device__ static int col4(int, int lane) { return 4 * (lane >> 4); }
  static constexpr bool SCALED = false;
  __device__ static v4f mma(v4f c, uint4 a, uint4 b) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a),
                                                   __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
  }
  // round to nearest even (inputs are finite)
  __device__ static T cvt(float x) {
    const uint32_t u = __float_as_uint(x);
    return (T)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
  }
  __device__ static float val(T x) { return __uint_as_float((uint32_t)x << 16); }
};

struct PFP8 {
  using T = uint8_t;  // OCP e4m3 (max 448)
  using Acc = v4f;
  static constexpr int ID = 2, KG = 64, TILE = 16;
  __device__ static int col4(int, int lane) { return 4 * (lane >> 4); }
  static constexpr bool SCALED = true;
  __device__ static v4f mma(v4f c, uint4 a, uint4 b) {
    const long a0 = ((long)a.y << 32) | a.x, a1 = ((long)a.w << 32) | a.z;
    const long b0 = ((long)b.y << 32) | b.x, b1 = ((long)b.w << 32) | b.z;
    c = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a0, b0, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a1, b1, c, 0, 0, 0);
    return c;
  }
  // round to nearest even, saturating at +-448
  __device__ static T cvt(float x) {
    x = fminf(fmaxf(x, -448.f), 448.f);
    return (T)(__builtin_amdgcn_cvt_pk_fp8_f32(x, 0.f, 0, false) & 0xff);
  }
  __device__ static float val(T x) { return __builtin_amdgcn_cvt_f32_fp8((int)x, 0); }
};

// BF16 on 32x32x16 tiles: the same storage, twice the FLOP per MFMA
// (32,768).  Lane l holds 8 consecutive k (8 * (l / 32) ..) of row l % 32 of
// either operand; the 16 accumulators of lane l are output columns
// 8 * (i / 4) + 4 * (l / 32) + i % 4 of row l % 32.  On gfx950 this
// instruction issues back to back where the 16x16x32 one leaves gaps.
struct PBF16W : PBF16 {
  using Acc = v16f;
  static constexpr int KG = 16, TILE = 32;
  __device__ static int col4(int g, int lane) { return 8 * g + 4 * (lane >> 5); }
  __device__ static v16f mma(v16f c, uint4 a, uint4 b) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a),
                                                   __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
  }
};

// Blocks per group: the window is processed a group of NG consecutive
// blocks at a time (the conv levels as one GEMM over all the group's
// positions, so each weight fragment serves NG times more rows), as many as
// the form's LDS budget allows beside the queue rings.
template <class Net, class P>
constexpr int group_blocks() {
  // (store latencies: the stores' ring takes LDS, so smaller groups)
  return Net::NCONV == 2 ? Net::NB : Net::MWQ ? (P::ID == 0 ? 1 : 2) : (P::ID == 0 ? 2 : 4);
}

template <class Net, class P>
struct Geo {
  using T = typename P::T;
  static constexpr int NT = Net::WAVES * 64;
  static constexpr int NG = group_blocks<Net, P>();
  static constexpr int PAD = 16 / sizeof(T);                       // 16 bytes of padding
  static constexpr int DP = padded_feat(Net::D, P::ID);            // features per slot
  // A conv reads rows of two consecutive input positions; each such pair is
  // followed by 16 bytes of padding, so the 16 rows of an MFMA tile (16
  // positions) fall in different LDS banks.  R* = elements per pair.
  static constexpr int RX = 2 * DP + PAD;                          // slot pair (conv1 row)
  static constexpr int R1 = 2 * Net::CH1 + PAD;                    // conv1 output pair
  static constexpr int R2 = 2 * Net::CH2 + PAD;                    // conv2 output pair (C3)
  static constexpr int SX = (NG * Net::BS / 2) * RX + PAD;         // a group's window rows, per window
  static constexpr int SA1 = (NG * Net::BS / 4) * R1 + PAD;        // conv1 output
  static constexpr int SA2 = Net::NCONV == 3 ? (NG * Net::BS / 8) * R2 + PAD  // conv2 output
                                             : NG * Net::CH2 + PAD;  // (last conv: flat)
  static constexpr int SA3 = (Net::NCONV == 3 ? NG * Net::CH3 : 0) + PAD;  // conv3 output (flat)
  static constexpr int SAL = Net::NCONV == 3 ? SA3 : SA2;          // last conv output
  // three conv levels: X and conv2's output share memory (X is dead once
  // conv1 has read it), and so do conv1's and conv3's outputs
  static constexpr bool ALIAS = Net::NCONV == 3;
  static constexpr int NXA2 = ALIAS ? (SX > SA2 ? MT * SX : MT * SA2) : MT * SX;
  static constexpr int NA1A3 = ALIAS ? (SA1 > SA3 ? MT * SA1 : MT * SA3) : MT * SA1;
  static constexpr int NA2 = ALIAS ? PAD : MT * SA2;
};

template <class Net, class P>
struct NetSmem {
  using G = Geo<Net, P>;
  // window rows of the group (X), then conv2's output; after the last group
  // also the final FC's cross-wave partial sums
  alignas(16) typename P::T xa2[G::NXA2];
  alignas(16) typename P::T a1a3[G::NA1A3]; // conv1's output, then conv3's output
  alignas(16) typename P::T a2own[G::NA2];  // conv2's output when it does not alias X
  float logit[MT][Net::NOUT];
  float x_inv[Net::D];  // FP8: reciprocal input scale of each window feature
  // The final FC on the VALU after the hidden layer (regression head): its
  // operands copied here once per launch (stage_head), so the end of every
  // prediction reads no global memory.  hb: hidden bias; FP8 hws, hai: the
  // hidden layer's weight and output scales; lw: final weights [NOUT][HID];
  // lb: final bias.
  static constexpr bool HL = Net::HID > 0 && Net::HEAD == 0;
  static constexpr int HLN = HL ? Net::HID : 1, HLS = HL && P::SCALED ? Net::HID : 1;
  float hb[HLN], hws[HLS], hai[HLS], lw[HL ? Net::NOUT * Net::HID : 1], lb[Net::NOUT];
  __device__ void stage_head(const DevWeights& wt, int tid, int nt) {
    if constexpr (HL) {
      // (weights without a final FC, as the training form's trunk has, leave
      // it unstaged: kernels that run the final FC are never given them)
      if (!wt.last_w || !wt.last_b || !wt.hid_b) return;
      for (int i = tid; i < Net::HID; i += nt) {
        hb[i] = wt.hid_b[i];
        if constexpr (P::SCALED) {
          hws[i] = wt.hid_ws[i];
          hai[i] = wt.hid_ai[i];
        }
      }
      for (int i = tid; i < Net::NOUT * Net::HID; i += nt) lw[i] = wt.last_w[i];
      for (int i = tid; i < Net::NOUT; i += nt) lb[i] = wt.last_b[i];
    }
  }
  __device__ typename P::T* x() { return xa2; }
  __device__ typename P::T* a1() { return a1a3; }
  __device__ typename P::T* a2() { return G::ALIAS ? xa2 : a2own; }
  __device__ typename P::T* a3() { return a1a3; }
  // [WAVES][MT][NOUT] partial sums of the final FC (X is dead by then)
  __device__ float* red() { return reinterpret_cast<float*>(xa2); }
  static_assert(Net::HID == 0 || sizeof(xa2) >= sizeof(float) * Net::WAVES * MT * Net::NOUT,
                "final-FC partial sums do not fit X's region");
};

// Epilogue of one accumulator element: bias, (FP8) dequantisation, ReLU.
template <class P>
__device__ __forceinline__ float activation(float acc, int col, const float* bias, const float* ws,
                                            bool relu) {
  float v;
  if constexpr (P::SCALED)
    v = fmaf(acc, ws[col], bias[col]);
  else
    v = acc + bias[col];
  return relu ? fmaxf(v, 0.f) : v;
}
// ... then (FP8) the next layer's input scale and conversion to storage.
template <class P>
__device__ __forceinline__ typename P::T to_storage(float v, int col, const float* ai) {
  if constexpr (P::SCALED) v *= ai[col];
  return P::cvt(v);
}
// The same two with the column's bias b, weight scale s and input scale a
// already in registers.
template <class P>
__device__ __forceinline__ float activation_v(float acc, float b, float s, bool relu) {
  float v;
  if constexpr (P::SCALED)
    v = fmaf(acc, s, b);
  else
    v = acc + b;
  return relu ? fmaxf(v, 0.f) : v;
}
template <class P>
__device__ __forceinline__ typename P::T to_storage_v(float v, float a) {
  if constexpr (P::SCALED) v *= a;
  return P::cvt(v);
}
// Calibration: running per-channel max of |activation| (LDS, as ordered bits).
__device__ __forceinline__ void cal_max(unsigned* cal, int i, float v) {
  atomicMax(cal + i, __float_as_uint(fabsf(v)));
}

// k-groups per chunk when streaming B: a chunk is at most FRAGS fragments
// (4 VGPRs each) and two chunks are in flight; must divide the k-groups.
constexpr int stream_chunk(int kgs, int tpw, int frags = 8) {
  int c = frags / tpw;
  if (c < 1) c = 1;
  if (c > kgs) c = kgs;
  while (kgs % c) --c;
  return c;
}

// One 16-byte weight fragment through a raw buffer load: the resource and
// the fragment's offset are wave-uniform (scalar registers), only the lane's
// 16-byte offset is per lane, so many fragments can be in flight without a
// 64-bit address register each.
__device__ __forceinline__ uint4 load_frag(__amdgpu_buffer_rsrc_t r, int lane_off, int frag_off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, frag_off, 0));
}

// Workgroup barrier ordering LDS only: global loads in flight (weight
// prefetches) stay in flight across it (__syncthreads waits for them).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t frag_rsrc(const uint4* Bp, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(Bp), (short)0, bytes, 0x00020000);
}

// The first chunk of a weight stream (see mma_stream), requested ahead of
// the stream: before the barrier that precedes it, so that its L2 latency
// passes during the barrier and the previous phase's tail instead of
// stalling every wave at the start of the phase.
template <int CH, int NPW>
struct StreamHead {
  uint4 b[CH][NPW];
};

template <int KGS, int NTILES, int NPW, int FRAGS = 8>
__device__ __forceinline__ StreamHead<stream_chunk(KGS, NPW, FRAGS), NPW> stream_head(
    const uint4* __restrict__ Bp, int nt0, int lane) {
  constexpr int CH = stream_chunk(KGS, NPW, FRAGS);
  const __amdgpu_buffer_rsrc_t rs = frag_rsrc(Bp, KGS * NTILES * 1024);
  const int lo = lane * 16;
  const int wn = __builtin_amdgcn_readfirstlane(nt0) * 1024;
  StreamHead<CH, NPW> h;
#pragma unroll
  for (int kg = 0; kg < CH; ++kg)
#pragma unroll
    for (int j = 0; j < NPW; ++j) h.b[kg][j] = load_frag(rs, lo, wn + (kg * NTILES + j) * 1024);
  return h;
}

// acc[i][j] += W(tile nt0 + j) x A(m-tile i: this lane's row of it), all K.
// The weight fragment is the MFMA's first operand, so lane l ends up
// holding row l % 16 of the activations and output columns 4*(l/16) .. +3
// of the tile: consecutive columns, stored with one vector write.  Each
// weight fragment serves MPW m-tiles.  Weight fragments are requested
// DEPTH - 1 chunks ahead of their use (DEPTH buffers) and the scheduler is
// kept from sinking the requests.  HEAD: the first chunk was requested by
// stream_head (same KGS, NTILES, NPW, FRAGS, Bp and nt0) and is passed in.
template <class P, int KGS, int NTILES, int NPW, int MPW, int FRAGS = 8, bool HEAD = false,
          int DEPTH = 2>
__device__ __forceinline__ void mma_stream(
    typename P::Acc (&acc)[MPW][NPW], const typename P::T* const (&ap)[MPW],
    const uint4* __restrict__ Bp, int nt0, int lane,
    const StreamHead<stream_chunk(KGS, NPW, FRAGS), NPW>* head = nullptr) {
  constexpr int CH = stream_chunk(KGS, NPW, FRAGS), NCH = KGS / CH;
  const __amdgpu_buffer_rsrc_t rs = frag_rsrc(Bp, KGS * NTILES * 1024);
  const int lo = lane * 16;
  const int wn = __builtin_amdgcn_readfirstlane(nt0) * 1024;
  uint4 b[DEPTH][CH][NPW];
  auto request = [&](int c) {
#pragma unroll
    for (int kg = 0; kg < CH; ++kg)
#pragma unroll
      for (int j = 0; j < NPW; ++j)
        b[c % DEPTH][kg][j] = load_frag(rs, lo, wn + ((c * CH + kg) * NTILES + j) * 1024);
  };
  if constexpr (HEAD) {
#pragma unroll
    for (int kg = 0; kg < CH; ++kg)
#pragma unroll
      for (int j = 0; j < NPW; ++j) b[0][kg][j] = head->b[kg][j];
  } else {
    request(0);
  }
#pragma unroll
  for (int c = 1; c < DEPTH - 1 && c < NCH; ++c) request(c);
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    if (c + DEPTH - 1 < NCH) request(c + DEPTH - 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kg = 0; kg < CH; ++kg) {
#pragma unroll
      for (int i = 0; i < MPW; ++i) {
        const uint4 a = *reinterpret_cast<const uint4*>(ap[i] + (c * CH + kg) * P::KG);
#pragma unroll
        for (int j = 0; j < NPW; ++j) acc[i][j] = P::mma(acc[i][j], b[c % DEPTH][kg][j], a);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// N consecutive storage elements written with the widest stores the
// destination's alignment (ALIGN bytes) allows.
template <int ALIGN, class T, int N>
__device__ __forceinline__ void store_run(T* dst, const T (&e)[N]) {
  constexpr int BYTES = N * (int)sizeof(T);
  constexpr int W = (ALIGN % 16 == 0 && BYTES % 16 == 0) ? 16
                    : (ALIGN % 8 == 0 && BYTES % 8 == 0) ? 8
                    : (ALIGN % 4 == 0 && BYTES % 4 == 0) ? 4 : (int)sizeof(T);
  uint32_t w[(BYTES + 3) / 4];
  __builtin_memcpy(w, e, BYTES);
  char* d = reinterpret_cast<char*>(dst);
#pragma unroll
  for (int o = 0; o < BYTES; o += W) {
    if constexpr (W == 16)
      *reinterpret_cast<uint4*>(d + o) = uint4{w[o / 4], w[o / 4 + 1], w[o / 4 + 2], w[o / 4 + 3]};
    else if constexpr (W == 8)
      *reinterpret_cast<uint2*>(d + o) = uint2{w[o / 4], w[o / 4 + 1]};
    else if constexpr (W == 4)
      *reinterpret_cast<uint32_t*>(d + o) = w[o / 4];
    else
      *reinterpret_cast<T*>(d + o) = e[o / sizeof(T)];
  }
}

// Waves along N for a conv level: two N tiles per wave where there are
// enough (each A fragment read from LDS then serves two MFMAs, each B
// fragment from L2 serves the wave's M tiles), and never more waves along M
// than there are M tiles.
constexpr int conv_wave_split(int ntiles, int mtiles, int waves) {
  int wn = ntiles / 2 < 1 ? 1 : ntiles / 2 < waves ? ntiles / 2 : waves;
  while (waves / wn > mtiles || waves % wn) wn *= 2;
  return wn;
}

// The tiling of one conv level as a GEMM (see conv_stage): MT windows x POS
// output positions of rows, N output channels, contraction K; the waves'
// split over N and M tiles and the type of the stream's first chunk.
template <class P, int K, int N, int POS, int WAVES>
struct ConvShape {
  static constexpr int ROWS = MT * POS;
  static constexpr int MTILES = ROWS / 16, NTILES = N / 16, KGS = K / P::KG;
  static constexpr int WN = conv_wave_split(NTILES, MTILES, WAVES), WM = WAVES / WN;
  static constexpr int MPW = MTILES / WM, NPW = NTILES / WN;
  static_assert(ROWS % 16 == 0 && N % 16 == 0 && K % P::KG == 0, "tile shape");
  static_assert(WAVES % WN == 0 && MTILES % WM == 0 && NTILES % WN == 0 && MPW >= 1,
                "wave split");
  // weight fragments per chunk: the BF16 form's conv levels run 1.3 %
  // faster with 16 (measured); FP32 and FP8 gain nothing
  static constexpr int FRAGS = P::ID == 1 ? 16 : 8;
  using Head = StreamHead<stream_chunk(KGS, NPW, FRAGS), NPW>;
};

// The first chunk of a conv level's weight stream for this wave (see
// StreamHead), requested ahead of conv_stage<..., HEAD = true>.
template <class P, int K, int N, int POS, int WAVES>
__device__ __forceinline__ typename ConvShape<P, K, N, POS, WAVES>::Head conv_head(
    const void* Bp, int wave, int lane) {
  using S = ConvShape<P, K, N, POS, WAVES>;
  return stream_head<S::KGS, S::NTILES, S::NPW, S::FRAGS>(static_cast<const uint4*>(Bp),
                                                (wave % S::WN) * S::NPW, lane);
}

// One conv level as a GEMM: rows (s, q) = MT windows x POS output positions,
// A row (s, q) is the K = 2*C_in contiguous elements of input positions 2q,
// 2q+1 at A + s*SA + q*IRS; output row (s, q) goes to O + s*SO + q*N, or,
// OPAIR, to O + s*SO + (q/2)*(2N + 16 bytes) + (q%2)*N (the padded pair
// layout the next conv reads).  The
// waves split the N tiles (conv_wave_split), then the M tiles; a wave runs
// MPW x NPW tiles.
// SAVE: also store each output row (s, q) to sv + s*sv_s + q*N (rows with
// s < sv_rows only), the layer's activations kept for the backward pass.
// Rows are numbered position-major, row = q * MT + s: an MFMA tile's 16
// rows are 16 windows at one position, whose window strides spread them
// over the LDS banks (the position stride of a wide level is a multiple of
// the bank count, so window-major tiles would collide).
// HEAD: the weight stream's first chunk was requested by conv_head and is
// passed in (head).
template <class P, int K, int N, int POS, int WAVES, int SA, int IRS, int SO, bool OPAIR,
          bool CAL = false, bool SAVE = false, bool HEAD = false>
__device__ __forceinline__ void conv_stage(
    const typename P::T* __restrict__ A, typename P::T* __restrict__ O,
    const uint4* __restrict__ Bp, const float* __restrict__ bias, const float* __restrict__ ws,
    const float* __restrict__ ai, bool relu, int wave, int lane, unsigned* cal = nullptr,
    const int* row_live = nullptr, typename P::T* sv = nullptr, int64_t sv_s = 0,
    int sv_rows = 0, const typename ConvShape<P, K, N, POS, WAVES>::Head* head = nullptr) {
  using T = typename P::T;
  using S = ConvShape<P, K, N, POS, WAVES>;
  constexpr int MTILES = S::MTILES, NTILES = S::NTILES, KGS = S::KGS;
  constexpr int WN = S::WN, MPW = S::MPW, NPW = S::NPW;
  (void)MTILES;
  const int wm = wave / WN, wn = wave % WN;
  const int nt0 = wn * NPW;
  const T* ap[MPW];
#pragma unroll
  for (int i = 0; i < MPW; ++i) {
    const int row = (wm * MPW + i) * 16 + (lane & 15);
    ap[i] = A + (row % MT) * SA + (row / MT) * IRS + (P::KG / 4) * (lane >> 4);
  }
  v4f acc[MPW][NPW];
#pragma unroll
  for (int i = 0; i < MPW; ++i)
#pragma unroll
    for (int j = 0; j < NPW; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  // the epilogue's operands for this lane's 4 columns of each tile, requested
  // before the products: after them, the wait for these loads would also
  // wait for every weight request in flight behind them
  constexpr int NS = P::SCALED ? NPW : 1;
  v4f eb[NPW], es[NS] = {}, ea[NS] = {};
#pragma unroll
  for (int j = 0; j < NPW; ++j) {
    const int col0 = (nt0 + j) * 16 + 4 * (lane >> 4);
    eb[j] = *reinterpret_cast<const v4f*>(bias + col0);
    if constexpr (P::SCALED) {
      es[j] = *reinterpret_cast<const v4f*>(ws + col0);
      ea[j] = *reinterpret_cast<const v4f*>(ai + col0);
    }
  }
  mma_stream<P, KGS, NTILES, NPW, MPW, S::FRAGS, HEAD>(acc, ap, Bp, nt0, lane, head);
#pragma unroll
  for (int i = 0; i < MPW; ++i) {
    const int row = (wm * MPW + i) * 16 + (lane & 15);
    constexpr int ORS = 2 * N + 16 / (int)sizeof(T);
    const int q = row / MT, s = row % MT;
    T* orow = O + s * SO + (OPAIR ? (q >> 1) * ORS + (q & 1) * N : q * N);
    const bool live = !CAL || row_live[s];
#pragma unroll
    for (int j = 0; j < NPW; ++j) {
      const int col0 = (nt0 + j) * 16 + 4 * (lane >> 4);
      T e[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float v = activation_v<P>(acc[i][j][q], eb[j][q], es[P::SCALED ? j : 0][q], relu);
        if constexpr (CAL)
          if (live) cal_max(cal, col0 + q, v);
        e[q] = to_storage_v<P>(v, ea[P::SCALED ? j : 0][q]);
      }
      store_run<4 * sizeof(T)>(orow + col0, e);
      if constexpr (SAVE)
        if (s < sv_rows) store_run<4 * sizeof(T)>(sv + s * sv_s + q * N + col0, e);
    }
  }
}

// Activations kept for the backward pass (training form, SAVE): per window
// b, channels-last, in storage precision: a1 [NB*BS/2][CH1], a2
// [NB*BS/4][CH2], a3 [NB][CH3], h [HID]; pointers already at the tile's
// first window, rows = windows of the tile that exist.
template <class T>
struct SavePtrs {
  T *a1, *a2, *a3, *h;
  int rows;
};

// Index of the hidden FC in the layer list (after the convs and the
// residual blocks' two pointwise layers each): its ReLU bit.
template <class Net>
constexpr int hidden_layer() {
  return Net::NCONV + 2 * Net::NRES;
}

// The hidden FC's weight stream for a group of NBG blocks (see hidden_fc):
// HT output tiles per wave, KGS k-groups, the packed weights' address.  CS:
// the workgroup computes one of CS equal slices of the output columns (the
// split step), wave w the tiles fc_tile0 .. + HT - 1.
template <class Net, class P, int NBG, int CS = 1>
struct FcShape {
  static constexpr int HT = (Net::HID / 16) / Net::WAVES / CS;
  static constexpr int KGS = NBG * Net::CHL / P::KG;
  using Head = StreamHead<stream_chunk(KGS, HT, Net::FC1_FRAGS), HT>;
  // the packed weights of blocks j0 .. j0 + NBG - 1
  static __device__ __forceinline__ const uint4* weights(const DevWeights& wt, int j0) {
    return static_cast<const uint4*>(wt.hid_w) +
           (size_t)j0 * (Net::CHL / P::KG) * (Net::HID / 16) * 64;
  }
  static __device__ __forceinline__ int tile0(int slice, int wave) {
    return slice * (Net::HID / 16 / CS) + wave * HT;
  }
};

// The first chunk of hidden_fc<..., HEAD = true>'s weight stream (see
// StreamHead).
template <class Net, class P, int NBG, int CS = 1>
__device__ __forceinline__ typename FcShape<Net, P, NBG, CS>::Head fc_head(const DevWeights& wt,
                                                                          int j0, int wave,
                                                                          int lane,
                                                                          int slice = 0) {
  using S = FcShape<Net, P, NBG, CS>;
  return stream_head<S::KGS, Net::HID / 16, S::HT, Net::FC1_FRAGS>(S::weights(wt, j0),
                                                                  S::tile0(slice, wave), lane);
}

// Hidden-FC contribution of NBG blocks from block j0: last = the blocks'
// last-conv output in LDS (window s at s * SAL, block-major), hacc += it
// times the per-block packed weights.  A fresh accumulator per group, then
// added, so the FP32 chain is per group.  HEAD: the stream's first chunk
// was requested by fc_head and is passed in (head).  The sums of one group
// do not depend on which workgroup or column slice computes them.
template <class Net, class P, int NBG, bool HEAD = false, int CS = 1>
__device__ __forceinline__ void hidden_fc(
    const DevWeights& wt, const typename P::T* last, int j0, v4f* hacc, int wave, int lane,
    const typename FcShape<Net, P, NBG, CS>::Head* head = nullptr, int slice = 0) {
  using G = Geo<Net, P>;
  using T = typename P::T;
  using S = FcShape<Net, P, NBG, CS>;
  constexpr int HT = S::HT;
  const T* const ap[1] = {last + (lane & 15) * G::SAL + (P::KG / 4) * (lane >> 4)};
  v4f bacc[1][HT];
#pragma unroll
  for (int jj = 0; jj < HT; ++jj) bacc[0][jj] = v4f{0.f, 0.f, 0.f, 0.f};
  mma_stream<P, S::KGS, Net::HID / 16, HT, 1, Net::FC1_FRAGS, HEAD, Net::FC1_DEPTH>(
      bacc, ap, S::weights(wt, j0), S::tile0(slice, wave), lane, head);
#pragma unroll
  for (int jj = 0; jj < HT; ++jj) hacc[jj] += bacc[0][jj];
}

// The conv levels and the hidden-FC (or final-FC) contribution of one group
// of NBG blocks starting at block j0, for the tile of MT windows whose
// window rows are in sm.x().  relu_mask bit l = ReLU after layer l.  Ends
// with the group's last-conv output consumed.  issue() requests the next
// group's rows into registers before the last conv level and finish(regs)
// writes them into sm.x() (the region conv2's output used, dead once the
// last level has read it) before the FC.  With three conv levels the first
// weight chunk of conv2, conv3 and the FC is requested before the barrier
// that precedes it (StreamHead) and the barriers order LDS only, so the
// requests stay in flight across them.  (Requesting conv1's across the
// group boundary as well made the hidden-FC stream spill registers.)
// TRUNK: the convolutions only, the last conv's output going to sv.a3 (a1
// and a2 are not written).  CS, slice: the hidden FC's column slice (hacc
// holds FcShape<..., CS>::HT tiles).
template <class Net, class P, int NBG, bool CAL, bool SAVE, bool TRUNK, int CS = 1, class Issue,
          class Finish>
__device__ __forceinline__ void run_group(
    const DevWeights& wt, uint32_t relu_mask, NetSmem<Net, P>& sm, int j0, unsigned* cal,
    const int* row_live, SavePtrs<typename P::T> sv, v4f* hacc, float& fpart, Issue&& issue,
    Finish&& finish, int slice = 0) {
  using G = Geo<Net, P>;
  using T = typename P::T;
  constexpr bool XPF = Net::NCONV == 3;  // weight streams requested across the barriers
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  constexpr int P1 = NBG * Net::BS / 2, P2 = NBG * Net::BS / 4;
  constexpr int Q1 = Net::BS / 2, Q2 = Net::BS / 4;  // positions per block
  conv_stage<P, 2 * G::DP, Net::CH1, P1, Net::WAVES, G::SX, G::RX, G::SA1, true, CAL,
             SAVE && !TRUNK>(
      sm.x(), sm.a1(), static_cast<const uint4*>(wt.conv_w[0]), wt.conv_b[0], wt.conv_ws[0],
      wt.conv_ai[0], relu_mask & 1u, wave, lane, cal + Net::D, row_live,
      sv.a1 + (size_t)j0 * Q1 * Net::CH1, (int64_t)Net::NB * Q1 * Net::CH1, sv.rows);
  typename ConvShape<P, 2 * Net::CH1, Net::CH2, P2, Net::WAVES>::Head h2;
  if constexpr (XPF) {
    h2 = conv_head<P, 2 * Net::CH1, Net::CH2, P2, Net::WAVES>(wt.conv_w[1], wave, lane);
    lds_barrier();
  } else {
    __syncthreads();
  }
  conv_stage<P, 2 * Net::CH1, Net::CH2, P2, Net::WAVES, G::SA1, G::R1, G::SA2, Net::NCONV == 3,
             CAL, SAVE && !TRUNK, XPF>(
      sm.a1(), sm.a2(), static_cast<const uint4*>(wt.conv_w[1]), wt.conv_b[1], wt.conv_ws[1],
      wt.conv_ai[1], relu_mask & 2u, wave, lane, cal + Net::D + Net::CH1, row_live,
      sv.a2 + (size_t)j0 * Q2 * Net::CH2, (int64_t)Net::NB * Q2 * Net::CH2, sv.rows, &h2);
  if constexpr (Net::NCONV == 3) {
    auto h3 = conv_head<P, 2 * Net::CH2, Net::CH3, NBG, Net::WAVES>(wt.conv_w[2], wave, lane);
    lds_barrier();
    // the next group's rows are requested now, held through conv3 and
    // written once conv3 has read conv2's output (X's region), so the FC's
    // weight stream has the registers to itself
    auto next_rows = issue();
    conv_stage<P, 2 * Net::CH2, Net::CH3, NBG, Net::WAVES, G::SA2, G::R2, G::SA3, false, CAL,
               SAVE, true>(
        sm.a2(), sm.a3(), static_cast<const uint4*>(wt.conv_w[2]), wt.conv_b[2], wt.conv_ws[2],
        wt.conv_ai[2], relu_mask & 4u, wave, lane, cal + Net::D + Net::CH1 + Net::CH2, row_live,
        sv.a3 + (size_t)j0 * Net::CH3, (int64_t)Net::NB * Net::CH3, sv.rows, &h3);
    if constexpr (!TRUNK && Net::HID > 0) {
      // hidden FC over the group's NBG*CHL inputs per window (block-major,
      // as the packed per-block matrices are consecutive)
      auto hf = fc_head<Net, P, NBG, CS>(wt, j0, wave, lane, slice);
      lds_barrier();
      if constexpr (!Net::LATE_COMMIT) finish(next_rows);
      hidden_fc<Net, P, NBG, true, CS>(wt, sm.a3(), j0, hacc, wave, lane, &hf, slice);
      if constexpr (Net::LATE_COMMIT) finish(next_rows);
      return;
    }
    lds_barrier();
    finish(next_rows);
  } else {
    __syncthreads();
  }
  const T* last = Net::NCONV == 3 ? sm.a3() : sm.a2();
  if constexpr (TRUNK) {
    (void)last;
  } else if constexpr (Net::HID > 0) {
    hidden_fc<Net, P, NBG>(wt, last, j0, hacc, wave, lane);
  } else {
    // final FC on the VALU straight after the convs: (s, o) pairs, LPP lanes
    // each; the next group's rows are requested before it and written after
    constexpr int LPP = G::NT / (MT * Net::NOUT);
    constexpr int CPL = Net::CHL / LPP;
    const int fpair = tid / LPP, fsub = tid % LPP;
    const int fs = fpair / Net::NOUT, fo = fpair % Net::NOUT;
    auto next_rows = issue();
#pragma unroll
    for (int jb = 0; jb < NBG; ++jb) {
      const float* wrow = wt.last_w + ((size_t)(j0 + jb) * Net::NOUT + fo) * Net::CHL + fsub * CPL;
      const T* arow = last + fs * G::SAL + jb * Net::CHL + fsub * CPL;
#pragma unroll
      for (int c = 0; c < CPL; ++c) fpart = fmaf(P::val(arow[c]), wrow[c], fpart);
    }
    finish(next_rows);
  }
}

// Hybrid head (NOUT outputs) after the hidden FC: the hidden layer's
// outputs (bias, ReLU, rounded to the form) go to LDS (X's region, dead
// after the last group), then the final FC runs as one MFMA tile row on the
// first NOUTP/16 waves; raw outputs to sm.logit.
template <class Net, class P, bool CAL>
__device__ __forceinline__ void hybrid_head(const DevWeights& wt, uint32_t relu_mask,
                                            NetSmem<Net, P>& sm, const v4f* hacc, unsigned* cal,
                                            const int* row_live) {
  using G = Geo<Net, P>;
  using T = typename P::T;
  constexpr int HT = (Net::HID / 16) / Net::WAVES;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  (void)tid;
  constexpr int NOUTP = (Net::NOUT + 15) / 16 * 16, NTL = NOUTP / 16;
  constexpr int SH = Net::HID + G::PAD;
  static_assert(sizeof(T) * MT * SH <= sizeof(sm.xa2) && NTL <= Net::WAVES, "hybrid head");
  T* hb = sm.x();
  const bool hrelu = relu_mask & (1u << hidden_layer<Net>());
  const int row = lane & 15;
  const bool live = !CAL || row_live[row];
#pragma unroll
  for (int jj = 0; jj < HT; ++jj) {
    const int col0 = (wave * HT + jj) * 16 + 4 * (lane >> 4);
    T e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float hv = activation<P>(hacc[jj][i], col0 + i, wt.hid_b, wt.hid_ws, hrelu);
      if constexpr (CAL)
        if (live) cal_max(cal, Net::D + Net::CH1 + Net::CH2 + Net::CH3 + col0 + i, hv);
      e[i] = to_storage<P>(hv, col0 + i, wt.hid_ai);
    }
    store_run<4 * sizeof(T)>(hb + row * SH + col0, e);
  }
  __syncthreads();
  if (wave < NTL) {
    const T* const ap[1] = {hb + row * SH + (P::KG / 4) * (lane >> 4)};
    v4f acc[1][1] = {{v4f{0.f, 0.f, 0.f, 0.f}}};
    mma_stream<P, Net::HID / P::KG, NTL, 1, 1>(acc, ap, static_cast<const uint4*>(wt.last_p),
                                               wave, lane);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int col = wave * 16 + 4 * (lane >> 4) + i;
      if (col < Net::NOUT) sm.logit[row][col] = acc[0][0][i] + wt.last_b[col];
    }
  }
}

// The rest of the predictor on a tile once the hidden layer's sums are in
// hacc (wave w's HT tiles): bias, ReLU, then the head, the raw outputs to
// sm.logit (regression head: sm.stage_head's copies must be there); SAVE:
// the hidden layer's output to sv.h instead (the training form's head is a
// separate product).  The caller synchronises before reading sm.logit.
template <class Net, class P, bool CAL, bool SAVE>
__device__ __forceinline__ void head_tile(const DevWeights& wt, uint32_t relu_mask,
                                          NetSmem<Net, P>& sm, const v4f* hacc, unsigned* cal,
                                          const int* row_live, SavePtrs<typename P::T> sv) {
  using T = typename P::T;
  constexpr int HT = (Net::HID / 16) / Net::WAVES;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  (void)tid;
  if constexpr (SAVE && Net::HID > 0) {
    // training form: the hidden layer's output is kept, the head runs as a
    // separate GEMM over the whole batch
    const bool hrelu = relu_mask & (1u << hidden_layer<Net>());
    const int row = lane & 15;
#pragma unroll
    for (int jj = 0; jj < HT; ++jj) {
      const int col0 = (wave * HT + jj) * 16 + 4 * (lane >> 4);
      T e[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        e[i] = to_storage<P>(activation<P>(hacc[jj][i], col0 + i, wt.hid_b, wt.hid_ws, hrelu),
                             col0 + i, wt.hid_ai);
      if (row < sv.rows) store_run<4 * sizeof(T)>(sv.h + (size_t)row * Net::HID + col0, e);
    }
  } else if constexpr (Net::HID > 0 && Net::HEAD == 1) {
    hybrid_head<Net, P, CAL>(wt, relu_mask, sm, hacc, cal, row_live);
  } else if constexpr (Net::HID > 0) {
    // bias + ReLU on the hidden layer, rounding to the form's precision, then
    // the final FC: lane l holds row l % 16 and 4 columns of each of its HT
    // tiles; reduce over the 4 lanes sharing the row, then over waves.
    const bool hrelu = relu_mask & (1u << hidden_layer<Net>());
    const int row = lane & 15;
    const bool live = !CAL || row_live[row];
    float p[Net::NOUT];
#pragma unroll
    for (int o = 0; o < Net::NOUT; ++o) p[o] = 0.f;
#pragma unroll
    for (int jj = 0; jj < HT; ++jj) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int col = (wave * HT + jj) * 16 + 4 * (lane >> 4) + i;
        const float hv = activation<P>(hacc[jj][i], col, sm.hb, sm.hws, hrelu);
        if constexpr (CAL)
          if (live) cal_max(cal, Net::D + Net::CH1 + Net::CH2 + Net::CH3 + col, hv);
        const float h = P::val(to_storage<P>(hv, col, sm.hai));
#pragma unroll
        for (int o = 0; o < Net::NOUT; ++o) p[o] = fmaf(h, sm.lw[o * Net::HID + col], p[o]);
      }
    }
#pragma unroll
    for (int o = 0; o < Net::NOUT; ++o) {
      float v = p[o];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (lane < 16) sm.red()[(wave * MT + row) * Net::NOUT + o] = v;
    }
    __syncthreads();
    if (tid < MT * Net::NOUT) {
      const int s = tid / Net::NOUT, o = tid % Net::NOUT;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < Net::WAVES; ++w) v += sm.red()[(w * MT + s) * Net::NOUT + o];
      v += sm.lb[o];
      if (relu_mask & (1u << (hidden_layer<Net>() + 1))) v = fmaxf(v, 0.f);
      sm.logit[s][o] = v;
    }
  }
}

// The whole predictor on one tile of MT windows.  The window arrives a group
// of NG blocks (NG*BS slots) at a time: load(j0, nb) requests the rows of
// blocks j0 .. j0+nb-1 into registers, commit(j0, nb, regs, X) writes them,
// in storage precision, to X at window s, slot t of the group, feature c
// (slot pairs padded, see Geo).
// The next group's rows are requested after the current group's conv levels
// and committed before its FC, so their memory latency is hidden.  Both are
// called by all threads; the raw outputs land in sm.logit.  CAL: also record
// per-channel max |input| of every layer into cal (offsets: window D, conv1
// out, conv2 out[, conv3 out, hidden out]), counting only tile rows whose
// row_live[s] is set.  TRUNK: the convolutions only, the last conv's
// output written to sv.a3 (nothing in sm.logit).
template <class Net, class P, bool CAL = false, bool SAVE = false, bool TRUNK = false, class Load,
          class Commit>
__device__ __forceinline__ void predict_tile(const DevWeights& wt, uint32_t relu_mask,
                                             NetSmem<Net, P>& sm, Load&& load, Commit&& commit,
                                             unsigned* cal = nullptr,
                                             const int* row_live = nullptr,
                                             SavePtrs<typename P::T> sv = {}) {
  using G = Geo<Net, P>;
  constexpr int NG = G::NG, NFULL = Net::NB / NG, TAIL = Net::NB % NG;
  const int tid = threadIdx.x;
  constexpr int HT = Net::HID > 0 ? (Net::HID / 16) / Net::WAVES : 1;
  v4f hacc[HT];
#pragma unroll
  for (int j = 0; j < HT; ++j) hacc[j] = v4f{0.f, 0.f, 0.f, 0.f};
  float fpart = 0.f;

  {
    auto regs = load(0, NFULL > 0 ? NG : TAIL);
    commit(0, NFULL > 0 ? NG : TAIL, regs, sm.x());
  }
  constexpr bool XPF = Net::NCONV == 3;  // LDS-only barriers (see run_group)
  for (int g = 0; g < NFULL; ++g) {
    if constexpr (XPF)
      lds_barrier();
    else
      __syncthreads();
    const int j0 = g * NG;
    const int nj = j0 + NG, nnb = g + 1 < NFULL ? NG : TAIL;
    run_group<Net, P, NG, CAL, SAVE, TRUNK>(
        wt, relu_mask, sm, j0, cal, row_live, sv, hacc, fpart, [&]() { return load(nj, nnb); },
        [&](const auto& regs) {
          if (nnb > 0) commit(nj, nnb, regs, sm.x());
        });
  }
  if constexpr (TAIL > 0) {
    if constexpr (XPF)
      lds_barrier();
    else
      __syncthreads();
    run_group<Net, P, TAIL, CAL, SAVE, TRUNK>(
        wt, relu_mask, sm, NFULL * NG, cal, row_live, sv, hacc, fpart, []() { return 0; },
        [](int) {});
  }
  if constexpr (TRUNK) {
    __syncthreads();
    return;
  }

  if constexpr (Net::HID > 0) {
    head_tile<Net, P, CAL, SAVE>(wt, relu_mask, sm, hacc, cal, row_live, sv);
  } else {
    constexpr int LPP = G::NT / (MT * Net::NOUT);
    const int fpair = tid / LPP, fsub = tid % LPP;
    const int fs = fpair / Net::NOUT, fo = fpair % Net::NOUT;
#pragma unroll
    for (int m = 1; m < LPP; m <<= 1) fpart += __shfl_xor(fpart, m);
    if (fsub == 0) {
      float v = fpart + wt.last_b[fo];
      if (relu_mask & (1u << Net::NCONV)) v = fmaxf(v, 0.f);
      sm.logit[fs][fo] = v;
    }
  }
  __syncthreads();
}

// One thread's share of a window row: CPT consecutive features from column
// c0.  FP8: the features' input scales are applied (xs: reciprocals by
// feature, in LDS).
template <class P, int CPT, int D>
__device__ __forceinline__ void window_elems(const float (&v)[CPT], const float* xs, int c0,
                                             typename P::T (&e)[CPT]) {
#pragma unroll
  for (int i = 0; i < CPT; ++i) {
    float x = v[i];
    if constexpr (P::SCALED) x *= xs[c0 + i < D ? c0 + i : 0];
    e[i] = P::cvt(x);
  }
}

// Registers carrying one thread's share of one window row between load and
// commit: FP32 feature pairs, or (H) BF16 feature pairs in one word each.
template <int CPT, bool H = false>
struct RowRegs {
  typename std::conditional<H, uint32_t, float2>::type v[CPT / 2];
  uint32_t code;
  float res, ex, sto;
  int valid;
  uint2 mem, cur_mem;  // dependency flags: this row's and slot 0's addresses
};

// The five memory dependency flags of a context instruction with addresses
// m against the current instruction's c (Sec. 2.1): same instruction cache
// line, same instruction page, same data address, data cache line, data
// page (64-byte lines, 4 KB pages; data flags need both addresses).
__device__ __forceinline__ float dep_flag(uint2 m, uint2 c, int f) {
  const bool both = m.y != 0u && c.y != 0u;
  switch (f) {
    case 0: return (m.x >> 6) == (c.x >> 6) ? 1.f : 0.f;
    case 1: return (m.x >> 12) == (c.x >> 12) ? 1.f : 0.f;
    case 2: return both && m.y == c.y ? 1.f : 0.f;
    case 3: return both && (m.y >> 6) == (c.y >> 6) ? 1.f : 0.f;
    default: return both && (m.y >> 12) == (c.y >> 12) ? 1.f : 0.f;
  }
}

// Rounded latency in cycles: nearest, ties to even; non-finite -> 0;
// clamped to [0, lat_max].
__device__ __forceinline__ int32_t round_latency(float v, int32_t lat_max, uint32_t& clamped,
                                                 uint32_t& nonfinite) {
  // (selects, not branches: this lies on the chain through every step)
  const bool finite = isfinite(v);
  const float r = rintf(v), top = (float)lat_max;
  const bool low = finite && r < 0.f, high = finite && r > top;
  nonfinite += !finite;
  clamped += low || high;
  const int32_t i = (int32_t)(finite && !low && !high ? r : 0.f);
  return high ? lat_max : i;
}

// Execution and store latency (each at most 65535) in one 32-bit word.
__device__ __forceinline__ int32_t pack_es(int32_t e, int32_t s) {
  return (int32_t)((uint32_t)e | ((uint32_t)s << 16));
}

// Hybrid head (Sec. 2.3): the most probable class (the first of equal
// scores; a NaN score never wins) is the latency, unless it is the last
// class ("larger"), which takes the direct output z[HYB_CLASSES], rounded.
__device__ __forceinline__ int32_t hybrid_latency(const float* z, int32_t lat_max,
                                                  uint32_t& clamped, uint32_t& nonfinite) {
  int best = 0;
#pragma unroll
  for (int c = 1; c < HYB_CLASSES; ++c)
    if (z[c] > z[best]) best = c;
  if (best < HYB_CLASSES - 1) return best;
  return round_latency(z[HYB_CLASSES], lat_max, clamped, nonfinite);
}

// Feature c of an instruction given as a packed code (trace encoding
// SIM_FEAT_CODE32): op class one-hot [0,5), three register ids one-hot in 7
// buckets each [5,26), data level one-hot [26,29), mispredict flag [29].
__device__ __forceinline__ float code_feature(uint32_t code, int c) {
  if (c < 5) return (int)(code & 7u) == c ? 1.f : 0.f;
  if (c < 26) {
    const int r = (c - 5) / 7, b = (c - 5) % 7;
    const int id = (int)((code >> (3 + 5 * r)) & 31u);
    return (id * 7) >> 5 == b ? 1.f : 0.f;
  }
  if (c < 29) return (int)((code >> 18) & 3u) == c - 26 ? 1.f : 0.f;
  if (c == 29) return (float)((code >> 20) & 1u);
  return 0.f;
}

// The gather of a group's window rows: TPR threads per (window, slot of the
// group) row, CPT features each.  H16: the BF16 form reads rows of a BF16
// copy of the trace (DS features each).
template <class Net, class P>
struct Gather {
  using G = Geo<Net, P>;
  static constexpr int GSL = G::NG * Net::BS;
  static constexpr int ROWS = MT * GSL, TPR = G::NT / ROWS, CPT = G::DP / TPR;
  static constexpr bool H16 = P::ID == 1;
  static constexpr int DS = staged_feat(Net::D);
  static_assert(G::NT % ROWS == 0 && G::DP % TPR == 0 && CPT % 2 == 0 && Net::D % 2 == 0,
                "gather split");
  static_assert(!H16 || (CPT % 8 == 0 && DS % 8 == 0), "BF16 rows");
  using Regs = RowRegs<CPT, H16>;
};

// A thread's share of trace row idx requested (-1: no instruction; every
// address is in bounds, so all are in flight together).  DEP: its addresses
// and those of the current instruction cur_idx; slot0: it is that one.
template <class Net, class P, bool DEP>
__device__ __forceinline__ void request_row(const StepParams& p, int64_t idx, bool slot0,
                                            int64_t cur_idx, int part,
                                            typename Gather<Net, P>::Regs& r) {
  using GA = Gather<Net, P>;
  constexpr int CPT = GA::CPT, TPR = GA::TPR, D = Net::D, DS = GA::DS;
  constexpr bool H16 = GA::H16;
  (void)slot0;
  (void)cur_idx;
  r.valid = idx >= 0;
  r.code = 0;
  if constexpr (DEP) {  // addresses of this row and of slot 0 (broadcast)
    r.mem = p.mem[idx < 0 ? 0 : idx];
    r.cur_mem = p.mem[cur_idx];
    if (slot0) r.valid = idx >= 0 ? 2 : 0;  // slot 0: no flags
  }
  if (p.codes) {
    r.code = p.codes[idx < 0 ? 0 : idx];
  } else if constexpr (H16) {
    // BF16 rows of DS features (16-byte aligned): whole 16-byte chunks
    const uint4* src = reinterpret_cast<const uint4*>(p.feat16 + (idx < 0 ? 0 : idx) * DS);
#pragma unroll
    for (int q = 0; q < CPT / 8; ++q) {
      const int c = part * CPT + 8 * q;
      const uint4 w = c < DS ? src[c / 8] : make_uint4(0u, 0u, 0u, 0u);
      r.v[4 * q] = w.x;
      r.v[4 * q + 1] = w.y;
      r.v[4 * q + 2] = w.z;
      r.v[4 * q + 3] = w.w;
    }
  } else {
    const float* src = p.feat + (idx < 0 ? 0 : idx) * D;
#pragma unroll
    for (int cc = 0; cc < CPT; cc += 2) {
      const int c = part * CPT + cc;
      // one thread per row: the padding columns are known at compile time
      if (TPR > 1 || cc < D)
        r.v[cc / 2] = *reinterpret_cast<const float2*>(src + (c < D ? c : D - 2));
      else
        r.v[cc / 2] = make_float2(0.f, 0.f);
    }
  }
}

// The share written to X (the group's window rows in LDS) at window gs, slot
// gt: dynamic columns, conversion, vector stores.
template <class Net, class P, bool CAL, bool DEP>
__device__ __forceinline__ void commit_row(const StepParams& p, const float* x_inv, int gs, int gt,
                                           int part, const typename Gather<Net, P>::Regs& r,
                                           typename P::T* X, unsigned* cal) {
  using G = Geo<Net, P>;
  using T = typename P::T;
  using GA = Gather<Net, P>;
  constexpr int CPT = GA::CPT, D = Net::D, DP = G::DP;
  constexpr bool H16 = GA::H16;
  (void)cal;
  T* dst = X + gs * G::SX + (gt >> 1) * G::RX + (gt & 1) * DP + part * CPT;
  // the row's column c, when this thread's share holds it, set to v
  auto put = [&](int c, float v) {
    if (c >= part * CPT && c < part * CPT + CPT) {
      if constexpr (P::SCALED) v *= x_inv[c < D ? c : 0];
      dst[c - part * CPT] = P::cvt(v);
    }
  };
  // the memory dependency flags (after the other columns, as below)
  auto put_dep = [&]() {
    if constexpr (DEP)
#pragma unroll
      for (int f = 0; f < 5; ++f)
        put(p.col_dep + f, r.valid == 1 ? dep_flag(r.mem, r.cur_mem, f) : 0.f);
  };
  if constexpr (!CAL) {
    // The share written whole, then the few columns that are not copied
    // features overwritten one by one: the same values as the per-feature
    // conversion below at a fraction of its VALU work.  The BF16 form's
    // rows are stored as loaded (its BF16 copy of the trace holds exactly
    // the values the conversion would produce).
    if constexpr (H16) {
      if (!p.codes) {
#pragma unroll
        for (int q = 0; q < CPT / 8; ++q) {
          const uint4 w = r.valid ? uint4{r.v[4 * q], r.v[4 * q + 1], r.v[4 * q + 2],
                                          r.v[4 * q + 3]}
                                  : uint4{0u, 0u, 0u, 0u};
          *reinterpret_cast<uint4*>(dst + 8 * q) = w;
        }
        put(p.col_res, r.res);
        put(p.col_exe, r.ex);
        put(p.col_sto, r.sto);
        put_dep();
        return;
      }
    }
    // packed codes: zeros, then the one-hot features of code_feature
    static_assert(D >= 30, "the code's features are columns 0 .. 29");
    if constexpr ((CPT * sizeof(T)) % 16 == 0) {
      if (p.codes) {
#pragma unroll
        for (int q = 0; q < CPT * (int)sizeof(T) / 16; ++q)
          *reinterpret_cast<uint4*>(reinterpret_cast<char*>(dst) + 16 * q) =
              uint4{0u, 0u, 0u, 0u};
        if (r.valid) {
          const uint32_t code = r.code;
          if ((code & 7u) < 5u) put((int)(code & 7u), 1.f);
#pragma unroll
          for (int g = 0; g < 3; ++g)
            put(5 + 7 * g + (((int)((code >> (3 + 5 * g)) & 31u) * 7) >> 5), 1.f);
          if (((code >> 18) & 3u) < 3u) put(26 + (int)((code >> 18) & 3u), 1.f);
          if ((code >> 20) & 1u) put(29, 1.f);
        }
        put(p.col_res, r.res);
        put(p.col_exe, r.ex);
        put(p.col_sto, r.sto);
        put_dep();
        return;
      }
    }
  }
  float v[CPT];
#pragma unroll
  for (int cc = 0; cc < CPT; ++cc) {
    const int c = part * CPT + cc;
    float x = 0.f;
    if (r.valid && c < D) {
      if (p.codes)
        x = code_feature(r.code, c);
      else if constexpr (H16)
        x = __uint_as_float(cc & 1 ? r.v[cc / 2] & 0xffff0000u : r.v[cc / 2] << 16);
      else
        x = cc & 1 ? r.v[cc / 2].y : r.v[cc / 2].x;
    }
    if (c == p.col_res) x = r.res;
    if (c == p.col_exe) x = r.ex;
    if (c == p.col_sto) x = r.sto;
    if constexpr (DEP)
      if (c >= p.col_dep && c < p.col_dep + 5)
        x = r.valid == 1 ? dep_flag(r.mem, r.cur_mem, c - p.col_dep) : 0.f;
    if constexpr (CAL)
      if (c < D && r.valid) cal_max(cal, c, x);
    v[cc] = x;
  }
  T e[CPT];
  window_elems<P, CPT, D>(v, x_inv, part * CPT, e);
  store_run<(CPT * sizeof(T)) % 16 == 0 ? 16 : 8>(dst, e);
}

// The same for explicit windows x [B][L][D] (FP32): slot t of window b.
template <class Net, int CPT, int TPR>
__device__ __forceinline__ RowRegs<CPT> request_window_row(const float* __restrict__ x, int64_t B,
                                                           int64_t b, int t, bool in_group,
                                                           int part) {
  constexpr int D = Net::D;
  RowRegs<CPT> r;
  r.valid = b < B && in_group;
  const float* src = x + ((r.valid ? b : 0) * Net::L + (r.valid ? t : 0)) * D;
#pragma unroll
  for (int cc = 0; cc < CPT; cc += 2) {
    const int c = part * CPT + cc;
    if (TPR > 1 || cc < D)
      r.v[cc / 2] = *reinterpret_cast<const float2*>(src + (c < D ? c : D - 2));
    else
      r.v[cc / 2] = make_float2(0.f, 0.f);
  }
  return r;
}

template <class Net, class P, int CPT>
__device__ __forceinline__ void commit_window_row(const float* x_inv, int s, int t, int part,
                                                  const RowRegs<CPT>& r, typename P::T* X) {
  using G = Geo<Net, P>;
  constexpr int D = Net::D;
  float v[CPT];
#pragma unroll
  for (int cc = 0; cc < CPT; ++cc) {
    const int c = part * CPT + cc;
    v[cc] = (r.valid && c < D) ? (cc & 1 ? r.v[cc / 2].y : r.v[cc / 2].x) : 0.f;
  }
  typename P::T e[CPT];
  window_elems<P, CPT, D>(v, x_inv, part * CPT, e);
  store_run<(CPT * sizeof(typename P::T)) % 16 == 0 ? 16 : 8>(
      X + s * G::SX + (t >> 1) * G::RX + (t & 1) * G::DP + part * CPT, e);
}

}  // namespace simnet

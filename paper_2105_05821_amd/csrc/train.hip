// Training-form kernels of libsimnet.so (gfx950): the pieces of a predictor
// training step that are not the fused trunk forward.
//
//   gemm kernels     C = op(A) x op(B), operands in FP32 or BF16, split-K with
//                    an ordered reduction when the output is small; epilogue
//                    with bias, ReLU mask (a saved activation > 0),
//                    accumulation and a column permutation of C (weight
//                    gradients stored in the parameters' own layout).  Used
//                    for the head and for every input-gradient and
//                    weight-gradient product of the backward pass (a kernel-2
//                    stride-2 convolution is a GEMM over position pairs).
//                    Operands in aligned rows go straight to LDS and are
//                    transposed on their way out (gemm_bf16_dma_kernel,
//                    gemm_f32_dma_kernel); operands of arbitrary strides and
//                    alignment take gemm_bf16_kernel (128x128 tiles, rounded
//                    to BF16 in LDS) and gemm_kernel (FP32 MFMA, 64x64 tiles).
//   gemm_group_kernel, group_reduce
//                    all weight gradients of a pass in one launch, with the
//                    row sums of their left operands (the trunk's bias
//                    gradients), their partials and the bias sums in another.
//   reductions       split-K partials summed in order with the epilogue.
//   loss_kernel      hybrid loss per window (400-bin cross-entropy + L1 on
//                    log1p(latency) per latency type) and its gradient
//                    w.r.t. the head outputs.
//   colsum kernels   bias gradients as chunk partials; sum_partials adds
//                    several lists of partials, each in a fixed order.
//   map_gather_multi weight re-layouts by index maps.
//   pad_rows         a row-major matrix copied with its rows padded.
//   adam kernels     Adam on FP32 master weights (and, fused, the re-layout
//                    of the updated weights).
#include <algorithm>
#include <type_traits>

#include "simnet_internal.h"

namespace simnet {

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float ld_elem(const void* p, int bf16, int64_t i) {
  if (bf16) return __uint_as_float((uint32_t)static_cast<const uint16_t*>(p)[i] << 16);
  return static_cast<const float*>(p)[i];
}

// Rows are grouped (row r at (r / grp) * gs + (r % grp) * rs) only where an
// operand skips memory between groups of rows; ungrouped operands carry
// grp >= NO_GROUP and take no division.  Grouped row indices are below
// 2^32 (the host checks), so their division is 32-bit.
__device__ __forceinline__ int64_t grouped_row(int64_t r, int64_t grp, int64_t gs, int64_t rs) {
  if (grp >= NO_GROUP) return r * rs;
  const uint32_t q = (uint32_t)r / (uint32_t)grp;
  return (int64_t)q * gs + (int64_t)((uint32_t)r - q * (uint32_t)grp) * rs;
}

__device__ __forceinline__ int64_t op_index(const GemmOperand& o, int64_t r, int64_t c) {
  return grouped_row(r, o.grp, o.gs, o.rs) + c * o.cs;
}

// Nearest-even BF16 bits of a finite float.
__device__ __forceinline__ uint16_t to_bf16(float x) {
  const uint32_t u = __float_as_uint(x);
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// Column n's offset in a row of C (N below 2^32 when permuted: the host
// checks).
__device__ __forceinline__ int64_t c_col(const GemmArgs& g, int64_t n) {
  if (g.ccg == 0) return n;
  const uint32_t q = (uint32_t)n / (uint32_t)g.ccg;
  return (int64_t)((uint32_t)n - q * (uint32_t)g.ccg) * g.ccm + q;
}

// C(m, n) epilogue shared by every GEMM path: bias, ReLU mask, accumulate,
// grouped row and permuted column addressing, BF16 output.
__device__ __forceinline__ void gemm_store(const GemmArgs& g, int64_t m, int64_t n, float v) {
  if (g.bias) v += g.bias[n];
  if (g.mask.p && !(ld_elem(g.mask.p, g.mask.bf16, op_index(g.mask, m, n)) > 0.f)) v = 0.f;
  const int64_t at = grouped_row(m, g.cgrp, g.cgs, g.ldc) + c_col(g, n);
  if (g.c_bf16) {
    reinterpret_cast<uint16_t*>(g.C)[at] = to_bf16(v);
    return;
  }
  float* c = g.C + at;
  *c = g.beta ? *c + v : v;
}

// The same for the columns n0 + 16*j (j < NJ) of one row m, with the row's
// addresses computed once; the caller has added the bias.
template <int NJ>
__device__ __forceinline__ void gemm_store_row(const GemmArgs& g, int64_t m, int64_t n0,
                                               const float (&v)[NJ]) {
  const int64_t crow = grouped_row(m, g.cgrp, g.cgs, g.ldc);
  const int64_t mrow = g.mask.p ? grouped_row(m, g.mask.grp, g.mask.gs, g.mask.rs) : 0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int64_t n = n0 + 16 * j;
    if (n >= g.N) continue;
    float x = v[j];
    if (g.mask.p && !(ld_elem(g.mask.p, g.mask.bf16, mrow + n * g.mask.cs) > 0.f)) x = 0.f;
    const int64_t at = crow + c_col(g, n);
    if (g.c_bf16) {
      reinterpret_cast<uint16_t*>(g.C)[at] = to_bf16(x);
    } else {
      float* c = g.C + at;
      *c = g.beta ? *c + x : x;
    }
  }
}

// Split-K: workgroup z covers k in [z*kc, min(K, (z+1)*kc)) and writes its
// raw partial product to part[z][M][N]; gemm_reduce sums the partials in
// order and applies the epilogue.
__device__ __forceinline__ void k_range(const GemmArgs& g, int step, int64_t z, int64_t* kb,
                                        int64_t* ke) {
  const int64_t per = (g.K + g.ksplit - 1) / g.ksplit;
  const int64_t kc = (per + step - 1) / step * step;
  *kb = z * kc;
  *ke = *kb + kc < g.K ? *kb + kc : g.K;
}

__device__ __forceinline__ void gemm_out(const GemmArgs& g, int64_t m, int64_t n, float v) {
  if (g.ksplit > 1)
    g.part[((int64_t)blockIdx.z * g.M + m) * g.N + n] = v;
  else
    gemm_store(g, m, n, v);
}

constexpr int GB = 64, GK = 16, GPAD = 4;

// One thread's four elements of a tile (rows r0.. of R, cols c0.. of C),
// read along whichever dimension is contiguous in memory.
__device__ __forceinline__ void load_tile(const GemmOperand& o, int64_t R, int64_t Cn, int64_t r0,
                                          int64_t c0, bool rows_are_k, int tid, float (&v)[4],
                                          int (&rr)[4], int (&cc)[4]) {
  // tile is GB (non-k) x GK (k); "along" = the contiguous dimension
  const bool k_contig = rows_are_k ? (o.rs == 1 && o.grp >= NO_GROUP) : (o.cs == 1);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    int kk, mm;
    if (k_contig) {
      mm = tid / 4;
      kk = (tid % 4) * 4 + e;
    } else {
      kk = tid / 16;
      mm = (tid % 16) * 4 + e;
    }
    // rows_are_k: operand rows index k (B operand); else rows index m (A)
    const int64_t r = rows_are_k ? r0 + kk : r0 + mm;
    const int64_t c = rows_are_k ? c0 + mm : c0 + kk;
    v[e] = (r < R && c < Cn) ? ld_elem(o.p, o.bf16, op_index(o, r, c)) : 0.f;
    rr[e] = kk;
    cc[e] = mm;
  }
}

// FP32 form: 64x64 tiles on mfma_f32_16x16x4f32, 2x2 waves of 32x32.
__global__ void __launch_bounds__(256) gemm_kernel(GemmArgs g) {
  __shared__ float As[GK][GB + GPAD];  // [k][m]
  __shared__ float Bs[GK][GB + GPAD];  // [k][n]
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t m0 = (int64_t)blockIdx.y * GB, n0 = (int64_t)blockIdx.x * GB;
  const int wm = wave >> 1, wn = wave & 1;
  int64_t kb, ke;
  k_range(g, GK, blockIdx.z, &kb, &ke);
  v4f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  float va[4], vb[4];
  int ka[4], ma[4], kb4[4], nb[4];
  load_tile(g.A, g.M, ke, m0, kb, false, tid, va, ka, ma);
  load_tile(g.B, ke, g.N, kb, n0, true, tid, vb, kb4, nb);
  for (int64_t k0 = kb; k0 < ke; k0 += GK) {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      As[ka[e]][ma[e]] = va[e];
      Bs[kb4[e]][nb[e]] = vb[e];
    }
    __syncthreads();
    if (k0 + GK < ke) {  // next tile in flight while this one is multiplied
      load_tile(g.A, g.M, ke, m0, k0 + GK, false, tid, va, ka, ma);
      load_tile(g.B, ke, g.N, k0 + GK, n0, true, tid, vb, kb4, nb);
    }
#pragma unroll
    for (int ks = 0; ks < GK; ks += 4) {
      const int k = ks + (lane >> 4);
      float a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = As[k][wm * 32 + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = Bs[k][wn * 32 + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
  // lane holds C[4*(lane/16) + r][lane % 16] of each 16x16 tile
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + wm * 32 + i * 16 + 4 * (lane >> 4) + r;
        const int64_t n = n0 + wn * 32 + j * 16 + (lane & 15);
        if (m < g.M && n < g.N) gemm_out(g, m, n, acc[i][j][r]);
      }
}

// BF16 form: 128x128 tiles, k-steps of 32 on mfma_f32_16x16x32_bf16, 2x2
// waves of 64x64, operands rounded to BF16 (nearest even) into LDS, FP32
// accumulation.  Both LDS tiles are [outer][k] so that a lane's fragment (8
// consecutive k of one row or column) is one 16-byte read.  Each thread
// stages 16 elements of each operand per k-step, read along the operand's
// contiguous dimension: mode 1 = along k (written to LDS as two 16-byte
// runs), mode 2 = along the outer dimension (written as 16 scalars, a
// transpose), mode 0 = no unit stride (scalar reads, k-major mapping).
constexpr int HB = 128, HK = 32, HLD = HK + 8;
static_assert(32 * (HB + 4) * sizeof(float) <= 2 * HB * HLD * sizeof(uint16_t),
              "the epilogue's staging fits one operand's LDS tiles");

typedef __bf16 v8bf_t __attribute__((ext_vector_type(8)));


// One thread's 16 staged elements of an operand: as floats (converted to
// BF16 when stored), or, raw, the 16 BF16 values as loaded (an operand
// already in BF16 needs no conversion: its values round to themselves).
struct Stage {
  union {
    float v[16];
    uint32_t w[8];  // raw: element 2q in the low half of w[q], 2q + 1 in the high
  };
  int raw;
};

// Element (outer, k) of an operand: A is (m, k), B is (k, n).
__device__ __forceinline__ int64_t elem_addr(const GemmOperand& o, bool is_b, int64_t outer,
                                             int64_t k) {
  return is_b ? op_index(o, k, outer) : op_index(o, outer, k);
}

__device__ __forceinline__ void stage_load(const GemmOperand& o, bool is_b, int mode, int vec,
                                           int64_t outer0, int64_t k0, int64_t outer_lim,
                                           int64_t k_lim, int tid, Stage& st) {
  int64_t outer, k;
  int cnt;
  if (mode == 2) {
    k = k0 + tid / 8;
    outer = outer0 + (tid % 8) * 16;
    const int64_t left = outer_lim - outer;
    cnt = k < k_lim ? (left > 16 ? 16 : (left > 0 ? (int)left : 0)) : 0;
  } else {
    outer = outer0 + tid / 2;
    k = k0 + (tid % 2) * 16;
    const int64_t left = k_lim - k;
    cnt = outer < outer_lim ? (left > 16 ? 16 : (left > 0 ? (int)left : 0)) : 0;
  }
  st.raw = 0;
  if (mode != 0 && vec == 1 && cnt == 16) {  // 8-byte vectors
    const int64_t a = elem_addr(o, is_b, outer, k);
    if (o.bf16) {
      const uint2* p = reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(o.p) + a);
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const uint2 w = p[h];
        st.w[2 * h] = w.x;
        st.w[2 * h + 1] = w.y;
      }
      st.raw = 1;
    } else {
      const float2* p = reinterpret_cast<const float2*>(static_cast<const float*>(o.p) + a);
#pragma unroll
      for (int h = 0; h < 8; ++h) {
        const float2 w = p[h];
        st.v[2 * h] = w.x;
        st.v[2 * h + 1] = w.y;
      }
    }
    return;
  }
  if (mode != 0 && vec == 2 && cnt == 16) {  // 16-byte vectors
    const int64_t a = elem_addr(o, is_b, outer, k);
    if (o.bf16) {
      const uint4* p = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(o.p) + a);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint4 w = p[h];
        st.w[4 * h] = w.x;
        st.w[4 * h + 1] = w.y;
        st.w[4 * h + 2] = w.z;
        st.w[4 * h + 3] = w.w;
      }
      st.raw = 1;
    } else {
      const float4* p = reinterpret_cast<const float4*>(static_cast<const float*>(o.p) + a);
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const float4 w = p[h];
        st.v[4 * h] = w.x;
        st.v[4 * h + 1] = w.y;
        st.v[4 * h + 2] = w.z;
        st.v[4 * h + 3] = w.w;
      }
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    float v = 0.f;
    if (e < cnt)
      v = ld_elem(o.p, o.bf16,
                  mode == 2 ? elem_addr(o, is_b, outer + e, k) : elem_addr(o, is_b, outer, k + e));
    st.v[e] = v;
  }
}

// LDS tiles hold 8-element (16-byte) k-chunks; chunk c of row r sits at
// position c ^ ((r >> 4) & 3), so that the transposing stores of rows 16
// apart (same banks otherwise) spread over four bank groups.
__device__ __forceinline__ int chunk_at(int row, int c) { return c ^ ((row >> 4) & 3); }

__device__ __forceinline__ void stage_store(uint16_t (*S)[HLD], int mode, int tid,
                                            const Stage& st) {
  if (mode == 2) {
    const int k = tid / 8, outer = (tid % 8) * 16;
    if (st.raw) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        S[outer + e][8 * chunk_at(outer + e, k >> 3) + (k & 7)] =
            (uint16_t)(e & 1 ? st.w[e / 2] >> 16 : st.w[e / 2] & 0xffffu);
      return;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e)
      S[outer + e][8 * chunk_at(outer + e, k >> 3) + (k & 7)] = to_bf16(st.v[e]);
  } else {
    const int outer = tid / 2, c0 = (tid % 2) * 2;
    uint32_t w[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      w[q] = st.raw ? st.w[q]
                    : (uint32_t)to_bf16(st.v[2 * q]) | ((uint32_t)to_bf16(st.v[2 * q + 1]) << 16);
    *reinterpret_cast<uint4*>(&S[outer][8 * chunk_at(outer, c0)]) = uint4{w[0], w[1], w[2], w[3]};
    *reinterpret_cast<uint4*>(&S[outer][8 * chunk_at(outer, c0 + 1)]) =
        uint4{w[4], w[5], w[6], w[7]};
  }
}

// The tile kernels' output: a TM x TN tile's accumulators (2 x 2 waves, wave
// (wm, wn) holding rows wm * TM/2 .., columns wn * TN/2 ..) to C through the
// epilogue (bias, ReLU mask, accumulate, BF16 output), or to the split-K
// partials.  E: LDS scratch of epilogue_floats<TN>(), free once the products
// end.
template <int TN>
constexpr int epilogue_floats() {
  return 32 * (TN + 4);
}

template <int TM, int TN>
__device__ __forceinline__ void gemm_tile_epilogue(const GemmArgs& g,
                                                   v4f (&acc)[TM / 32][TN / 32], float* E,
                                                   int64_t m0, int64_t n0, int64_t z, int wm,
                                                   int wn, int tid, int lane) {
  constexpr int MI = TM / 32, NI = TN / 32;
  if (g.evec) {
    // whole 16-byte rows: the tile goes through LDS 32 rows x TN columns at a
    // time, and each thread finishes CW consecutive columns of one row with
    // vector reads of the mask and previous C and vector stores (full cache
    // lines per row instead of 64-byte pieces)
    constexpr int ES = TN + 4;  // row stride of the staged rows, in floats
    constexpr int CW = TN / 8;
    const int er = tid / 8, ec = (tid % 8) * CW;
    const int64_t m = m0 + (er / 16) * (TM / 2) + (er % 16);  // + i * 16
    const int64_t n = n0 + ec;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          E[(wm * 16 + 4 * (lane >> 4) + r) * ES + wn * (TN / 2) + j * 16 + (lane & 15)] =
              acc[i][j][r];
      __syncthreads();
      const int64_t mi = m + i * 16;
      if (mi < g.M && n < g.N) {
        float v[CW];
#pragma unroll
        for (int q = 0; q < CW / 4; ++q) {
          const float4 t = *reinterpret_cast<const float4*>(&E[er * ES + ec + 4 * q]);
          v[4 * q] = t.x;
          v[4 * q + 1] = t.y;
          v[4 * q + 2] = t.z;
          v[4 * q + 3] = t.w;
        }
        if (g.ksplit > 1) {
          float4* cp = reinterpret_cast<float4*>(
              g.part + (z * g.M + mi) * g.N + n);
#pragma unroll
          for (int q = 0; q < CW / 4; ++q)
            cp[q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        } else {
          if (g.mask.p) {
            const int64_t a = grouped_row(mi, g.mask.grp, g.mask.gs, g.mask.rs) + n;
            float mk[CW];
            if (g.mask.bf16) {
              const uint4* mp =
                  reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(g.mask.p) + a);
#pragma unroll
              for (int h = 0; h < CW / 8; ++h) {
                const uint4 w = mp[h];
                const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  mk[8 * h + 2 * q] = __uint_as_float(ws[q] << 16);
                  mk[8 * h + 2 * q + 1] = __uint_as_float(ws[q] & 0xffff0000u);
                }
              }
            } else {
              const float4* mp =
                  reinterpret_cast<const float4*>(static_cast<const float*>(g.mask.p) + a);
#pragma unroll
              for (int q = 0; q < CW / 4; ++q) {
                const float4 w = mp[q];
                mk[4 * q] = w.x;
                mk[4 * q + 1] = w.y;
                mk[4 * q + 2] = w.z;
                mk[4 * q + 3] = w.w;
              }
            }
#pragma unroll
            for (int e = 0; e < CW; ++e)
              if (!(mk[e] > 0.f)) v[e] = 0.f;
          }
          const int64_t at = grouped_row(mi, g.cgrp, g.cgs, g.ldc) + n;
          if (g.c_bf16) {
            uint4* cp = reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(g.C) + at);
#pragma unroll
            for (int h = 0; h < CW / 8; ++h) {
              uint32_t w[4];
#pragma unroll
              for (int q = 0; q < 4; ++q)
                w[q] = (uint32_t)to_bf16(v[8 * h + 2 * q]) |
                       ((uint32_t)to_bf16(v[8 * h + 2 * q + 1]) << 16);
              cp[h] = uint4{w[0], w[1], w[2], w[3]};
            }
          } else {
            float4* cp = reinterpret_cast<float4*>(g.C + at);
#pragma unroll
            for (int q = 0; q < CW / 4; ++q) {
              float4 o = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
              if (g.beta) {
                const float4 c = cp[q];
                o = make_float4(c.x + o.x, c.y + o.y, c.z + o.z, c.w + o.w);
              }
              cp[q] = o;
            }
          }
        }
      }
      __syncthreads();
    }
    return;
  }
  const int64_t nb = n0 + wn * (TN / 2) + (lane & 15);
  // the bias of this lane's columns, read once (per row the compiler would
  // read it again after every store to C)
  float bj[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j)
    bj[j] = g.ksplit <= 1 && g.bias && nb + 16 * j < g.N ? g.bias[nb + 16 * j] : 0.f;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t m = m0 + wm * (TM / 2) + i * 16 + 4 * (lane >> 4) + r;
      if (m >= g.M) continue;
      float v[NI];
#pragma unroll
      for (int j = 0; j < NI; ++j) v[j] = acc[i][j][r] + bj[j];
      if (g.ksplit > 1) {
        float* prow = g.part + (z * g.M + m) * g.N;
#pragma unroll
        for (int j = 0; j < NI; ++j)
          if (nb + 16 * j < g.N) prow[nb + 16 * j] = v[j];
      } else {
        gemm_store_row(g, m, nb, v);
      }
    }
}

__global__ void __launch_bounds__(256) gemm_bf16_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(16))) uint16_t As[2][HB][HLD];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][HB][HLD];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t m0 = (int64_t)blockIdx.y * HB, n0 = (int64_t)blockIdx.x * HB;
  const int wm = wave >> 1, wn = wave & 1;
  int64_t kb, ke;
  k_range(g, HK, blockIdx.z, &kb, &ke);
  v4f acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  Stage sa, sb;
  stage_load(g.A, false, g.amode, g.avec, m0, kb, g.M, ke, tid, sa);
  stage_load(g.B, true, g.bmode, g.bvec, n0, kb, g.N, ke, tid, sb);
  stage_store(As[0], g.amode, tid, sa);
  stage_store(Bs[0], g.bmode, tid, sb);
  __syncthreads();
  int cur = 0;
  for (int64_t k0 = kb; k0 < ke; k0 += HK) {
    const bool more = k0 + HK < ke;
    if (more) {  // next k-step's operands in flight during this one's MFMAs
      stage_load(g.A, false, g.amode, g.avec, m0, k0 + HK, g.M, ke, tid, sa);
      stage_load(g.B, true, g.bmode, g.bvec, n0, k0 + HK, g.N, ke, tid, sb);
    }
    uint4 af[4], bfr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = wm * 64 + i * 16 + (lane & 15);
      af[i] = *reinterpret_cast<const uint4*>(&As[cur][row][8 * chunk_at(row, lane >> 4)]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = wn * 64 + j * 16 + (lane & 15);
      bfr[j] = *reinterpret_cast<const uint4*>(&Bs[cur][row][8 * chunk_at(row, lane >> 4)]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf_t, af[i]),
                                                           __builtin_bit_cast(v8bf_t, bfr[j]),
                                                           acc[i][j], 0, 0, 0);
    if (more) {
      stage_store(As[cur ^ 1], g.amode, tid, sa);
      stage_store(Bs[cur ^ 1], g.bmode, tid, sb);
    }
    __syncthreads();
    cur ^= 1;
  }
  gemm_tile_epilogue<HB, HB>(g, acc, reinterpret_cast<float*>(&As[0][0][0]), m0, n0, blockIdx.z, wm,
                             wn, tid, lane);
}

// out[n] = sum_{c < cnt} src[c * stride + n] for n < N, in a fixed order:
// 64 outputs per workgroup, four lanes per output summing every fourth c,
// then the four partial sums in lane order.  Split-K partials (with the
// GEMM epilogue) and column-sum partials both reduce through this.
template <bool GEMM>
__global__ void __launch_bounds__(256) strided_reduce(const float* __restrict__ src, int64_t cnt,
                                                      int64_t stride, int64_t N, GemmArgs g,
                                                      float* __restrict__ out, int beta) {
  __shared__ float red[4][64];
  const int col = threadIdx.x % 64, lane4 = threadIdx.x / 64;
  const int64_t n = (int64_t)blockIdx.x * 64 + col;
  float s = 0.f;
  if (n < N) {
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    int64_t c = lane4;
    for (; c + 12 < cnt; c += 16) {
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += src[(c + 4 * u) * stride + n];
    }
    for (; c < cnt; c += 4) acc[0] += src[c * stride + n];
    s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  }
  red[lane4][col] = s;
  __syncthreads();
  if (lane4 == 0 && n < N) {
    const float v = (red[0][col] + red[1][col]) + (red[2][col] + red[3][col]);
    if constexpr (GEMM) {
      gemm_store(g, n / g.N, n % g.N, v);
    } else {
      out[n] = beta ? out[n] + v : v;
    }
  }
}

// The same sums for long lists (cnt >= 64 partials): L lanes per output
// (16 or 64, one wave), lane l summing partials c = l, l + L, ... in order,
// then the L lane sums combined by a fixed butterfly (xor L/2, ..., 1), so
// the order is fixed and the latency is that of cnt / L loads, not cnt / 4.
template <bool GEMM>
__global__ void __launch_bounds__(256) strided_reduce_tree(const float* __restrict__ src,
                                                           int64_t cnt, int64_t stride, int64_t N,
                                                           int L, GemmArgs g,
                                                           float* __restrict__ out, int beta) {
  const int per_wg = 256 / L, sub = threadIdx.x % L;
  const int64_t n = (int64_t)blockIdx.x * per_wg + threadIdx.x / L;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  if (n < N) {
    int64_t c = sub;
    for (; c + 3 * L < cnt; c += 4 * L) {
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += src[(c + u * L) * stride + n];
    }
    for (; c < cnt; c += L) acc[0] += src[c * stride + n];
  }
  float v = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  for (int off = L / 2; off >= 1; off /= 2) v += __shfl_xor(v, off);
  if (sub == 0 && n < N) {
    if constexpr (GEMM) {
      gemm_store(g, n / g.N, n % g.N, v);
    } else {
      out[n] = beta ? out[n] + v : v;
    }
  }
}

// 16 waves per 64 outputs (coalesced: a wave reads 64 adjacent outputs of
// one partial), wave w summing partials c = w, w + 16, ... in order, the 16
// wave sums then combined in LDS by a fixed pairwise tree: for long lists
// of partials of many outputs (the split-K weight gradients).
template <bool GEMM>
__global__ void __launch_bounds__(1024) strided_reduce_wide(const float* __restrict__ src,
                                                            int64_t cnt, int64_t stride, int64_t N,
                                                            GemmArgs g, float* __restrict__ out,
                                                            int beta) {
  __shared__ float red[16][64];
  const int col = threadIdx.x % 64, w = threadIdx.x / 64;
  const int64_t n = (int64_t)blockIdx.x * 64 + col;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  if (n < N) {
    int64_t c = w;
    for (; c + 48 < cnt; c += 64) {
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += src[(c + 16 * u) * stride + n];
    }
    for (; c < cnt; c += 16) acc[0] += src[c * stride + n];
  }
  red[w][col] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  for (int h = 8; h >= 1; h /= 2) {
    if (w < h) red[w][col] += red[w + h][col];
    __syncthreads();
  }
  if (w == 0 && n < N) {
    const float v = red[0][col];
    if constexpr (GEMM) {
      gemm_store(g, n / g.N, n % g.N, v);
    } else {
      out[n] = beta ? out[n] + v : v;
    }
  }
}

// Split-K partials of a GEMM with few parts (cnt < 64) and N a multiple of
// 4: each thread finishes four adjacent outputs of one row, its partials
// read as 16-byte vectors and added in part order, then the epilogue.
__global__ void __launch_bounds__(256) reduce_gemm_vec4(const float* __restrict__ src, int64_t cnt,
                                                        int64_t MN, GemmArgs g) {
  const int64_t q = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (q >= MN) return;
  float4 a = *reinterpret_cast<const float4*>(src + q);
#pragma unroll 4
  for (int64_t c = 1; c < cnt; ++c) {
    const float4 t = *reinterpret_cast<const float4*>(src + c * MN + q);
    a.x += t.x;
    a.y += t.y;
    a.z += t.z;
    a.w += t.w;
  }
  const int64_t m = q / g.N, n = q - m * g.N;
  gemm_store(g, m, n, a.x);
  gemm_store(g, m, n + 1, a.y);
  gemm_store(g, m, n + 2, a.z);
  gemm_store(g, m, n + 3, a.w);
}

// The same for a permuted C (ccg > 0, N = ccg * ccm, no bias, mask or BF16
// output, 16-byte aligned rows): each thread finishes four adjacent outputs
// of one row in C's own order, d -> GEMM column (d % ccm) * ccg + d / ccm,
// so the stores are 16-byte vectors and the permutation falls on the reads
// (a wave's 256 outputs read about two cache lines per part and tap).
__global__ void __launch_bounds__(256) reduce_gemm_perm4(const float* __restrict__ src,
                                                         int64_t cnt, int64_t MN, GemmArgs g) {
  const int64_t q = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (q >= MN) return;
  const int64_t m = q / g.N, d0 = q - m * g.N;
  int64_t col[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int64_t d = d0 + e, t = d / g.ccm;
    col[e] = m * g.N + (d - t * g.ccm) * g.ccg + t;
  }
  float a[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) a[e] = src[col[e]];
#pragma unroll 4
  for (int64_t c = 1; c < cnt; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] += src[c * MN + col[e]];
  float4* cp = reinterpret_cast<float4*>(g.C + m * g.ldc + d0);
  float4 o = make_float4(a[0], a[1], a[2], a[3]);
  if (g.beta) {
    const float4 p = *cp;
    o = make_float4(p.x + o.x, p.y + o.y, p.z + o.z, p.w + o.w);
  }
  *cp = o;
}

// Reduce cnt partials of N outputs (see strided_reduce) with the kernel
// that suits the shape: few outputs and a long list (the bias sums): many
// lanes per output; many outputs and a long list: 16 waves per 64 outputs;
// otherwise 4.
template <bool GEMM>
static void launch_reduce(const float* src, int64_t cnt, int64_t stride, int64_t N,
                          const GemmArgs& g, float* out, int beta, hipStream_t stream) {
  if (cnt >= 64 && N <= 1024) {
    const int L = cnt >= 256 ? 64 : 16;
    const int64_t per_wg = 256 / L;
    hipLaunchKernelGGL(strided_reduce_tree<GEMM>, dim3((unsigned)((N + per_wg - 1) / per_wg)),
                       dim3(256), 0, stream, src, cnt, stride, N, L, g, out, beta);
  } else if (cnt >= 64) {
    hipLaunchKernelGGL(strided_reduce_wide<GEMM>, dim3((unsigned)((N + 63) / 64)), dim3(1024), 0,
                       stream, src, cnt, stride, N, g, out, beta);
  } else {
    hipLaunchKernelGGL(strided_reduce<GEMM>, dim3((unsigned)((N + 63) / 64)), dim3(256), 0,
                       stream, src, cnt, stride, N, g, out, beta);
  }
}

// The tile of workgroup id of nx x ny.  Workgroups go to the 8 XCDs in turn (id %
// 8), each XCD with its own L2: when the tiles of a k-split divide evenly,
// XCD x takes the x-th eighth of them in row-major order along the longer
// tile dimension, a band that shares the shorter operand whole and holds an
// eighth of the other, instead of tiles from everywhere.
__device__ __forceinline__ void xcd_tile(int64_t id, int64_t nx, int64_t ny, int64_t* tm,
                                         int64_t* tn) {
  const int64_t tiles = nx * ny;
  *tm = id / nx;
  *tn = id % nx;
  if (tiles % 8 != 0 || tiles < 64) return;
  const int64_t t = (id % 8) * (tiles / 8) + id / 8;
  if (ny >= nx) {
    *tm = t / nx;
    *tn = t % nx;
  } else {
    *tn = t / ny;
    *tm = t % ny;
  }
}

// The BF16 kernel for BF16 operands whose rows are 16-byte aligned: both
// operands go from memory to LDS as they are (global_load_lds, no registers,
// no conversion), three k-steps in flight in LDS stages of their own, one
// barrier per k-step.  An operand contiguous along k (mode 1) is staged
// [outer][32 k] and its fragments read as 16-byte runs; one contiguous along
// the outer dimension (mode 2, the weight gradients' operands) is staged
// [32 k][outer] and transposed on its way out of LDS (ds_read_b64_tr_b16:
// lane i of 16 gets element i of the four 16-element rows that the 16 lanes
// address).  Both layouts are permuted by the lanes' source addresses so that
// a fragment read spreads over the LDS banks.  Past M or N the tile is filled
// from rows or runs that exist (they reach only outputs that are not stored);
// a last k-step shorter than 32 (mode 2 only) is zeroed in LDS.  The same
// products in the same order as gemm_bf16_kernel.  Row sums of A (the bias
// gradients) are products with a fragment of ones.
// (The register-staged kernel before it wrote mode 2 to LDS element by
// element.)  us at 4,096 windows, before -> now: dA3 = dH W1 33 -> 28, dW1
// 49 -> 38, dW3 32 -> 29, dH 18 -> 11, conv1's weight gradient 31 -> 28; at
// 1,000 windows, where the batch's odd contractions took the general kernel:
// dW1 31 -> 22, dWh 29 -> 12, dW3 26 -> 21.  The 27 MB masks and outputs
// bound the conv input gradients (20 and 18 us against 17), the partials and
// LDS latency the weight gradients.
// Tiles of 128 x 128, for small outputs 64 x 64, for an FP32 right operand
// 64 x 128 (conv1's weight gradient, 64 x 100: one tile); waves 2 x 2.
// LDS byte address of a shared array (applied to the array itself).
template <class T>
__device__ __forceinline__ uint32_t lds_addr(T* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) T*)p;
}

// 16 bytes per lane from src straight to LDS, at byte address dst (the same
// in every lane) + 16 * lane.  In asm because the builtin makes the compiler
// wait for every such load in flight before most LDS reads; nothing here
// waits for it but dma_barrier (no register is written).  M0 is a reserved
// register: the compiler keeps no value in it, sets it right before each use
// of its own, and ignores it in a clobber list (with a warning).
__device__ __forceinline__ void dma16(const void* src, uint32_t dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(
                   __builtin_amdgcn_readfirstlane(dst)),
               "v"(src)
               : "memory");
}
template <int MODE, int T>
struct DmaOp {
  static constexpr int J = MODE == 3 ? 0 : T / 64;  // 16-byte loads per thread and k-step
  static constexpr int RPI = 1024 / (2 * T);     // mode 2: k rows per wave and load
  static constexpr int LPR = 64 / RPI, SEG = T / 16;
  const char* p[T / 64];
  int64_t ld;  // mode 2: bytes per k row; mode 1: per k-step
  int64_t k0;  // mode 2: this lane's k row of load 0 in k-step 0
  __device__ __forceinline__ void init(const GemmOperand& o, bool is_b, int64_t outer0,
                                       int64_t dim, int64_t kb, int w, int lane) {
    const uint16_t* base = static_cast<const uint16_t*>(o.p);
    if constexpr (MODE == 1) {
      const int64_t os = is_b ? o.cs : o.rs;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int r = (j * 4 + w) * 16 + (lane >> 2);
        const int64_t outer = outer0 + r < dim ? outer0 + r : dim - 1;
        p[j] = reinterpret_cast<const char*>(base + outer * os + kb +
                                             8 * ((lane & 3) ^ ((r >> 1) & 3)));
      }
      ld = 2 * HK;
    } else {
      const int64_t cap = o.ext ? o.ext : dim;  // a multiple of 8, at least dim
      ld = 2 * (is_b ? o.rs : o.cs);
      k0 = kb + w * RPI + lane / LPR;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int k = (j * 4 + w) * RPI + lane / LPR, c = lane % LPR;
        int64_t outer = outer0 + (((c >> 1) ^ (k & (SEG - 1))) * 16) + (c & 1) * 8;
        if (outer > cap - 8) outer = cap - 8;
        p[j] = reinterpret_cast<const char*>(base + outer);
      }
    }
  }
  // k-step i into the stage at LDS address `stage` (rows at or past ke: the
  // last row again)
  __device__ __forceinline__ void issue(uint32_t stage, int i, int64_t ke, int w) const {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const char* src;
      if constexpr (MODE == 1) {
        src = p[j] + i * ld;
      } else {
        int64_t k = k0 + i * HK + j * 4 * RPI;
        if (k > ke - 1) k = ke - 1;
        src = p[j] + k * ld;
      }
      dma16(src, stage + (j * 4 + w) * 1024);
    }
  }
  // fragment of the 16 outer elements of tile t: 8 consecutive k per lane
  static __device__ __forceinline__ uint4 frag(const uint16_t* stage, int t, int lane) {
    if constexpr (MODE == 1) {
      const int r = t * 16 + (lane & 15);
      return *reinterpret_cast<const uint4*>(stage + r * HK + 8 * ((lane >> 4) ^ ((r >> 1) & 3)));
    } else {
      typedef short v4s __attribute__((ext_vector_type(4)));
      const int k = 8 * (lane >> 4) + ((lane & 15) >> 2), c = (lane & 3) * 4;
      uint2 h[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int kk = k + 4 * u;
        h[u] = __builtin_bit_cast(
            uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                       (__attribute__((address_space(3))) v4s*)(stage + kk * T +
                                                                ((t ^ (kk & (SEG - 1))) * 16) + c)));
      }
      return uint4{h[0].x, h[0].y, h[1].x, h[1].y};
    }
  }
  // k rows [rem, 32) of the stage zeroed
  static __device__ __forceinline__ void zero_tail(uint16_t* stage, int rem, int tid) {
    if constexpr (MODE == 2)
      for (int i = rem * (T / 8) + tid; i < HK * (T / 8); i += 256)
        reinterpret_cast<uint4*>(stage)[i] = uint4{0u, 0u, 0u, 0u};
  }
};

// A right operand in FP32 contiguous along n in 8-byte pieces, rows (k)
// possibly grouped (mode 3: the windows), for T-wide tiles: a thread's T / 8
// elements of a k-step (k row tid / 8) through registers, loaded two k-steps
// ahead, zeros at or past ke; stored as mode 2's layout of the kernel's type
// (BF16: rounded to nearest even).
template <int T>
struct RegB {
  static constexpr int CW = T / 8, SEG = T / 16;
  const float* p;
  int64_t k0, grp, gs, rs;
  float2 v[CW / 2];
  int k, c;
  __device__ __forceinline__ void init(const GemmOperand& o, int64_t outer0, int64_t dim,
                                       int64_t kb, int tid) {
    const int64_t cap = o.ext ? o.ext : dim;  // a multiple of CW, at least dim
    k = tid >> 3;
    c = (tid & 7) * CW;
    int64_t outer = outer0 + c;
    if (outer > cap - CW) outer = cap - CW;
    p = static_cast<const float*>(o.p) + outer;
    k0 = kb + k;
    grp = o.grp;
    gs = o.gs;
    rs = o.rs;
  }
  __device__ __forceinline__ void load(int i, int64_t ke) {
    const int64_t r = k0 + (int64_t)i * HK;
    const float2* q =
        reinterpret_cast<const float2*>(p + grouped_row(r < ke ? r : ke - 1, grp, gs, rs));
#pragma unroll
    for (int h = 0; h < CW / 2; ++h) v[h] = q[h];
    if (r >= ke)
#pragma unroll
      for (int h = 0; h < CW / 2; ++h) v[h] = make_float2(0.f, 0.f);
  }
  __device__ __forceinline__ void store(float* stage) const {
    static_assert(T == 64, "FP32 tiles");
    float* d = stage + k * T + (((c >> 4) ^ ((k >> 2) & 3)) * 16) + (c & 15);
    *reinterpret_cast<float4*>(d) = make_float4(v[0].x, v[0].y, v[1].x, v[1].y);
    *reinterpret_cast<float4*>(d + 4) = make_float4(v[2].x, v[2].y, v[3].x, v[3].y);
  }
  __device__ __forceinline__ void store(uint16_t* stage) const {
    uint32_t w[CW / 2];
#pragma unroll
    for (int h = 0; h < CW / 2; ++h)
      w[h] = (uint32_t)to_bf16(v[h].x) | ((uint32_t)to_bf16(v[h].y) << 16);
    uint4* d = reinterpret_cast<uint4*>(stage + k * T + (((c >> 4) ^ (k & (SEG - 1))) * 16) +
                                        (c & 15));
#pragma unroll
    for (int q = 0; q < CW / 8; ++q)
      d[q] = uint4{w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]};
  }
};

// Waits until at most VM of this wave's memory requests are in flight, then
// the workgroup barrier; this wave's LDS reads have returned.
template <int VM>
__device__ __forceinline__ void dma_barrier() {
  static_assert(VM >= 0 && VM <= 4, "requests per k-step");
  if constexpr (VM == 0)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else if constexpr (VM == 1)
    asm volatile("s_waitcnt vmcnt(1) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else if constexpr (VM == 3)
    asm volatile("s_waitcnt vmcnt(3) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else if constexpr (VM == 2)
    asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else
    asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// three stages (A's tile, then B's); afterwards the epilogue's scratch
constexpr int dma_elems(int TM, int TN) { return 3 * (TM + TN) * HK; }

// st: LDS array of dma_elems(TM, TN), at byte address lds; id: the workgroup
// among the nx x ny tiles of k-split z.
// FOLD: the k-steps in runs of g.fold, each run's sums accumulated from zero
// and then added in order, as k-splits of that length and their reduction
// make them.
template <int AM, int BM, int TM, int TN, bool FOLD = false>
__device__ __forceinline__ void gemm_bf16_dma_tile(const GemmArgs& g, uint16_t* st, uint32_t lds,
                                                   int64_t id, int64_t nx, int64_t ny, int64_t z) {
  using OA = DmaOp<AM, TM>;
  using OB = DmaOp<BM, TN>;
  constexpr int MI = TM / 32, NI = TN / 32;  // 16-wide tiles per wave
  constexpr int SN = (TM + TN) * HK;
  static_assert(3 * SN >= 2 * epilogue_floats<TN>(), "epilogue scratch");
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int64_t tm, tn;
  xcd_tile(id, nx, ny, &tm, &tn);
  const int64_t m0 = tm * TM, n0 = tn * TN;
  const int wm = wave >> 1, wn = wave & 1;
  int64_t kb, ke;
  k_range(g, HK, z, &kb, &ke);
  v4f acc[MI][NI], rs[MI], tot[FOLD ? MI : 1][FOLD ? NI : 1] = {};
  int left = FOLD ? g.fold : 0;  // k-steps to the end of the run
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    rs[i] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  const int n = (int)((ke - kb + HK - 1) / HK);
  // the workgroups of the first column of tiles also sum A's rows
  const bool do_rs = g.rowsum != nullptr && tn == 0 && wn == 0;
  if (n > 0) {
    OA pa;
    OB pb;
    const int w = __builtin_amdgcn_readfirstlane(wave);
    pa.init(g.A, false, m0, g.M, kb, w, lane);
    RegB<TN> r3;
    if constexpr (BM == 3)
      r3.init(g.B, n0, g.N, kb, tid);
    else
      pb.init(g.B, true, n0, g.N, kb, w, lane);
    auto issue = [&](int i, int stage) __attribute__((always_inline)) {
      pa.issue(lds + stage * 2 * SN, i, ke, w);
      if constexpr (BM != 3) pb.issue(lds + stage * 2 * SN + 2 * TM * HK, i, ke, w);
    };
    auto compute = [&](const uint16_t* s) __attribute__((always_inline)) {
      uint4 af[MI], bf[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) af[i] = OA::frag(s, wm * MI + i, lane);
#pragma unroll
      for (int j = 0; j < NI; ++j) bf[j] = OB::frag(s + TM * HK, wn * NI + j, lane);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf_t, af[i]),
                                                             __builtin_bit_cast(v8bf_t, bf[j]),
                                                             acc[i][j], 0, 0, 0);
      if (do_rs) {
        const uint4 one = uint4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
#pragma unroll
        for (int i = 0; i < MI; ++i)
          rs[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf_t, af[i]),
                                                         __builtin_bit_cast(v8bf_t, one), rs[i],
                                                         0, 0, 0);
      }
      if constexpr (FOLD)
        if (--left == 0) {
          left = g.fold;
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
              tot[i][j] += acc[i][j];
              acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
            }
        }
    };
    // k-step i reads stage i % 3 (cur) once its loads have landed everywhere;
    // then the stage of step i - 1 (nxt), which every wave has read, takes
    // step i + 2's
    constexpr int L = OA::J + OB::J;  // loads per thread and k-step
    const int rem = (int)(ke - kb - (int64_t)(n - 1) * HK);
    auto step = [&](int i, uint16_t* cur, int nxt) __attribute__((always_inline)) {
      if (i + 1 < n) {
        dma_barrier<L>();
        if (i + 2 < n) issue(i + 2, nxt);
        if constexpr (BM == 3) {
          // (every wave has read the last use of the stage after cur)
          r3.store(st + (nxt == 0 ? 2 : nxt == 1 ? 0 : 1) * SN + TM * HK);
          if (i + 2 < n) r3.load(i + 2, ke);
        }
      } else {
        dma_barrier<0>();
        if (rem < HK) {
          OA::zero_tail(cur, rem, tid);
          if constexpr (BM != 3) OB::zero_tail(cur + TM * HK, rem, tid);
          __syncthreads();
        }
      }
      compute(cur);
    };
    if constexpr (BM == 3) {
      r3.load(0, ke);
      r3.store(st + TM * HK);
      if (n > 1) r3.load(1, ke);
    }
    issue(0, 0);
    if (n > 1) issue(1, 1);
    for (int i = 0; i < n; i += 3) {
      step(i, st, 2);
      if (i + 1 < n) {
        step(i + 1, st + SN, 0);
        if (i + 2 < n) step(i + 2, st + 2 * SN, 1);
      }
    }
    __syncthreads();
  }
  if constexpr (FOLD)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = tot[i][j] + acc[i][j];
  if (do_rs && (lane & 15) == 0) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + wm * (TM / 2) + i * 16 + 4 * (lane >> 4) + r;
        if (m < g.M) g.rowsum[z * g.M + m] = rs[i][r];
      }
  }
  gemm_tile_epilogue<TM, TN>(g, acc, reinterpret_cast<float*>(st), m0, n0, z, wm, wn, tid, lane);
}

template <int AM, int BM, int TM, int TN, bool FOLD = false>
__global__ void __launch_bounds__(256, TM == 128 ? 3 : 4) gemm_bf16_dma_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(1024))) uint16_t st[dma_elems(TM, TN)];
  gemm_bf16_dma_tile<AM, BM, TM, TN, FOLD>(g, st, lds_addr(st),
                                     (int64_t)blockIdx.y * gridDim.x + blockIdx.x, gridDim.x,
                                     gridDim.y, blockIdx.z);
}

// The FP32 kernel for operands in 16-byte aligned rows, staged straight into
// LDS like gemm_bf16_dma_kernel's: 64 x 64 tiles, 32 k per step, 2 x 2 waves
// of 32 x 32 on mfma_f32_16x16x4.  Mode 1 is staged [outer][32 k] and read in
// 16-byte runs, mode 2 [32 k][outer] and read by the element; mode 3 (the
// right operand: contiguous along n in 8-byte pieces, rows possibly grouped,
// e.g. the windows) as mode 2 but through registers, a k-step ahead (4-byte
// loads straight to LDS took 84 us for conv1's weight gradient of 4,096
// windows).  In a 16-deep block
// lane group g holds k = 4 g + t for the t-th MFMA, in both operands alike.
// Bound by the FP32 matrix rate (at 4,096 windows dA3 = dH W1 376 -> 130 us,
// 108 TFLOP/s; dW1 340 -> 162, its 416 tiles two to some CUs) and at small
// batches by the latency of a k-step (64 windows: head 39 -> 15 us); before
// are gemm_kernel's times.
constexpr int FT = 64;
template <int MODE>
struct DmaF32 {
  static constexpr int J = MODE == 3 ? 0 : 2;  // loads to LDS per thread and k-step
  const char* p[2];
  int64_t ld, k0;
  __device__ __forceinline__ void init(const GemmOperand& o, bool is_b, int64_t outer0,
                                       int64_t dim, int64_t kb, int w, int lane) {
    const float* base = static_cast<const float*>(o.p);
    if constexpr (MODE == 1) {
      const int64_t os = is_b ? o.cs : o.rs;
#pragma unroll
      for (int j = 0; j < 2; ++j) {  // 8 rows of 128 bytes per wave and load
        const int r = (j * 4 + w) * 8 + (lane >> 3);
        const int64_t outer = outer0 + r < dim ? outer0 + r : dim - 1;
        p[j] = reinterpret_cast<const char*>(base + outer * os + kb + 4 * ((lane & 7) ^ (r & 7)));
      }
      ld = 4 * HK;
    } else {
      static_assert(MODE == 2, "mode 3 is staged by RegB");
      const int64_t cap = o.ext ? o.ext : dim;  // a multiple of 4, at least dim
      ld = 4 * (is_b ? o.rs : o.cs);
      k0 = kb + w * 4 + (lane >> 4);
#pragma unroll
      for (int j = 0; j < 2; ++j) {  // 4 k rows of 256 bytes per wave and load
        const int k = (j * 4 + w) * 4 + (lane >> 4), c = lane & 15;
        int64_t outer = outer0 + (((c >> 2) ^ ((k >> 2) & 3)) * 16) + (c & 3) * 4;
        if (outer > cap - 4) outer = cap - 4;
        p[j] = reinterpret_cast<const char*>(base + outer);
      }
    }
  }
  __device__ __forceinline__ void issue(uint32_t stage, int i, int64_t ke, int w) const {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if constexpr (MODE == 1) {
        dma16(p[j] + i * ld, stage + (j * 4 + w) * 1024);
      } else {
        int64_t k = k0 + i * HK + j * 16;
        if (k > ke - 1) k = ke - 1;
        dma16(p[j] + k * ld, stage + (j * 4 + w) * 1024);
      }
    }
  }
  // elements t = 0 .. 3 of block b (16 k) of outer tile `tile`
  static __device__ __forceinline__ v4f frag(const float* stage, int tile, int b, int lane) {
    if constexpr (MODE == 1) {
      const int r = tile * 16 + (lane & 15);
      return *reinterpret_cast<const v4f*>(stage + r * HK + 4 * ((4 * b + (lane >> 4)) ^ (r & 7)));
    } else {
      const int g = lane >> 4;
      const float* q = stage + (16 * b + 4 * g) * FT + ((tile ^ g) * 16) + (lane & 15);
      return v4f{q[0], q[FT], q[2 * FT], q[3 * FT]};
    }
  }
  static __device__ __forceinline__ void zero_tail(float* stage, int rem, int tid) {
    if constexpr (MODE != 1)
      for (int i = rem * (FT / 4) + tid; i < HK * (FT / 4); i += 256)
        reinterpret_cast<uint4*>(stage)[i] = uint4{0u, 0u, 0u, 0u};
  }
};

// The products of F32_RUN k-steps (128 k, the shortest split that gemm_kernel
// makes) are accumulated from zero and the runs' sums then added, so that a
// result's error does not grow with the k that a workgroup takes (its splits
// are for the chip, not for the sums).  Against 64 bits, the head's weight
// gradient over 1,024 windows: gemm_kernel in four splits 2.7e-7, this kernel in
// one chain per split 3.8e-7, in runs 1.9e-7; 4,096 windows 5.2e-7, 7.4e-7, 2.0e-7.
// It costs 0.8 % of a pass of 200 windows (194.3 -> 195.8 us).
constexpr int F32_RUN = 4;
template <int AM, int BM>
__device__ __forceinline__ void gemm_f32_dma_tile(const GemmArgs& g, float* st, uint32_t lds,
                                                  int64_t id, int64_t nx, int64_t ny, int64_t z) {
  using OA = DmaF32<AM>;
  using OB = DmaF32<BM>;
  constexpr int TI = FT / 32, SN = 2 * FT * HK;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int64_t tm, tn;
  xcd_tile(id, nx, ny, &tm, &tn);
  const int64_t m0 = tm * FT, n0 = tn * FT;
  const int wm = wave >> 1, wn = wave & 1;
  int64_t kb, ke;
  k_range(g, HK, z, &kb, &ke);
  v4f acc[TI][TI], tot[TI][TI] = {};
  float rs[TI] = {}, rs_tot[TI] = {};
  int left = F32_RUN;  // k-steps to the end of the run
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TI; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  const int n = (int)((ke - kb + HK - 1) / HK);
  const bool do_rs = g.rowsum != nullptr && tn == 0 && wn == 0;
  if (n > 0) {
    OA pa;
    OB pb;
    const int w = __builtin_amdgcn_readfirstlane(wave);
    pa.init(g.A, false, m0, g.M, kb, w, lane);
    RegB<FT> r3;
    if constexpr (BM == 3)
      r3.init(g.B, n0, g.N, kb, tid);
    else
      pb.init(g.B, true, n0, g.N, kb, w, lane);
    auto issue = [&](int i, int stage) __attribute__((always_inline)) {
      pa.issue(lds + stage * 4 * SN, i, ke, w);
      if constexpr (BM != 3) pb.issue(lds + stage * 4 * SN + 4 * FT * HK, i, ke, w);
    };
    auto compute = [&](const float* s) __attribute__((always_inline)) {
#pragma unroll
      for (int b = 0; b < HK / 16; ++b) {
        v4f af[TI], bf[TI];
#pragma unroll
        for (int i = 0; i < TI; ++i) af[i] = OA::frag(s, wm * TI + i, b, lane);
#pragma unroll
        for (int j = 0; j < TI; ++j) bf[j] = OB::frag(s + FT * HK, wn * TI + j, b, lane);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TI; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i][t], bf[j][t], acc[i][j], 0, 0,
                                                               0);
        if (do_rs)
#pragma unroll
          for (int i = 0; i < TI; ++i) rs[i] += (af[i][0] + af[i][1]) + (af[i][2] + af[i][3]);
      }
      if (--left == 0) {
        left = F32_RUN;
#pragma unroll
        for (int i = 0; i < TI; ++i) {
          rs_tot[i] += rs[i];
          rs[i] = 0.f;
#pragma unroll
          for (int j = 0; j < TI; ++j) {
            tot[i][j] += acc[i][j];
            acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
          }
        }
      }
    };
    constexpr int L = OA::J + OB::J;
    const int rem = (int)(ke - kb - (int64_t)(n - 1) * HK);
    auto step = [&](int i, float* cur, int nxt) __attribute__((always_inline)) {
      if (i + 1 < n) {
        dma_barrier<L>();
        if (i + 2 < n) issue(i + 2, nxt);
        if constexpr (BM == 3) {
          // (every wave has read the last use of the stage after cur)
          r3.store(st + (nxt == 0 ? 2 : nxt == 1 ? 0 : 1) * SN + FT * HK);
          if (i + 2 < n) r3.load(i + 2, ke);
        }
      } else {
        dma_barrier<0>();
        if (rem < HK) {
          OA::zero_tail(cur, rem, tid);
          if constexpr (BM != 3) OB::zero_tail(cur + FT * HK, rem, tid);
          __syncthreads();
        }
      }
      compute(cur);
    };
    if constexpr (BM == 3) {
      r3.load(0, ke);
      r3.store(st + FT * HK);
      if (n > 1) r3.load(1, ke);
    }
    issue(0, 0);
    if (n > 1) issue(1, 1);
    for (int i = 0; i < n; i += 3) {
      step(i, st, 2);
      if (i + 1 < n) {
        step(i + 1, st + SN, 0);
        if (i + 2 < n) step(i + 2, st + 2 * SN, 1);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TI; ++j) acc[i][j] = tot[i][j] + acc[i][j];
  if (do_rs) {
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      float v = rs_tot[i] + rs[i];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      const int64_t m = m0 + wm * (FT / 2) + i * 16 + lane;
      if (lane < 16 && m < g.M) g.rowsum[z * g.M + m] = v;
    }
  }
  gemm_tile_epilogue<FT, FT>(g, acc, st, m0, n0, z, wm, wn, tid, lane);
}

template <int AM, int BM>
__global__ void __launch_bounds__(256, 3) gemm_f32_dma_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(1024))) float st[dma_elems(FT, FT)];
  gemm_f32_dma_tile<AM, BM>(g, st, lds_addr(st), (int64_t)blockIdx.y * gridDim.x + blockIdx.x,
                            gridDim.x, gridDim.y, blockIdx.z);
}

// Several weight gradients (mode 2 both operands, or the windows as mode 3)
// in one launch: workgroups first[p] .. of problem p, k-split by k-split.
// Each alone leaves the chip part idle (80 to 416 workgroups, some with a few
// k-steps, some with hundreds) and ends in a launch that adds its partials;
// together they are one round of workgroups of equal length and one such
// launch (group_reduce), and nothing is left for a second stream to overlap.
// Training step, a launch or two per product on one stream up to 1,024 windows
// (BF16) or 256 (FP32) and on two above -> grouped (us): BF16 16 152 -> 119,
// 512 191 -> 143, 1,024 217 -> 171, 2,048 277 -> 223, 4,096 400 -> 354; FP32 16 197
// -> 154, 256 231 -> 188, 1,024 391 -> 360, 4,096 1,004 -> 983.
template <bool BF>
__global__ void __launch_bounds__(256, 3) gemm_group_kernel(GemmGroup grp) {
  using T = typename std::conditional<BF, uint16_t, float>::type;
  constexpr int SZ = BF ? dma_elems(HB, HB) : dma_elems(FT, FT);
  __shared__ __attribute__((aligned(1024))) T st[SZ];
  int p = 0;
  while (p + 1 < grp.count && (int)blockIdx.x >= grp.at[p + 1].first) ++p;
  const GemmGroup::At at = grp.at[p];
  const int b = (int)blockIdx.x - at.first, tiles = at.nx * at.ny;
  const int z = b / tiles, id = b - z * tiles;
  const GemmArgs& g = grp.g[p];
  if (z >= g.ksplit) return;  // (first is a whole number of XCD rounds)
  const uint32_t lds = lds_addr(st);
  if constexpr (BF) {
    if (at.kind == 0)
      gemm_bf16_dma_tile<2, 2, HB, HB>(g, st, lds, id, at.nx, at.ny, z);
    else if (at.kind == 1)
      gemm_bf16_dma_tile<2, 2, 64, 64>(g, st, lds, id, at.nx, at.ny, z);
    else
      gemm_bf16_dma_tile<2, 3, 64, HB>(g, st, lds, id, at.nx, at.ny, z);
  } else {
    if (at.kind == 1)
      gemm_f32_dma_tile<2, 2>(g, st, lds, id, at.nx, at.ny, z);
    else
      gemm_f32_dma_tile<2, 3>(g, st, lds, id, at.nx, at.ny, z);
  }
}

// Operand access mode for the BF16 kernel (see gemm_bf16_kernel) and the
// vector reads a run of 16 elements allows: 2 = 16-byte, 1 = 8-byte (rows
// of an odd multiple of 8 bytes apart, e.g. windows of 111 x 50 FP32
// features), 0 = none.
static void operand_mode(const GemmOperand& o, bool is_b, int32_t* mode, int32_t* vec) {
  const bool grouped = o.grp < NO_GROUP;
  const int64_t k_stride = is_b ? o.rs : o.cs, outer_stride = is_b ? o.cs : o.rs;
  const bool k_is_row = is_b;  // grouping applies to the row index
  if (k_stride == 1 && !(k_is_row && grouped))
    *mode = 1;
  else if (outer_stride == 1 && !(!k_is_row && grouped))
    *mode = 2;
  else
    *mode = 0;
  const int64_t other = *mode == 1 ? outer_stride : k_stride;
  auto fits = [&](int64_t bytes) {
    const int64_t q = bytes / (o.bf16 ? 2 : 4);  // elements per vector
    return *mode != 0 && (reinterpret_cast<uintptr_t>(o.p) % bytes == 0) && other % q == 0 &&
           (!grouped || o.gs % q == 0);
  };
  *vec = fits(16) ? 2 : fits(8) ? 1 : 0;
}

// Which kernel takes a product: 0 the general ones, 2 the LDS-direct one, 3
// the same with the right operand FP32 in 8-byte pieces along n, rows
// possibly grouped (the windows).  Sets the operands' modes.
static int dma_mode(GemmArgs& g, int bf16_mma) {
  operand_mode(g.A, false, &g.amode, &g.avec);
  operand_mode(g.B, true, &g.bmode, &g.bvec);
  // operands of the form in aligned rows: staged straight into LDS (runs of
  // 16 bytes along the outer dimension within a readable extent; k in whole
  // steps where an operand is contiguous along it)
  auto direct = [&](const GemmOperand& o, int32_t mode, int32_t vec, int64_t dim) {
    const int64_t cap = o.ext ? o.ext : dim;
    return (o.bf16 != 0) == (bf16_mma != 0) && vec == 2 && o.grp >= NO_GROUP &&
           ((mode == 1 && g.K % HK == 0) ||
            (mode == 2 && cap % (o.bf16 ? 8 : 4) == 0 && cap >= dim));
  };
  const int64_t bcap = g.B.ext ? g.B.ext : g.N;
  if (!direct(g.A, g.amode, g.avec, g.M)) return 0;
  if (direct(g.B, g.bmode, g.bvec, g.N)) return 2;
  return !g.B.bf16 && g.bmode == 2 && g.bvec >= 1 && bcap % (bf16_mma ? 16 : 8) == 0 &&
                 bcap >= g.N
             ? 3
             : 0;
}

// Grouped rows are divided in 32 bits.
static bool rows_fit(const GemmArgs& g) {
  const int64_t big = (int64_t)1 << 32;
  return !((g.A.grp < NO_GROUP && g.M >= big) || (g.B.grp < NO_GROUP && g.K >= big) ||
           (g.mask.p && g.mask.grp < NO_GROUP && g.M >= big) || (g.cgrp < NO_GROUP && g.M >= big) ||
           (g.ccg != 0 && (g.ccg < 0 || g.N >= big)));
}

// C permuted whole rows at a time, in 16-byte aligned rows (reduce_gemm_perm4).
static bool perm_rows(const GemmArgs& g) {
  return g.ccg > 0 && g.N == g.ccg * g.ccm && !g.bias && !g.mask.p && !g.c_bf16 &&
         g.cgrp >= NO_GROUP && g.ldc % 4 == 0 && reinterpret_cast<uintptr_t>(g.C) % 16 == 0;
}

// The tiles' vector epilogue: split-K partials in whole 16-byte runs; else no
// bias, N whole 16-column runs, C and the mask in 16-byte aligned rows
// contiguous along n.
static bool vector_epilogue(const GemmArgs& g) {
  const int64_t mq = g.mask.bf16 ? 8 : 4;
  const int64_t cq = g.c_bf16 ? 8 : 4;  // elements per 16 bytes of C
  const bool c_ok = reinterpret_cast<uintptr_t>(g.C) % 16 == 0 && g.ldc % cq == 0 &&
                    (g.cgrp >= NO_GROUP || g.cgs % cq == 0);
  const bool m_ok = !g.mask.p || (g.mask.cs == 1 &&
                                  reinterpret_cast<uintptr_t>(g.mask.p) % 16 == 0 &&
                                  g.mask.rs % mq == 0 &&
                                  (g.mask.grp >= NO_GROUP || g.mask.gs % mq == 0));
  return g.N % 16 == 0 && (g.ksplit > 1 ? reinterpret_cast<uintptr_t>(g.part) % 16 == 0
                                        : !g.bias && g.ccg == 0 && c_ok && m_ok);
}

hipError_t launch_gemm(GemmArgs g, int bf16_mma, float* part, int64_t part_cap,
                       hipStream_t stream) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (!rows_fit(g)) return hipErrorInvalidValue;
  // (a left operand contiguous along the outer dimension, a weight gradient's,
  // goes through launch_gemm_group where the LDS-direct kernels can take it)
  const bool dma = dma_mode(g, bf16_mma) == 2 && g.amode == 1;
  g.rowsum = nullptr;
  auto tiles_of = [&](int64_t tm, int64_t tn) {
    return ((g.M + tm - 1) / tm) * ((g.N + tn - 1) / tn);
  };
  // (64 x 64 tiles where 128 x 128 ones would not fill the chip and k is too
  // short to split)
  const bool small = dma && tiles_of(HB, HB) < 192 && !(part && g.K >= 4096);
  const int T = !bf16_mma ? GB : small ? 64 : HB;
  const int64_t tiles = tiles_of(T, T);
  // split K when the output is too small to fill the chip, at least 8 k-steps
  // each, within the partial buffer: two workgroups per CU
  auto splits = [&](int64_t t, int64_t step) {
    int64_t n = 512 / t;
    const int64_t steps = g.K / (step * 8);
    if (n > steps) n = steps;
    if (n > part_cap / (g.M * g.N)) n = part_cap / (g.M * g.N);
    if (n > 65535) n = 65535;
    return n < 2 ? 1 : n;
  };
  int64_t ks = 1;
  g.fold = 0;
  if (g.c_bf16) {
    // The result is rounded to BF16, so its number of partial sums is part of
    // it: by 128 x 128 tiles whatever the kernel.  64 x 64 tiles add them up
    // themselves (two or three, k is short: a split's launch that adds its
    // partials costs more than it saves, 64 windows' step 114 us against 113,
    // 4,096 345 against 340).
    if (part && tiles_of(HB, HB) < 128) ks = splits(tiles_of(HB, HB), HK);
    if (small && ks > 1) {
      g.fold = (int32_t)(((g.K + ks - 1) / ks + HK - 1) / HK);
      ks = 1;
    }
  } else if (part && tiles < 128) {
    ks = splits(tiles, bf16_mma || dma ? HK : GK);
  }
  g.ksplit = (int32_t)ks;
  g.part = part;
  g.evec = (bf16_mma || dma) && vector_epilogue(g);
  const dim3 grid((unsigned)((g.N + T - 1) / T), (unsigned)((g.M + T - 1) / T), (unsigned)ks);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, g);
  };
  if (!dma)
    bf16_mma ? launch(gemm_bf16_kernel) : launch(gemm_kernel);
  else if (!bf16_mma)
    g.bmode == 1 ? launch(gemm_f32_dma_kernel<1, 1>) : launch(gemm_f32_dma_kernel<1, 2>);
  else if (!small)
    g.bmode == 1 ? launch(gemm_bf16_dma_kernel<1, 1, HB, HB>)
                 : launch(gemm_bf16_dma_kernel<1, 2, HB, HB>);
  else if (g.fold)
    g.bmode == 1 ? launch(gemm_bf16_dma_kernel<1, 1, 64, 64, true>)
                 : launch(gemm_bf16_dma_kernel<1, 2, 64, 64, true>);
  else
    g.bmode == 1 ? launch(gemm_bf16_dma_kernel<1, 1, 64, 64>)
                 : launch(gemm_bf16_dma_kernel<1, 2, 64, 64>);
  if (ks > 1) {
    const int64_t MN = g.M * g.N;
    if (ks < 64 && g.N % 4 == 0 && perm_rows(g))
      hipLaunchKernelGGL(reduce_gemm_perm4, dim3((unsigned)((MN / 4 + 255) / 256)), dim3(256), 0,
                         stream, part, ks, MN, g);
    else if (ks < 64 && g.N % 4 == 0)
      hipLaunchKernelGGL(reduce_gemm_vec4, dim3((unsigned)((MN / 4 + 255) / 256)), dim3(256), 0,
                         stream, part, ks, MN, g);
    else
      launch_reduce<true>(part, ks, MN, MN, g, nullptr, 0, stream);
  }
  return hipGetLastError();
}

// Several lists of partials summed in one launch: workgroup b serves the
// segment whose block range holds b; per segment L lanes per output (16 or
// 64, or 4 for short lists), lane l summing partials c = l, l + L, ... in
// order, then the L lane sums combined by a fixed butterfly.
__device__ __forceinline__ void sum_seg(const SumSegs& segs, int64_t b) {
  int s = 0;
  while (s + 1 < segs.count && b >= segs.seg[s].blocks) {
    b -= segs.seg[s].blocks;
    ++s;
  }
  const SumSeg& q = segs.seg[s];
  const int L = q.lanes, sub = threadIdx.x % L;
  const int64_t n = b * (256 / L) + threadIdx.x / L;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  if (n < q.N) {
    int64_t c = sub;
    for (; c + 3 * L < q.cnt; c += 4 * L) {
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += q.src[(c + u * L) * q.N + n];
    }
    for (; c < q.cnt; c += L) acc[0] += q.src[c * q.N + n];
  }
  float v = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  for (int off = L / 2; off >= 1; off /= 2) v += __shfl_xor(v, off);
  if (sub == 0 && n < q.N) q.out[n] = segs.beta ? q.out[n] + v : v;
}

__global__ void __launch_bounds__(256) sum_partials(SumSegs segs) { sum_seg(segs, blockIdx.x); }

// Lanes and blocks of each list; the blocks in all.
static int64_t plan_sums(SumSegs& segs) {
  int64_t blocks = 0;
  for (int s = 0; s < segs.count; ++s) {
    SumSeg& q = segs.seg[s];
    q.lanes = q.cnt >= 256 ? 64 : q.cnt >= 32 ? 16 : 4;
    q.blocks = (q.N + 256 / q.lanes - 1) / (256 / q.lanes);
    blocks += q.blocks;
  }
  return blocks;
}

// One launch that ends a group of weight gradients: the split-K partials of
// its products added in part order (within one of L lanes, the lanes by a
// fixed butterfly), four adjacent outputs per L lanes, in C's own order where
// its columns are permuted, then the bias sums (sum_seg).
__global__ void __launch_bounds__(256) group_reduce(GemmGroup grp, SumSegs segs) {
  int p = 0;
  int64_t b = blockIdx.x;
  while (p < grp.count && b >= grp.at[p].red_blocks) b -= grp.at[p++].red_blocks;
  if (p == grp.count) {
    sum_seg(segs, b);
    return;
  }
  const GemmArgs& g = grp.g[p];
  const int L = grp.at[p].red_lanes, sub = threadIdx.x % L;
  const int64_t MN = g.M * g.N, q = (b * (256 / L) + threadIdx.x / L) * 4;
  const bool on = q < MN;
  const int64_t m = on ? q / g.N : 0, n = on ? q - m * g.N : 0;
  float a[4] = {0.f, 0.f, 0.f, 0.f};
  if (on && grp.at[p].perm) {
    const float* src[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t d = (uint32_t)n + e, t = d / (uint32_t)g.ccm;
      src[e] = g.part + m * g.N + (int64_t)(d - t * (uint32_t)g.ccm) * g.ccg + t;
    }
#pragma unroll 4
    for (int c = sub; c < g.ksplit; c += L)
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] += src[e][c * MN];
  } else if (on) {
#pragma unroll 4
    for (int c = sub; c < g.ksplit; c += L) {
      const float4 t = *reinterpret_cast<const float4*>(g.part + c * MN + q);
      a[0] += t.x;
      a[1] += t.y;
      a[2] += t.z;
      a[3] += t.w;
    }
  }
  for (int off = L / 2; off >= 1; off /= 2)
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] += __shfl_xor(a[e], off);
  if (!on || sub != 0) return;
  if (grp.at[p].perm) {
    float4* c = reinterpret_cast<float4*>(g.C + m * g.ldc + n);
    float4 o = make_float4(a[0], a[1], a[2], a[3]);
    if (g.beta) {
      const float4 was = *c;
      o = make_float4(was.x + o.x, was.y + o.y, was.z + o.z, was.w + o.w);
    }
    *c = o;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) gemm_store(g, m, n + e, a[e]);
  }
}

// Workgroups a group's work is split for, in equal numbers of k-steps: BF16 two
// per CU (us per training step of 4,096 windows: 512 359, 640 379, 1,536 390;
// of 1,024: 171, 175, 183), FP32, whose tiles are a quarter the size, six
// (512 1,071, 1,024 1,009, 1,536 983, 2,048 972; of 1,024 windows 376, 365, 360,
// 368).  A k-step with the windows operand, through registers and half as
// much again to read, counts GROUP_X_COST times (BF16, 4,096 windows: 1 397,
// 2 359, 3 354, 4 354).  BF16 groups of less than GROUP_SMALL tiles' k-steps (about
// 560 windows) take 64 x 64 tiles (512 windows: 143 against 151 with 128 x 128).
constexpr int64_t GROUP_WGS_BF16 = 512, GROUP_WGS_F32 = 1536, GROUP_X_COST = 3,
                  GROUP_SMALL = 4096;

bool groups(GemmArgs g, int bf16_mma) {
  return g.M > 0 && g.N > 0 && g.K > 0 && g.N % 4 == 0 && rows_fit(g) &&
         dma_mode(g, bf16_mma) != 0 && g.amode == 2 && g.bmode == 2;
}

hipError_t launch_gemm_group(GemmGroup& grp, int bf16_mma, float* part, int64_t part_cap,
                             SumSegs& segs, hipStream_t stream) {
  // k-steps times tiles of the whole group, in 128 x 128 tiles (BF16) or 64 x 64
  // (FP32), to be spread over the workgroups the chip holds
  auto tiles_of = [](const GemmArgs& g, int64_t tm, int64_t tn) {
    return ((g.M + tm - 1) / tm) * ((g.N + tn - 1) / tn);
  };
  const int64_t T = bf16_mma ? HB : FT;
  int mode[GemmGroup::MAX];
  int64_t work = 0;
  for (int p = 0; p < grp.count; ++p) {
    GemmArgs& g = grp.g[p];
    mode[p] = dma_mode(g, bf16_mma);
    const int64_t tm = mode[p] == 3 ? 64 : T, tn = T;
    work += tiles_of(g, tm, tn) * ((g.K + HK - 1) / HK);
  }
  const bool small = bf16_mma && work < GROUP_SMALL;
  // k-steps a workgroup: at least 8
  int64_t per = work / (bf16_mma ? GROUP_WGS_BF16 : GROUP_WGS_F32);
  if (per < 8) per = 8;
  // (scratch kept for the products after this one, 64 splits of a small output)
  int64_t later[GemmGroup::MAX] = {};
  for (int p = grp.count - 2; p >= 0; --p) {
    const int64_t MN = grp.g[p + 1].M * grp.g[p + 1].N;
    later[p] = later[p + 1] + (MN <= 16 * 1024 ? 256 : MN <= 64 * 1024 ? 64 : 1) * ((MN + 63) / 64 * 64);
  }
  int64_t first = 0, red = 0;
  for (int p = 0; p < grp.count; ++p) {
    GemmArgs& g = grp.g[p];
    GemmGroup::At& at = grp.at[p];
    at.kind = mode[p] == 3 ? 2 : !bf16_mma || small ? 1 : 0;
    const int64_t tm = at.kind == 0 ? HB : 64, tn = at.kind == 1 ? 64 : T;
    const int64_t steps = (g.K + HK - 1) / HK, MN = g.M * g.N;
    const int64_t mine = mode[p] == 3 ? std::max<int64_t>(per / GROUP_X_COST, 8) : per;
    int64_t ks = (steps + mine - 1) / mine;
    if (ks > GROUP_SPLITS) ks = GROUP_SPLITS;
    const int64_t each = (MN + 63) / 64 * 64, room = part_cap - later[p];
    if (ks > room / each) ks = room / each;
    if (ks < 2) ks = 1;
    // (a large permuted output in two splits, stored whole rows at a time by
    // group_reduce, rather than element by element: FP32, 256 windows, 177 -> 172)
    if (ks < 2 && steps > 1 && MN > 64 * 1024 && perm_rows(g) && room / each >= 2) ks = 2;
    g.ksplit = (int32_t)ks;
    g.part = part;
    if (ks > 1) {
      part += ks * each;
      part_cap -= ks * each;
    }
    g.evec = vector_epilogue(g);
    at.nx = (int32_t)((g.N + tn - 1) / tn);
    at.ny = (int32_t)((g.M + tm - 1) / tm);
    at.first = (int32_t)first;
    first += ((int64_t)at.nx * at.ny * ks + 7) / 8 * 8;
    at.perm = perm_rows(g);
    at.red_lanes = ks < 8 ? 1 : ks < 32 ? 4 : ks < 128 ? 16 : 64;
    at.red_blocks = ks > 1 ? (int32_t)((MN / 4 + 256 / at.red_lanes - 1) / (256 / at.red_lanes)) : 0;
    red += at.red_blocks;
    if (g.rowsum) segs.seg[grp.bias[p]].cnt = ks;
  }
  if (first > INT32_MAX || red > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(bf16_mma ? gemm_group_kernel<true> : gemm_group_kernel<false>,
                     dim3((unsigned)first), dim3(256), 0, stream, grp);
  red += plan_sums(segs);
  if (red > 0)
    hipLaunchKernelGGL(group_reduce, dim3((unsigned)red), dim3(256), 0, stream, grp, segs);
  return hipGetLastError();
}

// Per latency type t the head outputs are n_bins class logits and one
// regression output; loss = CE(class min(lat, n_bins - 1)) + |reg -
// log1p(lat)| summed over t; dz = (softmax - onehot) / B, dreg = sign / B.
// One wavefront per (window, t), its logits held in registers (LOSS_PER per
// lane, lane l taking bins l, l + 64, ...), max and sum of exponentials
// reduced across the wave by a fixed butterfly; four waves (two windows) per
// workgroup, each window's two terms added in t order.
constexpr int LOSS_PER = 8;  // bins per lane: n_bins <= 64 * LOSS_PER
__global__ void __launch_bounds__(256)
    loss_kernel(const float* __restrict__ z, const int32_t* __restrict__ lat, int64_t B,
                int32_t n_bins, float* __restrict__ loss_b, float* __restrict__ dz) {
  __shared__ float part[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t b = (int64_t)blockIdx.x * 2 + (w >> 1);
  const int t = w & 1;
  const int per = n_bins + 1;
  float term = 0.f;
  if (b < B) {
    const float* zt = z + (b * 2 + t) * per;
    const int l = lat[b * 2 + t];
    const int bin = l < n_bins - 1 ? l : n_bins - 1;
    float v[LOSS_PER];
    float m = -INFINITY;
#pragma unroll
    for (int q = 0; q < LOSS_PER; ++q) {
      const int i = lane + 64 * q;
      v[q] = i < n_bins ? zt[i] : -INFINITY;
      m = fmaxf(m, v[q]);
    }
    for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    float se = 0.f;
#pragma unroll
    for (int q = 0; q < LOSS_PER; ++q)
      if (lane + 64 * q < n_bins) se += expf(v[q] - m);
    for (int o = 32; o >= 1; o >>= 1) se += __shfl_xor(se, o);
    const float lse = m + logf(se);
    const float zr = zt[n_bins], zb = zt[bin];
    const float r = zr - log1pf((float)l);
    const float inv = 1.f / (float)B;
    float* dzt = dz + (b * 2 + t) * per;
#pragma unroll
    for (int q = 0; q < LOSS_PER; ++q) {
      const int i = lane + 64 * q;
      if (i < n_bins) dzt[i] = inv * (expf(v[q] - lse) - (i == bin ? 1.f : 0.f));
    }
    if (lane == 0) dzt[n_bins] = inv * (r > 0.f ? 1.f : (r < 0.f ? -1.f : 0.f));
    term = lse - zb + fabsf(r);
  }
  if (lane == 0) part[w] = term;
  __syncthreads();
  if ((threadIdx.x & 127) == 0 && b < B) loss_b[b] = part[w] + part[w + 1];
}

// loss = mean of per-window losses, summed in a fixed order (one workgroup).
__global__ void __launch_bounds__(256) mean_kernel(const float* __restrict__ v, int64_t n,
                                                   float* __restrict__ out) {
  __shared__ double part[256];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) s += v[i];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = (float)(part[0] / (double)n);
}

hipError_t launch_loss(const float* z, const int32_t* lat, int64_t B, int32_t n_bins,
                       float* loss_b, float* loss, float* dz, hipStream_t stream) {
  if (n_bins < 1 || n_bins > 64 * LOSS_PER) return hipErrorInvalidValue;
  hipLaunchKernelGGL(loss_kernel, dim3((unsigned)((B + 1) / 2)), dim3(256), 0, stream, z, lat, B,
                     n_bins, loss_b, dz);
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(256), 0, stream, loss_b, B, loss);
  return hipGetLastError();
}

// Column sums of Y [M][ld] over rows in a fixed order: chunks of rows
// summed per workgroup, then the chunk partials through sum_partials.
// Partial column sums (rows without whole vectors): workgroup (x, c) sums rows [c*per, (c+1)*per) of
// columns [x*64*V, (x+1)*64*V), V adjacent columns per lane (V = 2 for BF16
// input, read as one 32-bit word), 4 row lanes per column, in a fixed order.
template <bool BF>
__global__ void __launch_bounds__(256) colsum_partial(const void* __restrict__ yv, int64_t M,
                                                      int64_t N, int64_t ld, int64_t per,
                                                      float* __restrict__ part) {
  constexpr int V = BF ? 2 : 1;
  __shared__ float red[4][64 * V];
  const int col = threadIdx.x % 64, lane4 = threadIdx.x / 64;
  const int64_t n = ((int64_t)blockIdx.x * 64 + col) * V;
  const int64_t c = blockIdx.y, lo = c * per, hi = lo + per < M ? lo + per : M;
  float acc[2][V];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[0][v] = acc[1][v] = 0.f;
  auto add = [&](int slot, int64_t m) {
    if constexpr (BF) {
      const uint16_t* y = static_cast<const uint16_t*>(yv) + m * ld + n;
      if (n + 1 < N) {  // (ld and n even: 4-byte aligned)
        const uint32_t w = *reinterpret_cast<const uint32_t*>(y);
        acc[slot][0] += __uint_as_float(w << 16);
        acc[slot][1] += __uint_as_float(w & 0xffff0000u);
      } else {
        acc[slot][0] += __uint_as_float((uint32_t)y[0] << 16);
      }
    } else {
      acc[slot][0] += static_cast<const float*>(yv)[m * ld + n];
    }
  };
  if (n < N) {
    int64_t m = lo + lane4;
    for (; m + 4 < hi; m += 8) {
      add(0, m);
      add(1, m + 4);
    }
    for (; m < hi; m += 4) add(0, m);
  }
#pragma unroll
  for (int v = 0; v < V; ++v) red[lane4][col * V + v] = acc[0][v] + acc[1][v];
  __syncthreads();
  if (lane4 == 0)
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (n + v < N)
        part[c * N + n + v] = (red[0][col * V + v] + red[1][col * V + v]) +
                              (red[2][col * V + v] + red[3][col * V + v]);
}

// Partial column sums for rows whose columns come in whole VB-byte vectors
// (VW columns each).  Workgroup (x, c) takes column block x (TPR vectors side
// by side) and rows [c*per, min(M, (c+1)*per)): RP = 256 / TPR row lanes,
// lane r summing rows lo + r, lo + r + RP, ... in order, four requests in
// flight; the RP lane sums are combined by a fixed pairwise tree in LDS into
// part[c][n], which sum_partials then adds over c.  (A single launch in
// which the last workgroup of a block adds the partials was slower: the
// device-scope release each workgroup needs before counting writes back its
// XCD's whole L2.)
template <bool BF, int VB>
struct ColVec {
  static constexpr int VW = VB / (BF ? 2 : 4);
  using T = typename std::conditional<VB == 16, uint4, uint2>::type;
  __device__ static __forceinline__ T load(const void* y, int64_t at) {
    return *reinterpret_cast<const T*>(static_cast<const char*>(y) + at * (BF ? 2 : 4));
  }
  __device__ static __forceinline__ void add(float (&a)[VW], const T& t) {
    const uint32_t* w = reinterpret_cast<const uint32_t*>(&t);
#pragma unroll
    for (int q = 0; q < VB / 4; ++q) {
      if constexpr (BF) {
        a[2 * q] += __uint_as_float(w[q] << 16);
        a[2 * q + 1] += __uint_as_float(w[q] & 0xffff0000u);
      } else {
        a[q] += __uint_as_float(w[q]);
      }
    }
  }
};

template <int VW>
__device__ __forceinline__ void lane_tree(float (&a)[VW], float* red, int r, int j, int tpr,
                                          int rp) {
#pragma unroll
  for (int v = 0; v < VW; ++v) red[(r * tpr + j) * VW + v] = a[v];
  __syncthreads();
  for (int h = rp / 2; h >= 1; h /= 2) {
    if (r < h)
#pragma unroll
      for (int v = 0; v < VW; ++v)
        red[(r * tpr + j) * VW + v] += red[((r + h) * tpr + j) * VW + v];
    __syncthreads();
  }
#pragma unroll
  for (int v = 0; v < VW; ++v) a[v] = red[j * VW + v];
}

template <bool BF, int VB>
__global__ void __launch_bounds__(256) colsum_vec(const void* __restrict__ y, int64_t M, int64_t N,
                                                  int64_t ld, int64_t per, int tpr,
                                                  float* __restrict__ part) {
  using V = ColVec<BF, VB>;
  constexpr int VW = V::VW;
  __shared__ float red[256 * VW];
  const int tid = threadIdx.x, j = tid % tpr, r = tid / tpr, rp = 256 / tpr;
  const int64_t n = (int64_t)blockIdx.x * tpr * VW + j * VW;
  const int64_t c = blockIdx.y, lo = c * per, hi = lo + per < M ? lo + per : M;
  const bool on = n < N;
  float a[VW];
#pragma unroll
  for (int v = 0; v < VW; ++v) a[v] = 0.f;
  if (on) {
    int64_t m = lo + r;
    for (; m + 3 * rp < hi; m += 4 * rp) {
      const typename V::T t0 = V::load(y, m * ld + n), t1 = V::load(y, (m + rp) * ld + n),
                          t2 = V::load(y, (m + 2 * rp) * ld + n),
                          t3 = V::load(y, (m + 3 * rp) * ld + n);
      V::add(a, t0);
      V::add(a, t1);
      V::add(a, t2);
      V::add(a, t3);
    }
    for (; m < hi; m += rp) V::add(a, V::load(y, m * ld + n));
  }
  lane_tree<VW>(a, red, r, j, tpr, rp);
  if (r == 0 && on)
#pragma unroll
    for (int v = 0; v < VW; ++v) part[c * N + n + v] = a[v];
}

hipError_t launch_colsum_partial(const void* y, int y_bf16, int64_t M, int64_t N, int64_t ld,
                                 float* work, int64_t* chunks_out, hipStream_t stream) {
  *chunks_out = 0;
  if (N <= 0) return hipSuccess;
  {
    // whole vectors along the rows: 16 bytes, else 8
    const int es = y_bf16 ? 2 : 4;
    const uintptr_t a = reinterpret_cast<uintptr_t>(y);
    auto fits = [&](int vb) {
      const int64_t vw = vb / es;
      return a % vb == 0 && N % vw == 0 && ld % vw == 0;
    };
    const int vb = fits(16) ? 16 : fits(8) ? 8 : 0;
    if (vb && M > 0) {
      const int vw = vb / es;
      int tpr = 1;
      while (tpr < 64 && (int64_t)tpr * vw < N) tpr *= 2;
      const int rp = 256 / tpr;
      const int64_t blocks = (N + (int64_t)tpr * vw - 1) / ((int64_t)tpr * vw);
      if (blocks <= 65535) {
        int64_t chunks = (M + rp * 8 - 1) / (rp * 8);  // about 8 rows per lane
        if (chunks > COLSUM_MAX_CHUNKS) chunks = COLSUM_MAX_CHUNKS;
        const int64_t per = (M + chunks - 1) / chunks;
        chunks = (M + per - 1) / per;
        const dim3 grid((unsigned)blocks, (unsigned)chunks);
#define SIMNET_COLSUM(BF, VB)                                                                   \
  hipLaunchKernelGGL((colsum_vec<BF, VB>), grid, dim3(256), 0, stream, y, M, N, ld, per, tpr, \
                     work)
        if (y_bf16 && vb == 16) SIMNET_COLSUM(true, 16);
        else if (y_bf16) SIMNET_COLSUM(true, 8);
        else if (vb == 16) SIMNET_COLSUM(false, 16);
        else SIMNET_COLSUM(false, 8);
#undef SIMNET_COLSUM
        *chunks_out = chunks;
        return hipGetLastError();
      }
    }
  }
  int64_t chunks = (M + 63) / 64;
  if (chunks > COLSUM_MAX_CHUNKS) chunks = COLSUM_MAX_CHUNKS;
  if (chunks < 1) chunks = 1;
  const int64_t per = (M + chunks - 1) / chunks;
  // (BF16: two adjacent columns per lane, which needs even N and ld)
  if (y_bf16 && N % 2 == 0 && ld % 2 == 0)
    hipLaunchKernelGGL(colsum_partial<true>, dim3((unsigned)((N + 127) / 128), (unsigned)chunks),
                       dim3(256), 0, stream, y, M, N, ld, per, work);
  else if (y_bf16)
    return hipErrorInvalidValue;
  else
    hipLaunchKernelGGL(colsum_partial<false>, dim3((unsigned)((N + 63) / 64), (unsigned)chunks),
                       dim3(256), 0, stream, y, M, N, ld, per, work);
  *chunks_out = chunks;
  return hipGetLastError();
}

hipError_t launch_sum_partials(SumSegs segs, hipStream_t stream) {
  if (segs.count < 1 || segs.count > SumSegs::MAX) return hipErrorInvalidValue;
  const int64_t blocks = plan_sums(segs);
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(sum_partials, dim3((unsigned)blocks), dim3(256), 0, stream, segs);
  return hipGetLastError();
}

// dst[r][c] = src[r][c] for c < cols, 0 for cols <= c < ld: rows padded to
// a stride whose 16-byte vectors the GEMM operand reads can use.
// One workgroup row per matrix row (grid x), 256 columns per workgroup
// (grid y).
__global__ void pad_rows(const float* __restrict__ src, int64_t cols, int64_t ld,
                         void* __restrict__ dst, int32_t dst_bf16) {
  const int64_t r = blockIdx.x, c = (int64_t)blockIdx.y * 256 + threadIdx.x;
  if (c >= ld) return;
  const float v = c < cols ? src[r * cols + c] : 0.f;
  if (dst_bf16)
    static_cast<uint16_t*>(dst)[r * ld + c] = to_bf16(v);
  else
    static_cast<float*>(dst)[r * ld + c] = v;
}

// The same for an even number of columns in 8-byte aligned rows, with the
// column sums of each chunk of `per` rows (grid y) in part[chunk][cols] on
// the way: 128 columns per workgroup, 4 row lanes, combined as in colsum_vec.
__global__ void __launch_bounds__(256) pad_rows_sum(const float* __restrict__ src, int64_t rows,
                                                    int64_t cols, int64_t ld, int64_t per,
                                                    void* __restrict__ dst, int32_t dst_bf16,
                                                    float* __restrict__ part) {
  __shared__ float red[512];
  const int j = threadIdx.x % 64, r = threadIdx.x / 64;
  const int64_t n = (int64_t)blockIdx.x * 128 + 2 * j;
  const int64_t c = blockIdx.y, lo = c * per, hi = lo + per < rows ? lo + per : rows;
  float a[2] = {0.f, 0.f};
  if (n < ld) {
#pragma unroll 4
    for (int64_t m = lo + r; m < hi; m += 4) {
      float2 v = make_float2(0.f, 0.f);
      if (n < cols) v = *reinterpret_cast<const float2*>(src + m * cols + n);
      if (dst_bf16)
        *reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(dst) + m * ld + n) =
            (uint32_t)to_bf16(v.x) | ((uint32_t)to_bf16(v.y) << 16);
      else
        *reinterpret_cast<float2*>(static_cast<float*>(dst) + m * ld + n) = v;
      a[0] += v.x;
      a[1] += v.y;
    }
  }
  lane_tree<2>(a, red, r, j, 64, 4);
  if (r == 0 && n < cols) *reinterpret_cast<float2*>(part + c * cols + n) = make_float2(a[0], a[1]);
}

hipError_t launch_pad_rows_sum(const float* src, int64_t rows, int64_t cols, int64_t ld, void* dst,
                               int32_t dst_bf16, float* work, int64_t* chunks,
                               hipStream_t stream) {
  if (rows <= 0 || cols % 2 || ld % 2 || reinterpret_cast<uintptr_t>(src) % 8 ||
      (ld + 127) / 128 > INT32_MAX) {
    const hipError_t e = launch_pad_rows(src, rows, cols, ld, dst, dst_bf16, stream);
    return e != hipSuccess ? e : launch_colsum_partial(src, 0, rows, cols, cols, work, chunks, stream);
  }
  int64_t n = (rows + 31) / 32;  // about 8 rows per lane
  if (n > COLSUM_MAX_CHUNKS) n = COLSUM_MAX_CHUNKS;
  const int64_t per = (rows + n - 1) / n;
  *chunks = (rows + per - 1) / per;
  hipLaunchKernelGGL(pad_rows_sum, dim3((unsigned)((ld + 127) / 128), (unsigned)*chunks), dim3(256),
                     0, stream, src, rows, cols, ld, per, dst, dst_bf16, work);
  return hipGetLastError();
}

hipError_t launch_pad_rows(const float* src, int64_t rows, int64_t cols, int64_t ld, void* dst,
                           int32_t dst_bf16, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  if (rows > INT32_MAX || (ld + 255) / 256 > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pad_rows, dim3((unsigned)rows, (unsigned)((ld + 255) / 256)), dim3(256), 0,
                     stream, src, cols, ld, dst, dst_bf16);
  return hipGetLastError();
}

// dst[i] = src[map[i]] (0 where map < 0), stored as FP32 or BF16 (nearest
// even), for several (map, n, dst) segments from one source in one launch:
// workgroup b serves the segment whose block range holds b (segments in
// order, each rounded up to whole workgroups).
__global__ void map_gather_multi(const float* __restrict__ src, GatherSegs segs) {
  int s = 0;
  int64_t b = blockIdx.x;
  while (s + 1 < segs.count && b >= (segs.seg[s].n + 255) / 256) {
    b -= (segs.seg[s].n + 255) / 256;
    ++s;
  }
  const GatherSeg& g = segs.seg[s];
  const int64_t i = b * 256 + threadIdx.x;
  if (i >= g.n) return;
  const int32_t k = g.map[i];
  const float v = k < 0 ? 0.f : src[k];
  if (g.bf16) {
    const uint32_t u = __float_as_uint(v);
    static_cast<uint16_t*>(g.dst)[i] = (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
  } else {
    static_cast<float*>(g.dst)[i] = v;
  }
}

hipError_t launch_map_gather_multi(const float* src, const GatherSegs& segs, hipStream_t stream) {
  if (segs.count < 1 || segs.count > GatherSegs::MAX) return hipErrorInvalidValue;
  int64_t blocks = 0;
  for (int s = 0; s < segs.count; ++s) blocks += (segs.seg[s].n + 255) / 256;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(map_gather_multi, dim3((unsigned)blocks), dim3(256), 0, stream, src, segs);
  return hipGetLastError();
}

// Columns from .. ld - 1 of every row of p [rows][ld] cleared.
__global__ void __launch_bounds__(256) zero_columns(float* __restrict__ p, int64_t rows, int64_t ld,
                                                    int64_t from) {
  const int64_t n = ld - from, total = rows * n;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * 256) {
    const int64_t r = i / n;
    p[r * ld + from + (i - r * n)] = 0.f;
  }
}

hipError_t launch_zero_columns(float* p, int64_t rows, int64_t ld, int64_t from,
                               hipStream_t stream) {
  if (rows <= 0 || from >= ld) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((rows * (ld - from) + 255) / 256, 4096);
  hipLaunchKernelGGL(zero_columns, dim3((unsigned)blocks), dim3(256), 0, stream, p, rows, ld, from);
  return hipGetLastError();
}

// One Adam step (Kingma & Ba, bias corrections c1 = 1 - b1^t, c2 = 1 -
// b2^t, no weight decay) on values: the moments updated in place, the new
// weight returned.  Every Adam kernel here applies this one function with
// contraction into fused multiply-adds off, so they all round alike.
__device__ __forceinline__ float adam_math(float gi, float& mi, float& vi, float wi, float lr,
                                           float b1, float b2, float eps, float c1, float c2) {
#pragma clang fp contract(off)
  mi = b1 * mi + (1.f - b1) * gi;
  vi = b2 * vi + (1.f - b2) * gi * gi;
  return wi - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Adam on FP32 master weights, step t >= 1.
__global__ void adam_kernel(float* __restrict__ w, const float* __restrict__ g,
                            float* __restrict__ m, float* __restrict__ v, int64_t n, float lr,
                            float b1, float b2, float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float mi = m[i], vi = v[i];
  const float wi = adam_math(g[i], mi, vi, w[i], lr, b1, b2, eps, c1, c2);
  m[i] = mi;
  v[i] = vi;
  w[i] = wi;
}

// adam_math on parameter i: moments stored, the new weight returned (and
// not yet stored).
__device__ __forceinline__ float adam_one(const float* __restrict__ w,
                                          const float* __restrict__ g, float* __restrict__ m,
                                          float* __restrict__ v, int64_t i, float lr, float b1,
                                          float b2, float eps, float c1, float c2) {
  float mi = m[i], vi = v[i];
  const float wi = adam_math(g[i], mi, vi, w[i], lr, b1, b2, eps, c1, c2);
  m[i] = mi;
  v[i] = vi;
  return wi;
}

// Adam as adam_kernel, the updated weight also written to a context's
// master copy and, where inv gives byte offsets (-1: none), to its packed and
// permuted copies in the form's precision (BF16 rounded to nearest even, as
// map_gather_multi writes them): the update and the re-layout in one pass.
// Index t is parameter t, or t + skip_n from skip_lo on (a range that
// adam_hidden_tile updates).
__device__ __forceinline__ void adam_relayout_one(
    int64_t i, float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
    float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float c1, float c2,
    float* __restrict__ master, const int2* __restrict__ inv, char* __restrict__ packed,
    char* __restrict__ perm, int32_t bf16, int64_t skip_lo, int64_t skip_n) {
  if (i >= skip_lo) i += skip_n;
  if (i >= n) return;
  const float wi = adam_one(w, g, m, v, i, lr, b1, b2, eps, c1, c2);
  w[i] = wi;
  master[i] = wi;
  const int2 d = inv[i];
  if (bf16) {
    const uint16_t h = to_bf16(wi);
    if (d.x >= 0) *reinterpret_cast<uint16_t*>(packed + d.x) = h;
    if (d.y >= 0) *reinterpret_cast<uint16_t*>(perm + d.y) = h;
  } else {
    if (d.x >= 0) *reinterpret_cast<float*>(packed + d.x) = wi;
    if (d.y >= 0) *reinterpret_cast<float*>(perm + d.y) = wi;
  }
}

// The hidden layer's weights (HO outputs x HC channels x HP positions,
// parameter o*HC*HP + c*HP + p) in tiles of HTO outputs x HTC channels: Adam
// on the tile's rows (contiguous runs of HTC*HP parameters, all of a thread's
// requested before any is used), the new weights to the master copy and to
// LDS, then from LDS to the permuted copy ([p*HC + c][o]: runs of HTO
// outputs) and the packed copy (per position p the K = HC x N = HO fragment
// order of the forward kernels: k-groups of KG channels, 16-output tiles,
// lane (k % KG) / E * 16 + o % 16, element k % E, E = KG / 4: whole 64 x E
// blocks), in the form's precision.
constexpr int HO = 512, HC = 256, HP = 13, HTO = 16, HTC = 32, HROW = HTC * HP + 1;
constexpr int AT = 1024;  // threads
__device__ __forceinline__ void adam_hidden_tile(
    int tile, float* T, float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
    float* __restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2,
    float* __restrict__ master, char* __restrict__ packed, char* __restrict__ perm, int32_t bf16,
    int32_t KG) {
  // T: [o - o0][(c - c0) * HP + p], rows padded by one
  constexpr int NT = HTO * HTC * HP, U = (NT + AT - 1) / AT;
  const int o0 = tile % (HO / HTO) * HTO, c0 = tile / (HO / HTO) * HTC;
  {
    int64_t ii[U];
    float gv[U], mv[U], vv[U], wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = threadIdx.x + u * AT;
      const int r = idx / (HTC * HP), col = idx - r * (HTC * HP);
      ii[u] = (int64_t)(o0 + r) * (HC * HP) + c0 * HP + col;
      if (idx < NT) {
        gv[u] = g[ii[u]];
        mv[u] = m[ii[u]];
        vv[u] = v[ii[u]];
        wv[u] = w[ii[u]];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = threadIdx.x + u * AT;
      if (idx >= NT) continue;
      float mi = mv[u], vi = vv[u];
      const float wi = adam_math(gv[u], mi, vi, wv[u], lr, b1, b2, eps, c1, c2);
      m[ii[u]] = mi;
      v[ii[u]] = vi;
      w[ii[u]] = wi;
      master[ii[u]] = wi;
      const int r = idx / (HTC * HP), col = idx - r * (HTC * HP);
      T[r * HROW + col] = wi;
    }
  }
  __syncthreads();
  // permuted copy: element (p, c, o) at (p*HC + c)*HO + o
  for (int idx = threadIdx.x; idx < NT; idx += AT) {
    const int ol = idx % HTO, rest = idx / HTO, cl = rest % HTC, p = rest / HTC;
    const float x = T[ol * HROW + cl * HP + p];
    const int64_t q = ((int64_t)p * HC + c0 + cl) * HO + o0 + ol;
    if (bf16)
      reinterpret_cast<uint16_t*>(perm)[q] = to_bf16(x);
    else
      reinterpret_cast<float*>(perm)[q] = x;
  }
  // packed copy: per position p, blocks (kg, nt) of 64 lanes x E elements
  const int E = KG / 4, BLK = 64 * E, NKG = HTC / KG, NNT = HTO / 16;
  for (int idx = threadIdx.x; idx < NT; idx += AT) {
    const int blk = idx / BLK, wi = idx - blk * BLK, lane = wi / E, e = wi - lane * E;
    const int ntl = blk % NNT, rest = blk / NNT, kgl = rest % NKG, p = rest / NKG;
    const int kg = c0 / KG + kgl, nt = o0 / 16 + ntl;
    const int c = kg * KG + (lane / 16) * E + e, o = nt * 16 + (lane & 15);
    const float x = T[(o - o0) * HROW + (c - c0) * HP + p];
    const int64_t q = (int64_t)p * (HC * HO) + ((int64_t)(kg * (HO / 16) + nt) * 64 + lane) * E + e;
    if (bf16)
      reinterpret_cast<uint16_t*>(packed)[q] = to_bf16(x);
    else
      reinterpret_cast<float*>(packed)[q] = x;
  }
}

// Both in one launch: workgroups 0 .. hid_tiles - 1 a tile of the hidden layer
// each, the others AT of the remaining parameters.  What bounds it is the
// latency of 16 bytes read and written per parameter: 16 waves per CU with all
// their reads in flight, and one launch (4,096 windows' step: 7 + 25 us as two
// launches of 256 threads with four reads in flight -> 18; 64 windows: 16).
__global__ void __launch_bounds__(AT)
    adam_relayout_kernel(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                         float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps,
                         float c1, float c2, float* __restrict__ master,
                         const int2* __restrict__ inv, char* __restrict__ packed,
                         char* __restrict__ perm, int32_t bf16, int32_t hid_tiles, int64_t hid_off,
                         int64_t hid_n, char* __restrict__ hid_packed,
                         char* __restrict__ hid_perm) {
  __shared__ float T[HTO * HROW];
  const int b = (int)blockIdx.x;
  if (b < hid_tiles)
    adam_hidden_tile(b, T, w + hid_off, g + hid_off, m + hid_off, v + hid_off, lr, b1, b2, eps, c1,
                     c2, master + hid_off, hid_packed, hid_perm, bf16, bf16 ? 32 : 16);
  else
    adam_relayout_one((int64_t)(b - hid_tiles) * AT + threadIdx.x, w, g, m, v, n, lr, b1, b2, eps,
                      c1, c2, master, inv, packed, perm, bf16, hid_off, hid_n);
}

hipError_t launch_adam_relayout(float* w, const float* g, float* m, float* v, int64_t n, float lr,
                                float b1, float b2, float eps, int32_t t, float* master,
                                const int2* inv, void* packed, void* perm, int32_t bf16,
                                int64_t hid_off, void* hid_packed, void* hid_perm,
                                hipStream_t stream) {
  const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
  const int64_t hn = hid_packed ? (int64_t)HO * HC * HP : 0;
  if (hid_packed && (hid_off < 0 || hid_off + hn > n)) return hipErrorInvalidValue;
  const int64_t rest = n - hn;
  const int32_t tiles = hid_packed ? HO / HTO * (HC / HTC) : 0;
  const int64_t blocks = tiles + (rest + AT - 1) / AT;
  if (blocks > 0)
    hipLaunchKernelGGL(adam_relayout_kernel, dim3((unsigned)blocks), dim3(AT), 0, stream, w, g, m, v,
                       n, lr, b1, b2, eps, c1, c2, master, inv, static_cast<char*>(packed),
                       static_cast<char*>(perm), bf16, tiles, hid_packed ? hid_off : n, hn,
                       static_cast<char*>(hid_packed), static_cast<char*>(hid_perm));
  return hipGetLastError();
}

hipError_t launch_adam(float* w, const float* g, float* m, float* v, int64_t n, float lr, float b1,
                       float b2, float eps, int32_t t, hipStream_t stream) {
  const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, w, g, m,
                     v, n, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

}  // namespace simnet

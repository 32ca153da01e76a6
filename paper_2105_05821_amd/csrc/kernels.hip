// HIP kernels of libsimnet.so for gfx950 (CDNA4).
//
// One workgroup owns a tile of MT = 16 sub-traces and runs the whole step
// loop for them inside one launch (persistent: sub-traces are independent,
// Sec. 3.3, so no grid-wide synchronisation is needed).  Each step:
//   gather   - builds the tile's windows block by block straight into LDS
//              from the trace rows (FP32, their BF16 copy in the BF16 form, or
//              packed codes) and the sub-trace's processor queue (Sec. 2.2:
//              current instruction with zero dynamic columns, then the
//              in-flight instructions newest first with residence and
//              execution latency; with store latencies, then the memory
//              write queue);
//   predict  - conv levels as MFMA GEMMs on LDS tiles (Sec. 2.3: kernel 2,
//              stride 2, ReLU), the hidden FC accumulated block by block in
//              MFMA accumulators, the final FC on the VALU (the hybrid head
//              as one MFMA tile row);
//   update   - rounding (or the hybrid head's class choice) and the clock /
//              queue update of Sec. 3.2 in its timestamp form: instruction i
//              enters at T_i = T_{i-1} + F_i and leaves at r_i = max(T_i +
//              E_i + 1, r_{i-1}, r_{i-W} + 1); the queue after the advance is
//              the suffix with r > T_i.
// The queue ring and the per-sub-trace scalars stay in LDS for the whole
// launch and are written back to HBM when the launch ends.  RB7, whose
// residual blocks do not fit this loop, runs each step as four launches
// (the step kernel's stages 1 and 2 around resblock_kernel and
// rb_head_kernel).  Few sub-traces (a slot for each, at most 2,048) take the
// split step of split.hip instead.
//
// Precision forms: weights and activations in FP32, BF16 or FP8 (OCP e4m3,
// per-channel power-of-two scales), products accumulated in FP32 in every
// form; biases and the final logits are FP32.
#include "predict.h"

namespace simnet {

template <class Net, class P>
struct StepSmem {
  static constexpr int CM = Net::MWQ ? Net::C : 1;
  NetSmem<Net, P> net;
  int32_t q_idx[MT][Net::C];
  int32_t q_e[MT][Net::C];
  int64_t q_t[MT][Net::C];
  int64_t q_r[MT][Net::C];
  int64_t rw[MT][WMAX];
  int64_t cur[MT], t_w[MT], r_prev[MT], pos[MT], first[MT], n_pos[MT], pred_off[MT];
  int32_t head[MT], count[MT], warm[MT], active[MT], kid[MT];
  // stores (store latencies only), as in DevState
  int32_t m_idx[MT][CM];
  int32_t m_es[MT][CM];
  int64_t m_t[MT][CM];
  int64_t m_r[MT][CM];
  int64_t m_x[MT][CM];
  int32_t m_head[MT], m_count[MT], m_inpq[MT];
  int64_t x_prev[MT];
};

// Slot s of the tile takes sub-trace k: its scalars come from the global
// state (the reset state for a sub-trace that has not started).
template <class SM>
__device__ __forceinline__ void load_slot(SM& sm, int s, int k, const DevState& st, int W) {
  sm.kid[s] = k;
  if (k < 0) {
    sm.active[s] = 0;
    return;
  }
  sm.cur[s] = st.cur[k];
  sm.t_w[s] = st.t_w[k];
  sm.r_prev[s] = st.r_prev[k];
  sm.pos[s] = st.pos[k];
  sm.first[s] = st.first[k];
  sm.n_pos[s] = st.n_pos[k];
  sm.pred_off[s] = st.pred_off[k];
  sm.head[s] = st.head[k];
  sm.count[s] = st.count[k];
  sm.warm[s] = st.warm[k];
  if (st.m_head) {
    sm.m_head[s] = st.m_head[k];
    sm.m_count[s] = st.m_count[k];
    sm.m_inpq[s] = st.m_inpq[k];
    sm.x_prev[s] = st.x_prev[k];
  }
  for (int i = 0; i < W; ++i) sm.rw[s][i] = st.rw[(size_t)k * WMAX + i];
  sm.active[s] = sm.pos[s] < sm.n_pos[s];
}

// Next unstarted sub-trace in claim order (longest first), or -1.
__device__ __forceinline__ int claim_subtrace(const DevState& st, int n_sub) {
  const unsigned q = atomicAdd(st.next, 1u);
  return q < (unsigned)n_sub ? st.order[q] : -1;
}

template <class Net>
constexpr int n_cal() {
  return Net::D + Net::CH1 + Net::CH2 + Net::CH3 + Net::HID;
}

// BF16 copy of an FP32 trace for the BF16 form: row i's D features rounded
// to BF16 (nearest even, as the window conversion does), then zeros to DS.
__global__ void stage_bf16_kernel(const float* __restrict__ feat, int64_t n, int D, int DS,
                                  uint16_t* __restrict__ out) {
  const int64_t total = n * DS;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / DS;
    const int c = (int)(i - r * DS);
    out[i] = c < D ? PBF16::cvt(feat[r * D + c]) : (uint16_t)0;
  }
}

hipError_t launch_stage_bf16(const float* feat, int64_t n, int D, uint16_t* out,
                             hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(stage_bf16_kernel, dim3(2048), dim3(256), 0, stream, feat, n, D,
                     staged_feat(D), out);
  return hipGetLastError();
}

// DEP: the window carries the memory dependency flags (a separate
// instantiation, so that runs without them pay no registers for them).
// STAGE (networks run as separate kernels per step, one step per launch):
// 1 = gather and convolutions only, the last conv's output to p.trunk_out
// and each slot's activity to p.active_out, the state not advanced;
// 2 = the update from the raw outputs in p.ext_logits, no gather.
template <class Net, class P, bool RUN_NET, bool CAL = false, bool DEP = false, int STAGE = 0>
__global__ void __launch_bounds__(Net::WAVES * 64)
    step_kernel(DevWeights wt, uint32_t relu_mask, DevState st, StepParams p) {
  using G = Geo<Net, P>;
  using T = typename P::T;
  constexpr int C = Net::C, NT = G::NT, D = Net::D, BS = Net::BS;
  __shared__ StepSmem<Net, P> sm;
  __shared__ unsigned cal[CAL ? n_cal<Net>() : 1];
  const int tid = threadIdx.x;
  const int slot0 = blockIdx.x * MT;
  if constexpr (CAL)
    for (int i = tid; i < n_cal<Net>(); i += NT) cal[i] = 0u;

  // Work queue: a slot keeps its sub-trace across launches; an empty slot
  // claims the next unstarted sub-trace (longest first).  Results are
  // indexed by sub-trace, so they do not depend on which slot runs it.
  if (tid < MT) {
    int k = st.slot_kid[slot0 + tid];
    if (k < 0) k = claim_subtrace(st, p.n_sub);
    load_slot(sm, tid, k, st, p.W);
  }
  if constexpr (RUN_NET) sm.net.stage_head(wt, tid, NT);
  __syncthreads();
  for (int i = tid; i < MT * C; i += NT) {
    const int s = i / C, e = i % C, k = sm.kid[s];
    if (k >= 0) {
      const size_t g = (size_t)k * C + e;
      sm.q_idx[s][e] = st.q_idx[g];
      sm.q_e[s][e] = st.q_e[g];
      sm.q_t[s][e] = st.q_t[g];
      sm.q_r[s][e] = st.q_r[g];
      if constexpr (Net::MWQ) {
        sm.m_idx[s][e] = st.m_idx[g];
        sm.m_es[s][e] = st.m_es[g];
        sm.m_t[s][e] = st.m_t[g];
        sm.m_r[s][e] = st.m_r[g];
        sm.m_x[s][e] = st.m_x[g];
      }
    }
  }
  uint32_t n_clamped = 0, n_nonfinite = 0, n_mismatch = 0, n_pred = 0;

  // Window gather: TPR threads per (sub-trace, slot-of-the-group) row, CPT
  // features each.
  using GA = Gather<Net, P>;
  constexpr int GSL = GA::GSL, TPR = GA::TPR, CPT = GA::CPT;
  constexpr bool H16 = GA::H16;
  const int grow = tid / TPR, part = tid % TPR;
  const int gs = grow / GSL, gt = grow % GSL;
  if constexpr (P::SCALED)
    for (int c = tid; c < D; c += NT) sm.net.x_inv[c] = wt.x_inv[c];
  // load(j0, nb): the row's trace index from the queue ring, then the row's
  // features requested (every address in bounds, so all are in flight
  // together); commit: dynamic columns, conversion, one vector store.
  auto load = [&](int j0, int nb) {
    RowRegs<CPT, H16> r;
    const int w = j0 * BS + gt;
    int64_t idx = -1;
    r.res = 0.f;
    r.ex = 0.f;
    r.sto = 0.f;
    if (gt < nb * BS && sm.active[gs]) {
      if (w == 0) {
        idx = sm.first[gs] + sm.pos[gs];
      } else if (w <= sm.count[gs]) {  // processor queue, newest first
        int e = sm.head[gs] + sm.count[gs] - w;
        e = e >= C ? e - C : e;
        idx = sm.q_idx[gs][e];
        r.res = (float)(sm.cur[gs] - sm.q_t[gs][e]);
        const int32_t es = sm.q_e[gs][e];
        r.ex = (float)(Net::MWQ ? es & 0xffff : es);
        if (Net::MWQ) r.sto = (float)((uint32_t)es >> 16);
      } else if (Net::MWQ && w <= sm.count[gs] + sm.m_count[gs] - sm.m_inpq[gs]) {
        // then the memory write queue, newest first: the stores that have
        // left the processor queue and not this one
        int e = sm.m_head[gs] + sm.m_count[gs] - sm.m_inpq[gs] - (w - sm.count[gs]);
        e = e >= C ? e - C : e;
        idx = sm.m_idx[gs][e];
        r.res = (float)(sm.cur[gs] - sm.m_t[gs][e]);
        r.ex = (float)(sm.m_es[gs][e] & 0xffff);
        r.sto = (float)((uint32_t)sm.m_es[gs][e] >> 16);
      }
    }
    request_row<Net, P, DEP>(p, idx, w == 0, sm.active[gs] ? sm.first[gs] + sm.pos[gs] : 0, part,
                             r);
    return r;
  };
  auto commit = [&](int j0, int nb, const RowRegs<CPT, H16>& r, T* X) {
    (void)j0;
    if (gt < nb * BS)  // (slots past a short group's blocks are never read)
      commit_row<Net, P, CAL, DEP>(p, sm.net.x_inv, gs, gt, part, r, X, cal);
  };

  if constexpr (STAGE == 1)
    if (tid < MT) p.active_out[slot0 + tid] = sm.active[tid];
  int any = __syncthreads_or(tid < MT ? sm.active[tid] : 0);

  for (int it = 0; it < p.n_steps && any; ++it) {
    if constexpr (RUN_NET && STAGE == 1) {
      SavePtrs<T> sv{};
      sv.a3 = static_cast<T*>(p.trunk_out) + (size_t)slot0 * Net::NB * Net::CH3;
      sv.rows = MT;
      predict_tile<Net, P, false, true, true>(wt, relu_mask, sm.net, load, commit, nullptr,
                                              nullptr, sv);
      break;  // the update is a separate launch
    } else if constexpr (RUN_NET && STAGE == 0) {
      predict_tile<Net, P, CAL>(wt, relu_mask, sm.net, load, commit, cal, sm.active);
    }

    if (tid < MT && sm.active[tid]) {
      const int s = tid, k = sm.kid[s];
      const int64_t pos = sm.pos[s];
      const int64_t g = sm.pred_off[s] + pos;
      int32_t lat[Net::NLAT];
      if (RUN_NET) {
        const float* z = STAGE == 2 ? p.ext_logits + (size_t)(slot0 + s) * Net::NOUT
                                    : sm.net.logit[s];
        if (p.logits_out)
          for (int o = 0; o < Net::NOUT; ++o) p.logits_out[g * Net::NOUT + o] = z[o];
#pragma unroll
        for (int o = 0; o < Net::NLAT; ++o) {
          if constexpr (Net::HEAD == 1)
            lat[o] = hybrid_latency(z + o * HYB_PER_TYPE, p.lat_max, n_clamped, n_nonfinite);
          else
            lat[o] = round_latency(z[o], p.lat_max, n_clamped, n_nonfinite);
        }
      }
      ++n_pred;  // positions advanced (the work a launch did)
      if (p.lat_mode != 0) {
#pragma unroll
        for (int o = 0; o < Net::NLAT; ++o) {
          const int32_t inj = p.lat_table[g * Net::NLAT + o];
          if (RUN_NET && inj != lat[o]) ++n_mismatch;
          lat[o] = inj;
        }
      }
      const int64_t Tn = sm.cur[s] + lat[0];
      int head = sm.head[s], count = sm.count[s];
      while (count > 0 && sm.q_r[s][head] <= Tn) {  // retired by Tn: a prefix (r is monotone)
        head = head + 1 == C ? 0 : head + 1;
        --count;
      }
      int64_t r = Tn + lat[1] + 1;
      r = r > sm.r_prev[s] ? r : sm.r_prev[s];
      const int wi = (int)(pos % p.W);
      if (pos >= p.W) {
        const int64_t rb = sm.rw[s][wi] + 1;
        r = r > rb ? r : rb;
      }
      sm.rw[s][wi] = r;
      int slot = head + count;
      slot = slot >= C ? slot - C : slot;
      if (count == C) {
        head = head + 1 == C ? 0 : head + 1;  // only the newest C stay visible
      } else {
        ++count;
      }
      const int64_t ii = sm.first[s] + pos;
      sm.q_idx[s][slot] = (int32_t)ii;
      // store latencies: E and S packed as 16-bit halves (lat_max <= 65535)
      sm.q_e[s][slot] = Net::MWQ ? pack_es(lat[1], lat[Net::NLAT - 1]) : lat[1];
      sm.q_t[s][slot] = Tn;
      sm.q_r[s][slot] = r;
      int64_t final_t = r;
      if constexpr (Net::MWQ) {
        // memory write queue (Sec. 3.2): a store enters it when it leaves
        // the processor queue (r) and leaves, in order, once its residence
        // exceeds its store latency: x = max(T + S + 1, r, previous x)
        int mh = sm.m_head[s], mc = sm.m_count[s];
        while (mc > 0 && sm.m_x[s][mh] <= Tn) {  // gone by Tn: a prefix (x is monotone)
          mh = mh + 1 == C ? 0 : mh + 1;
          --mc;
        }
        const bool is_store = p.codes ? code_feature(p.codes[ii], p.store_col) != 0.f
                                      : p.feat[ii * Net::D + p.store_col] != 0.f;
        if (is_store) {
          int64_t x = Tn + lat[2] + 1;
          x = x > r ? x : r;
          x = x > sm.x_prev[s] ? x : sm.x_prev[s];
          sm.x_prev[s] = x;
          int ms = mh + mc;
          ms = ms >= C ? ms - C : ms;
          if (mc == C) {
            mh = mh + 1 == C ? 0 : mh + 1;  // the newest C stores suffice for the window
          } else {
            ++mc;
          }
          sm.m_idx[s][ms] = (int32_t)ii;
          sm.m_es[s][ms] = pack_es(lat[1], lat[2]);
          sm.m_t[s][ms] = Tn;
          sm.m_r[s][ms] = r;
          sm.m_x[s][ms] = x;
        }
        // the newest stores still in the processor queue at Tn (r > Tn)
        int q = 0;
        while (q < mc) {
          int e = mh + mc - 1 - q;
          e = e >= C ? e - C : e;
          if (sm.m_r[s][e] <= Tn) break;
          ++q;
        }
        sm.m_head[s] = mh;
        sm.m_count[s] = mc;
        sm.m_inpq[s] = q;
        final_t = r > sm.x_prev[s] ? r : sm.x_prev[s];
      }
      sm.head[s] = head;
      sm.count[s] = count;
      sm.r_prev[s] = r;
      sm.cur[s] = Tn;
      sm.pos[s] = pos + 1;
      if (pos + 1 == sm.warm[s]) sm.t_w[s] = Tn;
      if (pos + 1 == sm.n_pos[s]) {  // last instruction: the drain ends (Eq. 1)
        st.fetch[k] = Tn - sm.t_w[s];
        st.drain[k] = final_t - Tn;
        st.final_tick[k] = final_t;
        st.warm_tick[k] = sm.t_w[s];
        st.pos[k] = pos + 1;
        st.cur[k] = Tn;
        // the finished sub-trace leaves the batch; the slot takes the next
        load_slot(sm, s, claim_subtrace(st, p.n_sub), st, p.W);
      }
    }
    any = __syncthreads_or(tid < MT ? sm.active[tid] : 0);
  }

  // (stage 1 leaves the state as it found it, apart from the slots' claims)
  if (tid < MT) {
    const int k = sm.kid[tid];
    st.slot_kid[slot0 + tid] = k;
    if (STAGE != 1 && k >= 0) {
      st.cur[k] = sm.cur[tid];
      st.t_w[k] = sm.t_w[tid];
      st.r_prev[k] = sm.r_prev[tid];
      st.pos[k] = sm.pos[tid];
      st.head[k] = sm.head[tid];
      st.count[k] = sm.count[tid];
      if constexpr (Net::MWQ) {
        st.m_head[k] = sm.m_head[tid];
        st.m_count[k] = sm.m_count[tid];
        st.m_inpq[k] = sm.m_inpq[tid];
        st.x_prev[k] = sm.x_prev[tid];
      }
      for (int i = 0; i < p.W; ++i) st.rw[(size_t)k * WMAX + i] = sm.rw[tid][i];
    }
    if (n_clamped) atomicAdd(&st.counters[0], (unsigned long long)n_clamped);
    if (n_nonfinite) atomicAdd(&st.counters[1], (unsigned long long)n_nonfinite);
    if (n_mismatch) atomicAdd(&st.counters[2], (unsigned long long)n_mismatch);
    if (n_pred) atomicAdd(&st.counters[3], (unsigned long long)n_pred);
  }
  if constexpr (CAL) {
    __syncthreads();
    for (int i = tid; i < n_cal<Net>(); i += NT)
      if (cal[i]) atomicMax(p.cal_out + i, cal[i]);
  }
  for (int i = tid; i < MT * C && STAGE != 1; i += NT) {
    const int s = i / C, e = i % C, k = sm.kid[s];
    if (k >= 0) {
      const size_t g = (size_t)k * C + e;
      st.q_idx[g] = sm.q_idx[s][e];
      st.q_e[g] = sm.q_e[s][e];
      st.q_t[g] = sm.q_t[s][e];
      st.q_r[g] = sm.q_r[s][e];
      if constexpr (Net::MWQ) {
        st.m_idx[g] = sm.m_idx[s][e];
        st.m_es[g] = sm.m_es[s][e];
        st.m_t[g] = sm.m_t[s][e];
        st.m_r[g] = sm.m_r[s][e];
        st.m_x[g] = sm.m_x[s][e];
      }
    }
  }
}

// ------------------------------------------ one wavefront per sub-trace ---
// The small network (16-slot windows of 32 features, conv 32 -> 32 -> 64,
// FC 256 -> 2) when a run has few sub-traces, so that the time of one step,
// not the throughput of many, bounds it: one wavefront (a workgroup of 64
// threads, one sub-trace slot) per sub-trace, no barrier between waves.
// The weights a lane needs stay in its registers for the whole launch; the
// window and the conv1 output pass through 3 KB of LDS; the products are
// VALU FMAs (a prediction is 33 k multiply-adds, ~520 cycles of one SIMD);
// the final FC is a lane reduction, so every lane holds the logits, and the
// clock and queue update runs on wave-uniform values, the retired prefix of
// the queue counted by one ballot over its entries (their retire times are
// non-decreasing along the queue).  The barriers order LDS only, so the next
// instruction's row, requested at the top of a step, stays in flight
// across them.  FP32 form, row or packed-code traces.
// Same state, work queue and results as step_kernel.
constexpr int WV_D = NetSmall::D, WV_C = NetSmall::C, WV_L = NetSmall::L;
constexpr int WV_C1 = NetSmall::CH1, WV_C2 = NetSmall::CH2, WV_NB = NetSmall::NB;

// Element B[k][n] of a weight matrix packed by the FP32 form (k-groups of
// 16, n-tiles of 16, lane = 16 * ((k % 16) / 4) + n % 16, 4 k per lane).
__device__ __forceinline__ float packed_f32(const float* Bp, int N, int k, int n) {
  const int kg = k >> 4, w = k & 15;
  return Bp[((((size_t)kg * (N >> 4) + (n >> 4)) * 64 + ((w >> 2) << 4) + (n & 15)) << 2) +
            (w & 3)];
}

template <bool RUN_NET>
__global__ void __launch_bounds__(64) wave_step_kernel(DevWeights wt, uint32_t relu_mask,
                                                       DevState st, StepParams p) {
  __shared__ __attribute__((aligned(16))) float x[WV_L][WV_D];        // the window
  __shared__ __attribute__((aligned(16))) float a1[WV_L / 2][WV_C1];  // conv1 output
  __shared__ int32_t q_e[WV_C];               // the queue ring
  __shared__ int64_t q_t[WV_C], q_r[WV_C];
  __shared__ int64_t rw[WMAX];                // retire times of the last W instructions
  __shared__ int claimed;
  const int lane = threadIdx.x, slot = blockIdx.x;
  constexpr int D = WV_D, C = WV_C;
  const int W = p.W;

  // weights this lane uses, kept in registers: conv1 output channel lane % 32
  // (its positions: lane / 32, +2, +4, +6), conv2 output channel lane, the
  // final FC's weights of conv2 channel lane at the 4 positions
  float w1[2][D], w2[2][WV_C1], wf[WV_NB][2];
  float b1 = 0.f, b2 = 0.f, bl[2] = {0.f, 0.f};
  const int c1 = lane & (WV_C1 - 1), half = lane >> 5;
  if (RUN_NET) {
    const float* W1 = static_cast<const float*>(wt.conv_w[0]);
    const float* W2 = static_cast<const float*>(wt.conv_w[1]);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int c = 0; c < D; ++c) w1[t][c] = packed_f32(W1, WV_C1, t * D + c, c1);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int c = 0; c < WV_C1; ++c) w2[t][c] = packed_f32(W2, WV_C2, t * WV_C1 + c, lane);
#pragma unroll
    for (int j = 0; j < WV_NB; ++j)
#pragma unroll
      for (int o = 0; o < 2; ++o) wf[j][o] = wt.last_w[((size_t)j * 2 + o) * WV_C2 + lane];
    b1 = wt.conv_b[0][c1];
    b2 = wt.conv_b[1][lane];
    bl[0] = wt.last_b[0];
    bl[1] = wt.last_b[1];
  }

  // the slot's sub-trace (a finished or empty slot claims the next one)
  int k = st.slot_kid[slot];
  if (k < 0) {
    if (lane == 0) claimed = claim_subtrace(st, p.n_sub);
    __syncthreads();
    k = claimed;
  }
  int64_t cur = 0, t_w = 0, r_prev = 0, pos = 0, first = 0, n_pos = 0, pred_off = 0;
  int32_t head = 0, count = 0, warm = 0;
  auto load_state = [&]() {
    if (k < 0) return;
    cur = st.cur[k];
    t_w = st.t_w[k];
    r_prev = st.r_prev[k];
    pos = st.pos[k];
    first = st.first[k];
    n_pos = st.n_pos[k];
    pred_off = st.pred_off[k];
    head = st.head[k];
    count = st.count[k];
    warm = st.warm[k];
    if (lane < C) {
      const size_t g = (size_t)k * C + lane;
      q_e[lane] = st.q_e[g];
      q_t[lane] = st.q_t[g];
      q_r[lane] = st.q_r[g];
    }
    if (lane < W) rw[lane] = st.rw[(size_t)k * WMAX + lane];
    lds_barrier();
  };
  // the window's static rows stay in registers: lane (slot w, 8 features)
  // holds trace row i - w; a step shifts them one slot (4 lanes) and takes
  // the next instruction's row, requested a step ahead, into slot 0
  const int ws = lane >> 2, wc = (lane & 3) * 8;
  float rowv[8];
  auto row_of = [&](int64_t row, float (&v)[8]) {
    if (p.codes) {
      const uint32_t code = p.codes[row];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = code_feature(code, wc + e);
    } else {
      const float4* src = reinterpret_cast<const float4*>(p.feat + row * D + wc);
      const float4 lo = src[0], hi = src[1];
      v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w;
      v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
    }
  };
  auto load_rows = [&]() {  // rows i - w that belong to the sub-trace
#pragma unroll
    for (int e = 0; e < 8; ++e) rowv[e] = 0.f;
    if (RUN_NET && k >= 0 && pos < n_pos && ws <= pos) row_of(first + pos - ws, rowv);
  };
  load_state();
  load_rows();
  uint32_t n_clamped = 0, n_nonfinite = 0, n_mismatch = 0, n_pred = 0;

  for (int it = 0; it < p.n_steps && k >= 0 && pos < n_pos; ++it) {
    const int64_t i = first + pos, g = pred_off + pos;
    float z[2] = {0.f, 0.f};
    float nxt[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // row i + 1 (slot 0), next step
    if (RUN_NET && ws == 0 && pos + 1 < n_pos) row_of(i + 1, nxt);
    if (RUN_NET) {
      // window: lane = (slot w, 8 features): the current instruction with
      // zero dynamic columns, then the queue newest first (instructions
      // i-1, i-2, ...: the queue holds consecutive ones), zeros past it
      {
        const int w = ws, c0 = wc;
        float res = 0.f, ex = 0.f;
        bool valid = w == 0;
        if (w >= 1 && w <= count) {
          int e = head + count - w;
          e = e >= C ? e - C : e;
          res = (float)(cur - q_t[e]);
          ex = (float)q_e[e];
          valid = true;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int c = c0 + e;
          float v = valid ? rowv[e] : 0.f;
          if (c == p.col_res) v = res;
          if (c == p.col_exe) v = ex;
          if (c == p.col_sto) v = 0.f;
          x[w][c] = v;
        }
      }
      lds_barrier();
      // conv1 (kernel 2, stride 2): channel c1 at positions half, half+2, ...
#pragma unroll
      for (int j = 0; j < WV_L / 4; ++j) {
        const int q = half + 2 * j;
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int c = 0; c < D; c += 4) {
            const float4 xv = *reinterpret_cast<const float4*>(&x[2 * q + t][c]);
            acc[0] = fmaf(w1[t][c], xv.x, acc[0]);
            acc[1] = fmaf(w1[t][c + 1], xv.y, acc[1]);
            acc[2] = fmaf(w1[t][c + 2], xv.z, acc[2]);
            acc[3] = fmaf(w1[t][c + 3], xv.w, acc[3]);
          }
        float v = b1 + ((acc[0] + acc[1]) + (acc[2] + acc[3]));
        if (relu_mask & 1u) v = fmaxf(v, 0.f);
        a1[q][c1] = v;
      }
      lds_barrier();
      // conv2: channel lane at positions 0..3, then the final FC's share
      float part[2] = {0.f, 0.f};
#pragma unroll
      for (int q = 0; q < WV_NB; ++q) {
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int c = 0; c < WV_C1; c += 4) {
            const float4 av = *reinterpret_cast<const float4*>(&a1[2 * q + t][c]);
            acc[0] = fmaf(w2[t][c], av.x, acc[0]);
            acc[1] = fmaf(w2[t][c + 1], av.y, acc[1]);
            acc[2] = fmaf(w2[t][c + 2], av.z, acc[2]);
            acc[3] = fmaf(w2[t][c + 3], av.w, acc[3]);
          }
        float v = b2 + ((acc[0] + acc[1]) + (acc[2] + acc[3]));
        if (relu_mask & 2u) v = fmaxf(v, 0.f);
        part[0] = fmaf(wf[q][0], v, part[0]);
        part[1] = fmaf(wf[q][1], v, part[1]);
      }
      // the final FC: sum over the 64 channels (a fixed butterfly)
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        float v = part[o];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
        v += bl[o];
        if (relu_mask & 4u) v = fmaxf(v, 0.f);
        z[o] = v;
      }
    }
    // round, or take the injected latencies
    int32_t lat[2];
    if (RUN_NET) {
      if (p.logits_out && lane == 0)
        for (int o = 0; o < 2; ++o) p.logits_out[g * 2 + o] = z[o];
#pragma unroll
      for (int o = 0; o < 2; ++o) lat[o] = round_latency(z[o], p.lat_max, n_clamped, n_nonfinite);
    }
    ++n_pred;
    if (p.lat_mode != 0) {
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const int32_t inj = p.lat_table[g * 2 + o];
        if (RUN_NET && inj != lat[o]) ++n_mismatch;
        lat[o] = inj;
      }
    }
    // clock and queue (Sec. 3.2): T = cur + F; the queue's retired prefix
    // (r <= T) leaves; r = max(T + E + 1, r_prev, r_{i-W} + 1); push
    const int64_t Tn = cur + lat[0];
    {
      bool gone = false;
      if (lane < count) {
        int e = head + lane;
        e = e >= C ? e - C : e;
        gone = q_r[e] <= Tn;
      }
      const int n_gone = __popcll(__ballot(gone));
      head += n_gone;
      head = head >= C ? head - C : head;
      count -= n_gone;
    }
    int64_t r = Tn + lat[1] + 1;
    r = r > r_prev ? r : r_prev;
    const int wi = (int)(pos % W);
    if (pos >= W) {
      const int64_t rb = rw[wi] + 1;
      r = r > rb ? r : rb;
    }
    int sl = head + count;
    sl = sl >= C ? sl - C : sl;
    if (count == C) {
      head = head + 1 == C ? 0 : head + 1;  // only the newest C stay visible
    } else {
      ++count;
    }
    lds_barrier();  // every lane has read the ring and rw for this step
    if (lane == 0) {
      rw[wi] = r;
      q_e[sl] = lat[1];
      q_t[sl] = Tn;
      q_r[sl] = r;
    }
    r_prev = r;
    cur = Tn;
    ++pos;
    if (pos == warm) t_w = Tn;
    if (pos == n_pos) {  // the drain ends (Eq. 1); the slot takes the next sub-trace
      if (lane == 0) {
        st.fetch[k] = Tn - t_w;
        st.drain[k] = r - Tn;
        st.final_tick[k] = r;
        st.warm_tick[k] = t_w;
        st.pos[k] = pos;
        st.cur[k] = Tn;
        claimed = claim_subtrace(st, p.n_sub);
      }
      lds_barrier();
      k = claimed;
      load_state();
      load_rows();
    } else {
      if (RUN_NET) {
        // slot w takes slot w-1's row; slot 0 the prefetched one
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float up = __shfl(rowv[e], lane >= 4 ? lane - 4 : lane);
          rowv[e] = ws == 0 ? nxt[e] : up;
        }
      }
      lds_barrier();
    }
  }

  // the slot's state back to memory
  if (lane == 0) {
    st.slot_kid[slot] = k;
    if (k >= 0) {
      st.cur[k] = cur;
      st.t_w[k] = t_w;
      st.r_prev[k] = r_prev;
      st.pos[k] = pos;
      st.head[k] = head;
      st.count[k] = count;
    }
    if (n_clamped) atomicAdd(&st.counters[0], (unsigned long long)n_clamped);
    if (n_nonfinite) atomicAdd(&st.counters[1], (unsigned long long)n_nonfinite);
    if (n_mismatch) atomicAdd(&st.counters[2], (unsigned long long)n_mismatch);
    if (n_pred) atomicAdd(&st.counters[3], (unsigned long long)n_pred);
  }
  if (k >= 0) {
    if (lane < C) {
      const size_t gq = (size_t)k * C + lane;
      st.q_idx[gq] = 0;
      st.q_e[gq] = q_e[lane];
      st.q_t[gq] = q_t[lane];
      st.q_r[gq] = q_r[lane];
    }
    if (lane < W) st.rw[(size_t)k * WMAX + lane] = rw[lane];
  }
}

// ------------------------------------------ queue in a row of 16 lanes ---
// The small network's processor queue (15 visible entries) held by 16
// consecutive lanes: lane j has the j-th newest instruction, a push moves
// every entry one lane up (DPP, no LDS), and the entries that have left stay
// behind the visible ones, so lane W - 1 always holds the retire time of the
// instruction W before.  The sub-trace's scalars are the same in all 16
// lanes.
constexpr int QL = 16;
static_assert(WV_C < QL && WMAX <= QL, "queue and retire history fit a row");

template <int CTRL>
__device__ __forceinline__ int32_t dpp(int32_t fill, int32_t x) {
  return __builtin_amdgcn_update_dpp(fill, x, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(dpp<CTRL>(0, __float_as_int(x)));
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E;  // quad permutations
constexpr int DPP_HALF_MIRROR = 0x141;           // lane i of 8 reads 7 - i
constexpr int DPP_ROR4 = 0x124, DPP_ROR8 = 0x128, DPP_SHR1 = 0x111;  // within 16

struct RowQueue {
  int32_t e;
  int64_t t, r;
  int64_t cur, t_w, r_prev, pos, n_pos, row, g;  // row: trace row of pos; g: prediction index
  int32_t count, warm;
  // sub-trace k's state (uniform over the 16 lanes); j: the lane's entry
  __device__ __forceinline__ void load(const DevState& st, int k, int j, int W) {
    cur = st.cur[k];
    t_w = st.t_w[k];
    r_prev = st.r_prev[k];
    pos = st.pos[k];
    n_pos = st.n_pos[k];
    row = st.first[k] + pos;
    g = st.pred_off[k] + pos;
    count = st.count[k];
    warm = st.warm[k];
    e = 0;
    t = r = 0;
    if (j < count) {
      int q = st.head[k] + count - 1 - j;
      q = q >= WV_C ? q - WV_C : q;
      const size_t at = (size_t)k * WV_C + q;
      e = st.q_e[at];
      t = st.q_t[at];
      r = st.q_r[at];
    } else if (j < W && j < pos) {
      r = st.rw[(size_t)k * WMAX + (pos - 1 - j) % W];
    }
  }
  // back to memory, the ring from entry 0 (head 0)
  __device__ __forceinline__ void store(const DevState& st, int k, int j, int W) const {
    if (j == 0) {
      st.cur[k] = cur;
      st.t_w[k] = t_w;
      st.r_prev[k] = r_prev;
      st.pos[k] = pos;
      st.head[k] = 0;
      st.count[k] = count;
    }
    if (j < count) {
      const size_t at = (size_t)k * WV_C + (count - 1 - j);
      st.q_idx[at] = (int32_t)(row - 1 - j);
      st.q_e[at] = e;
      st.q_t[at] = t;
      st.q_r[at] = r;
    }
    if (j < W && j < pos) st.rw[(size_t)k * WMAX + (pos - 1 - j) % W] = r;
  }
  // r_{i-W} + 1, or the least value before there are W instructions
  __device__ __forceinline__ int64_t retire_bound(int lane, int W) const {
    const int64_t rb = __shfl(r, (lane & ~(QL - 1)) + W - 1);
    return pos >= W ? rb + 1 : INT64_MIN;
  }
  // clock and queue (Sec. 3.2): T = cur + F; the retired prefix (r <= T)
  // leaves; r = max(T + E + 1, r_prev, r_{i-W} + 1); push.  Returns the
  // number of entries that were visible and stay so.
  __device__ __forceinline__ int advance(int32_t F, int32_t E, int64_t rb, int lane, int j) {
    const int64_t Tn = cur + F;
    const uint64_t gone = __ballot(j < count && r <= Tn);
    const int kept = count - __popc((uint32_t)(gone >> (lane & ~(QL - 1))) & 0xffffu);
    int64_t rn = Tn + E + 1;
    rn = rn > r_prev ? rn : r_prev;
    rn = rn > rb ? rn : rb;
    auto shift = [](int64_t fill, int64_t x) {
      const uint32_t lo = (uint32_t)dpp<DPP_SHR1>((int32_t)fill, (int32_t)x);
      const uint32_t hi = (uint32_t)dpp<DPP_SHR1>((int32_t)(fill >> 32), (int32_t)(x >> 32));
      return (int64_t)(((uint64_t)hi << 32) | lo);
    };
    e = dpp<DPP_SHR1>(E, e);
    t = shift(Tn, t);
    r = shift(rn, r);
    count = kept < WV_C ? kept + 1 : WV_C;  // only the newest C stay visible
    r_prev = rn;
    cur = Tn;
    ++pos;
    ++row;
    ++g;
    if (pos == warm) t_w = Tn;
    return kept;
  }
  // the drain ends (Eq. 1)
  __device__ __forceinline__ void finish(const DevState& st, int k) const {
    st.fetch[k] = cur - t_w;
    st.drain[k] = r_prev - cur;
    st.final_tick[k] = r_prev;
    st.warm_tick[k] = t_w;
    st.pos[k] = pos;
    st.cur[k] = cur;
  }
};

// Run counters of the lanes that own a sub-trace, added to the state's.
struct StepCounts {
  uint32_t clamped = 0, nonfinite = 0, mismatch = 0, pred = 0;
  __device__ __forceinline__ void add_to(const DevState& st) const {
    if (clamped) atomicAdd(&st.counters[0], (unsigned long long)clamped);
    if (nonfinite) atomicAdd(&st.counters[1], (unsigned long long)nonfinite);
    if (mismatch) atomicAdd(&st.counters[2], (unsigned long long)mismatch);
    if (pred) atomicAdd(&st.counters[3], (unsigned long long)pred);
  }
};

// LDS written by this wave and read by other lanes of it: the wave's LDS
// requests complete in order, so a compiler fence and a wait suffice
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// ------------------------------------------ four wavefronts per sub-trace ---
// The small network's FP32 step split over the four blocks of its kernel-2
// stride-2 tree: conv2's position j depends on window slots 4j .. 4j+3 only,
// so wave j builds those four slots, runs conv1 at positions 2j and 2j+1 and
// conv2 at position j (each wave reading only what it wrote), and multiplies
// its share of the final FC; the four partial sums meet in LDS, and every
// wave runs the same clock and queue update on the same values (wave 0
// alone writes the results and the state), each row of 16 lanes holding the
// whole queue.  Per lane that is 64 + 64 multiply-adds per prediction instead
// of the single wave's 768.  What bounds it is the chain of one step; the
// queue in registers leaves it one barrier, after the partial sums (written
// to alternating buffers), and the sums over a wave are DPP and lane swaps: 1.39
// us per step of one sub-trace (1.87 with the ring in LDS, a second barrier,
// LDS shuffles and a 64-bit remainder per step).  Three workgroups per CU
// instead of two spill 39 registers.  Same state, work queue and results as
// step_kernel.
constexpr int QW = 4;
static_assert(WV_NB == QW && WV_L == 16, "four blocks of four slots");

// s summed over the wave's 64 lanes, pairs 32, 16, 8, 4, 2, 1 apart in turn
__device__ __forceinline__ float wave_sum(float s) {
  auto halves = [](auto v) { return __uint_as_float(v[0]) + __uint_as_float(v[1]); };
  const uint32_t u = __float_as_uint(s);
  s = halves(__builtin_amdgcn_permlane32_swap(u, u, false, false));
  const uint32_t w = __float_as_uint(s);
  s = halves(__builtin_amdgcn_permlane16_swap(w, w, false, false));
  s += dpp<DPP_ROR8>(s);
  s += dpp<DPP_ROR4>(s);  // (lanes 8 apart hold the same by now)
  s += dpp<DPP_XOR2>(s);
  s += dpp<DPP_XOR1>(s);
  return s;
}

template <bool RUN_NET>
__global__ void __launch_bounds__(QW * 64) quad_step_kernel(DevWeights wt, uint32_t relu_mask,
                                                           DevState st, StepParams p) {
  constexpr int D = WV_D;
  __shared__ __attribute__((aligned(16))) float x[QW][4][D];   // each wave's four slots
  __shared__ __attribute__((aligned(16))) float a1[QW][2][WV_C1];  // its conv1 output
  __shared__ __attribute__((aligned(16))) float red[2][2][QW];   // partial sums of the final FC
  __shared__ int claimed;
  const int tid = threadIdx.x, v = tid >> 6, lane = tid & 63, slot = blockIdx.x;
  const int j = lane & (QL - 1), W = p.W;

  // this lane's weights: conv1 channel lane % 32 (position 2v + lane / 32),
  // conv2 channel lane (position v), the final FC's weights of that channel
  // at position v
  const int c1 = lane & (WV_C1 - 1), pl = lane >> 5;
  float w1[2][D], w2[2][WV_C1], wf[2];
  float b1 = 0.f, b2 = 0.f, bl[2] = {0.f, 0.f};
  if (RUN_NET) {
    const float* W1 = static_cast<const float*>(wt.conv_w[0]);
    const float* W2 = static_cast<const float*>(wt.conv_w[1]);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int c = 0; c < D; ++c) w1[t][c] = packed_f32(W1, WV_C1, t * D + c, c1);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int c = 0; c < WV_C1; ++c) w2[t][c] = packed_f32(W2, WV_C2, t * WV_C1 + c, lane);
#pragma unroll
    for (int o = 0; o < 2; ++o) wf[o] = wt.last_w[((size_t)v * 2 + o) * WV_C2 + lane];
    b1 = wt.conv_b[0][c1];
    b2 = wt.conv_b[1][lane];
    bl[0] = wt.last_b[0];
    bl[1] = wt.last_b[1];
  }

  int k = st.slot_kid[slot];
  if (k < 0) {
    if (tid == 0) claimed = claim_subtrace(st, p.n_sub);
    __syncthreads();
    k = claimed;
  }
  RowQueue q{};
  if (k >= 0) q.load(st, k, j, W);
  // this lane's window element pair: slot w = 4v + lane / 16, features
  // f0, f0 + 1; its trace row is that of the current instruction less w
  const int ls = lane >> 4, w = 4 * v + ls, f0 = j * 2;
  auto row_of = [&](int64_t row, float (&r)[2]) {
    if (p.codes) {
      const uint32_t code = p.codes[row];
      r[0] = code_feature(code, f0);
      r[1] = code_feature(code, f0 + 1);
    } else {
      const float2 t = *reinterpret_cast<const float2*>(p.feat + row * D + f0);
      r[0] = t.x;
      r[1] = t.y;
    }
  };
  float rowv[2] = {0.f, 0.f};
  auto load_row = [&]() {
    rowv[0] = rowv[1] = 0.f;
    if (RUN_NET && k >= 0 && q.pos < q.n_pos && w <= q.pos) row_of(q.row - w, rowv);
  };
  load_row();
  StepCounts n;

  for (int it = 0; it < p.n_steps && k >= 0 && q.pos < q.n_pos; ++it) {
    float nxt[2] = {0.f, 0.f};  // the next step's row for this lane
    if (RUN_NET && q.pos + 1 < q.n_pos && w <= q.pos + 1) row_of(q.row + 1 - w, nxt);
    const int64_t rb = q.retire_bound(lane, W);
    int32_t inj[2] = {0, 0};
    if (p.lat_mode != 0)
      for (int o = 0; o < 2; ++o) inj[o] = p.lat_table[q.g * 2 + o];
    float z[2] = {0.f, 0.f};
    if (RUN_NET) {
      // window: slot 0 the current instruction with zero dynamic columns,
      // slot w >= 1 the w-th newest queued one (lane w - 1's)
      {
        const int src = (lane & ~(QL - 1)) + (w >= 1 ? w - 1 : 0);
        float res = __shfl((float)(q.cur - q.t), src);
        float ex = __shfl((float)q.e, src);
        const bool queued = w >= 1 && w <= q.count, valid = w == 0 || queued;
        res = queued ? res : 0.f;
        ex = queued ? ex : 0.f;
        float2 val;
        val.x = valid ? rowv[0] : 0.f;
        val.y = valid ? rowv[1] : 0.f;
        auto put = [&](int c, float u) {
          val.x = f0 == c ? u : val.x;
          val.y = f0 + 1 == c ? u : val.y;
        };
        put(p.col_res, res);
        put(p.col_exe, ex);
        put(p.col_sto, 0.f);
        *reinterpret_cast<float2*>(&x[v][ls][f0]) = val;
      }
      wave_lds_sync();
      // conv1: channel c1 at position 2v + pl (slots 2 pl, 2 pl + 1 of the wave)
      {
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int c = 0; c < D; c += 4) {
            const float4 xv = *reinterpret_cast<const float4*>(&x[v][2 * pl + t][c]);
            acc[0] = fmaf(w1[t][c], xv.x, acc[0]);
            acc[1] = fmaf(w1[t][c + 1], xv.y, acc[1]);
            acc[2] = fmaf(w1[t][c + 2], xv.z, acc[2]);
            acc[3] = fmaf(w1[t][c + 3], xv.w, acc[3]);
          }
        float val = b1 + ((acc[0] + acc[1]) + (acc[2] + acc[3]));
        if (relu_mask & 1u) val = fmaxf(val, 0.f);
        a1[v][pl][c1] = val;
      }
      wave_lds_sync();
      // conv2: channel lane at position v, then its share of the final FC
      float part[2];
      {
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int c = 0; c < WV_C1; c += 4) {
            const float4 av = *reinterpret_cast<const float4*>(&a1[v][t][c]);
            acc[0] = fmaf(w2[t][c], av.x, acc[0]);
            acc[1] = fmaf(w2[t][c + 1], av.y, acc[1]);
            acc[2] = fmaf(w2[t][c + 2], av.z, acc[2]);
            acc[3] = fmaf(w2[t][c + 3], av.w, acc[3]);
          }
        float val = b2 + ((acc[0] + acc[1]) + (acc[2] + acc[3]));
        if (relu_mask & 2u) val = fmaxf(val, 0.f);
        part[0] = wf[0] * val;
        part[1] = wf[1] * val;
      }
      // (a wave writes this buffer again two barriers on, every wave having
      // read it before the first of them)
      float(&rd)[2][QW] = red[it & 1];
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const float s = wave_sum(part[o]);
        if (lane == 0) rd[o][v] = s;
      }
      lds_barrier();
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const float4 f = *reinterpret_cast<const float4*>(rd[o]);
        float s = ((f.x + f.y) + f.z) + f.w;
        s += bl[o];
        if (relu_mask & 4u) s = fmaxf(s, 0.f);
        z[o] = s;
      }
    }
    // round, or take the injected latencies (every wave alike)
    int32_t lat[2];
    if (RUN_NET) {
      if (p.logits_out && tid == 0)
        for (int o = 0; o < 2; ++o) p.logits_out[q.g * 2 + o] = z[o];
#pragma unroll
      for (int o = 0; o < 2; ++o) lat[o] = round_latency(z[o], p.lat_max, n.clamped, n.nonfinite);
    }
    ++n.pred;
    if (p.lat_mode != 0) {
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        if (RUN_NET && inj[o] != lat[o]) ++n.mismatch;
        lat[o] = inj[o];
      }
    }
    q.advance(lat[0], lat[1], rb, lane, j);
    if (q.pos == q.n_pos) {  // the slot takes the next sub-trace
      __syncthreads();  // every wave has read `claimed` of the sub-trace before
      if (tid == 0) {
        q.finish(st, k);
        claimed = claim_subtrace(st, p.n_sub);
      }
      __syncthreads();
      k = claimed;
      if (k >= 0) q.load(st, k, j, W);
      load_row();
    } else {
      rowv[0] = nxt[0];
      rowv[1] = nxt[1];
    }
  }

  // the slot's state back to memory
  if (tid == 0) {
    st.slot_kid[slot] = k;
    n.add_to(st);
  }
  if (k >= 0 && tid < QL) q.store(st, k, j, W);
}

// --------------------------------------- the small network's 16-slot tile ---
// Step of 16 sub-trace slots per workgroup (runs of more sub-traces than
// quad_step_kernel is for, and every BF16 and FP8 run): what bounds a step is
// the chain through it, not its 1.1 MFLOP per tile (MFMA FP32: 1.7 us, BF16
// 0.1).  So all weights stay in registers for the launch; the windows stay in
// LDS, a ring of 16 rows per slot turning one row per step (row of window
// slot w at step it: (it - w) % 16), of which a step writes the current
// instruction's row (requested a step before) and the dynamic columns; the
// queues are rows of 16 lanes (RowQueue; wave v holds slots 4v .. 4v + 3);
// wave v runs conv1 at positions 2v and 2v + 1 and conv2 at position v, so
// only the windows and conv2's outputs cross waves: two barriers.
// Against step_kernel<NetSmall, P>, which gathered the windows, streamed the
// weights and updated the queues one thread per slot anew each step (us per
// step over 120 steps, launch and results included; FP32, BF16, FP8): 3,000
// sub-traces 5.8 -> 3.7, 3.9 -> 2.2, 4.6 -> 2.4; 16,384: 18.8 -> 11.2, 8.8 ->
// 5.0, 13.0 -> 5.7.  Same products and sums in the same order as
// predict_tile<NetSmall, P>, same state, work queue and results.
// Sub-traces are claimed, and the run's counters added, once per workgroup:
// atomics on one address take ~17 ns each on the whole chip, and with one per
// wave (four times step_kernel's) runs of many short sub-traces were slower than
// that kernel (us, 20,000 and 100,000 sub-traces of 8 instructions, injected
// latencies: step_kernel 110, 320, one per wave 166, 501, one per workgroup 88,
// 254; BF16 predicting 164, 526, 209, 551, 121, 418).
template <class P>
struct SmallTile {
  using T = typename P::T;
  static constexpr int D = WV_D, PAD = 16 / (int)sizeof(T);
  static constexpr int KGS = 2 * D / P::KG;     // k-groups of either conv
  static constexpr int SX = WV_L * D + PAD;     // window ring, per slot
  static constexpr int SA = 2 * WV_C1 + PAD;    // a wave's conv1 output, per slot
  static constexpr int SO = QW * WV_C2 + PAD;   // conv2 output, per slot
  static_assert(WV_C1 == D && padded_feat(D, P::ID) == D && MT == 4 * QW, "small network shape");
  alignas(16) T x[MT * SX];
  alignas(16) T a1[QW][MT * SA];
  alignas(16) T out[MT * SO];
};

// The waves' agreement on which slots take a sub-trace, and when.
struct SmallClaims {
  alignas(16) uint32_t left[QW];   // per wave: steps to its first sub-trace's end
  alignas(16) uint32_t ended[QW];  // per wave: slots that take a sub-trace
  uint32_t claimed;                // the first of the claim order they take
  uint32_t counts[NCOUNTERS];      // the workgroup's run counters, at the end
};

template <class P, bool RUN_NET>
__global__ void __launch_bounds__(QW * 64, 2)
    small_step_kernel(DevWeights wt, uint32_t relu_mask, DevState st, StepParams p) {
  using S = SmallTile<P>;
  using T = typename P::T;
  constexpr int D = WV_D, KGS = S::KGS, KQ = P::KG / 4;
  constexpr int N1 = WV_C1 / 16, N2 = WV_C2 / 16, NS1 = P::SCALED ? N1 : 1,
                NS2 = P::SCALED ? N2 : 1;
  constexpr int CPL = WV_C2 / 8;  // final-FC channels per lane and block
  __shared__ S sm;  // (not there without the predictor)
  __shared__ SmallClaims cl;
  const int tid = threadIdx.x, v = tid >> 6, lane = tid & 63;
  const int s = tid >> 4, j = tid & (QL - 1), W = p.W;  // slot, queue entry
  const int mr = lane & 15, g4 = lane >> 4;             // MFMA row (slot), k quarter
  const int fo = j >> 3, fsub = j & 7, f0 = 2 * j;
  const int slot = blockIdx.x * MT + s;

  uint4 w1[KGS][N1], w2[KGS][N2];
  v4f b1[N1], b2[N2], s1[NS1] = {}, i1[NS1] = {}, s2[NS2] = {}, i2[NS2] = {};
  float wl[QW][CPL], lb = 0.f;
  float xi[2] = {1.f, 1.f}, xr = 1.f, xe = 1.f;  // FP8: input scales of this lane's columns
  if constexpr (RUN_NET) {
    const uint4* W1 = static_cast<const uint4*>(wt.conv_w[0]);
    const uint4* W2 = static_cast<const uint4*>(wt.conv_w[1]);
#pragma unroll
    for (int kg = 0; kg < KGS; ++kg) {
#pragma unroll
      for (int n = 0; n < N1; ++n) w1[kg][n] = W1[(kg * N1 + n) * 64 + lane];
#pragma unroll
      for (int n = 0; n < N2; ++n) w2[kg][n] = W2[(kg * N2 + n) * 64 + lane];
    }
#pragma unroll
    for (int n = 0; n < N1; ++n) {
      const int c = n * 16 + 4 * g4;
      b1[n] = *reinterpret_cast<const v4f*>(wt.conv_b[0] + c);
      if constexpr (P::SCALED) {
        s1[n] = *reinterpret_cast<const v4f*>(wt.conv_ws[0] + c);
        i1[n] = *reinterpret_cast<const v4f*>(wt.conv_ai[0] + c);
      }
    }
#pragma unroll
    for (int n = 0; n < N2; ++n) {
      const int c = n * 16 + 4 * g4;
      b2[n] = *reinterpret_cast<const v4f*>(wt.conv_b[1] + c);
      if constexpr (P::SCALED) {
        s2[n] = *reinterpret_cast<const v4f*>(wt.conv_ws[1] + c);
        i2[n] = *reinterpret_cast<const v4f*>(wt.conv_ai[1] + c);
      }
    }
#pragma unroll
    for (int b = 0; b < QW; ++b)
#pragma unroll
      for (int c = 0; c < CPL; ++c)
        wl[b][c] = wt.last_w[((size_t)b * 2 + fo) * WV_C2 + fsub * CPL + c];
    lb = wt.last_b[fo];
    if constexpr (P::SCALED) {
      auto scale = [&](int c) { return c >= 0 && c < D ? wt.x_inv[c] : 1.f; };
      xi[0] = scale(f0);
      xi[1] = scale(f0 + 1);
      xr = scale(p.col_res);
      xe = scale(p.col_exe);
    }
  }

  T* const xs = sm.x + s * S::SX;
  // trace row tr to `row` in storage precision, dynamic columns zero (the few
  // of them overwritten: a test per feature costs the kernel its scalar registers)
  auto put_row = [&](int64_t tr, T* row) {
    if (P::ID == 1 && !p.codes) {
      const uint4* src = reinterpret_cast<const uint4*>(p.feat16 + tr * staged_feat(D));
#pragma unroll
      for (int q = 0; q < D / 8; ++q) reinterpret_cast<uint4*>(row)[q] = src[q];
    } else {
      const uint32_t code = p.codes ? p.codes[tr] : 0u;
#pragma unroll
      for (int c = 0; c < D; c += 2) {
        float2 f;
        if (p.codes)
          f = make_float2(code_feature(code, c), code_feature(code, c + 1));
        else
          f = *reinterpret_cast<const float2*>(p.feat + tr * D + c);
        if constexpr (P::SCALED) f = make_float2(f.x * wt.x_inv[c], f.y * wt.x_inv[c + 1]);
        const T e[2] = {P::cvt(f.x), P::cvt(f.y)};
        store_run<2 * sizeof(T)>(row + c, e);
      }
    }
    for (int c : {p.col_res, p.col_exe, p.col_sto})
      if ((unsigned)c < (unsigned)D) row[c] = P::cvt(0.f);
  };
  // the current instruction's row: this lane's two features as they are in
  // the trace (or its code), requested a step ahead
  uint32_t raw[2] = {0u, 0u};
  auto request = [&](int64_t row) {
    if (p.codes) {
      raw[0] = p.codes[row];
    } else if constexpr (P::ID == 1) {
      raw[0] = *reinterpret_cast<const uint32_t*>(p.feat16 + row * staged_feat(D) + f0);
    } else {
      const uint2 r = *reinterpret_cast<const uint2*>(p.feat + row * D + f0);
      raw[0] = r.x;
      raw[1] = r.y;
    }
  };
  auto commit = [&](T* dst) {
    T e[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = f0 + i;
      float f = 0.f;
      if (p.codes) {
        f = code_feature(raw[0], c);
      } else if constexpr (P::ID == 1) {
        f = __uint_as_float(i ? raw[0] & 0xffff0000u : raw[0] << 16);
      } else {
        f = __uint_as_float(raw[i]);
      }
      const bool dyn = c == p.col_res || c == p.col_exe || c == p.col_sto;
      if constexpr (P::SCALED) f *= xi[i];
      e[i] = P::cvt(dyn ? 0.f : f);
      if constexpr (P::ID == 1)  // the BF16 rows' own bits
        if (!p.codes) e[i] = dyn ? (T)0 : (T)(i ? raw[0] >> 16 : raw[0]);
    }
    store_run<2 * sizeof(T)>(dst + f0, e);
  };
  auto zero_row = [&](T* row) {
#pragma unroll
    for (int q = 0; q < D * (int)sizeof(T) / 16; ++q)
      reinterpret_cast<uint4*>(row)[q] = make_uint4(0u, 0u, 0u, 0u);
  };

  RowQueue q{};
  bool active = false;
  int k = st.slot_kid[slot];
  // the slots with `take` set claim the next sub-traces, all at once
  auto claim = [&](bool take) {
    const uint64_t mine = __ballot(take && j == 0);
    if (lane == 0) cl.ended[v] = (uint32_t)__popcll(mine);
    lds_barrier();
    const uint4 c = *reinterpret_cast<const uint4*>(cl.ended);
    const uint32_t all = c.x + c.y + c.z + c.w;
    if (tid == 0 && all > 0) cl.claimed = atomicAdd(st.next, all);
    lds_barrier();
    if (!take) return;
    const uint32_t at = cl.claimed + (v > 0 ? c.x : 0) + (v > 1 ? c.y : 0) + (v > 2 ? c.z : 0) +
                        (uint32_t)__popcll(mine & ((1ull << (lane & ~(QL - 1))) - 1));
    k = at < (uint32_t)p.n_sub ? st.order[at] : -1;
  };
  claim(k < 0);
  // the slot's state, and its windows' rows but the current one's as step
  // `it` finds them (lane j: window slot j + 1)
  auto load = [&](int it) {
    active = false;
    if (k >= 0) {
      q.load(st, k, j, W);
      active = q.pos < q.n_pos;
    }
    if constexpr (RUN_NET) {
      T* row = xs + ((it - 1 - j) & (WV_L - 1)) * D;
      zero_row(row);
      if (active) {
        if (j < q.count) put_row(q.row - 1 - j, row);
        request(q.row);
      }
    }
  };
  load(0);
  StepCounts n;

  // up to the first end of a sub-trace in the workgroup, whose slots then take
  // the next ones together
  for (int it = 0; it < p.n_steps;) {
    uint32_t first = active ? (uint32_t)(q.n_pos - q.pos) : UINT32_MAX;  // (below 2^31)
    first = min(first, (uint32_t)__shfl_xor((int)first, 16));
    first = min(first, (uint32_t)__shfl_xor((int)first, 32));
    if (lane == 0) cl.left[v] = first;
    lds_barrier();
    const uint4 left = *reinterpret_cast<const uint4*>(cl.left);
    first = min(min(left.x, left.y), min(left.z, left.w));
    if (first == UINT32_MAX) break;  // (no slot has a sub-trace)
    const int end = it + (int)min(first, (uint32_t)(p.n_steps - it));
    for (; it < end; ++it) {
      const int64_t rb = q.retire_bound(lane, W);
      int32_t inj[2] = {0, 0};
      if (p.lat_mode != 0 && active)
        for (int o = 0; o < 2; ++o) inj[o] = p.lat_table[q.g * 2 + o];
      float z[2] = {0.f, 0.f};
      if constexpr (RUN_NET) {
        if (active) {
          commit(xs + (it & (WV_L - 1)) * D);
          if (j < q.count) {
            T* row = xs + ((it - 1 - j) & (WV_L - 1)) * D;
            auto put = [&](int c, float u, float inv) {
              if constexpr (P::SCALED) u *= inv;
              if ((unsigned)c < (unsigned)D) row[c] = P::cvt(u);
            };
            put(p.col_res, (float)(q.cur - q.t), xr);
            put(p.col_exe, (float)q.e, xe);
            put(p.col_sto, 0.f, 1.f);
          }
          if (q.pos + 1 < q.n_pos) request(q.row + 1);
        }
        lds_barrier();
        // conv1 at positions 2v, 2v + 1
        v4f acc[2][N1];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int n = 0; n < N1; ++n) acc[i][n] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kg = 0; kg < KGS; ++kg) {
          const int k0 = kg * P::KG + KQ * g4, tap = k0 / D, off = k0 % D;
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int row = (it - 2 * (2 * v + i) - tap) & (WV_L - 1);
            const uint4 a = *reinterpret_cast<const uint4*>(sm.x + mr * S::SX + row * D + off);
#pragma unroll
            for (int n = 0; n < N1; ++n) acc[i][n] = P::mma(acc[i][n], w1[kg][n], a);
          }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int n = 0; n < N1; ++n) {
            T e[4];
#pragma unroll
            for (int c = 0; c < 4; ++c)
              e[c] = to_storage_v<P>(activation_v<P>(acc[i][n][c], b1[n][c], s1[P::SCALED ? n : 0][c],
                                                     relu_mask & 1u),
                                     i1[P::SCALED ? n : 0][c]);
            store_run<4 * sizeof(T)>(&sm.a1[v][mr * S::SA + i * WV_C1 + n * 16 + 4 * g4], e);
          }
        wave_lds_sync();
        // conv2 at position v
        v4f acc2[N2];
#pragma unroll
        for (int n = 0; n < N2; ++n) acc2[n] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kg = 0; kg < KGS; ++kg) {
          const uint4 a = *reinterpret_cast<const uint4*>(
              &sm.a1[v][mr * S::SA + kg * P::KG + KQ * g4]);
#pragma unroll
          for (int n = 0; n < N2; ++n) acc2[n] = P::mma(acc2[n], w2[kg][n], a);
        }
#pragma unroll
        for (int n = 0; n < N2; ++n) {
          T e[4];
#pragma unroll
          for (int c = 0; c < 4; ++c)
            e[c] = to_storage_v<P>(activation_v<P>(acc2[n][c], b2[n][c], s2[P::SCALED ? n : 0][c],
                                                   relu_mask & 2u),
                                   i2[P::SCALED ? n : 0][c]);
          store_run<4 * sizeof(T)>(&sm.out[mr * S::SO + v * WV_C2 + n * 16 + 4 * g4], e);
        }
        lds_barrier();
        // final FC: 8 lanes per (slot, output)
        float f = 0.f;
#pragma unroll
        for (int b = 0; b < QW; ++b) {
          alignas(16) T a[CPL];
          __builtin_memcpy(a, __builtin_assume_aligned(
                                  &sm.out[s * S::SO + b * WV_C2 + fsub * CPL], CPL * sizeof(T) < 16
                                                                                   ? CPL * sizeof(T)
                                                                                   : 16),
                           sizeof a);
#pragma unroll
          for (int c = 0; c < CPL; ++c) f = fmaf(P::val(a[c]), wl[b][c], f);
        }
        f += dpp<DPP_XOR1>(f);
        f += dpp<DPP_XOR2>(f);
        f += dpp<DPP_HALF_MIRROR>(f);  // (lanes of a quad hold the same by now)
        f += lb;
        if (relu_mask & 4u) f = fmaxf(f, 0.f);
        const float other = dpp<DPP_ROR8>(f);
        z[0] = fo ? other : f;
        z[1] = fo ? f : other;
        if (p.logits_out && active && fsub == 0) p.logits_out[q.g * 2 + fo] = f;
      }
      int32_t lat[2] = {0, 0};
      const int32_t count = q.count;
      StepCounts m;
      if (RUN_NET) {
#pragma unroll
        for (int o = 0; o < 2; ++o)
          lat[o] = round_latency(z[o], p.lat_max, m.clamped, m.nonfinite);
      }
      if (p.lat_mode != 0) {
#pragma unroll
        for (int o = 0; o < 2; ++o) {
          if (RUN_NET && inj[o] != lat[o]) ++m.mismatch;
          lat[o] = inj[o];
        }
      }
      if (active) {
        ++n.pred;
        n.clamped += m.clamped;
        n.nonfinite += m.nonfinite;
        n.mismatch += m.mismatch;
        const int kept = q.advance(lat[0], lat[1], rb, lane, j);
        if constexpr (RUN_NET)
          // rows that left the window: that of the entry one lane down now (a
          // full queue's oldest is the next current row)
          if (j >= kept && j < count) zero_row(xs + ((it - 1 - j) & (WV_L - 1)) * D);
      }
    }
    const bool ended = active && q.pos == q.n_pos;
    if (ended && j == 0) q.finish(st, k);
    claim(ended);
    if (ended) load(it);
  }

  // (one atomic per counter and workgroup: those on one address take ~17 ns each)
  static_assert(NCOUNTERS == 4, "StepCounts");
  if (tid < NCOUNTERS) cl.counts[tid] = 0u;
  lds_barrier();
  if (j == 0) {
    st.slot_kid[slot] = k;
    atomicAdd(&cl.counts[0], n.clamped);
    atomicAdd(&cl.counts[1], n.nonfinite);
    atomicAdd(&cl.counts[2], n.mismatch);
    atomicAdd(&cl.counts[3], n.pred);
  }
  if (k >= 0) q.store(st, k, j, W);
  lds_barrier();
  if (tid < NCOUNTERS && cl.counts[tid])
    atomicAdd(&st.counters[tid], (unsigned long long)cl.counts[tid]);
}

// Predictor over explicit windows x [B][L][D] -> logits [B][NOUT]; TRUNK:
// the convolutions only, the last conv's output to trunk_out [B][NB][CH3].
template <class Net, class P, bool TRUNK = false>
__global__ void __launch_bounds__(Net::WAVES * 64)
    forward_kernel(DevWeights wt, uint32_t relu_mask, const float* __restrict__ x, int64_t B,
                   float* __restrict__ logits, void* __restrict__ trunk_out) {
  using G = Geo<Net, P>;
  using T = typename P::T;
  constexpr int NT = G::NT, D = Net::D, BS = Net::BS;
  __shared__ NetSmem<Net, P> sm;
  const int tid = threadIdx.x;
  const int64_t b0 = (int64_t)blockIdx.x * MT;
  using GA = Gather<Net, P>;
  constexpr int GSL = GA::GSL, TPR = GA::TPR, CPT = GA::CPT;
  const int row = tid / TPR, part = tid % TPR;
  const int s = row / GSL, t = row % GSL;
  if constexpr (P::SCALED)
    for (int c = tid; c < D; c += NT) sm.x_inv[c] = wt.x_inv[c];
  sm.stage_head(wt, tid, NT);
  __syncthreads();
  const int64_t b = b0 + s;
  // (request_window_row's loads, written out: through the function the FP32
  // form with store latencies spills scalar registers, 3,000 windows 272 us
  // against 256)
  auto load = [&](int j0, int nb) {
    RowRegs<CPT> r;
    r.valid = b < B && t < nb * BS;
    const float* src = x + ((r.valid ? b : 0) * Net::L + (r.valid ? j0 * BS + t : 0)) * D;
#pragma unroll
    for (int cc = 0; cc < CPT; cc += 2) {
      const int c = part * CPT + cc;
      if (TPR > 1 || cc < D)
        r.v[cc / 2] = *reinterpret_cast<const float2*>(src + (c < D ? c : D - 2));
      else
        r.v[cc / 2] = make_float2(0.f, 0.f);
    }
    return r;
  };
  auto commit = [&](int j0, int nb, const RowRegs<CPT>& r, T* X) {
    (void)j0;
    if (t < nb * BS) commit_window_row<Net, P>(sm.x_inv, s, t, part, r, X);
  };
  if constexpr (TRUNK) {
    SavePtrs<T> sv{};
    sv.a3 = static_cast<T*>(trunk_out) + b0 * Net::NB * Net::CH3;
    sv.rows = (int)(B - b0 < MT ? B - b0 : MT);
    predict_tile<Net, P, false, true, true>(wt, relu_mask, sm, load, commit, nullptr, nullptr, sv);
  } else {
    predict_tile<Net, P>(wt, relu_mask, sm, load, commit);
    if (tid < MT * Net::NOUT) {
      const int ss = tid / Net::NOUT, o = tid % Net::NOUT;
      if (b0 + ss < B) logits[(b0 + ss) * Net::NOUT + o] = sm.logit[ss][o];
    }
  }
}

// ------------------------------------------------------ residual blocks ---
// A tile of TM rows (window positions at the last conv level, CH3 channels
// each) stays in LDS through all NRES blocks.  Per block the expansion is
// produced EC channels at a time (bias, ReLU, rounded to the form, into one
// of two LDS buffers) and consumed by the projection in the next phase,
// while the following chunk is expanded; the projection's TM x CH3
// accumulators stay in registers for the whole block; then bias, the block
// input and the ReLU, rounded to the form, replace the tile.
// Bound by each CU's weight stream and LDS reads beside the MFMAs: BF16, 128
// rows 360 us (0.69 of the 32x32x16 instruction's sustained rate), 64 rows
// 205, 32 rows 172 (the weights' 100 us at the port's rate and their latency).

// The matrix instruction of a form in the residual blocks: BF16 on
// 32x32x16 tiles, FP32 on 16x16x4.
template <class P>
struct ResMma {
  using M = P;
};
template <>
struct ResMma<PBF16> {
  using M = PBF16W;
};

// Rows per tile TM and the waves' split: WNW along N (4: two along M, each
// weight fragment then requested by two waves; 8: one along M, each fragment
// requested once).  Chunks of EC expansion channels; the last may be shorter
// (ET), its expansion on the waves it reaches.
template <class P, int ROWS, int WN>
struct ResGeo {
  using T = typename P::T;
  using M = typename ResMma<P>::M;
  static constexpr int C = NetRB7::CH3, E = NetRB7::EXPAND;
  static constexpr int TM = ROWS, TILE = M::TILE, MTL = TM / TILE;
  static constexpr int EC = TILE * WN > 128 ? TILE * WN : 128, ET = E % EC;
  static constexpr int NCH = (E + EC - 1) / EC;
  static constexpr int PAD = 16 / sizeof(T);
  static constexpr int SXR = C + PAD, SHR = EC + PAD;  // padded LDS rows
  static constexpr int WAVES = 8, NT = WAVES * 64, WNW = WN, WMW = WAVES / WNW;
  static constexpr int MPW = MTL / WMW, NPE = EC / TILE / WNW, NPP = C / TILE / WNW;
  static_assert(MPW >= 1 && MTL % WMW == 0 && NPE * WNW * TILE == EC && NPP * WNW * TILE == C &&
                    E % (NPE * TILE) == 0 && ET % M::KG == 0,
                "wave split");
};

template <class P, int ROWS, int WN>
__global__ void __launch_bounds__((ResGeo<P, ROWS, WN>::NT))
    resblock_kernel(DevWeights wt, uint32_t relu_mask, typename P::T* __restrict__ x, int64_t rows,
                    const int32_t* __restrict__ active) {
  using RG = ResGeo<P, ROWS, WN>;
  using M = typename RG::M;
  using T = typename P::T;
  using Acc = typename M::Acc;
  using Net = NetRB7;
  constexpr int C = RG::C, E = RG::E, EC = RG::EC, TM = RG::TM, TILE = RG::TILE;
  constexpr int MPW = RG::MPW, NPE = RG::NPE, NPP = RG::NPP;
  constexpr int NG4 = TILE * TILE / 256;  // 4-column groups per lane and tile
  constexpr int CV = C * (int)sizeof(T) / 16, EPV = 16 / (int)sizeof(T);
  constexpr int KGE = C / M::KG, KGP = EC / M::KG, NCH = RG::NCH, NTE = E / TILE, NTP = C / TILE;
  __shared__ alignas(16) T xs[TM * RG::SXR];
  __shared__ alignas(16) T hs[2 * TM * RG::SHR];  // two expansion chunks
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t r0 = (int64_t)blockIdx.x * TM;
  const int64_t r1 = r0 + TM < rows ? r0 + TM : rows;  // rows [r0, r1) exist
  if (active) {  // windows none of whose rows is live are skipped
    int a = 0;
    for (int64_t w = r0 / Net::NB + tid; w <= (r1 - 1) / Net::NB; w += RG::NT) a |= active[w];
    if (!__syncthreads_or(a)) return;
  }
  for (int i = tid; i < TM * CV; i += RG::NT) {
    const int r = i / CV, v = i % CV;
    uint4 val = make_uint4(0u, 0u, 0u, 0u);
    if (r0 + r < r1) val = reinterpret_cast<const uint4*>(x + (r0 + r) * C)[v];
    *reinterpret_cast<uint4*>(xs + r * RG::SXR + v * EPV) = val;
  }
  __syncthreads();
  // a wave's A fragments (LDS) serve its NPE or NPP N tiles, its weight
  // fragments its MPW M tiles
  const int wn = wave % RG::WNW, wm = wave / RG::WNW;
  const int row = lane % TILE, ko = (lane / TILE) * (M::KG * TILE / 64);
  const T* apx[MPW];
  const T* aph[MPW];
#pragma unroll
  for (int i = 0; i < MPW; ++i) {
    const int r = (wm * MPW + i) * TILE + row;
    apx[i] = xs + r * RG::SXR + ko;
    aph[i] = hs + r * RG::SHR + ko;
  }
  const size_t half = (size_t)C * E * sizeof(T);
  Acc yacc[MPW][NPP];
#pragma unroll
  for (int i = 0; i < MPW; ++i)
#pragma unroll
    for (int j = 0; j < NPP; ++j) yacc[i][j] = Acc{};
  // Expansion of chunk u into hs buffer u & 1: bias, ReLU, rounded to the form.
  auto expand = [&](int u) {
    const int blk = u / NCH, ch = u % NCH;
    if (RG::ET && ch * EC + wn * NPE * TILE >= E) return;  // (past a short last chunk)
    const uint4* We = reinterpret_cast<const uint4*>(static_cast<const char*>(wt.res_w) +
                                                     (size_t)blk * wt.res_stride);
    const float* be = wt.res_b + (size_t)blk * (E + C);
    const bool erelu = relu_mask & (1u << (Net::NCONV + 2 * blk));
    float4 bev[NPE][NG4];  // requested before the weights (loads complete in order)
#pragma unroll
    for (int j = 0; j < NPE; ++j)
#pragma unroll
      for (int g = 0; g < NG4; ++g)
        bev[j][g] = *reinterpret_cast<const float4*>(be + ch * EC + (wn * NPE + j) * TILE +
                                                     M::col4(g, lane));
    Acc hacc[MPW][NPE];
#pragma unroll
    for (int i = 0; i < MPW; ++i)
#pragma unroll
      for (int j = 0; j < NPE; ++j) hacc[i][j] = Acc{};
    mma_stream<M, KGE, NTE, NPE, MPW>(hacc, apx, We, ch * (EC / TILE) + wn * NPE, lane);
    T* hb = hs + (u & 1) * TM * RG::SHR;
#pragma unroll
    for (int j = 0; j < NPE; ++j)
#pragma unroll
      for (int g = 0; g < NG4; ++g) {
        const int hc0 = (wn * NPE + j) * TILE + M::col4(g, lane);  // 4 channels of the chunk
        const float bq[4] = {bev[j][g].x, bev[j][g].y, bev[j][g].z, bev[j][g].w};
#pragma unroll
        for (int i = 0; i < MPW; ++i) {
          T e[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float v = hacc[i][j][4 * g + q] + bq[q];
            if (erelu) v = fmaxf(v, 0.f);
            e[q] = to_storage<P>(v, 0, nullptr);
          }
          store_run<4 * sizeof(T)>(hb + ((wm * MPW + i) * TILE + row) * RG::SHR + hc0, e);
        }
      }
  };
  // Projection of chunk u from hs buffer u & 1 into yacc.
  auto project = [&](int u) {
    const int blk = u / NCH, ch = u % NCH;
    const uint4* Wp = reinterpret_cast<const uint4*>(static_cast<const char*>(wt.res_w) +
                                                     (size_t)blk * wt.res_stride + half) +
                      (size_t)ch * KGP * NTP * 64;
    const int ho = (u & 1) * TM * RG::SHR;
    const T* aphu[MPW];
#pragma unroll
    for (int i = 0; i < MPW; ++i) aphu[i] = aph[i] + ho;
    if constexpr (RG::ET > 0)
      if (ch == NCH - 1) {
        mma_stream<M, RG::ET / M::KG, NTP, NPP, MPW>(yacc, aphu, Wp, wn * NPP, lane);
        return;
      }
    mma_stream<M, KGP, NTP, NPP, MPW>(yacc, aphu, Wp, wn * NPP, lane);
  };
  // Chunk u+1's expansion and chunk u's projection share a phase (one
  // barrier per chunk; the two products' chains interleave); a block's first
  // expansion waits for the previous block's output.
  constexpr int TT = Net::NRES * NCH;
  expand(0);
  lds_barrier();
  for (int t = 0; t < TT; ++t) {
    const int blk = t / NCH, ch = t % NCH;
    float4 bpv[NPP][NG4];
    if (ch == NCH - 1) {
      const float* bp = wt.res_b + (size_t)blk * (E + C) + E;
#pragma unroll
      for (int j = 0; j < NPP; ++j)
#pragma unroll
        for (int g = 0; g < NG4; ++g)
          bpv[j][g] = *reinterpret_cast<const float4*>(bp + (wn * NPP + j) * TILE +
                                                       M::col4(g, lane));
    } else {
      expand(t + 1);
    }
    project(t);
    lds_barrier();
    if (ch == NCH - 1) {
      // bias, the block input (as stored) and the activation replace the tile
      const bool orelu = relu_mask & (1u << (Net::NCONV + 2 * blk + 1));
#pragma unroll
      for (int j = 0; j < NPP; ++j)
#pragma unroll
        for (int g = 0; g < NG4; ++g) {
          const int col0 = (wn * NPP + j) * TILE + M::col4(g, lane);
          const float bq[4] = {bpv[j][g].x, bpv[j][g].y, bpv[j][g].z, bpv[j][g].w};
#pragma unroll
          for (int i = 0; i < MPW; ++i) {
            T* xr = xs + ((wm * MPW + i) * TILE + row) * RG::SXR + col0;
            T e[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              float v = yacc[i][j][4 * g + q] + bq[q] + P::val(xr[q]);
              if (orelu) v = fmaxf(v, 0.f);
              e[q] = to_storage<P>(v, 0, nullptr);
            }
            store_run<4 * sizeof(T)>(xr, e);
          }
        }
#pragma unroll
      for (int i = 0; i < MPW; ++i)
#pragma unroll
        for (int j = 0; j < NPP; ++j) yacc[i][j] = Acc{};
      lds_barrier();
      if (t + 1 < TT) {
        expand(t + 1);
        lds_barrier();
      }
    }
  }
  for (int i = tid; i < TM * CV; i += RG::NT) {
    const int r = i / CV, v = i % CV;
    if (r0 + r < r1)
      reinterpret_cast<uint4*>(x + (r0 + r) * C)[v] =
          *reinterpret_cast<const uint4*>(xs + r * RG::SXR + v * EPV);
  }
}

// FC 512 and the hybrid head over x [B][NB][CH3] (the blocks' output):
// each group of the tile's blocks is staged into LDS where the fused step
// keeps its last conv output, then the same hidden-FC and head code runs.
template <class P>
__global__ void __launch_bounds__(NetRB7::WAVES * 64)
    rb_head_kernel(DevWeights wt, uint32_t relu_mask, const typename P::T* __restrict__ x,
                   int64_t B, const int32_t* __restrict__ active, float* __restrict__ logits) {
  using Net = NetRB7;
  using G = Geo<Net, P>;
  using T = typename P::T;
  constexpr int NG = G::NG, NFULL = Net::NB / NG, TAIL = Net::NB % NG;
  constexpr int HT = (Net::HID / 16) / Net::WAVES, V = Net::CH3 * (int)sizeof(T) / 16;
  __shared__ NetSmem<Net, P> sm;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t b0 = (int64_t)blockIdx.x * MT;
  if (active) {
    const int a = tid < MT && b0 + tid < B ? active[b0 + tid] : 0;
    if (!__syncthreads_or(a)) return;
  }
  v4f hacc[HT];
#pragma unroll
  for (int j = 0; j < HT; ++j) hacc[j] = v4f{0.f, 0.f, 0.f, 0.f};
  auto stage = [&](int j0, int nb) {
    for (int i = tid; i < MT * nb * V; i += G::NT) {
      const int s = i / (nb * V), r = i % (nb * V), jb = r / V, v = r % V;
      uint4 val = make_uint4(0u, 0u, 0u, 0u);
      if (b0 + s < B)
        val = reinterpret_cast<const uint4*>(x + ((b0 + s) * Net::NB + j0 + jb) * Net::CH3)[v];
      *reinterpret_cast<uint4*>(sm.a3() + s * G::SAL + jb * Net::CH3 + v * (16 / (int)sizeof(T))) =
          val;
    }
    __syncthreads();
  };
  for (int g = 0; g < NFULL; ++g) {
    stage(g * NG, NG);
    hidden_fc<Net, P, NG>(wt, sm.a3(), g * NG, hacc, wave, lane);
    __syncthreads();
  }
  if constexpr (TAIL > 0) {
    stage(NFULL * NG, TAIL);
    hidden_fc<Net, P, TAIL>(wt, sm.a3(), NFULL * NG, hacc, wave, lane);
    __syncthreads();
  }
  hybrid_head<Net, P, false>(wt, relu_mask, sm, hacc, nullptr, nullptr);
  __syncthreads();
  if (tid < MT * Net::NOUT) {
    const int ss = tid / Net::NOUT, o = tid % Net::NOUT;
    if (b0 + ss < B) logits[(b0 + ss) * Net::NOUT + o] = sm.logit[ss][o];
  }
}

// Training-form forward over explicit windows: the trunk and the hidden
// layer, keeping every activation (the head runs as a GEMM afterwards).
template <class Net, class P>
__global__ void __launch_bounds__(Net::WAVES * 64)
    forward_save_kernel(DevWeights wt, uint32_t relu_mask, const float* __restrict__ x,
                        int64_t B, SaveBlock sb) {
  using G = Geo<Net, P>;
  using T = typename P::T;
  constexpr int NT = G::NT, D = Net::D, BS = Net::BS;
  __shared__ NetSmem<Net, P> sm;
  const int tid = threadIdx.x;
  const int64_t b0 = (int64_t)blockIdx.x * MT;
  using GA = Gather<Net, P>;
  constexpr int GSL = GA::GSL, TPR = GA::TPR, CPT = GA::CPT;
  const int row = tid / TPR, part = tid % TPR;
  const int s = row / GSL, t = row % GSL;
  if constexpr (P::SCALED)
    for (int c = tid; c < D; c += NT) sm.x_inv[c] = wt.x_inv[c];
  __syncthreads();
  const int64_t b = b0 + s;
  auto load = [&](int j0, int nb) {
    return request_window_row<Net, CPT, TPR>(x, B, b, j0 * BS + t, t < nb * BS, part);
  };
  auto commit = [&](int j0, int nb, const RowRegs<CPT>& r, T* X) {
    (void)j0;
    if (t < nb * BS) commit_window_row<Net, P>(sm.x_inv, s, t, part, r, X);
  };
  SavePtrs<T> sv;
  sv.a1 = static_cast<T*>(sb.a1) + b0 * (Net::NB * BS / 2) * Net::CH1;
  sv.a2 = static_cast<T*>(sb.a2) + b0 * (Net::NB * BS / 4) * Net::CH2;
  sv.a3 = static_cast<T*>(sb.a3) + b0 * Net::NB * Net::CH3;
  sv.h = static_cast<T*>(sb.h) + b0 * Net::HID;
  sv.rows = (int)(B - b0 < MT ? B - b0 : MT);
  predict_tile<Net, P, false, true>(wt, relu_mask, sm, load, commit, nullptr, nullptr, sv);
}

// (the hidden FC's 8-fragment weight chunks requested two ahead, as the step
// kernel's variant 3: 2 % faster than one ahead here, no spills)
template <class P>
static hipError_t launch_fwd_save_t(const DevWeights& w, uint32_t relu, const float* x, int64_t B,
                                    const SaveBlock& sb, hipStream_t stream) {
  const dim3 grid((unsigned)((B + MT - 1) / MT)), block(Geo<NetC3, P>::NT);
  hipLaunchKernelGGL((forward_save_kernel<NetC3V3, P>), grid, block, 0, stream, w, relu, x, B, sb);
  return hipGetLastError();
}

hipError_t launch_forward_save(int prec, const DevWeights& w, uint32_t relu, const float* x,
                               int64_t B, const SaveBlock& sb, hipStream_t stream) {
  return prec == 0 ? launch_fwd_save_t<PF32>(w, relu, x, B, sb, stream)
                   : launch_fwd_save_t<PBF16>(w, relu, x, B, sb, stream);
}

// Every sub-trace back to its first instruction.  The rings and the last
// retire times need not be cleared: with no instruction in flight and
// position 0 no entry is read before it is written, and clearing the rings
// took 63 of this kernel's 65 us at 1,000 sub-traces (440 strided stores a
// thread).  C: how many entries of each are cleared all the same (sim_reset).
__global__ void reset_kernel(DevState st, int32_t n_sub, int32_t C, int32_t n_slots) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_slots) st.slot_kid[i] = -1;
  if (i == 0) *st.next = 0u;
  if (i < n_sub) {
    st.cur[i] = 0;
    st.t_w[i] = 0;
    st.r_prev[i] = 0;
    st.pos[i] = 0;
    st.head[i] = 0;
    st.count[i] = 0;
    st.fetch[i] = 0;
    st.drain[i] = 0;
    st.final_tick[i] = 0;
    st.warm_tick[i] = 0;
    if (st.m_head) {
      st.m_head[i] = 0;
      st.m_count[i] = 0;
      st.m_inpq[i] = 0;
      st.x_prev[i] = 0;
    }
    for (int e = 0; e < C; ++e) {
      st.q_idx[i * C + e] = 0;
      st.q_e[i * C + e] = 0;
      st.q_t[i * C + e] = 0;
      st.q_r[i * C + e] = 0;
    }
  }
  if (i < NCOUNTERS) st.counters[i] = 0;
}

// total = sum_k (final_tick[k] - warm_tick[k]), one workgroup.
__global__ void __launch_bounds__(256) total_kernel(DevState st, int32_t n_sub, int64_t* total) {
  __shared__ long long part[4];
  long long acc = 0;
  for (int k = threadIdx.x; k < n_sub; k += 256) acc += st.final_tick[k] - st.warm_tick[k];
  for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) *total = part[0] + part[1] + part[2] + part[3];
}

template <class Net, class P>
static hipError_t launch_step_t(const DevWeights& w, uint32_t relu, const DevState& s,
                                const StepParams& p, hipStream_t stream) {
  const dim3 grid(p.n_wg), block(Geo<Net, P>::NT);
  if constexpr (std::is_same<Net, NetC3>::value) {
    if (p.lat_mode != 1 && p.col_dep >= 0) {
      hipLaunchKernelGGL((step_kernel<Net, P, true, false, true>), grid, block, 0, stream, w,
                         relu, s, p);
      return hipGetLastError();
    }
  }
  if (p.lat_mode == 1)
    hipLaunchKernelGGL((step_kernel<Net, P, false>), grid, block, 0, stream, w, relu, s, p);
  else
    hipLaunchKernelGGL((step_kernel<Net, P, true>), grid, block, 0, stream, w, relu, s, p);
  return hipGetLastError();
}

template <class Net>
static hipError_t launch_step_n(int prec, const DevWeights& w, uint32_t relu, const DevState& s,
                                const StepParams& p, hipStream_t stream) {
  if (prec == 0) return launch_step_t<Net, PF32>(w, relu, s, p, stream);
  if (prec == 1) return launch_step_t<Net, PBF16>(w, relu, s, p, stream);
  return launch_step_t<Net, PFP8>(w, relu, s, p, stream);
}

template <class Net>
static const void* c3_step_fn(int prec) {
  if (prec == 0) return reinterpret_cast<const void*>(&step_kernel<Net, PF32, true>);
  if (prec == 1) return reinterpret_cast<const void*>(&step_kernel<Net, PBF16, true>);
  return reinterpret_cast<const void*>(&step_kernel<Net, PFP8, true>);
}

static const void* small_step_fn(int prec, bool run_net) {
  auto fn = [&](auto form) {
    using P = decltype(form);
    return run_net ? reinterpret_cast<const void*>(&small_step_kernel<P, true>)
                   : reinterpret_cast<const void*>(&small_step_kernel<P, false>);
  };
  return prec == 0 ? fn(PF32{}) : prec == 1 ? fn(PBF16{}) : fn(PFP8{});
}

hipError_t c3_step_scratch(int prec, int variant, size_t* bytes) {
  const void* f = variant == 1   ? c3_step_fn<NetC3V1>(prec)
                  : variant == 2 ? c3_step_fn<NetC3V2>(prec)
                  : variant == 3 ? c3_step_fn<NetC3V3>(prec)
                                 : c3_step_fn<NetC3>(prec);
  hipFuncAttributes a{};
  const hipError_t e = hipFuncGetAttributes(&a, f);
  *bytes = e == hipSuccess ? a.localSizeBytes : 0;
  return e;
}

hipError_t launch_step(int net, int prec, int variant, const DevWeights& w, uint32_t relu,
                       const DevState& s, const StepParams& p, hipStream_t stream) {
  if (net == 1 && p.lat_mode != 1 && variant == 1)
    return launch_step_n<NetC3V1>(prec, w, relu, s, p, stream);
  if (net == 1 && p.lat_mode != 1 && variant == 2)
    return launch_step_n<NetC3V2>(prec, w, relu, s, p, stream);
  if (net == 1 && p.lat_mode != 1 && variant == 3)
    return launch_step_n<NetC3V3>(prec, w, relu, s, p, stream);
  if (net == 4) {  // store latencies: FP32 and BF16 forms
    if (prec == 0) return launch_step_t<NetC3S, PF32>(w, relu, s, p, stream);
    if (prec == 1) return launch_step_t<NetC3S, PBF16>(w, relu, s, p, stream);
    return hipErrorInvalidValue;
  }
  if (net == 3) {  // hybrid head: FP32 and BF16 forms
    if (prec == 0) return launch_step_t<NetC3Hyb, PF32>(w, relu, s, p, stream);
    if (prec == 1) return launch_step_t<NetC3Hyb, PBF16>(w, relu, s, p, stream);
    return hipErrorInvalidValue;
  }
  if (net == 0 && prec == 0 && variant == WAVE_VARIANT) {
    // one wavefront per slot
    const dim3 grid((unsigned)(p.n_wg * MT)), block(64);
    if (p.lat_mode == 1)
      hipLaunchKernelGGL(wave_step_kernel<false>, grid, block, 0, stream, w, relu, s, p);
    else
      hipLaunchKernelGGL(wave_step_kernel<true>, grid, block, 0, stream, w, relu, s, p);
    return hipGetLastError();
  }
  if (net == 0 && prec == 0 && variant == QUAD_VARIANT) {
    // four wavefronts per slot
    const dim3 grid((unsigned)(p.n_wg * MT)), block(QW * 64);
    if (p.lat_mode == 1)
      hipLaunchKernelGGL(quad_step_kernel<false>, grid, block, 0, stream, w, relu, s, p);
    else
      hipLaunchKernelGGL(quad_step_kernel<true>, grid, block, 0, stream, w, relu, s, p);
    return hipGetLastError();
  }
  if (net == 0) {
    const void* f = small_step_fn(prec, p.lat_mode != 1);
    DevWeights wa = w;
    DevState sa = s;
    StepParams pa = p;
    void* args[] = {&wa, &relu, &sa, &pa};
    return hipLaunchKernel(f, dim3(p.n_wg), dim3(QW * 64), args, 0, stream);
  }
  return launch_step_n<NetC3>(prec, w, relu, s, p, stream);
}

template <class Net, class P>
static hipError_t launch_forward_t(const DevWeights& w, uint32_t relu, const float* x, int64_t B,
                                   float* logits, hipStream_t stream) {
  const dim3 grid((unsigned)((B + MT - 1) / MT)), block(Geo<Net, P>::NT);
  hipLaunchKernelGGL((forward_kernel<Net, P>), grid, block, 0, stream, w, relu, x, B, logits,
                     nullptr);
  return hipGetLastError();
}

template <class Net>
static hipError_t launch_forward_n(int prec, const DevWeights& w, uint32_t relu, const float* x,
                                   int64_t B, float* logits, hipStream_t stream) {
  if (prec == 0) return launch_forward_t<Net, PF32>(w, relu, x, B, logits, stream);
  if (prec == 1) return launch_forward_t<Net, PBF16>(w, relu, x, B, logits, stream);
  return launch_forward_t<Net, PFP8>(w, relu, x, B, logits, stream);
}

template <class Net>
static hipError_t launch_cal_t(const DevWeights& w, uint32_t relu, const DevState& s,
                               const StepParams& p, hipStream_t stream) {
  const dim3 grid(p.n_wg), block(Geo<Net, PF32>::NT);
  if constexpr (std::is_same<Net, NetC3>::value) {
    if (p.col_dep >= 0) {
      hipLaunchKernelGGL((step_kernel<Net, PF32, true, true, true>), grid, block, 0, stream, w,
                         relu, s, p);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((step_kernel<Net, PF32, true, true>), grid, block, 0, stream, w, relu, s, p);
  return hipGetLastError();
}

hipError_t launch_calibrate(int net, const DevWeights& w, uint32_t relu, const DevState& s,
                            const StepParams& p, hipStream_t stream) {
  return net == 0 ? launch_cal_t<NetSmall>(w, relu, s, p, stream)
                  : launch_cal_t<NetC3>(w, relu, s, p, stream);
}

int calibration_size(int net) { return net == 0 ? n_cal<NetSmall>() : n_cal<NetC3>(); }

hipError_t launch_forward(int net, int prec, const DevWeights& w, uint32_t relu, const float* x,
                          int64_t B, float* logits, hipStream_t stream) {
  if (net == 4) {
    if (prec == 0) return launch_forward_t<NetC3S, PF32>(w, relu, x, B, logits, stream);
    if (prec == 1) return launch_forward_t<NetC3S, PBF16>(w, relu, x, B, logits, stream);
    return hipErrorInvalidValue;
  }
  if (net == 3) {
    if (prec == 0) return launch_forward_t<NetC3Hyb, PF32>(w, relu, x, B, logits, stream);
    if (prec == 1) return launch_forward_t<NetC3Hyb, PBF16>(w, relu, x, B, logits, stream);
    return hipErrorInvalidValue;
  }
  return net == 0 ? launch_forward_n<NetSmall>(prec, w, relu, x, B, logits, stream)
                  : launch_forward_n<NetC3>(prec, w, relu, x, B, logits, stream);
}

hipError_t launch_reset(const DevState& s, int32_t n_sub, int32_t C, int32_t n_slots,
                        hipStream_t stream) {
  const int threads = 256;
  const int n = n_sub > n_slots ? n_sub : n_slots;
  const int blocks = (n + threads - 1) / threads;
  hipLaunchKernelGGL(reset_kernel, dim3(blocks > 0 ? blocks : 1), dim3(threads), 0, stream, s,
                     n_sub, C, n_slots);
  return hipGetLastError();
}

hipError_t launch_total(const DevState& s, int32_t n_sub, int64_t* total, hipStream_t stream) {
  hipLaunchKernelGGL(total_kernel, dim3(1), dim3(256), 0, stream, s, n_sub, total);
  return hipGetLastError();
}

// The run as a graph of kernel nodes (no memset nodes): the persistent step
// kernel until every slot is empty, then the total.
template <class Net, class P>
static void* step_fn(bool run_net, bool dep = false) {
  if constexpr (std::is_same<Net, NetC3>::value)
    if (run_net && dep) return reinterpret_cast<void*>(&step_kernel<Net, P, true, false, true>);
  return run_net ? reinterpret_cast<void*>(&step_kernel<Net, P, true>)
                 : reinterpret_cast<void*>(&step_kernel<Net, P, false>);
}

hipError_t build_run_graph(int net, int prec, int variant, const DevWeights& w, uint32_t relu,
                           const DevState& s, const StepParams& p, int64_t* total,
                           hipGraph_t* out) {
  const bool run_net = p.lat_mode != 1;
  void* fn;
  int nt;
  int grid_x = p.n_wg;
  if (net == 1 && run_net && variant == 1) {
    fn = prec == 0 ? step_fn<NetC3V1, PF32>(run_net)
         : prec == 1 ? step_fn<NetC3V1, PBF16>(run_net) : step_fn<NetC3V1, PFP8>(run_net);
    nt = Geo<NetC3V1, PF32>::NT;
  } else if (net == 1 && run_net && variant == 2) {
    fn = prec == 0 ? step_fn<NetC3V2, PF32>(run_net)
         : prec == 1 ? step_fn<NetC3V2, PBF16>(run_net) : step_fn<NetC3V2, PFP8>(run_net);
    nt = Geo<NetC3V2, PF32>::NT;
  } else if (net == 1 && run_net && variant == 3) {
    fn = prec == 0 ? step_fn<NetC3V3, PF32>(run_net)
         : prec == 1 ? step_fn<NetC3V3, PBF16>(run_net) : step_fn<NetC3V3, PFP8>(run_net);
    nt = Geo<NetC3V3, PF32>::NT;
  } else if (net == 0 && prec == 0 && variant == WAVE_VARIANT) {
    fn = run_net ? reinterpret_cast<void*>(&wave_step_kernel<true>)
                 : reinterpret_cast<void*>(&wave_step_kernel<false>);
    nt = 64;
    grid_x = p.n_wg * MT;
  } else if (net == 0 && prec == 0 && variant == QUAD_VARIANT) {
    fn = run_net ? reinterpret_cast<void*>(&quad_step_kernel<true>)
                 : reinterpret_cast<void*>(&quad_step_kernel<false>);
    nt = QW * 64;
    grid_x = p.n_wg * MT;
  } else if (net == 0) {
    fn = const_cast<void*>(small_step_fn(prec, run_net));
    nt = QW * 64;
  } else if (net == 3) {
    if (prec > 1) return hipErrorInvalidValue;
    fn = prec == 0 ? step_fn<NetC3Hyb, PF32>(run_net) : step_fn<NetC3Hyb, PBF16>(run_net);
    nt = Geo<NetC3Hyb, PF32>::NT;
  } else if (net == 4) {
    if (prec > 1) return hipErrorInvalidValue;
    fn = prec == 0 ? step_fn<NetC3S, PF32>(run_net) : step_fn<NetC3S, PBF16>(run_net);
    nt = Geo<NetC3S, PF32>::NT;
  } else {
    const bool dep = p.col_dep >= 0;
    fn = prec == 0 ? step_fn<NetC3, PF32>(run_net, dep)
         : prec == 1 ? step_fn<NetC3, PBF16>(run_net, dep) : step_fn<NetC3, PFP8>(run_net, dep);
    nt = Geo<NetC3, PF32>::NT;
  }
  hipGraph_t g = nullptr;
  hipError_t e = hipGraphCreate(&g, 0);
  if (e != hipSuccess) return e;
  DevWeights wa = w;
  uint32_t ra = relu;
  DevState sa = s;
  StepParams pa = p;
  void* step_args[] = {&wa, &ra, &sa, &pa};
  hipKernelNodeParams kp{};
  kp.func = fn;
  kp.gridDim = dim3(grid_x);
  kp.blockDim = dim3(nt);
  kp.sharedMemBytes = 0;
  kp.kernelParams = step_args;
  kp.extra = nullptr;
  hipGraphNode_t step_node = nullptr, total_node = nullptr;
  e = hipGraphAddKernelNode(&step_node, g, nullptr, 0, &kp);
  int32_t n_sub = p.n_sub;
  int64_t* tot = total;
  void* total_args[] = {&sa, &n_sub, &tot};
  hipKernelNodeParams kt{};
  kt.func = reinterpret_cast<void*>(&total_kernel);
  kt.gridDim = dim3(1);
  kt.blockDim = dim3(256);
  kt.sharedMemBytes = 0;
  kt.kernelParams = total_args;
  kt.extra = nullptr;
  if (e == hipSuccess) e = hipGraphAddKernelNode(&total_node, g, &step_node, 1, &kt);
  if (e != hipSuccess) {
    (void)hipGraphDestroy(g);
    return e;
  }
  *out = g;
  return hipSuccess;
}

// ------------------------------------------------------------------ RB7 ---

template <class P>
static hipError_t launch_rb_stage_t(int stage, const DevWeights& w, uint32_t relu,
                                    const DevState& s, const StepParams& p, hipStream_t stream) {
  const dim3 grid(p.n_wg), block(Geo<NetRB7, P>::NT);
  if (stage == 1)
    hipLaunchKernelGGL((step_kernel<NetRB7, P, true, false, false, 1>), grid, block, 0, stream, w,
                       relu, s, p);
  else
    hipLaunchKernelGGL((step_kernel<NetRB7, P, true, false, false, 2>), grid, block, 0, stream, w,
                       relu, s, p);
  return hipGetLastError();
}

hipError_t launch_rb_stage(int prec, int stage, const DevWeights& w, uint32_t relu,
                           const DevState& s, const StepParams& p, hipStream_t stream) {
  if ((stage != 1 && stage != 2) || p.n_steps != 1) return hipErrorInvalidValue;
  if (prec == 0) return launch_rb_stage_t<PF32>(stage, w, relu, s, p, stream);
  if (prec == 1) return launch_rb_stage_t<PBF16>(stage, w, relu, s, p, stream);
  return hipErrorInvalidValue;
}

template <class P, int ROWS, int WN>
static hipError_t launch_resblocks_t(const DevWeights& w, uint32_t relu, void* x, int64_t rows,
                                     const int32_t* active, hipStream_t stream) {
  const int64_t tiles = (rows + ROWS - 1) / ROWS;
  if (tiles > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL((resblock_kernel<P, ROWS, WN>), dim3((unsigned)tiles),
                     dim3((ResGeo<P, ROWS, WN>::NT)), 0, stream, w, relu,
                     static_cast<typename P::T*>(x), rows, active);
  return hipGetLastError();
}

// Rows per tile.  BF16: a workgroup (one per CU) streams all 13.8 MB of
// weights whatever its rows, so few rows run on small tiles spread over the
// chip and many on large ones: the tile with the least rounds of workgroups x
// measured time per round (13,000 rows, 1,000 windows: 128-row tiles 357 us,
// 64-row 205; 39,000 rows: 128 x 2 rounds 735, 96 x 2 544).  FP32: 16-row
// tiles, two of which share a CU and hide each other's latency (3,328 rows
// 740 us against 1,860 with 64-row tiles; 53,248 rows 5.65 ms against 6.82),
// but 64-row ones where one round of those holds the rows and 48 per CU do
// not (13,000 rows: 1.89 ms against 2.0).
struct ResTile {
  int rows, us;
};

static int res_tile_bf16(int64_t rows, int n_cu) {
  constexpr ResTile t[] = {{128, 360}, {96, 275}, {64, 205}, {32, 172}};
  int best = 0;
  int64_t least = 0;
  for (const ResTile& r : t) {
    const int64_t cu = n_cu > 0 ? n_cu : 1, tiles = (rows + r.rows - 1) / r.rows;
    const int64_t us = (tiles + cu - 1) / cu * r.us;
    if (best == 0 || us < least) {
      least = us;
      best = r.rows;
    }
  }
  return best;
}

hipError_t launch_resblocks(int prec, const DevWeights& w, uint32_t relu, void* x, int64_t rows,
                            const int32_t* active, int n_cu, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  if (prec == 0) {
    if (rows > (int64_t)48 * n_cu && rows <= (int64_t)64 * n_cu)
      return launch_resblocks_t<PF32, 64, 4>(w, relu, x, rows, active, stream);
    return launch_resblocks_t<PF32, 16, 8>(w, relu, x, rows, active, stream);
  }
  if (prec != 1) return hipErrorInvalidValue;
  switch (res_tile_bf16(rows, n_cu)) {
    case 32: return launch_resblocks_t<PBF16, 32, 8>(w, relu, x, rows, active, stream);
    case 64: return launch_resblocks_t<PBF16, 64, 8>(w, relu, x, rows, active, stream);
    case 96: return launch_resblocks_t<PBF16, 96, 8>(w, relu, x, rows, active, stream);
    default: return launch_resblocks_t<PBF16, 128, 4>(w, relu, x, rows, active, stream);
  }
}

hipError_t launch_rb_head(int prec, const DevWeights& w, uint32_t relu, const void* x, int64_t B,
                          const int32_t* active, float* logits, hipStream_t stream) {
  if (B <= 0) return hipSuccess;
  const dim3 grid((unsigned)((B + MT - 1) / MT)), block(NetRB7::WAVES * 64);
  if (prec == 0)
    hipLaunchKernelGGL((rb_head_kernel<PF32>), grid, block, 0, stream, w, relu,
                       static_cast<const float*>(x), B, active, logits);
  else if (prec == 1)
    hipLaunchKernelGGL((rb_head_kernel<PBF16>), grid, block, 0, stream, w, relu,
                       static_cast<const PBF16::T*>(x), B, active, logits);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_rb_trunk(int prec, const DevWeights& w, uint32_t relu, const float* x, int64_t B,
                           void* out, hipStream_t stream) {
  if (B <= 0) return hipSuccess;
  const dim3 grid((unsigned)((B + MT - 1) / MT)), block(NetRB7::WAVES * 64);
  if (prec == 0)
    hipLaunchKernelGGL((forward_kernel<NetRB7, PF32, true>), grid, block, 0, stream, w, relu, x, B,
                       nullptr, out);
  else if (prec == 1)
    hipLaunchKernelGGL((forward_kernel<NetRB7, PBF16, true>), grid, block, 0, stream, w, relu, x,
                       B, nullptr, out);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace simnet

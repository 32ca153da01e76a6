// The C3 networks' step and forward for few windows (gfx950): one tile of
// MT windows spread over several workgroups.
//
// The persistent step (kernels.hip) gives a tile to one workgroup, whose
// time per step is that of streaming 3.4 MB (BF16) of hidden-FC weights
// through one CU's L2 port after four groups' convolutions, ~52 us, however
// many CUs idle.  Here a step is one launch of tiles x units x slices
// workgroups: unit u gathers and convolves a contiguous share of the
// window's block groups and multiplies their hidden-FC inputs by one of CS
// column slices of the weights, leaving each group's FP32 sums in memory.
// The next launch's workgroups all begin by adding the groups' sums in order,
// then run the head and the clock and queue update on the tile (redundantly,
// so that no second launch and no wait between workgroups is needed).  A
// launch reads one of two buffers and writes the other, both the sums (every
// workgroup its groups') and the new scalars (unit 0 slice 0), so no workgroup
// reads what another of its launch writes, whenever each of them starts: beside
// another stream's kernel some start after others have ended.  The sums are
// those of the one-workgroup step in the same order, so the results are
// identical.
//
// Time per step, one workgroup per tile -> split (uniform sub-traces, 24 steps
// a call): BF16 16 sub-traces 46 -> 16 us, 512 48 -> 20, 1,024 49 -> 26, 2,048 51
// -> 42; FP32 16 218 -> 33, 512 220 -> 47, 2,048 220 -> 134; a forward of one
// window BF16 47 -> 15, FP32 207 -> 28.  What bounds a small step now: ~6 us
// to launch, add the sums and run the head and the update, then ~9 us of one
// group's convolutions and its slice of the hidden layer, each layer waiting
// for the latency of its weights.  (The first group's trace rows requested
// before the head changed nothing.)
//
// RB7's step is three launches: this kernel with the convolutions only, the
// residual blocks, FC 512's group sums (1,000 windows BF16: 28 + 357 + 38 +
// 10 us in four launches -> 15 + 205 + 15).
//
// The queue is a ring of QN = 128 entries indexed by position mod 128: an
// entry outlives its place among the newest C = 110 by 17 pushes, so the
// push of a launch never lands on an entry that launch reads, the row of
// window slot w is instruction first + pos - w, and r_{i-W} of the retire
// rule is the ring's entry of position i - W.
#include "predict.h"

namespace simnet {

// Groups of blocks of a form (as predict_tile runs them).
template <class Net, class P>
struct Groups {
  static constexpr int NG = Geo<Net, P>::NG, NFULL = Net::NB / NG, TAIL = Net::NB % NG;
  static constexpr int N = NFULL + (TAIL > 0);
  __device__ static int blocks(int g) { return g < NFULL ? NG : TAIL; }
};

int split_groups(int net, int prec) {
  if (net == 4)
    return prec == 0 ? Groups<NetC3S, PF32>::N : Groups<NetC3S, PBF16>::N;
  return prec == 0 ? Groups<NetC3, PF32>::N
         : prec == 1 ? Groups<NetC3, PBF16>::N : Groups<NetC3, PFP8>::N;
}

// A group's sums of tile `tile` in memory: [tile][group][hidden tile][lane],
// four columns each, as the MFMA accumulators hold them.
template <class Net, class P>
__device__ __forceinline__ float4* group_sums(float4* part, int tile, int g) {
  return part + ((size_t)tile * Groups<Net, P>::N + g) * (Net::HID / 16) * 64;
}

// The tile's hidden-layer sums: every group's, added in group order (wave w's
// tiles).
template <class Net, class P>
__device__ __forceinline__ void add_groups(const float4* part, int tile, v4f* hacc, int wave,
                                           int lane) {
  constexpr int HT = (Net::HID / 16) / Net::WAVES;
#pragma unroll
  for (int j = 0; j < HT; ++j) hacc[j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int g = 0; g < Groups<Net, P>::N; ++g) {
    const float4* src = group_sums<Net, P>(const_cast<float4*>(part), tile, g) +
                        (size_t)wave * HT * 64 + lane;
#pragma unroll
    for (int j = 0; j < HT; ++j) {
      const float4 v = src[j * 64];
      hacc[j] += v4f{v.x, v.y, v.z, v.w};
    }
  }
}

// This workgroup's groups [gb, ge): convolutions and one slice of the hidden
// FC, each group's sums to memory.  load and commit as in predict_tile.
// TRUNK: the convolutions only, the last one's output to sv.a3.
template <class Net, class P, int CS, bool SAVE, bool TRUNK, class Load, class Commit>
__device__ __forceinline__ void run_units(const DevWeights& wt, uint32_t relu_mask,
                                          NetSmem<Net, P>& sm, int tile, int gb, int ge, int slice,
                                          float4* part, SavePtrs<typename P::T> sv, Load&& load,
                                          Commit&& commit) {
  using GR = Groups<Net, P>;
  constexpr int NG = GR::NG, HT = (Net::HID / 16) / Net::WAVES / CS;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  v4f hacc[HT];
  float unused = 0.f;
  auto store = [&](int g) {
    if constexpr (TRUNK) return;
    float4* dst = group_sums<Net, P>(part, tile, g) +
                  (size_t)FcShape<Net, P, NG, CS>::tile0(slice, wave) * 64 + lane;
#pragma unroll
    for (int j = 0; j < HT; ++j)
      dst[j * 64] = make_float4(hacc[j][0], hacc[j][1], hacc[j][2], hacc[j][3]);
  };
  auto clear = [&]() {
#pragma unroll
    for (int j = 0; j < HT; ++j) hacc[j] = v4f{0.f, 0.f, 0.f, 0.f};
  };
  {
    auto regs = load(gb * NG, GR::blocks(gb));
    commit(gb * NG, GR::blocks(gb), regs, sm.x());
  }
  for (int g = gb; g < (ge < GR::NFULL ? ge : GR::NFULL); ++g) {
    lds_barrier();
    const int nj = (g + 1) * NG, nnb = g + 1 < ge ? GR::blocks(g + 1) : 0;
    clear();
    run_group<Net, P, NG, false, SAVE, TRUNK, CS>(
        wt, relu_mask, sm, g * NG, nullptr, nullptr, sv, hacc, unused,
        [&]() { return load(nj, nnb); },
        [&](const auto& regs) {
          if (nnb > 0) commit(nj, nnb, regs, sm.x());
        },
        slice);
    store(g);
  }
  if constexpr (GR::TAIL > 0) {
    if (ge == GR::N) {
      lds_barrier();
      clear();
      run_group<Net, P, GR::TAIL, false, SAVE, TRUNK, CS>(
          wt, relu_mask, sm, GR::NFULL * NG, nullptr, nullptr, sv, hacc, unused,
          []() { return 0; }, [](int) {}, slice);
      store(GR::NFULL);
    }
  }
}

// Unit u's groups: equal contiguous shares of all N.
template <class Net, class P>
__device__ __forceinline__ int unit_begin(int u, int units) {
  return u * Groups<Net, P>::N / units;
}

// ------------------------------------------------------------ simulation ---

template <class Net, class P>
struct SplitSmem {
  NetSmem<Net, P> net;
  int64_t first[MT], pos[MT], cur[MT];
  int32_t count[MT], active[MT];
  int32_t lat_e[MT], lat_s[MT];     // the instruction just pushed
  int32_t m_new[MT], m_vis[MT];     // stores shown: m_vis of them, up to sequence number m_new
};

// One step of every tile: (finish) the previous launch's sums sp.part[in]
// through the head and the update, from scalars sp.scal[in] to the other
// buffer; (predict) this step's sums, to the buffer that goes with the scalars
// as they are now.  Grid: tiles x units x CS, tile by tile, or
// (xcd_tiles = tiles) tile t's workgroups t mod 8 + 8 i.
template <class Net, class P, bool DEP, int CS>
__global__ void __launch_bounds__(Net::WAVES * 64)
    split_step_kernel(DevWeights wt, uint32_t relu_mask, DevState st, StepParams p, SplitBufs sp,
                      int units, int xcd_tiles, int in, int finish, int predict) {
  using G = Geo<Net, P>;
  using GA = Gather<Net, P>;
  using T = typename P::T;
  constexpr int C = Net::C, BS = Net::BS, QN = SPLIT_RING;
  static_assert(G::NT == MT * 32 && QN > C + WMAX, "32 threads per slot");
  __shared__ SplitSmem<Net, P> sm;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int per = units * CS;
  int tile = blockIdx.x / per, uc = blockIdx.x % per;
  if (xcd_tiles) {
    const int q = blockIdx.x / 8;
    tile = q / per * 8 + blockIdx.x % 8;
    uc = q % per;
    if (tile >= xcd_tiles) return;
  }
  const int unit = uc / CS, slice = uc % CS;
  const bool writer = uc == 0;
  // this half-wave's slot
  const int s = tid >> 5, l = tid & 31, hbase = lane & 32;
  const size_t slot = (size_t)tile * MT + s;
  const SlotConst c = sp.cst[slot];
  SlotScalars z = sp.scal[in][slot];
  const bool act = z.pos < c.n_pos;
  if (!__syncthreads_or(act)) {  // nothing left in the tile: the scalars move on
    if (writer && finish && l == 0) sp.scal[in ^ 1][slot] = z;
    if (Net::NRES > 0 && writer && l == 0) p.active_out[slot] = 0;
    return;
  }
  if constexpr (P::SCALED)
    for (int i = tid; i < Net::D; i += G::NT) sm.net.x_inv[i] = wt.x_inv[i];
  int32_t lat[3] = {0, 0, 0};
  if (finish) {
    int64_t qr[4], mx[4], mr[4];  // this slot's rings, entries l + 32 i
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      qr[i] = sp.q_r[slot * QN + l + 32 * i];
      mx[i] = Net::MWQ ? sp.m_x[slot * QN + l + 32 * i] : 0;
      mr[i] = Net::MWQ ? sp.m_r[slot * QN + l + 32 * i] : 0;
    }
    const int64_t ii = c.first + z.pos;  // the instruction predicted
    bool is_store = false;
    if constexpr (Net::MWQ)
      if (act)
        is_store = p.codes ? code_feature(p.codes[ii], p.store_col) != 0.f
                           : p.feat[ii * Net::D + p.store_col] != 0.f;
    v4f hacc[(Net::HID / 16) / Net::WAVES];
    // (RB7's are written between the launches, always to the first buffer)
    add_groups<Net, P>(reinterpret_cast<const float4*>(sp.part[Net::NRES > 0 ? 0 : in]), tile, hacc,
                       wave, lane);
    sm.net.stage_head(wt, tid, G::NT);
    __syncthreads();
    head_tile<Net, P, false, false>(wt, relu_mask, sm.net, hacc, nullptr, nullptr, {});
    __syncthreads();
    // round and update (Sec. 3.2, as step_kernel's), every lane of the
    // half-wave on the same values
    const float* o = sm.net.logit[s];
    const int64_t g = c.pred_off + z.pos;
    uint32_t clamped = 0, nonfinite = 0, mismatch = 0;
#pragma unroll
    for (int i = 0; i < Net::NLAT; ++i) {
      if constexpr (Net::HEAD == 1)
        lat[i] = hybrid_latency(o + i * HYB_PER_TYPE, p.lat_max, clamped, nonfinite);
      else
        lat[i] = round_latency(o[i], p.lat_max, clamped, nonfinite);
    }
    if (p.lat_mode != 0 && act) {
#pragma unroll
      for (int i = 0; i < Net::NLAT; ++i) {
        const int32_t inj = p.lat_table[g * Net::NLAT + i];
        if (inj != lat[i]) ++mismatch;
        lat[i] = inj;
      }
    }
    const int64_t Tn = z.cur + lat[0];
    // entries of the queue still in flight at Tn (r is monotone, so they are
    // its newest)
    int n_live = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // the newest position the entry can hold
      const int64_t q = z.pos - 1 - ((z.pos - 1 - (l + 32 * i)) & (QN - 1));
      const bool live = act && q >= z.pos - z.count && qr[i] > Tn;
      n_live += __popc((uint32_t)(__ballot(live) >> hbase));
    }
    int64_t r = Tn + lat[1] + 1;
    r = r > z.r_prev ? r : z.r_prev;
    {
      const int e = (int)((z.pos - p.W) & (QN - 1));
      const int64_t v = e < 32 ? qr[0] : e < 64 ? qr[1] : e < 96 ? qr[2] : qr[3];
      const int64_t rb = __shfl(v, hbase | (e & 31)) + 1;
      if (z.pos >= p.W) r = r > rb ? r : rb;
    }
    int64_t final_t = r;
    const int64_t pos = z.pos;
    if constexpr (Net::MWQ) {
      // memory write queue: sequence numbers [m_n - m_count, m_n)
      int n_x = 0, n_r = 0;
      int32_t mc = z.m_count;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int32_t q = z.m_n - 1 - ((z.m_n - 1 - (l + 32 * i)) & (QN - 1));
        n_x += __popc((uint32_t)(__ballot(act && q >= z.m_n - mc && mx[i] > Tn) >> hbase));
      }
      mc = n_x;  // (x is monotone: those gone by Tn are the oldest)
      int64_t x = Tn + lat[2] + 1;
      x = x > r ? x : r;
      x = x > z.x_prev ? x : z.x_prev;
      if (is_store && mc == C) --mc;  // the newest C stores suffice for the window
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int32_t q = z.m_n - 1 - ((z.m_n - 1 - (l + 32 * i)) & (QN - 1));
        n_r += __popc((uint32_t)(__ballot(act && q >= z.m_n - mc && mr[i] > Tn) >> hbase));
      }
      if (act) {
        if (is_store) {
          if (writer && l == 0) {
            const size_t at = slot * QN + (z.m_n & (QN - 1));
            sp.m_idx[at] = (int32_t)ii;
            sp.m_es[at] = pack_es(lat[1], lat[2]);
            sp.m_t[at] = Tn;
            sp.m_r[at] = r;
            sp.m_x[at] = x;
          }
          z.x_prev = x;
          ++z.m_n;
          ++mc;
          ++n_r;
        }
        z.m_count = mc;
        z.m_inpq = n_r;
        final_t = r > z.x_prev ? r : z.x_prev;
      }
    }
    if (act) {
      z.cur = Tn;
      z.r_prev = r;
      z.pos = pos + 1;
      z.count = n_live + 1 < C ? n_live + 1 : C;  // only the newest C stay visible
      if (pos + 1 == c.warm) z.t_w = Tn;
      z.ctr[0] += clamped;
      z.ctr[1] += nonfinite;
      z.ctr[2] += mismatch;
      ++z.ctr[3];
    }
    if (writer && l == 0) {
      sp.scal[in ^ 1][slot] = z;
      if (act) {
        const size_t at = slot * QN + (pos & (QN - 1));
        sp.q_e[at] = Net::MWQ ? pack_es(lat[1], lat[Net::NLAT - 1]) : lat[1];
        sp.q_t[at] = Tn;
        sp.q_r[at] = r;
        if (p.logits_out)
          for (int i = 0; i < Net::NOUT; ++i) p.logits_out[g * Net::NOUT + i] = o[i];
        if (pos + 1 == c.n_pos) {  // last instruction: the drain ends (Eq. 1)
          st.fetch[c.kid] = Tn - z.t_w;
          st.drain[c.kid] = final_t - Tn;
          st.final_tick[c.kid] = final_t;
          st.warm_tick[c.kid] = z.t_w;
        }
      }
    }
  }
  if (!predict) return;
  if (l == 0) {
    sm.first[s] = c.first;
    sm.pos[s] = z.pos;
    sm.cur[s] = z.cur;
    sm.count[s] = z.count;
    sm.active[s] = z.pos < c.n_pos;
    sm.lat_e[s] = lat[1];
    sm.lat_s[s] = lat[2];
    // the stores shown: those that have left the processor queue and not
    // the memory write queue
    sm.m_new[s] = z.m_n - z.m_inpq;
    sm.m_vis[s] = z.m_count - z.m_inpq;
  }
  if (!__syncthreads_or(z.pos < c.n_pos)) {
    if (Net::NRES > 0 && writer && l == 0) p.active_out[slot] = 0;
    return;
  }

  constexpr int GSL = GA::GSL, TPR = GA::TPR;
  const int grow = tid / TPR, part = tid % TPR;
  const int gs = grow / GSL, gt = grow % GSL;
  auto load = [&](int j0, int nb) {
    typename GA::Regs r;
    const int w = j0 * BS + gt;
    int64_t idx = -1;
    r.res = 0.f;
    r.ex = 0.f;
    r.sto = 0.f;
    const size_t ring = ((size_t)tile * MT + gs) * QN;
    const int64_t i = sm.first[gs] + sm.pos[gs];
    if (gt < nb * BS && sm.active[gs]) {
      if (w <= sm.count[gs]) {  // (w = 0: the instruction itself)
        idx = i - w;
        if (w == 1 && finish) {  // pushed by this launch, at this tick
          r.ex = (float)sm.lat_e[gs];
          if (Net::MWQ) r.sto = (float)sm.lat_s[gs];
        } else if (w > 0) {
          const size_t e = ring + ((sm.pos[gs] - w) & (QN - 1));
          r.res = (float)(sm.cur[gs] - sp.q_t[e]);
          const int32_t es = sp.q_e[e];
          r.ex = (float)(Net::MWQ ? es & 0xffff : es);
          if (Net::MWQ) r.sto = (float)((uint32_t)es >> 16);
        }
      } else if (Net::MWQ && w <= sm.count[gs] + sm.m_vis[gs]) {
        const size_t e = ring + ((sm.m_new[gs] - (w - sm.count[gs])) & (QN - 1));
        idx = sp.m_idx[e];
        r.res = (float)(sm.cur[gs] - sp.m_t[e]);
        r.ex = (float)(sp.m_es[e] & 0xffff);
        r.sto = (float)((uint32_t)sp.m_es[e] >> 16);
      }
    }
    request_row<Net, P, DEP>(p, idx, w == 0, sm.active[gs] ? i : 0, part, r);
    return r;
  };
  auto commit = [&](int j0, int nb, const typename GA::Regs& r, T* X) {
    (void)j0;
    if (gt < nb * BS)
      commit_row<Net, P, false, DEP>(p, sm.net.x_inv, gs, gt, part, r, X, nullptr);
  };
  SavePtrs<T> sv{};
  constexpr bool TRUNK = Net::NRES > 0;  // (RB7: the rest of the network in its own kernels)
  if constexpr (TRUNK) {
    sv.a3 = static_cast<T*>(p.trunk_out) + (size_t)tile * MT * Net::NB * Net::CH3;
    sv.rows = MT;
    if (writer && l == 0) p.active_out[slot] = z.pos < c.n_pos;
  }
  run_units<Net, P, CS, TRUNK, TRUNK>(wt, relu_mask, sm.net, tile,
                                      unit_begin<Net, P>(unit, units),
                                      unit_begin<Net, P>(unit + 1, units), slice,
                                      reinterpret_cast<float4*>(sp.part[finish ? in ^ 1 : in]), sv,
                                      load, commit);
}

// Sub-trace state -> split form: slot i runs sub-trace order[i] (every
// sub-trace has a slot; longest first, so tiles finish from the last).
__global__ void __launch_bounds__(MT * 32)
    split_import_kernel(DevState st, SplitBufs sp, int32_t n_sub, int32_t C, int32_t W) {
  constexpr int QN = SPLIT_RING;
  const int s = threadIdx.x >> 5, l = threadIdx.x & 31;
  const size_t slot = (size_t)blockIdx.x * MT + s;
  const int k = slot < (size_t)n_sub ? st.order[slot] : -1;
  if (slot == 0 && l == 0) *st.next = (unsigned)n_sub;  // all claimed
  SlotConst c{};
  SlotScalars z{};
  c.kid = k;
  if (k >= 0) {
    c.first = st.first[k];
    c.n_pos = st.n_pos[k];
    c.pred_off = st.pred_off[k];
    c.warm = st.warm[k];
    z.cur = st.cur[k];
    z.t_w = st.t_w[k];
    z.r_prev = st.r_prev[k];
    z.pos = st.pos[k];
    z.count = st.count[k];
    if (st.m_head) {
      z.m_count = z.m_n = st.m_count[k];
      z.m_inpq = st.m_inpq[k];
      z.x_prev = st.x_prev[k];
    }
    // the ring: the retire times of the last W positions, then the queue
    for (int j = l; j < W && j < z.pos; j += 32) {
      const int64_t q = z.pos - 1 - j;
      if (q < z.pos - z.count) sp.q_r[slot * QN + (q & (QN - 1))] = st.rw[(size_t)k * WMAX + q % W];
    }
    const int head = st.head[k];
    for (int j = l; j < z.count; j += 32) {
      const int e = head + j < C ? head + j : head + j - C;
      const size_t from = (size_t)k * C + e;
      const size_t to = slot * QN + ((z.pos - z.count + j) & (QN - 1));
      sp.q_e[to] = st.q_e[from];
      sp.q_t[to] = st.q_t[from];
      sp.q_r[to] = st.q_r[from];
    }
    if (st.m_head) {
      const int mh = st.m_head[k];
      for (int j = l; j < z.m_count; j += 32) {
        const int e = mh + j < C ? mh + j : mh + j - C;
        const size_t from = (size_t)k * C + e, to = slot * QN + j;
        sp.m_idx[to] = st.m_idx[from];
        sp.m_es[to] = st.m_es[from];
        sp.m_t[to] = st.m_t[from];
        sp.m_r[to] = st.m_r[from];
        sp.m_x[to] = st.m_x[from];
      }
    }
  }
  if (l == 0) {
    sp.cst[slot] = c;
    sp.scal[0][slot] = z;  // (both: a tile with nothing left is in no launch)
    sp.scal[1][slot] = z;
  }
}

// Split form (scalars sp.scal[in]) -> sub-trace state, rings from entry 0;
// the counters added; finished sub-traces leave their slots.
__global__ void __launch_bounds__(MT * 32)
    split_export_kernel(DevState st, SplitBufs sp, int in, int32_t C, int32_t W) {
  constexpr int QN = SPLIT_RING;
  const int s = threadIdx.x >> 5, l = threadIdx.x & 31;
  const size_t slot = (size_t)blockIdx.x * MT + s;
  const SlotConst c = sp.cst[slot];
  const SlotScalars z = sp.scal[in][slot];
  const int k = c.kid;
  if (l == 0) {
    st.slot_kid[slot] = k >= 0 && z.pos < c.n_pos ? k : -1;
    for (int i = 0; i < NCOUNTERS; ++i)
      if (z.ctr[i]) atomicAdd(&st.counters[i], (unsigned long long)z.ctr[i]);
  }
  if (k < 0) return;
  for (int j = l; j < W && j < z.pos; j += 32) {
    const int64_t q = z.pos - 1 - j;
    st.rw[(size_t)k * WMAX + q % W] = sp.q_r[slot * QN + (q & (QN - 1))];
  }
  for (int j = l; j < z.count; j += 32) {
    const int64_t q = z.pos - z.count + j;
    const size_t from = slot * QN + (q & (QN - 1)), to = (size_t)k * C + j;
    st.q_idx[to] = (int32_t)(c.first + q);
    st.q_e[to] = sp.q_e[from];
    st.q_t[to] = sp.q_t[from];
    st.q_r[to] = sp.q_r[from];
  }
  if (st.m_head)
    for (int j = l; j < z.m_count; j += 32) {
      const size_t from = slot * QN + ((z.m_n - z.m_count + j) & (QN - 1)), to = (size_t)k * C + j;
      st.m_idx[to] = sp.m_idx[from];
      st.m_es[to] = sp.m_es[from];
      st.m_t[to] = sp.m_t[from];
      st.m_r[to] = sp.m_r[from];
      st.m_x[to] = sp.m_x[from];
    }
  if (l == 0) {
    st.cur[k] = z.cur;
    st.t_w[k] = z.t_w;
    st.r_prev[k] = z.r_prev;
    st.pos[k] = z.pos;
    st.head[k] = 0;
    st.count[k] = z.count;
    if (st.m_head) {
      st.m_head[k] = 0;
      st.m_count[k] = z.m_count;
      st.m_inpq[k] = z.m_inpq;
      st.x_prev[k] = z.x_prev;
    }
  }
}

hipError_t launch_split_import(const DevState& s, const SplitBufs& sp, int tiles, int32_t n_sub,
                               int32_t C, int32_t W, hipStream_t stream) {
  hipLaunchKernelGGL(split_import_kernel, dim3(tiles), dim3(MT * 32), 0, stream, s, sp, n_sub, C,
                     W);
  return hipGetLastError();
}

hipError_t launch_split_export(const DevState& s, const SplitBufs& sp, int tiles, int in,
                               int32_t C, int32_t W, hipStream_t stream) {
  hipLaunchKernelGGL(split_export_kernel, dim3(tiles), dim3(MT * 32), 0, stream, s, sp, in, C, W);
  return hipGetLastError();
}

// FC 512 of RB7's windows from x [windows][NB][CH3] (the blocks' output):
// each group's sums, a group staged into LDS where the fused step keeps its
// last conv output.  Tiles with no active window (NULL: all) are left out.
template <class P, int CS>
__global__ void __launch_bounds__(NetRB7::WAVES * 64)
    split_fc_kernel(DevWeights wt, const typename P::T* __restrict__ x, int64_t B,
                    const int32_t* __restrict__ active, float* __restrict__ sums, int units) {
  using Net = NetRB7;
  using G = Geo<Net, P>;
  using GR = Groups<Net, P>;
  constexpr int NG = GR::NG, HT = (Net::HID / 16) / Net::WAVES / CS;
  constexpr int EV = 16 / (int)sizeof(typename P::T), V = Net::CH3 / EV;
  __shared__ alignas(16) typename P::T a3[MT * G::SAL];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int per = units * CS, tile = blockIdx.x / per, uc = blockIdx.x % per;
  const int unit = uc / CS, slice = uc % CS;
  const int64_t b0 = (int64_t)tile * MT;
  if (active) {
    const int a = tid < MT && b0 + tid < B ? active[b0 + tid] : 0;
    if (!__syncthreads_or(a)) return;
  }
  auto group = [&](int g, auto nb_tag) {
    constexpr int NBG = decltype(nb_tag)::value;
    auto head = fc_head<Net, P, NBG, CS>(wt, g * NG, wave, lane, slice);
    for (int i = tid; i < MT * NBG * V; i += G::NT) {
      const int s = i / (NBG * V), r = i % (NBG * V), jb = r / V, v = r % V;
      uint4 val = make_uint4(0u, 0u, 0u, 0u);
      if (b0 + s < B)
        val = reinterpret_cast<const uint4*>(x + ((b0 + s) * Net::NB + g * NG + jb) * Net::CH3)[v];
      *reinterpret_cast<uint4*>(a3 + s * G::SAL + jb * Net::CH3 + v * EV) = val;
    }
    lds_barrier();
    v4f hacc[HT];
#pragma unroll
    for (int j = 0; j < HT; ++j) hacc[j] = v4f{0.f, 0.f, 0.f, 0.f};
    hidden_fc<Net, P, NBG, true, CS>(wt, a3, g * NG, hacc, wave, lane, &head, slice);
    float4* dst = group_sums<Net, P>(reinterpret_cast<float4*>(sums), tile, g) +
                  (size_t)FcShape<Net, P, NBG, CS>::tile0(slice, wave) * 64 + lane;
#pragma unroll
    for (int j = 0; j < HT; ++j)
      dst[j * 64] = make_float4(hacc[j][0], hacc[j][1], hacc[j][2], hacc[j][3]);
    lds_barrier();
  };
  const int gb = unit_begin<Net, P>(unit, units), ge = unit_begin<Net, P>(unit + 1, units);
  for (int g = gb; g < (ge < GR::NFULL ? ge : GR::NFULL); ++g)
    group(g, std::integral_constant<int, NG>{});
  if constexpr (GR::TAIL > 0)
    if (ge == GR::N) group(GR::NFULL, std::integral_constant<int, GR::TAIL>{});
}

template <class P>
static hipError_t launch_split_fc_t(const DevWeights& w, const void* x, int64_t B,
                                    const int32_t* active, float* sums, SplitShape sh,
                                    hipStream_t stream) {
  const dim3 grid((unsigned)((B + MT - 1) / MT * sh.units * sh.slices)), block(NetRB7::WAVES * 64);
  const auto* xt = static_cast<const typename P::T*>(x);
  if (sh.slices == 4)
    hipLaunchKernelGGL((split_fc_kernel<P, 4>), grid, block, 0, stream, w, xt, B, active, sums,
                       sh.units);
  else if (sh.slices == 2)
    hipLaunchKernelGGL((split_fc_kernel<P, 2>), grid, block, 0, stream, w, xt, B, active, sums,
                       sh.units);
  else
    hipLaunchKernelGGL((split_fc_kernel<P, 1>), grid, block, 0, stream, w, xt, B, active, sums,
                       sh.units);
  return hipGetLastError();
}

hipError_t launch_split_fc(int prec, const DevWeights& w, const void* x, int64_t B,
                           const int32_t* active, float* sums, SplitShape sh,
                           hipStream_t stream) {
  if (prec == 0) return launch_split_fc_t<PF32>(w, x, B, active, sums, sh, stream);
  if (prec == 1) return launch_split_fc_t<PBF16>(w, x, B, active, sums, sh, stream);
  return hipErrorInvalidValue;
}

template <class Net, class P, bool DEP>
static hipError_t launch_split_step_t(const DevWeights& w, uint32_t relu, const DevState& s,
                                      const StepParams& p, const SplitBufs& sp, SplitShape sh,
                                      int tiles, int in, int finish, int predict,
                                      hipStream_t stream) {
  const dim3 block(Geo<Net, P>::NT);
  if (!predict) sh = SplitShape{1, 1, 0};  // the head and the update only
  if (Net::NRES > 0) sh.slices = 1;      // no hidden FC here
  // A tile's workgroups on one XCD (workgroup b runs on XCD b mod 8), where
  // each XCD's CUs hold its share: the sums that all of them add then cross
  // from the memory side once per tile, not once per workgroup.  us per step,
  // tile by tile -> this: BF16 64 sub-traces 17.1 -> 16.6, 512 25.9 -> 21.1,
  // 1,024 31.5 -> 27.1, 2,048 46.0 -> 42.8; FP32 512 55.1 -> 50.8.  Not FP32
  // with fewer tiles than XCDs, whose 7.2 MB of weights want every L2 (64
  // sub-traces 36.1 against 39.1).
  const int per = sh.units * sh.slices, rows = (tiles + 7) / 8;
  const int xcd =
      predict && rows * per * 8 <= sh.max_wgs && (P::ID != 0 || tiles >= 8) ? tiles : 0;
  const dim3 grid((unsigned)(xcd ? rows * 8 * per : tiles * per));
  if constexpr (Net::NRES > 0) {
    hipLaunchKernelGGL((split_step_kernel<Net, P, DEP, 1>), grid, block, 0, stream, w, relu, s, p,
                       sp, sh.units, xcd, in, finish, predict);
    return hipGetLastError();
  } else if (sh.slices == 4)
    hipLaunchKernelGGL((split_step_kernel<Net, P, DEP, 4>), grid, block, 0, stream, w, relu, s, p,
                       sp, sh.units, xcd, in, finish, predict);
  else if (sh.slices == 2)
    hipLaunchKernelGGL((split_step_kernel<Net, P, DEP, 2>), grid, block, 0, stream, w, relu, s, p,
                       sp, sh.units, xcd, in, finish, predict);
  else
    hipLaunchKernelGGL((split_step_kernel<Net, P, DEP, 1>), grid, block, 0, stream, w, relu, s, p,
                       sp, sh.units, xcd, in, finish, predict);
  return hipGetLastError();
}

hipError_t launch_split_step(int net, int prec, const DevWeights& w, uint32_t relu,
                             const DevState& s, const StepParams& p, const SplitBufs& sp,
                             SplitShape sh, int tiles, int in, int finish, int predict,
                             hipStream_t stream) {
  auto go = [&](auto net_tag, auto form_tag, auto dep_tag) {
    return launch_split_step_t<decltype(net_tag), decltype(form_tag), decltype(dep_tag)::value>(
        w, relu, s, p, sp, sh, tiles, in, finish, predict, stream);
  };
  using No = std::false_type;
  using Yes = std::true_type;
  if (net == 1 && p.col_dep >= 0)
    return prec == 0   ? go(NetC3V3{}, PF32{}, Yes{})
           : prec == 1 ? go(NetC3V3{}, PBF16{}, Yes{}) : go(NetC3V3{}, PFP8{}, Yes{});
  if (net == 1)
    return prec == 0   ? go(NetC3V3{}, PF32{}, No{})
           : prec == 1 ? go(NetC3V3{}, PBF16{}, No{}) : go(NetC3V3{}, PFP8{}, No{});
  if (net == 3 && prec <= 1)
    return prec == 0 ? go(NetC3Hyb{}, PF32{}, No{}) : go(NetC3Hyb{}, PBF16{}, No{});
  if (net == 4 && prec <= 1)
    return prec == 0 ? go(NetC3S{}, PF32{}, No{}) : go(NetC3S{}, PBF16{}, No{});
  if (net == 5 && prec <= 1)
    return prec == 0 ? go(NetRB7{}, PF32{}, No{}) : go(NetRB7{}, PBF16{}, No{});
  return hipErrorInvalidValue;
}

// --------------------------------------------------------------- forward ---

// Explicit windows x [B][L][D]: each group's sums, as split_step_kernel;
// SAVE (training form): the convolutions' outputs kept too (by slice 0);
// RB7: the last conv's output to sb.a3 only.
template <class Net, class P, int CS, bool SAVE>
__global__ void __launch_bounds__(Net::WAVES * 64)
    split_forward_kernel(DevWeights wt, uint32_t relu_mask, const float* __restrict__ x, int64_t B,
                         float* __restrict__ sums, int units, SaveBlock sb) {
  using G = Geo<Net, P>;
  using GA = Gather<Net, P>;
  using T = typename P::T;
  constexpr int BS = Net::BS, GSL = GA::GSL, TPR = GA::TPR, CPT = GA::CPT;
  __shared__ NetSmem<Net, P> sm;
  const int tid = threadIdx.x;
  const int per = units * CS, tile = blockIdx.x / per, uc = blockIdx.x % per;
  const int unit = uc / CS, slice = uc % CS;
  const int64_t b0 = (int64_t)tile * MT;
  const int row = tid / TPR, part = tid % TPR;
  const int s = row / GSL, t = row % GSL;
  if constexpr (P::SCALED) {
    for (int i = tid; i < Net::D; i += G::NT) sm.x_inv[i] = wt.x_inv[i];
    __syncthreads();
  }
  auto load = [&](int j0, int nb) {
    return request_window_row<Net, CPT, TPR>(x, B, b0 + s, j0 * BS + t, t < nb * BS, part);
  };
  auto commit = [&](int j0, int nb, const RowRegs<CPT>& r, T* X) {
    (void)j0;
    if (t < nb * BS) commit_window_row<Net, P>(sm.x_inv, s, t, part, r, X);
  };
  constexpr bool TRUNK = Net::NRES > 0;
  SavePtrs<T> sv{};
  if constexpr (TRUNK) {
    sv.a3 = static_cast<T*>(sb.a3) + b0 * Net::NB * Net::CH3;
    sv.rows = (int)(B - b0 < MT ? B - b0 : MT);
  } else if constexpr (SAVE) {
    sv.a1 = static_cast<T*>(sb.a1) + b0 * (Net::NB * BS / 2) * Net::CH1;
    sv.a2 = static_cast<T*>(sb.a2) + b0 * (Net::NB * BS / 4) * Net::CH2;
    sv.a3 = static_cast<T*>(sb.a3) + b0 * Net::NB * Net::CH3;
    sv.rows = slice == 0 ? (int)(B - b0 < MT ? B - b0 : MT) : 0;
  }
  run_units<Net, P, CS, SAVE || TRUNK, TRUNK>(
      wt, relu_mask, sm, tile, unit_begin<Net, P>(unit, units),
      unit_begin<Net, P>(unit + 1, units), slice, reinterpret_cast<float4*>(sums), sv, load,
      commit);
}

// The head on a tile's sums: raw outputs, or (SAVE) the hidden layer.
template <class Net, class P, bool SAVE>
__global__ void __launch_bounds__(Net::WAVES * 64)
    split_head_kernel(DevWeights wt, uint32_t relu_mask, const float* __restrict__ sums, int64_t B,
                      float* __restrict__ logits, void* __restrict__ h) {
  using T = typename P::T;
  __shared__ NetSmem<Net, P> sm;
  const int tid = threadIdx.x, tile = blockIdx.x;
  const int64_t b0 = (int64_t)tile * MT;
  v4f hacc[(Net::HID / 16) / Net::WAVES];
  add_groups<Net, P>(reinterpret_cast<const float4*>(sums), tile, hacc, tid >> 6, tid & 63);
  SavePtrs<T> sv{};
  if constexpr (SAVE) {
    sv.h = static_cast<T*>(h) + b0 * Net::HID;
    sv.rows = (int)(B - b0 < MT ? B - b0 : MT);
  } else {
    sm.stage_head(wt, tid, Net::WAVES * 64);
    __syncthreads();
  }
  head_tile<Net, P, false, SAVE>(wt, relu_mask, sm, hacc, nullptr, nullptr, sv);
  if constexpr (!SAVE) {
    __syncthreads();
    if (tid < MT * Net::NOUT) {
      const int s = tid / Net::NOUT, o = tid % Net::NOUT;
      if (b0 + s < B) logits[(b0 + s) * Net::NOUT + o] = sm.logit[s][o];
    }
  }
}

template <class Net, class P, bool SAVE>
static hipError_t launch_split_head_t(const DevWeights& w, uint32_t relu, const float* sums,
                                      int64_t B, float* logits, void* h, hipStream_t stream) {
  hipLaunchKernelGGL((split_head_kernel<Net, P, SAVE>), dim3((unsigned)((B + MT - 1) / MT)),
                     dim3(Geo<Net, P>::NT), 0, stream, w, relu, sums, B, logits, h);
  return hipGetLastError();
}

// RB7: convolutions of explicit windows to out [B][NB][CH3].
template <class P>
static hipError_t launch_split_trunk_t(const DevWeights& w, uint32_t relu, const float* x,
                                       int64_t B, void* out, SplitShape sh, hipStream_t stream) {
  const dim3 grid((unsigned)((B + MT - 1) / MT * sh.units)), block(NetRB7::WAVES * 64);
  hipLaunchKernelGGL((split_forward_kernel<NetRB7, P, 1, false>), grid, block, 0, stream, w, relu,
                     x, B, nullptr, sh.units, SaveBlock{nullptr, nullptr, out, nullptr});
  return hipGetLastError();
}

hipError_t launch_split_trunk(int prec, const DevWeights& w, uint32_t relu, const float* x,
                              int64_t B, void* out, SplitShape sh, hipStream_t stream) {
  if (prec == 0) return launch_split_trunk_t<PF32>(w, relu, x, B, out, sh, stream);
  if (prec == 1) return launch_split_trunk_t<PBF16>(w, relu, x, B, out, sh, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_split_rb_head(int prec, const DevWeights& w, uint32_t relu, const float* sums,
                                int64_t B, float* logits, hipStream_t stream) {
  if (prec == 0)
    return launch_split_head_t<NetRB7, PF32, false>(w, relu, sums, B, logits, nullptr, stream);
  if (prec == 1)
    return launch_split_head_t<NetRB7, PBF16, false>(w, relu, sums, B, logits, nullptr, stream);
  return hipErrorInvalidValue;
}

template <class Net, class P, bool SAVE>
static hipError_t launch_split_forward_t(const DevWeights& w, uint32_t relu, const float* x,
                                         int64_t B, float* logits, const SaveBlock& sb,
                                         float* sums, SplitShape sh, hipStream_t stream) {
  const unsigned tiles = (unsigned)((B + MT - 1) / MT);
  const dim3 block(Geo<Net, P>::NT), grid(tiles * sh.units * sh.slices);
  if (sh.slices == 4)
    hipLaunchKernelGGL((split_forward_kernel<Net, P, 4, SAVE>), grid, block, 0, stream, w, relu,
                       x, B, sums, sh.units, sb);
  else if (sh.slices == 2)
    hipLaunchKernelGGL((split_forward_kernel<Net, P, 2, SAVE>), grid, block, 0, stream, w, relu,
                       x, B, sums, sh.units, sb);
  else
    hipLaunchKernelGGL((split_forward_kernel<Net, P, 1, SAVE>), grid, block, 0, stream, w, relu,
                       x, B, sums, sh.units, sb);
  return launch_split_head_t<Net, P, SAVE>(w, relu, sums, B, logits, sb.h, stream);
}

hipError_t launch_split_forward(int net, int prec, const DevWeights& w, uint32_t relu,
                                const float* x, int64_t B, float* logits, const SaveBlock& sb,
                                float* sums, SplitShape sh, hipStream_t stream) {
  auto go = [&](auto net_tag, auto form_tag, auto save_tag) {
    return launch_split_forward_t<decltype(net_tag), decltype(form_tag),
                                  decltype(save_tag)::value>(w, relu, x, B, logits, sb, sums, sh,
                                                             stream);
  };
  using No = std::false_type;
  using Yes = std::true_type;
  if (net == 1)
    return prec == 0   ? go(NetC3V3{}, PF32{}, No{})
           : prec == 1 ? go(NetC3V3{}, PBF16{}, No{}) : go(NetC3V3{}, PFP8{}, No{});
  if (net == 2 && prec <= 1)
    return prec == 0 ? go(NetC3V3{}, PF32{}, Yes{}) : go(NetC3V3{}, PBF16{}, Yes{});
  if (net == 3 && prec <= 1)
    return prec == 0 ? go(NetC3Hyb{}, PF32{}, No{}) : go(NetC3Hyb{}, PBF16{}, No{});
  if (net == 4 && prec <= 1)
    return prec == 0 ? go(NetC3S{}, PF32{}, No{}) : go(NetC3S{}, PBF16{}, No{});
  return hipErrorInvalidValue;
}

// ----------------------------------------------------------- many windows ---

// A batch of more windows than one workgroup per CU takes in a round: the
// fused forward streams 3.4 MB of hidden-FC weights through each CU's L2 port
// for every 16 windows, ~30 of a round's 67 us.  Here the convolutions write
// their outputs (6.7 KB a window) to memory, ~38 us a round, and one launch
// runs the hidden layer on M tiles per workgroup, so that a weight fragment
// serves M tiles (256 CUs, us: M = 2 43, M = 3 55, M = 4 65; the weight stream
// alone 37).  Forward of C3, BF16, fused -> this (us): 8,192 windows 135 ->
// 120, 16,384 269 -> 219, 20,480 328 -> 289, 65,536 1,017 -> 843.  FP8 halves
// the weights and gains nothing (16,384: 224 -> 216, 4,100: 95.7 -> 96.1), so
// it stays fused.  FP32 is bound by its matrix instructions.

// The hidden layer and the head on M tiles of MT windows from the last conv's
// outputs x [B][NB][CH3].  A block's rows are staged into one of two LDS
// buffers while the block before is multiplied; a group's sums accumulate
// across its blocks and are then added, as hidden_fc does.
template <class Net, class P, int M>
__global__ void __launch_bounds__(Net::WAVES * 64)
    rows_head_kernel(DevWeights wt, uint32_t relu_mask, const typename P::T* __restrict__ x,
                     int64_t B, float* __restrict__ logits) {
  using G = Geo<Net, P>;
  using GR = Groups<Net, P>;
  using T = typename P::T;
  using S = FcShape<Net, P, 1>;
  constexpr int HT = S::HT, K = Net::CHL, SA = K + G::PAD, NT = G::NT;
  constexpr int EV = 16 / (int)sizeof(T), V = K / EV, R = M * MT;
  constexpr int PER = (R * V + NT - 1) / NT;  // 16-byte pieces per thread and block
  __shared__ NetSmem<Net, P> sm;
  static_assert(2 * R * SA <= G::NXA2, "staged rows fit X's region");
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t b0 = (int64_t)blockIdx.x * R;
  T* const buf = sm.x();
  uint4 r[PER];
  auto request = [&](int j) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int i = q * NT + tid, row = i / V, v = i % V;
      r[q] = make_uint4(0u, 0u, 0u, 0u);
      if (row < R && b0 + row < B)
        r[q] = reinterpret_cast<const uint4*>(x + ((b0 + row) * Net::NB + j) * K)[v];
    }
  };
  auto commit = [&](int j) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int i = q * NT + tid, row = i / V, v = i % V;
      if (row < R) *reinterpret_cast<uint4*>(buf + (j & 1) * R * SA + row * SA + v * EV) = r[q];
    }
  };
  v4f hacc[M][HT], acc[M][HT];
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int t = 0; t < HT; ++t) hacc[m][t] = acc[m][t] = v4f{0.f, 0.f, 0.f, 0.f};
  request(0);
  commit(0);
  for (int j = 0; j < Net::NB; ++j) {
    if (j + 1 < Net::NB) request(j + 1);
    const auto head = fc_head<Net, P, 1>(wt, j, wave, lane);
    lds_barrier();
    const T* ap[M];
#pragma unroll
    for (int m = 0; m < M; ++m)
      ap[m] = buf + (j & 1) * R * SA + (m * MT + (lane & 15)) * SA + (P::KG / 4) * (lane >> 4);
    mma_stream<P, S::KGS, Net::HID / 16, HT, M, Net::FC1_FRAGS, true>(acc, ap, S::weights(wt, j),
                                                                      wave * HT, lane, &head);
    if (j + 1 < Net::NB) commit(j + 1);
    if ((j + 1) % GR::NG == 0 || j + 1 == Net::NB)  // the group's last block
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int t = 0; t < HT; ++t) {
          hacc[m][t] += acc[m][t];
          acc[m][t] = v4f{0.f, 0.f, 0.f, 0.f};
        }
  }
  sm.stage_head(wt, tid, NT);
#pragma unroll
  for (int m = 0; m < M; ++m) {
    __syncthreads();
    head_tile<Net, P, false, false>(wt, relu_mask, sm, hacc[m], nullptr, nullptr, {});
    __syncthreads();
    if (tid < MT * Net::NOUT) {
      const int s = tid / Net::NOUT, o = tid % Net::NOUT;
      const int64_t b = b0 + m * MT + s;
      if (b < B) logits[b * Net::NOUT + o] = sm.logit[s][o];
    }
  }
}

// Convolutions of explicit windows, one workgroup per tile, to rows.
template <class Net, class P>
__global__ void __launch_bounds__(Net::WAVES * 64)
    rows_trunk_kernel(DevWeights wt, uint32_t relu_mask, const float* __restrict__ x, int64_t B,
                      typename P::T* __restrict__ rows) {
  using G = Geo<Net, P>;
  using GA = Gather<Net, P>;
  using T = typename P::T;
  constexpr int BS = Net::BS, GSL = GA::GSL, TPR = GA::TPR, CPT = GA::CPT;
  __shared__ NetSmem<Net, P> sm;
  const int tid = threadIdx.x;
  const int64_t b0 = (int64_t)blockIdx.x * MT;
  const int row = tid / TPR, part = tid % TPR;
  const int s = row / GSL, t = row % GSL;
  if constexpr (P::SCALED) {
    for (int i = tid; i < Net::D; i += G::NT) sm.x_inv[i] = wt.x_inv[i];
    __syncthreads();
  }
  auto load = [&](int j0, int nb) {
    return request_window_row<Net, CPT, TPR>(x, B, b0 + s, j0 * BS + t, t < nb * BS, part);
  };
  auto commit = [&](int j0, int nb, const RowRegs<CPT>& r, T* X) {
    (void)j0;
    if (t < nb * BS) commit_window_row<Net, P>(sm.x_inv, s, t, part, r, X);
  };
  SavePtrs<T> sv{};
  sv.a3 = rows + b0 * Net::NB * Net::CH3;
  sv.rows = (int)(B - b0 < MT ? B - b0 : MT);
  predict_tile<Net, P, false, true, true>(wt, relu_mask, sm, load, commit, nullptr, nullptr, sv);
}

template <class Net>
static hipError_t launch_forward_rows_t(const DevWeights& w, uint32_t relu, const float* x,
                                        int64_t B, uint16_t* rows, float* logits, int n_cu,
                                        hipStream_t stream) {
  using P = PBF16;
  const int64_t tiles = (B + MT - 1) / MT;
  const dim3 block(Geo<Net, P>::NT);
  hipLaunchKernelGGL((rows_trunk_kernel<Net, P>), dim3((unsigned)tiles), block, 0, stream, w, relu,
                     x, B, rows);
  auto head = [&](auto kernel, int m) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((tiles + m - 1) / m)), block, 0, stream, w, relu,
                       rows, B, logits);
  };
  // as few row tiles per workgroup as one round of workgroups allows
  if (tiles <= 2 * (int64_t)n_cu)
    head(rows_head_kernel<Net, P, 2>, 2);
  else if (tiles <= 3 * (int64_t)n_cu)
    head(rows_head_kernel<Net, P, 3>, 3);
  else
    head(rows_head_kernel<Net, P, 4>, 4);
  return hipGetLastError();
}

hipError_t launch_forward_rows(int net, const DevWeights& w, uint32_t relu, const float* x,
                               int64_t B, uint16_t* rows, float* logits, int n_cu,
                               hipStream_t stream) {
  if (net == 1) return launch_forward_rows_t<NetC3>(w, relu, x, B, rows, logits, n_cu, stream);
  if (net == 3) return launch_forward_rows_t<NetC3Hyb>(w, relu, x, B, rows, logits, n_cu, stream);
  return hipErrorInvalidValue;
}

}  // namespace simnet

// C ABI of libsimnet.so (declared in include/simnet.h): validation, context
// and device-state ownership, weight re-layout, dispatch to the kernels.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/simnet.h"
#include "simnet_internal.h"

using namespace simnet;

// Training form (net 2: C3 trunk, hidden layer kept, head FC 512 -> 802):
// FP32 master parameters, index maps for the device-side re-layouts, the
// packed trunk weights in the form's precision, permuted copies in the
// form's precision used by the forward head and the backward products, and
// the backward workspace.
struct TrainState {
  float* master = nullptr;
  int32_t* maps = nullptr;
  size_t map_pack[4] = {0}, n_pack[4] = {0};
  size_t map_perm[5] = {0}, n_perm[5] = {0};  // w1c, w2c, w3, w1, w2
  void* packed = nullptr;
  size_t pack_off[4] = {0};
  float* perm = nullptr;
  size_t perm_off[5] = {0};
  float* work = nullptr;
  int64_t work_B = 0;
  void* save = nullptr;  // copy of a save buffer off a 16-byte boundary (backward)
  int64_t save_B = 0;
  int2* inv = nullptr;  // per parameter: byte offsets in packed and perm (-1: none)
  size_t woff[5] = {0}, boff[5] = {0};
  size_t n_params = 0;
};

struct sim_ctx {
  sim_config cfg;
  int32_t n_sub = 0;
  int64_t n_instr = 0;
  const float* feat = nullptr;
  uint16_t* feat16 = nullptr;  // BF16 form: BF16 copy of feat (owned)
  int net = -1;  // 0 NetSmall, 1 NetC3, 2 C3 training head, 3 C3 hybrid inference head,
                 // 4 C3 with store latencies (memory write queue), 5 RB7 (staged step)
  int C = 0;
  uint32_t relu = 0;
  bool weights = false;
  bool completed = false;
  int64_t max_pos = 0, n_pred = 0, n_meas = 0;
  int32_t n_wg = 0;                 // persistent workgroups; slots = n_wg * MT
  int32_t n_wg_max = 0;             // slots allocated at init
  int32_t variant = 0;              // tuning variant of the step kernel
  int32_t n_cu = 0;
  std::vector<char> results;  // host side of sim_run's one copy
  // split step and forward (C3 networks, few windows): buffers, steps taken
  // since the reset (a lower bound; 0 from a captured reset on, which may be
  // replayed after any step), each tile's longest sub-trace in claim order
  SplitBufs split{};
  int64_t steps_done = 0;
  bool reset_captured = false;
  std::vector<int64_t> tile_len;
  const uint32_t* codes = nullptr;  // packed trace (SIM_FEAT_CODE32)
  const uint2* mem = nullptr;       // addresses for the dependency flags
  float* logits_out = nullptr;
  hipStream_t stream = nullptr;
  void* dev_block = nullptr;  // state + table
  void* dev_weights = nullptr;
  void* dev_w32 = nullptr;          // FP8 form: FP32 weights for calibration
  DevWeights w32{};
  std::vector<float> params;        // FP8 form: FP32 parameters as loaded
  std::vector<float> act_scale;     // per layer-input channel, after calibration
  bool calibrated = false;
  bool ran_to_end = false;          // an unbounded step launch has been issued
  bool use_graph = false;           // sim_run replays a graph of its kernels
  hipGraphExec_t graph_exec = nullptr;
  int32_t graph_mode = -1;
  const int32_t* graph_table = nullptr;
  float* graph_logits = nullptr;
  bool has_trace = true;
  TrainState tr;
  int64_t* dev_total = nullptr;
  // RB7: per slot the last conv's output [NB][CH3], activity, raw outputs;
  // predictor_fwd's workspace for B windows
  void* rb_trunk = nullptr;
  int32_t* rb_active = nullptr;
  float* rb_logits = nullptr;
  void* rb_ws = nullptr;
  int64_t rb_ws_B = 0;
  DevState st{};
  DevWeights w{};
  std::string err;
  float* scratch = nullptr;  // this device's address of `scratch` (sim_loss_noalloc)
};

// Device scratch of sim_loss_noalloc: the per-window losses before their
// fixed-order mean.  One copy per GPU the library runs on, held until the
// process ends.  Host code never passes this name to a kernel or a copy (on
// the host it is only a stand-in for the symbol): it uses the address that
// hipGetSymbolAddress returns for the device.
static __device__ __align__(256) float scratch[SIM_NOALLOC_MAX_B];

namespace {

constexpr int SCRATCH_DEVICES = 64;
std::mutex g_scratch_mu;
float* g_scratch[SCRATCH_DEVICES] = {};  // per device id, once resolved

// The address of `scratch` on the current device (resolved once per device,
// with that device current).
hipError_t scratch_address(float** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= SCRATCH_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch[dev] = static_cast<float*>(ptr);
  }
  *out = g_scratch[dev];
  return hipSuccess;
}

int fail(sim_ctx* c, int code, const char* fmt, ...) __attribute__((format(printf, 3, 4)));
int fail(sim_ctx* c, int code, const char* fmt, ...) {
  if (c) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    c->err = buf;
  }
  return code;
}

int hip_fail(sim_ctx* c, hipError_t e, const char* what) {
  return fail(c, SIM_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

// Window shapes with a kernel: (n_feat, n_slot) -> net id.
int window_net(int32_t n_feat, int32_t n_slot) {
  if (n_feat == NetSmall::D && n_slot == NetSmall::L) return 0;
  if (n_feat == NetC3::D && n_slot == NetC3::L) return 1;
  return -1;
}

int check_cfg(const sim_config* cfg, const sim_trace* tr, std::string* why) {
  auto bad = [&](const char* m) {
    if (why) *why = m;
    return SIM_EINVAL;
  };
  if (!cfg || !tr) return bad("null config or trace");
  if (cfg->n_feat < 1 || cfg->n_slot < 2) return bad("n_feat must be >= 1 and n_slot >= 2");
  if (cfg->n_out != 2 && cfg->n_out != 3)
    return bad("n_out must be 2 (fetch, execution) or 3 (and store)");
  if (cfg->retire_width < 1 || cfg->retire_width > WMAX) return bad("retire_width must be 1..16");
  const int32_t cols[3] = {cfg->col_res, cfg->col_exe, cfg->col_sto};
  for (int i = 0; i < 3; ++i) {
    if (cols[i] < -1 || cols[i] >= cfg->n_feat) return bad("dynamic column out of range");
    for (int j = 0; j < i; ++j)
      if (cols[i] >= 0 && cols[i] == cols[j]) return bad("dynamic columns must differ");
  }
  if (cfg->lat_max < 1) return bad("lat_max must be >= 1");
  if (cfg->prec < SIM_FP32 || cfg->prec > SIM_FP8E4M3) return bad("unknown precision");
  if (cfg->col_dep < -1 || cfg->col_dep + 5 > cfg->n_feat) return bad("col_dep out of range");
  if (cfg->col_dep >= 0)
    for (int i = 0; i < 3; ++i)
      if (cols[i] >= cfg->col_dep && cols[i] < cfg->col_dep + 5)
        return bad("dependency-flag columns overlap a dynamic column");
  if (cfg->n_out == 3) {
    if (cfg->store_col < 0 || cfg->store_col >= cfg->n_feat) return bad("store_col out of range");
    if (cfg->lat_max > 65535) return bad("lat_max must be <= 65535 with store latencies");
  }
  if (tr->n_sub == 0 && !tr->feat) return SIM_OK;  // predictor-only context (no trace)
  if (!tr->feat) return bad("feat is NULL");
  if (cfg->col_dep >= 0 && !tr->mem) return bad("dependency flags need the trace's addresses");
  if (tr->feat_dtype != SIM_FEAT_F32 && tr->feat_dtype != SIM_FEAT_CODE32)
    return bad("unknown feat_dtype");
  if (tr->feat_dtype == SIM_FEAT_CODE32 && cfg->n_feat < 30)
    return bad("packed codes expand to 30 static features: n_feat must be >= 30");
  if (tr->n_instr < 1 || tr->n_instr >= (int64_t)1 << 31) return bad("n_instr must be in [1, 2^31)");
  if (tr->n_sub < 1) return bad("n_sub must be >= 1");
  if (!tr->start || !tr->len || !tr->warm) return bad("sub-trace table is NULL");
  for (int32_t k = 0; k < tr->n_sub; ++k) {
    if (tr->len[k] < 1) return bad("every sub-trace needs len >= 1");
    if (tr->warm[k] < 0 || tr->warm[k] > tr->start[k]) return bad("warm must be in [0, start]");
    if (tr->start[k] < 0 || tr->start[k] + tr->len[k] > tr->n_instr)
      return bad("sub-trace outside the trace");
  }
  return SIM_OK;
}

// Storage encodings of the precision forms (host side).
uint16_t bf16_bits(float x) {  // round to nearest even
  uint32_t u;
  memcpy(&u, &x, 4);
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
float bf16_value(uint16_t b) {
  const uint32_t u = (uint32_t)b << 16;
  float x;
  memcpy(&x, &u, 4);
  return x;
}
// OCP FP8 e4m3: 1 sign, 4 exponent (bias 7), 3 mantissa bits, no infinities,
// largest finite 448.  Codes 0x00..0x7e are the non-negative finite values.
float e4m3_value(uint8_t code) {
  const int e = (code >> 3) & 15, m = code & 7;
  const float mag = e == 0 ? ldexpf((float)m, -9) : ldexpf(1.f + m / 8.f, e - 7);
  return (code & 0x80) ? -mag : mag;
}
uint8_t e4m3_bits(float x) {  // round to nearest even, saturating at +-448
  const uint8_t sign = x < 0 ? 0x80 : 0;
  const float a = fminf(fabsf(x), 448.f);
  int lo = 0, hi = 0x7e;  // largest code with value <= a
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (e4m3_value((uint8_t)mid) <= a) lo = mid; else hi = mid - 1;
  }
  int c = lo;
  if (c < 0x7e) {
    const float d0 = a - e4m3_value((uint8_t)c), d1 = e4m3_value((uint8_t)(c + 1)) - a;
    if (d1 < d0 || (d1 == d0 && (c & 1))) c += 1;
  }
  return (uint8_t)(sign | c);
}

// Smallest power of two s with amax <= 448 * s (1 when amax is 0): the scale
// that maps a channel's largest magnitude into e4m3's finite range.
float pow2_scale(float amax) {
  if (!(amax > 0.f)) return 1.f;
  const double a = amax;
  int e = (int)ceil(log2(a / 448.0));
  while (a > 448.0 * ldexp(1.0, e)) ++e;
  while (a <= 448.0 * ldexp(1.0, e - 1)) --e;
  return (float)ldexp(1.0, e);
}

constexpr size_t elem_size(int prec) { return prec == 0 ? 4 : prec == 1 ? 2 : 1; }

void store_elem(int prec, float v, uint8_t* dst) {
  if (prec == 0) memcpy(dst, &v, 4);
  else if (prec == 1) { const uint16_t b = bf16_bits(v); memcpy(dst, &b, 2); }
  else *dst = e4m3_bits(v);
}
float round_to(int prec, float v) {
  return prec == 0 ? v : prec == 1 ? bf16_value(bf16_bits(v)) : e4m3_value(e4m3_bits(v));
}

// B[k][n] packed per (k-group of KG, n-tile of TILE) as 64 lanes x 16
// bytes: lane holds B[kg*KG + E*(lane/TILE) + e][nt*TILE + lane%TILE],
// e < E = KG*TILE/64 (16x16 tiles: KG/4 k per lane; 32x32 tiles: KG/2).
template <class F>
void pack_b_tile(int prec, int K, int N, int KG, int TILE, F&& B, uint8_t* out) {
  const int KGS = K / KG, NTL = N / TILE, E = KG * TILE / 64;
  const size_t es = elem_size(prec);
  if (prec == 1) {  // (the common case, without a copy call per element)
    uint16_t* dst = reinterpret_cast<uint16_t*>(out);
    for (int kg = 0; kg < KGS; ++kg)
      for (int nt = 0; nt < NTL; ++nt)
        for (int lane = 0; lane < 64; ++lane) {
          const int k = kg * KG + E * (lane / TILE), n = nt * TILE + lane % TILE;
          for (int e = 0; e < E; ++e) *dst++ = bf16_bits(B(k + e, n));
        }
    return;
  }
  for (int kg = 0; kg < KGS; ++kg)
    for (int nt = 0; nt < NTL; ++nt)
      for (int lane = 0; lane < 64; ++lane)
        for (int e = 0; e < E; ++e)
          store_elem(prec, B(kg * KG + E * (lane / TILE) + e, nt * TILE + lane % TILE),
                     out + ((((size_t)kg * NTL + nt) * 64 + lane) * E + e) * es);
}
template <class F>
void pack_b(int prec, int K, int N, F&& B, uint8_t* out) {
  pack_b_tile(prec, K, N, kgroup(prec), 16, B, out);
}

struct Expect {
  int32_t kind, c_in, c_out;
};

template <class Net>
std::vector<Expect> expected_layers() {
  std::vector<Expect> v;
  v.push_back({0, Net::D, Net::CH1});
  v.push_back({0, Net::CH1, Net::CH2});
  if (Net::NCONV == 3) v.push_back({0, Net::CH2, Net::CH3});
  for (int i = 0; i < Net::NRES; ++i) {  // residual blocks: expansion, projection
    v.push_back({2, Net::CH3, Net::EXPAND});
    v.push_back({3, Net::EXPAND, Net::CH3});
  }
  if (Net::HID > 0) {
    v.push_back({1, Net::CHL * Net::NB, Net::HID});
    v.push_back({1, Net::HID, Net::NOUT});
  } else {
    v.push_back({1, Net::CHL * Net::NB, Net::NOUT});
  }
  return v;
}

// Offsets (bytes) of every array inside the packed weight block.
struct Layout {
  size_t conv_w[3], conv_b[3], conv_ws[3], conv_ai[3], x_inv, hid_w, hid_b, hid_ws, hid_ai,
      last_w, last_b, last_p, res_w, res_stride, res_b;
};

// Re-lay-out PyTorch-order FP32 parameters for one network and precision.
// FP8 scales (scales != NULL): per layer l, in_scale[l][c] is the scale of
// input channel c of layer l (window features for l = 0), a power of two;
// weights are multiplied by their input channel's scale before quantising,
// and each output channel gets the power-of-two weight scale that maps its
// largest magnitude into e4m3's range.
template <class Net>
std::vector<uint8_t> relayout(int prec, const float* params,
                              const std::vector<std::vector<float>>* in_scale, Layout* L) {
  std::vector<const float*> w, b;
  size_t off = 0;
  for (const Expect& e : expected_layers<Net>()) {
    const size_t nw = (size_t)e.c_out * e.c_in * (e.kind == 0 ? 2 : 1);
    w.push_back(params + off);
    off += nw;
    b.push_back(params + off);
    off += e.c_out;
  }
  const int DP = padded_feat(Net::D, prec);
  const int chp[4] = {DP, Net::CH1, Net::CH2, Net::CH3};
  const int chr[4] = {Net::D, Net::CH1, Net::CH2, Net::CH3};
  const size_t es = elem_size(prec);
  const bool fp8 = prec == 2;
  std::vector<uint8_t> out;
  auto reserve = [&](size_t bytes) {  // 256-byte aligned sections
    const size_t at = (out.size() + 255) / 256 * 256;
    out.resize(at + bytes, 0);
    return at;
  };
  auto put_floats = [&](const std::vector<float>& v) {
    const size_t at = reserve(v.size() * 4);
    memcpy(out.data() + at, v.data(), v.size() * 4);
    return at;
  };
  auto sin = [&](int l, int c) { return fp8 ? (*in_scale)[l][c] : 1.f; };
  // per-output-channel power-of-two weight scale for e4m3 (1 otherwise)
  auto wscale = [&](int l, int K, int co, auto&& wv) {
    std::vector<float> s(co, 1.f);
    if (!fp8) return s;
    for (int n = 0; n < co; ++n) {
      float amax = 0.f;
      for (int k = 0; k < K; ++k) amax = fmaxf(amax, fabsf(wv(k, n)));
      s[n] = pow2_scale(amax);
    }
    (void)l;
    return s;
  };
  for (int l = 0; l < Net::NCONV; ++l) {
    const int K = 2 * chp[l], N = chp[l + 1], cin = chr[l];
    const float* wl = w[l];
    auto wv = [&](int k, int n) {  // weight with its input channel's scale folded in
      const int t = k / chp[l], c = k % chp[l];
      return c < cin ? wl[((size_t)n * cin + c) * 2 + t] * sin(l, c) : 0.f;
    };
    const std::vector<float> ws = wscale(l, K, N, wv);
    L->conv_w[l] = reserve((size_t)K * N * es);
    pack_b(prec, K, N, [&](int k, int n) { return fp8 ? wv(k, n) / ws[n] : wv(k, n); },
           out.data() + L->conv_w[l]);
    L->conv_b[l] = put_floats(std::vector<float>(b[l], b[l] + N));
    L->conv_ws[l] = put_floats(ws);
    std::vector<float> ai(N, 1.f);
    if (fp8) {
      const bool next_is_conv = l + 1 < Net::NCONV;
      for (int n = 0; n < N; ++n) {
        // next layer's input channel n: conv channel n, or (hidden FC) the
        // flattened inputs n*NB + j, which share one scale per channel
        ai[n] = 1.f / (*in_scale)[l + 1][n];  // next layer's input channel n
        (void)next_is_conv;
      }
    }
    L->conv_ai[l] = put_floats(ai);
  }
  {
    std::vector<float> xi(Net::D, 1.f);
    if (fp8)
      for (int c = 0; c < Net::D; ++c) xi[c] = 1.f / (*in_scale)[0][c];
    L->x_inv = put_floats(xi);
  }
  if (Net::NRES > 0) {
    // residual blocks (no FP8 form): per block the expansion B[c][e] =
    // E[e][c] (PyTorch [EXPAND][CH3][1]) then the projection B[e][c] =
    // P[c][e] ([CH3][EXPAND][1]), packed for the form's residual MFMA
    const int C3 = Net::CH3, E = Net::EXPAND;
    const size_t half = (size_t)C3 * E * es;
    L->res_stride = (2 * half + 255) / 256 * 256;
    L->res_w = reserve(L->res_stride * Net::NRES);
    std::vector<float> rb;
    for (int i = 0; i < Net::NRES; ++i) {
      const float* We = w[Net::NCONV + 2 * i];
      const float* Wp = w[Net::NCONV + 2 * i + 1];
      uint8_t* dst = out.data() + L->res_w + L->res_stride * i;
      // BF16 on 32x32x16 tiles (k-groups of 16), FP32 on 16x16 ones
      const int KG = prec == 1 ? 16 : kgroup(prec), TILE = prec == 1 ? 32 : 16;
      pack_b_tile(prec, C3, E, KG, TILE, [&](int k, int n) { return We[(size_t)n * C3 + k]; },
                  dst);
      pack_b_tile(prec, E, C3, KG, TILE, [&](int k, int n) { return Wp[(size_t)n * E + k]; },
                  dst + half);
      rb.insert(rb.end(), b[Net::NCONV + 2 * i], b[Net::NCONV + 2 * i] + E);
      rb.insert(rb.end(), b[Net::NCONV + 2 * i + 1], b[Net::NCONV + 2 * i + 1] + C3);
    }
    L->res_b = put_floats(rb);
  }
  const int li = Net::NCONV + 2 * Net::NRES;
  if (Net::HID > 0) {
    const int K = Net::CHL, N = Net::HID, NB = Net::NB;
    const float* W1 = w[li];
    // one per-output scale over all blocks of the hidden layer
    auto wv = [&](int kk, int n) {  // kk = c*NB + j (PyTorch flatten index)
      return W1[(size_t)n * (K * NB) + kk] * sin(li, kk / NB);
    };
    const std::vector<float> ws = wscale(li, K * NB, N, wv);
    const size_t per = (size_t)K * N * es;
    L->hid_w = reserve(per * NB);
    for (int j = 0; j < NB; ++j)
      pack_b(prec, K, N,
             [&](int c, int n) {
               const int kk = c * NB + j;
               return fp8 ? wv(kk, n) / ws[n] : W1[(size_t)n * (K * NB) + kk];
             },
             out.data() + L->hid_w + per * j);
    L->hid_b = put_floats(std::vector<float>(b[li], b[li] + N));
    L->hid_ws = put_floats(ws);
    std::vector<float> ai(N, 1.f);
    if (fp8)
      for (int n = 0; n < N; ++n) ai[n] = 1.f / (*in_scale)[li + 1][n];
    L->hid_ai = put_floats(ai);
    // final FC on the VALU: weights rounded to the form (scale of its input folded)
    std::vector<float> lw((size_t)Net::NOUT * N);
    for (int o = 0; o < Net::NOUT; ++o) {
      float amax = 0.f;
      for (int n = 0; n < N; ++n) amax = fmaxf(amax, fabsf(w[li + 1][(size_t)o * N + n] * sin(li + 1, n)));
      const float s = fp8 ? pow2_scale(amax) : 1.f;
      for (int n = 0; n < N; ++n)
        lw[(size_t)o * N + n] = round_to(prec, w[li + 1][(size_t)o * N + n] * sin(li + 1, n) / s) * s;
    }
    L->last_w = put_floats(lw);
    L->last_b = put_floats(std::vector<float>(b[li + 1], b[li + 1] + Net::NOUT));
    L->last_p = 0;
    if (Net::HEAD == 1) {
      // hybrid head: the same rounded weights packed for one MFMA tile row,
      // outputs padded to whole 16-column tiles with zeros
      constexpr int NOUTP = (Net::NOUT + 15) / 16 * 16;
      L->last_p = reserve((size_t)N * NOUTP * es);
      pack_b(prec, N, NOUTP, [&](int k, int n) { return n < Net::NOUT ? lw[(size_t)n * N + k] : 0.f; },
             out.data() + L->last_p);
    }
  } else {
    const int K = Net::CHL, NB = Net::NB;
    const float* Wf = w[li];
    std::vector<float> lw((size_t)NB * Net::NOUT * K);
    for (int o = 0; o < Net::NOUT; ++o) {
      float amax = 0.f;
      for (int kk = 0; kk < K * NB; ++kk)
        amax = fmaxf(amax, fabsf(Wf[(size_t)o * (K * NB) + kk] * sin(li, kk / NB)));
      const float s = fp8 ? pow2_scale(amax) : 1.f;
      for (int j = 0; j < NB; ++j)
        for (int c = 0; c < K; ++c)
          lw[((size_t)j * Net::NOUT + o) * K + c] =
              round_to(prec, Wf[(size_t)o * (K * NB) + c * NB + j] * sin(li, c) / s) * s;
    }
    L->hid_w = L->hid_b = L->hid_ws = L->hid_ai = 0;
    L->last_w = put_floats(lw);
    L->last_b = put_floats(std::vector<float>(b[li], b[li] + Net::NOUT));
  }
  return out;
}

template <class Net>
size_t param_count() {
  size_t n = 0;
  for (const Expect& e : expected_layers<Net>())
    n += (size_t)e.c_out * e.c_in * (e.kind == 0 ? 2 : 1) + e.c_out;
  return n;
}

template <class Net>
bool layers_match(const sim_layer* layers, int32_t n) {
  const std::vector<Expect> ex = expected_layers<Net>();
  if ((size_t)n != ex.size()) return false;
  for (int32_t i = 0; i < n; ++i)
    if (layers[i].kind != ex[i].kind || layers[i].c_in != ex[i].c_in ||
        layers[i].c_out != ex[i].c_out)
      return false;
  return true;
}

}  // namespace

// The split step's and forward's buffers, laid out from byte `at` of a block
// (`base` NULL: the size only); returns the end.  Group sums for
// SPLIT_MAX_TILES tiles, and for a simulation whose slots fit them the
// per-slot state and its tiles' group sums once more.
static size_t split_layout(const sim_ctx* c, char* base, size_t at, SplitBufs* out) {
  const int net = c->cfg.n_out == 3 ? 4 : 1;
  const size_t groups = (size_t)split_groups(net, c->cfg.prec);
  const size_t slots =
      c->has_trace && c->n_wg_max <= SPLIT_MAX_TILES ? (size_t)c->n_wg_max * MT : 0;
  const size_t ring = slots * SPLIT_RING, mring = net == 4 ? ring : 0;
  auto take = [&](auto*& p, size_t n) {
    using T = std::remove_reference_t<decltype(*p)>;
    p = base && n ? reinterpret_cast<T*>(base + at) : nullptr;
    at += (n * sizeof(T) + 255) / 256 * 256;
  };
  SplitBufs b{};
  take(b.part[0], (size_t)SPLIT_MAX_TILES * groups * MT * NetC3::HID);
  take(b.part[1], slots * groups * NetC3::HID);
  take(b.cst, slots);
  take(b.scal[0], slots);
  take(b.scal[1], slots);
  take(b.q_e, ring);
  take(b.q_t, ring);
  take(b.q_r, ring);
  take(b.m_idx, mring);
  take(b.m_es, mring);
  take(b.m_t, mring);
  take(b.m_r, mring);
  take(b.m_x, mring);
  if (out) *out = b;
  return at;
}

static void drop_graph(sim_ctx* c) {
  if (c->graph_exec) (void)hipGraphExecDestroy(c->graph_exec);
  c->graph_exec = nullptr;
  c->graph_mode = -1;
}

// Pack params for one precision and upload them into *dev (replacing any
// previous block); fills *w with the device pointers.
static int upload_weights(sim_ctx* c, int prec, const float* params,
                          const std::vector<std::vector<float>>* scales, void** dev,
                          DevWeights* w) {
  Layout lay{};
  std::vector<uint8_t> packed = c->net == 0   ? relayout<NetSmall>(prec, params, scales, &lay)
                                : c->net == 3 ? relayout<NetC3Hyb>(prec, params, scales, &lay)
                                : c->net == 5 ? relayout<NetRB7>(prec, params, scales, &lay)
                                : c->net == 4 ? relayout<NetC3S>(prec, params, scales, &lay)
                                              : relayout<NetC3>(prec, params, scales, &lay);
  void* dw = nullptr;
  hipError_t e = hipMalloc(&dw, packed.size());
  if (e != hipSuccess) return hip_fail(c, e, "hipMalloc weights");
  e = hipMemcpy(dw, packed.data(), packed.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(dw);
    return hip_fail(c, e, "upload weights");
  }
  if (*dev) {
    (void)hipStreamSynchronize(c->stream);
    (void)hipFree(*dev);
  }
  *dev = dw;
  drop_graph(c);
  char* base = static_cast<char*>(dw);
  auto F = [&](size_t o) { return reinterpret_cast<const float*>(base + o); };
  *w = DevWeights{};
  const int nconv = c->net == 0 ? NetSmall::NCONV : NetC3::NCONV;
  for (int l = 0; l < nconv; ++l) {
    w->conv_w[l] = base + lay.conv_w[l];
    w->conv_b[l] = F(lay.conv_b[l]);
    w->conv_ws[l] = F(lay.conv_ws[l]);
    w->conv_ai[l] = F(lay.conv_ai[l]);
  }
  w->x_inv = F(lay.x_inv);
  if (c->net == 1 || c->net == 3 || c->net == 4 || c->net == 5) {
    w->hid_w = base + lay.hid_w;
    w->hid_b = F(lay.hid_b);
    w->hid_ws = F(lay.hid_ws);
    w->hid_ai = F(lay.hid_ai);
  }
  w->last_w = F(lay.last_w);
  w->last_b = F(lay.last_b);
  w->last_p = c->net == 3 || c->net == 5 ? base + lay.last_p : nullptr;
  if (c->net == 5) {
    w->res_w = base + lay.res_w;
    w->res_stride = (int64_t)lay.res_stride;
    w->res_b = F(lay.res_b);
  }
  return SIM_OK;
}

// Shape of a split launch over `tiles` tiles: one unit per group and as many
// column slices as one workgroup per CU allows (a workgroup's LDS fills a
// CU); with more tiles, fewer units of several groups.  units < 2: not worth
// splitting (one workgroup per tile).  More workgroups than CUs lose, each
// round paying the head and the update again (us per step, BF16: 16 tiles 4
// units x 4 slices 18.2, x 2 19.6; 32 tiles 4 units x 2 slices 21, x 1 25, x 4
// 37; 85 tiles 3 units 36, 4 units 52, 2 units 40; 128 tiles 2 units 43, 4
// units 57, unsplit 51; 163 tiles 2 units 81 against 54 unsplit).
static SplitShape split_shape(const sim_ctx* c, int64_t tiles) {
  const int32_t max = c->n_cu / 8 * 8;
  if (!c->split.part[0] || tiles < 1 || tiles > SPLIT_MAX_TILES) return SplitShape{1, 1, max};
  const int64_t groups = split_groups(c->net, c->cfg.prec);
  for (int32_t s : {4, 2, 1})
    if (tiles * groups * s <= c->n_cu) return SplitShape{(int32_t)groups, s, max};
  return SplitShape{(int32_t)std::min<int64_t>(groups, c->n_cu / tiles), 1, max};
}

// ------------------------------------------------------------ training ---

constexpr int TRAIN_BINS = 400, TRAIN_OUT = 2 * (TRAIN_BINS + 1);
// the head's operand rows padded to whole 16-byte vectors (BF16 and FP32)
// the head's outputs padded to whole 32-deep k-steps (its input-gradient
// product runs over them, the padding zero)
constexpr int TRAIN_LD = (TRAIN_OUT + 31) / 32 * 32;

static bool train_layers_match(const sim_layer* l, int32_t n) {
  const int32_t want[5][4] = {{0, 50, 64, 1}, {0, 64, 128, 1}, {0, 128, 256, 1},
                              {1, 3328, 512, 1}, {1, 512, TRAIN_OUT, 0}};
  if (n != 5) return false;
  for (int i = 0; i < 5; ++i)
    if (l[i].kind != want[i][0] || l[i].c_in != want[i][1] || l[i].c_out != want[i][2] ||
        (l[i].relu != 0) != (want[i][3] != 0))
      return false;
  return true;
}

// Index maps (source parameter, -1 for padding) of every re-layout the
// training form uses; built once per context.
static void build_train_maps(sim_ctx* c, std::vector<int32_t>* maps) {
  TrainState& T = c->tr;
  const int prec = c->cfg.prec;
  const int chs[4] = {50, 64, 128, 256};
  size_t off = 0;
  const int douts[5] = {64, 128, 256, 512, TRAIN_OUT};
  const int dins[5] = {50 * 2, 64 * 2, 128 * 2, 3328, 512};
  for (int l = 0; l < 5; ++l) {
    T.woff[l] = off;
    off += (size_t)douts[l] * dins[l];
    T.boff[l] = off;
    off += douts[l];
  }
  T.n_params = off;
  auto packed = [&](int K, int N, auto&& idx) {  // same order as the kernels' B fragments
    const int KG = kgroup(prec), KGS = K / KG, NTL = N / 16, E = KG / 4;
    for (int kg = 0; kg < KGS; ++kg)
      for (int nt = 0; nt < NTL; ++nt)
        for (int lane = 0; lane < 64; ++lane)
          for (int e = 0; e < E; ++e)
            maps->push_back(idx(kg * KG + E * (lane / 16) + e, nt * 16 + lane % 16));
  };
  const int DP = padded_feat(50, prec);
  const int chp[3] = {DP, 64, 128};
  for (int l = 0; l < 3; ++l) {
    T.map_pack[l] = maps->size();
    const int cin = chs[l];
    packed(2 * chp[l], chs[l + 1], [&](int k, int n) {
      const int t = k / chp[l], ch = k % chp[l];
      return ch < cin ? (int32_t)(T.woff[l] + ((size_t)n * cin + ch) * 2 + t) : -1;
    });
    T.n_pack[l] = maps->size() - T.map_pack[l];
  }
  T.map_pack[3] = maps->size();
  for (int j = 0; j < 13; ++j)
    packed(256, 512, [&](int ch, int n) { return (int32_t)(T.woff[3] + (size_t)n * 3328 + ch * 13 + j); });
  T.n_pack[3] = maps->size() - T.map_pack[3];
  // row-major copies, each contiguous along the dimension its products sum
  // over: conv l as [2*c_in][c_out] (input column t*c_in + c) and the hidden
  // layer as [3328][512] (input column p*256 + c), the input-gradient
  // products' right operands; the head as [TRAIN_LD][512] (the FP32 layout,
  // rows past 802 zero), the forward's right operand and the head's
  // input-gradient one
  for (int l = 0; l < 3; ++l) {
    T.map_perm[l] = maps->size();
    const int ci = chs[l], co = chs[l + 1];
    for (int k = 0; k < 2 * ci; ++k)
      for (int o = 0; o < co; ++o)
        maps->push_back((int32_t)(T.woff[l] + ((size_t)o * ci + k % ci) * 2 + k / ci));
    T.n_perm[l] = maps->size() - T.map_perm[l];
  }
  T.map_perm[3] = maps->size();
  for (int k = 0; k < 3328; ++k)
    for (int o = 0; o < 512; ++o)
      maps->push_back((int32_t)(T.woff[3] + (size_t)o * 3328 + (k % 256) * 13 + k / 256));
  T.n_perm[3] = maps->size() - T.map_perm[3];
  T.map_perm[4] = maps->size();
  for (int o = 0; o < TRAIN_LD; ++o)
    for (int j = 0; j < 512; ++j)
      maps->push_back(o < TRAIN_OUT ? (int32_t)(T.woff[4] + (size_t)o * 512 + j) : -1);
  T.n_perm[4] = maps->size() - T.map_perm[4];
}

// Re-lay-out the master parameters on the device (packed trunk weights in
// the form's precision, FP32 permuted copies).
static int relayout_train(sim_ctx* c) {
  TrainState& T = c->tr;
  const int bf16 = c->cfg.prec == SIM_BF16;
  // one launch for the nine re-layouts
  GatherSegs segs{};
  for (int l = 0; l < 4; ++l)
    segs.seg[segs.count++] = GatherSeg{T.maps + T.map_pack[l], (int64_t)T.n_pack[l],
                                       static_cast<char*>(T.packed) + T.pack_off[l], bf16};
  // the transposed copies (the head's is the forward's operand, the others
  // serve the backward products) in the form's precision: the BF16 form's
  // products round their operands to BF16 (nearest even, as here) anyway,
  // and BF16 operands are staged without conversion
  for (int l = 0; l < 5; ++l)
    segs.seg[segs.count++] = GatherSeg{T.maps + T.map_perm[l], (int64_t)T.n_perm[l],
                                       T.perm + T.perm_off[l], bf16};
  const hipError_t e = launch_map_gather_multi(T.master, segs, c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "training re-layout");
  DevWeights& w = c->w;
  w = DevWeights{};
  for (int l = 0; l < 3; ++l) {
    w.conv_w[l] = static_cast<char*>(T.packed) + T.pack_off[l];
    w.conv_b[l] = T.master + T.boff[l];
  }
  w.hid_w = static_cast<char*>(T.packed) + T.pack_off[3];
  w.hid_b = T.master + T.boff[3];
  return SIM_OK;
}

static int load_train_weights(sim_ctx* c, const sim_layer* layers, int32_t n_layers,
                              const float* params, int32_t on_device) {
  TrainState& T = c->tr;
  hipError_t e = hipSuccess;
  if (!T.maps) {
    std::vector<int32_t> maps;
    build_train_maps(c, &maps);
    e = hipMalloc(&T.maps, maps.size() * 4);
    if (e == hipSuccess) e = hipMemcpy(T.maps, maps.data(), maps.size() * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMalloc(&T.master, T.n_params * 4);
    size_t pb = 0;
    for (int l = 0; l < 4; ++l) {
      T.pack_off[l] = pb;
      pb += (T.n_pack[l] * elem_size(c->cfg.prec) + 255) / 256 * 256;
    }
    if (e == hipSuccess) e = hipMalloc(&T.packed, pb);
    size_t qf = 0;
    for (int l = 0; l < 5; ++l) {
      T.perm_off[l] = qf;
      qf += (T.n_perm[l] + 63) / 64 * 64;
    }
    // (a context without a simulation: the split forward's sums too, if they fit)
    const size_t pf = (qf * 4 + 255) / 256 * 256;
    const bool split = !c->split.part[0];
    if (e == hipSuccess && split) {
      if (hipMalloc(&T.perm, split_layout(c, nullptr, pf, nullptr)) == hipSuccess) {
        split_layout(c, reinterpret_cast<char*>(T.perm), pf, &c->split);
      } else {
        (void)hipGetLastError();
        T.perm = nullptr;
      }
    }
    if (e == hipSuccess && !T.perm) e = hipMalloc(&T.perm, qf * 4);
    if (e != hipSuccess) return hip_fail(c, e, "training buffers");
    // per master parameter its byte offsets in the packed and permuted
    // copies (-1: none), for sim_adam_load's re-layout in the update pass
    // (left off if a parameter appeared twice in one copy)
    const size_t es = c->cfg.prec == SIM_BF16 ? 2 : 4;
    std::vector<int2> inv(T.n_params, int2{-1, -1});
    bool once = true;
    for (int l = 0; l < 4; ++l)
      for (size_t q = 0; q < T.n_pack[l]; ++q) {
        const int32_t k = maps[T.map_pack[l] + q];
        if (k < 0) continue;
        once = once && inv[k].x < 0;
        inv[k].x = (int32_t)(T.pack_off[l] + q * es);
      }
    for (int l = 0; l < 5; ++l)
      for (size_t q = 0; q < T.n_perm[l]; ++q) {
        const int32_t k = maps[T.map_perm[l] + q];
        if (k < 0) continue;
        once = once && inv[k].y < 0;
        inv[k].y = (int32_t)(T.perm_off[l] * 4 + q * es);
      }
    if (once) {
      e = hipMalloc(&T.inv, inv.size() * sizeof(int2));
      if (e == hipSuccess)
        e = hipMemcpy(T.inv, inv.data(), inv.size() * sizeof(int2), hipMemcpyHostToDevice);
      if (e != hipSuccess) return hip_fail(c, e, "re-layout offsets");
    }
  }
  e = hipMemcpyAsync(T.master, params, T.n_params * 4,
                     on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "copy parameters");
  if (!on_device)  // host parameters must stay valid until copied
    if ((e = hipStreamSynchronize(c->stream)) != hipSuccess) return hip_fail(c, e, "copy parameters");
  uint32_t relu = 0;
  for (int32_t i = 0; i < n_layers; ++i)
    if (layers[i].relu) relu |= 1u << i;
  c->relu = relu;
  int rc = relayout_train(c);
  if (rc != SIM_OK) return rc;
  c->weights = true;
  return SIM_OK;
}

static bool capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

// Backward workspace (floats): [0] per-window losses, [1] dH [B][512],
// [2] dY3 [B*13][256], [3] dY2 [B*26][128], [4] dY1 [B*52][64], [5] the
// five bias sums' chunk partials, [6] split-K partial products, [7] the
// head's output gradients with rows padded to TRAIN_LD.
constexpr size_t SPLITK_CAP = (size_t)16 << 20;
// floats for the chunk partials of the bias sums (head, hidden, conv3..1),
// each list starting on a 64-float boundary
constexpr size_t BIAS_PART = colsum_workspace_floats(TRAIN_OUT + 512 + 256 + 128 + 64) + 5 * 64;
static size_t train_work_off(int64_t B, int part) {
  const size_t sizes[8] = {(size_t)B, (size_t)B * 512, (size_t)B * 3328, (size_t)B * 3328,
                           (size_t)B * 3328, BIAS_PART, SPLITK_CAP, (size_t)B * TRAIN_LD};
  size_t off = 0;
  for (int i = 0; i < part; ++i) off += (sizes[i] + 63) / 64 * 64;
  return off;
}

static int ensure_train_work(sim_ctx* c, int64_t B) {
  TrainState& T = c->tr;
  if (T.work && T.work_B >= B) return SIM_OK;
  if (T.work) {
    (void)hipStreamSynchronize(c->stream);
    (void)hipFree(T.work);
    T.work = nullptr;
  }
  hipError_t e = hipMalloc(&T.work, train_work_off(B, 8) * 4);
  if (e != hipSuccess) return hip_fail(c, e, "training workspace");
  T.work_B = B;
  return SIM_OK;
}

// Per-window activation bytes kept by the training forward.
static int64_t save_bytes_per_window(int prec) {
  return (int64_t)(52 * 64 + 26 * 128 + 13 * 256 + 512) * (int64_t)elem_size(prec);
}

static SaveBlock save_block(const sim_ctx* c, void* save, int64_t B) {
  const size_t es = elem_size(c->cfg.prec);
  char* p = static_cast<char*>(save);
  SaveBlock sb;
  sb.a1 = p;
  sb.a2 = p + (size_t)B * 52 * 64 * es;
  sb.a3 = p + (size_t)B * (52 * 64 + 26 * 128) * es;
  sb.h = p + (size_t)B * (52 * 64 + 26 * 128 + 13 * 256) * es;
  return sb;
}

// The activations on a 16-byte boundary, as the backward products' LDS-direct
// kernels and grouped weight gradients read them: `save` itself, else a copy in
// memory kept by the context (without that, or where there is none yet under
// capture, `save`: the general kernels).  It holds as many windows as T.work and
// so moves only when that does.  BF16 backward of 4,096 windows off the boundary
// 500 us by the general kernels, 256 copied first (212 on it); 16 windows 177, 72.
static const void* aligned_save(sim_ctx* c, const void* save, int64_t B, hipError_t* e) {
  TrainState& T = c->tr;
  if (reinterpret_cast<uintptr_t>(save) % 16 == 0) return save;
  const int64_t per = save_bytes_per_window(c->cfg.prec);
  if (T.save_B < B) {
    if (capturing(c->stream)) return save;
    if (T.save) {
      (void)hipStreamSynchronize(c->stream);
      (void)hipFree(T.save);
      T.save_B = 0;
    }
    if (hipMalloc(&T.save, (size_t)(T.work_B * per)) != hipSuccess) {
      (void)hipGetLastError();
      T.save = nullptr;
      return save;
    }
    T.save_B = T.work_B;
  }
  *e = hipMemcpyAsync(T.save, save, (size_t)(B * per), hipMemcpyDeviceToDevice, c->stream);
  return T.save;
}

// Outputs per window of a network's inference head.
static int n_outputs(int net) {
  return net == 3 || net == 5 ? NetC3Hyb::NOUT : net == 4 ? NetC3S::NOUT : NetC3::NOUT;
}

static GemmOperand opnd(const void* p, int bf16, int64_t rs, int64_t cs,
                        int64_t grp = NO_GROUP, int64_t gs = 0) {
  GemmOperand o;
  o.p = p;
  o.bf16 = bf16;
  o.rs = rs;
  o.cs = cs;
  o.grp = grp;
  o.gs = gs;
  o.ext = 0;
  return o;
}

// The operand with `ext` elements readable along its contiguous outer
// dimension (a copy whose rows are padded past M or N).
static GemmOperand padded(GemmOperand o, int64_t ext) {
  o.ext = ext;
  return o;
}

static GemmArgs gemm(GemmOperand A, GemmOperand B, float* C, int64_t ldc, int64_t M, int64_t N,
                     int64_t K, int beta) {
  GemmArgs g{};
  g.A = A;
  g.B = B;
  g.mask = opnd(nullptr, 0, 0, 0);
  g.C = C;
  g.ldc = ldc;
  g.cgrp = NO_GROUP;
  g.cgs = 0;
  g.ccg = 0;
  g.ccm = 0;
  g.M = M;
  g.N = N;
  g.K = K;
  g.bias = nullptr;
  g.beta = beta;
  return g;
}

// Sub-traces up to which sim_run brings its results to the host in one copy and
// then to the caller's arrays (us for the four arrays, one copy -> straight to
// each: 1,000 sub-traces 6 -> 62, 20,000 41 -> 101, 100,000 252 -> 202, 1,000,000
// 3,131 -> 2,005).
constexpr int32_t ONE_COPY_MAX_SUB = 65536;

// Sub-traces up to which the small network's FP32 step defaults to one
// wavefront per sub-trace (sim_set_tuning / sim_autotune can change it).
constexpr int32_t WAVE_MAX_SUB = 1024;

extern "C" {

int sim_validate_config(const sim_config* cfg, const sim_trace* trace) {
  return check_cfg(cfg, trace, nullptr);
}

// Sec. 3.3: the trace is cut into n_sub contiguous sub-traces of equal
// length, the first n_instr mod n_sub of them one instruction longer; each
// also simulates the min(warm_max, start) instructions before its start.
int sim_partition(int64_t n_instr, int32_t n_sub, int32_t warm_max, int64_t* start, int64_t* len,
                  int32_t* warm) {
  if (n_sub < 1 || n_instr < n_sub || warm_max < 0 || !start || !len || !warm)
    return SIM_EINVAL;
  const int64_t q = n_instr / n_sub, r = n_instr % n_sub;
  int64_t at = 0;
  for (int32_t k = 0; k < n_sub; ++k) {
    start[k] = at;
    len[k] = q + (k < r ? 1 : 0);
    warm[k] = (int32_t)(at < warm_max ? at : warm_max);
    at += len[k];
  }
  return SIM_OK;
}

int sim_init(const sim_config* cfg, const sim_trace* tr, sim_ctx** out) {
  if (!out) return SIM_EINVAL;
  *out = nullptr;
  sim_ctx* c = new (std::nothrow) sim_ctx();
  if (!c) return SIM_ENOMEM;
  std::string why;
  int rc = check_cfg(cfg, tr, &why);
  if (rc != SIM_OK) {
    fprintf(stderr, "sim_init: %s\n", why.c_str());
    delete c;
    return rc;
  }
  c->net = window_net(cfg->n_feat, cfg->n_slot);
  if (cfg->n_out == 3) c->net = c->net == 1 ? 4 : -1;  // store latencies: the C3 window only
  if (c->net < 0) {
    fprintf(stderr, "sim_init: no kernel for window %dx%d at precision %d\n", cfg->n_slot,
            cfg->n_feat, cfg->prec);
    delete c;
    return SIM_EUNSUPPORTED;
  }
  c->cfg = *cfg;
  c->C = cfg->n_slot - 1;
  c->stream = static_cast<hipStream_t>(cfg->stream);
  {
    const hipError_t e = scratch_address(&c->scratch);
    if (e != hipSuccess) {
      fprintf(stderr, "sim_init: device scratch: %s\n", hipGetErrorString(e));
      delete c;
      return SIM_EDEVICE;
    }
  }
  if (tr->n_sub == 0) {  // predictor-only: forward/backward on explicit windows
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&c->n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
      (void)hipGetLastError();
      c->n_cu = 0;
    }
    c->has_trace = false;
    *out = c;
    return SIM_OK;
  }
  c->n_sub = tr->n_sub;
  c->n_instr = tr->n_instr;
  if (tr->feat_dtype == SIM_FEAT_CODE32)
    c->codes = static_cast<const uint32_t*>(tr->feat);
  else
    c->feat = static_cast<const float*>(tr->feat);
  c->mem = static_cast<const uint2*>(tr->mem);
  c->stream = static_cast<hipStream_t>(cfg->stream);
  if (c->feat && cfg->prec == SIM_BF16) {
    // the BF16 form gathers from a BF16 copy of the rows (the values its
    // windows hold anyway), half the bytes per row
    const size_t bytes = sizeof(uint16_t) * (size_t)tr->n_instr * staged_feat(cfg->n_feat);
    hipError_t e = hipMalloc(&c->feat16, bytes);
    if (e == hipSuccess)
      e = launch_stage_bf16(c->feat, tr->n_instr, cfg->n_feat, c->feat16, c->stream);
    if (e != hipSuccess) {
      fprintf(stderr, "sim_init: %s\n", hipGetErrorString(e));
      if (c->feat16) (void)hipFree(c->feat16);
      delete c;
      return SIM_ENOMEM;
    }
  }

  const int32_t K = tr->n_sub, C = c->C;
  std::vector<int64_t> first(K), npos(K), poff(K);
  std::vector<int32_t> warm(K);
  int64_t acc = 0;
  for (int32_t k = 0; k < K; ++k) {
    first[k] = tr->start[k] - tr->warm[k];
    npos[k] = tr->warm[k] + tr->len[k];
    warm[k] = tr->warm[k];
    poff[k] = acc;
    acc += npos[k];
    c->n_meas += tr->len[k];
    c->max_pos = std::max(c->max_pos, npos[k]);
  }
  c->n_pred = acc;
  // claim order: longest first (ties by index) so the long ones start early
  std::vector<int32_t> order(K);
  for (int32_t k = 0; k < K; ++k) order[k] = k;
  std::stable_sort(order.begin(), order.end(),
                   [&](int32_t a, int32_t b) { return npos[a] > npos[b]; });
  for (int32_t i = 0; i < K; i += MT) c->tile_len.push_back(npos[order[i]]);
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      n_cu < 1) {
    fprintf(stderr, "sim_init: cannot query the device\n");
    delete c;
    return SIM_EDEVICE;
  }
  c->n_cu = n_cu;
  // one persistent workgroup per CU for the large network (LDS-bound), a few
  // per CU for the small one
  const int per_cu = c->net == 0 ? 4 : 1;
  c->n_wg = (int32_t)std::min<int64_t>((K + MT - 1) / MT, (int64_t)n_cu * per_cu);
  c->n_wg_max = c->n_wg;
  // the small network's FP32 step runs one wavefront per sub-trace when
  // there are few (a step's latency bounds such runs)
  if (c->net == 0 && cfg->prec == SIM_FP32 && K <= WAVE_MAX_SUB) c->variant = QUAD_VARIANT;
  const int32_t n_slots = c->n_wg * MT;

  // one device block: table + state + results + counters + total
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += (bytes + 255) / 256 * 256;
    return at;
  };
  const size_t o_first = take(8 * K), o_npos = take(8 * K), o_warm = take(4 * K),
               o_poff = take(8 * K), o_cur = take(8 * K), o_tw = take(8 * K),
               o_rp = take(8 * K), o_pos = take(8 * K), o_head = take(4 * K),
               o_cnt = take(4 * K), o_rw = take(8 * (size_t)K * WMAX),
               o_qi = take(4 * (size_t)K * C), o_qe = take(4 * (size_t)K * C),
               o_qt = take(8 * (size_t)K * C), o_qr = take(8 * (size_t)K * C),
               o_fe = take(8 * K), o_dr = take(8 * K), o_fi = take(8 * K), o_wt = take(8 * K),
               o_ctr = take(8 * NCOUNTERS), o_tot = take(8), o_order = take(4 * K),
               o_slot = take(4 * (size_t)n_slots), o_next = take(4);
  const bool mwq = cfg->n_out == 3;
  const size_t KC = mwq ? (size_t)K * C : 0, KM = mwq ? (size_t)K : 0;
  const size_t o_mi = take(4 * KC), o_mes = take(4 * KC), o_mt = take(8 * KC), o_mr = take(8 * KC),
               o_mx = take(8 * KC), o_mh = take(4 * KM), o_mc = take(4 * KM), o_mq = take(4 * KM),
               o_xp = take(8 * KM);
  // the split step's buffers behind it (without them, if they do not fit,
  // every tile runs on one workgroup)
  const bool split = c->net != 0;
  hipError_t e = hipMalloc(&c->dev_block, split ? split_layout(c, nullptr, off, nullptr) : off);
  if (e == hipSuccess && split) {
    split_layout(c, static_cast<char*>(c->dev_block), off, &c->split);
  } else if (e != hipSuccess && split) {
    (void)hipGetLastError();
    e = hipMalloc(&c->dev_block, off);
  }
  if (e != hipSuccess) {
    fprintf(stderr, "sim_init: hipMalloc(%zu): %s\n", off, hipGetErrorString(e));
    if (c->feat16) (void)hipFree(c->feat16);
    delete c;
    return e == hipErrorOutOfMemory ? SIM_ENOMEM : SIM_EDEVICE;
  }
  char* base = static_cast<char*>(c->dev_block);
  DevState& s = c->st;
  s.first = reinterpret_cast<int64_t*>(base + o_first);
  s.n_pos = reinterpret_cast<int64_t*>(base + o_npos);
  s.warm = reinterpret_cast<int32_t*>(base + o_warm);
  s.pred_off = reinterpret_cast<int64_t*>(base + o_poff);
  s.cur = reinterpret_cast<int64_t*>(base + o_cur);
  s.t_w = reinterpret_cast<int64_t*>(base + o_tw);
  s.r_prev = reinterpret_cast<int64_t*>(base + o_rp);
  s.pos = reinterpret_cast<int64_t*>(base + o_pos);
  s.head = reinterpret_cast<int32_t*>(base + o_head);
  s.count = reinterpret_cast<int32_t*>(base + o_cnt);
  s.rw = reinterpret_cast<int64_t*>(base + o_rw);
  s.q_idx = reinterpret_cast<int32_t*>(base + o_qi);
  s.q_e = reinterpret_cast<int32_t*>(base + o_qe);
  s.q_t = reinterpret_cast<int64_t*>(base + o_qt);
  s.q_r = reinterpret_cast<int64_t*>(base + o_qr);
  s.fetch = reinterpret_cast<int64_t*>(base + o_fe);
  s.drain = reinterpret_cast<int64_t*>(base + o_dr);
  s.final_tick = reinterpret_cast<int64_t*>(base + o_fi);
  s.warm_tick = reinterpret_cast<int64_t*>(base + o_wt);
  s.counters = reinterpret_cast<unsigned long long*>(base + o_ctr);
  c->dev_total = reinterpret_cast<int64_t*>(base + o_tot);
  s.order = reinterpret_cast<int32_t*>(base + o_order);
  s.slot_kid = reinterpret_cast<int32_t*>(base + o_slot);
  s.next = reinterpret_cast<unsigned*>(base + o_next);
  if (mwq) {
    s.m_idx = reinterpret_cast<int32_t*>(base + o_mi);
    s.m_es = reinterpret_cast<int32_t*>(base + o_mes);
    s.m_t = reinterpret_cast<int64_t*>(base + o_mt);
    s.m_r = reinterpret_cast<int64_t*>(base + o_mr);
    s.m_x = reinterpret_cast<int64_t*>(base + o_mx);
    s.m_head = reinterpret_cast<int32_t*>(base + o_mh);
    s.m_count = reinterpret_cast<int32_t*>(base + o_mc);
    s.m_inpq = reinterpret_cast<int32_t*>(base + o_mq);
    s.x_prev = reinterpret_cast<int64_t*>(base + o_xp);
  }

  c->results.resize(o_tot + 8 - (K <= ONE_COPY_MAX_SUB ? o_fe : o_ctr));
  hipError_t e1 = hipMemcpyAsync(base + o_first, first.data(), 8 * K, hipMemcpyHostToDevice, c->stream);
  hipError_t e2 = hipMemcpyAsync(base + o_npos, npos.data(), 8 * K, hipMemcpyHostToDevice, c->stream);
  hipError_t e3 = hipMemcpyAsync(base + o_warm, warm.data(), 4 * K, hipMemcpyHostToDevice, c->stream);
  hipError_t e4 = hipMemcpyAsync(base + o_poff, poff.data(), 8 * K, hipMemcpyHostToDevice, c->stream);
  hipError_t e7 = hipMemcpyAsync(base + o_order, order.data(), 4 * K, hipMemcpyHostToDevice, c->stream);
  hipError_t e5 = launch_reset(s, K, 0, n_slots, c->stream);
  hipError_t e6 = hipStreamSynchronize(c->stream);  // host vectors die at return
  for (hipError_t x : {e1, e2, e3, e4, e7, e5, e6})
    if (x != hipSuccess) {
      fprintf(stderr, "sim_init: %s\n", hipGetErrorString(x));
      (void)hipFree(c->dev_block);
      if (c->feat16) (void)hipFree(c->feat16);
      delete c;
      return SIM_EDEVICE;
    }
  *out = c;
  return SIM_OK;
}

int sim_load_weights(sim_ctx* c, const sim_layer* layers, int32_t n_layers, const float* params,
                     int32_t on_device) {
  if (!c) return SIM_EINVAL;
  if (!layers || n_layers < 1 || !params) return fail(c, SIM_EINVAL, "null layers or params");
  if (c->net != 0 && train_layers_match(layers, n_layers)) {
    if (c->cfg.prec == SIM_FP8E4M3) return fail(c, SIM_EUNSUPPORTED, "no FP8 training form");
    c->net = 2;
    return load_train_weights(c, layers, n_layers, params, on_device);
  }
  if (c->net == 4) {  // store latencies: the trunk with three outputs only
    if (!layers_match<NetC3S>(layers, n_layers))
      return fail(c, SIM_EUNSUPPORTED, "with n_out = 3 the layer list must end in FC 512 -> 3");
    if (c->cfg.prec == SIM_FP8E4M3)
      return fail(c, SIM_EUNSUPPORTED, "no FP8 form with store latencies");
  }
  if (c->net == 2 || c->net == 3 || c->net == 5) c->net = 1;
  if (c->net == 1 && layers_match<NetRB7>(layers, n_layers)) {
    if (c->cfg.prec == SIM_FP8E4M3) return fail(c, SIM_EUNSUPPORTED, "no FP8 form of RB7");
    if (c->cfg.col_dep >= 0)
      return fail(c, SIM_EUNSUPPORTED, "dependency flags need the C3 regression network");
    c->net = 5;
  }
  if (c->net == 1 && layers_match<NetC3Hyb>(layers, n_layers)) {
    if (c->cfg.prec == SIM_FP8E4M3)
      return fail(c, SIM_EUNSUPPORTED, "no FP8 form of the hybrid head");
    c->net = 3;
  }
  const bool ok = c->net == 0   ? layers_match<NetSmall>(layers, n_layers)
                  : c->net >= 3 ? true
                                : layers_match<NetC3>(layers, n_layers);
  if (!ok) return fail(c, SIM_EUNSUPPORTED, "no kernel for this layer list");
  if (layers[n_layers - 1].relu)
    return fail(c, SIM_EUNSUPPORTED, "the output layer must not have ReLU");
  const size_t np = c->net == 0   ? param_count<NetSmall>()
                    : c->net == 3 ? param_count<NetC3Hyb>()
                    : c->net == 5 ? param_count<NetRB7>()
                    : c->net == 4 ? param_count<NetC3S>()
                                  : param_count<NetC3>();
  std::vector<float> host(np);
  if (on_device) {
    hipError_t e = hipMemcpy(host.data(), params, np * 4, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(c, e, "copy params to host");
  } else {
    memcpy(host.data(), params, np * 4);
  }
  for (size_t i = 0; i < np; ++i)
    if (!isfinite(host[i])) return fail(c, SIM_ENONFINITE, "parameter %zu is not finite", i);
  uint32_t relu = 0;
  for (int32_t i = 0; i < n_layers; ++i)
    if (layers[i].relu) relu |= 1u << i;
  c->relu = relu;
  if (c->cfg.prec == SIM_FP8E4M3) {
    // FP8 needs activation scales: keep the parameters, build FP32 weights
    // for the calibration pass; the FP8 weights are built by sim_calibrate.
    c->params = host;
    c->calibrated = false;
    int rc = upload_weights(c, SIM_FP32, host.data(), nullptr, &c->dev_w32, &c->w32);
    if (rc != SIM_OK) return rc;
    c->weights = true;
    return sim_reset(c);
  }
  int rc = upload_weights(c, c->cfg.prec, host.data(), nullptr, &c->dev_weights, &c->w);
  if (rc != SIM_OK) return rc;
  if (c->net == 5 && c->has_trace && !c->rb_trunk) {
    const int64_t slots = (int64_t)c->n_wg_max * MT;
    const size_t es = elem_size(c->cfg.prec);
    hipError_t e = hipMalloc(&c->rb_trunk, (size_t)slots * NetRB7::NB * NetRB7::CH3 * es);
    if (e == hipSuccess) e = hipMalloc(&c->rb_active, sizeof(int32_t) * slots);
    if (e == hipSuccess) e = hipMalloc(&c->rb_logits, sizeof(float) * slots * NetRB7::NOUT);
    if (e != hipSuccess) return hip_fail(c, e, "hipMalloc RB7 step buffers");
  }
  if (!c->has_trace && c->net != 0 && !c->split.part[0]) {  // the split forward's sums
    if (hipMalloc(&c->dev_block, split_layout(c, nullptr, 0, nullptr)) == hipSuccess) {
      split_layout(c, static_cast<char*>(c->dev_block), 0, &c->split);
    } else {
      (void)hipGetLastError();
      c->dev_block = nullptr;
    }
  }
  c->weights = true;
  return sim_reset(c);
}

int sim_reset(sim_ctx* c) {
  if (!c) return SIM_EINVAL;
  if (!c->has_trace) return SIM_OK;
  c->reset_captured = c->reset_captured || capturing(c->stream);
  // Where sub-traces outnumber the persistent kernel's slots, its workgroups
  // claim them longest first as they arrive, and arrive in a better order right
  // behind a kernel that fills the chip than on an idle one: the rings are
  // cleared, which lasts until the run arrives.  20,000 uneven C3 sub-traces,
  // BF16: 199.7 to 200.1 ms a run without, 197.6 to 197.9 with; 4,096 (a slot
  // each) 27.53 either way.  Fewer run split and the small network in tiles of
  // its own: these only pay for it (64 sub-traces 4.73 -> 4.76 ms).
  const bool clear =
      c->net != 0 && c->net != 5 && c->n_sub > (int64_t)c->n_wg_max * MT;
  hipError_t e =
      launch_reset(c->st, c->n_sub, clear ? c->C : 0, c->n_wg_max * MT, c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "reset");
  c->completed = false;
  c->ran_to_end = false;
  c->steps_done = 0;
  return SIM_OK;
}

int sim_calibrate(sim_ctx* c, int32_t n_steps, int32_t mode, const int32_t* table) {
  if (!c) return SIM_EINVAL;
  if (!c->has_trace) return fail(c, SIM_ESTATE, "context has no trace");
  if (c->net == 2) return fail(c, SIM_EUNSUPPORTED, "no FP8 training form");
  if (c->net >= 3) return fail(c, SIM_EUNSUPPORTED, "no FP8 form of this network");
  if (!c->weights) return fail(c, SIM_ESTATE, "weights not loaded");
  if (c->cfg.prec == SIM_BF16) return fail(c, SIM_EUNSUPPORTED, "calibration runs FP32 weights");
  if (n_steps < 1) return fail(c, SIM_EINVAL, "n_steps < 1");
  if (mode < SIM_LAT_PREDICT || mode > SIM_LAT_SHADOW) return fail(c, SIM_EINVAL, "bad lat_mode");
  if (mode != SIM_LAT_PREDICT && !table) return fail(c, SIM_EINVAL, "lat_table required");
  const DevWeights& w32 = c->cfg.prec == SIM_FP8E4M3 ? c->w32 : c->w;
  const int n = calibration_size(c->net);
  unsigned* amax = nullptr;
  hipError_t e = hipMalloc(&amax, sizeof(unsigned) * n);
  if (e != hipSuccess) return hip_fail(c, e, "hipMalloc calibration");
  int rc = sim_reset(c);
  std::vector<unsigned> host(n, 0u);
  if (rc == SIM_OK) {
    e = hipMemsetAsync(amax, 0, sizeof(unsigned) * n, c->stream);
    StepParams p{};
    p.feat = c->feat;
    p.codes = c->codes;
    p.mem = c->mem;
    p.col_dep = c->cfg.col_dep;
    p.n_wg = c->n_wg;
    p.n_sub = c->n_sub;
    p.W = c->cfg.retire_width;
    p.col_res = c->cfg.col_res;
    p.col_exe = c->cfg.col_exe;
    p.col_sto = c->cfg.col_sto;
    p.lat_max = c->cfg.lat_max;
    p.lat_mode = mode;
    p.lat_table = table;
    p.logits_out = nullptr;
    p.n_steps = n_steps;
    p.cal_out = amax;
    if (e == hipSuccess) e = launch_calibrate(c->net, w32, c->relu, c->st, p, c->stream);
    if (e == hipSuccess)
      e = hipMemcpyAsync(host.data(), amax, sizeof(unsigned) * n, hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) rc = hip_fail(c, e, "calibration run");
  }
  (void)hipFree(amax);
  if (rc != SIM_OK) return rc;
  // power-of-two scale per layer-input channel (window features first)
  c->act_scale.assign(n, 1.f);
  for (int i = 0; i < n; ++i) {
    float a;
    memcpy(&a, &host[i], 4);
    c->act_scale[i] = pow2_scale(a);
  }
  if (c->cfg.prec == SIM_FP8E4M3) {
    std::vector<int> sizes = c->net == 0 ? std::vector<int>{NetSmall::D, NetSmall::CH1, NetSmall::CH2}
                                         : std::vector<int>{NetC3::D, NetC3::CH1, NetC3::CH2,
                                                            NetC3::CH3, NetC3::HID};
    std::vector<std::vector<float>> per_layer;
    size_t off = 0;
    for (int sz : sizes) {
      per_layer.emplace_back(c->act_scale.begin() + off, c->act_scale.begin() + off + sz);
      off += sz;
    }
    rc = upload_weights(c, SIM_FP8E4M3, c->params.data(), &per_layer, &c->dev_weights, &c->w);
    if (rc != SIM_OK) return rc;
  }
  c->calibrated = true;
  return sim_reset(c);
}

int sim_set_graph(sim_ctx* c, int32_t enable) {
  if (!c) return SIM_EINVAL;
  c->use_graph = enable != 0;
  if (!c->use_graph) drop_graph(c);
  return SIM_OK;
}

int sim_act_scales(const sim_ctx* c, float* out, int32_t n) {
  if (!c || !out) return SIM_EINVAL;
  if (!c->calibrated) return SIM_ESTATE;
  if (n < (int32_t)c->act_scale.size()) return SIM_EINVAL;
  memcpy(out, c->act_scale.data(), sizeof(float) * c->act_scale.size());
  return SIM_OK;
}

int sim_record_logits(sim_ctx* c, float* logits) {
  if (!c) return SIM_EINVAL;
  c->logits_out = logits;
  return SIM_OK;
}

static StepParams step_params(const sim_ctx* c, int64_t n_steps, int32_t mode,
                              const int32_t* table) {
  StepParams p{};
  p.feat = c->feat;
  p.feat16 = c->feat16;
  p.codes = c->codes;
  p.mem = c->mem;
  p.col_dep = c->cfg.col_dep;
  p.n_wg = c->n_wg;
  p.n_sub = c->n_sub;
  p.W = c->cfg.retire_width;
  p.col_res = c->cfg.col_res;
  p.col_exe = c->cfg.col_exe;
  p.col_sto = c->cfg.col_sto;
  p.store_col = c->cfg.n_out == 3 ? c->cfg.store_col : 0;
  p.lat_max = c->cfg.lat_max;
  p.lat_mode = mode;
  p.lat_table = table;
  p.logits_out = c->logits_out;
  p.n_steps = (int32_t)std::min<int64_t>(n_steps, INT32_MAX);
  p.cal_out = nullptr;
  p.trunk_out = c->rb_trunk;
  p.active_out = c->rb_active;
  p.ext_logits = c->rb_logits;
  return p;
}

// RB7: one step = gather and convolutions (stage 1), the residual blocks
// over every slot's 13 positions, FC 512 and the head, then the update
// (stage 2).  Slots with nothing left to simulate are skipped by every part.
static hipError_t rb_step(sim_ctx* c, int32_t mode, const int32_t* table) {
  StepParams p = step_params(c, 1, mode, table);
  const int64_t slots = (int64_t)p.n_wg * MT;
  hipError_t e = launch_rb_stage(c->cfg.prec, 1, c->w, c->relu, c->st, p, c->stream);
  if (e == hipSuccess)
    e = launch_resblocks(c->cfg.prec, c->w, c->relu, c->rb_trunk, slots * NetRB7::NB,
                         c->rb_active, c->n_cu, c->stream);
  if (e == hipSuccess)
    e = launch_rb_head(c->cfg.prec, c->w, c->relu, c->rb_trunk, slots, c->rb_active,
                       c->rb_logits, c->stream);
  if (e == hipSuccess) e = launch_rb_stage(c->cfg.prec, 2, c->w, c->relu, c->st, p, c->stream);
  return e;
}

// RB7 steps; n_steps = INT32_MAX runs until every position has been
// advanced (checked on the host every RB_CHECK steps).
constexpr int RB_CHECK = 16;
static int rb_launch(sim_ctx* c, int64_t n_steps, int32_t mode, const int32_t* table) {
  const bool to_end = n_steps >= INT32_MAX;
  for (int64_t done = 0; to_end || done < n_steps;) {
    const int64_t chunk = to_end ? RB_CHECK : std::min<int64_t>(RB_CHECK, n_steps - done);
    for (int64_t i = 0; i < chunk; ++i) {
      hipError_t e = rb_step(c, mode, table);
      if (e != hipSuccess) return hip_fail(c, e, "RB7 step launch");
    }
    done += chunk;
    if (!to_end) continue;
    unsigned long long adv = 0;
    hipError_t e = hipMemcpyAsync(&adv, c->st.counters + 3, sizeof adv, hipMemcpyDeviceToHost,
                                  c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return hip_fail(c, e, "RB7 progress");
    if ((int64_t)adv >= c->n_pred) break;
    if (done > c->n_pred + RB_CHECK)  // every step advances at least one position
      return fail(c, SIM_EDEVICE, "RB7 run did not finish");
  }
  return SIM_OK;
}

// n_steps steps of every sub-trace launched.
static void count_steps(sim_ctx* c, int64_t n_steps) {
  if (!c->reset_captured) c->steps_done = std::min(c->max_pos, c->steps_done + n_steps);
}

// Whether a call of n_steps steps in this many tiles is split over several
// workgroups per tile: a C3 network running its predictor, every sub-trace in a
// slot of its own (so that `steps` launches are known to end the run), and not
// under capture (a graph takes the persistent kernel's one node).  Nor a short
// call on many tiles: the state's way in and out and the last head and update
// cost a call ~33 us, and with two units per tile (86 to 128 tiles) a BF16 or FP8
// step gains less than that (us a call, one workgroup per tile -> split, 2,048
// sub-traces: C3 BF16 1 step 64 -> 75, 2 steps 115 -> 116, 4 216 -> 197; hybrid 1
// 64 -> 65, 2 116 -> 106; store latencies 80 -> 84, 139 -> 129).  With three units
// (1,360 sub-traces) one step 63 -> 58, in FP32 (2,048) 232 -> 168, RB7 462 -> 451.
static bool split_step(const sim_ctx* c, int64_t n_steps, int32_t mode, int32_t n_wg) {
  if (!((c->net == 1 || c->net >= 3) && mode != SIM_LAT_INJECT && c->split.cst &&
        (int64_t)n_wg * MT >= c->n_sub && !capturing(c->stream)))
    return false;
  const int32_t units = split_shape(c, n_wg).units;
  n_steps = std::min(n_steps, c->max_pos - c->steps_done);  // (a run's)
  const bool brief = units == 2 && c->cfg.prec != SIM_FP32 && c->net != 5 &&
                     n_steps < (c->net == 1 ? 3 : 2);
  return units >= 2 && !brief;
}

// n_steps split steps (to the end at most): launch i finishes step i - 1 and
// begins step i.  Slots run the sub-traces longest first, so tiles end from
// the last; an ended tile stays for one launch that copies its final scalars
// to the buffer the next launches read.
static hipError_t split_steps(sim_ctx* c, int64_t n_steps, int32_t mode, const int32_t* table) {
  const int64_t n = std::min(n_steps, c->max_pos - c->steps_done);
  if (n <= 0) return hipSuccess;
  const StepParams p = step_params(c, 1, mode, table);
  const int all = (int)c->tile_len.size();
  hipError_t e = launch_split_import(c->st, c->split, all, c->n_sub, c->C, c->cfg.retire_width,
                                     c->stream);
  int tiles = all, in = 0;
  for (int64_t i = 0; i <= n && e == hipSuccess; ++i) {
    while (tiles > 1 && c->tile_len[tiles - 1] + 1 < c->steps_done + i) --tiles;
    e = launch_split_step(c->net, c->cfg.prec, c->w, c->relu, c->st, p, c->split,
                          split_shape(c, tiles), tiles, in, i > 0, i < n, c->stream);
    if (i > 0) in ^= 1;
    if (c->net == 5 && i < n && e == hipSuccess) {  // the blocks, then FC 512's sums
      const int64_t win = std::min<int64_t>((int64_t)tiles * MT, c->n_sub);
      e = launch_resblocks(c->cfg.prec, c->w, c->relu, c->rb_trunk, win * NetRB7::NB,
                           c->rb_active, c->n_cu, c->stream);
      if (e == hipSuccess)
        e = launch_split_fc(c->cfg.prec, c->w, c->rb_trunk, win, c->rb_active, c->split.part[0],
                            split_shape(c, tiles), c->stream);
    }
  }
  if (e == hipSuccess)
    e = launch_split_export(c->st, c->split, all, in, c->C, c->cfg.retire_width, c->stream);
  return e;
}

static int step_launch(sim_ctx* c, int64_t n_steps, int32_t mode, const int32_t* table) {
  if (!c->has_trace) return fail(c, SIM_ESTATE, "context has no trace");
  if (c->cfg.col_dep >= 0 && c->net != 1 && mode != SIM_LAT_INJECT)
    return fail(c, SIM_EUNSUPPORTED, "dependency flags need the C3 regression network");
  if (c->net == 2) return fail(c, SIM_EUNSUPPORTED, "the training head does not drive the simulation");
  if (mode < SIM_LAT_PREDICT || mode > SIM_LAT_SHADOW) return fail(c, SIM_EINVAL, "bad lat_mode");
  if (mode != SIM_LAT_PREDICT && !table) return fail(c, SIM_EINVAL, "lat_table required");
  if (mode != SIM_LAT_INJECT && !c->weights) return fail(c, SIM_ESTATE, "weights not loaded");
  if (mode != SIM_LAT_INJECT && c->cfg.prec == SIM_FP8E4M3 && !c->calibrated)
    return fail(c, SIM_ESTATE, "FP8 form needs sim_calibrate first");
  if (c->completed) return fail(c, SIM_ESTATE, "run completed; call sim_reset");
  if (c->ran_to_end) return SIM_OK;  // every sub-trace has already finished
  if (n_steps == 0) return SIM_OK;   // checks only
  if (n_steps >= INT32_MAX) c->ran_to_end = true;
  if (split_step(c, n_steps, mode, c->n_wg)) {
    const hipError_t e = split_steps(c, n_steps, mode, table);
    if (e != hipSuccess) return hip_fail(c, e, "split step launch");
    count_steps(c, n_steps);
    return SIM_OK;
  }
  if (c->net == 5 && mode != SIM_LAT_INJECT) return rb_launch(c, n_steps, mode, table);
  const StepParams p = step_params(c, n_steps, mode, table);
  // (injected latencies need no predictor: RB7 shares the hybrid head's step)
  hipError_t e = launch_step(c->net == 5 ? 3 : c->net, c->cfg.prec, c->variant, c->w, c->relu,
                             c->st, p, c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "step launch");
  // (launches under capture may never run, and slots that refill lag)
  if ((int64_t)c->n_wg * MT >= c->n_sub && !capturing(c->stream)) count_steps(c, n_steps);
  return SIM_OK;
}

int sim_step(sim_ctx* c, int32_t n_steps, int32_t mode, const int32_t* table) {
  if (!c) return SIM_EINVAL;
  if (n_steps < 0) return fail(c, SIM_EINVAL, "n_steps < 0");
  if (n_steps == 0) return SIM_OK;
  return step_launch(c, n_steps, mode, table);
}

int sim_run(sim_ctx* c, int32_t mode, const int32_t* table, sim_result* res) {
  if (!c) return SIM_EINVAL;
  if (!res) return fail(c, SIM_EINVAL, "null result");
  hipError_t e = hipSuccess;
  // (RB7 and split steps run eagerly)
  if (c->use_graph && !c->ran_to_end && c->net != 5 && !split_step(c, INT32_MAX, mode, c->n_wg)) {
    // same checks as a step launch, then replay (rebuilt when its inputs change)
    int rc = step_launch(c, 0, mode, table);
    if (rc != SIM_OK) return rc;
    if (!c->graph_exec || c->graph_mode != mode || c->graph_table != table ||
        c->graph_logits != c->logits_out) {
      drop_graph(c);
      hipGraph_t g = nullptr;
      e = build_run_graph(c->net, c->cfg.prec, c->variant, c->w, c->relu, c->st,
                          step_params(c, INT32_MAX, mode, table), c->dev_total, &g);
      if (e == hipSuccess) e = hipGraphInstantiate(&c->graph_exec, g, nullptr, nullptr, 0);
      if (g) (void)hipGraphDestroy(g);
      if (e != hipSuccess) return hip_fail(c, e, "build run graph");
      c->graph_mode = mode;
      c->graph_table = table;
      c->graph_logits = c->logits_out;
    }
    e = hipGraphLaunch(c->graph_exec, c->stream);
    if (e != hipSuccess) return hip_fail(c, e, "graph launch");
    c->ran_to_end = true;
  } else {
    int rc = step_launch(c, INT32_MAX, mode, table);
    if (rc != SIM_OK) return rc;
    e = launch_total(c->st, c->n_sub, c->dev_total, c->stream);
    if (e != hipSuccess) return hip_fail(c, e, "total launch");
  }
  // The results lie one after another (fetch, drain, final and warm ticks,
  // counters, total).  Few sub-traces: one copy to the host from the first that
  // is asked for, its pieces to the caller's arrays; many: the counters and the
  // total, and each array straight to its place.
  const struct {
    int64_t* to;
    const int64_t* from;
  } arrays[] = {{res->fetch_cycles, c->st.fetch},
                {res->drain_cycles, c->st.drain},
                {res->final_tick, c->st.final_tick},
                {res->warm_tick, c->st.warm_tick}};
  const bool few = c->n_sub <= ONE_COPY_MAX_SUB;
  const size_t kb = 8 * (size_t)c->n_sub;
  const char* from = reinterpret_cast<const char*>(c->st.counters);
  const char* const end = reinterpret_cast<const char*>(c->dev_total) + 8;
  e = hipSuccess;
  for (const auto& a : arrays) {
    if (few && a.to) from = std::min(from, reinterpret_cast<const char*>(a.from));
    if (!few && a.to && e == hipSuccess)
      e = hipMemcpyAsync(a.to, a.from, kb, hipMemcpyDeviceToHost, c->stream);
  }
  if (e == hipSuccess)
    e = hipMemcpyAsync(c->results.data(), from, end - from, hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "sim_run results");
  auto host = [&](const void* dev) {
    return c->results.data() + (static_cast<const char*>(dev) - from);
  };
  for (const auto& a : arrays)
    if (few && a.to) memcpy(a.to, host(a.from), kb);
  unsigned long long ctr[NCOUNTERS];
  memcpy(ctr, host(c->st.counters), sizeof ctr);
  memcpy(&res->total_cycles, host(c->dev_total), 8);
  res->measured_instr = c->n_meas;
  res->predicted_instr = c->n_pred;
  res->n_clamped = (int64_t)ctr[0];
  res->n_nonfinite = (int64_t)ctr[1];
  res->n_shadow_mismatch = (int64_t)ctr[2];
  c->completed = true;
  return SIM_OK;
}

// At least n windows' last-conv outputs in c->rb_ws, kept for later calls.
static hipError_t trunk_workspace(sim_ctx* c, int64_t n) {
  if (n <= c->rb_ws_B) return hipSuccess;
  if (c->rb_ws) {
    (void)hipStreamSynchronize(c->stream);
    (void)hipFree(c->rb_ws);
    c->rb_ws = nullptr;
    c->rb_ws_B = 0;
  }
  const size_t per = NetC3::NB * NetC3::CH3 * elem_size(c->cfg.prec);
  hipError_t e = hipMalloc(&c->rb_ws, (size_t)n * per);
  if (e == hipSuccess) c->rb_ws_B = n;
  return e;
}

int predictor_fwd(sim_ctx* c, const void* x, int64_t B, float* logits, void* save_or_null) {
  if (!c) return SIM_EINVAL;
  if (!c->weights) return fail(c, SIM_ESTATE, "weights not loaded");
  if (c->cfg.prec == SIM_FP8E4M3 && !c->calibrated)
    return fail(c, SIM_ESTATE, "FP8 form needs sim_calibrate first");
  if (B < 0 || (B > 0 && (!x || !logits))) return fail(c, SIM_EINVAL, "bad batch arguments");
  if (B == 0) return SIM_OK;
  if ((B + MT - 1) / MT > INT32_MAX) return fail(c, SIM_EINVAL, "batch too large");
  // A captured call may be replayed on any stream, beside other replays and
  // the context's own work, so under capture nothing of the context's memory
  // is written where the network needs none (RB7 does): one workgroup per tile.
  const bool captured = capturing(c->stream);
  auto shape = [&](int64_t n) {
    return captured || c->net == 0 ? SplitShape{1, 1, 0} : split_shape(c, (n + MT - 1) / MT);
  };
  if (c->net == 2) {
    if (!save_or_null) return fail(c, SIM_EINVAL, "the training form needs a save buffer");
    const SaveBlock sb = save_block(c, save_or_null, B);
    const SplitShape sh = shape(B);
    hipError_t e =
        sh.units >= 2 ? launch_split_forward(2, c->cfg.prec, c->w, c->relu,
                                             static_cast<const float*>(x), B, nullptr, sb,
                                             c->split.part[0], sh, c->stream)
                      : launch_forward_save(c->cfg.prec, c->w, c->relu,
                                            static_cast<const float*>(x), B, sb, c->stream);
    TrainState& T = c->tr;
    const int bf = c->cfg.prec == SIM_BF16;
    GemmArgs g = gemm(opnd(sb.h, bf, 512, 1), opnd(T.perm + T.perm_off[4], bf, 1, 512),
                      logits, TRAIN_OUT, B, TRAIN_OUT, 512, 0);
    g.bias = T.master + T.boff[4];
    if (e == hipSuccess) e = launch_gemm(g, bf, nullptr, 0, c->stream);
    if (e != hipSuccess) return hip_fail(c, e, "training forward");
    return SIM_OK;
  }
  if (save_or_null) return fail(c, SIM_EUNSUPPORTED, "save buffer not supported");
  if (c->net == 5) {  // convolutions, residual blocks, FC 512 and head over a workspace
    if (B > INT64_MAX / (NetRB7::NB * NetRB7::CH3 * 4)) return fail(c, SIM_EINVAL, "batch too large");
    if (hipError_t e = trunk_workspace(c, B); e != hipSuccess)
      return hip_fail(c, e, "hipMalloc RB7 workspace");
    const SplitShape sh = shape(B);
    const bool split = sh.units >= 2;
    hipError_t e = split ? launch_split_trunk(c->cfg.prec, c->w, c->relu,
                                              static_cast<const float*>(x), B, c->rb_ws, sh,
                                              c->stream)
                         : launch_rb_trunk(c->cfg.prec, c->w, c->relu,
                                           static_cast<const float*>(x), B, c->rb_ws, c->stream);
    if (e == hipSuccess)
      e = launch_resblocks(c->cfg.prec, c->w, c->relu, c->rb_ws, B * NetRB7::NB, nullptr, c->n_cu,
                           c->stream);
    if (e == hipSuccess && split) {
      e = launch_split_fc(c->cfg.prec, c->w, c->rb_ws, B, nullptr, c->split.part[0], sh, c->stream);
      if (e == hipSuccess)
        e = launch_split_rb_head(c->cfg.prec, c->w, c->relu, c->split.part[0], B, logits, c->stream);
    } else if (e == hipSuccess) {
      e = launch_rb_head(c->cfg.prec, c->w, c->relu, c->rb_ws, B, nullptr, logits, c->stream);
    }
    if (e != hipSuccess) return hip_fail(c, e, "RB7 forward");
    return SIM_OK;
  }
  // n windows: few split over several workgroups per tile (split_shape), at
  // most one round of workgroups in one kernel, more through rows (BF16,
  // FWD_ROUNDS rounds at a time, in memory of one size; without it, or under
  // capture, in one kernel too).  The first such call has no memory yet: it
  // takes the one kernel and allocates behind it.
  const int64_t round = (int64_t)MT * c->n_cu, most = FWD_ROUNDS * round;
  // (a predictor-only context may not know its device's CUs: one kernel then)
  const bool many = (c->net == 1 || c->net == 3) && c->cfg.prec == SIM_BF16 && round > 0 &&
                    B > round && !captured;
  const bool rows = many && most <= c->rb_ws_B;
  // a few windows beyond whole rounds cost less split than as one more round
  // (us, 4,100 windows: 102 in one piece, 82 as 4,096 and 4; 8,200: 141, 134)
  const int64_t over = rows ? B % round : 0, rest = over <= round / 8 ? over : 0;
  const int64_t whole = rows ? B - rest : 0;
  hipError_t e = hipSuccess;
  for (int64_t at = 0, n; at < B && e == hipSuccess; at += n) {
    n = at < whole ? std::min(whole - at, most) : B - at;
    const float* xs = static_cast<const float*>(x) + at * c->cfg.n_slot * c->cfg.n_feat;
    float* out = logits + at * n_outputs(c->net);
    const SplitShape sh = shape(n);
    e = sh.units >= 2 ? launch_split_forward(c->net, c->cfg.prec, c->w, c->relu, xs, n, out,
                                             SaveBlock{}, c->split.part[0], sh, c->stream)
        : rows && n > round
            ? launch_forward_rows(c->net, c->w, c->relu, xs, n, static_cast<uint16_t*>(c->rb_ws),
                                  out, c->n_cu, c->stream)
            : launch_forward(c->net, c->cfg.prec, c->w, c->relu, xs, n, out, c->stream);
  }
  if (e != hipSuccess) return hip_fail(c, e, "forward launch");
  if (many && !rows && trunk_workspace(c, most) != hipSuccess) (void)hipGetLastError();
  return SIM_OK;
}

int sim_set_tuning(sim_ctx* c, int32_t variant, int32_t n_wg) {
  if (!c) return SIM_EINVAL;
  if (!c->has_trace) return fail(c, SIM_ESTATE, "context has no trace");
  if (variant < 0 || variant >= N_VARIANTS) return fail(c, SIM_EINVAL, "unknown variant");
  if (variant != 0 && c->cfg.col_dep >= 0)
    return fail(c, SIM_EUNSUPPORTED, "with dependency flags only variant 0 exists");
  if (n_wg < 1 || n_wg > c->n_wg_max) return fail(c, SIM_EINVAL, "n_wg out of range");
  drop_graph(c);
  c->variant = variant;
  c->n_wg = n_wg;
  return sim_reset(c);
}

int sim_autotune(sim_ctx* c, int32_t n_steps, int32_t lat_mode, const int32_t* lat_table,
                 sim_tuning* out) {
  if (!c) return SIM_EINVAL;
  if (!c->has_trace) return fail(c, SIM_ESTATE, "context has no trace");
  if (n_steps < 1 || !out) return fail(c, SIM_EINVAL, "bad arguments");
  // candidates: every kernel variant (C3 with the predictor running) x
  // 4/4, 3/4 and 1/2 of the slots
  // (the small network's FP32 step: the workgroup tile or one wave per slot)
  const int nv = (c->net == 1 && lat_mode != SIM_LAT_INJECT && c->cfg.col_dep < 0) ? N_VARIANTS
                 : (c->net == 0 && c->cfg.prec == SIM_FP32)                       ? 3
                                                                                  : 1;
  std::vector<int32_t> shapes;
  for (int q : {4, 3, 2}) {
    const int32_t n = std::max<int32_t>(1, c->n_wg_max * q / 4);
    if (std::find(shapes.begin(), shapes.end(), n) == shapes.end()) shapes.push_back(n);
  }
  // kernels that need scratch memory (register spills) are tried only when
  // every candidate does
  bool skip[N_VARIANTS] = {};
  if (nv == N_VARIANTS) {
    size_t sc[N_VARIANTS];
    bool any_free = false;
    for (int v = 0; v < nv; ++v) {
      const hipError_t e = c3_step_scratch(c->cfg.prec, v, &sc[v]);
      if (e != hipSuccess) return hip_fail(c, e, "kernel attributes");
      any_free = any_free || sc[v] == 0;
    }
    for (int v = 0; v < nv; ++v) skip[v] = any_free && sc[v] > 0;
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  if (e != hipSuccess) return hip_fail(c, e, "events");
  *out = sim_tuning{};
  float best = -1.f;
  int rc = SIM_OK;
  auto trial = [&](int v, int32_t nw) {
    if ((rc = sim_set_tuning(c, v, nw)) != SIM_OK) return;
    // one untimed launch (first use of a kernel), then the timed one
    if ((rc = step_launch(c, n_steps, lat_mode, lat_table)) != SIM_OK) return;
    if ((rc = sim_reset(c)) != SIM_OK) return;
    float ms = 0.f;
    unsigned long long ctr[NCOUNTERS] = {0, 0, 0, 0};
    e = hipEventRecord(e0, c->stream);
    if (e == hipSuccess) rc = step_launch(c, n_steps, lat_mode, lat_table);
    if (e == hipSuccess && rc == SIM_OK) e = hipEventRecord(e1, c->stream);
    if (e == hipSuccess && rc == SIM_OK)
      e = hipMemcpyAsync(ctr, c->st.counters, sizeof ctr, hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess && rc == SIM_OK) e = hipStreamSynchronize(c->stream);
    if (e == hipSuccess && rc == SIM_OK) e = hipEventElapsedTime(&ms, e0, e1);
    if (e != hipSuccess) rc = hip_fail(c, e, "timing");
    if (rc != SIM_OK) return;
    // the objective is time per position advanced: fewer slots do less
    // work per step
    ms = ctr[3] ? ms * 1e6f / (float)ctr[3] : ms * 1e6f;
    if (out->n_tried < 16) {
      out->tried_variant[out->n_tried] = v;
      out->tried_n_wg[out->n_tried] = nw;
      out->tried_ms[out->n_tried] = ms;
      ++out->n_tried;
    }
    if (best < 0.f || ms < best) {
      best = ms;
      out->variant = v;
      out->n_wg = nw;
      out->ms = ms;
    }
  };
  // The split step is one kernel whatever the variant: it is timed once, last,
  // with the variant that was best in the other shapes, which steps that are
  // not split (under capture) then run.
  int first = 0;
  while (skip[first]) ++first;
  out->variant = first;
  for (int v = first; v < nv && rc == SIM_OK; ++v)
    for (int32_t nw : shapes)
      if (!skip[v] && rc == SIM_OK && !split_step(c, n_steps, lat_mode, nw)) trial(v, nw);
  for (int32_t nw : shapes)
    if (rc == SIM_OK && split_step(c, n_steps, lat_mode, nw)) trial(out->variant, nw);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != SIM_OK) return rc;
  return sim_set_tuning(c, out->variant, out->n_wg);
}

int sim_variant_scratch(sim_ctx* c, int32_t variant, int64_t* bytes) {
  if (!c || !bytes) return SIM_EINVAL;
  if (c->net != 1) return fail(c, SIM_EUNSUPPORTED, "scratch query: C3 step variants only");
  if (variant < 0 || variant >= N_VARIANTS) return fail(c, SIM_EINVAL, "variant out of range");
  size_t b = 0;
  const hipError_t e = c3_step_scratch(c->cfg.prec, variant, &b);
  if (e != hipSuccess) return hip_fail(c, e, "kernel attributes");
  *bytes = (int64_t)b;
  return SIM_OK;
}

int64_t predictor_save_bytes(const sim_ctx* c, int64_t B) {
  if (!c || c->net != 2 || B < 0) return -1;
  return B * save_bytes_per_window(c->cfg.prec);
}

int sim_loss(sim_ctx* c, const float* logits, const int32_t* labels, int64_t B, float* loss,
             float* dlogits) {
  if (!c) return SIM_EINVAL;
  if (c->net != 2) return fail(c, SIM_EUNSUPPORTED, "the loss needs the training head");
  if (B < 1 || !logits || !labels || !loss || !dlogits) return fail(c, SIM_EINVAL, "bad arguments");
  int rc = ensure_train_work(c, B);
  if (rc != SIM_OK) return rc;
  hipError_t e = launch_loss(logits, labels, B, TRAIN_BINS, c->tr.work, loss, dlogits, c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "loss");
  return SIM_OK;
}

int sim_loss_noalloc(sim_ctx* c, const float* logits, const int32_t* labels, int64_t B,
                     float* loss, float* dlogits) {
  if (!c) return SIM_EINVAL;
  if (c->net != 2) return fail(c, SIM_EUNSUPPORTED, "the loss needs the training head");
  if (B < 1 || !logits || !labels || !loss || !dlogits) return fail(c, SIM_EINVAL, "bad arguments");
  if (B > SIM_NOALLOC_MAX_B)
    return fail(c, SIM_EINVAL, "B = %lld exceeds the scratch's %d windows", (long long)B,
                SIM_NOALLOC_MAX_B);
  if (!c->scratch) return fail(c, SIM_ESTATE, "no device scratch");
  // the same kernels as sim_loss, the per-window losses in this device's
  // static scratch instead of the context's training workspace
  hipError_t e = launch_loss(logits, labels, B, TRAIN_BINS, c->scratch, loss, dlogits, c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "loss");
  return SIM_OK;
}

int predictor_bwd(sim_ctx* c, const void* x, const void* save, const float* dlogits, int64_t B,
                  float* dx, float* dparams, int32_t accumulate) {
  if (!c) return SIM_EINVAL;
  if (c->net != 2) return fail(c, SIM_EUNSUPPORTED, "the backward pass needs the training head");
  if (!c->weights) return fail(c, SIM_ESTATE, "weights not loaded");
  if (B < 1 || !x || !save || !dlogits || !dparams) return fail(c, SIM_EINVAL, "bad arguments");
  int rc = ensure_train_work(c, B);
  if (rc != SIM_OK) return rc;
  TrainState& T = c->tr;
  const int bf = c->cfg.prec == SIM_BF16;
  const int beta = accumulate ? 1 : 0;
  hipError_t e = hipSuccess;
  const SaveBlock sb = save_block(c, const_cast<void*>(aligned_save(c, save, B, &e)), B);
  if (e != hipSuccess) return hip_fail(c, e, "copy of the save buffer");
  float* W = T.work;
  float* dH = W + train_work_off(B, 1);
  float* dY3 = W + train_work_off(B, 2);
  float* dY2 = W + train_work_off(B, 3);
  float* dY1 = W + train_work_off(B, 4);
  float* csw_next = W + train_work_off(B, 5);
  float* part = W + train_work_off(B, 6);
  void* dZp = W + train_work_off(B, 7);
  // The input-gradient chain product by product, then all weight gradients
  // together (launch_gemm_group).
  hipStream_t s = c->stream;
  auto run = [&](const GemmArgs& g) {
    if (e == hipSuccess) e = launch_gemm(g, bf, part, (int64_t)SPLITK_CAP, s);
  };
  // the bias sums: lists of partials now (column-sum chunks or a weight
  // gradient's per-split row sums), all five added in one launch at the end
  GemmGroup grp{};
  SumSegs bias{};
  bias.beta = beta;
  auto sums = [&](int64_t parts, int64_t N, float* out) {
    bias.seg[bias.count++] = SumSeg{csw_next, parts, N, out, 0, 0};
    csw_next += (parts * N + 63) / 64 * 64;
  };
  // trunk layer l's weight gradient, [c_out][input column] with
  // input column t*c_in + c (p*256 + c for the hidden layer), stored
  // straight into the parameters' layout ([c_out][c_in][2], [512][256][13]);
  // its bias gradient the column sums of dy (y [rows][c_out]).  In the group
  // where it may join, the bias from the same product's row sums of dy^T (one
  // list of partials per k-split for the final sum), else (windows off an
  // 8-byte boundary, a save buffer that could not be copied) by itself, the bias
  // as a column sum.
  auto wgrad = [&](const GemmOperand& dyt, const GemmOperand& act, int l, int64_t c_out,
                   int64_t cols, int64_t c_in, int64_t taps, int64_t rows, const void* y) {
    GemmArgs g = gemm(dyt, act, dparams + T.woff[l], cols, c_out, cols, rows, beta);
    g.ccg = c_in;
    g.ccm = taps;
    g.rowsum = csw_next;
    if (groups(g, bf)) {
      grp.bias[grp.count] = bias.count;
      sums(GROUP_SPLITS, c_out, dparams + T.boff[l]);  // (the group sets the number)
      grp.g[grp.count++] = g;
      return;
    }
    int64_t parts = 0;
    run(g);
    if (e == hipSuccess)
      e = launch_colsum_partial(y, bf, rows, c_out, c_out, csw_next, &parts, s);
    if (e == hipSuccess) sums(parts, c_out, dparams + T.boff[l]);
  };
  // The output gradients of the hidden layer and the convolutions (dH, dY3,
  // dY2, dY1, masked by their layer's ReLU) are written in the form's
  // precision: BF16 in the BF16 form, where every product and the bias sum
  // take them rounded; FP32 in the FP32 form.
  // head: dH = dZ W2 through the ReLU of the hidden layer; dW2 = dZ^T H. dZ
  // is read from a copy with rows padded to TRAIN_LD with zeros, in the
  // form's precision (the BF16 products round it to BF16 anyway), so both
  // products read it in vectors and dH's runs over whole k-steps (the head
  // copy's padding rows are zero too); the copy also leaves the bias sums'
  // partials, of the FP32 gradients.
  {
    int64_t chunks = 0;
    e = launch_pad_rows_sum(dlogits, B, TRAIN_OUT, TRAIN_LD, dZp, bf, csw_next, &chunks, s);
    sums(chunks, TRAIN_OUT, dparams + T.boff[4]);
  }
  GemmArgs g = gemm(opnd(dZp, bf, TRAIN_LD, 1), opnd(T.perm + T.perm_off[4], bf, 512, 1), dH,
                    512, B, 512, TRAIN_LD, 0);
  g.mask = opnd(sb.h, bf, 512, 1);
  g.c_bf16 = bf;
  run(g);
  // hidden layer: dA3 = dH W1 (columns p*256 + c) through conv3's ReLU
  g = gemm(opnd(dH, bf, 512, 1), opnd(T.perm + T.perm_off[3], bf, 1, 512), dY3, 3328, B, 3328,
           512, 0);
  g.mask = opnd(sb.a3, bf, 3328, 1);
  g.c_bf16 = bf;
  run(g);
  wgrad(opnd(dH, bf, 1, 512), opnd(sb.a3, bf, 3328, 1), 3, 512, 3328, 256, 13, B, dH);
  // conv3: rows (b, p), 13 per window; input pairs of conv2 positions
  g = gemm(opnd(dY3, bf, 256, 1), opnd(T.perm + T.perm_off[2], bf, 1, 256), dY2, 256, B * 13, 256,
           256, 0);
  g.mask = opnd(sb.a2, bf, 256, 1);
  g.c_bf16 = bf;
  run(g);
  wgrad(opnd(dY3, bf, 1, 256), opnd(sb.a2, bf, 256, 1), 2, 256, 256, 128, 2, B * 13, dY3);
  g = gemm(padded(opnd(dZp, bf, 1, TRAIN_LD), TRAIN_LD), opnd(sb.h, bf, 512, 1),
           dparams + T.woff[4], 512, TRAIN_OUT, 512, B, beta);
  if (groups(g, bf))
    grp.g[grp.count++] = g;
  else
    run(g);
  // conv2: rows (b, p), 26 per window
  g = gemm(opnd(dY2, bf, 128, 1), opnd(T.perm + T.perm_off[1], bf, 1, 128), dY1, 128, B * 26, 128,
           128, 0);
  g.mask = opnd(sb.a1, bf, 128, 1);
  g.c_bf16 = bf;
  run(g);
  wgrad(opnd(dY2, bf, 1, 128), opnd(sb.a1, bf, 128, 1), 1, 128, 128, 64, 2, B * 26, dY2);
  // conv1: rows (b, p), 52 per window; input pairs of window slots, rows of
  // window b at x + b*111*50 (the last 7 slots feed no output)
  const int64_t win = (int64_t)c->cfg.n_slot * c->cfg.n_feat;
  // (x read in runs of 16 along the 100 columns of a pair: up to column 111
  // of the last pair, slot 104, still inside its window)
  wgrad(opnd(dY1, bf, 1, 64), padded(opnd(x, 0, 100, 1, 52, win), 112), 0, 64, 100, 50, 2,
        B * 52, dY1);
  if (e == hipSuccess && grp.count > 0)
    e = launch_gemm_group(grp, bf, part, (int64_t)SPLITK_CAP, bias, s);
  if (dx) {
    // (the products write 52 pairs of slots; the last 7 slots feed no output)
    if (e == hipSuccess) e = launch_zero_columns(dx, B, win, 52 * 100, s);
    g = gemm(opnd(dY1, bf, 64, 1), opnd(T.perm + T.perm_off[0], bf, 1, 64), dx, 100, B * 52, 100,
             64, 0);
    g.cgrp = 52;
    g.cgs = win;
    run(g);
  }
  if (e == hipSuccess && grp.count == 0) e = launch_sum_partials(bias, s);
  if (e != hipSuccess) return hip_fail(c, e, "backward");
  return SIM_OK;
}

int sim_adam_load(sim_ctx* c, float* params, const float* grads, float* m, float* v, int64_t n,
                  float lr, float beta1, float beta2, float eps, int32_t step) {
  if (!c) return SIM_EINVAL;
  if (!params || !grads || !m || !v || step < 1) return fail(c, SIM_EINVAL, "bad arguments");
  if (c->net != 2) return fail(c, SIM_EUNSUPPORTED, "sim_adam_load needs the training head");
  if (!c->weights) return fail(c, SIM_ESTATE, "weights not loaded");
  TrainState& T = c->tr;
  if (n != (int64_t)T.n_params)
    return fail(c, SIM_EINVAL, "n = %lld but the network has %lld parameters", (long long)n,
                (long long)T.n_params);
  if (!T.inv) return fail(c, SIM_EUNSUPPORTED, "no one-to-one re-layout for this network");
  // (the hidden layer's 1.7 M weights through the tiled kernel)
  hipError_t e = launch_adam_relayout(
      params, grads, m, v, n, lr, beta1, beta2, eps, step, T.master, T.inv, T.packed, T.perm,
      c->cfg.prec == SIM_BF16, (int64_t)T.woff[3], static_cast<char*>(T.packed) + T.pack_off[3],
      T.perm + T.perm_off[3], c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "adam");
  return SIM_OK;
}

int sim_adam(sim_ctx* c, float* params, const float* grads, float* m, float* v, int64_t n,
             float lr, float beta1, float beta2, float eps, int32_t step) {
  if (!c) return SIM_EINVAL;
  if (!params || !grads || !m || !v || n < 0 || step < 1) return fail(c, SIM_EINVAL, "bad arguments");
  hipError_t e = launch_adam(params, grads, m, v, n, lr, beta1, beta2, eps, step, c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "adam");
  return SIM_OK;
}

void sim_destroy(sim_ctx* c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->stream);
  drop_graph(c);
  if (c->dev_weights) (void)hipFree(c->dev_weights);
  if (c->dev_w32) (void)hipFree(c->dev_w32);
  if (c->tr.master) (void)hipFree(c->tr.master);
  if (c->tr.maps) (void)hipFree(c->tr.maps);
  if (c->tr.packed) (void)hipFree(c->tr.packed);
  if (c->tr.perm) (void)hipFree(c->tr.perm);
  if (c->tr.inv) (void)hipFree(c->tr.inv);
  if (c->tr.work) (void)hipFree(c->tr.work);
  if (c->tr.save) (void)hipFree(c->tr.save);
  if (c->dev_block) (void)hipFree(c->dev_block);
  if (c->rb_trunk) (void)hipFree(c->rb_trunk);
  if (c->rb_active) (void)hipFree(c->rb_active);
  if (c->rb_logits) (void)hipFree(c->rb_logits);
  if (c->rb_ws) (void)hipFree(c->rb_ws);
  if (c->feat16) (void)hipFree(c->feat16);
  delete c;
}

const char* sim_last_error(const sim_ctx* c) { return c ? c->err.c_str() : "null context"; }

}  // extern "C"

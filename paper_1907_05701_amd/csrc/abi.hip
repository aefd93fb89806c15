// Host-side plumbing of the C ABI: dims validation, the flat parameter layout
// (PyTorch nn.LSTM order, as the paper trains with PyTorch, Section 5.1),
// workspace layout, error strings and the optional kernel-timing hooks.
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <string>
#include <vector>

#include "common.hpp"
#include "gemm_kc.hpp"
#include "lstm_persist.hpp"

static thread_local char g_err[512] = "";

int blstm_fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

int blstm_check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return blstm_fail(BLSTM_EHIP, "%s: %s", what, hipGetErrorString(e));
  return BLSTM_OK;
}

extern "C" const char* blstm_last_error(void) { return g_err; }

// Split-K factor of a product with Mo x No outputs (per batch) and Kr-long
// reductions.
// bf16 (direct-to-LDS kernel): enough workgroups to cover the chip, at least 4
// k-tiles per split, below 256 tiles; aims at 256 workgroups (measured: more
// splits cost more in the partial reduction than they gain).
// float32: the split of least estimated time; a 64x64 block takes 0.25 us of a
// CU per 16-deep k-step, and partials cost their bytes at 4.5 TB/s and a
// launch.
int plan_splits(int64_t Mo, int64_t No, int64_t Kr, int BMt, int BNt, int BK, int batches, bool lp, bool alone) {
  const int64_t tiles = cdiv(Mo, BMt) * cdiv(No, BNt) * batches;
  const int64_t kt = cdiv(Kr, BK);
  if (!lp) {
    int best = 1;
    double lim = 0;
    // the head's products (alone) split no further than 512 workgroups ask
    // for, and not at all from 256: the static entry point takes dims by the
    // size of the head workspace, which the partials are part of
    const int64_t most = !alone ? 16 : tiles >= 256 ? 1 : cdiv(512, tiles);
    for (int s = 1; s <= 16 && s <= most && (s == 1 || kt / s >= 4); ++s) {
      const double t = (double)cdiv(tiles * s, 256) * (double)cdiv(kt, s) * 0.25 +
                       kc_us_partials((double)batches * (double)Mo * (double)No, s);
      if (s == 1 || t < 0.95 * lim) { best = s; lim = t; }
    }
    return best;
  }
  if (tiles >= 256) return 1;
  // a product launched alone fills one round of two blocks per CU without
  // starting a second; the backward layer products share a grouped launch and
  // split to half a round each
  int64_t s = alone ? std::max<int64_t>(512 / tiles, 1) : cdiv(256, tiles);
  s = std::min<int64_t>(s, std::max<int64_t>(kt / 4, 1));
  s = std::min<int64_t>(s, 16);
  return (int)std::max<int64_t>(s, 1);
}

// Tiles and splits of the deferred weight gradients (one grouped launch of
// every layer's dW_ih and dW_hh): 256x256 blocks when they are 5 % faster by
// the estimate of kc_plan.  One such block runs on a CU at a time and all are
// about as long, so the blocks past the last whole round would take a round
// of their own: the first products in launch order stay whole and the last
// ones (layer 0 is the last) are split so that their shorter blocks fill it.
static void plan_dw(const blstm_dims* d, Layout& L) {
  const int64_t H = d->H, M = L.M, kt = cdiv(M, 64);
  const int n = 2 * d->L;
  int64_t tiles[2 * MAX_LAYERS], small = 0, total = 0;
  double elems[2 * MAX_LAYERS];
  for (int i = 0; i < n; ++i) {   // launch order: top layer first, dW_ih then dW_hh
    const int l = d->L - 1 - i / 2;
    const int64_t N = (i & 1) ? H : L.layer_in(l);
    tiles[i] = 2 * cdiv(4 * H, 256) * cdiv(N, 256);
    elems[i] = 2.0 * 4 * H * N;
    small += 2 * cdiv(4 * H, 128) * cdiv(N, 128);
    total += tiles[i];
    L.sp_dw[i] = 1;
  }
  double lim = 0.95 * kc_us_small(small, kt);
  if (4 * H < 192 || H < 192) return;
  for (int j = 0; j <= n; ++j) {   // the products from j on are split
    int64_t whole = 0, rest = 0;
    double e = 0;
    for (int i = 0; i < n; ++i) (i < j ? whole : rest) += tiles[i];
    for (int i = j; i < n; ++i) e += elems[i];
    for (int s = 2; s <= 8 && kt / s >= 8; ++s) {
      if (j == n && s > 2) break;
      const int64_t in_last = whole % 256 ? 256 - whole % 256 : 0;   // CUs idle in the whole blocks' last round
      const int64_t left = rest * s - in_last * s;
      const double t = kc_us_big((double)cdiv(whole, 256), kt) +
                       (left > 0 ? kc_us_big((double)cdiv(left, 256), cdiv(kt, s)) : 0) +
                       (j < n ? kc_us_partials(e, s) : 0);
      if (t < lim) {
        lim = t;
        L.big_dw = true;
        for (int i = 0; i < n; ++i) L.sp_dw[i] = i < j ? 1 : s;
      }
    }
  }
}

// The float32 form: one split for all of them, of least estimated time (as
// plan_splits; one launch of all products, so their blocks count together).
static void plan_dw32(const blstm_dims* d, Layout& L) {
  const int64_t H = d->H, kt = cdiv(L.M, 16);
  int64_t tiles = 0;
  double elems = 0, lim = 0;
  for (int l = 0; l < d->L; ++l)
    for (int64_t N : {(int64_t)L.layer_in(l), H}) {
      tiles += 2 * cdiv(4 * H, 64) * cdiv(N, 64);
      elems += 2.0 * 4 * H * N;
    }
  int best = 1;
  for (int s = 1; s <= 16 && (s == 1 || kt / s >= 4); ++s) {
    const double t = (double)cdiv(tiles * s, 256) * (double)cdiv(kt, s) * 0.25 + kc_us_partials(elems, s);
    if (s == 1 || t < 0.95 * lim) { best = s; lim = t; }
  }
  for (int i = 0; i < 2 * d->L; ++i) L.sp_dw[i] = best;
}

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

int make_layout(const blstm_dims* d, Layout* lo) {
  if (!d || !lo) return blstm_fail(BLSTM_EINVAL, "null dims");
  if (d->L < 1 || d->D < 1 || d->H < 1 || d->P < 1 || d->K < 1 || d->T < 1 || d->B < 1)
    return blstm_fail(BLSTM_EINVAL, "all dims must be positive (L=%d D=%d H=%d P=%d K=%d T=%d B=%d)",
                      d->L, d->D, d->H, d->P, d->K, d->T, d->B);
  if (d->precision != BLSTM_FP32 && d->precision != BLSTM_BF16)
    return blstm_fail(BLSTM_EINVAL, "precision must be BLSTM_FP32 or BLSTM_BF16");
  if (d->L > MAX_LAYERS) return blstm_fail(BLSTM_EUNSUPPORTED, "L > %d", MAX_LAYERS);
  const int hq = d->precision == BLSTM_BF16 ? 32 : 16;
  if (d->H % hq) return blstm_fail(BLSTM_EUNSUPPORTED, "H must be a multiple of %d", hq);
  if (d->P % 8) return blstm_fail(BLSTM_EUNSUPPORTED, "P must be a multiple of 8");
  if (d->D % 4) return blstm_fail(BLSTM_EUNSUPPORTED, "D must be a multiple of 4");
  if ((int64_t)d->T * d->B > (1 << 24)) return blstm_fail(BLSTM_EUNSUPPORTED, "T*B too large");
  if (d->B > 65535 * 16) return blstm_fail(BLSTM_EUNSUPPORTED, "B too large");

  Layout& L = *lo;
  memset(&L, 0, sizeof(L));
  L.L = d->L; L.D = d->D; L.H = d->H; L.P = d->P; L.K = d->K; L.T = d->T; L.B = d->B;
  L.prec = d->precision;
  L.M = (int64_t)d->T * d->B;
  L.Dp0 = (int)rup(d->D, 8);
  L.Kp = (int)rup(d->K, 8);
  L.es = d->precision == BLSTM_BF16 ? 2 : 4;
  const int64_t H = d->H;
  int64_t off = 0;
  for (int l = 0; l < d->L; ++l) {
    const int64_t Dl = l == 0 ? d->D : 2 * H;
    for (int dir = 0; dir < 2; ++dir) {
      L.Wih[l][dir] = off; off += 4 * H * Dl;
      L.Whh[l][dir] = off; off += 4 * H * H;
      L.bih[l][dir] = off; off += 4 * H;
      L.bhh[l][dir] = off; off += 4 * H;
    }
  }
  L.Wl = off; off += (int64_t)d->P * 2 * H;
  L.bl = off; off += d->P;
  L.Ws = off; off += (int64_t)d->K * d->P;
  L.bs = off; off += d->K;
  L.n = off;

  // act_ws
  const size_t es = L.es;
  const int64_t M = L.M;
  size_t a = 0;
  L.X0 = a; a = align256(a + (size_t)M * L.Dp0 * es);
  for (int l = 0; l < d->L; ++l) {
    if (l < d->L - 1) { L.Y[l] = a; a = align256(a + (size_t)M * 2 * H * es); }
    L.G[l] = a; a = align256(a + (size_t)M * 8 * H * es);
    L.C[l] = a; a = align256(a + (size_t)M * 2 * H * 4);
  }
  L.GX = a; a = align256(a + (size_t)M * 8 * H * es);
  L.DYa = a; a = align256(a + (size_t)M * 2 * H * 4);
  L.DYb = a; a = align256(a + (size_t)M * 2 * H * 4);
  L.DC = a; a = align256(a + (size_t)2 * d->B * H * 4);
  L.WT = a; a = align256(a + (size_t)2 * d->L * 4 * H * H * es);
  L.WP0_bytes = es == 2 && d->D % 8 != 0 ? (size_t)2 * 4 * H * L.Dp0 * es : 0;
  L.WP0 = a; a = align256(a + L.WP0_bytes);
  // da [M][8H], one per layer (the weight gradients of every layer run after
  // the last BPTT); the top layer's in the forward's input projection, which
  // the backward does not read
  L.da_bytes = align256((size_t)M * 8 * H * es);
  for (int l = 0; l < d->L - 1; ++l) { L.DA[l] = a; a += L.da_bytes; }
  L.DA[d->L - 1] = L.GX;
  // per-step 16-row partials (per-step BPTT) or per-workgroup partials over
  // all steps (persistent BPTT)
  // (8-row workgroups in bf16, 4-row ones in float32)
  L.dbp_bytes = align256((size_t)std::max<int64_t>((int64_t)d->T * cdiv(d->B, 16), cdiv(d->B, es == 2 ? 8 : 4)) * 8 * H * 4);
  L.DBP = a; a += (size_t)std::max(2, d->L) * L.dbp_bytes;   // per layer when the bias sums wait for the last BPTT
  L.CSP = a; a = align256(a + (size_t)COLSUM_MAX_CHUNKS * 8 * H * 4);
  // split-K plans and partial buffers of the backward GEMMs: a layer's dX, and
  // after the last dX the deferred weight gradients (disjoint regions within
  // their one launch)
  const int BMt = es == 2 ? GemmCfg<bf16>::BM : GemmCfg<float>::BM;
  const int BNt = es == 2 ? GemmCfg<bf16>::BN : GemmCfg<float>::BN;
  const int BKt = es == 2 ? GemmCfg<bf16>::BK : GemmCfg<float>::BK;
  size_t skp = 0;
  const bool lp = es == 2;
  for (int l = 0; l < d->L; ++l) {
    const int64_t Dl = l == 0 ? d->D : 2 * H;
    L.sp_dX[l] = l > 0 ? plan_splits(M, Dl, 8 * H, BMt, BNt, BKt, 1, lp, lp) : 1;
    if (lp && l > 0) {
      const KcPlan p = kc_plan(M, Dl, 8 * H, 1, L.sp_dX[l]);
      L.big_dX[l] = p.big;
      L.sp_dX[l] = p.splits;
    }
    if (L.sp_dX[l] > 1) skp = std::max(skp, (size_t)L.sp_dX[l] * M * Dl * 4);
  }
  if (lp) plan_dw(d, L);
  else plan_dw32(d, L);
  size_t dw = 0;
  for (int i = 0; i < 2 * d->L; ++i) {
    const int64_t Nw = (i & 1) ? H : L.layer_in(d->L - 1 - i / 2);
    L.skp_dw[i] = dw;
    if (L.sp_dw[i] > 1) dw += align256((size_t)L.sp_dw[i] * 2 * 4 * H * Nw * 4);
  }
  skp = std::max(skp, dw);
  L.SKP = a; a = align256(a + skp);
  L.XCH = a; a = align256(a + (es == 2 ? persist_xch_bytes(d->B, d->H) : persist32_xch_bytes(d->B, d->H)));   // recurrent step exchange
  L.GST = a; a = align256(a + (es == 2 ? persist_state_bytes(d->B, d->H) : persist32_state_bytes(d->B, d->H)));
  // recurrence status block, the last PERSIST_STATUS_BYTES of act_ws
  L.SYNC = a; a += PERSIST_STATUS_BYTES;
  L.act_bytes = a;

  // head_ws
  size_t h = 0;
  const int64_t P = d->P;
  L.Z = h; h = align256(h + (size_t)M * P * es);
  // float32: the logits, overwritten by ds; bf16: ds only (the logits stay
  // in the products' accumulators) plus the per-(frame, class strip)
  // statistics and the per-frame log-sum-exp
  L.S = h; h = align256(h + (size_t)M * L.Kp * es);
  L.LST = h; h = align256(h + (es == 2 ? (size_t)M * cdiv(d->K, 64) * 8 : 0));
  L.LSE = h; h = align256(h + (es == 2 ? (size_t)M * 4 : 0));
  L.LDB = h; h = align256(h + (es == 2 ? (size_t)cdiv(M, 32) * L.Kp * 4 : 0));   // db_s partials per frame tile (32 frames or more)
  // bf16: db_l shares of the 128-class strips (W_s^T db_s, per strip)
  L.DBLP = h; h = align256(h + (es == 2 ? (size_t)cdiv(d->K, 128) * d->P * 4 : 0));
  L.RL = h; h = align256(h + (size_t)M * 4);
  L.DZ = h; h = align256(h + (size_t)M * P * 4);
  L.DZT = h; h = align256(h + (size_t)M * P * es);
  // float32: column-sum partials of db_s (those of db_l in HSKP)
  L.HCSP = h; h = align256(h + (es == 2 ? 0 : (size_t)COLSUM_MAX_CHUNKS * std::max<int64_t>(L.Kp, P) * 4));
  size_t hsk = 0;
  L.sp_z = es == 2 ? plan_splits(M, P, 2 * H, BMt, BNt, BKt, 1, true, true) : 1;
  if (L.sp_z > 1) hsk = std::max(hsk, (size_t)L.sp_z * M * P * 4);
  L.sp_dz = plan_splits(M, P, d->K, BMt, BNt, BKt, 1, es == 2, true);
  if (es == 2) {
    const KcPlan p = kc_plan(M, P, d->K, 1, L.sp_dz);
    L.big_dz = p.big;
    L.sp_dz = p.splits;
  }
  hsk = std::max(hsk, (size_t)L.sp_dz * M * P * 4);  // dz always goes through partials
  L.sp_dWs = plan_splits(d->K, P, M, BMt, BNt, BKt, 1, es == 2, true);
  if (es == 2) {
    const KcPlan p = kc_plan(d->K, P, M, 1, L.sp_dWs);
    L.big_dWs = p.big;
    L.sp_dWs = p.splits;
  }
  if (L.sp_dWs > 1) hsk = std::max(hsk, (size_t)L.sp_dWs * d->K * P * 4);
  L.sp_dWl = plan_splits(P, 2 * H, M, BMt, BNt, BKt, 1, es == 2, true);
  if (L.sp_dWl > 1) hsk = std::max(hsk, (size_t)L.sp_dWl * P * 2 * H * 4);
  L.sp_dy = plan_splits(M, 2 * H, P, BMt, BNt, BKt, 1, es == 2, true);
  if (L.sp_dy > 1) hsk = std::max(hsk, (size_t)L.sp_dy * M * 2 * H * 4);
  L.HSKP = h; h = align256(h + hsk);
  L.head_bytes = h;
  L.ytop_bytes = (size_t)M * 2 * H * es;
  return BLSTM_OK;
}

extern "C" int64_t blstm_param_count(const blstm_dims* dims) {
  Layout lo;
  int rc = make_layout(dims, &lo);
  if (rc != BLSTM_OK) return rc;
  return lo.n;
}

extern "C" int blstm_workspace_bytes(const blstm_dims* dims, size_t* act_ws, size_t* head_ws,
                                     size_t* theta_lp, size_t* y_top) {
  Layout lo;
  int rc = make_layout(dims, &lo);
  if (rc != BLSTM_OK) return rc;
  if (act_ws) *act_ws = lo.act_bytes;
  if (head_ws) *head_ws = lo.head_bytes;
  if (theta_lp) *theta_lp = lo.prec == BLSTM_BF16 ? (size_t)lo.n * 2 : 0;
  if (y_top) *y_top = lo.ytop_bytes;
  return BLSTM_OK;
}

// ---------------------------------------------------------------------------
// Kernel timing: HIP events around selected launches.
// ---------------------------------------------------------------------------
bool g_timing_on = false;
static std::string g_prefix;
struct TimedLaunch {
  std::string name;
  hipEvent_t start, stop;
  int launches;
};
static std::vector<TimedLaunch> g_launches;
static std::vector<hipEvent_t> g_pool;

static hipEvent_t take_event() {
  if (!g_pool.empty()) {
    hipEvent_t e = g_pool.back();
    g_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

int timing_pre(const char* name, hipStream_t s) { return timing_pre_n(name, s, 1); }

int timing_pre_n(const char* name, hipStream_t s, int launches) {
  if (strncmp(name, g_prefix.c_str(), g_prefix.size()) != 0) return -1;
  TimedLaunch t;
  t.name = name;
  t.launches = launches;
  t.start = take_event();
  t.stop = take_event();
  if (!t.start || !t.stop) return -1;
  hipEventRecord(t.start, s);
  g_launches.push_back(t);
  return (int)g_launches.size() - 1;
}

void timing_post(int slot, hipStream_t s) { hipEventRecord(g_launches[slot].stop, s); }

extern "C" int blstm_timing_begin(const char* prefix) {
  for (auto& t : g_launches) {
    g_pool.push_back(t.start);
    g_pool.push_back(t.stop);
  }
  g_launches.clear();
  g_prefix = prefix ? prefix : "";
  g_timing_on = true;
  return BLSTM_OK;
}

extern "C" int blstm_timing_end(blstm_kernel_time* out, int32_t cap, int32_t* count) {
  g_timing_on = false;
  std::vector<blstm_kernel_time> agg;
  for (auto& t : g_launches) {
    if (hipEventSynchronize(t.stop) != hipSuccess)
      return blstm_fail(BLSTM_EHIP, "hipEventSynchronize failed");
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, t.start, t.stop) != hipSuccess)
      return blstm_fail(BLSTM_EHIP, "hipEventElapsedTime failed");
    size_t i = 0;
    for (; i < agg.size(); ++i)
      if (t.name == agg[i].name) break;
    if (i == agg.size()) {
      blstm_kernel_time k;
      memset(&k, 0, sizeof(k));
      snprintf(k.name, sizeof(k.name), "%s", t.name.c_str());
      agg.push_back(k);
    }
    agg[i].launches += t.launches;
    agg[i].total_ms += ms;
  }
  if (count) *count = (int32_t)agg.size();
  for (size_t i = 0; i < agg.size() && (int32_t)i < cap; ++i) out[i] = agg[i];
  return BLSTM_OK;
}

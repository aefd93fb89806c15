// Persistent recurrent kernels of the float32 path: one launch runs all T
// steps of one layer, for both directions at once, with the W_hh slice of
// each workgroup in registers for the whole chunk.
//
// Work split.  A "member" owns PU = 16 NCB hidden units (32, 64 or 128: the
// most whose 4 PU gate rows of W_hh fill the 256 KB of half a register file),
// so a layer of up to 128 cells is one workgroup per (direction, batch slice)
// and needs no exchange at all, one of up to 256 cells four members and one
// of up to 512 cells sixteen.  A batch slice is RV = 4 RT rows: the products
// run on v_mfma_f32_4x4x1_16b_f32, which multiplies 4 batch rows by 64
// columns with the row operand broadcast to its 16 blocks.  Its rate equals
// that of the 16x16x4 form (126 TFLOP/s measured over the chip) without
// padding a slice to 16 rows, so a small batch spreads over all CUs: at
// H = 512 a batch of 32 takes 2 directions x 8 slices of 4 rows x 16 members
// = 256 workgroups, each step costing 128 such instructions per wave.
//   forward : wave (cb, ks) multiplies h_prev (RV rows, its k part of the H
//             units) by 64 gate columns (16 units x gates i, f, g, o, the
//             gate fastest); the k parts meet in LDS; each thread then owns
//             one gate of one cell, and the four threads of a cell swap
//             their gates with DPP quad permutations.
//   backward: each thread forms one gate's da of its cell; wave (cb, ks)
//             multiplies the member's own da (k = 128 of its gate rows) by
//             W_hh for 64 hidden units: partial sums of dh_rec for all H
//             units, summed by the owner of each unit in part order.
// Steps exchange h (forward) and the partial sums (backward) as 8-byte words
// holding one float32 and a 32-bit tag (launch position and step), in two
// slots alternating by step; the reasoning about slot reuse, residency and
// bounded waits is that of the bf16 kernels (lstm_persist.hip).
//
// What bounds it: at 4 rows the step's exchange round trip (about 1 us) and
// the products (0.9 us of matrix-core time per 4 rows) about equally; at 16
// rows the products.  The per-step launches that these kernels replace took
// 19.8 us (forward) and 30.5 us (backward) per step at H = 512, B = 32, and
// 5.7 and 7.1 us at H = 64, B = 8.
#include <stdlib.h>

#include "common.hpp"
#include "lstm_persist.hpp"

#define P32_THREADS 512
#define P32_KW 128                 // k values of W_hh per wave (registers per lane)

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

template <int CTRL>
__device__ __forceinline__ float quad(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
#define QUAD_0 0x00     // the quad's lane 0 in every lane, ...
#define QUAD_1 0x55
#define QUAD_2 0xAA
#define QUAD_3 0xFF
#define QUAD_XOR1 0xB1
#define QUAD_XOR2 0x4E

// acc += a(4 rows, k = 16 values of this register) * w[0..15]: lane 4 b + i
// of `a` holds row i at the b-th k value, lane l of w[b] column l; lane l of
// acc receives rows 0..3 of column l.
template <int N>
__device__ __forceinline__ f32x4 mfma_rows4(float a, const float* w, f32x4 acc) {
  if constexpr (N > 0) {
    acc = mfma_rows4<N - 1>(a, w, acc);
    acc = __builtin_amdgcn_mfma_f32_4x4x1f32(a, w[N - 1], acc, 4, N - 1, 0);
  }
  return acc;
}

__device__ __forceinline__ void p32_publish(uint64_t* p, float v, uint32_t tag, bool local) {
  ll_store64(p, ((uint64_t)tag << 32) | __builtin_bit_cast(uint32_t, v), local);
}

// LDS row pitch (floats) of a row operand of n k values: the 4 rows x 16 k
// of one operand read fall in 64 distinct banks.
__host__ __device__ static inline int p32_pitch(int n) { return (n + 63) / 64 * 64 + 16; }

// ---------------------------------------------------------------------------
// Forward.
// ---------------------------------------------------------------------------
// SOLO: one member (no exchange; h stays in LDS).  One pass runs steps
// [tau0, tau1) of member `mem`, with the group's other members beside it or
// (ONE) one step of one member after the other, as in the bf16 kernels.
template <int NCB, int RT, bool SOLO, bool ONE>
__device__ __forceinline__ int fwd32_pass(const Persist32Args& a, char* lds_raw, int g, int mem, int nmem, int tau0,
                                          int tau1) {
  constexpr int PU = 16 * NCB, KS = 8 / NCB, RV = 4 * RT, NCOL = 64 * NCB;
  constexpr int IT = RV * NCOL / P32_THREADS;   // gate values per thread
  constexpr int RPI = P32_THREADS / NCOL;       // rows between a thread's items
  const int H = a.H, B = a.B, Tn = a.Tn;
  const int d = g & 1, s = g >> 1;
  const int u0 = mem * PU;
  const int tid = pass_thread<ONE, false>(), lane = tid & 63, w = tid >> 6;
  const int cb = w % NCB, ks = w / NCB;
  const int KQ = (H + 16 * KS - 1) / (16 * KS) * 16;   // k values per part (whole groups of 16)
  const int k0 = ks * KQ;

  // W_hh rows of this lane's gate column, k0 .. k0 + KQ (zeros past H), through
  // a wave's own piece of LDS so that the global loads take whole lines (8
  // rows of 32 k values per instruction; a lane loading its own row by itself
  // touches 64 lines per instruction: 17.0 -> 10.6 us for a one-step launch
  // at H = 512)
  float bw[P32_KW];
  {
    constexpr int SP = 36;   // staging pitch (floats): 16-byte aligned rows
    float* stg = (float*)lds_raw + w * 64 * SP;
    const float* wd = a.W + (d ? a.whh1 : a.whh0);
#pragma unroll
    for (int c = 0; c < P32_KW / 32; ++c) {
      f32x4u v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int cl = i * 8 + (lane >> 3), kk = c * 32 + (lane & 7) * 4;
        const int un = u0 + cb * 16 + (cl >> 2);
        const bool ok = un < H && kk < KQ && k0 + kk < H;   // H and KQ are multiples of 16
        v[i] = ok ? *(const f32x4u*)(wd + ((int64_t)(cl & 3) * H + un) * H + k0 + kk) : f32x4u{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) *(f32x4*)&stg[(i * 8 + (lane >> 3)) * SP + (lane & 7) * 4] = v[i];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const f32x4 r = *(const f32x4*)&stg[lane * SP + j * 4];
#pragma unroll
        for (int e = 0; e < 4; ++e) bw[c * 32 + j * 4 + e] = r[e];
      }
    }
    __syncthreads();   // the step buffers reuse this LDS
  }

  const int HS = p32_pitch(H);
  float* hl = (float*)lds_raw;        // h of the previous step [RV][HS]
  float* red = hl + RV * HS;          // products by k part [KS][RV][NCOL]
  for (int i = tid; i < RV * HS; i += P32_THREADS) hl[i] = 0.f;
  lds_barrier();

  const int rowbase = a.b0 + s * RV, rend = a.b0 + a.rows;
  const int64_t slot_stride = (int64_t)2 * a.rows * H;
  // items: gate column `col` of row tid / NCOL + RPI i
  const int col = tid % NCOL, q = col & 3, unit = u0 + (col >> 2), r0 = tid / NCOL;
  const bool uok = unit < H;
  const int unitc = min(unit, H - 1);
  float creg[IT], gxn[IT];
  auto load_gx = [&](int tt) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int row = min(rowbase + r0 + RPI * i, rend - 1);
      gxn[i] = a.Gx[((int64_t)tt * B + row) * 8 * H + (int64_t)d * 4 * H + (int64_t)q * H + unitc];
    }
  };
#pragma unroll
  for (int i = 0; i < IT; ++i) creg[i] = ONE && tau0 > 0 ? group_state(a.state, g, mem, nmem)[i] : 0.f;
  load_gx(d ? Tn - 1 - tau0 : tau0);
  int how = GROUP_APART;
  if (!SOLO && !ONE && Tn > 1) {
    how = group_meet(group_word(a.words, a.seq, g), a.words, a.seq, g, mem, nmem, a.wait);
    if (how >= GROUP_ALONE) return how;
  }
  const bool local = how == GROUP_LOCAL;

  for (int tau = tau0; tau < tau1; ++tau) {
    const int t = d ? Tn - 1 - tau : tau;
    float sum[IT];
    if (tau > 0) {
      if constexpr (!SOLO) {
        // h of the previous step: the slice's RV rows x H words are
        // contiguous; up to GB words per thread at a time
        constexpr int GB = RV < 8 ? RV : 8;
        const int nwords = RV * H;
        const uint64_t* src = a.X + ((tau - 1) & 1) * slot_stride + ((int64_t)d * a.rows + (rowbase - a.b0)) * H;
        const uint32_t want = a.tag0 + tau;
        for (int j0 = tid; j0 < nwords; j0 += GB * P32_THREADS) {
          uint64_t wv[GB];
          uint32_t off[GB];
#pragma unroll
          for (int j = 0; j < GB; ++j) {
            const int idx = j0 + j * P32_THREADS;
            off[j] = (uint32_t)idx;
            wv[j] = idx < nwords && rowbase + idx / H < rend ? ll_load(src + idx) : (uint64_t)want << 32;
          }
          poll_tagged<GB>(wv, src, off, want, a.status);
#pragma unroll
          for (int j = 0; j < GB; ++j) {
            const int idx = j0 + j * P32_THREADS;
            if (idx < nwords) hl[(idx / H) * HS + idx % H] = __builtin_bit_cast(float, (uint32_t)wv[j]);
          }
        }
      }
      lds_barrier();
      f32x4 acc[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
      const float* ab = hl + (lane & 3) * HS + k0 + (lane >> 2);
#pragma unroll
      for (int kg = 0; kg < P32_KW / 16; ++kg) {
        if (kg * 16 >= KQ) break;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt] = mfma_rows4<16>(ab[rt * 4 * HS + kg * 16], &bw[kg * 16], acc[rt]);
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(ks * RV + rt * 4 + r) * NCOL + cb * 64 + lane] = acc[rt][r];
      lds_barrier();
#pragma unroll
      for (int i = 0; i < IT; ++i) {
        sum[i] = red[(r0 + RPI * i) * NCOL + col];
#pragma unroll
        for (int p = 1; p < KS; ++p) sum[i] += red[(p * RV + r0 + RPI * i) * NCOL + col];
      }
    }
    float pre[IT];   // (the projection not before here: waiting for it at the step's start waits for the last stores too)
#pragma unroll
    for (int i = 0; i < IT; ++i) pre[i] = tau > 0 ? gxn[i] + sum[i] : gxn[i];
    uint64_t* xo = a.X + (tau & 1) * slot_stride;
    float hv[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      // this thread's gate, then the cell in all four threads of the quad
      const float sg = sigmoidf_(q == 2 ? 2.0f * pre[i] : pre[i]);
      const float act = q == 2 ? 2.0f * sg - 1.0f : sg;
      const float ig = quad<QUAD_0>(act), fg = quad<QUAD_1>(act), gg = quad<QUAD_2>(act), og = quad<QUAD_3>(act);
      creg[i] = fg * creg[i] + ig * gg;
      hv[i] = og * tanhf_(creg[i]);
    }
    if (q == 0) {
#pragma unroll
      for (int i = 0; i < IT; ++i) {
        const int rl = r0 + RPI * i, row = rowbase + rl;
        if constexpr (SOLO) {
          // (rows past the batch feed only themselves; a unit past H, a copy
          // of the last one here, meets zero weights)
          if (tau + 1 < Tn) hl[rl * HS + unit] = hv[i];
        } else if (uok && row < rend) {
          p32_publish(xo + ((int64_t)d * a.rows + (row - a.b0)) * H + unit, hv[i], a.tag0 + tau + 1, local);
        }
      }
    }
    // the prefetch before the stores: its wait then leaves them in flight
    if (tau + 1 < tau1) load_gx(d ? Tn - 2 - tau : tau + 1);
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int row = rowbase + r0 + RPI * i;
      if (!uok || row >= rend) continue;
      const int64_t f = (int64_t)t * B + row;
      a.G[f * 8 * H + (int64_t)d * 4 * H + (int64_t)unit * 4 + q] = pre[i];
      if (q == 1 || q == 2) (q == 1 ? a.C : a.Y)[f * 2 * H + (int64_t)d * H + unit] = q == 1 ? creg[i] : hv[i];
    }
  }
  if constexpr (ONE) {
#pragma unroll
    for (int i = 0; i < IT; ++i) group_state(a.state, g, mem, nmem)[i] = creg[i];
    __syncthreads();   // the next pass reuses the LDS
  }
  return how;
}

// A group that runs on this workgroup alone.
template <int NCB, int RT>
__device__ __attribute__((noinline)) void fwd32_alone(const Persist32Args* at, lds_base_t lds, int gv, int nmemv) {
  const int g = scalar(gv), nmem = scalar(nmemv), Tn = pass_args(at).Tn;
#pragma nounroll
  for (int tau = 0; tau < Tn; ++tau)
#pragma nounroll
    for (int m = 0; m < nmem; ++m)
      fwd32_pass<NCB, RT, false, true>(pass_args(at), (char*)lds, g, m, nmem, tau, tau + 1);
}

template <int NCB, int RT, bool SOLO>
__global__ __launch_bounds__(P32_THREADS) void lstm_fwd_persist32(const Persist32Args a) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  if constexpr (SOLO) {
    fwd32_pass<NCB, RT, true, false>(a, lds_raw, blockIdx.x, 0, 1, 0, a.Tn);
  } else {
    const int nmem = gridDim.x / a.NG;
    int g, mem;
    group_of(a.NG, nmem, &g, &mem);
    if (g >= 2 * a.NS) return;   // padding (see persist_groups)
    if (a.Tn > 1) group_arrive(a.words, a.seq, g, mem, a.wait);
    if (fwd32_pass<NCB, RT, false, false>(a, lds_raw, g, mem, nmem, 0, a.Tn) != GROUP_ALONE) return;
    if (threadIdx.x == 0) a.status[1] = 1;
    fwd32_alone<NCB, RT>(kernel_args<Persist32Args>(), (lds_base_t)lds_raw, g, nmem);
  }
}

// ---------------------------------------------------------------------------
// Backward (BPTT).
// ---------------------------------------------------------------------------
// KS: k parts of the own gate rows; SOLO: one member (the partial sums stay
// in LDS).
template <int NCB, int RT, int KS, bool SOLO, bool ONE>
__device__ __forceinline__ int bwd32_pass(const Persist32Args& a, char* lds_raw, int g, int mem, int nmem, int tau0,
                                          int tau1) {
  constexpr int PU = 16 * NCB, RV = 4 * RT, NCOL = 64 * NCB;   // NCOL own gate rows
  constexpr int CBS = 8 / KS, KW = NCOL / KS;                  // unit blocks of 64; own rows per k part
  static_assert(KW <= P32_KW && KW % 16 == 0, "W_hh slice in registers");
  constexpr int IT = RV * NCOL / P32_THREADS, RPI = P32_THREADS / NCOL;
  constexpr int MEMS = SOLO ? 1 : NCB == 2 ? 16 : 4;           // members at most
  constexpr int MPP = (MEMS * KS + 3) / 4;                     // partial sums per thread of a quad
  constexpr int AS = (NCOL + 63) / 64 * 64 + 16;
  const int H = a.H, B = a.B, Tn = a.Tn;
  const int d = g & 1, s = g >> 1;
  const int u0 = mem * PU;
  const int tid = pass_thread<ONE, false>(), lane = tid & 63, w = tid >> 6;
  const int cb = w % CBS, ks = w / CBS;
  const int hu = cb * 64 + lane;   // hidden unit of this lane's product column
  const int parts = nmem * KS;

  // W_hh[own gate row][hu], own row 4 (unit - u0) + gate, the KW rows of part ks
  float bw[KW];
  {
    const float* wd = a.W + (d ? a.whh1 : a.whh0) + min(hu, H - 1);
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const int unit = u0 + ks * (KW / 4) + (k >> 2);
      const bool ok = unit < H && hu < H;
      const float v = wd[((int64_t)(k & 3) * H + min(unit, H - 1)) * H];
      bw[k] = ok ? v : 0.f;
    }
  }

  float* al = (float*)lds_raw;            // own da by step parity [2][RV][AS]
  float* dhl = al + 2 * RV * AS;          // one member: the partial sums [KS][RV][PU]
  const int rowbase = a.b0 + s * RV, rend = a.b0 + a.rows;
  const int64_t slot_stride = (int64_t)2 * parts * a.rows * H;
  const int col = tid % NCOL, q = col & 3, unit = u0 + (col >> 2), r0 = tid / NCOL;
  const bool uok = unit < H;
  const int unitc = min(unit, H - 1);
  float dcreg[IT], dbacc[IT], cc[IT], cpn[IT], dyn[IT], gn[IT];
  auto rowc = [&](int i) { return min(rowbase + r0 + RPI * i, rend - 1); };
  auto fetch = [&](int tau_) {
    const int t_ = d ? tau_ : Tn - 1 - tau_;
    const int tp_ = d ? t_ + 1 : t_ - 1;
    const bool hp = tp_ >= 0 && tp_ < Tn;
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int64_t f = (int64_t)t_ * B + rowc(i);
      dyn[i] = a.DY[f * 2 * H + (int64_t)d * H + unitc];
      gn[i] = a.G[f * 8 * H + (int64_t)d * 4 * H + (int64_t)unitc * 4 + q];
      const float c = a.C[((int64_t)(hp ? tp_ : t_) * B + rowc(i)) * 2 * H + (int64_t)d * H + unitc];
      cpn[i] = hp ? c : 0.f;
    }
  };
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    dcreg[i] = ONE && tau0 > 0 ? group_state(a.state, g, mem, nmem)[4 + i] : 0.f;
    dbacc[i] = ONE && tau0 > 0 ? group_state(a.state, g, mem, nmem)[i] : 0.f;
    cc[i] = a.C[((int64_t)(d ? tau0 : Tn - 1 - tau0) * B + rowc(i)) * 2 * H + (int64_t)d * H + unitc];
  }
  fetch(tau0);
  int how = GROUP_APART;
  if (!SOLO && !ONE && Tn > 1) {
    how = group_meet(group_word(a.words, a.seq, g), a.words, a.seq, g, mem, nmem, a.wait);
    if (how >= GROUP_ALONE) return how;
  }
  const bool local = how == GROUP_LOCAL;

  for (int tau = tau0; tau < tau1; ++tau) {
    const int t = d ? tau : Tn - 1 - tau;
    float* alp = al + (tau & 1) * RV * AS;
    // the gathered dh_rec of each item: the quad's threads take MPP parts
    // each in part order, the four sums are added by pairs
    float dhr[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) dhr[i] = 0.f;
    if (tau > 0) {
      if constexpr (!SOLO) {
        const uint64_t* src = a.X + ((tau - 1) & 1) * slot_stride;
        const uint32_t want = a.tag0 + tau;
        constexpr int IB = IT * MPP <= 8 ? IT : 8 / MPP;   // items gathered at a time
#pragma unroll
        for (int i0 = 0; i0 < IT; i0 += IB) {
          uint64_t wv[IB * MPP];
          uint32_t off[IB * MPP];
#pragma unroll
          for (int j = 0; j < IB * MPP; ++j) {
            const int row = rowbase + r0 + RPI * (i0 + j / MPP), p = q * MPP + j % MPP;
            const bool ok = uok && row < rend && p < parts;
            off[j] = (uint32_t)((((int64_t)d * parts + (ok ? p : 0)) * a.rows + (ok ? row - a.b0 : 0)) * H + unitc);
            wv[j] = ok ? ll_load(src + off[j]) : (uint64_t)want << 32;
          }
          poll_tagged<IB * MPP>(wv, src, off, want, a.status);
#pragma unroll
          for (int j = 0; j < IB * MPP; ++j) dhr[i0 + j / MPP] += __builtin_bit_cast(float, (uint32_t)wv[j]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < IT; ++i)
#pragma unroll
          for (int p = 0; p < MPP; ++p)
            if (q * MPP + p < KS) dhr[i] += dhl[((q * MPP + p) * RV + r0 + RPI * i) * PU + (col >> 2)];
      }
#pragma unroll
      for (int i = 0; i < IT; ++i) {
        dhr[i] += quad<QUAD_XOR1>(dhr[i]);
        dhr[i] += quad<QUAD_XOR2>(dhr[i]);
      }
    }
    float da[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const float sg = sigmoidf_(q == 2 ? 2.0f * gn[i] : gn[i]);
      const float act = q == 2 ? 2.0f * sg - 1.0f : sg;
      const float ig = quad<QUAD_0>(act), fg = quad<QUAD_1>(act), gg = quad<QUAD_2>(act), og = quad<QUAD_3>(act);
      const float dh = dhr[i] + dyn[i];
      const float tc = tanhf_(cc[i]);
      const float dc = dh * og * (1.f - tc * tc) + dcreg[i];
      dcreg[i] = dc * fg;
      const float v0 = dc * gg * ig * (1.f - ig);
      const float v1 = dc * cpn[i] * fg * (1.f - fg);
      const float v2 = dc * ig * (1.f - gg * gg);
      const float v3 = dh * tc * og * (1.f - og);
      const float v = q == 0 ? v0 : q == 1 ? v1 : q == 2 ? v2 : v3;
      const int rl = r0 + RPI * i;
      da[i] = uok && rowbase + rl < rend ? v : 0.f;
      alp[rl * AS + col] = da[i];
      dbacc[i] += da[i];
      cc[i] = cpn[i];
    }
    lds_barrier();   // own da complete (and, one member, the sums of dhl read)
    if (tau + 1 < Tn) {
      f32x4 acc[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
      const float* ab = alp + (lane & 3) * AS + ks * KW + (lane >> 2);
#pragma unroll
      for (int kg = 0; kg < KW / 16; ++kg)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt] = mfma_rows4<16>(ab[rt * 4 * AS + kg * 16], &bw[kg * 16], acc[rt]);
      if constexpr (!SOLO) {
        uint64_t* xo = a.X + (tau & 1) * slot_stride + ((int64_t)d * parts + mem * KS + ks) * a.rows * H + hu;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = rowbase + rt * 4 + r;
            if (hu < H && row < rend) p32_publish(xo + (int64_t)(row - a.b0) * H, acc[rt][r], a.tag0 + tau + 1, local);
          }
      } else {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (CBS * 64 <= PU || hu < PU) dhl[(ks * RV + rt * 4 + r) * PU + hu] = acc[rt][r];
      }
      if (tau + 1 < tau1) fetch(tau + 1);
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int row = rowbase + r0 + RPI * i;
      if (uok && row < rend)
        a.DA[((int64_t)t * B + row) * 8 * H + (int64_t)d * 4 * H + (int64_t)q * H + unit] = da[i];
    }
    if constexpr (SOLO) lds_barrier();   // the partial sums in LDS
  }
  if constexpr (ONE) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      group_state(a.state, g, mem, nmem)[4 + i] = dcreg[i];
      group_state(a.state, g, mem, nmem)[i] = dbacc[i];
    }
    __syncthreads();   // the next pass reuses the LDS
    if (tau1 < Tn) return how;
  }
  // bias partials: the slice's rows in order
  __syncthreads();
#pragma unroll
  for (int i = 0; i < IT; ++i) al[(r0 + RPI * i) * AS + col] = dbacc[i];
  __syncthreads();
  if (tid < NCOL && uok) {
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < RV; ++r) sum += al[r * AS + tid];
    a.DBP[(int64_t)(rowbase / RV) * 8 * H + (int64_t)d * 4 * H + (int64_t)q * H + unit] = sum;
  }
  if constexpr (ONE) __syncthreads();
  return how;
}

template <int NCB, int RT, int KS>
__device__ __attribute__((noinline)) void bwd32_alone(const Persist32Args* at, lds_base_t lds, int gv, int nmemv) {
  const int g = scalar(gv), nmem = scalar(nmemv), Tn = pass_args(at).Tn;
#pragma nounroll
  for (int tau = 0; tau < Tn; ++tau)
#pragma nounroll
    for (int m = 0; m < nmem; ++m)
      bwd32_pass<NCB, RT, KS, false, true>(pass_args(at), (char*)lds, g, m, nmem, tau, tau + 1);
}

template <int NCB, int RT, int KS, bool SOLO>
__global__ __launch_bounds__(P32_THREADS) void lstm_bwd_persist32(const Persist32Args a) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  if constexpr (SOLO) {
    bwd32_pass<NCB, RT, KS, true, false>(a, lds_raw, blockIdx.x, 0, 1, 0, a.Tn);
  } else {
    const int nmem = gridDim.x / a.NG;
    int g, mem;
    group_of(a.NG, nmem, &g, &mem);
    if (g >= 2 * a.NS) return;   // padding (see persist_groups)
    if (a.Tn > 1) group_arrive(a.words, a.seq, g, mem, a.wait);
    if (bwd32_pass<NCB, RT, KS, false, false>(a, lds_raw, g, mem, nmem, 0, a.Tn) != GROUP_ALONE) return;
    if (threadIdx.x == 0) a.status[1] = 1;
    bwd32_alone<NCB, RT, KS>(kernel_args<Persist32Args>(), (lds_base_t)lds_raw, g, nmem);
  }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
namespace {
struct Plan32 {
  int ncb, rt, members, chunk;   // column blocks per member, row tiles, members per group, rows per launch
  int bks;                       // k parts of the backward
};
}  // namespace

// One member while its 4H gate rows fit (H up to 128: no exchange), of the
// least width that holds them (a 64-cell layer on 64-unit members halves each
// thread's cells and splits the products' k over all waves); else members as
// large as the registers allow, 64 units up to 256 cells, 32 above.  Slices of
// 4 rows while they all fit the chip at one workgroup per CU, then of 8, then
// of 16 (32-unit members only: the cell registers of wider ones spill more; of
// these the backward spills 18 registers), in as many launches as it takes.
static bool plan32(int H, int B, Plan32* p) {
  const int cus = std::min(persist_max_wg(), 256);   // the exchange buffer is sized for 256
  p->ncb = H <= 32 ? 2 : H <= 64 ? 4 : H <= 128 ? 8 : H <= 256 ? 4 : 2;
  p->members = (int)cdiv(H, 16 * p->ncb);
  p->bks = p->members == 1 ? (p->ncb == 8 ? 4 : 8) : p->ncb / 2;
  const int slices = cus / (2 * p->members);
  if (slices < 1) return false;
  const int top = p->ncb == 2 ? 4 : 2;
  p->rt = 1;
  while (p->rt < top && cdiv(B, 4 * p->rt) > slices) p->rt *= 2;
  p->chunk = (int)std::min<int64_t>(B, (int64_t)slices * 4 * p->rt);
  return true;
}

bool persist32_supported(int H) { return H % 16 == 0 && H >= 16 && H <= 512; }

int persist32_rows_per_workgroup(int H, int B) {
  Plan32 p;
  return plan32(H, B, &p) ? 4 * p.rt : 16;
}

size_t persist32_xch_bytes(int B, int H) {
  if (!persist32_supported(H) || H <= 128) return 0;
  // as many rows per launch as the largest slices allow on 256 CUs
  const int ncb = H <= 256 ? 4 : 2;
  const int64_t members = cdiv(H, 16 * ncb);
  const int64_t rows = std::min<int64_t>(B, 256 / (2 * members) * (ncb == 2 ? 16 : 8));
  return (size_t)2 * 2 * members * (ncb / 2) * rows * H * 8 + GROUP_WORDS * 8;
}

size_t persist32_state_bytes(int B, int H) {
  if (!persist32_supported(H) || H <= 128) return 0;
  const int64_t members = cdiv(H, H <= 256 ? 64 : 32);
  return (size_t)(2 * std::min<int64_t>(cdiv(B, 4), 256 / (2 * members)) * members) * P32_THREADS * GROUP_STATE * 4;
}

hipError_t persist32_clear(bool backward, const Persist32Args& a, hipStream_t s) {
  Plan32 p;
  if (!plan32(a.H, a.B, &p)) return hipErrorInvalidValue;
  int64_t words = 0;   // one member exchanges nothing
  if (p.members > 1)
    words = GROUP_WORDS + (int64_t)2 * 2 * (backward ? p.members * p.bks : 1) * p.chunk * a.H;
  if (backward && words == 0) return hipSuccess;
  return persist_clear_words(a.words, words / 2, backward ? nullptr : a.status, s);
}

template <int NCB, int RT, int BKS, bool SOLO>
static const void* fn32(bool backward) {
  return backward ? (const void*)lstm_bwd_persist32<NCB, RT, BKS, SOLO> : (const void*)lstm_fwd_persist32<NCB, RT, SOLO>;
}

hipError_t persist32_layer(bool backward, Persist32Args a, hipStream_t s) {
  Plan32 p;
  if (!plan32(a.H, a.B, &p)) return hipErrorInvalidValue;
  const bool solo = p.members == 1;
  const void* fn = nullptr;
  switch (p.ncb * 100 + p.rt * 10 + (solo ? 1 : 0)) {
    case 210: fn = fn32<2, 1, 1, false>(backward); break;
    case 220: fn = fn32<2, 2, 1, false>(backward); break;
    case 240: fn = fn32<2, 4, 1, false>(backward); break;
    case 410: fn = fn32<4, 1, 2, false>(backward); break;
    case 420: fn = fn32<4, 2, 2, false>(backward); break;
    case 211: fn = fn32<2, 1, 8, true>(backward); break;
    case 221: fn = fn32<2, 2, 8, true>(backward); break;
    case 241: fn = fn32<2, 4, 8, true>(backward); break;
    case 411: fn = fn32<4, 1, 8, true>(backward); break;
    case 421: fn = fn32<4, 2, 8, true>(backward); break;
    case 811: fn = fn32<8, 1, 4, true>(backward); break;
    case 821: fn = fn32<8, 2, 4, true>(backward); break;
    default: return hipErrorInvalidValue;
  }
  const int RV = 4 * p.rt, ncol = 64 * p.ncb;
  size_t lds = backward ? ((size_t)2 * RV * (ncol + 16) + (size_t)p.bks * RV * 16 * p.ncb) * 4
                        : ((size_t)RV * p32_pitch(a.H) + (size_t)8 / p.ncb * RV * ncol) * 4;
  if (!backward) lds = std::max(lds, (size_t)8 * 64 * 36 * 4);   // W_hh staging
  const uint32_t wait = persist_group_wait();
  for (int b0 = 0; b0 < a.B; b0 += p.chunk) {
    Persist32Args c = a;
    c.b0 = b0;
    c.rows = std::min(p.chunk, a.B - b0);
    c.NS = (int)cdiv(c.rows, RV);
    c.NG = solo ? 2 * c.NS : persist_groups(2 * c.NS, p.members);
    // tags of one call's launches never meet: the launch's position times T,
    // plus the step (1 .. T); T B <= 2^24 keeps the product below 2^32
    c.seq = a.tag0 * (uint32_t)cdiv(a.B, p.chunk) + (uint32_t)(b0 / p.chunk);
    c.tag0 = c.seq * (uint32_t)a.Tn;
    c.wait = wait;
    const hipError_t e = persist_launch(backward ? "lstm_rec_bwd_persist32" : "lstm_rec_fwd_persist32", fn,
                                        dim3(c.NG * p.members), P32_THREADS, lds, &c, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

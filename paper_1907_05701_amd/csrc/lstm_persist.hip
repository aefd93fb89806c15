// Persistent recurrent kernels (bf16 operands): one launch runs all T steps
// of one layer, for both directions at once, and each workgroup keeps its
// slice of W_hh in registers for the whole chunk.
//
// Work split.  The batch is cut into slices of RV rows (8, 16 or 32: launch_rows),
// each on 16-row MFMA tiles; a group of NM = ceil(H/64) workgroups ("members")
// owns one (direction, slice) pair, and member m owns hidden units
// [64m, 64m + 64), i.e. 256 gate rows
// of W_hh (256 KB at H = 512: 128 VGPRs in each of the workgroup's 8
// waves).  Eight members per group instead of sixteen halves the chip-wide
// exchange volume of every step; at the paper's B = 128 a launch takes 256
// workgroups (2 directions x 16 slices of 8 rows x 8 members).
//   forward : wave (ub, kh) = (w % 4, w / 4) multiplies h_prev (all H units
//             of the slice, gathered from the members' published h) by the
//             four gates of the 16 units of block ub over the k half kh; the
//             two halves meet in LDS; the owning waves add the input
//             projection, apply the cell, publish h and write h, c and the
//             gate pre-activations for the backward.
//   backward: the gate derivatives of the member's 64 units (dc stays in
//             registers), then wave w multiplies the member's own da block
//             [16 x 256 own gate rows] by its W_hh rows for the unit blocks
//             w, w+8, w+16, w+24: partial dh_rec for all H units, published;
//             each member sums the NM partials of its own units in member
//             order.
//
// Step-to-step exchange without barriers or cache maintenance.  The values
// one member needs from the others (h, or partial dh) are published in an
// exchange buffer as 8-byte words holding four 15-bit values and a 4-bit
// tag (see h4_tag; the accesses: lstm_persist.hpp).  A word is written and
// read whole, so a reader that sees the expected tag in a word also sees that
// word's payload; readers poll the words they need (bounded; the status flag
// is set if a poll ever gives up).  Two slots alternate by step parity: a
// member overwrites a slot only after it has consumed the next step from
// every member, which those members produce only after they have consumed
// the slot's current contents.  The buffer is cleared once per forward or
// backward call, and the tag tells a word of the expected step from one of
// step n - 2 and from one left by either of the two previous launches of the
// call.  The members of a group start their steps only once all of them run
// (see group_meet); the launch is plain when the occupancy query shows that the
// whole grid fits on an idle device, cooperative otherwise (see persist_launch).
#include <stdlib.h>
#include <string.h>

#include "common.hpp"
#include "lstm_persist.hpp"
#include "dma.hpp"
#include "gemm_kc.hpp"

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

#define PU 64                 // hidden units per member
#define NTH 512               // threads per workgroup (8 waves)
// the LDS holds one workgroup: the compiler need not save registers for a
// second (the 32-row forward at B = 512: 373 -> 367 us for two layers)
#define ONE_PER_CU __attribute__((amdgpu_waves_per_eu(2, 2)))
#define KH_MAX 8              // forward: 32-deep k-steps per k half at H = 512
#define STAGE_BYTES (128 * 1024)   // W_hh staging buffer (half of a member's slice)
// backward: LDS offset of the summed dy (past the two da buffers)
__host__ __device__ constexpr int bwd_dy_lds(int RV) { return 2 * 32 * ((RV > 16 ? 32 : 16) + 1) * 16; }

// the value of lane l ^ 1 (a DPP quad permutation, no LDS round trip)
__device__ __forceinline__ float lane_xor1(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false));
}

__device__ __forceinline__ float lane_xor2(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, false));
}

// the value of lane l ^ 2
__device__ __forceinline__ uint32_t lane_xor2(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);
}

// Forward words: four bf16 h of one row
// (units 4i .. 4i+3, the first in the low half-word).  |h| = |o tanh(c)| <= 1,
// and a bf16 below 2 in magnitude has a zero top exponent bit (bit 14), so
// the four such bits carry a 4-bit tag: bit 0 always set (a cleared word
// never matches), bit 1 = bit 1 of the step number (a slot alternates
// between steps n and n - 2), bits 2-3 = the launch's sequence number in
// its call modulo 4 (a word can be left by one of the two launches before).
// Readers clear the four bits, so the exchanged values are exactly the bf16 of
// h.  A NaN would be clipped to a magnitude between 1 and 2, which no h has;
// where 64 does not divide H, readers give such a value its bit 14 back, so a
// NaN travels on as in the per-step kernels, which ran these widths before.
// (For the other widths it reaches the other members clipped, as it always has,
// while the layer output keeps it: the two instructions a word cost a 21-step
// launch at H = 512 1.5 to 5 us.)
#define H4_TAG_BITS 0x4000400040004000ull
template <bool NANS>
__device__ __forceinline__ uint64_t h4_decode(uint64_t w) {
  const uint64_t v = w & ~H4_TAG_BITS;
  if constexpr (!NANS) return v;
  // magnitude + 0x7F reaches bit 14 from 0x3F81 on (1.0 is 0x3F80), and no further
  return v | ((v + 0x007F007F007F007Full) & H4_TAG_BITS);
}
//
// BPTT words: four partial sums (rows 4i
// .. 4i+3 of one unit) in a 15-bit form that frees the same bits: the bf16
// of x * 2^-64 (so bf16 exponents 65 .. 190, i.e. 2^-62 <= |x| < 2^65, keep
// bit 14 clear and the 8-bit significand of the bf16 of x), with x * 2^-64
// clamped to +-(2 - 2^-7), the largest bf16 below 2: larger magnitudes and
// infinities saturate there, and a NaN becomes -(2 - 2^-7) (v_med3_f32
// returns the minimum of the non-NaN inputs when one is a quiet NaN); tiny
// values become bf16 subnormals.  Readers add the scaled values and
// multiply the sum by 2^64 (exact, as is every step of it: the scaled
// values stay below 2 in magnitude and bf16 subnormals add exactly).
// two bf16 values in one dword, `lo` in the low half
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{lo, hi}), bf16x2_t));   // one v_cvt_pk_bf16_f32
}
// the 15-bit form of four partial sums in one word (tag bits clear)
__device__ __forceinline__ uint64_t p15x4_encode(f32x4 v) {
  constexpr float M = 1.9921875f;   // bf16 0x3FFF
  float c[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) c[q] = __builtin_amdgcn_fmed3f(v[q] * 0x1p-64f, -M, M);
  const uint32_t lo = pack_bf16x2(c[0], c[1]), hi = pack_bf16x2(c[2], c[3]);
  return ((uint64_t)hi << 32) | lo;
}
// the four scaled partial sums of a word (x * 2^-64; tag bits ignored)
__device__ __forceinline__ f32x4 p15x4_decode_scaled(uint64_t w) {
  const uint32_t lo = (uint32_t)w & 0xBFFFBFFFu, hi = (uint32_t)(w >> 32) & 0xBFFFBFFFu;
  return f32x4{__builtin_bit_cast(float, lo << 16), __builtin_bit_cast(float, lo & 0xFFFF0000u),
               __builtin_bit_cast(float, hi << 16), __builtin_bit_cast(float, hi & 0xFFFF0000u)};
}
__device__ __forceinline__ uint64_t h4_tag(uint32_t seq, int n) {
  const uint32_t t = 1u | (((uint32_t)n >> 1 & 1u) << 1) | ((seq & 3u) << 2);
  return ((uint64_t)(t & 1u) << 14) | ((uint64_t)(t >> 1 & 1u) << 30) | ((uint64_t)(t >> 2 & 1u) << 46) |
         ((uint64_t)(t >> 3 & 1u) << 62);
}

// Polls the N words base[j * stride] (want: the expected tag bits; a word
// already holding `want` is never read) until every word carries the tag;
// gives up after PERSIST_SPIN_LIMIT polls, or at once when any wait anywhere has
// given up (the status flag is set), so every wave ends.
template <int N>
__device__ __forceinline__ void poll_words(uint64_t (&wv)[N], const uint64_t* base, int stride, uint64_t want,
                                           int* status) {
  for (unsigned it = 0;; ++it) {
    bool bad = false;
#pragma unroll
    for (int j = 0; j < N; ++j) bad |= (wv[j] & H4_TAG_BITS) != want;
    if (!bad) break;
    if (it > PERSIST_SPIN_LIMIT ||
        ((it & 63) == 63 && __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
      __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      break;
    }
    __builtin_amdgcn_s_sleep(1);
#pragma unroll
    for (int j = 0; j < N; ++j)
      if ((wv[j] & H4_TAG_BITS) != want) wv[j] = ll_load(base + (int64_t)j * stride);
  }
}

// lanes 32-63 of x replaced by lanes 0-31 of y (v_permlane32_swap_b32;
// lanes 0-31 of x are kept)
__device__ __forceinline__ float upper_from_lower(float x, float y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y),
                                                  false, false);
  return __builtin_bit_cast(float, r[0]);
}

// ---------------------------------------------------------------------------
// Input projection inside the forward launch (when the caller passes the
// layer input): before its steps, each workgroup computes
//   G_x[t][row][d 4H + q H + u0 + ul] = x[t][row] . W_ih[d][q H + u0 + ul] + b_ih + b_hh
// for its own RV rows at every step and its member's 256 gate columns
// (q < 4, ul < 64), the entries its own steps read.  The work is split
// evenly over the whole chip, with no launch of its own.  The sum runs as
// in the separate product: 64-deep k-tiles in ascending order, each on two
// v_mfma_f32_16x16x32_bf16 steps, the biases added to the float32 sum
// before the rounding to bf16; so the values are bit for bit the same.
// Rows (step, slice row) in passes of GXR; both operands staged by
// direct-to-LDS loads in the K-contiguous tile layout of gemm_kc.hpp (in
// the LDS that the W_hh staging and the steps use afterwards); wave w owns
// gate columns 32w .. 32w+31.
// ---------------------------------------------------------------------------
#define GXR 176   // rows per pass (11 MFMA row tiles)
// LDS of the projection: two stages of 64-deep k-tiles (x and W_ih rows of
// 128 bytes) and one scratch KB (the destination of load instructions that
// have no rows, so every wave issues as many loads per k-tile as every other
// and one vmcnt bound serves them all).  Measured on MI355X: 32-deep tiles
// in 3-5 stages, and a third W_ih stage, were slower.
#define GX_BK 64
#define GX_ST 2
static constexpr size_t gx_lds_bytes = (size_t)GX_ST * (GXR + 4 * PU) * 2 * GX_BK + 1024;
template <int RV>
__device__ __forceinline__ void gx_prologue(const PersistArgs& a, char* lds, int d, int u0, int rowbase, int rend) {
  constexpr int BK = GX_BK, ST = GX_ST, ROWB = 2 * BK, FM = GXR / 16, FN = 2;
  constexpr int CPR = ROWB / 16, RPI = 64 / CPR;      // 16-byte chunks per tile row, rows per load instruction
  constexpr int NA = GXR / RPI, NB = 4 * PU / RPI;    // load instructions per k-tile
  constexpr int QA = (NA + 7) / 8, QB = NB / 8;       // per wave
  constexpr int TA = GXR * ROWB, STG = (GXR + 4 * PU) * ROWB;
  static_assert(NB % 8 == 0 && GXR % RPI == 0, "tile rows split over the waves");
  static_assert(BK == 32 || BK == 64, "k-tile depth");
  const int H = a.H, B = a.B, K = a.Kin;
  const int rows = a.Tn * RV;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int fr = lane & 15, fc = lane >> 4;
  const int lr = lane / CPR, ls = lane % CPR;   // load lanes: row within the instruction, 16-byte slot
  char* scratch = lds + ST * STG;
  const __amdgpu_buffer_rsrc_t rx = dma_rsrc(a.Xin);
  const __amdgpu_buffer_rsrc_t rw = dma_rsrc(a.Wih + (d ? a.wih_d : 0));
  const int ntiles = (K + BK - 1) / BK;
  // W_ih rows of this lane's loads (instruction q 8 + w fills tile rows
  // RPI ins .. RPI ins + RPI - 1; tile row br is gate br / 64 of unit
  // u0 + br % 64)
  int64_t wrow[QB];   // negative: a unit past H (reads as zeros)
#pragma unroll
  for (int q = 0; q < QB; ++q) {
    const int br = (q * 8 + w) * RPI + lr;
    wrow[q] = u0 + (br & 63) < H ? ((int64_t)(br >> 6) * H + u0 + (br & 63)) * a.ldw : -1;
  }
  float bv[FN];
#pragma unroll
  for (int jn = 0; jn < FN; ++jn) {
    const int n = 32 * w + jn * 16 + fr;
    const int64_t gi = (d ? a.b_d : 0) + (int64_t)(n >> 6) * H + min(u0 + (n & 63), H - 1);
    float v = 0.f;
    v += a.bih[gi];
    v += a.bhh[gi];
    bv[jn] = v;
  }
  for (int m0 = 0; m0 < rows; m0 += GXR) {
    // frame rows of this lane's A loads
    int64_t xrow[QA];
    bool xok[QA];
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int ins = q * 8 + w;
      const int m = m0 + ins * RPI + lr;
      const int r = m % RV;
      xok[q] = ins < NA && m < rows && rowbase + r < rend;
      xrow[q] = xok[q] ? ((int64_t)(m / RV) * B + rowbase + r) * a.ldx : 0;
    }
    auto issue = [&](int j) {
      char* st = lds + (j % ST) * STG;
      const int64_t k0 = (int64_t)j * BK;
#pragma unroll
      for (int q = 0; q < QA; ++q) {
        const int ins = q * 8 + w;
        const int64_t k = k0 + kc_slot<BK>(ls, ins * RPI + lr) * 8;
        dma16(rx, xok[q] && k < K ? (uint32_t)((xrow[q] + k) * 2) : DMA_OFF_NONE,
              ins < NA ? st + ins * 1024 : scratch);
      }
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        const int ins = q * 8 + w;
        const int64_t k = k0 + kc_slot<BK>(ls, ins * RPI + lr) * 8;
        dma16(rw, k < K && wrow[q] >= 0 ? (uint32_t)((wrow[q] + k) * 2) : DMA_OFF_NONE, st + TA + ins * 1024);
      }
    };
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int jn = 0; jn < FN; ++jn) acc[i][jn] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < ST - 1; ++j)
      if (j < ntiles) issue(j);
    for (int j = 0; j < ntiles; ++j) {
      if (j + ST - 2 < ntiles)
        kc_wait_vm<(ST - 2) * (QA + QB)>();
      else
        kc_wait_vm<0>();
      __syncthreads();   // tile j in LDS; every wave is done with tile j - 1
      if (j + ST - 1 < ntiles) issue(j + ST - 1);
      const char* st = lds + (j % ST) * STG;
#pragma unroll
      for (int ks = 0; ks < BK / 32; ++ks) {
        bf16x8 bf[FN];
#pragma unroll
        for (int jn = 0; jn < FN; ++jn) {
          const int br = 32 * w + jn * 16 + fr;
          bf[jn] = *(const bf16x8*)(st + TA + br * ROWB + kc_slot<BK>(ks * 4 + fc, fr) * 16);
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const bf16x8 af = *(const bf16x8*)(st + (i * 16 + fr) * ROWB + kc_slot<BK>(ks * 4 + fc, fr) * 16);
#pragma unroll
          for (int jn = 0; jn < FN; ++jn) acc[i][jn] = Mfma<bf16>::mma(af, bf[jn], acc[i][jn]);
        }
      }
    }
    __syncthreads();   // the stages are free for the next pass
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int m = m0 + i * 16 + fc * 4 + rr;
        const int r = m % RV;
        if (m < rows && rowbase + r < rend) {
          bf16* o = a.Gx + ((int64_t)(m / RV) * B + rowbase + r) * 8 * H + (int64_t)d * 4 * H + u0;
#pragma unroll
          for (int jn = 0; jn < FN; ++jn) {
            const int n = 32 * w + jn * 16 + fr;
            if (u0 + (n & 63) < H) o[(n >> 6) * H + (n & 63)] = (bf16)(acc[i][jn][rr] + bv[jn]);
          }
        }
      }
  }
  // the projection stored (the steps read it back through the same CU's
  // cache) and the LDS free for the W_hh staging
  __syncthreads();
}

// The same entries for member columns u0 .. u0 + 63 without the LDS, for a
// group that runs alone (the same sums, so the same bits).
template <int RV>
__device__ __forceinline__ void gx_member(const PersistArgs& a, int d, int u0, int rowbase, int rend) {
  const int tid = pass_thread<true>(), lane = tid & 63, w = tid >> 6;
  const int fr = lane & 15, fc = lane >> 4;
  const int H = a.H, B = a.B, rows = a.Tn * RV;
  for (int tile = w; tile < (rows + 15) / 16 * 16; tile += 8) {
    const int m0 = (tile >> 4) * 16, n = (tile & 15) * 16 + fr, un = u0 + (n & 63);
    const int r = (m0 + fr) % RV;
    const bool xok = m0 + fr < rows && rowbase + r < rend, wok = un < H;
    const bf16* xr = a.Xin + (xok ? ((int64_t)((m0 + fr) / RV) * B + rowbase + r) * a.ldx : 0);
    const bf16* wr = a.Wih + (d ? a.wih_d : 0) + (wok ? ((int64_t)(n >> 6) * H + un) * a.ldw : 0);
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < a.Kin; k0 += 32) {
      const int k = k0 + fc * 8;
      const bf16x8 x = xok && k < a.Kin ? *(const bf16x8*)(xr + k) : Mfma<bf16>::zero();
      const bf16x8 v = wok && k < a.Kin ? *(const bf16x8*)(wr + k) : Mfma<bf16>::zero();
      acc = Mfma<bf16>::mma(x, v, acc);
    }
    const int64_t gi = (d ? a.b_d : 0) + (int64_t)(n >> 6) * H + min(un, H - 1);
    float bv = 0.f;
    bv += a.bih[gi];
    bv += a.bhh[gi];
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int m = m0 + fc * 4 + rr, ro = m % RV;
      if (m < rows && rowbase + ro < rend && wok)
        a.Gx[((int64_t)(m / RV) * B + rowbase + ro) * 8 * H + (int64_t)d * 4 * H + (n >> 6) * H + un] =
            (bf16)(acc[rr] + bv);
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Forward.
//
// RV rows of the batch per workgroup (8, 16 or 32) on 16-row MFMA tiles (with
// RV = 8 the tiles' rows 8-15 are zeros, and after the k halves meet the
// owner lanes swap the valid rows of lanes 0-31 into lanes 32-63, so that
// every lane applies the cell to 2 rows instead of 4).  With 32 rows the waves
// of k half kh own row tile kh; with fewer, sharing the cells between both
// halves measured slower (100.7 -> 127 us per 42 steps at RV = 8).
// ---------------------------------------------------------------------------
//
// One pass runs steps [tau0, tau1) of member `mem`: all of them with the
// group's other members beside it (ONE false; returns how the group runs, see
// group_meet, and does nothing if it does not run together), or one step of
// one member after the other (ONE, see lstm_fwd_persist), with the member's
// registers kept in a.state between its steps.
template <int RV, bool NANS, bool ONE>
__device__ __forceinline__ int fwd_pass(const PersistArgs& a, char* lds_raw, int g, int mem, int tau0, int tau1) {
  static_assert(RV == 8 || RV == 16 || RV == 32, "rows per workgroup");
  constexpr int NT = RV > 16 ? 2 : 1;   // MFMA row tiles
  constexpr int R = 16 * NT;            // LDS rows of h
  constexpr bool BOTH = RV == 32;       // both k halves' waves own cells
  constexpr int NR = RV == 8 ? 2 : 4;   // cell rows per owner lane
  const int H = a.H, B = a.B, Tn = a.Tn;
  const int d = g & 1, s = g >> 1;
  const int u0 = mem * PU;
  const int tid = pass_thread<ONE, (RV < 32)>(), lane = tid & 63, w = tid >> 6;
  const int ub = w & 3, kh = w >> 2;
  const int NM = (H + PU - 1) / PU, HP = NM * PU;   // members; units with the last member's padding
  const int KH = NM;                                // 32-deep k-steps per k half
  const bool owner = BOTH || kh == 0;

  // W_hh fragments (B operand): gate q of unit u0 + ub*16 + lane%16, k-step
  // kh*KH + i, k = 8*(lane/16) .. +8 within it.  Staged by direct-to-LDS
  // loads one k half at a time: 256 local rows lr = q*64 + b*16 + u (gate q,
  // unit u0 + 16b + u), 512 bytes each (k past the half read as zeros), the
  // 16-byte chunk c of row lr in slot c ^ (lr & 15) so that the 16 rows of
  // one fragment read fall in distinct bank groups.
  bf16x8 bw[KH_MAX][4];
  int how = GROUP_APART;
  const bool meets = Tn > 1 && NM > 1;
  uint64_t word = 0;   // (asked for while the staging loads are in flight)
  {
    char* stg = lds_raw;
    const __amdgpu_buffer_rsrc_t rw = dma_rsrc(a.W + (d ? a.whh1 : a.whh0));
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        // one instruction fills rows 2 ins, 2 ins + 1 (w < 8: said, it shortens the masks)
        const int ins = q * 8 + (w & 7);
        const int lr = ins * 2 + (lane >> 5);
        const int c = (lane & 31) ^ (lr & 15);      // chunk held by this lane's slot
        const int un = u0 + ((lr >> 4) & 3) * 16 + (lr & 15), k = p * (HP / 2) + c * 8;
        const int64_t grow = (int64_t)(lr >> 6) * H + un;
        const bool ok = c * 8 < HP / 2 && k < H && un < H;
        dma16(rw, ok ? (uint32_t)((grow * H + k) * 2) : DMA_OFF_NONE, stg + ins * 1024);
      }
      dma_wait_all();
      __syncthreads();
      if (!ONE && p == 1 && meets) word = group_word(a.words, a.seq, g);
      if (kh == p) {
#pragma unroll
        for (int i = 0; i < KH_MAX; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int lr = q * 64 + ub * 16 + (lane & 15);
            const int c = min(i, KH - 1) * 4 + (lane >> 4);
            bw[i][q] = *(const bf16x8*)(stg + lr * 512 + (c ^ (lr & 15)) * 16);
          }
      }
      __syncthreads();   // the next half (then the step buffers) reuse this LDS
    }
  }

  // LDS during the steps: gathered h [HP/8][R + 1][8] (MFMA A layout; rows
  // RV..15 and units past H stay zero), the k-half partial sums, and step buffers (by step
  // parity) of c [RV][64] (float), h [RV][64] and gate pre-activations
  // [RV][64][4] (bf16), staged for 16-byte stores
  const int rend = a.b0 + a.rows;
  const int rowbase = a.b0 + s * RV;
  bf16* hl = (bf16*)lds_raw;
  f32x4* red = (f32x4*)(lds_raw + (size_t)(HP / 8) * (R + 1) * 16);   // [receiving half][4 unit blocks][4 gates][64]
  char* stage0 = (char*)(red + (BOTH ? 2 : 1) * 4 * 4 * 64);
  constexpr int STEP_STAGE = RV * PU * (4 + 2 + 8);
  auto stC = [&](int par) { return (float*)(stage0 + par * STEP_STAGE); };
  auto stY = [&](int par) { return (bf16*)(stage0 + par * STEP_STAGE + RV * PU * 4); };
  auto stG = [&](int par) { return (bf16*)(stage0 + par * STEP_STAGE + RV * PU * 6); };
  // c, h and the gates of step tt in 16-byte pieces (the NT threads from
  // first): per row, the 64 units x 4 gates are 512 contiguous bytes (32
  // pieces), c 256 bytes (16) and h 128 bytes (8)
  auto store_step = [&](int tt, int par, int first, int nt) {
    const float* sC = stC(par);
    const bf16* sY = stY(par);
    const bf16* sG = stG(par);
    for (int pc = tid - first; pc < RV * 56; pc += nt) {
      if (pc < RV * 32) {
        const int rl = pc >> 5, c = pc & 31;
        if (rowbase + rl < rend && u0 + c * 2 < H)
          *(uint4*)(a.G + ((int64_t)tt * B + rowbase + rl) * 8 * H + (int64_t)d * 4 * H + (int64_t)u0 * 4 + c * 8) =
              *(const uint4*)&sG[rl * PU * 4 + c * 8];
      } else if (pc < RV * 48) {
        const int rl = (pc - RV * 32) >> 4, c = (pc - RV * 32) & 15;
        if (rowbase + rl < rend && u0 + c * 4 < H)
          *(float4*)(a.C + ((int64_t)tt * B + rowbase + rl) * 2 * H + (int64_t)d * H + u0 + c * 4) =
              *(const float4*)&sC[rl * PU + c * 4];
      } else {
        const int rl = (pc - RV * 48) >> 3, c = (pc - RV * 48) & 7;
        if (rowbase + rl < rend && u0 + c * 8 < H)
          *(uint4*)(a.Y + ((int64_t)tt * B + rowbase + rl) * 2 * H + (int64_t)d * H + u0 + c * 8) =
              *(const uint4*)&sY[rl * PU + c * 8];
      }
    }
  };
  if (RV < R || HP > H)
    for (int i = tid; i < (HP / 8) * (R + 1); i += NTH) *(uint4*)&hl[i * 8] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();

  const int unit = u0 + ub * 16 + (lane & 15);
  const int wpr = H / 4;   // exchange words per row
  const int64_t slot_stride = (int64_t)2 * a.rows * wpr;
  // the slice rows of an owner lane's NR cell rows
  auto lrow = [&](int r) {
    return RV == 8 ? ((lane >> 4) & 1) * 4 + (lane >> 5) * 2 + r : (BOTH ? kh * 16 : 0) + (lane >> 4) * 4 + r;
  };

  if (!ONE && meets) how = group_meet(word, a.words, a.seq, g, mem, NM, a.wait);
  if (!ONE && how >= GROUP_ALONE) return how;
  const bool local = how == GROUP_LOCAL;
  float creg[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) creg[r] = ONE && tau0 > 0 ? group_state(a.state, g, mem, NM)[r] : 0.f;

  // input projection of a step (independent of h), loaded one step ahead so
  // that its latency hides behind the previous step's exchange
  bf16 gxn[NR][4];
  auto load_gx = [&](int tt) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int row = rowbase + lrow(r);
      const bf16* p =
          a.Gx + ((int64_t)tt * B + (row < rend ? row : a.b0)) * 8 * H + (int64_t)d * 4 * H + min(unit, H - 1);
#pragma unroll
      for (int q = 0; q < 4; ++q) gxn[r][q] = p[q * H];
    }
  };
  if (owner) load_gx(d ? Tn - 1 - tau0 : tau0);

  constexpr int NGT = NTH;   // gathering threads
  constexpr int WPT = (RV * 128 + NGT - 1) / NGT;     // gathered words per thread (at H = 512)
  for (int tau = tau0; tau < tau1; ++tau) {
    const int t = d ? Tn - 1 - tau : tau;

    f32x4 acc[NT][4];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[i][q] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (tau > 0) {
      // h of the previous step (RV rows x H/4 words of this slice, contiguous
      // in the exchange buffer), polled by the gathering threads in whole
      // cache lines and staged in LDS in the MFMA A layout
      if (tid < NGT) {
        const int nwords = RV * wpr;
        const uint64_t* src = a.X + ((tau - 1) & 1) * slot_stride + ((int64_t)d * a.rows + (rowbase - a.b0)) * wpr;
        const uint64_t want = h4_tag(a.seq, tau);
        uint64_t wv[WPT];
#pragma unroll
        for (int j = 0; j < WPT; ++j) {
          const int idx = tid + NGT * j;
          const bool ok = idx < nwords && rowbase + idx / wpr < rend;
          wv[j] = ok ? ll_load(src + idx) : want;
        }
        poll_words<WPT>(wv, src + tid, NGT, want, a.status);
#pragma unroll
        for (int j = 0; j < WPT; ++j) {
          const int idx = tid + NGT * j;
          if (idx >= nwords) break;
          const int row = idx / wpr, wc = idx % wpr;   // units 4 wc .. 4 wc + 3
          const bool ok = rowbase + row < rend;
          *(uint64_t*)&hl[((wc >> 1) * (R + 1) + row) * 8 + 4 * (wc & 1)] = ok ? h4_decode<NANS>(wv[j]) : 0ull;
        }
      }
      lds_barrier();
#pragma unroll
      for (int i = 0; i < KH_MAX; ++i) {
        if (i >= KH) break;
        const int kg = (kh * KH + i) * 4 + (lane >> 4);
#pragma unroll
        for (int tl = 0; tl < NT; ++tl) {
          const bf16x8 af = *(const bf16x8*)&hl[(kg * (R + 1) + tl * 16 + (lane & 15)) * 8];
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[tl][q] = Mfma<bf16>::mma(af, bw[i][q], acc[tl][q]);
        }
      }
    }
    // the two k halves meet at the owner (k half 0; with two row tiles, k half
    // kh owns tile kh)
    if (BOTH || !owner) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        red[((BOTH && kh == 0 ? 16 : 0) + ub * 4 + q) * 64 + lane] = BOTH && kh ? acc[0][q] : acc[NT - 1][q];
    }
    lds_barrier();
    if (owner) {
      // cell math of all owned rows, then h published (the other members
      // wait for it), then the saved activations (only read after the launch)
      uint64_t* xo = a.X + (tau & 1) * slot_stride;
      f32x4 pre[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        pre[q] = (BOTH && kh ? acc[NT - 1][q] : acc[0][q]) + red[((BOTH ? kh * 16 : 0) + ub * 4 + q) * 64 + lane];
        if constexpr (RV == 8) {
          // rows 2, 3 (lanes 0-15) and 6, 7 (lanes 16-31) into lanes 32-63
          pre[q][0] = upper_from_lower(pre[q][0], pre[q][2]);
          pre[q][1] = upper_from_lower(pre[q][1], pre[q][3]);
        }
      }
      float hv[NR], gv[NR][4];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
#pragma unroll
        for (int q = 0; q < 4; ++q) gv[r][q] = pre[q][r] + (float)gxn[r][q];
        const float ig = sigmoidf_(gv[r][0]), fg = sigmoidf_(gv[r][1]);
        const float gg = tanhf_(gv[r][2]), og = sigmoidf_(gv[r][3]);
        const float c = fg * creg[r] + ig * gg;
        creg[r] = c;
        hv[r] = og * tanhf_(c);
      }
      // every row's h before the first publish (the empty asm pins the
      // values here, so the compiler cannot sink their math past a publish)
#pragma unroll
      for (int r = 0; r < NR; ++r) __asm__ volatile("" : "+v"(hv[r]));
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int row = rowbase + lrow(r);
        const float h_next_unit = lane_xor1(hv[r]);   // lanes of one row, units u and u^1
        // lane 4i stores units 4i .. 4i+3 (the pairs of lanes 4i and 4i+2)
        const uint32_t p2 = pack_bf16x2(hv[r], h_next_unit);
        const uint32_t p4 = lane_xor2(p2);
        if (row < rend && unit < H && (lane & 3) == 0)
          ll_store64(xo + ((int64_t)d * a.rows + (row - a.b0)) * wpr + unit / 4,
                     ((((uint64_t)p4 << 32) | p2) & ~H4_TAG_BITS) | h4_tag(a.seq, tau + 1), local);
      }
      // into LDS; the whole workgroup writes them out after the barrier
      const int ul = ub * 16 + (lane & 15);
      float* sC = stC(tau & 1);
      bf16* sY = stY(tau & 1);
      bf16* sG = stG(tau & 1);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int rl = lrow(r);
        sC[rl * PU + ul] = creg[r];
        sY[rl * PU + ul] = (bf16)hv[r];
        bf16x4 g4;
#pragma unroll
        for (int q = 0; q < 4; ++q) g4[q] = (bf16)gv[r][q];
        *(bf16x4*)&sG[(rl * PU + ul) * 4] = g4;
      }
      if (tau + 1 < tau1) load_gx(d ? Tn - 2 - tau : tau + 1);
    }
    // the step's saved activations by the whole workgroup (the next step's
    // gather barrier comes before this buffer is rewritten)
    lds_barrier();
    store_step(t, tau & 1, 0, NTH);
  }
  if constexpr (ONE) {
#pragma unroll
    for (int r = 0; r < NR; ++r) group_state(a.state, g, mem, NM)[r] = creg[r];
    __syncthreads();   // the next pass reuses the LDS
  }
  return how;
}

// A group that runs on this workgroup alone: every member's input projection,
// then every member's part of each step.
template <int RV, bool NANS>
__device__ __attribute__((noinline)) void fwd_alone(const PersistArgs* at, lds_base_t lds, int gv, int memv) {
  char* lds_raw = (char*)lds;
  const int g = scalar(gv), mem = scalar(memv);
  const PersistArgs a = pass_args(at);
  const int NM = (a.H + PU - 1) / PU;
  if (a.Xin)
#pragma nounroll
    for (int m = 0; m < NM; ++m)
      if (m != mem) gx_member<RV>(pass_args(at), g & 1, m * PU, a.b0 + (g >> 1) * RV, a.b0 + a.rows);
#pragma nounroll
  for (int tau = 0; tau < a.Tn; ++tau)
#pragma nounroll
    for (int m = 0; m < NM; ++m) fwd_pass<RV, NANS, true>(pass_args(at), lds_raw, g, m, tau, tau + 1);
}

template <int RV, bool NANS>
__global__ __launch_bounds__(NTH) ONE_PER_CU void lstm_fwd_persist(const PersistArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  const int NM = (a.H + PU - 1) / PU;
  int g, mem;
  group_of(a.NG, NM, &g, &mem);
  if (g >= 2 * a.NS) return;   // padding (see persist_groups)
  if (a.Tn > 1 && NM > 1) group_arrive(a.words, a.seq, g, mem, a.wait);
  if (a.Xin) gx_prologue<RV>(a, lds_raw, g & 1, mem * PU, a.b0 + (g >> 1) * RV, a.b0 + a.rows);
  if (fwd_pass<RV, NANS, false>(a, lds_raw, g, mem, 0, a.Tn) != GROUP_ALONE) return;
  if (threadIdx.x == 0) a.status[1] = 1;
  fwd_alone<RV, NANS>(kernel_args<PersistArgs>(), (lds_base_t)lds_raw, g, mem);
}

// ---------------------------------------------------------------------------
// Backward (BPTT).
//
// dh_rec[b][j] = sum over all 4H gate rows g of da[b][g] W_hh[g][j].  Member
// m owns the 256 gate rows of its 64 units, so it computes the partial sums
// P_m = da[:, own rows] W_hh[own rows, :] for ALL H units from data it
// already holds (its own da in LDS, its W_hh rows in registers), publishes
// P_m as exchange words, and gathers for its own 64 units the partials of
// all members.  An exchange word holds one unit's partials for four adjacent
// rows; words are ordered (row quad, member, unit), so a member publishes
// whole cache lines and a reader takes 512 contiguous bytes of each member.
// RV rows per workgroup (8, 16 or 32) on 16-row MFMA tiles (with RV = 8 the
// da block's rows 8-15 stay zero).
//
// Every thread gathers and owns cells: the LPI = 32 / RV adjacent lanes of
// one (row quad, unit) take 8 / LPI members' words each, add them in member
// order, and swap partial sums with DPP so that each lane ends with the
// total of its 4 / LPI rows, whose cells it then computes.  So the gathered
// sums never pass through LDS and a step has one barrier (own da complete).
//
// F32X: the partial sums travel as float32, one word each (row quad, member,
// row, unit; a 32-bit tag): four times the words, for the widths that 64 does
// not divide, whose recurrence has always kept them in float32 (the per-step
// kernels, which ran these widths before at 6.1 / 11.9 us a step for H = 96 /
// 480, B = 128, T = 21; now 2.2 / 4.1, and the forward 5.3 / 7.4 -> 1.9 / 2.8).
// ---------------------------------------------------------------------------
//
// Passes as in the forward.
template <int RV, bool F32X, bool ONE>
__device__ __forceinline__ int bwd_pass(const PersistArgs& a, char* lds_raw, int g, int mem, int tau0, int tau1) {
  static_assert(RV == 8 || RV == 16 || RV == 32, "rows per workgroup");
  constexpr int NT = RV > 16 ? 2 : 1;   // MFMA row tiles
  constexpr int R = 16 * NT;            // LDS rows of da
  constexpr int LPI = 32 / RV;          // lanes per (row quad, unit)
  constexpr int RPT = 4 / LPI;          // cell rows per lane
  constexpr int MPL = 8 / LPI;          // members' words per lane (at most)
  const int H = a.H, B = a.B, Tn = a.Tn;
  const int NM = (H + PU - 1) / PU;
  const int d = g & 1, s = g >> 1;
  const int u0 = mem * PU;
  const int tid = pass_thread<ONE>(), lane = tid & 63, w = tid >> 6;
  const int NB = H / 16;                // unit blocks of the partial product

  // W_hh of the 256 own gate rows as the B operand: k = own row kk (gate
  // (kk>>4)&3, unit u0 + (kk>>6)*16 + (kk&15)), n = unit.  Wave w holds the
  // unit blocks nb = w + 8j (j < 4) for all 8 k-steps.  Staged from W_hh as
  // it lies, 128 own rows at a time, by direct-to-LDS loads ([kk][512
  // units], 1 KB rows, the 16-byte chunk c of row kk in slot c ^ wswz(kk);
  // units past H read as zeros), then each lane takes its fragments with
  // transposing LDS reads (ds_read_b64_tr_b16: in a 16-lane group lane r
  // addresses 4 consecutive units of k row r/4 and receives unit column r's
  // values over those 4 rows; two reads give the 8 consecutive k of the
  // MFMA B operand).  The swizzle spreads the 16 rows of one read over
  // distinct chunk pairs.
  bf16x8 bw[8][4];
  int how = GROUP_APART;
  const bool meets = Tn > 1 && NM > 1;
  uint64_t word = 0;
  {
    auto wswz = [](int k) { return 2 * ((k & 3) | (((k >> 3) & 1) << 2)); };
    char* stg = lds_raw;
    const __amdgpu_buffer_rsrc_t rw = dma_rsrc(a.W + (d ? a.whh1 : a.whh0));
    const int gq = lane >> 4, r = lane & 15;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int kl = q * 8 + w;   // one 1 KB row per load instruction
        const int kk = p * 128 + kl;
        const int c = lane ^ wswz(kl);
        const int un = u0 + (kk >> 6) * 16 + (kk & 15);
        const int64_t grow = (int64_t)((kk >> 4) & 3) * H + un;
        dma16(rw, c * 8 < H && un < H ? (uint32_t)((grow * H + c * 8) * 2) : DMA_OFF_NONE, stg + kl * 1024);
      }
      dma_wait_all();
      __syncthreads();
      if (!ONE && p == 1 && meets) word = group_word(a.words, a.seq, g);
#pragma unroll
      for (int ksl = 0; ksl < 4; ++ksl)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int mn = (w + 8 * j) * 16 + 4 * (r & 3);
          bf16x4 h[2];
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const int k = ksl * 32 + 8 * gq + 4 * hh + (r >> 2);
            const char* pa = stg + k * 1024 + ((mn >> 3) ^ wswz(k)) * 16 + (mn & 7) * 2;
            h[hh] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)(pa));
          }
          bw[4 * p + ksl][j] = bf16x8{h[0][0], h[0][1], h[0][2], h[0][3], h[1][0], h[1][1], h[1][2], h[1][3]};
        }
      __syncthreads();   // the next rows (then the step buffers) reuse this LDS
    }
  }

  // LDS during the steps: own da as the A operand, by step parity
  // [2][32 k groups][R + 1][8] (k = own row; with RV = 8 rows 8..15 stay
  // zero), and with dy given as partial sums, the summed dy of every step
  // [T][RV][64] behind them
  constexpr int ALS = 32 * (R + 1) * 8;
  bf16* al0 = (bf16*)lds_raw;
  float* dyl = (float*)(lds_raw + bwd_dy_lds(RV));
  if constexpr (RV < R) {
    for (int i = tid; i < 2 * 32 * (R - RV); i += NTH)
      *(uint4*)&al0[((i / (R - RV)) * (R + 1) + RV + i % (R - RV)) * 8] = make_uint4(0u, 0u, 0u, 0u);
  }

  const int rend = a.b0 + a.rows;
  const int rowbase = a.b0 + s * RV;
  const int rquads = (a.rows + 3) / 4;             // row quads of this launch
  constexpr int WPQ = F32X ? 4 : 1;                // words per (row quad, member, unit)
  const int64_t slot_stride = (int64_t)2 * rquads * NM * H * WPQ;
  // this lane's item: unit cu of row quad qd, rows rl0 .. rl0 + RPT - 1
  const int sub = tid % LPI, item = tid / LPI;
  const int cu = item & 63, qd = item >> 6, rl0 = qd * 4 + sub * RPT;
  if (!ONE && meets) how = group_meet(word, a.words, a.seq, g, mem, NM, a.wait);
  if (!ONE && how >= GROUP_ALONE) return how;
  const bool local = how == GROUP_LOCAL;
  float dcreg[RPT], dbacc[4];
#pragma unroll
  for (int i = 0; i < RPT; ++i) dcreg[i] = ONE && tau0 > 0 ? group_state(a.state, g, mem, NM)[4 + i] : 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) dbacc[q] = ONE && tau0 > 0 ? group_state(a.state, g, mem, NM)[q] : 0.f;

  // everything the cell derivative needs besides dh_rec: dy, the gate
  // pre-activations and c at t, c at the step's predecessor in forward time
  // (which is the next step's t).  Fetched one step ahead, right after the
  // previous step's gather, so that no gather waits for them; c at t is the
  // previous step's predecessor value.  Per-row element offsets are fixed
  // (32-bit, row and unit); a step adds its frame base to the pointers.
  float dyn[RPT], cpn[RPT], cc[RPT];
  bf16x4 gtn[RPT];
  uint32_t oc[RPT];   // cell offsets into [B][2H] frames (C, DY); 4 oc into [B][2H][4] (G)
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    int row = rowbase + rl0 + i;
    row = row < rend ? row : a.b0;
    oc[i] = (uint32_t)(row * 2 * H + d * H + min(u0 + cu, H - 1));
  }
  const int64_t fc = (int64_t)B * 2 * H, fg = (int64_t)B * 8 * H;   // elements per frame
  if (a.ndy > 0) {
    // dy of the slice at every step, [T][RV][64] in LDS: the partial sums
    // added in split order, four units per 16-byte load (item = step, row,
    // unit quad); DYI items per thread at a time with all their loads (up
    // to three partials each) issued together
    constexpr int DYI = 3;
    const int nitems = Tn * RV * (PU / 4);
    for (int i0 = 0; i0 < nitems; i0 += DYI * NTH) {
      float4 v[DYI][3];
#pragma unroll
      for (int j = 0; j < DYI; ++j) {
        const int it = min(i0 + j * NTH + tid, nitems - 1);
        const int rs = it >> 4, t_ = rs / RV, r = rs % RV;
        const int row = rowbase + r < rend ? rowbase + r : a.b0;
        const float* p = a.DYP + (int64_t)t_ * fc + (int64_t)row * 2 * H + d * H + min(u0 + (it & 15) * 4, H - 4);
#pragma unroll
        for (int k = 0; k < 3; ++k) v[j][k] = *(const float4*)(p + (int64_t)min(k, a.ndy - 1) * a.dy_kstride);
      }
#pragma unroll
      for (int j = 0; j < DYI; ++j) {
        const int it = i0 + j * NTH + tid;
        if (it >= nitems) break;
        const int rs = it >> 4, t_ = rs / RV, r = rs % RV;
        float4 sum = v[j][0];
#pragma unroll
        for (int k = 1; k < 3; ++k)
          if (k < a.ndy) { sum.x += v[j][k].x; sum.y += v[j][k].y; sum.z += v[j][k].z; sum.w += v[j][k].w; }
        for (int k = 3; k < a.ndy; ++k) {
          const int row = rowbase + r < rend ? rowbase + r : a.b0;
          const float4 w4 = *(const float4*)(a.DYP + (int64_t)k * a.dy_kstride + (int64_t)t_ * fc +
                                             (int64_t)row * 2 * H + d * H + min(u0 + (it & 15) * 4, H - 4));
          sum.x += w4.x; sum.y += w4.y; sum.z += w4.z; sum.w += w4.w;
        }
        if (!(rowbase + r < rend)) sum = make_float4(0.f, 0.f, 0.f, 0.f);
        *(float4*)&dyl[(t_ * RV + r) * PU + (it & 15) * 4] = sum;
      }
    }
    __syncthreads();
  }
  auto fetch = [&](int tau_) {
    const int t_ = d ? tau_ : Tn - 1 - tau_;
    const int tp_ = d ? t_ + 1 : t_ - 1;
    const bool hp = tp_ >= 0 && tp_ < Tn;
    const float* dyt = a.DY + t_ * fc;
    const float* cpt = a.C + (hp ? tp_ : 0) * fc;
    const bf16* gt = a.G + t_ * fg;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      dyn[i] = a.ndy > 0 ? dyl[(t_ * RV + rl0 + i) * PU + cu] : dyt[oc[i]];
      cpn[i] = hp ? cpt[oc[i]] : 0.f;
      gtn[i] = *(const bf16x4*)(gt + 4 * oc[i]);   // the unit's four gates: one 8-byte load
    }
  };
  {
    const float* ct = a.C + (d ? tau0 : Tn - 1 - tau0) * fc;
#pragma unroll
    for (int i = 0; i < RPT; ++i) cc[i] = ct[oc[i]];
  }
  fetch(tau0);

  const int m0 = sub * MPL, mcount = max(0, min(NM, m0 + MPL) - m0);
  const uint32_t ogath =
      (uint32_t)((((int64_t)d * rquads + (rowbase - a.b0) / 4 + qd) * NM + m0) * WPQ * H + u0 + cu);
  // word offset (within a slot) of the first published word; unit block j and
  // row tile tl are 128 j units and 4 tl row quads further
  const uint32_t opub = (uint32_t)((((int64_t)d * rquads + (rowbase - a.b0) / 4 + (lane >> 4)) * NM + mem) * WPQ * H +
                                   w * 16 + (lane & 15));
  const uint32_t tag0 = a.seq * (uint32_t)Tn + 1;   // F32X: + step; launches of a call never meet (T B <= 2^24)
  // da out: pieces of 8 own gate rows of one row
  constexpr int NDT = RV == 8 ? NTH / 2 : NTH;   // threads writing DA: waves 4-7 when that is one piece each
  constexpr int NDA = 32 * RV / NDT;
  const int dtid = tid - (NTH - NDT);
  uint32_t oda[NDA];
#pragma unroll
  for (int c0 = 0; c0 < NDA; ++c0) {
    const int c = c0 * NDT + max(dtid, 0), kk = (c & 31) * 8, r = c >> 5;
    oda[c0] = (uint32_t)((rowbase + r) * 8 * H + d * 4 * H + ((kk >> 4) & 3) * H + u0 + (kk >> 6) * 16 + (kk & 15));
  }

  for (int tau = tau0; tau < tau1; ++tau) {
    const int t = d ? tau : Tn - 1 - tau;
    bf16* al = al0 + (tau & 1) * ALS;
    // the step's gate activations from the prefetched pre-activations,
    // before the gather (whose polls wait for the other members anyway)
    float ga[RPT][4], tc[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      ga[i][0] = sigmoidf_((float)gtn[i][0]);
      ga[i][1] = sigmoidf_((float)gtn[i][1]);
      ga[i][2] = tanhf_((float)gtn[i][2]);
      ga[i][3] = sigmoidf_((float)gtn[i][3]);
      tc[i] = tanhf_(cc[i]);
    }

    float dhr[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) dhr[i] = 0.f;
    if (tau > 0) {
      const uint64_t* base = a.X + ((tau - 1) & 1) * slot_stride + ogath;
      const uint64_t want = h4_tag(a.seq, tau);
      f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
      if (rowbase + 4 * qd < rend && u0 + cu < H) {
        if constexpr (F32X) {
          // two members (eight words) at a time
#pragma unroll
          for (int k0 = 0; k0 < MPL; k0 += 2) {
            uint64_t wv[8];
            uint32_t off[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const bool ok = k0 + j / 4 < mcount;
              off[j] = ok ? (uint32_t)(((k0 + j / 4) * 4 + j % 4) * H) : 0;
              wv[j] = ok ? ll_load(base + off[j]) : (uint64_t)(tag0 + tau) << 32;
            }
            poll_tagged<8>(wv, base, off, tag0 + tau, a.status);
#pragma unroll
            for (int j = 0; j < 8; ++j) sum[j % 4] += __builtin_bit_cast(float, (uint32_t)wv[j]);
          }
        } else {
          uint64_t wv[MPL];
#pragma unroll
          for (int k = 0; k < MPL; ++k) wv[k] = k < mcount ? ll_load(base + (int64_t)k * H) : want;
          poll_words<MPL>(wv, base, H, want, a.status);
#pragma unroll
          for (int k = 0; k < MPL; ++k)
            if (k < mcount) sum += p15x4_decode_scaled(wv[k]);
          sum *= 0x1p64f;
        }
      }
      // the lanes of one (row quad, unit) add their members' sums
      if constexpr (LPI == 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) dhr[i] = sum[i];
      } else if constexpr (LPI == 2) {
        const bool hi = sub & 1;
        dhr[0] = (hi ? sum[2] : sum[0]) + lane_xor1(hi ? sum[0] : sum[2]);
        dhr[1] = (hi ? sum[3] : sum[1]) + lane_xor1(hi ? sum[1] : sum[3]);
      } else {
        const bool hi = sub & 2, odd = sub & 1;
        const float k0 = (hi ? sum[2] : sum[0]) + lane_xor2(hi ? sum[0] : sum[2]);
        const float k1 = (hi ? sum[3] : sum[1]) + lane_xor2(hi ? sum[1] : sum[3]);
        dhr[0] = (odd ? k1 : k0) + lane_xor1(odd ? k0 : k1);
      }
    }
    float dy[RPT], cp[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      dy[i] = dyn[i];
      cp[i] = cpn[i];
    }

    // cell derivatives; da goes to LDS (next partial product) and from there
    // to global memory (weight and input gradients)
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = rl0 + i;
      const float ig = ga[i][0], fg_ = ga[i][1], gg = ga[i][2], og_ = ga[i][3];
      const float dh = dhr[i] + dy[i];
      const float dc = dh * og_ * (1.f - tc[i] * tc[i]) + dcreg[i];
      dcreg[i] = dc * fg_;
      float da[4];
      da[0] = dc * gg * ig * (1.f - ig);
      da[1] = dc * cp[i] * fg_ * (1.f - fg_);
      da[2] = dc * ig * (1.f - gg * gg);
      da[3] = dh * tc[i] * og_ * (1.f - og_);
      const bool ok = rowbase + r < rend && u0 + cu < H;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float dq = ok ? da[q] : 0.f;
        // own row kk = (cu >> 4)*64 + q*16 + (cu & 15)
        const int kk = (cu >> 4) * 64 + q * 16 + (cu & 15);
        al[((kk >> 3) * (R + 1) + r) * 8 + (kk & 7)] = (bf16)dq;
        dbacc[q] += dq;   // the bias gradient sums da before it is rounded
      }
      cc[i] = cp[i];   // c at the next step's t
    }
    if (tau + 1 < tau1) fetch(tau + 1);
    lds_barrier();

    // P = da_own [RV x 256] * W_own [256 x H]; unit blocks w + 8j of this
    // wave.  On the critical path, so before the global copies of da.
    if (tau + 1 < Tn) {
      uint64_t* xo = a.X + (tau & 1) * slot_stride;
      const uint64_t tg = h4_tag(a.seq, tau + 1);
      // one row tile after the other, the first one's words on their way
      // while the second multiplies
#pragma unroll
      for (int tl = 0; tl < NT; ++tl) {
        f32x4 acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        // the A fragments one k-step ahead of the products (two in registers:
        // the registers holding W_hh leave no room for all eight)
        const bf16* ab = &al[((lane >> 4) * (R + 1) + tl * 16 + (lane & 15)) * 8];
        bf16x8 af = *(const bf16x8*)ab, an;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          if (ks + 1 < 8) an = *(const bf16x8*)(ab + (ks + 1) * 4 * (R + 1) * 8);
          // (unit blocks past H hold zero fragments; their sums are not published)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j] = Mfma<bf16>::mma(af, bw[ks][j], acc[j]);
          af = an;
        }
        // publish: word (row quad, member, unit), the lane's four rows
        const int rl = tl * 16 + (lane >> 4) * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if constexpr (F32X) {
            if (rl < RV && rowbase + rl < rend && w + 8 * j < NB) {
              uint64_t* xw = xo + opub + (uint32_t)(tl * 16 * NM * H + j * 128);
#pragma unroll
              for (int r = 0; r < 4; ++r)
                ll_store64(xw + r * H, ((uint64_t)(tag0 + tau + 1) << 32) | __float_as_uint(acc[j][r]), local);
            }
          } else {
            const uint64_t v = p15x4_encode(acc[j]);   // (inside the branch, two registers spill at RV = 32)
            if (rl < RV && rowbase + rl < rend && w + 8 * j < NB)
              ll_store64(xo + opub + (uint32_t)(tl * 4 * NM * H + j * 128), v | tg, local);
          }
        }
      }
    }

    // da in frame-major rows, 16 bytes of LDS and of DA per piece (8 own gate
    // rows of one row)
    if (dtid >= 0) {
      bf16* dat = a.DA + (int64_t)t * fg;
#pragma unroll
      for (int c0 = 0; c0 < NDA; ++c0) {
        const int c = c0 * NDT + dtid, kg = c & 31, r = c >> 5;
        if (rowbase + r < rend && u0 + (kg >> 3) * 16 + (kg & 1) * 8 < H)
          *(uint4*)(dat + oda[c0]) = *(const uint4*)&al[(kg * (R + 1) + r) * 8];
      }
    }
  }
  if constexpr (ONE) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) group_state(a.state, g, mem, NM)[4 + i] = dcreg[i];
#pragma unroll
    for (int q = 0; q < 4; ++q) group_state(a.state, g, mem, NM)[q] = dbacc[q];
  }
  if (a.DBP && tau1 == Tn) {
    // bias partials: every lane's sum over its rows and steps, added over
    // the slice's row groups in order
    float* red = (float*)lds_raw;   // [RV / RPT][64 units][4 gates]
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) red[((qd * LPI + sub) * PU + cu) * 4 + q] = dbacc[q];
    __syncthreads();
    if (tid < 4 * PU && rowbase < rend && u0 + (tid >> 2) < H) {
      float sum = 0.f;
#pragma unroll
      for (int r = 0; r < RV / RPT; ++r) sum += red[r * PU * 4 + tid];
      a.DBP[(int64_t)s * 8 * H + (int64_t)d * 4 * H + (int64_t)(tid & 3) * H + u0 + (tid >> 2)] = sum;
    }
  }
  if constexpr (ONE) __syncthreads();   // the next pass reuses the LDS
  return how;
}

template <int RV, bool F32X>
__device__ __attribute__((noinline)) void bwd_alone(const PersistArgs* at, lds_base_t lds, int gv) {
  char* lds_raw = (char*)lds;
  const int g = scalar(gv);
  const PersistArgs a = pass_args(at);
  const int NM = (a.H + PU - 1) / PU;
#pragma nounroll
  for (int tau = 0; tau < a.Tn; ++tau)
#pragma nounroll
    for (int m = 0; m < NM; ++m) bwd_pass<RV, F32X, true>(pass_args(at), lds_raw, g, m, tau, tau + 1);
}

template <int RV, bool F32X>
__global__ __launch_bounds__(NTH) ONE_PER_CU void lstm_bwd_persist(const PersistArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];
  const int NM = (a.H + PU - 1) / PU;
  int g, mem;
  group_of(a.NG, NM, &g, &mem);
  if (g >= 2 * a.NS) return;   // padding (see persist_groups)
  if (a.Tn > 1 && NM > 1) group_arrive(a.words, a.seq, g, mem, a.wait);
  if (bwd_pass<RV, F32X, false>(a, lds_raw, g, mem, 0, a.Tn) != GROUP_ALONE) return;
  if (threadIdx.x == 0) a.status[1] = 1;
  bwd_alone<RV, F32X>(kernel_args<PersistArgs>(), (lds_base_t)lds_raw, g);
}

// The recurrence status block (at the end of the activation workspace): an
// int set to 1 by any exchange wait that gives up, and a 64-bit tag that
// says whether the block has been initialised.  The flag is sticky: only
// status_reset_kernel (blstm_recurrence_ok) clears it, and the forward pass
// initialises it only when the tag is missing (a fresh workspace), so one
// query covers every call since the previous query.
#define STATUS_TAG 0x5354415455535f31ull   // "STATUS_1"

__device__ __forceinline__ void status_init_if_fresh(int* status) {
  uint64_t* tag = (uint64_t*)(status + 2);
  if (*tag != STATUS_TAG) {
    status[0] = status[1] = 0;
    *tag = STATUS_TAG;
  }
}

// exchange words cleared; status (if non-null) initialised when fresh
__global__ __launch_bounds__(256) void clear_exchange_kernel(uint4* p, int64_t n16, int* status) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
    p[i] = make_uint4(0u, 0u, 0u, 0u);
  if (status && blockIdx.x == 0 && threadIdx.x == 0) status_init_if_fresh(status);
}

__global__ void status_reset_kernel(int* status) {
  status[0] = status[1] = 0;
  *(uint64_t*)(status + 2) = STATUS_TAG;
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
static int members(int H) { return (int)cdiv(H, PU); }

size_t persist_lds_bytes(int H, bool backward, int RV) {
  const int R = RV > 16 ? 32 : 16;
  const size_t run = backward ? (size_t)bwd_dy_lds(RV)
                              : (size_t)(rup(H, PU) / 8) * (R + 1) * 16 + (size_t)(RV > 16 ? 2 : 1) * 4 * 4 * 64 * 16 +
                                    (size_t)2 * RV * PU * (4 + 2 + 8);
  return std::max(std::max(run, (size_t)STAGE_BYTES), backward ? (size_t)0 : gx_lds_bytes);
}

// Compute units: one persistent workgroup fits per CU (its 8 waves hold
// the W_hh slice in half of the register file and the rest in working
// registers).
int persist_max_wg() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  return cus;
}

bool persist_supported(int H, int T) {
  (void)T;   // any length: the tag holds only bit 1 of the step number
  return H % 32 == 0 && H >= 32 && H <= 512;
}

// Launch mode.  A cooperative launch has all its workgroups resident at once,
// at a measured cost of about 15 us per launch on MI355X (12 launches per
// learner step).  A plain launch is used instead when the occupancy query shows
// that the whole grid fits on the device at once (one workgroup per CU here):
// its groups all run together unless other launches hold CUs, and a group that
// does not get all of its own in time is done by one workgroup (group_meet).
// ADPSGD_BLSTM_COOPERATIVE=1 forces cooperative launches, for comparisons.
static bool force_cooperative() {
  const char* e = getenv("ADPSGD_BLSTM_COOPERATIVE");
  return e && e[0] == '1';
}

hipError_t persist_launch(const char* name, const void* fn, dim3 grid, int threads, size_t lds, void* arg,
                          hipStream_t s) {
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const dim3 block(threads);
  void* args[] = {arg};
  // the whole grid resident at once? (per device; the answer depends only
  // on the kernel and its resources)
  bool fits = false;
  if (!force_cooperative()) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds) == hipSuccess)
      fits = (int64_t)per_cu * persist_max_wg() >= (int64_t)grid.x;
    else
      (void)hipGetLastError();
  }
  const int slot = g_timing_on ? timing_pre(name, s) : -1;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  e = hipStreamIsCapturing(s, &cap);
  if (e != hipSuccess) return e;
  if (fits) {
    e = hipLaunchKernel(fn, grid, block, args, lds, s);
  } else if (cap == hipStreamCaptureStatusNone) {
    e = hipLaunchCooperativeKernel(fn, grid, block, args, (unsigned)lds, s);
  } else {
    // recorded into a graph as a kernel node with the cooperative attribute
    hipLaunchAttribute attr;
    memset(&attr, 0, sizeof(attr));
    attr.id = hipLaunchAttributeCooperative;
    attr.val.cooperative = 1;
    hipLaunchConfig_t cfg;
    memset(&cfg, 0, sizeof(cfg));
    cfg.gridDim = grid;
    cfg.blockDim = block;
    cfg.dynamicSmemBytes = lds;
    cfg.stream = s;
    cfg.attrs = &attr;
    cfg.numAttrs = 1;
    e = hipLaunchKernelExC(&cfg, fn, args);
  }
  if (slot >= 0) timing_post(slot, s);
  return e;
}

uint32_t persist_group_wait() {
  const char* e = getenv("ADPSGD_BLSTM_GROUP_WAIT_US");
  return 100u * (uint32_t)(e ? std::min(std::max(atoi(e), 0), 1000000) : 1000);
}

int persist_groups(int groups, int members) {
  const int padded = (int)rup(groups, 8);
  return padded * members <= persist_max_wg() ? padded : groups;
}

template <int RV, bool BWD>
static hipError_t launch_one(PersistArgs a, hipStream_t s) {
  const void* fn;
  // (widths that 64 does not divide take at most 16 rows, see persist_plan)
  constexpr bool ODD = RV < 32;
  if (BWD)
    fn = ODD && a.H % PU ? (const void*)lstm_bwd_persist<RV, ODD> : (const void*)lstm_bwd_persist<RV, false>;
  else
    fn = ODD && a.H % PU ? (const void*)lstm_fwd_persist<RV, ODD> : (const void*)lstm_fwd_persist<RV, false>;
  return persist_launch(BWD ? "lstm_rec_bwd_persist" : "lstm_rec_fwd_persist", fn, dim3(a.NG * members(a.H)), NTH,
                        persist_lds_bytes(a.H, BWD, RV), &a, s);
}

// Rows per workgroup of a launch over `rows` rows: the fewest that take them all
// at one workgroup per CU, 8 (half of each MFMA tile idle, half the cell work
// and exchange per workgroup), 16, or 32 (the most; 16 where 64 does not divide
// H: the gather of more rows' float32 partial sums spills).
// ADPSGD_BLSTM_ROWS_PER_WG=16 or 32 keeps that many at any batch (fewer
// workgroups at small batches, for measurements and tests).
static int max_slices(int H) { return std::min(persist_max_wg(), 256) / (2 * members(H)); }
static int launch_rows(int H, int rows) {
  const int most = H % PU ? 16 : 32, ns = max_slices(H);
  if (const char* e = getenv("ADPSGD_BLSTM_ROWS_PER_WG"))
    if (atoi(e) == 16 || atoi(e) == 32) return std::min(atoi(e), most);
  return (rows + 7) / 8 <= ns ? 8 : (rows + 15) / 16 <= ns ? 16 : most;
}
// Rows per workgroup of a batch's largest launches, and rows per launch (the
// last one takes what is left, with rows per workgroup of its own: 520
// sequences at H = 512, T = 21 run as 512 + 8, forward 322 us a layer with 32
// rows per workgroup in both, 229 now).  False if no launch fits.
static bool persist_plan(int H, int B, int* RVo, int* chunko) {
  if (max_slices(H) < 1) return false;
  const int RV = launch_rows(H, B);
  *RVo = RV;
  *chunko = std::min(B, max_slices(H) * RV);
  return true;
}

bool persist_short_fwd(int H, int B, int T) {
  if (H % PU == 0) return false;
  int RV, chunk;
  if (!persist_plan(H, B, &RV, &chunk)) return false;
  return T <= (chunk == B ? 2 : 2 * (B % chunk) > chunk || B % chunk == 0 ? 3 : 5);
}

bool persist_fuse_gx(int H, int B, int T, int K) {
  int RV, chunk;
  if (!persist_plan(H, B, &RV, &chunk)) return false;
  const int64_t rows = (int64_t)T * RV;
  if (K <= 128 && rows <= 32) return true;
  return 2 * cdiv(chunk, RV) * members(H) >= 192 && 4 * rows >= 3 * GXR * cdiv(rows, GXR);
}

int persist_bias_rows(int H, int B) {
  int RV, chunk;
  if (!persist_plan(H, B, &RV, &chunk)) return 0;
  const int left = B % chunk;
  return (int)cdiv(B - left, RV) + (left ? (int)cdiv(left, launch_rows(H, left)) : 0);
}

bool persist_bwd_dy_partials_ok(int H, int B, int T) {
  int RV, chunk;
  if (!persist_plan(H, B, &RV, &chunk)) return false;
  return (size_t)bwd_dy_lds(RV) + (size_t)T * RV * PU * 4 <= persist_lds_bytes(H, true, RV);
}

hipError_t persist_clear(bool backward, const PersistArgs& a, hipStream_t s) {
  int RV, chunk;
  if (!persist_plan(a.H, a.B, &RV, &chunk)) return hipErrorInvalidValue;
  // both exchange slots start without any valid tag; the forward's clear
  // also initialises the status block of a fresh workspace
  const int64_t part = (int64_t)((chunk + 3) / 4) * members(a.H) * a.H * (a.H % PU ? 4 : 1);
  const int64_t words = GROUP_WORDS + 2 * 2 * (backward ? part : (int64_t)chunk * (a.H / 4));
  return persist_clear_words(a.words, words / 2, backward ? nullptr : a.status, s);
}

hipError_t persist_clear_words(void* p, int64_t n16, int* status, hipStream_t s) {
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(cdiv(n16, 256), 2048));
  hipLaunchKernelGGL(clear_exchange_kernel, dim3(grid), dim3(256), 0, s, (uint4*)p, n16, status);
  return hipGetLastError();
}

hipError_t persist_status_init(int* status, hipStream_t s) { return persist_clear_words(nullptr, 0, status, s); }

hipError_t persist_status_reset(int* status, hipStream_t s) {
  hipLaunchKernelGGL(status_reset_kernel, dim3(1), dim3(1), 0, s, status);
  return hipGetLastError();
}

hipError_t persist_layer(bool backward, PersistArgs a, hipStream_t s) {
  int RV, chunk;
  if (!persist_plan(a.H, a.B, &RV, &chunk)) return hipErrorInvalidValue;
  const uint32_t wait = persist_group_wait();
  for (int b0 = 0; b0 < a.B; b0 += chunk) {
    PersistArgs c = a;
    c.b0 = b0;
    c.rows = std::min(chunk, a.B - b0);
    if (a.DBP) c.DBP = a.DBP + (int64_t)(b0 / RV) * 8 * a.H;
    const int rv = c.rows < chunk ? launch_rows(a.H, c.rows) : RV;
    c.NS = (c.rows + rv - 1) / rv;
    c.NG = persist_groups(2 * c.NS, members(a.H));
    // the launch's position in the call (the caller's tag numbers the layers
    // in the order the call runs them)
    c.seq = a.tag * (uint32_t)cdiv(a.B, chunk) + (uint32_t)(b0 / chunk);
    c.wait = wait;
    const hipError_t e = rv == 8    ? (backward ? launch_one<8, true>(c, s) : launch_one<8, false>(c, s))
                         : rv == 16 ? (backward ? launch_one<16, true>(c, s) : launch_one<16, false>(c, s))
                                    : (backward ? launch_one<32, true>(c, s) : launch_one<32, false>(c, s));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

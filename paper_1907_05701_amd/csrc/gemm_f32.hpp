// float32 GEMM C[m][n] = sum_k A(m, k) B(n, k) with each operand K-contiguous
// (element (mn, k) at mn*ld + k) or MN-contiguous (at k*ld + mn): 64x64 output
// blocks of four waves (32x32 each, v_mfma_f32_16x16x4_f32), 32-deep k-tiles
// staged by direct-to-LDS loads into a three-stage ring (48 KB, three
// workgroups per CU).
//
// The float32 matrix rate (256 operations per clock and CU) asks little of
// the LDS and the caches at this block size (16 operand bytes per clock and CU
// from L2); what bounded the register-staged kernel it replaces was the memory
// latency of every 16-deep k-tile.  Here two k-tiles are in flight while the
// third is multiplied, and 12 waves per CU cover each other's waits.
// Measured at 672 frames of two 512-cell layers, register-staged / this one:
// input projections 54.2 / 42.3 us on average, weight gradients 47.4 / 38.6,
// dX (672 x 1024 x 4096, with its partial sums) 120 / 69.
//
// LDS layout.  K-contiguous: rows of 32 k (128 bytes), 16-byte chunk c of row
// r in slot c ^ (r & 7); a fragment read takes 16 bytes per lane, i.e. four k
// of one row, which feed four MFMAs (lane group g = lane / 16 supplies k =
// 4 g + s in MFMA s).  MN-contiguous: rows of 64 mn (256 bytes) of one k,
// chunk c of row k in slot c ^ (4 (k / 4 mod 4)); MFMA s reads the rows 4 g + s
// (4 bytes per lane, the four rows in distinct bank groups).
#pragma once

#include "dma.hpp"
#include "gemm.hpp"

struct F32Args {
  const float* A;
  int64_t lda, azs, arows;   // rows (KC) or contiguous extent (MNC) of A, batch stride azs
  const float* B;
  int64_t ldb, bzs, brows;
  int64_t bseg, bsegs;       // MN-contiguous B: k rows from bseg on start bsegs elements after the first (0: one segment)
  int64_t M, N, K, ksplit;   // k range of split s: [s*ksplit, min(K, (s+1)*ksplit))
  int splits, ntm, ntn, total;
};

#define F32_BT 64
#define F32_BK 32
#define F32_ST 3
#define F32_RUN 8
static constexpr size_t f32_lds_bytes = (size_t)F32_ST * 2 * F32_BT * F32_BK * 4;

template <bool KC>
struct F32Operand {
  static constexpr int CPR = KC ? F32_BK / 4 : F32_BT / 4;   // 16-byte chunks per LDS row
  static constexpr int RPI = 64 / CPR;                       // rows per load instruction
  static constexpr int LOADS = F32_BT * F32_BK * 4 / 1024 / 4;   // load instructions per wave and k-tile
  __device__ __forceinline__ static int slot(int c, int r) { return KC ? c ^ (r & 7) : c ^ (((r >> 2) & 3) << 2); }
  // rows: valid rows from the tile's first (KC), or the contiguous extent left (MNC)
  __device__ __forceinline__ static void issue(const float* base, int64_t ld, int64_t seg, int64_t segs, int64_t mn0,
                                               int64_t rows, int64_t k0, int64_t kend, char* tile, int wid, int lane) {
    const int lr = lane / CPR, ls = lane % CPR;
    const int64_t kb = KC ? mn0 * ld + k0 : (seg && k0 >= seg ? segs + (k0 - seg) * ld : k0 * ld) + mn0;
    const __amdgpu_buffer_rsrc_t r = dma_rsrc(base + kb);
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
      const int row = (q * 4 + wid) * RPI + lr;
      const int c = slot(ls, row) * 4;
      const bool ok = KC ? row < rows && k0 + c < kend : k0 + row < kend && c < rows;
      dma16(r, ok ? (uint32_t)((row * ld + c) * 4) : DMA_OFF_NONE, tile + (q * 4 + wid) * 1024);
    }
  }
  // the lane's values of MFMAs s = 0..3 of 16-deep step ks, for the 16 rows from mnb
  __device__ __forceinline__ static f32x4 frag(const char* tile, int mnb, int ks, int lane) {
    const int fr = lane & 15, g = lane >> 4;
    if constexpr (KC) {
      const int row = mnb + fr;
      return *(const f32x4*)(tile + row * (F32_BK * 4) + slot(ks * 4 + g, row) * 16);
    } else {
      f32x4 v;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = ks * 16 + g * 4 + s, mn = mnb + fr;
        v[s] = *(const float*)(tile + k * (F32_BT * 4) + slot(mn >> 2, k) * 16 + (mn & 3) * 4);
      }
      return v;
    }
  }
};

// One output block of one product; w is the workgroup's index within the
// product's workgroups (those at or past p.total have no block).
template <bool AKC, bool BKC, class Epi>
__device__ __forceinline__ void gemm_f32_tile(const F32Args& p, const Epi& epi, int w) {
  typedef F32Operand<AKC> OA;
  typedef F32Operand<BKC> OB;
  constexpr int TA = F32_BT * F32_BK * 4, STAGE = 2 * TA;
  extern __shared__ __attribute__((aligned(1024))) char f32_lds[];
  if (w >= p.total) return;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int wm = wid & 1, wn = wid >> 1;
  int zs, tm, tn;
  kc_tile_of(p, w, 4, zs, tm, tn);
  const int z = zs / p.splits, sp = zs % p.splits;
  const int64_t m0 = (int64_t)tm * F32_BT, n0 = (int64_t)tn * F32_BT;
  const int64_t kbeg = (int64_t)sp * p.ksplit, kend = min(p.K, kbeg + p.ksplit);
  const int ntiles = kend > kbeg ? (int)((kend - kbeg + F32_BK - 1) / F32_BK) : 0;
  const float* ab = p.A + (int64_t)z * p.azs;
  const float* bb = p.B + (int64_t)z * p.bzs;
  auto issue = [&](int j) {
    const int64_t k0 = kbeg + (int64_t)j * F32_BK;
    char* st = f32_lds + (j % F32_ST) * STAGE;
    OA::issue(ab, p.lda, 0, 0, m0, p.arows - m0, k0, kend, st, wid, lane);
    OB::issue(bb, p.ldb, p.bseg, p.bsegs, n0, p.brows - n0, k0, kend, st + TA, wid, lane);
  };
  // two sums per output, of the even and the odd 16-deep steps, moved into a
  // total every F32_RUN k-tiles: chains of roundings of at most K / 256 + 32
  // steps instead of K / 4 (the split-K partials used to shorten them)
  f32x4 acc[2][2][2], total[2][2];
  auto clear = [&](f32x4 (&v)[2][2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) v[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  auto flush = [&]() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) total[i][j] += acc[0][i][j] + acc[1][i][j];
    clear(acc[0]);
    clear(acc[1]);
  };
  clear(total);
  clear(acc[0]);
  clear(acc[1]);
#pragma unroll
  for (int j = 0; j < F32_ST - 1; ++j)
    if (j < ntiles) issue(j);
  for (int it = 0; it < ntiles; ++it) {
    if (it + F32_ST - 2 < ntiles)
      kc_wait_vm<(F32_ST - 2) * (OA::LOADS + OB::LOADS)>();
    else
      kc_wait_vm<0>();
    kc_barrier();   // tile it in LDS; every wave is done with tile it - 1
    if (it + F32_ST - 1 < ntiles) issue(it + F32_ST - 1);
    const char* st = f32_lds + (it % F32_ST) * STAGE;
#pragma unroll
    for (int ks = 0; ks < F32_BK / 16; ++ks) {
      f32x4 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = OA::frag(st, wm * 32 + i * 16, ks, lane);
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = OB::frag(st + TA, wn * 32 + j * 16, ks, lane);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[ks & 1][i][j] = Mfma<float>::mma(a[i][s], b[j][s], acc[ks & 1][i][j]);
    }
    if (it % F32_RUN == F32_RUN - 1) flush();
  }
  flush();
  epi.template apply<2, 2>(z, sp, m0 + wm * 32, n0 + wn * 32, total, lane);
}

template <bool AKC, bool BKC, class Epi>
__global__ __launch_bounds__(256, 3) void gemm_f32_kernel(const F32Args p, const Epi epi) {
  gemm_f32_tile<AKC, BKC, Epi>(p, epi, blockIdx.x);
}

// Several products of one layout in one launch (product i owns workgroups
// [start[i], start[i + 1]), starts multiples of 8), and two of different
// layouts (the first owns [0, n1)): one launch and one partial round of the
// chip instead of several.
#define F32_MAX_GROUP 12
template <class Epi>
struct F32Group {
  F32Args p[F32_MAX_GROUP];
  Epi e[F32_MAX_GROUP];
  int start[F32_MAX_GROUP + 1];
  int n;
};
template <bool AKC, bool BKC, class Epi>
__global__ __launch_bounds__(256, 3) void gemm_f32_group_kernel(const F32Group<Epi> g) {
  int i = 0;
#pragma unroll
  for (int k = 1; k < F32_MAX_GROUP; ++k) i += (k < g.n && (int)blockIdx.x >= g.start[k]);
  gemm_f32_tile<AKC, BKC, Epi>(g.p[i], g.e[i], (int)blockIdx.x - g.start[i]);
}
template <bool AKC1, bool BKC1, bool AKC2, bool BKC2, class Epi>
__global__ __launch_bounds__(256, 3) void gemm_f32_pair_kernel(const F32Args p1, const Epi e1, const F32Args p2,
                                                               const Epi e2, int n1) {
  if ((int)blockIdx.x < n1)
    gemm_f32_tile<AKC1, BKC1, Epi>(p1, e1, (int)blockIdx.x);
  else
    gemm_f32_tile<AKC2, BKC2, Epi>(p2, e2, (int)blockIdx.x - n1);
}

// Whether an operand can be staged: 16-byte aligned rows, batches and
// segments, the whole k range inside it (K-contiguous: to the end of its last
// chunk, with finite values there that meet the MN-contiguous other operand's
// zeros).
static inline bool f32_operand_ok(const Opnd& o, int64_t K, bool kc, bool seg_ok) {
  if (o.ilH != 0 || o.ld % 4 != 0 || o.zstride % 4 != 0 || ((uintptr_t)o.base & 15) != 0) return false;
  if (kc) return o.seg == 0 && o.ext >= rup(K, 4) && 64 * o.ld * 4 < 0x7ffffff0;
  if (o.seg != 0 && !(seg_ok && o.seg % F32_BK == 0 && K <= 2 * o.seg && o.segstride % 4 == 0)) return false;
  return o.rows >= K && o.ext % 4 == 0 && F32_BK * o.ld * 4 < 0x7ffffff0;
}

// False if an operand cannot be staged.
template <bool AKC, bool BKC>
static inline bool f32_args(const Opnd& A, const Opnd& B, int64_t M, int64_t N, int64_t K, int batches, int splits,
                            F32Args* q) {
  if (AKC && BKC && K % 4 != 0) return false;
  if (!f32_operand_ok(A, K, AKC, false) || !f32_operand_ok(B, K, BKC, true)) return false;
  F32Args& p = *q;
  p.A = (const float*)A.base; p.lda = A.ld; p.azs = A.zstride; p.arows = AKC ? std::min<int64_t>(A.rows, M) : A.ext;
  p.B = (const float*)B.base; p.ldb = B.ld; p.bzs = B.zstride; p.brows = BKC ? std::min<int64_t>(B.rows, N) : B.ext;
  p.bseg = BKC ? 0 : B.seg; p.bsegs = B.segstride;
  p.M = M; p.N = N; p.K = K;
  p.ksplit = splits > 1 ? rup(cdiv(K, splits), F32_BK) : (K > 0 ? K : 1);
  p.splits = splits;
  p.ntm = (int)cdiv(M, F32_BT);
  p.ntn = (int)cdiv(N, F32_BT);
  const int64_t total = (int64_t)batches * splits * p.ntm * p.ntn;
  p.total = (int)total;
  return total <= (1 << 30);
}

// One product; false (and nothing launched) if an operand cannot be staged.
template <bool AKC, bool BKC, class Epi>
static inline bool gemm_f32_dma(const char* name, hipStream_t s, const Opnd& A, const Opnd& B, int64_t M, int64_t N,
                                int64_t K, int batches, int splits, const Epi& epi) {
  F32Args p;
  if (!f32_args<AKC, BKC>(A, B, M, N, K, batches, splits, &p)) return false;
  auto fn = gemm_f32_kernel<AKC, BKC, Epi>;
  BLSTM_LAUNCH(name, fn, dim3((unsigned)p.total), dim3(256), f32_lds_bytes, s, p, epi);
  return true;
}

// Fused transition layer (MegaFold Section IV: fused layer-norm & linear
// projection, fused SwiGLU and the fused transition layer built from them;
// forward and backward in the appendix listing of the transition layer).
// Per row x of the pair representation (C = 128 features):
//   o1 = (x - mean) rstd * gamma + beta
//   [a | b] = o1 W1              W1 [C][2F]
//   u = a sigmoid(a) b           (SwiGLU)
//   out = u W2                   W2 [F][C]
//
// Differences from the paper's design (separate layer-norm-linear, SwiGLU
// and matmul kernels with o1 and o2 written to memory, atomics for the
// weight gradients), for gfx950:
//  - the forward is ONE kernel: a wave keeps its 32 rows' normalised
//    features and its output accumulators in registers and walks the hidden
//    width in chunks of 32 columns; [a | b] and u of a chunk never leave the
//    registers (u goes straight from the accumulators into the B operand of
//    the W2 product);
//  - the backward recomputes [a | b] instead of reading it back (the matrix
//    cores have room, HBM does not): one kernel computes dx (du, the
//    recomputed a and b, dh = [da | db], do1 = dh W1^T, the layer-norm
//    backward), a second one the sums over rows per column group of the
//    hidden width (G = xhat^T dh, s = column sums of dh, dW2 = u^T dout),
//    each into its own partial-sum block, reduced in a fixed order:
//    dW1 = gamma G + beta s^T, dgamma = sum_n W1 o G, dbeta = W1 s
//    (o1 = xhat gamma + beta regrouped), bitwise reproducible;
//  - products are formed transposed where that keeps a lane on one row
//    (out^T = W2^T u^T, do1^T = W1 dh^T), so the elementwise steps stay in
//    the lane that holds the row.
//
// Weights reach the kernels through per-chunk images that a small packing
// kernel writes into the workspace (the contraction slots of the
// accumulator-fed operands already in accumulator order); a workgroup streams
// them into an LDS ring.
#include <algorithm>
#include <type_traits>

#include "dma.h"
#include "kernels.h"
#include "timing.h"

namespace triattn {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int TRN_WAVES = 8;
constexpr int TRN_THREADS = 64 * TRN_WAVES;
constexpr int TRN_NT = TRN_C / 16;  // MFMA steps over the features
constexpr int TRN_ROWS = 32 * TRN_WAVES;  // rows per workgroup block

// image of one chunk j (hidden columns fb = 32 j .. fb + 31), bytes:
//   forward : A1a [0, 8K)  A1b [8K, 16K)  A2 [16K, 24K)
//   backward: A1a [0, 8.5K)  A1b [8.5K, 17K)  A3 [17K, 25.5K)  A4 [25.5K, 43.5K), padded to 44K
// A1a / A1b: W1^T rows fb + r (a) / F + fb + r (b), 16 pieces (16 bytes) of 8 features.
// A2: W2^T for output tile t, row r = output column 32 t + r, 4 pieces
//     (k-step s, half g) of hidden columns in accumulator order.
// A3: W2 rows fb + r, 16 pieces of 8 output columns.
// A4: W1 for feature tile t, row r = feature 32 t + r, 8 pieces (k-step
//     s = 0..3, half g): s < 2 the a columns, s >= 2 the b columns of the
//     chunk, in accumulator order.
// In LDS every row is followed by 16 unused bytes: rows r, r + 1, .. then start
// an odd number of 16-byte pieces apart, so an operand read (one piece of 32
// consecutive rows) is free of bank conflicts and all of a lane's reads of a
// chunk are one address per row pitch plus constants (a permutation of the
// pieces takes 16 to 24 address registers, which the kernels spend on operands
// in flight instead).  The backward's images hold the gaps too (its workspace
// has the room, and without them trn_bwd_w, which reads rows from the images,
// takes 1.6 us more and trn_bwd_dx, with an address per copy, 0.8); the
// forward's do not, which keeps its workspace at 24 KB per chunk: its copies
// leave the gaps, each lane with its own address in the image.
constexpr int IMG_A2 = 16384;                                      // forward image
constexpr int P1 = 256 + 16, P2 = 64 + 16, P4 = 128 + 16;         // row pitches in LDS
constexpr int OFF_A1B = 32 * P1, OFF_A2 = 64 * P1;                // forward
constexpr int OFF_A3 = 64 * P1, OFF_A4 = 96 * P1;                 // backward
constexpr int FWD_SLOT = 27648;                                   // whole copies of 1 KB
static_assert(OFF_A2 + 128 * P2 <= FWD_SLOT && FWD_SLOT % 1024 == 0, "slot size");
static_assert(IMG_A2 + 128 * 64 == TRN_FWD_IMG, "image size");
static_assert(OFF_A4 + 128 * P4 <= TRN_BWD_IMG && TRN_BWD_IMG % 1024 == 0, "image size");

// Accumulator order of a 16-wide contraction step s: slot e of half g holds
// index 16 s + 8 (e / 4) + 4 g + e % 4 (the rows a 32x32 accumulator gives
// a lane in its registers 8 s .. 8 s + 7).
__device__ inline int acc_k(int s, int g, int e) { return 16 * s + 8 * (e >> 2) + 4 * g + (e & 3); }

__device__ inline float sigm(float x) { return __builtin_amdgcn_rcpf(1.f + __expf(-x)); }

__device__ inline f32x4 mma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---- weight images -------------------------------------------------------------------

// One thread per 16-byte piece of the images of all chunks.
__global__ __launch_bounds__(256) void trn_pack_kernel(const bf16* w1, const bf16* w2, int f,
                                                       int bwd, char* img) {
  const int img_bytes = bwd ? TRN_BWD_IMG : TRN_FWD_IMG;
  const int per = img_bytes / 16;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)(f / TRN_FC) * per) return;
  const int j = (int)(idx / per), o = 16 * (int)(idx % per), fb = TRN_FC * j;
  const int n1 = 2 * f;  // W1 row length
  bf16x8 v = {};         // gaps stay zero
  const int p1 = bwd ? P1 : 256;
  if (o < 64 * p1) {  // A1a, A1b
    const int r = o / p1, c = o % p1 >> 4;
    const int col = (r >> 5) * f + fb + (r & 31);
    if (c < 16) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = w1[(int64_t)(8 * c + e) * n1 + col];
    }
  } else if (!bwd) {  // A2
    const int r = (o - IMG_A2) / 64, c = o % 64 >> 4;  // r: output column
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = w2[(int64_t)(fb + acc_k(c >> 1, c & 1, e)) * TRN_C + r];
  } else if (o < OFF_A4) {  // A3
    const int r = (o - OFF_A3) / P1, c = ((o - OFF_A3) % P1) >> 4;
    if (c < 16) v = *(const bf16x8*)(w2 + (int64_t)(fb + r) * TRN_C + 8 * c);
  } else {  // A4
    const int r = (o - OFF_A4) / P4, c = ((o - OFF_A4) % P4) >> 4;  // r: feature
    const int s = c >> 1, g = c & 1;
    const int base = (s < 2 ? 0 : f) + fb;
    if (r < TRN_C && c < 8) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = w1[(int64_t)r * n1 + base + acc_k(s & 1, g, e)];
    }
  }
  *(bf16x8*)(img + (int64_t)j * img_bytes + o) = v;
}

// Row statistics and o1 (bf16, the B operand over the features) of a lane's
// row: half g holds features 16 t + 8 g .. + 7.
__device__ inline void ln_row(const bf16x8 (&xr)[TRN_NT], const float (&gb)[2][TRN_C], int g,
                              float eps, float& mean, float& rstd, bf16x8 (&of)[TRN_NT]) {
  float xv[TRN_NT][8];
  float s = 0.f;
#pragma unroll
  for (int t = 0; t < TRN_NT; ++t)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      xv[t][e] = (float)xr[t][e];
      s += xv[t][e];
    }
  mean = wave_xor32_sum(s) * (1.f / TRN_C);
  float v = 0.f;
#pragma unroll
  for (int t = 0; t < TRN_NT; ++t)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      xv[t][e] -= mean;
      v = fmaf(xv[t][e], xv[t][e], v);
    }
  rstd = 1.f / sqrtf(wave_xor32_sum(v) * (1.f / TRN_C) + eps);
#pragma unroll
  for (int t = 0; t < TRN_NT; ++t)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = 16 * t + 8 * g + e;
      of[t][e] = (bf16)fmaf(xv[t][e] * rstd, gb[0][k], gb[1][k]);
    }
}

// o1 from saved statistics.
__device__ inline void ln_row_saved(const bf16x8 (&xr)[TRN_NT], const float (&gb)[2][TRN_C], int g,
                                    float mean, float rstd, bf16x8 (&of)[TRN_NT]) {
#pragma unroll
  for (int t = 0; t < TRN_NT; ++t)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = 16 * t + 8 * g + e;
      of[t][e] = (bf16)fmaf(((float)xr[t][e] - mean) * rstd, gb[0][k], gb[1][k]);
    }
}

__device__ inline void load_row(const bf16* base, int64_t row, int64_t m, int g,
                                bf16x8 (&xr)[TRN_NT]) {
  const bf16* p = base + (row < m ? row : m - 1) * TRN_C + 8 * g;
#pragma unroll
  for (int t = 0; t < TRN_NT; ++t) xr[t] = *(const bf16x8*)(p + 16 * t);
}

// Store a lane's 4 x 16 accumulated values (feature 32 t + 8 j + 4 g + i)
// of its row as bf16, 8 bytes per run.
__device__ inline void store_row(bf16* base, int64_t row, int g, const f32x16 (&acc)[4]) {
  bf16* p = base + row * TRN_C + 4 * g;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *(bf16x4*)(p + 32 * t + 8 * j) =
          bf16x4{(bf16)acc[t][4 * j], (bf16)acc[t][4 * j + 1], (bf16)acc[t][4 * j + 2],
                 (bf16)acc[t][4 * j + 3]};
}

// Chunk images HBM -> LDS by DMA, pieces of 1 KB dealt to the waves in turn (the
// last piece several times, so that no wave branches); real = false reads no
// memory and fills the slot with zeros.  Written as instructions: after the
// builtin the compiler holds the next LDS read, whatever it reads, until the
// copy has landed, which put a chunk's whole copy latency into every chunk of
// the kernels that read other slots meanwhile.  It does not count these copies
// either, so chunk_wait() must stand before the slot's readers; its own counted
// waits only get stricter by them.
// m0 (the LDS address) is an operand, so that the compiler knows what it holds.
// It does not see to the wait states here: five before the first load, in case
// a scalar operand has just come back from a vector register, and one after a
// write of m0.
#define TRN_COPY(m, v, s) "s_mov_b32 m0, " m "\n\ts_nop 0\n\tbuffer_load_dwordx4 " v ", %1, " s " offen lds\n\t"

__device__ inline u32x4 chunk_rsrc(const char* src, bool real, int bytes) {
  const uint64_t b = (uint64_t)src;
  return u32x4{(uint32_t)b, (uint32_t)(b >> 32) & 0xffffu, real ? (uint32_t)bytes : 0u, 0x00020000u};
}

struct FwdCopy {
  static constexpr int PIECES = FWD_SLOT / 1024, N = (PIECES + TRN_WAVES - 1) / TRN_WAVES;
  static_assert(N == 4, "pieces per wave");
  uint32_t at[N];  // where the wave's pieces go in the slot
  uint32_t v[N];   // and this lane's 16 bytes of them in the image (past its end in a gap: zeros)

  // (In units of 16 bytes, with the divisions as 24-bit products and without a
  // branch: the kernel's first copies wait for this.)
  __device__ inline FwdCopy(int wave, int lane) {
    constexpr uint32_t R1 = OFF_A2 / 16;  // rows of 16 units and a gap up to here, then of 4
    static_assert(R1 % 64 == 0, "a piece holds rows of one kind");
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint32_t piece = min(wave + TRN_WAVES * i, PIECES - 1);
      at[i] = 1024 * piece;
      const uint32_t u = 64 * piece + lane;
      // u / 17, q / 5: exact below 2^16
      const uint32_t r1 = __umul24(u, 61681) >> 20, c1 = u - __umul24(r1, 17);
      const uint32_t q = (u - R1) & 0xffff, r2 = __umul24(q, 52429) >> 18, c2 = q - __umul24(r2, 5);
      const uint32_t v1 = c1 < 16 ? 256 * r1 + 16 * c1 : TRN_FWD_IMG;
      const uint32_t v2 = c2 < 4 && r2 < TRN_C ? IMG_A2 + 64 * r2 + 16 * c2 : TRN_FWD_IMG;
      if (TRN_WAVES * (i + 1) <= R1 / 64)
        v[i] = v1;
      else if (TRN_WAVES * i >= R1 / 64)
        v[i] = v2;
      else
        v[i] = piece < R1 / 64 ? v1 : v2;
    }
  }

  __device__ inline void operator()(const char* src, char* dst, bool real) const {
    const uint32_t to = lds_addr(dst);
    uint32_t m0 = to + at[0];
    asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %2, %1, 0 offen lds\n\t"
                 TRN_COPY("%3", "%4", "0") TRN_COPY("%5", "%6", "0") TRN_COPY("%7", "%8", "0")
                 : "+{m0}"(m0)
                 : "s"(chunk_rsrc(src, real, TRN_FWD_IMG)), "v"(v[0]), "s"(to + at[1]), "v"(v[1]),
                   "s"(to + at[2]), "v"(v[2]), "s"(to + at[3]), "v"(v[3])
                 : "memory");
  }
};

__device__ inline void bwd_copy(const char* src, char* dst, int wave, int lane, bool real) {
  constexpr int PIECES = TRN_BWD_IMG / 1024, N = (PIECES + TRN_WAVES - 1) / TRN_WAVES;
  static_assert(N == 6, "pieces per wave");
  const uint32_t to = lds_addr(dst);
  uint32_t at[N];
#pragma unroll
  for (int i = 0; i < N; ++i) at[i] = 1024 * min(wave + TRN_WAVES * i, PIECES - 1);
  uint32_t m0 = to + at[0];
  asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %2, %1, %3 offen lds\n\t"
               TRN_COPY("%4", "%2", "%5") TRN_COPY("%6", "%2", "%7") TRN_COPY("%8", "%2", "%9")
               TRN_COPY("%10", "%2", "%11") TRN_COPY("%12", "%2", "%13")
               : "+{m0}"(m0)
               : "s"(chunk_rsrc(src, real, TRN_BWD_IMG)), "v"(16 * lane), "s"(at[0]), "s"(to + at[1]),
                 "s"(at[1]), "s"(to + at[2]), "s"(at[2]), "s"(to + at[3]), "s"(at[3]),
                 "s"(to + at[4]), "s"(at[4]), "s"(to + at[5]), "s"(at[5])
               : "memory");
}
#undef TRN_COPY

// Every copy, load and store of this wave has landed.
__device__ inline void chunk_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---- forward -------------------------------------------------------------------------
//
// Persistent workgroups of 8 waves (one per CU); a workgroup takes blocks of
// 256 rows (32 per wave) and walks the F / 32 chunks, whose images arrive in a
// ring of three by DMA, one barrier per chunk.  Per chunk a wave forms hb, the
// next chunk's ha and the chunk's share of out^T, 8 MFMAs each: u of the chunk
// is multiplied out under the next ha and the sigmoids of the next chunk run
// under out^T and hb, so that no MFMA waits for the elementwise step; eight
// operand fragments are in flight per wave, across chunks.  The next block's
// rows are loaded ahead of this block's stores (loads and stores retire in
// order).  Weights copied through registers and reads left to the compiler
// measured 61.8 us at m = 345^2, F = 512 (forward call), against 59.4.  No unit
// is full (m = 768^2): the matrix cores are busy 44% of the time, the LDS 24%
// (a fragment per MFMA is half of its 256 bytes per clock at the MFMA's full
// rate), and the waves wait for memory or the barrier 26% of theirs and are
// ready without being issued 43%: two waves per SIMD do not cover each other's
// latencies.  64 rows per wave halve the reads, but at one wave per SIMD the
// same schedule (442 registers) took 71.6 us.
__global__ __launch_bounds__(TRN_THREADS, 1) void trn_fwd_kernel(TrnFwdArgs a) {
  constexpr int SLOTS = 3;
  __shared__ __align__(16) char ring[SLOTS * FWD_SLOT];
  __shared__ __align__(16) float gb[2][TRN_C];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t nblk = (a.m + TRN_ROWS - 1) / TRN_ROWS;
  if ((int64_t)blockIdx.x >= nblk) return;  // whole workgroup, before any barrier
  const int nch = a.f / TRN_FC;             // at least 4 (F is a multiple of 128)
  // (in 32 bits, at most 2^23 blocks: a 64-bit division takes 0.2 us)
  const int nsteps = (int)(((uint32_t)nblk - blockIdx.x + gridDim.x - 1) / gridDim.x) * nch;
  int dj = 0, ds = 0;  // chunk index and slot of the next DMA
  int issued = 0;
  const FwdCopy copy(wave, lane);
  auto issue = [&] {
    copy(a.img + (int64_t)dj * TRN_FWD_IMG, ring + ds * FWD_SLOT, issued < nsteps);
    dj = dj + 1 == nch ? 0 : dj + 1;
    ds = ds + 1 == SLOTS ? 0 : ds + 1;
    ++issued;
  };
  issue();
  issue();
  int64_t row = (int64_t)blockIdx.x * TRN_ROWS + wave * 32 + l32;
  bf16x8 xr[TRN_NT], of[TRN_NT];
  load_row(a.x, row, a.m, g, xr);
  if (tid < TRN_C) {
    gb[0][tid] = (float)a.gamma[tid];
    gb[1][tid] = (float)a.beta[tid];
  }
  chunk_wait();
  __syncthreads();

  const uint32_t base = lds_addr(ring);
  const uint32_t b1 = base + l32 * P1 + 16 * g, b2 = base + OFF_A2 + l32 * P2 + 16 * g;
  uint32_t so = 0;  // slot offset of the current chunk
  bf16x8 fq[8];     // operand fragments in flight
  auto f1a = [&](uint32_t o, int i) { return lds_load16<bf16x8>(b1 + o + 32 * i); };
  auto f1b = [&](uint32_t o, int i) { return lds_load16<bf16x8>(b1 + o + OFF_A1B + 32 * i); };
  // (tile i % 4, step i / 4)
  auto f2 = [&](uint32_t o, int i) {
    return lds_load16<bf16x8>(b2 + o + (i & 3) * 32 * P2 + 32 * (i >> 2));
  };
#pragma unroll
  for (int i = 0; i < 8; ++i) fq[i] = f1a(0, i);

  for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    float mean, rstd;
    ln_row(xr, gb, g, a.eps, mean, rstd, of);
    if (row < a.m && g == 0) {
      a.mean[row] = mean;
      a.rstd[row] = rstd;
    }
    f32x16 acc[4] = {}, ha = {};
    float si[16];  // exp2, then the sigmoid, then a sigmoid(a)
    // stage w of the gate: a pair of elements starts per stage, w = 1 .. 8
    auto gate = [&](int w) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int e0 = 2 * (w - 1) + k, e1 = e0 - 2, e2 = e0 - 4;
        if (e0 >= 0 && e0 < 16) si[e0] = __builtin_amdgcn_exp2f(-LOG2E * ha[e0]);
        if (e1 >= 0 && e1 < 16) si[e1] = __builtin_amdgcn_rcpf(1.f + si[e1]);
        if (e2 >= 0 && e2 < 16) si[e2] = ha[e2] * si[e2];
      }
    };
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      ha = Mma<bf16>::mma(fq[i], of[i], ha);
      fq[i] = f1b(so, i);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int w = 0; w < 8; ++w) gate(w);
    auto chunk = [&](auto lastc) {
      constexpr bool LAST = decltype(lastc)::value;  // the block's last chunk: no next ha
      chunk_wait();  // the next chunk has landed; every wave has left the previous one
      lds_barrier();
      issue();
      const uint32_t sn = so == (SLOTS - 1) * FWD_SLOT ? 0u : so + FWD_SLOT;
      f32x16 hb = {};
      bf16x8 uf[2];
      auto mul = [&](int w) {  // u of elements 2 w, 2 w + 1
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int e = 2 * w + k;
          if (e >= 0) uf[e >> 3][e & 7] = (bf16)(si[e] * hb[e]);
        }
      };
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        hb = Mma<bf16>::mma(fq[i], of[i], hb);
        fq[i] = LAST ? f2(so, i) : f1a(sn, i);
        gate(8 + i);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (LAST) {
#pragma unroll
        for (int w = 0; w < 8; ++w) mul(w);
      } else {
        ha = f32x16{};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          ha = Mma<bf16>::mma(fq[i], of[i], ha);
          fq[i] = f2(so, i);
          mul(i - 1);
          __builtin_amdgcn_sched_barrier(0);
        }
        mul(7);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        acc[i & 3] = Mma<bf16>::mma(fq[i], uf[i >> 2], acc[i & 3]);
        fq[i] = LAST ? f1a(sn, i) : f1b(sn, i);
        if constexpr (!LAST) gate(i);
        __builtin_amdgcn_sched_barrier(0);
      }
      so = sn;
    };
    for (int j = 0; j + 1 < nch; ++j) chunk(std::false_type{});
    chunk(std::true_type{});
    const int64_t done = row;
    row += (int64_t)gridDim.x * TRN_ROWS;
    load_row(a.x, row, a.m, g, xr);  // (past the last block: the last row again)
    __builtin_amdgcn_sched_barrier(0);
    if (done < a.m) store_row(a.out, done, g, acc);
  }
  chunk_wait();  // the copies past the last chunk land before the workgroup ends
}

// ---- backward: dx ----------------------------------------------------------------------

// Persistent workgroups of 8 waves as in the forward, 32 rows per wave.  Per
// chunk a wave forms du, ha and hb (24 MFMAs) and adds the chunk's share of
// do1 (16).  The chunk images arrive in a ring of three by DMA; a wave's
// operand reads run TRN_NQ fragments ahead of their use, across chunks, and
// the elementwise step is dealt over the MFMAs after ha in stages of a pair
// of elements, so that it waits for neither.  Weights copied through
// registers and reads left to the compiler (one fragment ahead) measured
// 483 us at m = 768^2, F = 512, against 456 us on the same card (845 TFLOP/s
// of the ten products).  Of what remains the operand reads, one LDS fragment
// per MFMA, cost most (without them, a third less), by their latency and issue:
// the LDS is busy 23% of the time, the matrix cores 42%.  64 rows per wave
// would halve them, but at one wave per SIMD the forward built that way was
// slower (314 against 268 us).

constexpr int TRN_NQ = 8;  // operand fragments in flight per wave

__global__ __launch_bounds__(TRN_THREADS, 1) void trn_bwd_dx_kernel(TrnBwdArgs a) {
  constexpr int SLOTS = 3, NQ = TRN_NQ;
  __shared__ __align__(16) char ring[SLOTS * TRN_BWD_IMG];
  __shared__ __align__(16) float gb[2][TRN_C];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t nblk = (a.m + TRN_ROWS - 1) / TRN_ROWS;
  if ((int64_t)blockIdx.x >= nblk) return;
  const int nch = a.f / TRN_FC;
  // (in 32 bits, at most 2^23 blocks: a 64-bit division takes 0.2 us)
  const int nsteps = (int)(((uint32_t)nblk - blockIdx.x + gridDim.x - 1) / gridDim.x) * nch;
  int dj = 0, ds = 0;  // chunk index and slot of the next DMA
  int issued = 0;
  auto issue = [&] {
    bwd_copy(a.img + (int64_t)dj * TRN_BWD_IMG, ring + ds * TRN_BWD_IMG, wave, lane,
             issued < nsteps);
    dj = dj + 1 == nch ? 0 : dj + 1;
    ds = ds + 1 == SLOTS ? 0 : ds + 1;
    ++issued;
  };
  issue();
  issue();
  if (tid < TRN_C) {
    gb[0][tid] = (float)a.gamma[tid];
    gb[1][tid] = (float)a.beta[tid];
  }
  chunk_wait();
  __syncthreads();

  const uint32_t base = lds_addr(ring);
  const uint32_t b1 = base + l32 * P1 + 16 * g, b4 = base + OFF_A4 + l32 * P4 + 16 * g;
  uint32_t so = 0;  // slot offset of the current chunk
  // operand fragments of a chunk in the order of use: A3 (du), A1a (ha), A1b
  // (hb), 8 steps each, then A4 of the b columns (steps 2, 3) and of the a
  // columns (steps 0, 1), four feature tiles each
  bf16x8 fq[NQ];
  auto frag = [&](uint32_t o, int i) {
    if (i < 24) {
      const int off = i < 8 ? OFF_A3 : (i < 16 ? 0 : OFF_A1B);
      return lds_load16<bf16x8>(b1 + o + off + 32 * (i & 7));
    }
    const int s = ((i - 24) >> 2) ^ 2, t = i & 3;
    return lds_load16<bf16x8>(b4 + o + t * 32 * P4 + 32 * s);
  };
#pragma unroll
  for (int i = 0; i < NQ; ++i) fq[i] = frag(0, i);

  for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const int64_t row = blk * TRN_ROWS + wave * 32 + l32;
    const int64_t rc = row < a.m ? row : a.m - 1;
    bf16x8 xr[TRN_NT], of[TRN_NT], df[TRN_NT];
    load_row(a.x, row, a.m, g, xr);
    load_row(a.dout, row, a.m, g, df);
    const float mean = a.mean[rc], rstd = a.rstd[rc];
    ln_row_saved(xr, gb, g, mean, rstd, of);
    f32x16 d1[4] = {};  // do1^T: feature 32 t + acc row, lane <-> row
    for (int j = 0; j < nch; ++j) {
      const uint32_t sn = so == (SLOTS - 1) * TRN_BWD_IMG ? 0u : so + TRN_BWD_IMG;
      f32x16 ha = {}, hb = {}, du = {};
      bf16x8 dh[4];
      float ex[16], si[16], sg[16];
      // elementwise work that goes with MFMA w, a pair of elements per stage:
      // dh[0], dh[1] = da and dh[2], dh[3] = db
      auto valu = [&](int w) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int e0 = 2 * (w - 17) + k, e1 = e0 - 2, e2 = e0 - 4, eb = e0 - 6, ea = 2 * (w - 26) + k;
          if (e0 >= 0 && e0 < 16) ex[e0] = __builtin_amdgcn_exp2f(-LOG2E * ha[e0]);
          if (e1 >= 0 && e1 < 16) ex[e1] = __builtin_amdgcn_rcpf(1.f + ex[e1]);
          if (e2 >= 0 && e2 < 16) {
            si[e2] = ha[e2] * ex[e2];                     // a sigmoid(a)
            sg[e2] = fmaf(si[e2], 1.f - ex[e2], ex[e2]);  // sigmoid(a) (1 + a (1 - sigmoid(a)))
          }
          if (eb >= 0 && eb < 16) dh[2 + (eb >> 3)][eb & 7] = (bf16)(du[eb] * si[eb]);
          if (ea >= 0 && ea < 16) dh[ea >> 3][ea & 7] = (bf16)(du[ea] * hb[ea] * sg[ea]);
        }
      };
      auto refill = [&](int i) {
        fq[i % NQ] = i + NQ < 40 ? frag(so, i + NQ) : frag(sn, i + NQ - 40);
      };
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        du = Mma<bf16>::mma(fq[i % NQ], df[i], du);  // du^T = W2 rows . dout^T
        refill(i);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 8; i < 16; ++i) {
        ha = Mma<bf16>::mma(fq[i % NQ], of[i - 8], ha);
        refill(i);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 16; i < 24; ++i) {
        hb = Mma<bf16>::mma(fq[i % NQ], of[i - 16], hb);
        refill(i);
        valu(i);
        __builtin_amdgcn_sched_barrier(0);
      }
      chunk_wait();  // the next chunk has landed; every wave has left the previous one
      lds_barrier();
      issue();
#pragma unroll
      for (int i = 24; i < 40; ++i) {
        d1[i & 3] = Mma<bf16>::mma(fq[i % NQ], dh[((i - 24) >> 2) ^ 2], d1[i & 3]);
        refill(i);
        valu(i);
        __builtin_amdgcn_sched_barrier(0);
      }
      so = sn;
    }
    // layer-norm backward: wdy = do1 gamma, dx = rstd (wdy - c1 xhat - c2)
    float xh[4][16], wdy[4][16];
    float c1 = 0.f, c2 = 0.f;
    const bf16* xp = a.x + rc * TRN_C + 4 * g;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bf16x4 xv = *(const bf16x4*)(xp + 32 * t + 8 * j);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = 32 * t + 8 * j + 4 * g + i, v = 4 * j + i;
          xh[t][v] = ((float)xv[i] - mean) * rstd;
          wdy[t][v] = d1[t][v] * gb[0][k];
          c1 = fmaf(xh[t][v], wdy[t][v], c1);
          c2 += wdy[t][v];
        }
      }
    c1 = wave_xor32_sum(c1) * (1.f / TRN_C);
    c2 = wave_xor32_sum(c2) * (1.f / TRN_C);
    f32x16 dx[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) dx[t][v] = (wdy[t][v] - c1 * xh[t][v] - c2) * rstd;
    if (row < a.m) store_row(a.dx, row, g, dx);
  }
  chunk_wait();  // the copies past the last chunk land before the workgroup ends
}

// ---- backward: sums over rows ----------------------------------------------------------
//
// Workgroup (part p, column group cg): rows of part p, hidden columns
// cg * 128 .. + 127.  Wave w owns hidden columns f0 = cg * 128 + 16 w .. + 15
// and keeps W1's a and b columns and W2's rows for them in registers.  All
// products are 16x16x32 MFMAs.  Per block of 32 rows (o1, xhat and dout
// staged in LDS by all threads, shared by the waves):
//   ha, hb, du [32 rows x 16 hidden columns] = o1 W1 (a, b), dout W2^T
//   dh = [da | db] and u = a sigmoid(a) b, one element per lane and register
//   G_a, G_b [128 features x 16] += xhat^T dh,  s += column sums of dh
//   dW2 [16 x 128 out] += u^T dout
// The accumulators of ha, hb and du feed the sums over rows as they are: lane
// group q holds rows 4 q .. + 3 of both 16-row tiles, the eight contraction
// slots of a 16x16x32 operand, and the transposed reads of xhat and dout
// fetch the same rows.
//
// Why 16-wide tiles: the sums' accumulators take 96 registers per 16 hidden
// columns, so at two waves per SIMD a wave can own 16.  32x32 tiles of ha and
// hb then held a and b of the same 16 columns side by side, formed du twice
// and did the elementwise step in both lanes of a pair: 88 instead of 80
// (half-size) MFMA slots, 350 instead of 243 vector instructions and 44
// instead of 40 KB of LDS reads per wave and block: 0.87 ms at m = 768^2,
// F = 512, against 0.68-0.78 ms now (770 GFLOP of MFMAs: 990-1140 TFLOP/s; the
// launches of one run differ from 0.70 to 0.95 as the clock follows the load).
// A loop of nothing but this mix of MFMAs, LDS reads and vector instructions
// (80 : 56 : 280), two waves per SIMD on random operands, takes 2.24 us per
// block, 0.645 ms for this shape: issue and the clock under that load bound the
// kernel.  Its matrix cores are busy 49% of the time, its LDS 45%, a third of
// that for bank conflicts.  Four waves of 32 columns (one per
// SIMD, 490 registers) measured 0.735 ms: one wave issues at most an
// instruction every four to five cycles.
// The x and dout tiles are stored as four 32-column blocks of 64-byte rows
// (blk_off).

// One ring slot: o1 (bf16), xhat (bf16), dout and the low part of o1
// (o1 - bf16(o1), rounded to bf16) tiles of 32 rows, each as four 32-column
// blocks of 64-byte rows (blk_off).  The staging threads normalise once per
// block for all waves.  a and b are recomputed from o1 as the pair hi + lo:
// rounding o1 to one bf16 moves a and b by up to 2^-9 of the l2 norm of
// their terms, which is large against a or b where the terms cancel, and a
// sum over a few rows does not average that out.
// Blocks sit W_BLK bytes apart (2 KB + 64): the staging stores of one wave
// touch the four blocks of a row at once, and the extra 64 bytes put them on
// different banks.  Every read stays inside one block.
constexpr int W_BLK = 2048 + 64;
constexpr int W_TILE = 4 * W_BLK;
constexpr int W_SLOT = 4 * W_TILE;
constexpr int W_XH = W_TILE, W_DO = 2 * W_TILE, W_OL = 3 * W_TILE;

// One operand of two transposed reads (rows in the order described above).
// This kernel stages through registers, so the compiler's own waits serve.
typedef short s16x4_v __attribute__((__vector_size__(4 * sizeof(short))));
__device__ inline bf16x8 tr_pair(uint32_t a0, uint32_t a1) {
  const auto lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((TRIATTN_LDS s16x4_v*)(uintptr_t)a0);
  const auto hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((TRIATTN_LDS s16x4_v*)(uintptr_t)a1);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

__global__ __launch_bounds__(TRN_THREADS, 1) void trn_bwd_w_kernel(TrnBwdArgs a, int64_t rpp) {
  __shared__ __align__(16) char ring[2][W_SLOT];
  const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, l16 = lane & 15;
  const int wave = tid >> 6;
  const int f = a.f, p = blockIdx.x, cg = blockIdx.y;
  const int f0 = cg * TRN_GROUP + 16 * wave;
  const int fl = f0 + l16;  // this lane's hidden column: columns fl (a) and f + fl (b) of W1
  const int64_t r0 = (int64_t)p * rpp, r1 = r0 + rpp < a.m ? r0 + rpp : a.m;
  const int nb = r1 > r0 ? (int)((r1 - r0 + 31) / 32) : 0;

  // the wave's B operands W1[k][fl], W1[k][f + fl] and W2[fl][k],
  // k = 32 s + 8 q + e, kept in registers for the whole launch (read from the
  // chunk images, which hold them 8 features at a time)
  const char* img = a.img + (int64_t)(f0 / TRN_FC) * TRN_BWD_IMG;
  bf16x8 w1a[4], w1b[4], w2r[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const char* o = img + ((f0 & 31) + l16) * P1 + 16 * (4 * s + q);
    w1a[s] = *(const bf16x8*)o;
    w1b[s] = *(const bf16x8*)(o + OFF_A1B);
    w2r[s] = *(const bf16x8*)(o + OFF_A3);
  }

  // staging: thread tid takes 8 features (chunk tid % 16) of row tid / 16:
  // x, dout and the row's statistics; it writes o1 (hi and lo), xhat and dout
  // in bf16.  Rows past the part's end read as zeros (range-checked loads):
  // their dh is zero, so they contribute nothing.
  const int sr = tid >> 4, sc = tid & 15;
  const uint32_t soff = (sc >> 2) * W_BLK + blk_off(sr, sc & 3);
  float gm[8], bt[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    gm[e] = (float)a.gamma[8 * sc + e];
    bt[e] = (float)a.beta[8 * sc + e];
  }
  struct Staged {
    u32x4 x, d;
    uint32_t mean, rstd;
  };
  auto stage_load = [&](int ib, Staged& v) {
    const int64_t row = r0 + 32 * (int64_t)ib;
    const uint32_t left = (uint32_t)min(r1 - row, (int64_t)32);
    const rsrc_t rx = buf_rsrc_n(a.x + row * TRN_C, left * TRN_C * 2);
    const rsrc_t rd = buf_rsrc_n(a.dout + row * TRN_C, left * TRN_C * 2);
    const rsrc_t rm = buf_rsrc_n(a.mean + row, left * 4), rr = buf_rsrc_n(a.rstd + row, left * 4);
    v.x = __builtin_amdgcn_raw_buffer_load_b128(rx, 16 * tid, 0, 0);
    v.d = __builtin_amdgcn_raw_buffer_load_b128(rd, 16 * tid, 0, 0);
    v.mean = __builtin_amdgcn_raw_buffer_load_b32(rm, 4 * sr, 0, 0);
    v.rstd = __builtin_amdgcn_raw_buffer_load_b32(rr, 4 * sr, 0, 0);
  };
  auto stage_store = [&](char* slot, const Staged& v) {
    const bf16x8 x = __builtin_bit_cast(bf16x8, v.x);
    const float mean = __uint_as_float(v.mean), rstd = __uint_as_float(v.rstd);
    bf16x8 o1, ol, xh;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float h = ((float)x[e] - mean) * rstd;
      xh[e] = (bf16)h;
      const float o = fmaf(h, gm[e], bt[e]);
      o1[e] = (bf16)o;
      ol[e] = (bf16)(o - (float)o1[e]);
    }
    *(bf16x8*)(slot + soff) = o1;
    *(bf16x8*)(slot + W_XH + soff) = xh;
    *(u32x4*)(slot + W_DO + soff) = v.d;
    *(bf16x8*)(slot + W_OL + soff) = ol;
  };

  f32x4 Ga[8] = {}, Gb[8] = {}, W2a[8] = {};
  float sa = 0.f, sb = 0.f;
  // Row m of a 16-row tile is x row perm(m) (bits 2 and 3 swapped), so that
  // lane groups 2 i and 2 i + 1 of a transposed read take rows 8 apart, whose
  // pieces the slot permutation puts on different banks.
  const int prow = (l16 & 3) | ((l16 & 4) << 1) | ((l16 & 8) >> 1);
  const uint32_t ao = blk_off(prow, q);  // rows perm(l16) (+ 16: + 1024), features 8 q ..
  // transposed reads: lane 4 e + j of group q supplies columns 4 j .. + 3 of
  // row perm(4 q + e); columns 16 further on are two chunks further (to[1])
  const int trow = ((lane >> 2) & 3) | ((q & 1) << 3) | ((q & 2) << 1);
  const uint32_t to[2] = {(uint32_t)(blk_off(trow, (lane >> 1) & 1) + 8 * (lane & 1)),
                          (uint32_t)(blk_off(trow, 2 + ((lane >> 1) & 1)) + 8 * (lane & 1))};

  Staged sv;
  if (nb > 0) {
    stage_load(0, sv);
    stage_store(ring[0], sv);
    stage_load(min(1, nb - 1), sv);
  }
  __syncthreads();
  for (int ib = 0; ib < nb; ++ib) {
    const uint32_t cur = lds_addr(ring[ib & 1]);
    // hidden tiles: rows = x rows, lanes = hidden columns
    f32x4 ha[2] = {}, hb[2] = {}, du[2] = {};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const uint32_t o = cur + ao + s * W_BLK + 1024 * r;
        const bf16x8 oh = lds_load16<bf16x8>(o), ol = lds_load16<bf16x8>(o + W_OL);
        const bf16x8 dd = lds_load16<bf16x8>(o + W_DO);
        ha[r] = mma16(oh, w1a[s], ha[r]);
        hb[r] = mma16(oh, w1b[s], hb[r]);
        du[r] = mma16(dd, w2r[s], du[r]);
        ha[r] = mma16(ol, w1a[s], ha[r]);
        hb[r] = mma16(ol, w1b[s], hb[r]);
      }
    stage_store(ring[(ib + 1) & 1], sv);
    stage_load(min(ib + 2, nb - 1), sv);
    // dh = [da | db] as bf16 pairs and u, in the slot order of the sums over rows
    bf16x8 ah, al, bh, bl, uf;
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      const float av = ha[v >> 2][v & 3], bv = hb[v >> 2][v & 3], dv = du[v >> 2][v & 3];
      const float sg = sigm(av), si = av * sg;
      const float da = dv * (bv * fmaf(si, 1.f - sg, sg));  // b sigmoid(a) (1 + a (1 - sigmoid(a)))
      const float db = dv * si;
      sa += da;
      sb += db;
      ah[v] = (bf16)da;
      al[v] = (bf16)(da - (float)ah[v]);
      bh[v] = (bf16)db;
      bl[v] = (bf16)(db - (float)bh[v]);
      uf[v] = (bf16)(si * bv);
    }
    // the first step's fragments are read and waited for at once; the others'
    // reads are the compiler's to place under the MFMAs before them (3.5%
    // faster than a wait per step)
    s16x4 tr0[4];
    tr_read4_wait(cur + to[0] + W_XH, cur + to[0] + W_XH + 1024, cur + to[0] + W_DO,
                  cur + to[0] + W_DO + 1024, tr0);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const uint32_t o = cur + to[t & 1] + (t >> 1) * W_BLK;
      const bf16x8 xf = t == 0 ? tr_frag(tr0, 0) : tr_pair(o + W_XH, o + W_XH + 1024);
      const bf16x8 df = t == 0 ? tr_frag(tr0, 1) : tr_pair(o + W_DO, o + W_DO + 1024);
      Ga[t] = mma16(xf, ah, Ga[t]);
      Gb[t] = mma16(xf, bh, Gb[t]);
      W2a[t] = mma16(uf, df, W2a[t]);
      Ga[t] = mma16(xf, al, Ga[t]);
      Gb[t] = mma16(xf, bl, Gb[t]);
    }
    __syncthreads();
  }

  // partial sums of part p: G [C][2F], s [2F], dW2 [F][C]; 16x16 accumulators:
  // lane group q holds rows 4 q + i of column l16
  float* out = a.part + (int64_t)p * trn_part_floats(f);
  float* w2o = out + (int64_t)TRN_C * 2 * f + 2 * f;
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float* o = out + (int64_t)(16 * t + 4 * q + i) * 2 * f + fl;
      o[0] = Ga[t][i];
      o[f] = Gb[t][i];
      w2o[(int64_t)(f0 + 4 * q + i) * TRN_C + 16 * t + l16] = W2a[t][i];
    }
  sa += __shfl_xor(sa, 16);
  sb += __shfl_xor(sb, 16);
  sa = wave_xor32_sum(sa);
  sb = wave_xor32_sum(sb);
  if (q == 0) {
    out[(int64_t)TRN_C * 2 * f + fl] = sa;
    out[(int64_t)TRN_C * 2 * f + f + fl] = sb;
  }
}

// Fixed-order sum of the partial blocks: G and s into gsum (part 0's place:
// an entry is read and written by one thread only), dW2 into its output.
__global__ __launch_bounds__(256) void trn_reduce_kernel(TrnBwdArgs a) {
  const int64_t per = trn_part_floats(a.f);
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= per) return;
  float s = 0.f;
#pragma unroll 16
  for (int p = 0; p < a.nparts; ++p) s += a.part[(int64_t)p * per + i];
  const int64_t ng = (int64_t)TRN_C * 2 * a.f + 2 * a.f;
  if (i < ng)
    a.gsum[i] = s;
  else
    a.dw2[i - ng] = s;
}

// dW1 = gamma G + beta s^T, dgamma = sum_n W1 o G, dbeta = W1 s; one
// workgroup per feature, fixed-order tree over the columns.
__global__ __launch_bounds__(256) void trn_finish_kernel(TrnBwdArgs a) {
  __shared__ float red[2][256];
  const int k = blockIdx.x, tid = threadIdx.x, n = 2 * a.f;
  const float gm = (float)a.gamma[k], bt = (float)a.beta[k];
  const float* G = a.gsum + (int64_t)k * n;
  const float* s = a.gsum + (int64_t)TRN_C * n;
  float dg = 0.f, db = 0.f;
  for (int c = tid; c < n; c += 256) {
    const float w = (float)a.w1[(int64_t)k * n + c];
    a.dw1[(int64_t)k * n + c] = gm * G[c] + bt * s[c];
    dg = fmaf(w, G[c], dg);
    db = fmaf(w, s[c], db);
  }
  red[0][tid] = dg;
  red[1][tid] = db;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) {
      red[0][tid] += red[0][tid + w];
      red[1][tid] += red[1][tid + w];
    }
    __syncthreads();
  }
  if (tid == 0) {
    a.dgamma[k] = red[0][0];
    a.dbeta[k] = red[1][0];
  }
}

constexpr int TRN_GRID = 256;  // persistent workgroups (one per CU)

}  // namespace

int trn_bwd_parts(int64_t m, int f) {
  const int groups = f / TRN_GROUP;
  int p = TRN_GRID / groups;
  if (p < 1) p = 1;
  const int64_t blocks = (m + 31) / 32;
  if (p > blocks) p = (int)blocks;
  return p;
}

hipError_t launch_trn_fwd(const TrnFwdArgs& a, hipStream_t s) {
  const int64_t slots = (int64_t)(a.f / TRN_FC) * (TRN_FWD_IMG / 16);
  {
    KernelTimer t(K_TRN_PACK, s);
    hipLaunchKernelGGL(trn_pack_kernel, dim3((unsigned)((slots + 255) / 256)), dim3(256), 0, s,
                       a.w1, a.w2, a.f, 0, a.img);
  }
  const int64_t nblk = (a.m + TRN_ROWS - 1) / TRN_ROWS;
  {
    KernelTimer t(K_TRN_FWD, s);
    hipLaunchKernelGGL(trn_fwd_kernel, dim3((unsigned)std::min<int64_t>(nblk, TRN_GRID)),
                       dim3(TRN_THREADS), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_trn_bwd(const TrnBwdArgs& a, hipStream_t s) {
  const int64_t slots = (int64_t)(a.f / TRN_FC) * (TRN_BWD_IMG / 16);
  {
    KernelTimer t(K_TRN_PACK, s);
    hipLaunchKernelGGL(trn_pack_kernel, dim3((unsigned)((slots + 255) / 256)), dim3(256), 0, s,
                       a.w1, a.w2, a.f, 1, a.img);
  }
  const int64_t nblk = (a.m + TRN_ROWS - 1) / TRN_ROWS;
  {
    KernelTimer t(K_TRN_BWD_DX, s);
    hipLaunchKernelGGL(trn_bwd_dx_kernel, dim3((unsigned)std::min<int64_t>(nblk, TRN_GRID)),
                       dim3(TRN_THREADS), 0, s, a);
  }
  {
    // rows per part: a multiple of 32
    const int64_t blocks = (a.m + 31) / 32;
    const int64_t rpp = (blocks + a.nparts - 1) / a.nparts * 32;
    KernelTimer t(K_TRN_BWD_W, s);
    hipLaunchKernelGGL(trn_bwd_w_kernel, dim3((unsigned)a.nparts, (unsigned)(a.f / TRN_GROUP)),
                       dim3(TRN_THREADS), 0, s, a, rpp);
  }
  {
    const int64_t per = trn_part_floats(a.f);
    KernelTimer t(K_TRN_REDUCE, s);
    hipLaunchKernelGGL(trn_reduce_kernel, dim3((unsigned)((per + 255) / 256)), dim3(256), 0, s,
                       a);
  }
  {
    KernelTimer t(K_TRN_FINISH, s);
    hipLaunchKernelGGL(trn_finish_kernel, dim3(TRN_C), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace triattn

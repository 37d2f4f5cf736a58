// Per-call preparation shared by the forward and the backward: the bias in
// accumulator order and the key-valid bits.  Device pieces for 256-thread
// workgroups; the kernels that run them (prep_kernel in fwd.hip,
// bwd_prep_kernel in bwd.hip) deal a one-dimensional grid over the pieces, so
// that a call spends one launch on all of its preparation: at N = 256 the bias
// and the bits took 4 + 3 us as two launches, nearly all of it launch and
// latency, and they do not depend on each other.
#pragma once

#include "dma.h"
#include "kernels.h"

namespace triattn {

// bias / scale over the zero-padded np x np map, in accumulator order (see
// frag_tile): in tile (t1, t2), element 256 j + 4 l + e has x = 32 t1 + l % 32
// as the lane's column and y = 32 t2 + 8 j + 4 (l / 32) + e as its row.  bt
// holds bias(query x, key y) for the kernels whose lanes own queries; btT
// holds bias(query y, key x) for the kernel whose lanes own keys.  The
// starting node reads bias[q][k][h], the ending node bias[k][q][h].
//
// One workgroup per 32 x 32 block (query tile qa, key tile kb) of the map,
// four heads at a time: the block goes through LDS once and leaves as bt tile
// (qa, kb) and btT tile (kb, qa), both written 16 bytes per thread.
template <typename T>
__device__ inline void load_heads4(const T* p, float (&x)[4]);
template <>
__device__ inline void load_heads4(const bf16* p, float (&x)[4]) {
  const bf16x4 v = *(const bf16x4*)p;
#pragma unroll
  for (int j = 0; j < 4; ++j) x[j] = (float)v[j];
}
template <>
__device__ inline void load_heads4(const float* p, float (&x)[4]) {
  const f32x4 v = *(const f32x4*)p;
#pragma unroll
  for (int j = 0; j < 4; ++j) x[j] = v[j];
}

template <typename T>
__device__ inline void prep_bias_block(const Geom& G, int node, int block, const T* bias,
                                       float* bt, float* btT) {
  const int nt = G.nkt, n = G.n;
  const int qa = block % nt, kb = block / nt;
  const int tid = threadIdx.x;
  constexpr int HG = 4;  // heads per pass through LDS
  __shared__ float tl[HG][32][33];  // [head][query][key] of HG heads: bias / scale
  // loads: query r, keys c0 .. c0 + 3 of the block, HG heads each (one
  // vector load per key when the head count is a multiple of HG)
  const int r = tid >> 3, c0 = 4 * (tid & 7);
  const int q = 32 * qa + r;
  const bool vec = G.H % HG == 0;
  // stores: element 4 tid .. 4 tid + 3 of a tile (j = tid / 64, l = tid % 64)
  const int l = tid & 63, x = l & 31, y0 = 8 * (tid >> 6) + 4 * (l >> 5);
  for (int h0 = 0; h0 < G.H; h0 += HG) {
    const int hn = min(HG, G.H - h0);
    float v[4][HG];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = 32 * kb + c0 + e;
      const int qc = min(q, n - 1), kc = min(k, n - 1);  // in bounds; zero outside the map
      const int64_t at = (node == 0 ? (int64_t)qc * n + kc : (int64_t)kc * n + qc) * G.H + h0;
      if (vec) {
        load_heads4(bias + at, v[e]);
      } else {
#pragma unroll
        for (int j = 0; j < HG; ++j) v[e][j] = j < hn ? (float)bias[at + j] : 0.f;
      }
      if (!(q < n && k < n)) {
#pragma unroll
        for (int j = 0; j < HG; ++j) v[e][j] = 0.f;
      }
    }
    __syncthreads();  // the previous heads' tiles have been read
#pragma unroll
    for (int j = 0; j < HG; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) tl[j][r][c0 + e] = v[e][j] / G.scale;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < HG; ++j) {
      if (j >= hn) break;
      const int h = h0 + j;
      const f32x4 o = {tl[j][x][y0], tl[j][x][y0 + 1], tl[j][x][y0 + 2], tl[j][x][y0 + 3]};
      *(f32x4*)(bt + (((int64_t)h * nt + qa) * nt + kb) * 1024 + 4 * tid) = o;
      if (btT) {
        const f32x4 p = {tl[j][y0][x], tl[j][y0 + 1][x], tl[j][y0 + 2][x], tl[j][y0 + 3][x]};
        *(f32x4*)(btT + (((int64_t)h * nt + kb) * nt + qa) * 1024 + 4 * tid) = p;
      }
    }
  }
}

// kbits[row][t]: bit e set iff key 32 t + e < n and mask(row, key) != 0.
// rowfull[row] = 1 iff every key < n is valid for the row.
//
// Starting node, mask[row][key] (a row's keys contiguous): one workgroup per
// row; each wave reads 64 consecutive keys per load and forms two words with
// a ballot.
__device__ inline void prep_kbits_start(const Geom& G, int row, const uint8_t* mask,
                                        uint32_t* kbits, uint32_t* rowfull) {
  const int n = G.n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bool full = true;
  for (int k0 = 64 * wave; k0 < G.np; k0 += 256) {
    const int key = k0 + lane;
    const bool in = key < n;
    const bool ok = in && (mask == nullptr || mask[(int64_t)row * n + min(key, n - 1)] != 0);
    const uint64_t b = __ballot(ok), want = __ballot(in);
    full = full && b == want;
    const int t = k0 >> 5;
    if (lane == 0) kbits[(int64_t)row * G.nkt + t] = (uint32_t)b;
    if (lane == 1 && t + 1 < G.nkt) kbits[(int64_t)row * G.nkt + t + 1] = (uint32_t)(b >> 32);
  }
  const int all = __syncthreads_and(full);
  if (threadIdx.x == 0) rowfull[row] = all ? 1u : 0u;
}

// Ending node, mask[key][row] (consecutive rows contiguous): one workgroup
// per 64 rows, lane <-> row; wave w builds words w, w + 4, ... of the 64
// rows, one 64-byte read of a key's row of the mask per bit.
__device__ inline void prep_kbits_end(const Geom& G, int block, const uint8_t* mask,
                                      uint32_t* kbits, uint32_t* rowfull) {
  const int n = G.n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = 64 * block + lane;
  const bool rin = row < G.nr;
  const int rowc = min(row, G.nr - 1);  // in-bounds address for lanes past the last row
  bool full = true;
  for (int t = wave; t < G.nkt; t += 4) {
    const uint32_t want = in_range_bits(t, n);
    uint32_t bits = rin ? want : 0u;
    if (mask != nullptr) {
      // every load first (addresses clamped in bounds), then the bits
      uint8_t m[32];
#pragma unroll
      for (int e = 0; e < 32; ++e) m[e] = mask[(int64_t)min(32 * t + e, n - 1) * n + rowc];
#pragma unroll
      for (int e = 0; e < 32; ++e)
        if (m[e] == 0) bits &= ~(1u << e);
    }
    if (rin) kbits[(int64_t)row * G.nkt + t] = bits;
    full = full && bits == want;
  }
  __shared__ uint32_t part[4][64];
  part[wave][lane] = full ? 1u : 0u;
  __syncthreads();
  if (wave == 0 && rin) {
    uint32_t all = 1u;
#pragma unroll
    for (int w = 0; w < 4; ++w) all &= part[w][lane];
    rowfull[row] = all;
  }
}

// Workgroups of the key bits; the bias takes nkt * nkt more.
inline unsigned prep_kbits_blocks(const Geom& g, int node) {
  return (unsigned)(node == 0 ? g.nr : (g.nr + 63) / 64);
}
inline unsigned prep_blocks(const Geom& g, int node) {
  return prep_kbits_blocks(g, node) + (unsigned)(g.nkt * g.nkt);
}

// Block `b` of the preparation (b < prep_blocks): the key bits first, their
// chains of dependent loads being the longer.
template <typename T>
__device__ inline void prep_block(const Geom& G, int node, int b, int nkb, const T* bias,
                                  const uint8_t* mask, const Prep& p) {
  if (b >= nkb)
    prep_bias_block(G, node, b - nkb, at_sample(bias, G.bBias), ws_at_sample(p.bt, G.bWs),
                    ws_at_sample(p.btT, G.bWs));
  else if (node == 0)
    prep_kbits_start(G, b, at_sample(mask, G.bMask), ws_at_sample(p.kbits, G.bWs),
                     ws_at_sample(p.rowfull, G.bWs));
  else
    prep_kbits_end(G, b, at_sample(mask, G.bMask), ws_at_sample(p.kbits, G.bWs),
                   ws_at_sample(p.rowfull, G.bWs));
}

}  // namespace triattn

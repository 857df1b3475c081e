// Batched-row GEMMs on MFMA: y[m][n] = sum_k x[m][k] W[n][k] for up to
// SPEC_MAX_ROWS rows, with the same fused epilogues as the thin GEMV kernels
// (1/rms row scale, rotary + paged KV append, residual + next-norm input,
// SwiGLU, per-tile argmax, or k-split partial sums).  Two kernels:
//   * k_gemm_wide (below k_gemm): passes of more than 32 rows over the
//     tile-packed weights (several sequences verified together);
//   * k_gemm: row-major weights (SPEC_FLAG_ROWMAJOR) for passes of more than
//     16 rows, 17..32-row passes whose width the thin GEMV cannot stage, and
//     the q/k/v projection of wider packed passes where it is not k-split
//     (narrow models).
//
// k_gemm: a workgroup owns kGemmTiles = 4 output tiles of 16 columns and the k-range
// of split blockIdx.y, walked in chunks of 32 * kSteps columns (kSteps
// 32-wide MFMA steps; kSteps = 4 or 2 by the row count).  It has two kinds
// of waves:
//   * 2 * kSteps MFMA waves.  Wave w = 2q + p multiplies tile pair p (tiles
//     2p, 2p+1) by step q of every chunk: each x operand it reads from LDS
//     feeds two MFMAs, and the step groups split the k-range (their partial
//     tiles are summed through LDS at the end).  They stream only weights,
//     kStages chunks ahead.
//   * 4 loader waves.  They stage every chunk's x rows (all rows) into one of
//     two LDS buffers, loading kStages chunks ahead.
// Loads complete in issue order per wave, so a wave that waited for x would
// also wait for every weight load issued before it; with x in waves of its
// own, the weight loads stay kStages chunks deep.  One workgroup barrier per
// chunk hands a staged buffer to the MFMA waves; barriers wait for LDS
// traffic only, never for loads in flight.  Both loops run a whole number of
// kStages-chunk rounds with no early exit (chunks past the k-range load
// nothing and add zeros): an exit inside the unrolled round would make the
// compiler drain every load in flight at the loop head.
//
// v_mfma_f32_16x16x32_bf16 takes the weight fragment as A (lane l: row l&15,
// k 8*(l>>4)..+8) and x^T as B (lane l: x row l&15, same k); lane l then
// holds y[n0 + 4*(l>>4) + i][row l&15 of the block] for each 16-row block.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>

#include "ctx.h"
#include "device.h"
#include "gemv.h"
#include "sgemv.h"

namespace specdec {

namespace {

constexpr int kLoadWaves = 4;                 // waves that stage x
constexpr int kOut = 0x7FFFFF00;              // buffer offset past every operand: the load returns zeros
constexpr int kRsrcWord3 = 0x00020000;        // raw buffer resource, 32-bit data
constexpr int kNt = 2;                        // non-temporal hint of the weight loads
constexpr int NL = kLoadWaves * 64;           // loader threads
constexpr int kYStride = 17;                  // floats per row of an output tile in LDS

// Step groups (32-wide k-steps per chunk, one MFMA wave pair each) and chunks
// of loads in flight, by 16-row blocks: up to 3 blocks 2 groups and 8 chunks
// (8 waves of at most 128 registers: two workgroups per CU); 4-5 blocks 4
// groups and 5 chunks (12 waves, 168 registers each); from 6 blocks, whose
// accumulators need more registers, 2 groups and 8 chunks (8 waves of 256).
// The compiler waits for all of a wave's loads once per round of kStages
// chunks, so a deep round is what keeps enough bytes in flight per CU.
constexpr int steps_for(int mb) { return (mb >= 6 || mb <= 3) ? 2 : 4; }
constexpr int stages_for(int mb) { return (mb >= 6 || mb <= 3) ? 8 : 5; }
constexpr int threads_for(int mb) { return (2 * steps_for(mb) + kLoadWaves) * 64; }
constexpr int xstride_for(int mb) { return 32 * steps_for(mb) + 8; }   // bf16 per LDS x row (16-byte pad)
static_assert(kGemmTiles == 4, "MFMA wave w = 2q + p: tile pair p, step group q");
// Sums of squares each thread of the 1/rms prologue loads, with `parts`
// threads per row: enough for hidden 8192 (512 sums) where registers allow.
constexpr int lpt_for(int parts) { return (512 + parts - 1) / parts < 96 ? (512 + parts - 1) / parts : 96; }

// two x buffers of 16 mb rows plus a spare row each (the target of loader
// stores past the last row, so that no branch skips a store)
size_t x_lds_bytes(int mb) { return (size_t)2 * (16 * mb + 1) * xstride_for(mb) * sizeof(bf16_t); }
// output tiles, plus (4 step groups) the partial tiles of groups 2 and 3 while they are summed
size_t y_lds_bytes(int mb) {
  return (size_t)(steps_for(mb) == 4 ? 2 : 1) * kGemmTiles * (16 * mb) * kYStride * sizeof(float);
}

template <int MB, int EPI>
__global__ __launch_bounds__(threads_for(MB)) void k_gemm(GemvArgs a) {
  constexpr int ROWS = MB * 16;
  constexpr int kSteps = steps_for(MB), kStages = stages_for(MB), NT = threads_for(MB);
  constexpr int kMfmaWaves = 2 * kSteps;
  constexpr int kChunk = 32 * kSteps;                         // k columns per stage
  constexpr int kXStride = xstride_for(MB);
  constexpr int CV = kChunk / 8;                              // x vectors per row and chunk
  constexpr int XV = (ROWS * CV + NL - 1) / NL;               // x vectors per loader thread and chunk
  constexpr bool kNorm = EPI == EPI_ROPE || EPI == EPI_SWIGLU || EPI == EPI_ARGMAX;
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ float inv_rms[ROWS];
  __shared__ int live_s[ROWS];
  __shared__ float rms_part[kNorm ? NT : 1];

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const bool loader = wave >= kMfmaWaves;                    // wave-uniform role
  const int pair = wave & 1, q = (wave >> 1) & (kSteps - 1);
  const int lt = threadIdx.x - kMfmaWaves * 64;               // loader thread index
  const int split = blockIdx.y;
  const int Kd = a.Kd, M = a.M, N = a.N;
  const int T = (Kd + 31) >> 5;
  const int s0 = (int)((long long)split * T / a.splits);
  const int s1 = (int)((long long)(split + 1) * T / a.splits);
  const int nch = (s1 - s0 + kSteps - 1) / kSteps;
  const int kq = 8 * (lane >> 4);
  const int kend = min(s1 * 32, Kd);

  // Weights are read through buffer resources, x through one over its rows:
  // every load is issued unconditionally, and one that a lane does not need
  // (past the split, a dead row, a tile past N) gets offset kOut and returns
  // zeros without a memory access.  With no branch around a load, the
  // compiler's wait counts stay exact and loads stay kStages chunks deep.
  //
  // MFMA waves, tile t of the pair: on the tile-packed copy, block (tile,
  // step) is 1 KB at (tile * T + step) * 1 KB with lane l at 16 l; on
  // row-major weights, lane l reads row l & 15 of the tile.  SwiGLU tiles
  // come in pairs on both (tile 2c: gate rows 16c..16c+16, tile 2c+1: the up
  // rows of the same features), so every tile is one load per step.
  const bool packed = a.pw != nullptr;
  __amdgpu_buffer_rsrc_t rw[2];
  int wbase[2];          // byte offset of this lane's fragment at step 0 (kOut: tile unused)
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int tile = blockIdx.x * kGemmTiles + 2 * pair + t;
    const int n0 = tile * kTile;
    const bool on = !loader && n0 < N;
    const int r = lane & 15;
    if (packed) {
      rw[t] = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.pw), 0, (N / kTile) * T * 1024, kRsrcWord3);
      wbase[t] = on ? tile * T * 1024 + 16 * lane : kOut;
    } else if constexpr (EPI == EPI_SWIGLU) {
      const int F = N / 2;
      rw[t] = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.w[tile & 1]), 0, F * Kd * 2, kRsrcWord3);
      wbase[t] = on ? (((tile >> 1) * kTile + r) * Kd + kq) * 2 : kOut;
    } else {
      int sg = 0;
#pragma unroll
      for (int i = 1; i < 3; ++i)
        if (i < a.nseg && n0 >= a.row0[i]) sg = i;
      const int rows = (sg + 1 < a.nseg ? a.row0[sg + 1] : N) - a.row0[sg];
      rw[t] = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.w[sg]), 0, rows * Kd * 2, kRsrcWord3);
      wbase[t] = on ? ((n0 - a.row0[sg] + r) * Kd + kq) * 2 : kOut;
    }
  }
  const __amdgpu_buffer_rsrc_t rx =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.x), 0, M * a.ldx * 2, kRsrcWord3);

  // live rows: row m is row m % rps of sequence m / rps, live while below
  // that sequence's row count
  for (int m = threadIdx.x; m < ROWS; m += NT) {
    int lv = 0;
    if (m < M) {
      const int b = m / a.rps;
      lv = (m - b * a.rps) < a.st[b].count ? 1 : 0;
    }
    live_s[m] = lv;
  }
  __syncthreads();

  // 1/rms of each live row from the per-16-column sums of squares, at the
  // start.  ss_in is [H/16][mpad]: for one column group the rows are
  // contiguous, so thread (part p, row m) sums groups p*per .. (p+1)*per - 1
  // of row m with loads that are coalesced across the rows, all issued before
  // the first add (one memory round trip per workgroup); the parts are then
  // added in order.  inv_rms is read after the K loop's barriers.
  if constexpr (kNorm) {
    constexpr int P = NT / ROWS;              // parts per row (>= 3)
    constexpr int LPT = lpt_for(P);           // loads per thread (H/16 <= LPT * P, checked on the host)
    const int nt = a.H / kTile, per = (nt + P - 1) / P;
    const int m = threadIdx.x % ROWS, p = threadIdx.x / ROWS;
    float v[LPT];
#pragma unroll
    for (int j = 0; j < LPT; ++j) v[j] = a.ss_in[(size_t)min(p * per + j, nt - 1) * a.mpad + m];
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < LPT; ++j) sum += (p < P && j < per && p * per + j < nt) ? v[j] : 0.f;
    rms_part[threadIdx.x] = sum;
    __syncthreads();
    if (threadIdx.x < ROWS) {
      float t = 0.f;
      for (int q2 = 0; q2 < P; ++q2) t += rms_part[q2 * ROWS + threadIdx.x];
      inv_rms[threadIdx.x] = live_s[threadIdx.x] ? rsqrtf(t / a.H + a.eps) : 0.f;
    }
  }

  // Loader waves, chunk c: x vector v (v < ROWS*CV) is row v / CV, columns
  // 8*(v % CV) .. +8 of the chunk.  MFMA waves, chunk c: step q of the chunk
  // for both tiles.  Dead rows, columns past the split or past Kd read as
  // zeros (Kd % 8 == 0, so a vector starting below the end lies inside).
  auto issue_x = [&](int c, u32x4 (&xr)[XV]) {
    const int kc = (s0 + kSteps * c) * 32;
#pragma unroll
    for (int i = 0; i < XV; ++i) {
      const int v = lt + NL * i;
      const int m = v / CV, k = kc + 8 * (v % CV);
      const int mm = m < ROWS ? m : ROWS - 1;   // (no branch around the LDS read)
      const bool ok = (v < ROWS * CV) & (m < M) & (live_s[mm] != 0) & (k < kend);
      xr[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? (m * a.ldx + k) * 2 : kOut, 0, 0);
    }
  };
  auto issue_w = [&](int c, u32x4 (&wr)[2]) {
    const int st = s0 + kSteps * c + q;
    const bool ok = packed ? st < s1 : st * 32 + kq < kend;
    const int step_bytes = packed ? 1024 : 64;
#pragma unroll
    for (int t = 0; t < 2; ++t)
      wr[t] = __builtin_amdgcn_raw_buffer_load_b128(rw[t], (ok && wbase[t] != kOut) ? wbase[t] + st * step_bytes : kOut,
                                                    0, kNt);
  };

  bf16_t* xs = reinterpret_cast<bf16_t*>(lds);
  float* y = reinterpret_cast<float*>(lds);   // output tiles once the x buffers are free
  // Both roles pass the same barriers: one per chunk, then the sums' (five
  // with four step groups, three with two).
  if (loader) {
    u32x4 xr[kStages][XV];
#pragma unroll
    for (int u = 0; u < kStages; ++u) issue_x(u, xr[u]);
    for (int c0 = 0; c0 < nch; c0 += kStages) {   // workgroup-uniform
#pragma unroll
      for (int u = 0; u < kStages; ++u) {
        const int c = c0 + u;   // chunks past the last one load nothing and stage zeros
        // buffer c&1 was last read in chunk c-2, before every wave passed
        // chunk c-1's barrier
        bf16_t* xb = xs + (size_t)(c & 1) * (ROWS + 1) * kXStride;
#pragma unroll
        for (int i = 0; i < XV; ++i) {
          const int v = lt + NL * i;
          const int row = v < ROWS * CV ? v / CV : ROWS;
          *reinterpret_cast<u32x4*>(xb + row * kXStride + 8 * (v % CV)) = xr[u][i];
        }
        issue_x(c + kStages, xr[u]);   // past the last chunk: zeros, no memory access
        __syncthreads();   // chunk c's x rows are visible to every wave
      }
    }
    for (int i = 0; i < (kSteps == 4 ? 5 : 3); ++i) __syncthreads();
  } else {
    u32x4 wr[kStages][2];
#pragma unroll
    for (int u = 0; u < kStages; ++u) issue_w(u, wr[u]);
    f32x4 acc[2][MB];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc[t][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < nch; c0 += kStages) {   // workgroup-uniform
#pragma unroll
      for (int u = 0; u < kStages; ++u) {
        const int c = c0 + u;   // chunks past the last one multiply zeros
        const bf16_t* xb = xs + (size_t)(c & 1) * (ROWS + 1) * kXStride;
        __syncthreads();   // chunk c's x rows are visible to every wave
        const u32x4 w0 = wr[u][0], w1 = wr[u][1];
        issue_w(c + kStages, wr[u]);   // past the last chunk: zeros, no memory access
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const u32x4 xv = *reinterpret_cast<const u32x4*>(xb + (mb * 16 + (lane & 15)) * kXStride + 32 * q + kq);
          acc[0][mb] = mfma16x16x32(w0, xv, acc[0][mb]);
          acc[1][mb] = mfma16x16x32(w1, xv, acc[1][mb]);
        }
      }
    }
    __syncthreads();   // 1: x buffers are free

    // Sum the step groups' partial tiles in a fixed order, ((q0 + q2) + (q1 + q3))
    // with four groups (2 and 3 store, 0 and 1 add; 1 stores, 0 adds) or
    // q0 + q1 with two; group 0 scales by 1/rms and leaves the result in
    // y[tile][m][c].
    auto tile_at = [&](float* base, int t, int mb, int i) -> float& {
      const int m = mb * 16 + (lane & 15);
      return base[((2 * pair + t) * ROWS + m) * kYStride + 4 * (lane >> 4) + i];
    };
    auto store = [&](float* dst) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int i = 0; i < 4; ++i) tile_at(dst, t, mb, i) = acc[t][mb][i];
    };
    if constexpr (kSteps == 4) {
      float* yp = y + (size_t)kGemmTiles * ROWS * kYStride;   // the upper partial tiles
      if (q >= 2) store(q == 2 ? y : yp);
      __syncthreads();   // 2
      if (q < 2) {
        float* src = q == 0 ? y : yp;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[t][mb][i] += tile_at(src, t, mb, i);
      }
      __syncthreads();   // 3
    }
    if (q == 1) store(y);
    __syncthreads();   // 4 (two groups: 2)
    if (q == 0) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const float sc = kNorm ? inv_rms[mb * 16 + (lane & 15)] : 1.f;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float& d = tile_at(y, t, mb, i);
            d = (acc[t][mb][i] + d) * sc;
          }
        }
    }
    __syncthreads();   // 5 (two groups: 3)
  }

  // epilogues: items of (tile w, row m, column or pair)
  if constexpr (EPI == EPI_STORE) {
    for (int idx = threadIdx.x; idx < kGemmTiles * ROWS * 16; idx += NT) {
      const int w = idx / (ROWS * 16), r = idx % (ROWS * 16), m = r >> 4, cc = r & 15;
      const int nw = (blockIdx.x * kGemmTiles + w) * kTile;
      if (nw < N && m < M) a.out[((size_t)split * M + m) * N + nw + cc] = y[(w * ROWS + m) * kYStride + cc];
    }
  } else if constexpr (EPI == EPI_ROPE) {
    for (int idx = threadIdx.x; idx < kGemmTiles * ROWS * 8; idx += NT) {
      const int w = idx / (ROWS * 8), r = idx % (ROWS * 8), m = r >> 3, pr = r & 7;
      const int nw = (blockIdx.x * kGemmTiles + w) * kTile;
      if (nw >= N || m >= M || !live_s[m]) continue;
      const int b = m / a.rps, j = m - b * a.rps;
      const int slot = a.st[b].base + j;
      const int head = nw / a.D, d = ((nw % a.D) >> 1) + pr;
      const float e = y[(w * ROWS + m) * kYStride + 2 * pr], o = y[(w * ROWS + m) * kYStride + 2 * pr + 1];
      if (head < a.nq + a.nkv) {
        const float2 cs = a.rcs[(size_t)m * (a.D / 2) + d];
        const float re = e * cs.x - o * cs.y, ro = e * cs.y + o * cs.x;
        if (head < a.nq) {
          *reinterpret_cast<uint32_t*>(a.q + ((size_t)m * a.nq + head) * a.D + 2 * d) = pack2(re, ro);
        } else {
          const size_t pg = (size_t)a.pt[b * a.pps + slot / kAttnChunk] * a.nkv + (head - a.nq);
          *reinterpret_cast<uint32_t*>(a.kc + (pg * kAttnChunk + slot % kAttnChunk) * a.D + 2 * d) =
              pack2(re, ro);
        }
      } else {
        const size_t pg = (size_t)a.pt[b * a.pps + slot / kAttnChunk] * a.nkv + (head - a.nq - a.nkv);
        bf16_t* vp = a.vt + (pg * a.D + 2 * d) * kAttnChunk + slot % kAttnChunk;
        vp[0] = f2bf(e);
        vp[kAttnChunk] = f2bf(o);
      }
    }
  } else if constexpr (EPI == EPI_RESID) {
    // 16 consecutive threads share (w, m): the row's sum of squares over the
    // tile is a 16-lane reduction
    for (int idx = threadIdx.x; idx < kGemmTiles * ROWS * 16; idx += NT) {
      const int w = idx / (ROWS * 16), r = idx % (ROWS * 16), m = r >> 4, cc = r & 15;
      const int nw = (blockIdx.x * kGemmTiles + w) * kTile;
      const bool ok = nw < N && m < M;
      float xn = 0.f;
      if (ok) {
        const int n = nw + cc;
        xn = a.x32[(size_t)m * N + n];
        if (live_s[m]) {                      // rows of idle sequences keep their stream
          xn += y[(w * ROWS + m) * kYStride + cc];
          a.x32[(size_t)m * N + n] = xn;
        }
        a.xg[(size_t)m * N + n] = f2bf(xn * bf2f(a.gain[n]));
      }
      float sq = xn * xn;
      for (int o = 1; o < 16; o <<= 1) sq += __shfl_xor(sq, o);
      if (ok && cc == 0) a.ss_out[(size_t)(nw / kTile) * a.mpad + m] = sq;
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    // tiles 2j, 2j+1: gate and up rows of features 16 j' .. +16, j' = 2 blockIdx.x + j
    const int F = N / 2;
    for (int idx = threadIdx.x; idx < 2 * ROWS * 16; idx += NT) {
      const int j = idx / (ROWS * 16), r = idx % (ROWS * 16), m = r >> 4, cc = r & 15;
      const int f = (2 * blockIdx.x + j) * kTile + cc;
      if (f >= F || m >= M) continue;
      const float g = y[(2 * j * ROWS + m) * kYStride + cc];
      const float up = y[((2 * j + 1) * ROWS + m) * kYStride + cc];
      a.u[(size_t)m * F + f] = f2bf(g / (1.f + expf(-g)) * up);
    }
  } else {   // EPI_ARGMAX
    bf16_t* lg = a.allow_logits && a.st[0].want_logits ? a.st[0].logits : nullptr;
    if (lg) {
      for (int idx = threadIdx.x; idx < kGemmTiles * ROWS * 16; idx += NT) {
        const int w = idx / (ROWS * 16), r = idx % (ROWS * 16), m = r >> 4, cc = r & 15;
        const int nw = (blockIdx.x * kGemmTiles + w) * kTile;
        if (nw < N && m < M)
          st_global(lg + (size_t)m * N + nw + cc, f2bf(y[(w * ROWS + m) * kYStride + cc]));
      }
    }
    for (int idx = threadIdx.x; idx < kGemmTiles * ROWS; idx += NT) {
      const int w = idx / ROWS, m = idx % ROWS;
      const int nw = (blockIdx.x * kGemmTiles + w) * kTile;
      if (nw >= N || m >= M) continue;
      float best = -INFINITY;
      int bi = nw;
      bool nan = false;
      for (int cc = 0; cc < 16; ++cc) {
        float v = y[(w * ROWS + m) * kYStride + cc];
        if (v != v) {
          nan = true;
          v = -INFINITY;
        }
        if (v > best) {
          best = v;
          bi = nw + cc;
        }
      }
      a.amax_v[(size_t)(nw / kTile) * a.mpad + m] = best;
      a.amax_i[(size_t)(nw / kTile) * a.mpad + m] = bi;
      if (nan && live_s[m]) atomicOr(const_cast<int32_t*>(&a.st[m / a.rps].err), ERR_NUMERIC);
    }
  }
}

// ---------------------------------------------------------------------------
// Wide-unit GEMM over the tile-packed weights for passes of 33 to 160 rows
// (3 to 10 row blocks): the gate/up and LM-head projections in one launch, and
// the q/k/v, o and down projections as k-split partial sums.
//
// A unit is a pair of tiles (32 output columns; a gate/up pair).  A workgroup
// takes a contiguous run of units over the k-range of its split, walked in
// chunks of at most P units.  Two loader waves only stage x; P x KG worker waves
// multiply: worker (p, kg) owns unit p of the chunk and, of every stage of
// KG x NS k-steps, the kg-th NS steps, for all row blocks, so that each x
// operand read from LDS feeds two MFMAs and each weight block MB of them.
//
// x: the loaders stage each stage's x operands (all rows, a share each) by
// buffer-to-LDS loads, in MFMA operand order (block rb of a step: 16 rows x 32
// columns, lane l's 16 bytes at 16 l), into a ring of 2 to kWideStages LDS
// buffers, as many as fit, all but one ahead of the workers; one workgroup
// barrier per stage.  Weights go straight to the workers' registers, kWideDepth
// steps ahead.  With x in waves of its own, a worker's only outstanding memory
// operations are its weight loads, so the compiler's wait counts are exact and
// the loads stay in flight across the barriers.
//
// What bounds it: the weights, read once from HBM, then the work at both ends
// of a launch.  x comes from the XCD's L2 (a workgroup reads up to 112 GB/s per
// CU of lines its neighbours share, against 27 GB/s per CU of HBM at full
// rate), so narrow column ranges with few k-splits beat wide ones with many:
// re-reading x is cheaper than writing and re-reading fp32 partial sums.  One
// barrier per stage instead of per k-step, x in waves of its own, and no 64-bit
// division, dependent load or unrolled epilogue around the loop: at 144 rows
// and 7B widths gate/up 87 -> 56 us, LM head 315 -> 205, down 40 -> 33, q/k/v
// 21 -> 16, o 22 -> 15; at 45 rows 51 -> 45, 201 -> 182, 27 (unchanged), 15 ->
// 10 and 15 -> 9.  Of the 56 us, 42 are the loop (39 us of weights at the
// read rate), 4 the time to the first staged x and 5 the epilogue.
//
// A weight load past the k-range or the unit range gets an offset past the
// operand and returns zeros without a memory access; steps past the k-range
// are not multiplied; rows past M read other rows' x and are never stored.
// ---------------------------------------------------------------------------
constexpr int kWideLoaders = 2;     // waves that stage x
// worker waves: 14, or 10 from 7 row blocks, whose accumulators (8 registers
// per row block) leave no room for the weights in a 16-wave workgroup's 128
constexpr int wide_workers(int mb) { return mb <= 6 ? 14 : 10; }
constexpr int kWideDepth = 4;       // weight k-steps in flight per worker

// Buffer-to-LDS load of 16 bytes per lane; IMM is added to both addresses.
template <int IMM>
__device__ __forceinline__ void lds_load16(__amdgpu_buffer_rsrc_t r, unsigned char* dst, int voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(dst), 16, voff, 0, IMM, 0);
}

// Workgroup barrier that waits for this wave's LDS operations only.
__device__ __forceinline__ void wide_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// k-steps per worker and stage for KG k-groups of MB row blocks, and the stage
// buffers
constexpr size_t kWideRing = 144 * 1024;
constexpr int kWideStages = 6;
int wide_ns(int mb, int kg) {
  for (int ns : {4, 2})
    if ((size_t)2 * kg * ns * mb * 1024 <= kWideRing) return ns;
  return 1;
}
int wide_nb(int mb, int kg) {
  return (int)std::min<size_t>(kWideStages, kWideRing / ((size_t)kg * wide_ns(mb, kg) * mb * 1024));
}

// Row blocks whose partial tiles (P units, KG k-groups) pass through LDS at once.
int wide_rb(int mb, int P, int KG) { return std::max(1, std::min(mb, (int)(kWideRing / ((size_t)KG * P * 2 * 1024)))); }
// The x stage buffers, reused by the partial tiles; the LM head's running
// (max, index) of every unit slot and row.
size_t wide_lds_bytes(int mb, int P, int KG, int epi) {
  const size_t ring = (size_t)wide_nb(mb, KG) * KG * wide_ns(mb, KG) * mb * 1024;
  const size_t sums = (size_t)wide_rb(mb, P, KG) * KG * P * 2 * 1024;
  return std::max(ring, sums) + (epi == EPI_ARGMAX ? (size_t)P * 16 * mb * 8 : 0);
}

// Waits until at most n of the wave's vector memory operations are in flight
// (n rounded down to a multiple of four).
__device__ __forceinline__ void wait_vm(int n) {
  switch (min(n, 60) >> 2) {
#define WVM(i) case i: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * i) : "memory"); break;
    WVM(1) WVM(2) WVM(3) WVM(4) WVM(5) WVM(6) WVM(7) WVM(8) WVM(9) WVM(10) WVM(11) WVM(12) WVM(13) WVM(14) WVM(15)
#undef WVM
    default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
}

template <int MB, int EPI, int NS>
__global__ __launch_bounds__((wide_workers(MB) + kWideLoaders) * 64) void k_gemm_wide(GemvArgs a) {
  static_assert(EPI == EPI_SWIGLU || EPI == EPI_ARGMAX || EPI == EPI_STORE, "wide-unit epilogues");
  constexpr bool kNorm = EPI != EPI_STORE;
  constexpr int ROWS = 16 * MB, D = kWideDepth, U = D / NS;   // U stages per unrolled round
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ float inv_rms[ROWS];       // 0 for rows past the pass or idle
  __shared__ int live_s[ROWS];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int M = a.M, N = a.N, T = (a.Kd + 31) >> 5, ntiles = N / kTile;
  // The divisions are the host's: the code ahead of the first loads is fetched
  // cold by every launch.
  const int P = a.wp, KG = a.wkg, NB = a.wnb, nch = a.wnch, cu = a.wcu, nst = a.wnst;
  // Splits are dealt first: consecutive workgroups go to the 8 XCDs in turn, so
  // with 2, 4 or 8 splits an XCD's workgroups share one split's x in its L2.
  const int split = blockIdx.x % a.splits, blk = blockIdx.x / a.splits;
  const int s0 = split * a.wsq + min(split, a.wsr), s1 = s0 + a.wsq + (split < a.wsr ? 1 : 0);
  const int u0 = blk * a.wuq + min(blk, a.wur), u1 = u0 + a.wuq + (blk < a.wur ? 1 : 0);
  const int SS = KG * NS;                                     // k-steps per stage
  const int stage_bytes = SS * MB * 1024;
  float* best_v = reinterpret_cast<float*>(lds + a.wlds - (size_t)P * ROWS * 8);   // LM head: [P][ROWS] running
  int* best_i = reinterpret_cast<int*>(best_v + P * ROWS);                          // maximum and its index

  if (wave < kWideLoaders) {
    // The loaders share every stage's x blocks.  Operand-order x: a stage is
    // one contiguous run, four 1 KB blocks per address.  Row-major x: lane l
    // reads row 16 b + (l & 15), 16 bytes at column 32 step + 8 (l >> 4).
    // (Steps past the range are never multiplied.)
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.x), 0,
                                                                        a.xpk ? T * MB * 1024 : M * a.ldx * 2, kRsrcWord3);
    const int nblk = SS * MB, b0 = nblk * wave / kWideLoaders, b1 = nblk * (wave + 1) / kWideLoaders, cnt = b1 - b0;
    auto issue = [&](int st, int slot) {
      unsigned char* dst = lds + slot * stage_bytes;
      const int step0 = s0 + st * SS;
      if (a.xpk) {
        int off = (step0 * MB + b0) * 1024 + 16 * lane;
        int k = b0;
        for (; k + 4 <= b1; k += 4, off += 4096) {
          lds_load16<0>(rx, dst + k * 1024, off);
          lds_load16<1024>(rx, dst + k * 1024, off);
          lds_load16<2048>(rx, dst + k * 1024, off);
          lds_load16<3072>(rx, dst + k * 1024, off);
        }
        for (; k < b1; ++k, off += 1024) lds_load16<0>(rx, dst + k * 1024, off);
      } else {
        const int xlane = ((lane & 15) * a.ldx + 8 * (lane >> 4)) * 2;
        for (int k = b0; k < b1; ++k)
          lds_load16<0>(rx, dst + k * 1024, xlane + (step0 + k / MB) * 64 + (k % MB) * 32 * a.ldx);
      }
    };
    // what the epilogues need: loaded first (one round trip, beside the x
    // loads), stored to LDS below
    constexpr int RPT = (ROWS + kWideLoaders * 64 - 1) / (kWideLoaders * 64);   // rows per loader thread
    int cnt_r[RPT] = {}, row_j[RPT] = {};
    float inv_r[RPT] = {};
    if constexpr (kNorm) {
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const int m = min((int)threadIdx.x + i * kWideLoaders * 64, M - 1), b = m / a.rps;
        row_j[i] = m - b * a.rps;
        cnt_r[i] = a.st[b].count;
        inv_r[i] = a.rinv[m];
      }
    }
    for (int ch = 0; ch < nch; ++ch) {
      const int ahead = min(NB - 1, nst);
      for (int st = 0; st < ahead; ++st) issue(st, st);
      if (ch == 0) {
        if constexpr (kNorm) {
#pragma unroll
          for (int i = 0; i < RPT; ++i) {
            const int m = threadIdx.x + i * kWideLoaders * 64;
            const bool lv = m < M && row_j[i] < cnt_r[i];
            if (m < ROWS) {
              live_s[m] = lv ? 1 : 0;
              inv_rms[m] = lv ? inv_r[i] : 0.f;
            }
          }
        }
        if constexpr (EPI == EPI_ARGMAX) {
          for (int i = threadIdx.x; i < P * ROWS; i += kWideLoaders * 64) {
            best_v[i] = -INFINITY;
            best_i[i] = 0x7fffffff;
          }
        }
      }
      int slot = ahead == NB ? 0 : ahead;     // the next stage's buffer
      if (slot >= NB) slot -= NB;
      for (int st = 0; st < nst; ++st) {
        wait_vm(min(NB - 2, nst - 1 - st) * cnt);
        wide_barrier();                       // stage st is staged; the buffer of stage st - 1 is free
        if (st + NB - 1 < nst) {
          issue(st + NB - 1, slot);
          if (++slot == NB) slot = 0;
        }
      }
      wide_barrier();                         // the workers are done with the last stage
      if (EPI == EPI_STORE && KG == 1) continue;
      for (int r0 = 0; r0 < MB; r0 += a.wrb) {
        wide_barrier();
        wide_barrier();
      }
    }
  } else {
    // where the logits go, if anywhere
    bf16_t* lg = EPI == EPI_ARGMAX && a.allow_logits && a.st[0].want_logits ? a.st[0].logits : nullptr;
    const int wi = wave - kWideLoaders, kg = (wi * a.wrp) >> 16, pi = wi - kg * P;
    // Weights of the chunk being refilled: one buffer per tile, ending at the
    // split's last step, so that later steps (and, with no bytes at all, a slot
    // without a unit) read zeros without a memory access or a branch.
    __amdgpu_buffer_rsrc_t rw[2];
    auto open_w = [&](int ch) {
      const int unit = u0 + ch * cu + pi;
      const bool on = ch < nch && pi < cu && unit < u1;
      const bf16_t* p = a.pw + (size_t)(on ? 2 * unit : 0) * T * 512;
      rw[0] = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), 0, on ? s1 * 1024 : 0, kRsrcWord3);
      rw[1] = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p + (size_t)T * 512), 0,
                                                on && 2 * unit + 1 < ntiles ? s1 * 1024 : 0, kRsrcWord3);
    };
    const int w0 = (s0 + kg * NS) * 1024 + 16 * lane;         // the worker's first step of stage 0
    u32x4 w[D][2];
    auto issue_w = [&](u32x4 (&wr)[2], int off) {
      wr[0] = __builtin_amdgcn_raw_buffer_load_b128(rw[0], off, 0, kNt);
      wr[1] = __builtin_amdgcn_raw_buffer_load_b128(rw[1], off, 0, kNt);
    };
    open_w(0);
#pragma unroll
    for (int uu = 0; uu < U; ++uu)
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        issue_w(w[uu * NS + i], w0 + (uu * SS + i) * 1024);
        asm volatile("" ::: "memory");   // in this order: the wait counts of the loop's first round follow it
      }

    for (int ch = 0; ch < nch; ++ch) {
      f32x4 acc[2][MB];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[t][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
      int slot = 0;                                           // the stage's buffer
      for (int st0 = 0; st0 < nst; st0 += U) {
        int wn = w0 + (st0 + U) * SS * 1024;                  // the refills' steps
        if (st0 + U >= nst) {                                 // ... which belong to the next chunk
          open_w(ch + 1);
          wn = w0;
        }
#pragma unroll
        for (int uu = 0; uu < U; ++uu) {
          wide_barrier();
          const unsigned char* xb = lds + slot * stage_bytes + kg * NS * MB * 1024 + 16 * lane;
          if (++slot == NB) slot = 0;
#pragma unroll
          for (int i = 0; i < NS; ++i) {
            u32x4(&ws)[2] = w[uu * NS + i];
            if (s0 + (st0 + uu) * SS + kg * NS + i < s1) {    // wave-uniform
              u32x4 xv[MB];
#pragma unroll
              for (int mb = 0; mb < MB; ++mb) xv[mb] = *reinterpret_cast<const u32x4*>(xb + (i * MB + mb) * 1024);
#pragma unroll
              for (int mb = 0; mb < MB; ++mb) {
                acc[0][mb] = mfma16x16x32(ws[0], xv[mb], acc[0][mb]);
                acc[1][mb] = mfma16x16x32(ws[1], xv[mb], acc[1][mb]);
              }
              // kXv operand reads ahead of the products that use them
              constexpr int kXv = MB < 4 ? MB : MB == 6 ? 3 : 4;
              __builtin_amdgcn_sched_group_barrier(0x100, kXv, 0);
#pragma unroll
              for (int mb = 0; mb < MB - kXv; ++mb) {
                __builtin_amdgcn_sched_group_barrier(0x8, 2, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
              }
              __builtin_amdgcn_sched_group_barrier(0x8, 2 * kXv, 0);
            }
            issue_w(ws, wn + (uu * SS + i) * 1024);
          }
        }
      }
      wide_barrier();
      const int unit = u0 + ch * cu + pi, grp = lane >> 4;
      const bool mine = pi < cu && unit < u1;                 // wave-uniform
      const bool two = 2 * unit + 1 < ntiles;                 // the last unit may be a single tile
      if constexpr (EPI == EPI_STORE) {
        if (KG == 1) {   // complete sums of this split: out[split][m][n]
          float* o = a.out + ((size_t)split * M + (lane & 15)) * N + 2 * unit * kTile + 4 * grp;
#pragma unroll
          for (int mb = 0; mb < MB; ++mb, o += (size_t)16 * N)
            if (mine && mb * 16 + (lane & 15) < M) {
              *reinterpret_cast<f32x4*>(o) = acc[0][mb];
              if (two) *reinterpret_cast<f32x4*>(o + kTile) = acc[1][mb];
            }
          continue;
        }
      }
      // The partial tiles go through LDS, a.wrb row blocks at a time; worker
      // (p, kg) then completes unit p's row blocks kg, kg + KG, .., adding the
      // k-groups' partial tiles in order.  That loop is kept rolled: unrolled
      // over the row blocks it would be several KB of code that every launch
      // fetches once.
      f32x4* red = reinterpret_cast<f32x4*>(lds) + lane;      // [KG][P][2][wrb][64]
      for (int r0 = 0; r0 < MB; r0 += a.wrb) {
        const int nr = min(a.wrb, MB - r0);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          if (mb >= r0 && mb < r0 + nr) {                     // wave-uniform
            f32x4* r = red + ((kg * P + pi) * 2 * a.wrb + mb - r0) * 64;
            r[0] = acc[0][mb];
            r[a.wrb * 64] = acc[1][mb];
          }
        wide_barrier();
#pragma unroll 1
        for (int rb = mine ? kg : nr; rb < nr; rb += KG) {
          f32x4 y0 = f32x4{0.f, 0.f, 0.f, 0.f}, y1 = y0;
#pragma unroll 1
          for (int k = 0; k < KG; ++k) {
            const f32x4* r = red + ((k * P + pi) * 2 * a.wrb + rb) * 64;
            y0 += r[0];
            y1 += r[a.wrb * 64];
          }
          const int m = (r0 + rb) * 16 + (lane & 15);
          if constexpr (EPI == EPI_STORE) {
            // fp32 partial sums of this split: out[split][m][n]
            if (m < M) {
              float* o = a.out + ((size_t)split * M + m) * N + 2 * unit * kTile + 4 * grp;
              *reinterpret_cast<f32x4*>(o) = y0;
              if (two) *reinterpret_cast<f32x4*>(o + kTile) = y1;
            }
          } else if constexpr (EPI == EPI_SWIGLU) {
            // the gate and up rows of features 16 unit .. +16
            const int F = N / 2, f = unit * kTile + 4 * grp;
            const float r = inv_rms[m];
            const bool lv = live_s[m];
            float o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float g = y0[i] * r, up = y1[i] * r;
              o[i] = lv ? g / (1.f + expf(-g)) * up : 0.f;
            }
            if (m < M) {
              const size_t at = a.upk ? xop_at(m, f, MB) : (size_t)m * F + f;
              *reinterpret_cast<u32x2*>(a.u + at) = u32x2{pack2(o[0], o[1]), pack2(o[2], o[3])};
            }
          } else {   // EPI_ARGMAX: the (max, index) of each row over the unit's 32 logits
            const int n = 2 * unit * kTile + 4 * grp;
            const bool lv = live_s[m];
            const float r = inv_rms[m];
            float y[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              y[i] = lv ? y0[i] * r : 0.f;
              y[4 + i] = lv ? y1[i] * r : 0.f;
            }
            if (lg && m < M) {
              bf16_t* lo = lg + (size_t)m * N + n;
              st_global(lo, u32x2{pack2(y[0], y[1]), pack2(y[2], y[3])});
              if (two) st_global(lo + kTile, u32x2{pack2(y[4], y[5]), pack2(y[6], y[7])});
            }
            float best = -INFINITY;
            int bi = n;
            int nan = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              float v = y[i];
              if (i >= 4 && !two) v = -INFINITY;
              if (v != v) {
                nan = 1;
                v = -INFINITY;
              }
              if (v > best) {
                best = v;
                bi = n + (i & 3) + (i >> 2) * kTile;
              }
            }
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
              const float v2 = __shfl_xor(best, o);
              const int i2 = __shfl_xor(bi, o);
              nan |= __shfl_xor(nan, o);
              amax_merge(best, bi, v2, i2);
            }
            if (grp == 0) {
              float bv = best_v[pi * ROWS + m];
              int bx = best_i[pi * ROWS + m];
              amax_merge(bv, bx, best, bi);
              best_v[pi * ROWS + m] = bv;
              best_i[pi * ROWS + m] = bx;
              if (nan && lv) atomicOr(const_cast<int32_t*>(&a.st[m / a.rps].err), ERR_NUMERIC);
            }
          }
        }
        wide_barrier();
      }
    }
  }
  if constexpr (EPI == EPI_ARGMAX) {
    // one (max, index) per row for the whole workgroup
    wide_barrier();
    for (int m = threadIdx.x; m < M; m += blockDim.x) {
      float bv = -INFINITY;
      int bx = 0x7fffffff;
      for (int p = 0; p < P; ++p) amax_merge(bv, bx, best_v[p * ROWS + m], best_i[p * ROWS + m]);
      a.amax_v[(size_t)blk * a.mpad + m] = bv;
      a.amax_i[(size_t)blk * a.mpad + m] = bx;
    }
  }
}

// CUs of the current device (the wide kernel's grid for SwiGLU and argmax)
int wide_cus() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      n < 1) {
    (void)hipGetLastError();
    return 256;
  }
  return n;
}

// Geometry of a wide-unit launch: G workgroups per k-split, chunks of at most
// P units, KG k-groups.  Workgroups divide the units evenly; P x KG workers
// (at most wide_workers) share a workgroup's chunk.
struct WidePlan {
  int G, S, P, KG;
};

WidePlan wide_plan(int epi, int N, int Kd, int M, int ncu) {
  const int mb = (M + 15) / 16, T = (Kd + 31) / 32, units = (N / kTile + 1) / 2;
  auto shape = [&](int S) {
    WidePlan p;
    p.S = S;
    p.G = std::max(1, std::min(ncu / S, units));
    const int upw = (units + p.G - 1) / p.G;                 // units of the busiest workgroup
    // Few long chunks before many k-groups: each chunk stages all of x again.  10
    // units are the workers of the wider passes (chunks of 7 at 144 rows: LM head
    // 152064 x 3584 226 us against 205, gate/up of 32768 x 3584 99 against 82, down
    // of 8192 x 28672 106 against 86; of 5: 241, 99 and 104).
    constexpr int pmax = 10;
    static_assert(pmax <= wide_workers(SPEC_MAX_ROWS / 16), "a worker per unit of a chunk");
    const int chunks = (upw + pmax - 1) / pmax;
    p.P = (upw + chunks - 1) / chunks;
    // as many k-groups as the workers and the LDS (two stage buffers) allow; the
    // groups' partial tiles pass through it as many row blocks at a time as fit
    p.KG = std::max(1, std::min(wide_workers(mb) / p.P, (T + S - 1) / S));
    while (p.KG > 1 && (size_t)2 * p.KG * mb * 1024 > kWideRing)
      --p.KG;
    return p;
  };
  if (epi != EPI_STORE) return shape(1);
  // k-splits (a power of two, see the kernel): the least bytes a workgroup
  // waits for: its weights from HBM, x from L2 at about four times that rate,
  // and its share of the fp32 partial sums, written once and read once by the
  // finishing kernel.  (Counting the partial sums half or twice: 16-scene
  // verify 1058 and 1067 us against 1056.)
  WidePlan best{};
  double least = 0;
  // (at most as many as 256-column workgroups would fill the CUs once with, of 16
  // k-steps or more: that bounds the scratch a pass needs)
  const int most = std::max(1, std::min(ncu / ((N / kTile + 15) / 16), T / 16));
  for (int S = 1; S <= std::min(16, most); S *= 2) {
    const WidePlan p = shape(S);
    const int upw = (units + p.G - 1) / p.G;
    const double steps = (T + S - 1) / S;
    const double cost = upw * 2048.0 * steps + steps * mb * 256.0 + 8.0 * S * M * N / ncu;
    if (S == 1 || cost < least) {
      least = cost;
      best = p;
    }
  }
  return best;
}

template <int MB, int EPI>
hipError_t launch_wide_mb(const GemvArgs& g, int ns, const dim3& grid, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const dim3 block((g.wp * g.wkg + kWideLoaders) * 64);
  switch (ns) {
    case 1: hipExtLaunchKernelGGL((k_gemm_wide<MB, EPI, 1>), grid, block, g.wlds, s, e0, e1, 0, g); break;
    case 2: hipExtLaunchKernelGGL((k_gemm_wide<MB, EPI, 2>), grid, block, g.wlds, s, e0, e1, 0, g); break;
    case 4: hipExtLaunchKernelGGL((k_gemm_wide<MB, EPI, 4>), grid, block, g.wlds, s, e0, e1, 0, g); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int EPI>
hipError_t launch_wide(GemvArgs g, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const int mb = (g.M + 15) / 16;
  WidePlan p = wide_plan(EPI, g.N, g.Kd, g.M, wide_cus());
  if (p.S != g.splits) return hipErrorInvalidValue;   // the caller sized its partial sums with gemm_wide_splits
  g.wp = p.P;
  g.wkg = p.KG;
  g.wnb = wide_nb(mb, p.KG);
  g.wrb = wide_rb(mb, p.P, p.KG);
  const int T = (g.Kd + 31) / 32, units = (g.N / kTile + 1) / 2, upw = (units + p.G - 1) / p.G;
  const int ns = wide_ns(mb, p.KG), round = kWideDepth / ns, steps = (T + p.S - 1) / p.S;
  g.wsq = T / p.S;
  g.wsr = T % p.S;
  g.wuq = units / p.G;
  g.wur = units % p.G;
  g.wnch = (upw + p.P - 1) / p.P;
  g.wcu = (upw + g.wnch - 1) / g.wnch;
  const int st = (steps + p.KG * ns - 1) / (p.KG * ns);
  g.wnst = (st + round - 1) / round * round;   // a whole number of unrolled rounds
  g.wrp = (65536 + p.P - 1) / p.P;
  g.wlds = (int)wide_lds_bytes(mb, p.P, p.KG, EPI);
  const dim3 grid(p.G * p.S);
  switch (mb) {
    case 3: return launch_wide_mb<3, EPI>(g, ns, grid, s, e0, e1);
    case 4: return launch_wide_mb<4, EPI>(g, ns, grid, s, e0, e1);
    case 5: return launch_wide_mb<5, EPI>(g, ns, grid, s, e0, e1);
    case 6: return launch_wide_mb<6, EPI>(g, ns, grid, s, e0, e1);
    case 7: return launch_wide_mb<7, EPI>(g, ns, grid, s, e0, e1);
    case 8: return launch_wide_mb<8, EPI>(g, ns, grid, s, e0, e1);
    case 9: return launch_wide_mb<9, EPI>(g, ns, grid, s, e0, e1);
    case 10: return launch_wide_mb<10, EPI>(g, ns, grid, s, e0, e1);
    default: return hipErrorInvalidValue;
  }
}

template <int MB, int EPI>
void set_wide_attr(int limit) {
  const void* f[3] = {reinterpret_cast<const void*>(&k_gemm_wide<MB, EPI, 1>),
                      reinterpret_cast<const void*>(&k_gemm_wide<MB, EPI, 2>),
                      reinterpret_cast<const void*>(&k_gemm_wide<MB, EPI, 4>)};
  for (const void* p : f) (void)hipFuncSetAttribute(p, hipFuncAttributeMaxDynamicSharedMemorySize, limit - 2048);
}

template <int MB>
void set_wide_attributes(int limit) {
  set_wide_attr<MB, EPI_SWIGLU>(limit);
  set_wide_attr<MB, EPI_ARGMAX>(limit);
  set_wide_attr<MB, EPI_STORE>(limit);
}

template <int EPI>
hipError_t launch_mb(const GemvArgs& g, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const int mb = (g.M + 15) / 16;
  const dim3 grid((g.N + kGemmTiles * kTile - 1) / (kGemmTiles * kTile), g.splits), block(threads_for(mb));
  const size_t lds = gemm_lds_bytes(g.M);
  switch (mb) {
    case 2: hipExtLaunchKernelGGL((k_gemm<2, EPI>), grid, block, lds, s, e0, e1, 0, g); break;
    case 3: hipExtLaunchKernelGGL((k_gemm<3, EPI>), grid, block, lds, s, e0, e1, 0, g); break;
    case 4: hipExtLaunchKernelGGL((k_gemm<4, EPI>), grid, block, lds, s, e0, e1, 0, g); break;
    case 5: hipExtLaunchKernelGGL((k_gemm<5, EPI>), grid, block, lds, s, e0, e1, 0, g); break;
    case 6: hipExtLaunchKernelGGL((k_gemm<6, EPI>), grid, block, lds, s, e0, e1, 0, g); break;
    case 7: hipExtLaunchKernelGGL((k_gemm<7, EPI>), grid, block, lds, s, e0, e1, 0, g); break;
    case 8: hipExtLaunchKernelGGL((k_gemm<8, EPI>), grid, block, lds, s, e0, e1, 0, g); break;
    case 9: hipExtLaunchKernelGGL((k_gemm<9, EPI>), grid, block, lds, s, e0, e1, 0, g); break;
    case 10: hipExtLaunchKernelGGL((k_gemm<10, EPI>), grid, block, lds, s, e0, e1, 0, g); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int MB>
void set_mb_attributes(int limit) {
  const int lds = (int)std::max(x_lds_bytes(MB), y_lds_bytes(MB));
  if (lds > limit) return;   // such a launch is rejected by the host-side LDS check
  const void* f[5] = {reinterpret_cast<const void*>(&k_gemm<MB, EPI_STORE>),
                      reinterpret_cast<const void*>(&k_gemm<MB, EPI_ROPE>),
                      reinterpret_cast<const void*>(&k_gemm<MB, EPI_RESID>),
                      reinterpret_cast<const void*>(&k_gemm<MB, EPI_SWIGLU>),
                      reinterpret_cast<const void*>(&k_gemm<MB, EPI_ARGMAX>)};
  for (const void* p : f) (void)hipFuncSetAttribute(p, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}

}  // namespace

size_t gemm_lds_bytes(int M) {
  const int mb = (M + 15) / 16;
  return std::max(x_lds_bytes(mb), y_lds_bytes(mb));
}

void gemm_set_attributes(int limit) {
  set_mb_attributes<2>(limit);
  set_mb_attributes<3>(limit);
  set_mb_attributes<4>(limit);
  set_mb_attributes<5>(limit);
  set_mb_attributes<6>(limit);
  set_mb_attributes<7>(limit);
  set_mb_attributes<8>(limit);
  set_mb_attributes<9>(limit);
  set_mb_attributes<10>(limit);
  set_wide_attributes<3>(limit);
  set_wide_attributes<4>(limit);
  set_wide_attributes<5>(limit);
  set_wide_attributes<6>(limit);
  set_wide_attributes<7>(limit);
  set_wide_attributes<8>(limit);
  set_wide_attributes<9>(limit);
  set_wide_attributes<10>(limit);
}

bool gemm_takes_wide(int epi, const GemvArgs& g) {
  return g.pw && g.M > kSgMaxRows && g.M <= SPEC_MAX_ROWS &&
         (epi == EPI_STORE || ((epi == EPI_SWIGLU || epi == EPI_ARGMAX) && g.splits == 1 && g.rinv));
}

int gemm_argmax_entries(const GemvArgs& g) {
  return gemm_takes_wide(EPI_ARGMAX, g) ? wide_plan(EPI_ARGMAX, g.N, g.Kd, g.M, wide_cus()).G : g.N / kTile;
}

hipError_t gemm_launch(int epi, const GemvArgs& g, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (g.M <= kSgMaxRowsGemm || g.M > SPEC_MAX_ROWS || g.splits < 1 || (epi != EPI_STORE && g.splits != 1) ||
      g.N % kTile != 0 || g.Kd % 8 != 0)
    return hipErrorInvalidValue;
  // k_gemm's 1/rms prologue reads at most lpt_for(parts) sums of squares per
  // thread, in threads_for / rows parts per row
  if (!gemm_takes_wide(epi, g)) {
    const int mb = (g.M + 15) / 16, parts = threads_for(mb) / (16 * mb);
    if ((epi == EPI_ROPE || epi == EPI_SWIGLU || epi == EPI_ARGMAX) &&
        (g.H < kTile || g.H / kTile > lpt_for(parts) * parts))
      return hipErrorInvalidValue;
  }
  // every operand is addressed with 32-bit byte offsets below kOut
  if ((long long)g.N * ((g.Kd + 31) / 32) * 64 >= kOut || (long long)g.M * g.ldx * 2 >= kOut) return hipErrorInvalidValue;
  if (gemm_takes_wide(epi, g)) {
    if (epi == EPI_STORE) return launch_wide<EPI_STORE>(g, s, e0, e1);
    return epi == EPI_SWIGLU ? launch_wide<EPI_SWIGLU>(g, s, e0, e1) : launch_wide<EPI_ARGMAX>(g, s, e0, e1);
  }
  if (g.xpk) return hipErrorInvalidValue;   // only the wide kernel reads operand-order x
  switch (epi) {
    case EPI_STORE: return launch_mb<EPI_STORE>(g, s, e0, e1);
    case EPI_ROPE: return launch_mb<EPI_ROPE>(g, s, e0, e1);
    case EPI_RESID: return launch_mb<EPI_RESID>(g, s, e0, e1);
    case EPI_SWIGLU: return launch_mb<EPI_SWIGLU>(g, s, e0, e1);
    case EPI_ARGMAX: return launch_mb<EPI_ARGMAX>(g, s, e0, e1);
    default: return hipErrorInvalidValue;
  }
}

// k-splits of the down projection over M > kThinRows rows: as many as fit
// the resident workgroup slots in one round (a count that overflows them
// leaves a second round for the few workgroups left over, which doubles the
// projection's time: 56 groups x 5 splits = 280 workgroups on 256 slots),
// at least 8 k-steps per split.
int gemm_down_splits(int N, int Kd, int ncu) {
  const int groups = (N + kGemmTiles * kTile - 1) / (kGemmTiles * kTile);
  const int T = (Kd + 31) / 32;
  int s = std::max(1, ncu / groups);
  return std::max(1, std::min(s, T / 8));
}

int gemm_wide_splits(int N, int Kd, int M, int ncu) { return wide_plan(EPI_STORE, N, Kd, M, ncu).S; }

int gemm_wgs_per_cu(int M) {
  // only the 8-wave shape of up to three row blocks is sized for two
  // workgroups per CU; the wider ones keep one, so that their (larger) k-split
  // partials do not double
  const int mb = (M + 15) / 16;
  const void* f = nullptr;
  switch (mb) {
    case 2: f = reinterpret_cast<const void*>(&k_gemm<2, EPI_STORE>); break;
    case 3: f = reinterpret_cast<const void*>(&k_gemm<3, EPI_STORE>); break;
    default: return 1;
  }
  int n = 0;
  const size_t lds = gemm_lds_bytes(M);
  if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, threads_for(mb), lds) != hipSuccess) {
    (void)hipGetLastError();
    return 1;
  }
  return std::max(1, std::min(n, 2));
}

int gemm_qkv_splits(int N, int Kd, int M, int ncu) {
  const int groups = (N + kGemmTiles * kTile - 1) / (kGemmTiles * kTile);
  if (2 * groups >= ncu) return 1;
  // one workgroup per CU: measured faster here than filling both slots, as
  // the doubled partials outweigh the extra streams
  const int s = gemm_down_splits(N, Kd, ncu);
  // Passes of more than 32 rows always split: such a GEMM is far from
  // streaming its weights at full rate (the time goes into each workgroup's
  // MFMA and x-operand work), so spreading it over s times the workgroups
  // pays for the partials (144 rows: 72 workgroups -> 3 x 72).  Fewer rows
  // split only while 2 * s * M * N fp32 partial bytes <= (N * Kd bf16 weight
  // bytes) / 10.
  return (M > kSgMaxRows || (long long)40 * s * M <= Kd) ? s : 1;
}

int gemm_qkv_splits_for(int N, int Kd, int M, int ncu, bool wide) {
  return (wide && M > kSgMaxRows) ? gemm_wide_splits(N, Kd, M, ncu) : gemm_qkv_splits(N, Kd, M, ncu);
}

}  // namespace specdec

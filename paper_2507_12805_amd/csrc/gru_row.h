// One row of the BiGRU (h <= 32 units per direction) in one workgroup: the
// device code shared by its inference (tf_kernels.hip) and its training
// (gru_train.hip).
//
// What bounds a row is the chain over its t positions: a position's hidden
// products need the previous position's state.  So only that chain is run
// serially, by one wave per direction; everything that does not need the
// state is done for all positions at once by the whole workgroup (the input
// products here; in the training also the weight gradients, the input
// gradients and the embedding sums).  In the chain's wave, lane l holds unit
// u = l % 32: lanes 0-31 its reset and candidate rows, lanes 32-63 its update
// row, the rows' hidden weights in registers, the state broadcast from LDS,
// so a position costs two in-order dot products of 32 and no barrier.
//
// Widths below the compiled ones (32 units, the padded input width) are
// padded with zero weights: a padded term adds an exact zero, so every sum
// keeps its value and its order (unit, then gate r, z, n).  A padded gate
// row's input part and a padded unit's dh are set to zero, not summed: zero
// weights times an infinite input would make them NaN, and they are factors
// of the other units' padded terms.
#pragma once
#include "pmklc_internal.h"
#include "seq_loop.h"

namespace pmklc {
namespace gru {

constexpr int kU = 32;         // padded units per direction
constexpr int kG = 3 * kU;     // padded gate rows per direction: r, z, n

__device__ __forceinline__ float sigm(float x) { return 1.0f / (1.0f + __expf(-x)); }
__device__ __forceinline__ float tanh_f(float x) { return 1.0f - 2.0f / (__expf(2.0f * x) + 1.0f); }

// LDS written and read by one wave: the LDS serves a wave's accesses in the
// order they were issued, so the compiler keeping that order is enough (no
// barrier, and no wait for the write before the read).
__device__ __forceinline__ void wave_sync() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// The gate rows of both directions, w[d] rows 3h x cols, into LDS as
// dst[(d 96 + gate 32 + u) (NP + 1) + c], zero past the real units and
// columns; column slot c holds real column col(c), zero where negative.
// Read along a row by its lane: an odd pitch, so the reads meet no bank
// conflict, and global memory is read in order (a lane reading its own row
// from global memory costs a cache line per lane and load).
template <int NP, class Col>
__device__ __forceinline__ void stage_gates(const float *W, const int64_t (&off)[2], int h, int cols, Col col,
                                            float *dst, int nt) {
  constexpr int kFly = 8;   // loads in flight per thread
  for (int x0 = threadIdx.x; x0 < 2 * kG * NP; x0 += kFly * nt) {
    float v[kFly];
#pragma unroll
    for (int y = 0; y < kFly; y++) {
      const int x = x0 + y * nt, row = x / NP, k = col(x % NP), d = row >= kG, g = row - d * kG, u = g % kU;
      v[y] = x < 2 * kG * NP && u < h && k >= 0 ? W[off[d] + (int64_t)((g / kU) * h + u) * cols + k] : 0.0f;
    }
#pragma unroll
    for (int y = 0; y < kFly; y++) {
      const int x = x0 + y * nt;
      if (x < 2 * kG * NP) dst[x + x / NP] = v[y];
    }
  }
}
template <int NP>
__device__ __forceinline__ void load_row(const float *rows, int row, float (&v)[NP]) {
#pragma unroll
  for (int c = 0; c < NP; c++) v[c] = rows[row * (NP + 1) + c];
}

// acc += w[0] x[0], then w[1] x[1], ... over C products, C a multiple of 8.
// The products of a group of 8 are formed while the previous group's are
// added: a lone wave's dependent multiply-add pairs would otherwise wait out
// both latencies 2 C times.
template <int C>
__device__ __forceinline__ float dot_in_order(float acc, const float (&w)[C], const float (&x)[C]) {
  float p[8];
#pragma unroll
  for (int c = 0; c < 8; c++) p[c] = w[c] * x[c];
#pragma unroll
  for (int c0 = 8; c0 <= C; c0 += 8) {
    __builtin_amdgcn_sched_barrier(0);
    float n[8];
    if (c0 < C) {
#pragma unroll
      for (int c = 0; c < 8; c++) n[c] = w[c0 + c] * x[c0 + c];
    }
#pragma unroll
    for (int c = 0; c < 8; c++) acc += p[c];
    if (c0 < C) {
#pragma unroll
      for (int c = 0; c < 8; c++) p[c] = n[c];
    }
  }
  return acc;
}
// 4-float runs of LDS (16-byte aligned) into v
template <int C>
__device__ __forceinline__ void lds_run(const float *p, float *v) {
#pragma unroll
  for (int c = 0; c < C; c += 4) {
    const float4 x = *reinterpret_cast<const float4 *>(p + c);
    v[c] = x.x; v[c + 1] = x.y; v[c + 2] = x.z; v[c + 3] = x.w;
  }
}

// Input parts of every position: pa[(d t + p) 96 + row] = b_i + W_i x_p, one
// thread per (direction, row) and share of the positions (blockDim / 192
// shares), the row's weights in registers (the constructor reads them from
// the staged rows).  xat(p, c): columns c..c+3 of the position's padded
// input, 16-byte aligned in LDS.
template <int NP>
struct InputParts {
  float w[NP], b;
  int d, row, share, shares;
  bool real;   // not a padded row
  __device__ __forceinline__ InputParts(const float *rows, const float *W, const int64_t (&bih)[2], int h) {
    shares = (int)blockDim.x / (2 * kG);
    const int item = (int)threadIdx.x % (2 * kG);
    share = (int)threadIdx.x / (2 * kG);
    d = item / kG;
    row = item % kG;
    const int gate = row / kU, u = row % kU;
    real = u < h;
    load_row<NP>(rows, item, w);
    b = real ? W[bih[d] + gate * h + u] : 0.0f;
  }
  template <class X>
  __device__ __forceinline__ void run(int t, X xat, float *pa) const {
    if (share >= shares) return;
    for (int p = share; p < t; p += shares) {
      float x[NP];
#pragma unroll
      for (int c = 0; c < NP; c += 4) lds_run<4>(xat(p, c), x + c);
      const float a = dot_in_order<NP>(b, w, x);
      pa[(d * t + p) * kG + row] = real ? a : 0.0f;
    }
  }
};

// The recurrence of direction d by one wave (the constructor reads its
// hidden weights from the staged rows).  hq: the state before the first step
// (zeros) at hq, after step s at hq + (s + 1) hstep (hstep 32 keeps them all,
// 0 only the last).  save(s, u, r, z, n, bn): the gates and the candidate's
// hidden part of step s, called by lanes 0-31.
struct Recurrence {
  float w0[kU], w1[kU], b0i, b1i;
  __device__ __forceinline__ Recurrence(const float *rows, const float *W, const int64_t (&bhh)[2], int d, int h) {
    const int lane = threadIdx.x & 63, u = lane & (kU - 1);
    const bool lower = lane < kU;
    load_row<kU>(rows, d * kG + (lower ? 0 : kU) + u, w0);
    load_row<kU>(rows, d * kG + 2 * kU + u, w1);
    b0i = u < h ? W[bhh[d] + (lower ? 0 : h) + u] : 0.0f;
    b1i = u < h ? W[bhh[d] + 2 * h + u] : 0.0f;
  }
  template <class Save>
  __device__ __forceinline__ void run(int t, int d, const float *pa, float *hq, int hstep, Save save) const {
    const int lane = threadIdx.x & 63, u = lane & (kU - 1);
    const bool lower = lane < kU;
    float hold = 0.0f;
    if (lower) hq[u] = 0.0f;
    wave_sync();
    for (int s = 0; s < t; s++) {
      const int p = d == 0 ? s : t - 1 - s;
      const float *ap = pa + (d * t + p) * kG;
      const float a0 = ap[(lower ? 0 : kU) + u], an = ap[2 * kU + u];
      float hv[kU];
      lds_run<kU>(hq + s * hstep, hv);
      float b0 = b0i, bn = b1i;
#pragma unroll
      for (int c = 0; c < kU; c++) {
        b0 += w0[c] * hv[c];
        bn += w1[c] * hv[c];
      }
      const float g0 = sigm(a0 + b0);              // lanes 0-31 r, 32-63 z
      const float z = __shfl_xor(g0, kU);          // z in lanes 0-31
      const float n = tanh_f(an + g0 * bn);
      const float hn = (1.0f - z) * n + z * hold;
      if (lower) {
        hold = hn;
        hq[(s + 1) * hstep + u] = hn;
        save(s, u, g0, z, n, bn);
      }
      wave_sync();
    }
  }
};

}  // namespace gru
}  // namespace pmklc

// The Transformer DM's attention block in BF16 for the paper's widths (t 32,
// E 64, A 256 in heads of 32, V 64): included by tf_kernels.hip.
//
// A row's keys and values are a product over E = 64 inputs, so computing
// them again costs the matrix cores little, while keeping them costs memory:
// [k | v] of 16 blocks of 320 rows is 335 MB per step, written once and read
// three times, and their gradient the same again.  So neither is ever in
// memory here: the forward and the backward each rebuild a row's [k | v]
// from its tokens in LDS, and the gradient of [k | v], an outer product per
// head (dk_p = ds_p q, dv_p = a_p do), is formed as the matrix cores'
// fragments where it is used.  What is kept per row is the probabilities a
// and ds (H t floats each), q and do.
//
// Values: each product's k-steps, each split's slices and each sum over
// positions or head columns run in the order of the general kernels
// (gemm_kernel, attn_fwd_kernel, attn_bwd_kernel), so both give the same
// bits and a container decodes with either.
#pragma once

struct PaperAttn {
  static constexpr int T = 32, E = 64, A = 256, DH = 32, H = A / DH, V = 64;
};
bool is_paper_attn(const TfShape &s) {
  typedef PaperAttn P;
  return s.arch == 1 && s.bf16 && s.t == P::T && s.E == P::E && s.A == P::A && s.dh == P::DH && s.V == P::V;
}

typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4a __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4_t mma_bf16(bf16x8_t a, bf16x8_t b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// Matrix-core results read past a branch: keep their wait states explicit
// (as in gemm_kernel)
__device__ __forceinline__ void mma_settle() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void load8(const float *p, float (&v)[8]) {
  const f32x4a x = *reinterpret_cast<const f32x4a *>(p), y = *reinterpret_cast<const f32x4a *>(p + 4);
#pragma unroll
  for (int c = 0; c < 4; c++) {
    v[c] = x[c];
    v[4 + c] = y[c];
  }
}
__device__ __forceinline__ bf16x8_t pack8(const float (&v)[8]) {
  bf16x8_t f;
#pragma unroll
  for (int c = 0; c < 8; c++) f[c] = (__bf16)v[c];
  return f;
}
// LDS exchanges inside one wave: its accesses are served in order
__device__ __forceinline__ void wave_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// x_p = Emb[c_p] + Pos[p], 8 columns from e0
__device__ __forceinline__ bf16x8_t ctx_x8(const TfShape &s, const float *W, int tok, int p, int e0) {
  float a[8], b[8];
  load8(W + s.off_emb + (int64_t)tok * PaperAttn::E + e0, a);
  load8(W + s.off_pos + (int64_t)p * PaperAttn::E + e0, b);
#pragma unroll
  for (int c = 0; c < 8; c++) a[c] = a[c] + b[c];
  return pack8(a);
}

// A row's [k | v] (T x 2A) in LDS from its tokens.  Wave w of four owns
// columns 128 w .. 128 w + 127: their weights stay in its registers for all
// rows of the workgroup.
struct RowKv {
  typedef PaperAttn P;
  static constexpr int XP = P::E + 8;         // pitch of the X rows (BF16)
  static constexpr int KP = 2 * P::A + 4;     // pitch of the [k | v] rows: 4 rows apart are 16 banks apart
  static constexpr int NT = 8;                // column tiles per wave
  bf16x8_t w[NT][2];
  float bias[NT];
  int lane, r, q, col0;
  __device__ __forceinline__ void load(const TfShape &s, const float *W, int wave) {
    lane = threadIdx.x & 63;
    r = lane & 15;
    q = lane >> 4;
    col0 = 16 * NT * wave + r;
    const float *wk = W + s.off_W[0] + P::A + col0;
#pragma unroll
    for (int n = 0; n < NT; n++) {
#pragma unroll
      for (int ks = 0; ks < 2; ks++) {
        float v[8];
#pragma unroll
        for (int c = 0; c < 8; c++) v[c] = wk[(int64_t)(32 * ks + 8 * q + c) * 3 * P::A + 16 * n];
        w[n][ks] = pack8(v);
      }
      bias[n] = W[s.off_b[0] + P::A + col0 + 16 * n];
    }
  }
  // the row's X into LDS (256 threads, 8 columns each)
  __device__ __forceinline__ static void stage_x(const TfShape &s, const float *W, const uint8_t *tok, __bf16 *xs) {
    const int p = (int)threadIdx.x >> 3, e0 = ((int)threadIdx.x & 7) * 8;
    *reinterpret_cast<bf16x8_t *>(xs + p * XP + e0) = ctx_x8(s, W, tok[p], p, e0);
  }
  __device__ __forceinline__ void product(const __bf16 *xs, float *kv) const {
    bf16x8_t a[2][2];
#pragma unroll
    for (int m = 0; m < 2; m++)
#pragma unroll
      for (int ks = 0; ks < 2; ks++)
        a[m][ks] = *reinterpret_cast<const bf16x8_t *>(xs + (16 * m + r) * XP + 32 * ks + 8 * q);
    f32x4_t acc[NT][2];
#pragma unroll
    for (int n = 0; n < NT; n++)
#pragma unroll
      for (int m = 0; m < 2; m++) acc[n][m] = mma_bf16(a[m][0], w[n][0], f32x4_t{0.0f, 0.0f, 0.0f, 0.0f});
#pragma unroll
    for (int n = 0; n < NT; n++)
#pragma unroll
      for (int m = 0; m < 2; m++) acc[n][m] = mma_bf16(a[m][1], w[n][1], acc[n][m]);
#pragma unroll
    for (int n = 0; n < NT; n++)
#pragma unroll
      for (int m = 0; m < 2; m++)
#pragma unroll
        for (int c = 0; c < 4; c++) kv[(16 * m + 4 * q + c) * KP + col0 + 16 * n] = acc[n][m][c] + bias[n];
  }
};

// max over the 32 lanes of a head
__device__ __forceinline__ float head_max(float x) {
#pragma unroll
  for (int o = 16; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
  return x;
}
// sum of 32 consecutive LDS floats, first to last
__device__ __forceinline__ float sum32(const float *p) {
  float s = 0.0f;
#pragma unroll
  for (int c = 0; c < 32; c += 4) {
    const f32x4a x = *reinterpret_cast<const f32x4a *>(p + c);
    s += x[0];
    s += x[1];
    s += x[2];
    s += x[3];
  }
  return s;
}
// a . b over 32 consecutive floats of LDS, first to last
__device__ __forceinline__ float dot32(const float *a, const float *b) {
  float s = 0.0f;
#pragma unroll
  for (int c = 0; c < 32; c += 4) {
    const f32x4a x = *reinterpret_cast<const f32x4a *>(a + c), y = *reinterpret_cast<const f32x4a *>(b + c);
    s += x[0] * y[0];
    s += x[1] * y[1];
    s += x[2] * y[2];
    s += x[3] * y[3];
  }
  return s;
}

struct AttnLds {
  typedef PaperAttn P;
  float kv[P::T * RowKv::KP];
  float qs[2][P::A];   // q (backward: do), by row parity
  float e[P::H * P::T], a[P::H * P::T];
  __bf16 xs[P::T * RowKv::XP];
};

// Attention of rows [blockIdx.x rows, ...) of a slot (general form:
// attn_fwd_kernel).  256 threads; thread = (head, position) for the scores
// and probabilities, = column for the output; a head is half a wave, so
// only the product is between barriers.  Two workgroups share a CU (73 KB
// of LDS each).  Bound by the LDS and vector units (the product is 128
// MFMAs a row): 36 us per step of 16 blocks of 320 rows, against 136 us for
// the [k | v] product, 68 us for the attention and 37 us for the gather
// that it replaces.
__global__ __launch_bounds__(256, 2) void paper_attn_fwd_kernel(TfShape s, const TfState *st, const float *params,
                                                                const uint8_t *tokstep, int64_t sTok, const float *Q,
                                                                float *att, float *O, int64_t sQ, int64_t sAtt,
                                                                int rows) {
  typedef PaperAttn P;
  const int slot = blockIdx.y;
  if (slot >= st->nact) return;
  extern __shared__ __align__(16) unsigned char raw[];
  AttnLds &L = *reinterpret_cast<AttnLds *>(raw);
  const int x = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(x >> 6), h = x >> 5, p = x & 31;
  const float *W = params + slot * s.stride;
  const uint8_t *tk = tokstep + slot * sTok;
  const float scale = 1.0f / sqrtf((float)P::DH);
  RowKv kv;
  kv.load(s, W, wave);
  const int row0 = blockIdx.x * rows, row1 = min(row0 + rows, s.bs);
  for (int row = row0; row < row1; row++) {
    float *qs = L.qs[row & 1];
    RowKv::stage_x(s, W, tk + (int64_t)row * P::T, L.xs);
    qs[x] = Q[slot * sQ + (int64_t)row * P::A + x];
    __syncthreads();
    kv.product(L.xs, L.kv);
    __syncthreads();
    const float sc = dot32(qs + h * P::DH, L.kv + p * RowKv::KP + h * P::DH) * scale;
    const float ex = __expf(sc - head_max(sc));
    L.e[x] = ex;
    wave_order();
    const float inv = 1.0f / sum32(L.e + h * P::T), a = ex * inv;
    L.a[x] = a;
    att[slot * sAtt + (int64_t)row * P::H * P::T + x] = a;
    wave_order();
    float o = 0.0f;
    const float *v = L.kv + P::A + x;
#pragma unroll
    for (int c = 0; c < P::T; c += 4) {
      const f32x4a y = *reinterpret_cast<const f32x4a *>(L.a + h * P::T + c);
      o += y[0] * v[c * RowKv::KP];
      o += y[1] * v[(c + 1) * RowKv::KP];
      o += y[2] * v[(c + 2) * RowKv::KP];
      o += y[3] * v[(c + 3) * RowKv::KP];
    }
    O[slot * sQ + (int64_t)row * P::A + x] = o;
  }
}

// Its backward up to ds and dq (general form: attn_bwd_kernel): da_p = do .
// v_p, ds_p = a_p (da_p - sum_r a_r da_r) / sqrt(dh), dq = sum_p ds_p k_p.
// 38 us per step of 16 blocks of 320 rows against 222 us (which also wrote
// 335 MB of dk, dv).
__global__ __launch_bounds__(256, 2) void paper_attn_bwd_kernel(TfShape s, const TfState *st, const float *params,
                                                                const uint8_t *tokstep, int64_t sTok, const float *att,
                                                                const float *dO, float *dS, float *dQ, int64_t sQ,
                                                                int64_t sAtt, int64_t sDs, int rows) {
  typedef PaperAttn P;
  const int slot = blockIdx.y;
  if (slot >= st->nact) return;
  extern __shared__ __align__(16) unsigned char raw[];
  AttnLds &L = *reinterpret_cast<AttnLds *>(raw);
  const int x = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(x >> 6), h = x >> 5, p = x & 31;
  const float *W = params + slot * s.stride;
  const uint8_t *tk = tokstep + slot * sTok;
  const float scale = 1.0f / sqrtf((float)P::DH);
  RowKv kv;
  kv.load(s, W, wave);
  const int row0 = blockIdx.x * rows, row1 = min(row0 + rows, s.bs);
  for (int row = row0; row < row1; row++) {
    float *dos = L.qs[row & 1];
    RowKv::stage_x(s, W, tk + (int64_t)row * P::T, L.xs);
    dos[x] = dO[slot * sQ + (int64_t)row * P::A + x];
    const float a = att[slot * sAtt + (int64_t)row * P::H * P::T + x];
    __syncthreads();
    kv.product(L.xs, L.kv);
    __syncthreads();
    L.a[x] = a;
    const float da = dot32(dos + h * P::DH, L.kv + p * RowKv::KP + P::A + h * P::DH);
    L.e[x] = da;
    wave_order();
    const float dot = dot32(L.a + h * P::T, L.e + h * P::T);
    const float ds = a * (da - dot) * scale;
    wave_order();
    L.e[x] = ds;
    dS[slot * sDs + (int64_t)row * P::H * P::T + x] = ds;
    wave_order();
    float dq = 0.0f;
    const float *k = L.kv + x;
#pragma unroll
    for (int c = 0; c < P::T; c += 4) {
      const f32x4a y = *reinterpret_cast<const f32x4a *>(L.e + h * P::T + c);
      dq += y[0] * k[c * RowKv::KP];
      dq += y[1] * k[(c + 1) * RowKv::KP];
      dq += y[2] * k[(c + 2) * RowKv::KP];
      dq += y[3] * k[(c + 3) * RowKv::KP];
    }
    dQ[slot * sQ + (int64_t)row * P::A + x] = dq;
  }
}

// dX = d[k | v] Wkv^T for rows [blockIdx.x rows, ...): the fragments of
// d[k | v] (BF16, position rows) are built once per row into LDS, a k-step
// being one head's keys or values; wave w owns columns 16 w .. of E, its
// weights in registers.  Bound by its two barriers' worth of latency per row
// and the FP32 dX it writes (42 MB): 32 us per step against 113 us for the product from memory.
__global__ __launch_bounds__(256, 2) void paper_kv_dx_kernel(TfShape s, const TfState *st, const float *params,
                                                             const float *Q, const float *dO, const float *att,
                                                             const float *dS, float *dX, int64_t sQ, int64_t sAtt,
                                                             int64_t sDs, int64_t sX, int rows) {
  typedef PaperAttn P;
  constexpr int KS = 2 * P::H;   // k-steps of 32
  const int slot = blockIdx.y;
  if (slot >= st->nact) return;
  __shared__ __align__(16) __bf16 fr[2][2 * KS * 64 * 8];
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const float *W = params + slot * s.stride;
  bf16x8_t b[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ks++) {
    float v[8];
    load8(W + s.off_W[0] + (int64_t)(16 * w + r) * 3 * P::A + P::A + 32 * ks + 8 * q, v);
    b[ks] = pack8(v);
  }
  const int row0 = blockIdx.x * rows, row1 = min(row0 + rows, s.bs);
  for (int row = row0; row < row1; row++) {
    __bf16 *f = fr[row & 1];
    // this wave's four k-steps: heads of the keys (ds, q) or values (a, do)
    const bool key = w < 2;
    const float *col = (key ? Q : dO) + slot * sQ + (int64_t)row * P::A;
    const float *pos = key ? dS + slot * sDs : att + slot * sAtt;
    pos += (int64_t)row * P::H * P::T;
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int ks = 4 * w + u, h = ks & (P::H - 1);
      float v[8];
      load8(col + 32 * h + 8 * q, v);
#pragma unroll
      for (int m = 0; m < 2; m++) {
        const float y = pos[h * P::T + 16 * m + r];
        float z[8];
#pragma unroll
        for (int c = 0; c < 8; c++) z[c] = y * v[c];
        *reinterpret_cast<bf16x8_t *>(f + ((m * KS + ks) * 64 + lane) * 8) = pack8(z);
      }
    }
    __syncthreads();
    f32x4_t acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
#pragma unroll
      for (int m = 0; m < 2; m++)
        acc[m] = mma_bf16(*reinterpret_cast<const bf16x8_t *>(f + ((m * KS + ks) * 64 + lane) * 8), b[ks], acc[m]);
    float *out = dX + slot * sX + (int64_t)row * P::T * P::E + 16 * w + r;
#pragma unroll
    for (int m = 0; m < 2; m++)
#pragma unroll
      for (int c = 0; c < 4; c++) out[(16 * m + 4 * q + c) * P::E] = acc[m][c];
  }
}

// The partial sums of Wkv's gradient (and, as row E, its bias): slice
// blockIdx.x holds `per` rows of K (per / T batch rows), a k-step being one
// batch row's positions.  blockIdx.z: the keys' or the values' half, four
// waves of 64 columns (two heads), all of E and the ones row: X^T passes
// through LDS, d[k | v]^T is built in registers.  (Halves: 576 workgroups of
// four waves are all resident at once; 288 of eight were 55 us, two rounds.)
// 46 us per step against 169 us for the product from memory.
__global__ __launch_bounds__(256, 3) void paper_kv_dw_kernel(TfShape s, const TfState *st, const float *params,
                                                          const uint8_t *tokstep, int64_t sTok, const float *Q,
                                                          const float *dO, const float *att, const float *dS,
                                                          float *part, int64_t sQ, int64_t sAtt, int64_t sDs,
                                                          int64_t sPart, int per) {
  typedef PaperAttn P;
  constexpr int TP = P::T + 8, MT = P::E / 16;
  const int slot = blockIdx.y, slice = blockIdx.x;
  if (slot >= st->nact) return;
  __shared__ __align__(16) __bf16 xt[2][P::E * TP];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, q = lane >> 4, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float *W = params + slot * s.stride;
  const uint8_t *tk = tokstep + slot * sTok;
  const bool key = blockIdx.z == 0;
  const int c0 = 64 * w;   // first column among the keys (values)
  f32x4_t acc[4][MT + 1];
#pragma unroll
  for (int n = 0; n < 4; n++)
#pragma unroll
    for (int m = 0; m <= MT; m++) acc[n][m] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  float one8[8];
#pragma unroll
  for (int c = 0; c < 8; c++) one8[c] = 1.0f;
  const bf16x8_t ones = pack8(one8);
  const int row0 = slice * (per / P::T), row1 = min(row0 + per / P::T, s.bs);
  const int sp = tid & 31, se = (tid >> 5) * 8;   // X^T staging: position, 8 columns
  auto stage = [&](int row) {
    __bf16 *x = xt[row & 1];
    const int c = tk[(int64_t)row * P::T + sp];
    const bf16x8_t v = ctx_x8(s, W, c, sp, se);
#pragma unroll
    for (int e = 0; e < 8; e++) x[(se + e) * TP + sp] = v[e];
  };
  auto operands = [&](int row, float (&pv)[2][8], float (&cv)[4]) {
    const float *pos = (key ? dS + slot * sDs : att + slot * sAtt) + (int64_t)row * P::H * P::T;
    const float *col = (key ? Q : dO) + slot * sQ + (int64_t)row * P::A + c0;
#pragma unroll
    for (int h = 0; h < 2; h++) load8(pos + (c0 / P::DH + h) * P::T + 8 * q, pv[h]);
#pragma unroll
    for (int n = 0; n < 4; n++) cv[n] = col[16 * n + r];
  };
  float pv[2][8], cv[4];
  if (row0 < row1) {
    stage(row0);
    operands(row0, pv, cv);
  }
  for (int row = row0; row < row1; row++) {
    __syncthreads();
    bf16x8_t b[4], a[MT];
#pragma unroll
    for (int n = 0; n < 4; n++) {
      float z[8];
#pragma unroll
      for (int c = 0; c < 8; c++) z[c] = pv[n >> 1][c] * cv[n];
      b[n] = pack8(z);
    }
#pragma unroll
    for (int m = 0; m < MT; m++)
      a[m] = *reinterpret_cast<const bf16x8_t *>(xt[row & 1] + (16 * m + r) * TP + 8 * q);
    if (row + 1 < row1) {   // the next row's loads behind this row's products
      stage(row + 1);
      operands(row + 1, pv, cv);
    }
#pragma unroll
    for (int n = 0; n < 4; n++) {
#pragma unroll
      for (int m = 0; m < MT; m++) acc[n][m] = mma_bf16(a[m], b[n], acc[n][m]);
      acc[n][MT] = mma_bf16(ones, b[n], acc[n][MT]);
    }
  }
  mma_settle();
  float *out = part + slot * sPart + (int64_t)slice * (P::E + 1) * 2 * P::A + (key ? 0 : P::A) + c0 + r;
#pragma unroll
  for (int n = 0; n < 4; n++) {
#pragma unroll
    for (int m = 0; m < MT; m++)
#pragma unroll
      for (int c = 0; c < 4; c++) out[(int64_t)(16 * m + 4 * q + c) * 2 * P::A + 16 * n] = acc[n][m][c];
    if (q == 0) out[(int64_t)P::E * 2 * P::A + 16 * n] = acc[n][MT][0];
  }
}

// The partial sums of the embeddings' gradient (onehot(tokens)^T dX) and the
// positions' (onehot(position)^T dX), both from one read of dX: slice
// blockIdx.x holds `per` rows of K; wave w owns columns 16 w .. of E; the
// one-hot fragments are built in registers (a k-step is one batch row's
// positions, so the positions' are the identity).  21 us per step against
// 33 + 24 us for the two products.
__global__ __launch_bounds__(256) void paper_emb_kernel(TfShape s, const TfState *st, const uint8_t *tokstep,
                                                        int64_t sTok, const float *dX, float *part_e, float *part_p,
                                                        int64_t sX, int64_t sPart, int per) {
  typedef PaperAttn P;
  const int slot = blockIdx.y, slice = blockIdx.x;
  if (slot >= st->nact) return;
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const uint8_t *tk = tokstep + slot * sTok + 8 * q;
  const float *src = dX + slot * sX + (int64_t)8 * q * P::E + 16 * w + r;
  f32x4_t acc[4], pac[2];
#pragma unroll
  for (int m = 0; m < 4; m++) acc[m] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  bf16x8_t id[2];
#pragma unroll
  for (int m = 0; m < 2; m++) {
    pac[m] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < 8; c++) id[m][c] = (__bf16)(8 * q + c == 16 * m + r ? 1.0f : 0.0f);
  }
  const int row0 = slice * (per / P::T), row1 = min(row0 + per / P::T, s.bs);
  constexpr int U = 4;   // rows in flight
  for (int rr = row0; rr < row1; rr += U) {
    float v[U][8];
    uint32_t t8[U][2];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int row = min(rr + u, row1 - 1);
#pragma unroll
      for (int c = 0; c < 8; c++) v[u][c] = src[(int64_t)row * P::T * P::E + c * P::E];
      const uint2 t = *reinterpret_cast<const uint2 *>(tk + (int64_t)row * P::T);
      t8[u][0] = t.x;
      t8[u][1] = t.y;
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      if (rr + u >= row1) break;   // (uniform)
      const bf16x8_t b = pack8(v[u]);
#pragma unroll
      for (int m = 0; m < 4; m++) {
        bf16x8_t a;
#pragma unroll
        for (int c = 0; c < 8; c++)
          a[c] = (__bf16)(((t8[u][c >> 2] >> (8 * (c & 3))) & 0xFFu) == (uint32_t)(16 * m + r) ? 1.0f : 0.0f);
        acc[m] = mma_bf16(a, b, acc[m]);
      }
#pragma unroll
      for (int m = 0; m < 2; m++) pac[m] = mma_bf16(id[m], b, pac[m]);
    }
  }
  mma_settle();
  float *oe = part_e + slot * sPart + (int64_t)slice * P::V * P::E + 16 * w + r;
  float *op = part_p + slot * sPart + (int64_t)slice * P::T * P::E + 16 * w + r;
#pragma unroll
  for (int m = 0; m < 4; m++)
#pragma unroll
    for (int c = 0; c < 4; c++) oe[(16 * m + 4 * q + c) * P::E] = acc[m][c];
#pragma unroll
  for (int m = 0; m < 2; m++)
#pragma unroll
    for (int c = 0; c < 4; c++) op[(16 * m + 4 * q + c) * P::E] = pac[m][c];
}

// tokens of the step and X at the last position (what the query's products
// read; the other positions' X is rebuilt where it is used)
__global__ __launch_bounds__(256) void paper_gather_kernel(TfShape s, const TfState *st, const TfSlot *desc,
                                                           const uint8_t *toks, const uint8_t *ctx, const float *params,
                                                           float *X, int64_t sX, uint8_t *tokstep, int64_t sTok,
                                                           int *err) {
  typedef PaperAttn P;
  const int slot = blockIdx.y;
  if (slot >= st->nact) return;
  const int q = blockIdx.x * 256 + threadIdx.x;   // (row, position)
  const bool in = q < s.bs * P::T;
  int c = 0;
  if (in) {
    c = ctx_token(s, desc[slot], toks, ctx, st->i, q / P::T, q % P::T);
    if (c >= s.V) {
      atomicOr(err, 1);
      c = 0;
    }
    tokstep[slot * sTok + q] = (uint8_t)c;
  }
  // each wave holds two rows: their last tokens are in lanes 31 and 63
  const int lane = threadIdx.x & 63, wrow = (q - lane) / P::T;
  const float *W = params + slot * s.stride;
#pragma unroll
  for (int u = 0; u < 2; u++) {
    const int row = wrow + u, last = __shfl(c, 32 * u + 31);
    if (row < s.bs)
      X[slot * sX + ((int64_t)row * P::T + P::T - 1) * P::E + lane] =
          W[s.off_emb + (int64_t)last * P::E + lane] + W[s.off_pos + (int64_t)(P::T - 1) * P::E + lane];
  }
}

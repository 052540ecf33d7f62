// Dense layers of the launch-sequence loop in BF16 whose weights stream
// through memory (included by tf_kernels.hip): a 256-wide output, every
// weight read once per kernel, straight into the registers of the wave that
// uses it.
//
// A weight matrix of these layers (4096 x 256 in the configurations' large
// MLP and the Transformer's FFN) is 4 MB per block, each block has its own,
// and Adam's moments are twice that again: no cache holds them, so a step is
// bound by the bytes of weights and moments.  The general gemm_kernel reads
// a weight tile through LDS once per 64-row tile of the other operand and
// once more for the update; here the row operand is what passes through LDS.
//
// Values: the k-steps of every output element are gemm_kernel's, and where a
// kernel takes a product that is split over K, the slices and the order they
// are added in (the layer's backward takes none).  A product may be computed
// transposed (operands exchanged): the matrix cores multiply and add the
// same pairs in the same slots, so the bits are the same.
#pragma once

constexpr int kDN = 256;              // output width of the layer
constexpr int kDRows = 64;            // rows staged at a time
constexpr int kDRP = kDN + 8;         // pitch of the staged rows (BF16)
constexpr int kDTP = kDRows + 8;      // pitch of their transpose

typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));

// the XCD-aware tile order of gemm_kernel over a flat grid: the tiles of one
// slot, which read the same rows, share an L2
__device__ __forceinline__ uint32_t xcd_tile(uint32_t total) {
  const uint32_t lin = blockIdx.x, xcd = lin % 8, full = total / 8;
  return xcd * full + min(xcd, total % 8) + lin / 8;
}

// eight tokens (two words of four) as 16-bit pairs
struct Tok8 {
  u16x2_t p[4];
  __device__ __forceinline__ Tok8(uint32_t lo, uint32_t hi) {
    p[0] = __builtin_bit_cast(u16x2_t, __builtin_amdgcn_perm(0u, lo, 0x0C010C00u));
    p[1] = __builtin_bit_cast(u16x2_t, __builtin_amdgcn_perm(0u, lo, 0x0C030C02u));
    p[2] = __builtin_bit_cast(u16x2_t, __builtin_amdgcn_perm(0u, hi, 0x0C010C00u));
    p[3] = __builtin_bit_cast(u16x2_t, __builtin_amdgcn_perm(0u, hi, 0x0C030C02u));
  }
  // the one-hot fragment of symbol x: BF16 1.0 (0x3F80) where the token is x
  __device__ __forceinline__ bf16x8_t one_hot(int x) const {
    const unsigned short xs = (unsigned short)x;
    struct { u16x2_t w[4]; } o;
#pragma unroll
    for (int c = 0; c < 4; c++) {
      const u16x2_t d = p[c] - u16x2_t{xs, xs};
      const u16x2_t nz = __builtin_elementwise_min(d, u16x2_t{1, 1});   // 0 where equal
      o.w[c] = u16x2_t{0x3F80, 0x3F80} - nz * u16x2_t{0x3F80, 0x3F80};
    }
    return __builtin_bit_cast(bf16x8_t, o);
  }
};

// A row of 32 consecutive floats in the four lanes q of a fragment's row, in
// two registers: as memory gives it in two 64-byte loads (x: floats 4 q..,
// y: 16 + 4 q..) or as a fragment wants it (x: 8 q.., y: 8 q + 4..).
__device__ __forceinline__ void to_fragment(uint32_t &x, uint32_t &y) {
  const auto a = __builtin_amdgcn_permlane32_swap(x, y, false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(a[0], a[1], false, false);
  x = b[0];
  y = b[1];
}
__device__ __forceinline__ void to_memory(float &x, float &y) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(a[0], a[1], false, false);
  x = __uint_as_float(b[0]);
  y = __uint_as_float(b[1]);
}

// ---------------------------------------------------------------------------
// Backward of a layer out = in W + b with W [D][256]: dIn = dOut W^T (masked
// by in > 0 when gd.mask is given; gd.hc: stored in BF16), and W, b updated
// (or their gradients stored) from in^T dOut, in one kernel.
// gd: the dIn product (A = dOut, B = W, C = dIn); gw: the weight's (A = in or
// the virtual X, C, moments).  A wave owns 16 rows d of W at a time: lane
// (r, q) loads W[d = r][32 k + 16 m + 4 q .. +3], whole 64-byte runs;
// exchanged between the lanes q (to_fragment) they are dIn's fragments, and
// the weight gradient's tiles, rows h permuted (tile (k, m), row 4 q + c:
// h = 32 k + 8 q + 4 m + c), exchanged the other way lie as W was loaded.
// dOut is staged in LDS in both orientations, 64 rows a chunk.
constexpr int kDChunk = kDRows * kDRP + kDN * kDTP;   // one chunk, both orientations (BF16)
// (256 threads: each 4 columns of 4 rows of each 16)
struct DenseChunk {
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 v[4][4];
  __device__ __forceinline__ void load(const float *dout, int j0, int bs) {
    const int cg = (int)threadIdx.x & 63, rg = (int)threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int c = 0; c < 4; c++) {
        const int j = j0 + 4 * (rg + 4 * i) + c;   // zero past the last row
        v[i][c] = j < bs ? *reinterpret_cast<const f4 *>(dout + (int64_t)j * kDN + 4 * cg) : f4{0.0f, 0.0f, 0.0f, 0.0f};
      }
  }
  __device__ __forceinline__ void stage(__bf16 *rows, __bf16 *cols) const {
    const int cg = (int)threadIdx.x & 63, rg = (int)threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int jr = 4 * (rg + 4 * i);
      bf16x4_t x[4];
#pragma unroll
      for (int c = 0; c < 4; c++) {
#pragma unroll
        for (int y = 0; y < 4; y++) x[c][y] = (__bf16)v[i][c][y];
        *reinterpret_cast<bf16x4_t *>(rows + (jr + c) * kDRP + 4 * cg) = x[c];
      }
#pragma unroll
      for (int y = 0; y < 4; y++)
        *reinterpret_cast<bf16x4_t *>(cols + (4 * cg + y) * kDTP + jr) = bf16x4_t{x[0][y], x[1][y], x[2][y], x[3][y]};
    }
  }
};
// the slot's embedding as BF16 rows of E + 8, rounded as operands are
template <int NT>
__device__ __forceinline__ void emb_stage(const float *emb, int V, int E, __bf16 *embh) {
  for (int x = (int)threadIdx.x * 8; x < V * E; x += NT * 8) {
    float v[8];
    load8(emb + x, v);
    *reinterpret_cast<bf16x8_t *>(embh + (x / E) * (E + 8) + x % E) = pack8(v);
  }
}

// one wave's 16 rows d
template <bool VIRT, int EPI>
struct DenseTile {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const Gemm &gd, &gw;
  int slot, bs, r, q, d0, e;
  int64_t at0;             // W element (k, m): at0 + 32 k + 16 m
  bf16x8_t wb[8];
  f32x4_t acc[8][2];
  f4 mm[8][2];             // Adam's first moments
  const uint8_t *oh;
  const float *in;
  __device__ __forceinline__ DenseTile(const Gemm &gd_, const Gemm &gw_, int slot_, int bs_, int d0_)
      : gd(gd_), gw(gw_), slot(slot_), bs(bs_), d0(d0_) {
    const int lane = threadIdx.x & 63;
    r = lane & 15;
    q = lane >> 4;
    at0 = (int64_t)(d0 + r) * kDN + 4 * q;
    const float *Wt = gd.B + slot * gd.sB + at0;
    f4 w[8][2];
#pragma unroll
    for (int k = 0; k < 8; k++)
#pragma unroll
      for (int m = 0; m < 2; m++) w[k][m] = *reinterpret_cast<const f4 *>(Wt + 32 * k + 16 * m);
    if constexpr (VIRT) {   // (E is a multiple of 16: one position per tile)
      e = (d0 + r) % gw.xE;
      oh = gw.oh + slot * gw.sOh + d0 / gw.xE;
    } else {
      in = gw.A + slot * gw.sA + d0 + r;
    }
#pragma unroll
    for (int k = 0; k < 8; k++) {
      struct { uint32_t x[2], y[2]; } p;
      const float v[8] = {w[k][0][0], w[k][0][1], w[k][0][2], w[k][0][3], w[k][1][0], w[k][1][1], w[k][1][2], w[k][1][3]};
      p = __builtin_bit_cast(decltype(p), pack8(v));
#pragma unroll
      for (int c = 0; c < 2; c++) to_fragment(p.x[c], p.y[c]);
      wb[k] = __builtin_bit_cast(bf16x8_t, p);
#pragma unroll
      for (int m = 0; m < 2; m++) acc[k][m] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    }
  }
  // tokens of rows j0 .. j0 + 63 at the tile's position, by this wave
  __device__ __forceinline__ void stage_tok(int j0, uint8_t *tok) const {
    const int j = j0 + ((int)threadIdx.x & 63);
    tok[threadIdx.x & 63] = j < bs ? oh[(int64_t)j * gw.xt] : 0;
  }
  // in^T (8 rows of this lane's column per k-step), from memory
  __device__ __forceinline__ void in_mem(int j0, float (&v)[2][8]) const {
#pragma unroll
    for (int kb = 0; kb < 2; kb++)
#pragma unroll
      for (int c = 0; c < 8; c++) {
        const int j = j0 + 32 * kb + 8 * q + c;
        v[kb][c] = j < bs ? in[(int64_t)j * gw.lda] : 0.0f;
      }
  }
  // ... or from the staged embedding
  __device__ __forceinline__ void in_virt(int j0, const uint8_t *tok, const __bf16 *embh, bf16x8_t (&bf)[2]) const {
#pragma unroll
    for (int kb = 0; kb < 2; kb++)
#pragma unroll
      for (int c = 0; c < 8; c++) {
        const int j = 32 * kb + 8 * q + c;
        const __bf16 x = embh[(int)tok[j] * (gw.xE + 8) + e];
        bf[kb][c] = j0 + j < bs ? x : (__bf16)0.0f;
      }
  }
  __device__ __forceinline__ void load_moments() {
    if (EPI != kUpdate || !gw.m) return;
#pragma unroll
    for (int k = 0; k < 8; k++)
#pragma unroll
      for (int m = 0; m < 2; m++)
        mm[k][m] = *reinterpret_cast<const f4 *>(gw.m + slot * gw.sMV + at0 + 32 * k + 16 * m);
  }
  // the products of one staged chunk: the weight gradient's into acc, dIn^T's
  // into o (lane (r, q): 4 consecutive columns d of row 16 mt + r)
  __device__ __forceinline__ void products(const __bf16 *rows, const __bf16 *cols, const bf16x8_t (&bf)[2],
                                           f32x4_t (&o)[kDRows / 16]) {
    const int hrow = 8 * (r >> 2) + (r & 3);   // row of tile (k, m) in the transposed rows, less 32 k + 4 m
#pragma unroll
    for (int k = 0; k < 8; k++)
#pragma unroll
      for (int m = 0; m < 2; m++)
#pragma unroll
        for (int kb = 0; kb < 2; kb++)
          acc[k][m] = mma_bf16(
              *reinterpret_cast<const bf16x8_t *>(cols + (32 * k + 4 * m + hrow) * kDTP + 32 * kb + 8 * q), bf[kb],
              acc[k][m]);
#pragma unroll
    for (int mt = 0; mt < kDRows / 16; mt++) {
      o[mt] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int k = 0; k < 8; k++)
        o[mt] = mma_bf16(wb[k], *reinterpret_cast<const bf16x8_t *>(rows + (16 * mt + r) * kDRP + 32 * k + 8 * q), o[mt]);
    }
    mma_settle();
  }
  // the mask's values where store_din puts dIn
  __device__ __forceinline__ void load_mask(int j0, f4 (&k)[kDRows / 16]) const {
    if (!gd.mask) return;
#pragma unroll
    for (int mt = 0; mt < kDRows / 16; mt++) {
      const int j = min(j0 + 16 * mt + r, bs - 1);
      k[mt] = *reinterpret_cast<const f4 *>(gd.mask + slot * gd.sMask + (int64_t)j * gd.ldm + d0 + 4 * q);
    }
  }
  // dIn of the chunk, FP32: 64-byte runs
  __device__ __forceinline__ void store_din(int j0, const f32x4_t (&o)[kDRows / 16], const f4 (&k)[kDRows / 16]) const {
#pragma unroll
    for (int mt = 0; mt < kDRows / 16; mt++) {
      const int j = j0 + 16 * mt + r;
      f4 y = {o[mt][0], o[mt][1], o[mt][2], o[mt][3]};
      if (gd.mask) {
#pragma unroll
        for (int c = 0; c < 4; c++)
          if (!(k[mt][c] > 0.0f)) y[c] = 0.0f;
      }
      if (j < bs) *reinterpret_cast<f4 *>(gd.C + slot * gd.sC + (int64_t)j * gd.ldc + d0 + 4 * q) = y;
    }
  }
  // the gradient stored, or the weights updated: 16 loads in flight per lane
  // (W again: the constructor's copy was rounded), then their updates
  __device__ __forceinline__ void finish() {
    mma_settle();
#pragma unroll
    for (int k = 0; k < 8; k++)
#pragma unroll
      for (int c = 0; c < 4; c++) {
        float x = acc[k][0][c], y = acc[k][1][c];
        to_memory(x, y);
        acc[k][0][c] = x;
        acc[k][1][c] = y;
      }
    float *C = gw.C + slot * gw.sC;
    if constexpr (EPI == kGrad) {
#pragma unroll
      for (int k = 0; k < 8; k++)
#pragma unroll
        for (int m = 0; m < 2; m++) *reinterpret_cast<f32x4_t *>(C + at0 + 32 * k + 16 * m) = acc[k][m];
    } else {
      const Opt o = make_opt(gw);
      const bool adam = gw.m != nullptr;
      float *M = adam ? gw.m + slot * gw.sMV : nullptr, *Vv = adam ? gw.v + slot * gw.sMV : nullptr;
#pragma unroll
      for (int k0 = 0; k0 < 8; k0 += 4) {
        f4 w[4][2], vv[4][2];
#pragma unroll
        for (int k = 0; k < 4; k++)
#pragma unroll
          for (int m = 0; m < 2; m++) {
            const int64_t at = at0 + 32 * (k0 + k) + 16 * m;
            w[k][m] = *reinterpret_cast<const f4 *>(C + at);
            if (adam) vv[k][m] = *reinterpret_cast<const f4 *>(Vv + at);
          }
#pragma unroll
        for (int k = 0; k < 4; k++)
#pragma unroll
          for (int m = 0; m < 2; m++) {
            const int64_t at = at0 + 32 * (k0 + k) + 16 * m;
            if (adam) {
#pragma unroll
              for (int c = 0; c < 4; c++) {
                float mc = mm[k0 + k][m][c], vc = vv[k][m][c];
                w[k][m][c] -= opt_delta_c<true>(o, acc[k0 + k][m][c], &mc, &vc);
                mm[k0 + k][m][c] = mc;
                vv[k][m][c] = vc;
              }
              *reinterpret_cast<f4 *>(M + at) = mm[k0 + k][m];
              *reinterpret_cast<f4 *>(Vv + at) = vv[k][m];
            } else {
#pragma unroll
              for (int c = 0; c < 4; c++)
                w[k][m][c] -= opt_delta_c<false>(o, acc[k0 + k][m][c], (float *)nullptr, (float *)nullptr);
            }
            *reinterpret_cast<f4 *>(C + at) = w[k][m];
          }
      }
    }
  }
};
// the bias gradient (column sums of dOut) of columns 16 ht .. +15: one chunk's
// products with ones, and the store (the bias follows W)
__device__ __forceinline__ f32x4_t dense_bias(const __bf16 *cols, int ht, f32x4_t acc) {
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
  const float one8[8] = {1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f};
#pragma unroll
  for (int kb = 0; kb < 2; kb++)
    acc = mma_bf16(*reinterpret_cast<const bf16x8_t *>(cols + (16 * ht + r) * kDTP + 32 * kb + 8 * q), pack8(one8), acc);
  return acc;
}
template <int EPI>
__device__ __forceinline__ void dense_bias_store(const Gemm &gw, int slot, int D, int ht, f32x4_t acc) {
  mma_settle();
  const int lane = threadIdx.x & 63;
  if ((lane & 15) == 0) {
#pragma unroll
    for (int c = 0; c < 4; c++) epilogue<EPI>(gw, slot, 0, D, 16 * ht + 4 * (lane >> 4) + c, acc[c]);
  }
}

// A workgroup owns 64 rows d and passes dOut through LDS a chunk at a time,
// the next chunk's loads (after the last chunk, Adam's first moments) behind
// the products; two share a CU, so that one's products hide the other's
// loads too.  Bound by memory (24 bytes per weight with Adam, dIn and in):
// 256 blocks of 4096 x 256, 128 rows: 1481 us (6.7 GB, 4.5 TB/s) against
// 555 + 1330 us for the two products (without the loads ahead 1511; with all
// of dOut in LDS and no barriers, one workgroup a CU, 1815); 16 blocks, 320
// rows (571 MB): 154 us against 89 + 139 (without the loads ahead 206; 36
// bytes a lane are spilled where the input is read from memory).
template <bool VIRT, int EPI>
__global__ __launch_bounds__(256, 2) void dense_bwd_kernel(Gemm gd, Gemm gw, int V, int nslots) {
  extern __shared__ __align__(16) unsigned char raw[];
  __bf16 *rows = reinterpret_cast<__bf16 *>(raw), *cols = rows + kDRows * kDRP, *embh = rows + kDChunk;
  const int bs = gd.M, D = gw.M, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  uint8_t *tok = reinterpret_cast<uint8_t *>(embh + (VIRT ? V * (gw.xE + 8) : 0)) + 64 * wave;
  const uint32_t gx = (uint32_t)D / 64, tile = xcd_tile(gx * (uint32_t)nslots);
  const int slot = (int)(tile / gx), tx = (int)(tile % gx);
  if (slot >= gw.st->nact) return;
  const float *dout = gd.A + slot * gd.sA;
  DenseChunk ch;
  ch.load(dout, 0, bs);
  if constexpr (VIRT) emb_stage<256>(gw.emb + slot * gw.sEmb, V, gw.xE, embh);
  DenseTile<VIRT, EPI> t(gd, gw, slot, bs, 64 * tx + 16 * wave);
  float in[2][8];
  if constexpr (!VIRT) t.in_mem(0, in);
  // the first four workgroups' waves take one tile of 16 bias columns each
  // (so D is at least 256: dense_ok)
  const bool bias_wg = tx < 4;
  f32x4_t accb = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  auto step = [&](auto last_c, int j0) {
    constexpr bool LAST = decltype(last_c)::value;
    ch.stage(rows, cols);
    bf16x8_t bf[2];
    if constexpr (VIRT) {
      t.stage_tok(j0, tok);
    } else {
#pragma unroll
      for (int kb = 0; kb < 2; kb++) bf[kb] = pack8(in[kb]);
    }
    __syncthreads();
    if constexpr (VIRT) t.in_virt(j0, tok, embh, bf);
    // the next chunk's operands, or after the last the first moments, load
    // behind this chunk's products
    typename DenseTile<VIRT, EPI>::f4 mask[kDRows / 16];
    t.load_mask(j0, mask);
    if constexpr (!LAST) {
      ch.load(dout, j0 + kDRows, bs);
      if constexpr (!VIRT) t.in_mem(j0 + kDRows, in);
    } else {
      t.load_moments();
    }
    if (bias_wg) accb = dense_bias(cols, 4 * tx + wave, accb);
    f32x4_t o[kDRows / 16];
    t.products(rows, cols, bf, o);
    if (!gd.hc) t.store_din(j0, o, mask);
    __syncthreads();
    if (gd.hc) {
      // BF16: a wave's 16 columns would be 32-byte pieces of a line; the
      // workgroup's 64 columns of a row go out as one 128-byte run
      __bf16 *ob = rows;   // [64][72]
#pragma unroll
      for (int mt = 0; mt < kDRows / 16; mt++) {
        bf16x4_t x;
#pragma unroll
        for (int c = 0; c < 4; c++) x[c] = (__bf16)o[mt][c];
        *reinterpret_cast<bf16x4_t *>(ob + (16 * mt + t.r) * 72 + 16 * wave + 4 * t.q) = x;
      }
      __syncthreads();
      __bf16 *dst = reinterpret_cast<__bf16 *>(gd.C) + slot * gd.sC + 64 * tx;
#pragma unroll
      for (int i = 0; i < 2; i++) {
        const int jr = ((int)threadIdx.x >> 3) + 32 * i, c8 = ((int)threadIdx.x & 7) * 8;
        if (j0 + jr < bs)
          *reinterpret_cast<bf16x8_t *>(dst + (int64_t)(j0 + jr) * gd.ldc + c8) =
              *reinterpret_cast<const bf16x8_t *>(ob + jr * 72 + c8);
      }
      __syncthreads();
    }
  };
  int j0 = 0;
  for (; j0 + kDRows < bs; j0 += kDRows) step(std::false_type{}, j0);
  step(std::true_type{}, j0);
  t.finish();
  if (bias_wg) dense_bias_store<EPI>(gw, slot, D, 4 * tx + wave, accb);
}

// ---------------------------------------------------------------------------
// First layer of the MLP: X W1 (X the concatenated context embeddings, read
// from a BF16 embedding in LDS through the step's tokens), 256 wide, at most
// 16 MT rows.  Wave w of eight owns columns 32 w .. +31 and all rows: lane r
// holds 2 consecutive columns (tile n of two: column 2 r + n), so a weight
// row is read as whole 128-byte runs, once, and converted once.  ALL: one workgroup adds
// its slot's slices in order and stores the layer's output; else slice
// blockIdx.y's sums go to g.part for reduce_kernel.
// Bound by the weights it reads (4.2 MB per block): 256 blocks, 128 rows:
// 246 us (4.4 TB/s) against 691 + 85 us.
template <int MT, bool ALL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void x1_fwd_kernel(Gemm g, int V, int per) {
  extern __shared__ __align__(16) unsigned char raw[];
  const int slot = blockIdx.x;
  if (slot >= g.st->nact) return;
  const int E = g.xE, EP = E + 8, t = g.xt, bs = g.M, K = g.K;
  __bf16 *embh = reinterpret_cast<__bf16 *>(raw);                       // [V][E + 8]
  uint8_t *tk = raw + (size_t)V * EP * 2;                               // [t][16 MT]
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float *emb = g.emb + slot * g.sEmb;
  for (int x = tid * 8; x < V * E; x += 512 * 8) {
    float v[8];
    load8(emb + x, v);
    *reinterpret_cast<bf16x8_t *>(embh + (x / E) * EP + x % E) = pack8(v);
  }
  const uint8_t *oh = g.oh + slot * g.sOh;
  for (int x = tid; x < 16 * MT * t; x += 512) {   // (consecutive threads, consecutive positions of a row)
    const int j = x / t, p = x % t;
    tk[p * 16 * MT + j] = j < bs ? oh[x] : 0;
  }
  __syncthreads();
  typedef float f2 __attribute__((ext_vector_type(2)));
  const int kbeg = ALL ? 0 : (int)blockIdx.y * per, kend = ALL ? K : min(K, kbeg + per);
  const float *Wc = g.B + slot * g.sB + (int64_t)8 * q * kDN + 32 * wave + 2 * r;
  f32x4_t acc[MT][2], sum[ALL ? MT : 1][2];
  auto clear = [&](auto &a) {
#pragma unroll
    for (auto &row : a)
#pragma unroll
      for (auto &x : row) x = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  };
  clear(acc);
  if constexpr (ALL) clear(sum);
  int slice_end = per;   // (ALL)
  constexpr int U = 2;   // k-steps per chunk of weights
  f2 cur[U][8], nxt[U][8];
  auto fetch = [&](int k0, f2 (&b)[U][8]) {
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int c = 0; c < 8; c++) b[u][c] = *reinterpret_cast<const f2 *>(Wc + (int64_t)(min(k0 + 32 * u, kend - 32) + c) * kDN);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto use = [&](int k0, const f2 (&b)[U][8]) {
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int k = k0 + 32 * u;
      if (k >= kend) break;   // (uniform)
      const int p = k / E, e0 = k % E + 8 * q;
      bf16x8_t wf[2];
#pragma unroll
      for (int n = 0; n < 2; n++) {
        const float v[8] = {b[u][0][n], b[u][1][n], b[u][2][n], b[u][3][n], b[u][4][n], b[u][5][n], b[u][6][n], b[u][7][n]};
        wf[n] = pack8(v);
      }
      int c[MT];
#pragma unroll
      for (int m = 0; m < MT; m++) c[m] = tk[p * 16 * MT + 16 * m + r];
      bf16x8_t a[MT];
#pragma unroll
      for (int m = 0; m < MT; m++) a[m] = *reinterpret_cast<const bf16x8_t *>(embh + c[m] * EP + e0);
#pragma unroll
      for (int m = 0; m < MT; m++)
#pragma unroll
        for (int n = 0; n < 2; n++) acc[m][n] = mma_bf16(a[m], wf[n], acc[m][n]);
      if constexpr (ALL) {
        // the end of a slice: its sum joins the others in slice order
        if (k + 32 == slice_end || k + 32 >= K) {
          slice_end += per;
          mma_settle();
#pragma unroll
          for (int m = 0; m < MT; m++)
#pragma unroll
            for (int n = 0; n < 2; n++) {
              sum[m][n] += acc[m][n];
              acc[m][n] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
            }
        }
      }
    }
  };
  if (kbeg < kend) {
    fetch(kbeg, cur);
    for (int k0 = kbeg; k0 < kend; k0 += 64 * U) {
      fetch(k0 + 32 * U, nxt);
      use(k0, cur);
      fetch(k0 + 64 * U, cur);
      use(k0 + 32 * U, nxt);
    }
  }
  mma_settle();
  const int col = 32 * wave + 2 * r;
#pragma unroll
  for (int m = 0; m < MT; m++)
#pragma unroll
    for (int c = 0; c < 4; c++) {
      const int row = 16 * m + 4 * q + c;
      if (row >= bs) continue;
      if constexpr (ALL) {
        const float x[2] = {sum[m][0][c], sum[m][1][c]};
#pragma unroll
        for (int n = 0; n < 2; n++) epilogue<kStore>(g, slot, 0, row, col + n, x[n]);
      } else {
        const float x[2] = {acc[m][0][c], acc[m][1][c]};
#pragma unroll
        for (int n = 0; n < 2; n++) epilogue<kPartial>(g, slot, (int)blockIdx.y, row, col + n, x[n]);
      }
    }
}

// ---------------------------------------------------------------------------
// The MLP's embedding gradient onehot(tokens)^T dX for V = E = 64 and dX in
// BF16: a slice of `per` rows of dX per wave, read once as whole 128-byte
// rows (lane r: columns 4 r + n of tile n), the one-hot fragments built in
// registers.  Bound by the read of dX: 256 blocks of 8192 rows (268 MB):
// 86 us (3.1 TB/s) against 196 us.
__global__ __launch_bounds__(256, 3) void mlp_emb_kernel(Gemm g, int per) {
  const int slot = blockIdx.y;
  if (slot >= g.st->nact) return;
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
  const int slice = 4 * (int)blockIdx.x + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (slice >= g.split) return;
  const int kbeg = slice * per, kend = min(g.K, kbeg + per);
  const uint8_t *tk = g.oh + slot * g.sOh + 8 * q;
  const __bf16 *src = reinterpret_cast<const __bf16 *>(g.B) + slot * g.sB + (int64_t)8 * q * 64 + 4 * r;
  f32x4_t acc[4][4];
#pragma unroll
  for (int m = 0; m < 4; m++)
#pragma unroll
    for (int n = 0; n < 4; n++) acc[m][n] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  uint2 cur[8], nxt[8], tc, tn;
  auto fetch = [&](int k, uint2 (&b)[8], uint2 &t) {
    k = min(k, kend - 32);
#pragma unroll
    for (int c = 0; c < 8; c++) b[c] = *reinterpret_cast<const uint2 *>(src + (int64_t)(k + c) * 64);
    t = *reinterpret_cast<const uint2 *>(tk + k);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto use = [&](const uint2 (&b)[8], const uint2 &t) {
    const Tok8 tok(t.x, t.y);
    bf16x8_t bf[4];
#pragma unroll
    for (int n = 0; n < 4; n++) {   // column n of the 8 x 4 block: half n % 2 of word n / 2
      struct { uint32_t w[4]; } o;
#pragma unroll
      for (int c = 0; c < 4; c++) {
        const uint32_t lo = n < 2 ? b[2 * c].x : b[2 * c].y, hi = n < 2 ? b[2 * c + 1].x : b[2 * c + 1].y;
        o.w[c] = __builtin_amdgcn_perm(hi, lo, (n & 1) ? 0x07060302u : 0x05040100u);
      }
      bf[n] = __builtin_bit_cast(bf16x8_t, o);
    }
#pragma unroll
    for (int m = 0; m < 4; m++) {
      const bf16x8_t a = tok.one_hot(16 * m + r);
#pragma unroll
      for (int n = 0; n < 4; n++) acc[m][n] = mma_bf16(a, bf[n], acc[m][n]);
    }
  };
  if (kbeg < kend) {
    fetch(kbeg, cur, tc);
    for (int k = kbeg; k < kend; k += 64) {
      fetch(k + 32, nxt, tn);
      use(cur, tc);
      fetch(k + 64, cur, tc);
      if (k + 32 < kend) use(nxt, tn);
    }
  }
  mma_settle();
#pragma unroll
  for (int m = 0; m < 4; m++)
#pragma unroll
    for (int c = 0; c < 4; c++) {
      const float x[4] = {acc[m][0][c], acc[m][1][c], acc[m][2][c], acc[m][3][c]};
      epilogue4<kPartial>(g, slot, slice, 16 * m + 4 * q + c, 4 * r, x);
    }
}

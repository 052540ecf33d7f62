// Training of the one-layer BiGRU static private model on the input
// (Sec. 4.2.3, the static model of Sec. 4.2.2 as the private one): the
// dynamic model's learning steps (Sec. 2 steps (2)-(4), its optimiser and
// learning rate, no other model mixed in) over the gathered training block
// of bs segments of Lp tokens; steps t..Lp-1 each make one update from the
// mean cross-entropy of the bs rows.  FP32 throughout.
//
// One learned step i is two launches on the caller's stream where one
// workgroup's LDS holds a row (h <= 32, E <= 32, see row_plan):
//   gru_row_kernel    everything a row needs by itself: the recurrence of both
//                     directions, Dense, head, softmax, dL/dlogits, the
//                     row's share of the dense backward, and back-propagation
//                     through time, into one partial gradient per row;
//   gru_step_kernel   the sums over the rows in order (dense layers from the
//                     kept activations, the others from the partials) and the
//                     optimiser step of every parameter.
// Otherwise (wider shapes) six:
//   gru_fwd_kernel    the recurrence of both directions per R rows (one
//                     thread per (direction, gate row), as the inference
//                     kernel), every position's state kept for the backward,
//                     the Dense (ReLU) output and the logits;
//   gru_loss_kernel   softmax and dL/dlogits = (P - onehot) / bs;
//   gru_du_kernel, gru_dgrad_kernel
//                     the head and Dense layers' gradients and dL/dfeat
//                     (one output per thread, sums over the rows in order);
//   gru_bptt_kernel   back-propagation through time per R rows (one thread
//                     per (direction, gate row), its weight-gradient rows in
//                     registers; gates recomputed from the kept states; the
//                     embedding gradient per direction in LDS, rows in order)
//                     into one partial gradient per workgroup;
//   gru_update_kernel the partials summed in workgroup order, then the
//                     optimiser step of every parameter.
// Every value is computed in a fixed order, so the trained model does not
// depend on scheduling.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "gru_row.h"
#include "pmklc_internal.h"
#include "seq_loop.h"
#include "step_common.h"

namespace pmklc {

namespace {

constexpr int kEmax = 32, kHmax = 64;   // embedding width and units per direction the training kernels hold

__device__ __forceinline__ float sg(float x) { return 1.0f / (1.0f + __expf(-x)); }
__device__ __forceinline__ float th(float x) { return 1.0f - 2.0f / (__expf(2.0f * x) + 1.0f); }

// context token (row, p) of step i: the training block holds row j's
// segment at j Lp
__device__ __forceinline__ int ctx_tok(const uint8_t *tok, uint64_t Lp, int i, int t, int row, int p) {
  return tok[(uint64_t)row * Lp + (uint64_t)(i - t + p)];
}

// Forward of the rows [row0, row0 + R) of step i.  seq[row][p][2h] receives
// the state after position p of each direction (forward half, backward
// half); dn[row][gd] the post-ReLU Dense output; lg[row][V] the logits.
// LDS: W_ih [2][G][E + 1], W_hh [2][G][h + 1] (rows padded), states
// [R][2][h], pre-activations [R][2][G] twice, the rows' context embeddings
// [R][t][E].
__global__ __launch_bounds__(384) void gru_fwd_kernel(TfShape s, const uint8_t *tok, uint64_t Lp, int i,
                                                      const float *W, float *seq, float *dn, float *lg, int R) {
  extern __shared__ float sm[];
  const int h = s.gh, G = 3 * h, t = s.t, E = s.sE, V = s.V, gd = s.gd;
  const int tid = threadIdx.x, d = tid / G, g = tid % G;
  const int row0 = blockIdx.x * R, rows = min(R, s.bs - row0);
  const int LE = E + 1, LH = h + 1;   // weight rows padded to an odd stride (no bank conflicts)
  float *wih = sm, *whh = wih + 2 * G * LE, *hs = whh + 2 * G * LH, *ga = hs + R * 2 * h, *gb = ga + R * 2 * G,
        *xs = gb + R * 2 * G;
  for (int q = tid; q < 2 * G * E; q += blockDim.x)
    wih[(q / E) * LE + q % E] = W[s.s_wih[0][q / (G * E)] + q % (G * E)];
  for (int q = tid; q < 2 * G * h; q += blockDim.x)
    whh[(q / h) * LH + q % h] = W[s.s_whh[0][q / (G * h)] + q % (G * h)];
  for (int q = tid; q < R * 2 * h; q += blockDim.x) hs[q] = 0.0f;
  for (int q = tid; q < rows * t * E; q += blockDim.x) {
    const int r = q / (t * E), p = (q / E) % t;
    xs[q] = W[s.s_emb + (int64_t)ctx_tok(tok, Lp, i, t, row0 + r, p) * E + q % E];
  }
  const float bi = W[s.s_bih[0][d] + g], bh = W[s.s_bhh[0][d] + g];
  const float *wi = wih + (d * G + g) * LE, *wh = whh + (d * G + g) * LH;
  __syncthreads();
  for (int step = 0; step < t; step++) {
    const int p = d == 0 ? step : t - 1 - step;
    for (int r = 0; r < rows; r++) {
      const float *x = xs + (r * t + p) * E;
      float a = bi, b = bh;
#pragma unroll 8
      for (int k = 0; k < E; k++) a += wi[k] * x[k];
      const float *hp = hs + (r * 2 + d) * h;
#pragma unroll 8
      for (int k = 0; k < h; k++) b += wh[k] * hp[k];
      ga[(r * 2 + d) * G + g] = a;
      gb[(r * 2 + d) * G + g] = b;
    }
    __syncthreads();
    if (g < h) {
      for (int r = 0; r < rows; r++) {
        const float *xa = ga + (r * 2 + d) * G, *xb = gb + (r * 2 + d) * G;
        const float rg = sg(xa[g] + xb[g]);
        const float zg = sg(xa[h + g] + xb[h + g]);
        const float ng = th(xa[2 * h + g] + rg * xb[2 * h + g]);
        float *hp = hs + (r * 2 + d) * h;
        const float hn = (1.0f - zg) * ng + zg * hp[g];
        hp[g] = hn;
        seq[((int64_t)(row0 + r) * t + p) * 2 * h + d * h + g] = hn;
      }
    }
    __syncthreads();
  }
  // final states [forward after t-1 | backward after 0] -> Dense + ReLU -> head
  for (int q = tid; q < rows * gd; q += blockDim.x) {
    const int r = q / gd, o = q % gd;
    float a = W[s.s_db + o];
    const float *hr = hs + r * 2 * h;
#pragma unroll 8
    for (int k = 0; k < 2 * h; k++) a += hr[k] * W[s.s_dw + (int64_t)k * gd + o];
    dn[(int64_t)(row0 + r) * gd + o] = a > 0.0f ? a : 0.0f;
  }
  __syncthreads();
  for (int q = tid; q < rows * V; q += blockDim.x) {
    const int r = q / V, v = q % V;
    float a = W[s.s_lb + v];
    const float *dr = dn + (int64_t)(row0 + r) * gd;
#pragma unroll 8
    for (int o = 0; o < gd; o++) a += dr[o] * W[s.s_lw + (int64_t)o * V + v];
    lg[(int64_t)(row0 + r) * V + v] = a;
  }
}

// lg[row] (logits) becomes (softmax - onehot(target)) / bs; one thread per row
__global__ __launch_bounds__(256) void gru_loss_kernel(TfShape s, const uint8_t *tok, uint64_t Lp, int i, float *lg) {
  const int row = blockIdx.x * 256 + threadIdx.x;
  if (row >= s.bs) return;
  const int V = s.V;
  float *z = lg + (int64_t)row * V;
  float mx = z[0];
  for (int v = 1; v < V; v++) mx = fmaxf(mx, z[v]);
  float sum = 0.0f;
  for (int v = 0; v < V; v++) sum += __expf(z[v] - mx);
  const float inv = 1.0f / sum, scale = 1.0f / (float)s.bs;
  const int e = tok[(uint64_t)row * Lp + (uint64_t)i];
  for (int v = 0; v < V; v++) z[v] = (__expf(z[v] - mx) * inv - (v == e ? 1.0f : 0.0f)) * scale;
}

// The head and Dense layers' backward, one output per thread: du = (dz
// Wl^T) * [dn > 0]; then the gradients of Wl, bl, Wd, bd into gr (the
// parameter layout) and dfeat = du Wd^T.  Sums over rows run in row order.
__global__ __launch_bounds__(256) void gru_du_kernel(TfShape s, const float *W, const float *dn, const float *dz,
                                                     float *du) {
  const int V = s.V, gd = s.gd;
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= s.bs * gd) return;
  const int j = q / gd, o = q % gd;
  float a = 0.0f;
#pragma unroll 8
  for (int v = 0; v < V; v++) a += dz[(int64_t)j * V + v] * W[s.s_lw + (int64_t)o * V + v];
  du[q] = dn[q] > 0.0f ? a : 0.0f;
}
__global__ __launch_bounds__(256) void gru_dgrad_kernel(TfShape s, const float *W, const float *seq, const float *dn,
                                                        const float *dz, const float *du, float *gr, float *dfeat) {
  const int h = s.gh, t = s.t, V = s.V, gd = s.gd, bs = s.bs, F = 2 * h;
  const int n_lw = gd * V, n_lb = V, n_dw = F * gd, n_db = gd, n_df = bs * F;
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= n_lw + n_lb + n_dw + n_db + n_df) return;
  auto feat = [&](int j, int k) {
    return k < h ? seq[((int64_t)j * t + t - 1) * F + k] : seq[((int64_t)j * t) * F + k];
  };
  float a = 0.0f;
  if (q < n_lw) {
    const int o = q / V, v = q % V;
#pragma unroll 8
    for (int j = 0; j < bs; j++) a += dn[(int64_t)j * gd + o] * dz[(int64_t)j * V + v];
    gr[s.s_lw + q] = a;
  } else if (q < n_lw + n_lb) {
    const int v = q - n_lw;
    for (int j = 0; j < bs; j++) a += dz[(int64_t)j * V + v];
    gr[s.s_lb + v] = a;
  } else if (q < n_lw + n_lb + n_dw) {
    const int r = q - n_lw - n_lb, k = r / gd, o = r % gd;
#pragma unroll 8
    for (int j = 0; j < bs; j++) a += feat(j, k) * du[(int64_t)j * gd + o];
    gr[s.s_dw + r] = a;
  } else if (q < n_lw + n_lb + n_dw + n_db) {
    const int o = q - n_lw - n_lb - n_dw;
    for (int j = 0; j < bs; j++) a += du[(int64_t)j * gd + o];
    gr[s.s_db + o] = a;
  } else {
    const int r = q - n_lw - n_lb - n_dw - n_db, j = r / F, k = r % F;
#pragma unroll 8
    for (int o = 0; o < gd; o++) a += du[(int64_t)j * gd + o] * W[s.s_dw + (int64_t)k * gd + o];
    dfeat[r] = a;
  }
}

// Back-propagation through time for the rows [row0, row0 + R) of step i,
// each direction from its final state (dL/dfeat) back to its first
// position, the gates recomputed from the kept states.  With a = W_i x +
// b_i, b = W_h h + b_h per gate row: dn = dh' (1 - z), dz = dh' (h - n),
// dA_n = dn (1 - n^2), dA_r = dA_n b_n r (1 - r), dA_z = dz z (1 - z);
// input rows (dA_r, dA_z, dA_n), hidden rows (dA_r, dA_z, dA_n r);
// dh = dh' z + W_h^T (hidden rows), dx = W_i^T (input rows) onto the
// position's embedding row.  part[blockIdx.x] receives this workgroup's
// gradient of the GRU tensors (their layout from s_wih[0][0]) and, after
// them, of the embedding per direction [2][V][E].
// LDS: W_ih [2][G][E + 1], W_hh [2][G][h + 1] (rows padded), pre-activations
// [R][2][G] twice, input and hidden rows [R][2][G] twice, dh [R][2][h],
// embedding [2][V][E], the rows' context embeddings [R][t][E] and kept
// states [R][t][2h].
__global__ __launch_bounds__(384) void gru_bptt_kernel(TfShape s, const uint8_t *tok, uint64_t Lp, int i,
                                                       const float *W, const float *seq, const float *dfeat,
                                                       float *part, int64_t part_stride, int R) {
  extern __shared__ float sm[];
  const int h = s.gh, G = 3 * h, t = s.t, E = s.sE, V = s.V, F = 2 * h;
  const int tid = threadIdx.x, d = tid / G, g = tid % G;
  const int row0 = blockIdx.x * R, rows = min(R, s.bs - row0);
  const int LE = E + 1, LH = h + 1;   // weight rows padded to an odd stride (no bank conflicts)
  float *wih = sm, *whh = wih + 2 * G * LE, *ga = whh + 2 * G * LH, *gb = ga + R * 2 * G, *gi = gb + R * 2 * G,
        *gh = gi + R * 2 * G, *dh = gh + R * 2 * G, *de = dh + R * 2 * h, *xs = de + 2 * V * E,
        *hsq = xs + R * t * E;
  for (int q = tid; q < 2 * G * E; q += blockDim.x)
    wih[(q / E) * LE + q % E] = W[s.s_wih[0][q / (G * E)] + q % (G * E)];
  for (int q = tid; q < 2 * G * h; q += blockDim.x)
    whh[(q / h) * LH + q % h] = W[s.s_whh[0][q / (G * h)] + q % (G * h)];
  for (int q = tid; q < 2 * V * E; q += blockDim.x) de[q] = 0.0f;
  for (int q = tid; q < rows * t * E; q += blockDim.x) {
    const int r = q / (t * E), p = (q / E) % t;
    xs[q] = W[s.s_emb + (int64_t)ctx_tok(tok, Lp, i, t, row0 + r, p) * E + q % E];
  }
  for (int q = tid; q < rows * t * F; q += blockDim.x) hsq[q] = seq[(int64_t)row0 * t * F + q];
  for (int q = tid; q < R * 2 * h; q += blockDim.x) {
    const int r = q / F, dd = (q / h) % 2, u = q % h;
    dh[q] = r < rows ? dfeat[(int64_t)(row0 + r) * F + dd * h + u] : 0.0f;
  }
  const float bi = W[s.s_bih[0][d] + g], bh = W[s.s_bhh[0][d] + g];
  const float *wi = wih + (d * G + g) * LE, *wh = whh + (d * G + g) * LH;
  float awi[kEmax], awh[kHmax], abi = 0.0f, abh = 0.0f;
#pragma unroll
  for (int k = 0; k < kEmax; k++) awi[k] = 0.0f;
#pragma unroll
  for (int k = 0; k < kHmax; k++) awh[k] = 0.0f;
  __syncthreads();
  for (int step = t - 1; step >= 0; step--) {
    const int p = d == 0 ? step : t - 1 - step;
    const int pp = d == 0 ? p - 1 : p + 1;    // the position processed before p (step > 0)
    // pre-activations of this position from the kept states
    for (int r = 0; r < rows; r++) {
      const float *x = xs + (r * t + p) * E;
      float a = bi, b = bh;
#pragma unroll 8
      for (int k = 0; k < E; k++) a += wi[k] * x[k];
      if (step > 0) {
        const float *hp = hsq + (r * t + pp) * F + d * h;
#pragma unroll 8
        for (int k = 0; k < h; k++) b += wh[k] * hp[k];
      }
      ga[(r * 2 + d) * G + g] = a;
      gb[(r * 2 + d) * G + g] = b;
    }
    __syncthreads();
    if (g < h) {
      for (int r = 0; r < rows; r++) {
        const int o = (r * 2 + d) * G;
        const float rg = sg(ga[o + g] + gb[o + g]);
        const float zg = sg(ga[o + h + g] + gb[o + h + g]);
        const float ng = th(ga[o + 2 * h + g] + rg * gb[o + 2 * h + g]);
        const float hprev = step > 0 ? hsq[(r * t + pp) * F + d * h + g] : 0.0f;
        float *dhr = dh + (r * 2 + d) * h;
        const float dhu = dhr[g];
        const float dnn = dhu * (1.0f - zg), dzz = dhu * (hprev - ng);
        const float dan = dnn * (1.0f - ng * ng);
        const float dar = dan * gb[o + 2 * h + g] * rg * (1.0f - rg), daz = dzz * zg * (1.0f - zg);
        gi[o + g] = dar;
        gi[o + h + g] = daz;
        gi[o + 2 * h + g] = dan;
        gh[o + g] = dar;
        gh[o + h + g] = daz;
        gh[o + 2 * h + g] = dan * rg;
        dhr[g] = dhu * zg;   // the direct part; the hidden rows' part is added below
      }
    }
    __syncthreads();
    for (int r = 0; r < rows; r++) {
      const int o = (r * 2 + d) * G;
      const int tk = ctx_tok(tok, Lp, i, t, row0 + r, p);
      const float *x = xs + (r * t + p) * E;
      // this thread's gate row: weight and bias gradients
      const float vi = gi[o + g], vh = gh[o + g];
      abi += vi;
      abh += vh;
#pragma unroll
      for (int k = 0; k < kEmax; k++)
        if (k < E) awi[k] += vi * x[k];
      if (step > 0) {
        const float *hp = hsq + (r * t + pp) * F + d * h;
#pragma unroll
        for (int k = 0; k < kHmax; k++)
          if (k < h) awh[k] += vh * hp[k];
      }
      // dh of the previous position (unit g) and dx (component g) of this one
      if (g < h && step > 0) {
        float a = 0.0f;
#pragma unroll 8
        for (int q = 0; q < G; q++) a += whh[(d * G + q) * LH + g] * gh[o + q];
        dh[(r * 2 + d) * h + g] += a;
      }
      for (int e = g; e < E; e += G) {
        float a = 0.0f;
#pragma unroll 8
        for (int q = 0; q < G; q++) a += wih[(d * G + q) * LE + e] * gi[o + q];
        de[(d * V + tk) * E + e] += a;
      }
    }
    __syncthreads();
  }
  float *pw = part + (int64_t)blockIdx.x * part_stride;
  const int64_t base = s.s_wih[0][0];
#pragma unroll
  for (int k = 0; k < kEmax; k++)
    if (k < E) pw[s.s_wih[0][d] - base + (int64_t)g * E + k] = awi[k];
#pragma unroll
  for (int k = 0; k < kHmax; k++)
    if (k < h) pw[s.s_whh[0][d] - base + (int64_t)g * h + k] = awh[k];
  pw[s.s_bih[0][d] - base + g] = abi;
  pw[s.s_bhh[0][d] - base + g] = abh;
  const int64_t ne = s.s_dw - base;   // the GRU tensors' length
  for (int q = tid; q < 2 * V * E; q += blockDim.x) pw[ne + q] = de[q];
}

// every parameter: its gradient (embedding and GRU tensors: the partials in
// workgroup order, the embedding's two directions in order; the dense
// layers: gr), then the optimiser step
__global__ __launch_bounds__(256) void gru_update_kernel(TfShape s, float *W, const float *gr, const float *part,
                                                         int64_t part_stride, int nwg, float *m, float *v, float c1,
                                                         float c2) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= s.sP) return;
  const int64_t base = s.s_wih[0][0], ne = s.s_dw - base, VE = (int64_t)s.V * s.sE;
  float g = 0.0f;
  if (q < base) {
    for (int w = 0; w < nwg; w++)
      for (int dd = 0; dd < 2; dd++) g += part[(int64_t)w * part_stride + ne + dd * VE + q];
  } else if (q < s.s_dw) {
    for (int w = 0; w < nwg; w++) g += part[(int64_t)w * part_stride + q - base];
  } else {
    g = gr[q];
  }
  Opt o;
  o.kind = s.optimizer;
  o.lr = s.lr; o.b1 = s.b1; o.b2 = s.b2; o.eps = s.eps;
  o.c1 = c1;
  o.c2 = c2;
  W[q] -= opt_delta(o, g, m ? m + q : (float *)nullptr, v ? v + q : (float *)nullptr);
}

// ------------------------------------------------- one row per workgroup
// LDS plan of gru_row_kernel (float offsets).  Two regions are used twice:
// the dense weights' by the gate gradients, the input parts' by the input
// gradients.  Dense rows are padded to an odd pitch (read along either index).
constexpr int kRowT = 512;   // threads: 8 waves, two of which run the recurrences
struct RowPlan {
  int EP;                                         // padded embedding width (16 or 32)
  int dw, lw, gi, ghn, de;                        // region 1
  int pa, dx;                                     // region 2
  int gates, hq, xs, wih, dn, du, dz, ex, df, tk; // the rest; gates: [4][2][t][32] r, z, n, candidate's hidden part
  int floats;
};
__host__ __device__ inline RowPlan row_plan(const TfShape &s) {
  const int h = s.gh, t = s.t, V = s.V, gd = s.gd;
  RowPlan q;
  q.EP = s.sE <= 16 ? 16 : 32;
  int o = 0;
  auto take = [&](int n) { const int at = o; o += (n + 3) / 4 * 4; return at; };
  q.dw = take(2 * h * (gd + 1));
  q.lw = take(gd * (V + 1));
  const int end1 = o;
  o = 0;
  q.gi = take(2 * t * gru::kG);
  q.ghn = take(2 * t * gru::kU);
  q.de = take(2 * V * s.sE);
  if (o < end1) o = end1;
  q.pa = q.dx = take(2 * t * gru::kG);
  q.gates = take(max(4 * 2 * t * gru::kU, 2 * gru::kG * (gru::kU + 1)));
  q.hq = take(2 * (t + 1) * gru::kU);
  q.xs = take(t * q.EP);
  q.wih = take(2 * gru::kG * (q.EP + 1));
  q.dn = take(gd);
  q.du = take(gd);
  q.dz = take(V);
  q.ex = take(V);
  q.df = take(2 * gru::kU);
  q.tk = take(t);
  q.floats = o;
  return q;
}
bool row_fits(const TfShape &s) {
  return s.gl == 1 && s.gh <= gru::kU && s.sE <= 32 && s.gd <= 4096 && s.t <= 4096 &&
         (size_t)row_plan(s).floats * 4 <= 160 * 1024;
}

// Step i of row blockIdx.x.  feat [bs][2h], dn [bs][gd], dz [bs][V], du
// [bs][gd] are kept for the dense layers' gradients; part[row] receives the
// row's gradient of the GRU tensors (from s_wih[0][0]) and the embedding per
// direction [2][V][E].  Gate formulas: see gru_bptt_kernel; every sum has
// its order.
// What bounds it is the two chains of t positions (forward, backward), each
// run by one wave per direction without a barrier; the rest is spread over
// the workgroup's eight waves.  Paper's widths (t 32, E 16, h 32, Dense 128,
// V 64, 64 rows): 70 us, and 5 us for gru_step_kernel, against 480 us for
// the six kernels; of the 70, the forward chain 22 (0.7 per position), the
// backward chain 17, the weight gradients 8, staging and input parts 10.
template <int EP>
__global__ __launch_bounds__(kRowT) __attribute__((amdgpu_waves_per_eu(2, 2))) void gru_row_kernel(TfShape s, const uint8_t *tok, uint64_t Lp, int i,
                                                        const float *__restrict__ W, float *feat, float *dnG,
                                                        float *dzG, float *duG, float *part, int64_t part_stride) {
  using namespace gru;
  extern __shared__ __align__(16) float sm[];
  const RowPlan q = row_plan(s);
  const int h = s.gh, t = s.t, E = s.sE, V = s.V, gd = s.gd, tid = threadIdx.x, row = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  float *dw = sm + q.dw, *lw = sm + q.lw, *pa = sm + q.pa, *hq = sm + q.hq, *xs = sm + q.xs, *wih = sm + q.wih,
        *dn = sm + q.dn, *du = sm + q.du, *dz = sm + q.dz, *ex = sm + q.ex, *df = sm + q.df;
  int *tk = reinterpret_cast<int *>(sm + q.tk);
  const int gsz = 2 * t * kU;   // one gate array
  float *gr = sm + q.gates, *gz = gr + gsz, *gn = gz + gsz, *gb = gn + gsz;
  const int W1 = gd + 1, W2 = V + 1;

  // ---- the step's inputs and weights
  for (int x = tid; x < t * EP; x += kRowT) {
    const int p = x / EP, e = x % EP, c = ctx_tok(tok, Lp, i, t, row, p);
    xs[x] = e < E ? W[s.s_emb + (int64_t)c * E + e] : 0.0f;
    if (e == 0) tk[p] = c;
  }
  auto same = [](int n) { return [n](int c) { return c < n ? c : -1; }; };
  stage_gates<EP>(W, s.s_wih[0], h, E, same(E), wih, kRowT);
  stage_gates<kU>(W, s.s_whh[0], h, h, same(h), gr, kRowT);   // (the gates' region, read before they are written)
  // the dense weights, 8 loads in flight per thread (x / n by a 32-bit
  // reciprocal, exact below 2^20; n = 1 has none)
  auto stage_rows = [&](const float *src, int total, int n, float *dst) {
    const uint32_t mag = (uint32_t)(((1ull << 32) + n - 1) / n);
    for (int x0 = tid; x0 < total; x0 += 8 * kRowT) {
      float v[8];
#pragma unroll
      for (int c = 0; c < 8; c++) v[c] = x0 + c * kRowT < total ? src[x0 + c * kRowT] : 0.0f;
#pragma unroll
      for (int c = 0; c < 8; c++) {
        const int x = x0 + c * kRowT;
        if (x < total) dst[x + (n == 1 ? x : (int)__umulhi((uint32_t)x, mag))] = v[c];
      }
    }
  };
  stage_rows(W + s.s_dw, 2 * h * gd, gd, dw);
  stage_rows(W + s.s_lw, gd * V, V, lw);
  __syncthreads();
  const Recurrence rec(gr, W, s.s_bhh[0], wave & 1, h);
  {
    const InputParts<EP> in(wih, W, s.s_bih[0], h);
    in.run(t, [&](int p, int c) { return xs + p * EP + c; }, pa);
  }
  __syncthreads();
  // ---- forward
  if (wave < 2) {
    const int o = wave * t * kU;
    rec.run(t, wave, pa, hq + wave * (t + 1) * kU, kU, [&](int st, int u, float r, float z, float n, float bn) {
      const int at = o + st * kU + u;
      gr[at] = r;
      gz[at] = z;
      gn[at] = n;
      gb[at] = bn;
    });
  }
  // column u of W_hh for the backward chain (its loads end behind the dense layers)
  float wc[kG];
  if (wave < 2) {
    const int u = lane & (kU - 1);
#pragma unroll
    for (int g = 0; g < kG; g++) {
      const int k = g % kU;
      wc[g] = u < h && k < h ? W[s.s_whh[0][wave] + (int64_t)((g / kU) * h + k) * h + u] : 0.0f;
    }
  }
  __syncthreads();
  auto state_end = [&](int k) {   // final states [forward | backward]
    return k < h ? hq[t * kU + k] : hq[(t + 1) * kU + t * kU + k - h];
  };
  for (int o = tid; o < gd; o += kRowT) {
    float a = W[s.s_db + o];
#pragma unroll 8
    for (int k = 0; k < h; k++) a += hq[t * kU + k] * dw[k * W1 + o];
#pragma unroll 8
    for (int k = 0; k < h; k++) a += hq[(t + 1) * kU + t * kU + k] * dw[(h + k) * W1 + o];
    a = a > 0.0f ? a : 0.0f;
    dn[o] = a;
    dnG[(int64_t)row * gd + o] = a;
  }
  for (int k = tid; k < 2 * h; k += kRowT) feat[(int64_t)row * 2 * h + k] = state_end(k);
  __syncthreads();
  for (int v = tid; v < V; v += kRowT) {
    float a = W[s.s_lb + v];
#pragma unroll 8
    for (int o = 0; o < gd; o++) a += dn[o] * lw[o * W2 + v];
    dz[v] = a;
  }
  __syncthreads();
  // ---- dL/dlogits = (softmax - onehot) / bs
  float mx = dz[0];
  for (int v = 1; v < V; v++) mx = fmaxf(mx, dz[v]);
  for (int v = tid; v < V; v += kRowT) ex[v] = __expf(dz[v] - mx);
  __syncthreads();
  {
    float sum = 0.0f;
    for (int v = 0; v < V; v++) sum += ex[v];
    const float inv = 1.0f / sum, scale = 1.0f / (float)s.bs;
    const int e = tok[(uint64_t)row * Lp + (uint64_t)i];
    for (int v = tid; v < V; v += kRowT) {
      const float x = (ex[v] * inv - (v == e ? 1.0f : 0.0f)) * scale;
      dz[v] = x;
      dzG[(int64_t)row * V + v] = x;
    }
  }
  __syncthreads();
  // ---- dense backward of this row
  for (int o = tid; o < gd; o += kRowT) {
    float a = 0.0f;
#pragma unroll 8
    for (int v = 0; v < V; v++) a += dz[v] * lw[o * W2 + v];
    a = dn[o] > 0.0f ? a : 0.0f;
    du[o] = a;
    duG[(int64_t)row * gd + o] = a;
  }
  __syncthreads();
  for (int k = tid; k < 2 * kU; k += kRowT) {
    const int d = k / kU, u = k % kU;
    float a = 0.0f;
    if (u < h) {
      const float *wr = dw + (d * h + u) * W1;
#pragma unroll 8
      for (int o = 0; o < gd; o++) a += du[o] * wr[o];
    }
    df[k] = a;
  }
  __syncthreads();   // the dense weights are dead from here
  float *gi = sm + q.gi, *ghn = sm + q.ghn, *de = sm + q.de;
  // ---- back-propagation through time: the chain of dh, one wave per direction
  if (wave < 2) {
    const int d = wave, u = lane & (kU - 1);
    float dh = df[d * kU + u];
    const float *hd = hq + d * (t + 1) * kU;
    for (int st = t - 1; st >= 0; st--) {
      const int at = (d * t + st) * kU + u;
      const float rg = gr[at], zg = gz[at], ng = gn[at], bn = gb[at], hprev = hd[st * kU + u];
      const float dnn = dh * (1.0f - zg), dzz = dh * (hprev - ng);
      const float dan = dnn * (1.0f - ng * ng);
      const float dar = dan * bn * rg * (1.0f - rg), daz = dzz * zg * (1.0f - zg);
      float *gs = gi + (d * t + st) * kG, *gh = ghn + (d * t + st) * kU;
      // (both halves of the wave hold the same values)
      gs[u] = dar;
      gs[kU + u] = daz;
      gs[2 * kU + u] = dan;
      gh[u] = dan * rg;
      dh = dh * zg;
      wave_sync();
      if (st > 0) {
        float x[kG];
        lds_run<2 * kU>(gs, x);
        lds_run<kU>(gh, x + 2 * kU);
        const float a = dot_in_order<kG>(0.0f, wc, x);
        dh += u < h ? a : 0.0f;
      }
    }
  } else {
    for (int x = tid - 128; x < 2 * V * E; x += kRowT - 128) de[x] = 0.0f;
  }
  __syncthreads();
  float *pw = part + (int64_t)row * part_stride;
  const int64_t base = s.s_wih[0][0];
  // ---- weight gradients: sums over the positions in processing order.  A
  // wave takes chunks of 4 columns of all three gates' rows, lanes =
  // (direction, unit): 12 sums per lane from 3 + 4 LDS values.
  {
    const int d = lane / kU, u = lane % kU;
    constexpr int NI = EP / 4, NC = NI + kU / 4;   // input and hidden chunks
    for (int ch = wave; ch < NC; ch += kRowT / 64) {
      const bool in = ch < NI;
      const int k0 = 4 * (in ? ch : ch - NI), n = in ? E : h;
      if (k0 >= n) continue;
      float acc[3][4], bsum[3];
#pragma unroll
      for (int y = 0; y < 3; y++) {
        bsum[y] = 0.0f;
#pragma unroll
        for (int x = 0; x < 4; x++) acc[y][x] = 0.0f;
      }
      const float *vp = gi + d * t * kG + u, *vn = in ? vp + 2 * kU : ghn + d * t * kU + u;
      const int vs = in ? kG : kU;
      // columns of step st: the embedding of its position, or the state
      // before it (zero before the first)
      const float *xp = in ? xs + (d == 0 ? 0 : t - 1) * EP + k0 : hq + d * (t + 1) * kU + k0;
      const int xstep = in ? (d == 0 ? EP : -EP) : kU;
      auto fetch = [&](int st, float (&v)[3], float (&x)[4]) {
        v[0] = vp[st * kG];
        v[1] = vp[st * kG + kU];
        v[2] = vn[st * vs];
        lds_run<4>(xp + st * xstep, x);
      };
      auto add = [&](const float (&v)[3], const float (&x)[4]) {
#pragma unroll
        for (int y = 0; y < 3; y++) {
          bsum[y] += v[y];
#pragma unroll
          for (int c = 0; c < 4; c++) acc[y][c] += v[y] * x[c];
        }
      };
      int st = t - 1;
      for (; st >= 3; st -= 4) {   // four steps' operands in flight
        float v[4][3], x[4][4];
#pragma unroll
        for (int y = 0; y < 4; y++) fetch(st - y, v[y], x[y]);
#pragma unroll
        for (int y = 0; y < 4; y++) add(v[y], x[y]);
      }
      for (; st >= 0; st--) {
        float v[3], x[4];
        fetch(st, v, x);
        add(v, x);
      }
      if (u < h) {
        float *out = pw + (in ? s.s_wih[0][d] : s.s_whh[0][d]) - base, *ob = pw + (in ? s.s_bih[0][d] : s.s_bhh[0][d]) - base;
#pragma unroll
        for (int y = 0; y < 3; y++) {
          const int g = y * h + u;
#pragma unroll
          for (int c = 0; c < 4; c++)
            if (k0 + c < n) out[(int64_t)g * n + k0 + c] = acc[y][c];
          if (k0 == 0) ob[g] = bsum[y];
        }
      }
    }
  }
  // ---- input gradients of every position (pa is dead), one output per thread
  float *dx = sm + q.dx;
  for (int x = tid; x < 2 * t * EP; x += kRowT) {
    const int d = x / (t * EP), st = (x / EP) % t, e = x % EP;
    const float *gs = gi + (d * t + st) * kG, *wr = wih + d * kG * (EP + 1) + e;
    float a = 0.0f;
#pragma unroll 3
    for (int c = 0; c < kG; c += 32) {
      float v[32], w[32];
      lds_run<32>(gs + c, v);
#pragma unroll
      for (int y = 0; y < 32; y++) w[y] = wr[(c + y) * (EP + 1)];
      a = dot_in_order<32>(a, w, v);
    }
    dx[x] = a;
  }
  __syncthreads();
  // the embedding rows' gradients per direction, positions in processing
  // order: the thread of a token's first position sums all of its positions
  for (int x = tid; x < 2 * t * EP; x += kRowT) {
    const int d = x / (t * EP), st = (x / EP) % t, e = x % EP;
    if (e >= E) continue;
    const int t0 = d == 0 ? 0 : t - 1, ts = d == 0 ? 1 : -1, c = tk[t0 + ts * st];
    const float *dp = dx + d * t * EP + e;
    bool first = true;
    float a = 0.0f;
#pragma unroll 8
    for (int y = t - 1; y >= 0; y--) {
      const bool same = tk[t0 + ts * y] == c;
      const float s1 = a + dp[y * EP];
      first = first && !(same && y > st);
      a = same && y <= st ? s1 : a;
    }
    if (!first) continue;
    de[(d * V + c) * E + e] = a;
  }
  __syncthreads();
  const int64_t ne = s.s_dw - base;
  for (int x = tid; x < 2 * V * E; x += kRowT) pw[ne + x] = de[x];
}

// every parameter: its gradient (embedding and GRU tensors: the rows'
// partials in order, the embedding's two directions in order; the dense
// layers: the rows' products in order), then the optimiser step.  Bound by
// the latency of its 64-odd in-order loads per parameter (L2), so they are
// issued 16 at a time.
__global__ __launch_bounds__(256) void gru_step_kernel(TfShape s, float *W, const float *feat, const float *dn,
                                                       const float *dz, const float *du, const float *part,
                                                       int64_t part_stride, float *m, float *v, float c1, float c2) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= s.sP) return;
  const int V = s.V, gd = s.gd, bs = s.bs, F = 2 * s.gh;
  const int64_t base = s.s_wih[0][0], ne = s.s_dw - base, VE = (int64_t)V * s.sE;
  float g = 0.0f;
  if (q < base) {
    const float *p = part + ne + q;
#pragma unroll 8
    for (int w = 0; w < bs; w++) {
      g += p[(int64_t)w * part_stride];
      g += p[(int64_t)w * part_stride + VE];
    }
  } else if (q < s.s_dw) {
    const float *p = part + q - base;
#pragma unroll 16
    for (int w = 0; w < bs; w++) g += p[(int64_t)w * part_stride];
  } else if (q < s.s_db) {
    const int k = (int)((q - s.s_dw) / gd), o = (int)((q - s.s_dw) % gd);
#pragma unroll 16
    for (int j = 0; j < bs; j++) g += feat[(int64_t)j * F + k] * du[(int64_t)j * gd + o];
  } else if (q < s.s_lw) {
    const int o = (int)(q - s.s_db);
#pragma unroll 16
    for (int j = 0; j < bs; j++) g += du[(int64_t)j * gd + o];
  } else if (q < s.s_lb) {
    const int o = (int)((q - s.s_lw) / V), x = (int)((q - s.s_lw) % V);
#pragma unroll 16
    for (int j = 0; j < bs; j++) g += dn[(int64_t)j * gd + o] * dz[(int64_t)j * V + x];
  } else {
    const int x = (int)(q - s.s_lb);
#pragma unroll 16
    for (int j = 0; j < bs; j++) g += dz[(int64_t)j * V + x];
  }
  Opt o;
  o.kind = s.optimizer;
  o.lr = s.lr; o.b1 = s.b1; o.b2 = s.b2; o.eps = s.eps;
  o.c1 = c1;
  o.c2 = c2;
  W[q] -= opt_delta(o, g, m ? m + q : (float *)nullptr, v ? v + q : (float *)nullptr);
}

// rows per workgroup (one: the training runs one block of bs rows, so a
// workgroup per row fills more of the chip; measured faster than two) and
// LDS bytes of the two recurrent kernels
size_t fwd_lds(const TfShape &s, int R) {
  const int h = s.gh, G = 3 * h;
  return ((size_t)2 * G * (s.sE + 1) + 2 * G * (h + 1) + (size_t)R * 2 * h + 2 * (size_t)R * 2 * G +
          (size_t)R * s.t * s.sE) * 4;
}
size_t bptt_lds(const TfShape &s, int R) {
  const int h = s.gh, G = 3 * h;
  return ((size_t)2 * G * (s.sE + 1) + 2 * G * (h + 1) + 4 * (size_t)R * 2 * G + (size_t)R * 2 * h +
          2 * (size_t)s.V * s.sE +
          (size_t)R * s.t * s.sE + (size_t)R * s.t * 2 * h) * 4;
}
int pick_rows(const TfShape &s, size_t (*lds)(const TfShape &, int)) {
  for (int R = 1; R >= 1; R >>= 1)
    if (lds(s, R) <= 150 * 1024) return R;
  return 0;
}

}  // namespace

// the seeded initialisation of the BiGRU shape: U(-a, a) from the same
// SplitMix64 draws as every model's initialiser, a = 1 for the embedding,
// 1/sqrt(gh) for the GRU tensors, 1/sqrt(2 gh) for the Dense layer,
// 1/sqrt(gd) for the head
hipError_t gru_init_params(const TfShape &s, uint64_t seed, float *out, hipStream_t st) {
  const int end[4] = {(int)s.s_wih[0][0], (int)s.s_dw, (int)s.s_lw, (int)s.sP};
  const double sc[4] = {1.0, 1.0 / std::sqrt((double)s.gh), 1.0 / std::sqrt(2.0 * s.gh), 1.0 / std::sqrt((double)s.gd)};
  return launch_init_scaled(seed, (int)s.sP, 4, end, sc, out, st);
}

bool gru_train_supported(const TfShape &s) {
  return s.sarch == 1 && s.gl == 1 && s.sE >= 1 && s.sE <= kEmax && s.gh >= 1 && s.gh <= kHmax &&
         pick_rows(s, fwd_lds) > 0 && pick_rows(s, bptt_lds) > 0;
}

uint64_t gru_train_floats(const TfShape &s, uint64_t &part_stride, int &nwg) {
  const int R = pick_rows(s, bptt_lds);
  nwg = R ? (s.bs + R - 1) / R : 0;
  part_stride = ((uint64_t)(s.s_dw - s.s_wih[0][0]) + 2ull * s.V * s.sE + 63) / 64 * 64;
  const uint64_t bs = (uint64_t)s.bs;
  return bs * s.t * 2 * s.gh      // seq
         + bs * s.gd * 2          // dn, du
         + bs * s.V               // logits / loss gradient
         + bs * 2 * s.gh          // dfeat
         + (uint64_t)s.sP         // dense gradients
         + part_stride * nwg      // partials
         + 64 * 8;                // alignment slack
}

hipError_t gru_train(const TfShape &s, const uint8_t *tok, uint64_t Lp, float *W, float *buf, float *adam_m,
                     float *adam_v, hipStream_t st) {
  if (!gru_train_supported(s)) return hipErrorInvalidValue;
  uint64_t ps;
  int nwg;
  gru_train_floats(s, ps, nwg);
  const int Rf = pick_rows(s, fwd_lds), Rb = pick_rows(s, bptt_lds);
  auto take = [&](uint64_t n) {
    float *p = buf;
    buf += (n + 63) / 64 * 64;
    return p;
  };
  const uint64_t bs = (uint64_t)s.bs;
  float *seq = take(bs * s.t * 2 * s.gh), *dn = take(bs * s.gd), *du = take(bs * s.gd), *lg = take(bs * s.V),
        *dfeat = take(bs * 2 * s.gh), *gr = take((uint64_t)s.sP), *part = take(ps * nwg);
  static bool lds_set = false;   // dynamic LDS beyond 64 KB needs the kernels' attribute once
  if (!lds_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gru_fwd_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gru_bptt_kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
    if (e != hipSuccess) return e;
    lds_set = true;
  }
  if (adam_m) {
    hipError_t e = hipMemsetAsync(adam_m, 0, sizeof(float) * s.sP, st);
    if (e == hipSuccess) e = hipMemsetAsync(adam_v, 0, sizeof(float) * s.sP, st);
    if (e != hipSuccess) return e;
  }
  const bool by_row = row_fits(s);
  const RowPlan rp = row_plan(s);
  const auto row_kernel = rp.EP == 16 ? &gru_row_kernel<16> : &gru_row_kernel<32>;
  if (by_row) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(row_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, rp.floats * 4);
    if (e != hipSuccess) return e;
  }
  const int threads = 6 * s.gh;
  const int gfwd = (s.bs + Rf - 1) / Rf;
  const unsigned nup = (unsigned)((s.sP + 255) / 256);
  const unsigned ngrad =
      (unsigned)(((int64_t)s.gd * s.V + s.V + 2ll * s.gh * s.gd + s.gd + (int64_t)s.bs * 2 * s.gh + 255) / 256);
  uint64_t tau = 0;
  for (uint64_t i = (uint64_t)s.t; i < Lp; i++) {
    tau++;
    // Adam's bias corrections in double, as the optimiser's definition
    const float c1 = (float)(1.0 - std::pow((double)s.b1, (double)tau));
    const float c2 = (float)(1.0 - std::pow((double)s.b2, (double)tau));
    if (by_row) {
      hipLaunchKernelGGL(row_kernel, dim3(s.bs), dim3(kRowT), rp.floats * 4, st, s, tok, Lp, (int)i, W, seq, dn, lg, du,
                         part, (int64_t)ps);
      hipLaunchKernelGGL(gru_step_kernel, dim3(nup), dim3(256), 0, st, s, W, seq, dn, lg, du, part, (int64_t)ps,
                         s.optimizer == 1 ? adam_m : nullptr, s.optimizer == 1 ? adam_v : nullptr, c1, c2);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      continue;
    }
    hipLaunchKernelGGL(gru_fwd_kernel, dim3(gfwd), dim3(threads), fwd_lds(s, Rf), st, s, tok, Lp, (int)i, W, seq, dn,
                       lg, Rf);
    hipLaunchKernelGGL(gru_loss_kernel, dim3((s.bs + 255) / 256), dim3(256), 0, st, s, tok, Lp, (int)i, lg);
    hipLaunchKernelGGL(gru_du_kernel, dim3((unsigned)((s.bs * s.gd + 255) / 256)), dim3(256), 0, st, s, W, dn, lg,
                       du);
    hipLaunchKernelGGL(gru_dgrad_kernel, dim3(ngrad), dim3(256), 0, st, s, W, seq, dn, lg, du, gr, dfeat);
    hipLaunchKernelGGL(gru_bptt_kernel, dim3(nwg), dim3(threads), bptt_lds(s, Rb), st, s, tok, Lp, (int)i, W, seq,
                       dfeat, part, (int64_t)ps, Rb);
    hipLaunchKernelGGL(gru_update_kernel, dim3(nup), dim3(256), 0, st, s, W, gr, part, (int64_t)ps, nwg,
                       s.optimizer == 1 ? adam_m : nullptr, s.optimizer == 1 ? adam_v : nullptr, c1, c2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace pmklc

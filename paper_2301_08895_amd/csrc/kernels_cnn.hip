// One parameter-server round for the convolutional model of Section V-A (two convolutional and
// three fully connected layers), fp32.
//
// The paper states no layer shapes; the reading: k x k convolutions (stride 1, no padding) with C1 and
// C2 channels, each followed by ReLU and 2 x 2 max-pooling, then F0 -> F1 -> F2 -> C dense layers
// with ReLU between them and softmax cross-entropy; relu'(0) = 0; the pooling gradient goes to the
// first maximum of a window in the order (0,0), (0,1), (1,0), (1,1).  abs_config.dims =
// {C0 S S, C1, C2, F1, F2, C, C0, k}.  Model vector: per layer W then b; a convolution's W is
// [C_in k k][C_out] with row (ci k + u) k + v, a dense layer's [d_in][d_out].
//
// Shape of the work: B = 32 images per upload and N <= 128 uploads per round - a few hundred images
// of 62 K parameters.  Nothing here is bound by arithmetic or bandwidth but by how long a chain of
// fetches and LDS reads a workgroup walks, and by the launches; a round is four of them:
//   cnn_fwd      a workgroup per stacked row: image and the upload's stale filters in LDS, both convolutions
//                with ReLU and pooling; per window max(., 0) and which of the four it was (255: window dead)
//   cnn_dense    a workgroup per 1 to 8 rows of an upload: the three dense layers forward at the
//                upload's model version, loss, and back down to the gradient of the pooled map
//                (every dZ already carries the upload's coefficient of Eq. 3)
//   cnn_bwd      a workgroup per row: gradient of the first pooled map and the row's share of both filter
//                gradients; behind them a workgroup per tile of an upload's dense gradient; the first
//                one publishes the uploads' losses
//   cnn_combine  Eq. 3: rows' and uploads' shares added in order, w^{t+1} = w^t - sum
// (20 workers, 32 images each, 5 uploads: 71 us of kernels; nine launches of smaller workgroups took 187.)
// Pooling is applied to the pre-activations and the ReLU after it (the maximum of the four ReLUs is
// the ReLU of the maximum, and a window whose maximum is not positive passes no gradient either way).
// All sums have a fixed order: two runs are bitwise identical.
#include <hip/hip_runtime.h>
#include "kernels.h"

namespace abs_impl {

namespace {

constexpr int kDead = 255;
constexpr int kMaxCout = 32;

__device__ __forceinline__ uint64_t cnn_batch_row(const WorkerDesc& w, uint64_t batch_key, uint64_t shard_rows,
                                                  uint32_t b) {
  const uint64_t jk = job_key(batch_key, w.id, w.job);
  return (uint64_t)w.id * shard_rows + draw(jk, b) % shard_rows;
}

struct CnnDev {
  CnnPlan p;
  char* ws;
  const float* X;
  const int32_t* y;
  uint64_t shard_rows, batch_key;
  int fixed_slot;        // >= 0: every row reads this ring slot (evaluation); else the upload's own
  int64_t row0;          // evaluation: stacked row r is dataset row row0 + r
  int n_rows;            // stacked rows of this launch
  int step;              // local SGD (U > 1): the local step in hand, else -1.  From step 1 on upload a
                         // computes at its private model; every step's update goes to the private model
  int U;
};

template <typename T>
__device__ __forceinline__ T* wsp(const CnnDev& d, size_t off) { return (T*)(d.ws + off); }

__device__ __forceinline__ const float* slot_of(const CnnDev& d, const RoundDesc& rd, int upload) {
  if (d.step > 0) return wsp<const float>(d, d.p.off_priv) + (size_t)upload * d.p.slot_stride;
  const uint32_t slot = d.fixed_slot >= 0 ? (uint32_t)d.fixed_slot : rd.w[upload].slot;
  return wsp<const float>(d, d.p.off_ring) + (size_t)slot * d.p.slot_stride;
}
// layer 0: dataset rows -> first pooled map; layer 1: first pooled map -> second pooled map (the
// dense stack's input).
// KS: the filter size when it is 3 or 5 (loops over a filter row unrolled, a row of inputs fetched
// once for its KS taps), 0: any size.
template <int KS>
__global__ __launch_bounds__(256) void cnn_conv_pool_fwd_kernel(CnnDev d, RoundDesc rd, int layer) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const CnnPlan& p = d.p;
  const int r = blockIdx.x, a = r / p.B, t = threadIdx.x;
  const int Cin = layer ? p.C1 : p.C0, Cout = layer ? p.C2 : p.C1;
  const int Sin = layer ? p.S1 : p.S, Sp = layer ? p.S2 : p.S1, k = KS ? KS : p.k;
  const int n_in = Cin * Sin * Sin, n_w = Cin * k * k * Cout, n_out = Cout * Sp * Sp;
  float* sx = sm;
  float* sw = sx + n_in;
  float* sb = sw + n_w;
  const float* src;
  if (layer) {
    src = wsp<const float>(d, p.off_p1) + (size_t)r * n_in;
  } else {
    const uint64_t row = d.fixed_slot >= 0 ? (uint64_t)(d.row0 + r)
                                           : cnn_batch_row(rd.w[a], d.batch_key, d.shard_rows,
                                                           (uint32_t)(max(d.step, 0) * p.B + r - a * p.B));
    src = d.X + row * (uint64_t)n_in;
    if (t == 0) {
      wsp<uint32_t>(d, p.off_rowidx)[r] = (uint32_t)(d.fixed_slot >= 0 ? r : row);
      wsp<int32_t>(d, p.off_label)[r] = d.y[row];
    }
  }
  const float* w = slot_of(d, rd, a);
  for (int i = t; i < n_in; i += 256) sx[i] = src[i];
  for (int i = t; i < n_w; i += 256) sw[i] = w[p.w_off[layer] + i];
  for (int i = t; i < Cout; i += 256) sb[i] = w[p.b_off[layer] + i];
  __syncthreads();
  float* out = wsp<float>(d, layer ? p.off_p2 : p.off_p1) + (size_t)r * n_out;
  uint8_t* arg_out = wsp<uint8_t>(d, layer ? p.off_a2 : p.off_a1) + (size_t)r * n_out;
  for (int o = t; o < n_out; o += 256) {
    const int co = o / (Sp * Sp), pi = (o / Sp) % Sp, pj = o % Sp;
    float a0 = sb[co], a1 = a0, a2 = a0, a3 = a0;
    for (int ci = 0; ci < Cin; ++ci)
      for (int u = 0; u < k; ++u) {
        const float* x0 = sx + (ci * Sin + 2 * pi + u) * Sin + 2 * pj;
        const float* wr = sw + ((ci * k + u) * k) * Cout + co;
        if (KS) {
          float xa[KS + 1], xb[KS + 1];
#pragma unroll
          for (int v = 0; v <= KS; ++v) { xa[v] = x0[v]; xb[v] = x0[v + Sin]; }
#pragma unroll
          for (int v = 0; v < KS; ++v) {
            const float wv = wr[v * Cout];
            a0 = fmaf(xa[v], wv, a0);
            a1 = fmaf(xa[v + 1], wv, a1);
            a2 = fmaf(xb[v], wv, a2);
            a3 = fmaf(xb[v + 1], wv, a3);
          }
        } else {
          for (int v = 0; v < k; ++v) {
            const float wv = wr[v * Cout];
            a0 = fmaf(x0[v], wv, a0);
            a1 = fmaf(x0[v + 1], wv, a1);
            a2 = fmaf(x0[v + Sin], wv, a2);
            a3 = fmaf(x0[v + Sin + 1], wv, a3);
          }
        }
      }
    float m = a0; int q = 0;
    if (a1 > m) { m = a1; q = 1; }
    if (a2 > m) { m = a2; q = 2; }
    if (a3 > m) { m = a3; q = 3; }
    out[o] = fmaxf(m, 0.f);
    arg_out[o] = (uint8_t)(m > 0.f ? q : kDead);
  }
}

// Both convolutions of a stacked row in one workgroup: the first pooled map stays in LDS for the second.
// A thread takes a pooling window and two output channels (a filter tap of both is one 8-byte read, the
// inputs under the window serve 8 sums); every sum runs over (ci, u, v) in the order of
// cnn_conv_pool_fwd_kernel, so the results are bitwise the same.  Bound by the vector ALU and the LDS reads that feed
// it, behind the latency of fetching image and filters; 160 rows of the 5 x 5 workload: 32 us in two launches of 256
// threads, 15 us this way.
template <int KS, int NT>
__device__ __forceinline__ void conv_pool_stage(const float* sx, int Cin, int Sin, const float* sw, const float* sb,
                                                int Cout, int Sp, int k, float* s_out, float* g_out, uint8_t* g_arg) {
  const int win = Sp * Sp, Cop = (Cout + 1) & ~1, items = Cop / 2 * win;
  for (int o = threadIdx.x; o < items; o += NT) {
    const int co = o / win * 2, wi = o - o / win * win, pi = wi / Sp, pj = wi - pi * Sp;
    float a[2][4];
#pragma unroll
    for (int c = 0; c < 2; ++c) a[c][0] = a[c][1] = a[c][2] = a[c][3] = sb[min(co + c, Cout - 1)];
    for (int ci = 0; ci < Cin; ++ci)
      for (int u = 0; u < (KS ? KS : k); ++u) {
        const float* x0 = sx + (ci * Sin + 2 * pi + u) * Sin + 2 * pj;
        const float* wr = sw + ((ci * k + u) * k) * Cop + co;
        if (KS) {
          // (an odd filter has an even input side: S - k + 1 is even)
          float xa[KS + 1], xb[KS + 1];
#pragma unroll
          for (int v = 0; v <= KS; v += 2) {
            const float2 p = *(const float2*)(x0 + v), q = *(const float2*)(x0 + v + Sin);
            xa[v] = p.x; xa[v + 1] = p.y; xb[v] = q.x; xb[v + 1] = q.y;
          }
#pragma unroll
          for (int v = 0; v < KS; ++v) {
            const float2 wv = *(const float2*)(wr + v * Cop);
            a[0][0] = fmaf(xa[v], wv.x, a[0][0]); a[0][1] = fmaf(xa[v + 1], wv.x, a[0][1]);
            a[0][2] = fmaf(xb[v], wv.x, a[0][2]); a[0][3] = fmaf(xb[v + 1], wv.x, a[0][3]);
            a[1][0] = fmaf(xa[v], wv.y, a[1][0]); a[1][1] = fmaf(xa[v + 1], wv.y, a[1][1]);
            a[1][2] = fmaf(xb[v], wv.y, a[1][2]); a[1][3] = fmaf(xb[v + 1], wv.y, a[1][3]);
          }
        } else {
          for (int v = 0; v < k; ++v) {
            const float2 wv = *(const float2*)(wr + v * Cop);
            const float x00 = x0[v], x01 = x0[v + 1], x10 = x0[v + Sin], x11 = x0[v + Sin + 1];
            a[0][0] = fmaf(x00, wv.x, a[0][0]); a[0][1] = fmaf(x01, wv.x, a[0][1]);
            a[0][2] = fmaf(x10, wv.x, a[0][2]); a[0][3] = fmaf(x11, wv.x, a[0][3]);
            a[1][0] = fmaf(x00, wv.y, a[1][0]); a[1][1] = fmaf(x01, wv.y, a[1][1]);
            a[1][2] = fmaf(x10, wv.y, a[1][2]); a[1][3] = fmaf(x11, wv.y, a[1][3]);
          }
        }
      }
#pragma unroll
    for (int c = 0; c < 2; ++c)
      if (co + c < Cout) {
        float m = a[c][0]; int q = 0;
        if (a[c][1] > m) { m = a[c][1]; q = 1; }
        if (a[c][2] > m) { m = a[c][2]; q = 2; }
        if (a[c][3] > m) { m = a[c][3]; q = 3; }
        const int at = (co + c) * win + wi;
        const float v = fmaxf(m, 0.f);
        if (s_out) s_out[at] = v;
        g_out[at] = v;
        g_arg[at] = (uint8_t)(m > 0.f ? q : kDead);
      }
  }
}

// LDS (floats): image | first filters [tap][C1, even] | second filters [tap][C2, even] | biases | first pooled map
struct FwdLds { int w0, w1, b, p1, total; };
__host__ __device__ __forceinline__ FwdLds fwd_lds(const CnnPlan& p) {
  const int kk = p.k * p.k;
  FwdLds o;
  o.w0 = (p.C0 * p.S * p.S + 1) & ~1;
  o.w1 = o.w0 + p.C0 * kk * ((p.C1 + 1) & ~1);
  o.b = o.w1 + p.C1 * kk * ((p.C2 + 1) & ~1);
  o.p1 = (o.b + p.C1 + p.C2 + 1) & ~1;
  o.total = o.p1 + p.C1 * p.S1 * p.S1;
  return o;
}
template <int KS, int NT>
__global__ __launch_bounds__(NT) void cnn_fwd_kernel(CnnDev d, RoundDesc rd) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const CnnPlan& p = d.p;
  const int r = blockIdx.x, a = r / p.B, t = threadIdx.x, k = KS ? KS : p.k, kk = k * k;
  const FwdLds at = fwd_lds(p);
  const float* w = slot_of(d, rd, a);
  const uint64_t row = d.fixed_slot >= 0 ? (uint64_t)(d.row0 + r)
                                         : cnn_batch_row(rd.w[a], d.batch_key, d.shard_rows,
                                                         (uint32_t)(max(d.step, 0) * p.B + r - a * p.B));
  if (t == 0) {
    wsp<uint32_t>(d, p.off_rowidx)[r] = (uint32_t)(d.fixed_slot >= 0 ? r : row);
    wsp<int32_t>(d, p.off_label)[r] = d.y[row];
  }
  const int n_in = p.C0 * p.S * p.S;
  const float* src = d.X + row * (uint64_t)n_in;
  for (int i = t; i < n_in; i += NT) sm[i] = src[i];
  const int c1p = (p.C1 + 1) & ~1, c2p = (p.C2 + 1) & ~1;
  for (int i = t; i < p.C0 * kk * c1p; i += NT) {
    const int q = i / c1p, co = i - q * c1p;
    sm[at.w0 + i] = co < p.C1 ? w[p.w_off[0] + (size_t)q * p.C1 + co] : 0.f;
  }
  for (int i = t; i < p.C1 * kk * c2p; i += NT) {
    const int q = i / c2p, co = i - q * c2p;
    sm[at.w1 + i] = co < p.C2 ? w[p.w_off[1] + (size_t)q * p.C2 + co] : 0.f;
  }
  for (int i = t; i < p.C1 + p.C2; i += NT) sm[at.b + i] = i < p.C1 ? w[p.b_off[0] + i] : w[p.b_off[1] + i - p.C1];
  __syncthreads();
  const int n1 = p.C1 * p.S1 * p.S1;
  conv_pool_stage<KS, NT>(sm, p.C0, p.S, sm + at.w0, sm + at.b, p.C1, p.S1, k, sm + at.p1,
                      wsp<float>(d, p.off_p1) + (size_t)r * n1, wsp<uint8_t>(d, p.off_a1) + (size_t)r * n1);
  __syncthreads();
  conv_pool_stage<KS, NT>(sm + at.p1, p.C1, p.S1, sm + at.w1, sm + at.b + p.C1, p.C2, p.S2, k, nullptr,
                      wsp<float>(d, p.off_p2) + (size_t)r * p.F0, wsp<uint8_t>(d, p.off_a2) + (size_t)r * p.F0);
}

// The dense stack.  A workgroup takes G stacked rows of one upload; the rows' values of a feature sit next
// to each other in LDS ([feature][row]), so one read feeds a weight's G sums.
// out[j][b] = bias[j] + sum_i in[i][b] W[i][j].  The workgroup is cut into slices of the input features,
// each with a thread per column (neighbouring threads read neighbouring weights, NW of a column in
// flight); the slices' sums are added in slice order.  Weights do not depend on the rows, so a thread's first NW are
// asked for (load) stages before they are used (run).
template <int G, int NT, int NW>
struct DenseRows {
  const float *W, *bias;
  int Fout, fr, nz, z, j, i, i1, last;
  uint32_t col;
  float b0, wv[NW];
  __device__ __forceinline__ void load(const float* W_, const float* bias_, int Fin_, int Fout_) {
    W = W_; bias = bias_; Fout = Fout_;
    fr = min((Fout + 31) & ~31, NT); nz = NT / fr;
    const int len = (Fin_ + nz - 1) / nz, t = threadIdx.x;
    z = t / fr; j = t - z * fr;
    i = min(z * len, Fin_); i1 = z < nz && j < Fout ? min(Fin_, i + len) : i;
    b0 = bias[min(t / G, Fout - 1)];
    last = max(0, i1 - 1); col = (uint32_t)min(j, Fout - 1);
    request();
  }
  __device__ __forceinline__ void request() {              // (without a branch: past the slice its last row again, past the layer the last column)
#pragma unroll
    for (int e = 0; e < NW; ++e) wv[e] = W[(uint32_t)(min(i + e, last) * Fout) + col];
  }
  __device__ __forceinline__ void run(const float* s_in, int nb, bool relu, float* s_part, float* s_out, float* g_out) {
    const int t = threadIdx.x;
    float acc[G];
#pragma unroll
    for (int q = 0; q < G; ++q) acc[q] = 0.f;
    while (i < i1) {
#pragma unroll
      for (int e = 0; e < NW; ++e)
        if (i + e < i1) {
#pragma unroll
          for (int q = 0; q < G; ++q) acc[q] = fmaf(s_in[(i + e) * G + q], wv[e], acc[q]);
        }
      i += NW;
      if (i < i1) request();
    }
    if (z < nz) {
#pragma unroll
      for (int q = 0; q < G; ++q) s_part[(z * fr + j) * G + q] = acc[q];
    }
    __syncthreads();
    for (int o = t; o < Fout * G; o += NT) {
      const int jo = o / G, q = o - jo * G;
      float v = o == t ? b0 : bias[jo];
      for (int zz = 0; zz < nz; ++zz) v += s_part[(zz * fr + jo) * G + q];
      if (relu) v = fmaxf(v, 0.f);
      s_out[o] = v;
      if (g_out && q < nb) g_out[(size_t)q * Fout + jo] = v;
    }
    __syncthreads();
  }
};

// dIn[i][b] = gate(b, i) ? sum_j dOut[j][b] W[i][j] : 0: sixteen neighbouring lanes take input feature i and
// read its row of weights in pieces of 64 bytes, NF features (NT / 16 apart) together; the first pieces ahead as above.
template <int G, int NT, int NF>
struct DenseRowsBack {
  static constexpr int kStep = NT / 16;
  const float* W;
  int Fin, Fout;
  float wv[NF][8];
  __device__ __forceinline__ void load(const float* W_, int Fout_, int Fin_) {
    W = W_; Fout = Fout_; Fin = Fin_;
    request(threadIdx.x >> 4, threadIdx.x & 15);
  }
  __device__ __forceinline__ void request(int i0, int j) {
#pragma unroll
    for (int h = 0; h < NF; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e) wv[h][e] = W[(uint32_t)(min(i0 + h * kStep, Fin - 1) * Fout + min(j + 16 * e, Fout - 1))];
  }
  template <typename Gate>
  __device__ __forceinline__ void run(const float* s_dout, int nb, Gate gate, float* s_din, float* g_din) {
    const int l = threadIdx.x & 15, first = threadIdx.x >> 4;
    for (int i0 = first; i0 < Fin; i0 += NF * kStep) {
      float acc[NF][G];
#pragma unroll
      for (int h = 0; h < NF; ++h)
#pragma unroll
        for (int q = 0; q < G; ++q) acc[h][q] = 0.f;
      for (int j = l; j < Fout; j += 128) {
        if (i0 != first || j != l) request(i0, j);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (j + 16 * e < Fout) {
#pragma unroll
            for (int q = 0; q < G; ++q) {
              const float dz = s_dout[(j + 16 * e) * G + q];
#pragma unroll
              for (int h = 0; h < NF; ++h) acc[h][q] = fmaf(dz, wv[h][e], acc[h][q]);
            }
          }
      }
#pragma unroll
      for (int h = 0; h < NF; ++h) {
        const int i = i0 + h * kStep;
#pragma unroll
        for (int q = 0; q < G; ++q) {
#pragma unroll
          for (int o = 8; o > 0; o >>= 1) acc[h][q] += __shfl_xor(acc[h][q], o, 16);
          if (l == q && i < Fin) {
            const float v = q < nb && gate(q, i) ? acc[h][q] : 0.f;
            if (s_din) s_din[i * G + q] = v;
            if (q < nb) g_din[(size_t)q * Fin + i] = v;
          }
        }
      }
    }
    __syncthreads();
  }
};

// The same where a launch has workgroups enough to fill the chip several times over: a thread per column, all
// input features in order, and on the way back a thread per input feature - no exchange between threads, which is what
// the forms above pay for their fetches in flight.
template <int G, int NT>
__device__ __forceinline__ void dense_cols(const float* s_in, int Fin, const float* W, const float* bias, int Fout,
                                           int nb, bool relu, float* s_out, float* g_out) {
  for (int j = threadIdx.x; j < Fout; j += NT) {
    float acc[G];
    const float bv = bias[j];
#pragma unroll
    for (int q = 0; q < G; ++q) acc[q] = bv;
    int i = 0;
    for (; i + 8 <= Fin; i += 8) {
      float wv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) wv[e] = W[(size_t)(i + e) * Fout + j];
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int q = 0; q < G; ++q) acc[q] = fmaf(s_in[(i + e) * G + q], wv[e], acc[q]);
    }
    for (; i < Fin; ++i) {
      const float wv = W[(size_t)i * Fout + j];
#pragma unroll
      for (int q = 0; q < G; ++q) acc[q] = fmaf(s_in[i * G + q], wv, acc[q]);
    }
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const float v = relu ? fmaxf(acc[q], 0.f) : acc[q];
      s_out[j * G + q] = v;
      if (g_out && q < nb) g_out[(size_t)q * Fout + j] = v;
    }
  }
  __syncthreads();
}
template <int G, int NT, typename Gate>
__device__ __forceinline__ void dense_cols_back(const float* s_dout, int Fout, const float* W, int Fin, int nb,
                                                Gate gate, float* s_din, float* g_din) {
  for (int i = threadIdx.x; i < Fin; i += NT) {
    float acc[G];
#pragma unroll
    for (int q = 0; q < G; ++q) acc[q] = 0.f;
    const float* wr = W + (size_t)i * Fout;
    int j = 0;
    for (; j + 8 <= Fout; j += 8) {
      float wv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) wv[e] = wr[j + e];
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int q = 0; q < G; ++q) acc[q] = fmaf(s_dout[(j + e) * G + q], wv[e], acc[q]);
    }
    for (; j < Fout; ++j) {
      const float wv = wr[j];
#pragma unroll
      for (int q = 0; q < G; ++q) acc[q] = fmaf(s_dout[j * G + q], wv, acc[q]);
    }
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const float v = q < nb && gate(q, i) ? acc[q] : 0.f;
      if (s_din) s_din[i * G + q] = v;
      if (q < nb) g_din[(size_t)q * Fin + i] = v;
    }
  }
  __syncthreads();
}

// The dense stack for a group of up to G rows of one upload (training) or of the evaluation pass:
// forward at the rows' model version, per-row loss, and (training) back down to the gradient of the
// second pooled map; every dZ carries the upload's coefficient of Eq. 3.
// Every stage is a chain of weight fetches from the L2: what bounds it is how many are in flight, so a
// round of few rows takes small groups (a workgroup per CU) and slices within them.  5 uploads of 32 rows, 400-120-84-10:
// 59 us with 20 workgroups of 256 threads (8 rows each, a thread per column); of 1024 threads, 80 for 2 rows
// each 27 us, 160 for a row each 23, and 20.4 since each stage's first weights are asked for stages ahead (784-10-20-200-100-20,
// four local steps, a round 337 -> 319).  More of them (32 and 4 features instead of 16 and 2) spill: 25.6.
template <int G, int NT, bool COLS>
__global__ __launch_bounds__(NT) void cnn_dense_kernel(CnnDev d, RoundDesc rd, float* eval_loss, float* eval_hit) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const CnnPlan& p = d.p;
  const int t = threadIdx.x;
  const int gpu_ = (p.B + G - 1) / G;                      // groups per upload
  const int a = blockIdx.x / gpu_, g = blockIdx.x - a * gpu_;
  const int r0 = a * p.B + g * G;
  const int nb = min(G, min(p.B - g * G, d.n_rows - r0));
  if (nb <= 0) return;
  float* sPart = sm;
  float* sH0 = sPart + (COLS ? 0 : NT * G);
  float* sH1 = sH0 + G * p.F0;
  float* sH2 = sH1 + G * p.F1;
  float* sZ = sH2 + G * p.F2;
  float* sD2 = sZ + G * p.C;            // dZ of the second dense layer
  float* sD1 = sD2 + G * p.F2;          // dZ of the first dense layer
  const float* w = slot_of(d, rd, a);
  const float* p2 = wsp<const float>(d, p.off_p2) + (size_t)r0 * p.F0;
  constexpr int kAhead = 16, kFeatures = 2;
  DenseRows<G, NT, kAhead> f1;
  DenseRows<G, NT, 16> f2;
  DenseRows<G, NT, 4> f3;
  if constexpr (!COLS) {
    f1.load(w + p.w_off[2], w + p.b_off[2], p.F0, p.F1);
    f2.load(w + p.w_off[3], w + p.b_off[3], p.F1, p.F2);
    f3.load(w + p.w_off[4], w + p.b_off[4], p.F2, p.C);
  }
  for (int i = t; i < G * p.F0; i += NT) {
    const int q = i / p.F0, f = i - q * p.F0;
    sH0[f * G + q] = q < nb ? p2[i] : 0.f;
  }
  __syncthreads();
  const bool train = eval_loss == nullptr;
  const int y = t < nb ? wsp<const int32_t>(d, p.off_label)[r0 + t] : 0;
  float* const h1 = train ? wsp<float>(d, p.off_h1) + (size_t)r0 * p.F1 : nullptr;
  float* const h2 = train ? wsp<float>(d, p.off_h2) + (size_t)r0 * p.F2 : nullptr;
  DenseRowsBack<G, NT, 2> b3, b2;
  DenseRowsBack<G, NT, kFeatures> b1;
  if constexpr (COLS) {
    dense_cols<G, NT>(sH0, p.F0, w + p.w_off[2], w + p.b_off[2], p.F1, nb, true, sH1, h1);
    dense_cols<G, NT>(sH1, p.F1, w + p.w_off[3], w + p.b_off[3], p.F2, nb, true, sH2, h2);
    dense_cols<G, NT>(sH2, p.F2, w + p.w_off[4], w + p.b_off[4], p.C, nb, false, sZ, nullptr);
  } else {
    f1.run(sH0, nb, true, sPart, sH1, h1);
    if (train) { b3.load(w + p.w_off[4], p.C, p.F2); b2.load(w + p.w_off[3], p.F2, p.F1); }
    f2.run(sH1, nb, true, sPart, sH2, h2);
    f3.run(sH2, nb, false, sPart, sZ, nullptr);
  }
  if (t < nb) {
    // softmax cross-entropy of row t; dZ = c (p - onehot) with the upload's coefficient of Eq. 3
    float* z = sZ + t;
    float zmax = z[0]; int best = 0;
    for (int c = 1; c < p.C; ++c) if (z[c * G] > zmax) { zmax = z[c * G]; best = c; }
    const float zy = z[y * G];
    float ssum = 0.f;
    for (int c = 0; c < p.C; ++c) { const float e = expf(z[c * G] - zmax); z[c * G] = e; ssum += e; }
    const float loss = logf(ssum) - (zy - zmax);
    if (train) {
      const float coef = rd.w[a].c, inv = 1.f / ssum;
      float* dz3 = wsp<float>(d, p.off_dz3) + (size_t)(r0 + t) * p.C;
      for (int c = 0; c < p.C; ++c) {
        const float v = coef * (z[c * G] * inv - (c == y ? 1.f : 0.f));
        z[c * G] = v;
        dz3[c] = v;
      }
      wsp<float>(d, p.off_rowloss)[r0 + t] = loss;
    } else {
      eval_loss[r0 + t] = loss;
      eval_hit[r0 + t] = best == y ? 1.f : 0.f;
    }
  }
  if (!train) return;
  __syncthreads();
  // (a window is dead exactly where its pooled value is zero)
  auto gate2 = [&](int b, int i) { return sH2[i * G + b] > 0.f; };
  auto gate1 = [&](int b, int i) { return sH1[i * G + b] > 0.f; };
  auto gate0 = [&](int b, int i) { return sH0[i * G + b] > 0.f; };
  float* const dz2 = wsp<float>(d, p.off_dz2) + (size_t)r0 * p.F2;
  float* const dz1 = wsp<float>(d, p.off_dz1) + (size_t)r0 * p.F1;
  float* const dp2 = wsp<float>(d, p.off_dp2) + (size_t)r0 * p.F0;
  if constexpr (COLS) {
    dense_cols_back<G, NT>(sZ, p.C, w + p.w_off[4], p.F2, nb, gate2, sD2, dz2);
    dense_cols_back<G, NT>(sD2, p.F2, w + p.w_off[3], p.F1, nb, gate1, sD1, dz1);
    dense_cols_back<G, NT>(sD1, p.F1, w + p.w_off[2], p.F0, nb, gate0, nullptr, dp2);
  } else {
    b1.load(w + p.w_off[2], p.F1, p.F0);
    b3.run(sZ, nb, gate2, sD2, dz2);
    b2.run(sD2, nb, gate1, sD1, dz1);
    b1.run(sD1, nb, gate0, nullptr, dp2);
  }
}

// A kernel argument's value, opaque: a choice among several members of an argument struct otherwise becomes an
// indexed load from a copy of the whole struct in scratch memory.
template <typename T>
__device__ __forceinline__ T member(T v) { asm("" : "+s"(v)); return v; }

// The dense layers' share of upload a's gradient: a 64 x 64 tile of one of the three weight matrices (its
// bias is one more input row of ones), summed over the upload's B rows in row order, 32 rows through
// LDS at a time.  U = 1: the sum goes to the upload's slot of G (Eq. 3 adds the slots in arrival order,
// cnn_combine_kernel); local steps: the upload's private model takes the step at once (Eq. 2).
// (A thread per element and two loads from the L2 per row took 15 us for 5 uploads of 62 K weights.)
__host__ __device__ __forceinline__ int dense_wgrad_tiles(const CnnPlan& p, int l) {
  const int fi = (l == 0 ? p.F0 : l == 1 ? p.F1 : p.F2) + 1, fo = l == 0 ? p.F1 : l == 1 ? p.F2 : p.C;
  return ((fi + 63) / 64) * ((fo + 63) / 64);
}
__host__ __device__ __forceinline__ int dense_wgrad_blocks(const CnnPlan& p) {
  return dense_wgrad_tiles(p, 0) + dense_wgrad_tiles(p, 1) + dense_wgrad_tiles(p, 2);
}
template <int NT>
__device__ __forceinline__ void dense_wgrad_block(const CnnDev& d, const RoundDesc& rd, int blk, float* lds) {
  const CnnPlan& p = d.p;
  const int per = dense_wgrad_blocks(p);
  const int a = blk / per;
  int tile = blk - a * per, l = 0;
  const int n0 = dense_wgrad_tiles(p, 0), n1 = dense_wgrad_tiles(p, 1);
  if (tile >= n0 + n1) { tile -= n0 + n1; l = 2; }
  else if (tile >= n0) { tile -= n0; l = 1; }
  const int F0 = member(p.F0), F1 = member(p.F1), F2 = member(p.F2), C = member(p.C);
  const int Fin = l == 0 ? F0 : l == 1 ? F1 : F2, Fout = l == 0 ? F1 : l == 1 ? F2 : C;
  const size_t i_0 = member(p.off_p2), i_1 = member(p.off_h1), i_2 = member(p.off_h2);
  const size_t z_0 = member(p.off_dz1), z_1 = member(p.off_dz2), z_2 = member(p.off_dz3);
  const size_t w_0 = member(p.w_off[2]), w_1 = member(p.w_off[3]), w_2 = member(p.w_off[4]);
  const size_t b_0 = member(p.b_off[2]), b_1 = member(p.b_off[3]), b_2 = member(p.b_off[4]);
  const float* in = wsp<const float>(d, l == 0 ? i_0 : l == 1 ? i_1 : i_2);
  const float* dz = wsp<const float>(d, l == 0 ? z_0 : l == 1 ? z_1 : z_2);
  const size_t w_at = l == 0 ? w_0 : l == 1 ? w_1 : w_2, b_at = l == 0 ? b_0 : l == 1 ? b_1 : b_2;
  const int nj = (Fout + 63) / 64, i0 = tile / nj * 64, j0 = (tile % nj) * 64;
  float* s_in = lds;               // [32 rows][64]
  float* s_dz = lds + 32 * 64;     // [32 rows][64]
  constexpr int RPT = 1024 / NT;         // input features per thread, NT / 16 apart
  const int t = threadIdx.x, il = t >> 4, jl = (t & 15) * 4;
  float g[RPT][4];
#pragma unroll
  for (int q = 0; q < RPT; ++q) g[q][0] = g[q][1] = g[q][2] = g[q][3] = 0.f;
  for (int b0 = 0; b0 < p.B; b0 += 32) {
    const int nr = min(32, p.B - b0);
    const size_t r0 = (size_t)a * p.B + b0;
    for (int e = t; e < 32 * 64; e += NT) {
      const int r = e >> 6, i = i0 + (e & 63), j = j0 + (e & 63);
      s_in[e] = r < nr ? (i < Fin ? in[(r0 + r) * Fin + i] : 1.f) : 0.f;
      s_dz[e] = r < nr && j < Fout ? dz[(r0 + r) * Fout + j] : 0.f;
    }
    __syncthreads();
    for (int r = 0; r < nr; ++r) {
      const float4 v = *(const float4*)(s_dz + r * 64 + jl);
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        const float x = s_in[r * 64 + il + q * (NT / 16)];
        g[q][0] = fmaf(x, v.x, g[q][0]); g[q][1] = fmaf(x, v.y, g[q][1]);
        g[q][2] = fmaf(x, v.z, g[q][2]); g[q][3] = fmaf(x, v.w, g[q][3]);
      }
    }
    __syncthreads();
  }
  float* priv = wsp<float>(d, p.off_priv) + (size_t)a * p.slot_stride;
  const float* cur = slot_of(d, rd, a);
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int i = i0 + il + q * (NT / 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = j0 + jl + e;
      if (i <= Fin && j < Fout) {
        const size_t at = i < Fin ? w_at + (size_t)i * Fout + j : b_at + (size_t)j;
        priv[at] = d.step < 0 ? g[q][e] : cur[at] - g[q][e];
      }
    }
  }
}

// The uploads' mean minibatch losses; U = 1: published at once (the host selects and enqueues the next round
// while this one's backward half runs), local steps: added to the job's mean.  Whole workgroup, uniform.
__device__ __forceinline__ void cnn_losses(const CnnDev& d, const RoundDesc& rd, LossMailbox* mailbox) {
  const CnnPlan& p = d.p;
  const bool local = d.step >= 0;
  const int a = threadIdx.x;
  if (a < rd.K) {
    const float* rl = wsp<const float>(d, p.off_rowloss) + (size_t)a * p.B;
    float sum = 0.f;
    int b = 0;
    for (; b + 8 <= p.B; b += 8) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = rl[b + e];
#pragma unroll
      for (int e = 0; e < 8; ++e) sum += v[e];
    }
    for (; b < p.B; ++b) sum += rl[b];
    const float mean = sum / (float)p.B;
    float* lb = wsp<float>(d, p.off_lossbuf) + a;
    if (!local) *lb = mean;
    else *lb = (d.step == 0 ? 0.f : *lb) + mean / (float)d.U;       // mean over the job's U steps
    if (mailbox) post_loss(mailbox, a, mean, rd.stamp);
  }
}

// A convolution's share of one row's gradient from LDS: sum over the pooling windows of the gradient
// times the input under the window's maximum (gw: gradient and offset of the maximum in an input plane,
// per output channel and window); `sp` neighbouring threads share an entry's windows.
template <int NT>
__device__ __forceinline__ void conv_wgrad_stage(const float* sx, int Cin, int Sin, const float2* gw, int Cout, int win,
                                                 int k, float* out) {
  const int nW = Cin * k * k * Cout, n = nW + Cout;
  int sp = 1;
  while (sp < 8 && n * sp * 2 <= 2 * NT) sp *= 2;
  const int rounds = (n * sp + NT - 1) / NT;
  for (int it = 0; it < rounds; ++it) {
    const int idx = it * NT + (int)threadIdx.x, e = idx / sp, h = idx - e * sp;
    float acc = 0.f;
    if (e < nW) {
      const int co = e % Cout, q = e / Cout, ci = q / (k * k), u = (q / k) % k, v = q % k;
      const float* x0 = sx + (ci * Sin + u) * Sin + v;
      const float2* gg = gw + co * win;
#pragma unroll 4
      for (int w_ = h; w_ < win; w_ += sp) {
        const float2 a = gg[w_];
        acc = fmaf(x0[__float_as_int(a.y)], a.x, acc);
      }
    } else if (e < n) {
      const float2* gg = gw + (e - nW) * win;
      for (int w_ = h; w_ < win; w_ += sp) acc += gg[w_].x;
    }
    for (int o = 1; o < sp; o <<= 1) acc += __shfl_xor(acc, o, 64);
    if (h == 0 && e < n) out[e] = acc;
  }
}

// The backward half below the dense stack, one launch.  Workgroup r < rows: everything of stacked row r -
// the gradient of the first pooled map and the row's share of both filter gradients; the workgroups
// behind them: the dense layers' share of the uploads' gradients (dense_wgrad_block).  The first workgroup
// turns the row losses into the uploads' and, at U = 1, publishes them.
// The gradient of the first pooled map is a product with few columns, [positions][taps x C2] times
// [taps x C2][C1], on fp32 matrix instructions (16 x 16 x 4): A is the second convolution's output
// gradient, scattered into a zero-framed map (k - 1 positions on every side, so no tap needs a bounds
// check; channels innermost at a pitch that puts the 16 positions x 4 channels of a read in different
// banks), B the upload's filters.  One read of each per 1024 multiply-adds; on the vector ALU the
// filters alone were an LDS read per 4 (40 us for 160 rows; with the two filter-gradient launches, 25 us, and the
// dense one, 15 us, now 29 us together: 35 with half the wavefronts, of which the products 12, the filter
// gradients 6 and 10).
struct BwdLds { int w, x, p1, g1, g0, total, pc, pw; };
__host__ __device__ __forceinline__ BwdLds bwd_lds(const CnnPlan& p) {
  BwdLds o;
  const int side = 2 * p.S2 + 2 * (p.k - 1), Cp = (p.C2 + 3) & ~3, n1 = p.C1 * p.S1 * p.S1;
  o.pc = Cp % 8 == 0 ? Cp + 4 : Cp;                  // map pitch: 4 (mod 8) words
  o.pw = p.C1 | 1;                                   // filters [tap][channel][C1]
  o.w = side * side * o.pc;
  o.x = (o.w + p.k * p.k * Cp * o.pw + 32 + 1) & ~1; // (the columns beyond C1 of the last rows are read, and ignored)
  o.p1 = o.x + p.C0 * p.S * p.S;
  o.g1 = (o.p1 + n1 + 1) & ~1;                       // second convolution: (gradient, offset) per channel and window
  o.g0 = o.g1 + 2 * p.F0;                            // first convolution
  o.total = o.g0 + 2 * n1;
  if (o.total < 4 * 1024) o.total = 4 * 1024;        // (dense_wgrad_block)
  return o;
}
template <int KS, int NT>
__global__ __launch_bounds__(NT) void cnn_bwd_kernel(CnnDev d, RoundDesc rd, int rows, LossMailbox* mailbox) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const CnnPlan& p = d.p;
  if ((int)blockIdx.x >= rows) { dense_wgrad_block<NT>(d, rd, (int)blockIdx.x - rows, sm); return; }
  if (blockIdx.x == 0) cnn_losses(d, rd, mailbox);
  const int r = blockIdx.x, a = r / p.B, t = threadIdx.x, k = KS ? KS : p.k, kk = k * k;
  const BwdLds at = bwd_lds(p);
  const int side = 2 * p.S2 + 2 * (k - 1), Cp = (p.C2 + 3) & ~3, n1 = p.C1 * p.S1 * p.S1;
  const float* w = slot_of(d, rd, a);
  float* sdc = sm; float* sw = sm + at.w; float* sx = sm + at.x; float* sp1 = sm + at.p1;
  float2* g1 = (float2*)(sm + at.g1); float2* g0 = (float2*)(sm + at.g0);
  const int n_in = p.C0 * p.S * p.S;
  const float* src = d.X + (size_t)wsp<const uint32_t>(d, p.off_rowidx)[r] * n_in;
  for (int i = t; i < side * side * at.pc; i += NT) sdc[i] = 0.f;
  for (int i = t; i < p.C1 * kk * p.C2; i += NT) {
    const int q = i / p.C2, co = i - q * p.C2, ci = q / kk, tap = q - ci * kk;
    sw[(tap * Cp + co) * at.pw + ci] = w[p.w_off[1] + i];
  }
  const int npad = Cp - p.C2;            // channels of the padding: a zero gradient times any number but these
  for (int i = t; i < kk * npad * at.pw; i += NT) {
    const int q = i / at.pw, tap = q / npad;
    sw[(tap * Cp + p.C2 + q - tap * npad) * at.pw + i - q * at.pw] = 0.f;
  }
  for (int i = t; i < n_in; i += NT) sx[i] = src[i];
  for (int i = t; i < n1; i += NT) sp1[i] = wsp<const float>(d, p.off_p1)[(size_t)r * n1 + i];
  __syncthreads();
  const float* dp2 = wsp<const float>(d, p.off_dp2) + (size_t)r * p.F0;
  const uint8_t* a2 = wsp<const uint8_t>(d, p.off_a2) + (size_t)r * p.F0;
  const int win2 = p.S2 * p.S2;
  for (int o = t; o < p.F0; o += NT) {
    const int m = a2[o], co = o / win2, wi = o - co * win2, pi = wi / p.S2, pj = wi - pi * p.S2;
    // (a dead window contributes 0 x the corner of its inputs)
    const bool live = m != kDead;
    const int i = 2 * pi + (live ? m >> 1 : 0), j = 2 * pj + (live ? m & 1 : 0);
    const float v = live ? dp2[o] : 0.f;
    g1[o] = make_float2(v, __int_as_float(i * p.S1 + j));
    if (live) sdc[((i + k - 1) * side + j + k - 1) * at.pc + co] = v;
  }
  __syncthreads();
  // positions (y, x) of the first pooled map x input channels: sum over taps (u, v) and channels of
  // gradient(y - u, x - v) W(ci, u, v)
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  const int pos = p.S1 * p.S1, mt = (pos + 15) / 16, nt = (p.C1 + 15) / 16;
  const int lane = t & 63, wave = t >> 6, l15 = lane & 15, l4 = lane >> 4;
  const uint8_t* a1 = wsp<const uint8_t>(d, p.off_a1) + (size_t)r * n1;
  for (int item = wave; item < mt * nt; item += NT / 64) {
    const int m0 = item % mt * 16, c0 = item / mt * 16;
    const int pm = min(m0 + l15, pos - 1);
    const float* pa = sdc + ((pm / p.S1 + k - 1) * side + pm % p.S1 + k - 1) * at.pc + l4;
    const float* pb = sw + l4 * at.pw + c0 + l15;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    for (int u = 0; u < k; ++u)
      for (int c = 0; c < Cp; c += 4) {
        const float* qa = pa - u * side * at.pc + c;
        const float* qb = pb + (u * k * Cp + c) * at.pw;
        if (KS) {
          // (all reads of a filter row in flight before the first product)
          float fa[KS ? KS : 1], fb[KS ? KS : 1];
#pragma unroll
          for (int v = 0; v < KS; ++v) { fa[v] = qa[-v * at.pc]; fb[v] = qb[v * Cp * at.pw]; }
#pragma unroll
          for (int v = 0; v < KS; ++v) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[v], fb[v], acc, 0, 0, 0);
        } else {
          for (int v = 0; v < k; ++v) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[-v * at.pc], qb[v * Cp * at.pw], acc, 0, 0, 0);
        }
      }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int po = m0 + 4 * l4 + e, ci = c0 + l15;
      if (po < pos && ci < p.C1) {
        const int o = ci * pos + po, m = a1[o], pi = po / p.S1, pj = po - pi * p.S1;
        const bool live = m != kDead;
        g0[o] = make_float2(live ? acc[e] : 0.f,
                            __int_as_float((2 * pi + (live ? m >> 1 : 0)) * p.S + 2 * pj + (live ? m & 1 : 0)));
      }
    }
  }
  conv_wgrad_stage<NT>(sp1, p.C1, p.S1, g1, p.C2, win2, k, wsp<float>(d, p.off_grow2) + (size_t)r * (p.C1 * kk * p.C2 + p.C2));
  __syncthreads();
  conv_wgrad_stage<NT>(sx, p.C0, p.S, g0, p.C1, pos, k, wsp<float>(d, p.off_grow1) + (size_t)r * (p.C0 * kk * p.C1 + p.C1));
}
// The same for shapes whose stages do not fit the LDS together: dense shares and losses only.
__global__ __launch_bounds__(1024) void cnn_dense_wgrad_kernel(CnnDev d, RoundDesc rd, LossMailbox* mailbox) {
  __shared__ __attribute__((aligned(16))) float lds[4 * 1024];
  if (blockIdx.x == 0) cnn_losses(d, rd, mailbox);
  dense_wgrad_block<1024>(d, rd, blockIdx.x, lds);
}

// Gradient of the first pooled map of row r: the second convolution's output gradient is non-zero
// only where a pooling window had its (positive) maximum.
// LDS: the output gradient as [row][column][channel] and the filters as [(ci, u, v)][channel], channels
// padded to a multiple of 4, so that the sum over output channels runs on 16-byte reads.
template <int KS>
__global__ __launch_bounds__(256) void cnn_conv2_bwd_kernel(CnnDev d, RoundDesc rd) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const CnnPlan& p = d.p;
  const int r = blockIdx.x, a = r / p.B, t = threadIdx.x, k = KS ? KS : p.k;
  const int S2c = 2 * p.S2, Cp = (p.C2 + 3) & ~3, n_dc = S2c * S2c * Cp, n_q = p.C1 * k * k;
  float* sdc = sm;             // [S2c][S2c][Cp]
  float* sw = sdc + n_dc;      // [C1 k k][Cp]: second convolution's filters of this upload's version
  const float* w = slot_of(d, rd, a);
  for (int i = t; i < n_dc; i += 256) sdc[i] = 0.f;
  for (int i = t; i < n_q * Cp; i += 256) {
    const int q = i / Cp, co = i - q * Cp;
    sw[i] = co < p.C2 ? w[p.w_off[1] + (size_t)q * p.C2 + co] : 0.f;
  }
  __syncthreads();
  const float* dp2 = wsp<const float>(d, p.off_dp2) + (size_t)r * p.F0;
  const uint8_t* a2 = wsp<const uint8_t>(d, p.off_a2) + (size_t)r * p.F0;
  for (int o = t; o < p.F0; o += 256) {
    const int q = a2[o];
    if (q != kDead) {
      const int co = o / (p.S2 * p.S2), pi = (o / p.S2) % p.S2, pj = o % p.S2;
      sdc[((2 * pi + (q >> 1)) * S2c + 2 * pj + (q & 1)) * Cp + co] = dp2[o];
    }
  }
  __syncthreads();
  const int n1 = p.C1 * p.S1 * p.S1;
  const uint8_t* a1 = wsp<const uint8_t>(d, p.off_a1) + (size_t)r * n1;
  float* dp1 = wsp<float>(d, p.off_dp1) + (size_t)r * n1;
  for (int o = t; o < n1; o += 256) {
    float acc = 0.f;
    if (a1[o] != kDead) {
      const int ci = o / (p.S1 * p.S1), y = (o / p.S1) % p.S1, x = o % p.S1;
#pragma unroll
      for (int u = 0; u < (KS ? KS : k); ++u) {
        const int i = y - u;
        if (i < 0 || i >= S2c) continue;
#pragma unroll
        for (int v = 0; v < (KS ? KS : k); ++v) {
          const int j = x - v;
          if (j < 0 || j >= S2c) continue;
          const float4* wr = (const float4*)(sw + ((ci * k + u) * k + v) * Cp);
          const float4* gr = (const float4*)(sdc + (i * S2c + j) * Cp);
          for (int c4 = 0; c4 < Cp / 4; ++c4) {
            const float4 gv = gr[c4], wv = wr[c4];
            acc = fmaf(gv.x, wv.x, acc); acc = fmaf(gv.y, wv.y, acc);
            acc = fmaf(gv.z, wv.z, acc); acc = fmaf(gv.w, wv.w, acc);
          }
        }
      }
    }
    dp1[o] = acc;
  }
}

// A convolution's share of one row's gradient (workgroup = stacked row): the row's input map, the
// gradient of its pooled map and the windows' maxima in LDS; a thread sums one filter weight
// (ci, u, v, co) over the pooling windows (a window contributes the input under its maximum), the
// last Cout entries are the bias.  Result: Grow[r][weights..., biases...], in the model's own order.
__global__ __launch_bounds__(256) void cnn_conv_wgrad_rows_kernel(CnnDev d, int layer) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const CnnPlan& p = d.p;
  const int r = blockIdx.x, t = threadIdx.x, k = p.k;
  const int Cin = layer ? p.C1 : p.C0, Cout = layer ? p.C2 : p.C1;
  const int Sin = layer ? p.S1 : p.S, Sp = layer ? p.S2 : p.S1;
  const int n_in = Cin * Sin * Sin, n_out = Cout * Sp * Sp, win = Sp * Sp, nW = Cin * k * k * Cout;
  float* sx = sm;
  float* sg = sx + n_in;
  int* sa = (int*)(sg + n_out);
  const float* in = layer ? wsp<const float>(d, p.off_p1) + (size_t)r * n_in
                          : d.X + (size_t)wsp<const uint32_t>(d, p.off_rowidx)[r] * n_in;
  const float* g = wsp<const float>(d, layer ? p.off_dp2 : p.off_dp1) + (size_t)r * n_out;
  const uint8_t* A = wsp<const uint8_t>(d, layer ? p.off_a2 : p.off_a1) + (size_t)r * n_out;
  for (int i = t; i < n_in; i += 256) sx[i] = in[i];
  for (int i = t; i < n_out; i += 256) {
    const int m = A[i], w_ = i % win, pi = w_ / Sp, pj = w_ - pi * Sp;
    sg[i] = m == kDead ? 0.f : g[i];
    // offset of the window's maximum inside an input plane (a dead window contributes 0 x its corner)
    sa[i] = (2 * pi + (m == kDead ? 0 : (m >> 1))) * Sin + 2 * pj + (m == kDead ? 0 : (m & 1));
  }
  __syncthreads();
  float* out = wsp<float>(d, layer ? p.off_grow2 : p.off_grow1) + (size_t)r * (nW + Cout);
  for (int e = t; e < nW + Cout; e += 256) {
    float acc = 0.f;
    if (e < nW) {
      const int co = e % Cout, q = e / Cout, ci = q / (k * k), u = (q / k) % k, v = q % k;
      const float* x0 = sx + (ci * Sin + u) * Sin + v;
      const float* gg = sg + co * win;
      const int* aa = sa + co * win;
      for (int w_ = 0; w_ < win; ++w_) acc = fmaf(x0[aa[w_]], gg[w_], acc);
    } else {
      const float* gg = sg + (e - nW) * win;
      for (int w_ = 0; w_ < win; ++w_) acc += gg[w_];
    }
    out[e] = acc;
  }
}

// Local steps: a convolution parameter's shares of the upload's own rows (blockIdx.y = upload), added in row
// order; the upload's private model takes the step (Eq. 2; the dense parameters took theirs already).
__device__ __forceinline__ float conv_rows_sum(const CnnDev& d, size_t e, int a) {
  const CnnPlan& p = d.p;
  const int layer = e >= p.w_off[1] ? 1 : 0;
  const size_t n = (layer ? p.w_off[2] : p.w_off[1]) - p.w_off[layer];
  const float* G = wsp<const float>(d, layer ? p.off_grow2 : p.off_grow1) + (size_t)a * p.B * n + (e - p.w_off[layer]);
  float sum = 0.f;
  int r = 0;
  for (; r + 8 <= p.B; r += 8) {
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = G[(size_t)(r + q) * n];
#pragma unroll
    for (int q = 0; q < 8; ++q) sum += v[q];
  }
  for (; r < p.B; ++r) sum += G[(size_t)r * n];
  return sum;
}
__global__ __launch_bounds__(256) void cnn_conv_step_kernel(CnnDev d, RoundDesc rd) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int a = blockIdx.y;
  if (e >= d.p.w_off[2]) return;
  wsp<float>(d, d.p.off_priv)[(size_t)a * d.p.slot_stride + e] = slot_of(d, rd, a)[e] - conv_rows_sum(d, e, a);
}

// U = 1: Eq. 3, w^{t+1} = w^t - the uploads' shares added in arrival order.  The first conv_blocks workgroups
// take 32 convolution parameters each, eight groups of 32 threads adding the rows' shares of an upload
// in row order; the others a dense parameter per thread, its shares in the uploads' slots of G.
__global__ __launch_bounds__(256) void cnn_combine_kernel(CnnDev d, RoundDesc rd, int conv_blocks) {
  __shared__ float s_up[ABS_MAX_WORKERS * 32];
  const CnnPlan& p = d.p;
  const float* cur = wsp<const float>(d, p.off_ring) + (size_t)rd.slot_cur * p.slot_stride;
  float* nxt = wsp<float>(d, p.off_ring) + (size_t)rd.slot_next * p.slot_stride;
  const int t = threadIdx.x;
  if ((int)blockIdx.x < conv_blocks) {
    const size_t e = (size_t)blockIdx.x * 32 + (t & 31);
    const bool ok = e < p.w_off[2];
    for (int a = t >> 5; a < rd.K; a += 8) s_up[a * 32 + (t & 31)] = ok ? conv_rows_sum(d, e, a) : 0.f;
    __syncthreads();
    if (t < 32 && ok) {
      float sum = 0.f;
      for (int a = 0; a < rd.K; ++a) sum += s_up[a * 32 + t];
      nxt[e] = cur[e] - sum;
    }
    return;
  }
  const size_t e = p.w_off[2] + (size_t)((int)blockIdx.x - conv_blocks) * 256 + t;
  if (e >= p.P) return;
  const float* G = wsp<const float>(d, p.off_priv) + e;
  float sum = 0.f;
  int a = 0;
  for (; a + 4 <= rd.K; a += 4) {
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = G[(size_t)(a + q) * p.slot_stride];
#pragma unroll
    for (int q = 0; q < 4; ++q) sum += v[q];
  }
  for (; a < rd.K; ++a) sum += G[(size_t)a * p.slot_stride];
  nxt[e] = cur[e] - sum;
}

// Eq. 3 after U local steps: w^{t+1} = w^t - (1/K) sum_a (w^{t - tau_a} - w_a^U), uploads in arrival
// order; the first workgroup publishes the uploads' mean local losses.
__global__ __launch_bounds__(256) void cnn_delta_update_kernel(CnnDev d, RoundDesc rd, LossMailbox* mailbox) {
  const CnnPlan& p = d.p;
  if (blockIdx.x == 0 && mailbox && (int)threadIdx.x < rd.K)
    post_loss(mailbox, threadIdx.x, wsp<const float>(d, p.off_lossbuf)[threadIdx.x], rd.stamp);
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= p.P) return;
  const float* ring = wsp<const float>(d, p.off_ring);
  const float* priv = wsp<const float>(d, p.off_priv);
  float sum = 0.f;
  for (int a = 0; a < rd.K; ++a)
    sum += ring[(size_t)rd.w[a].slot * p.slot_stride + e] - priv[(size_t)a * p.slot_stride + e];
  wsp<float>(d, p.off_ring)[(size_t)rd.slot_next * p.slot_stride + e] =
      ring[(size_t)rd.slot_cur * p.slot_stride + e] - sum / (float)rd.K;
}

size_t conv_fwd_lds(const CnnPlan& p, int layer) {
  const int Cin = layer ? p.C1 : p.C0, Cout = layer ? p.C2 : p.C1, Sin = layer ? p.S1 : p.S;
  return ((size_t)Cin * Sin * Sin + (size_t)Cin * p.k * p.k * Cout + Cout) * 4;
}
// (what decides whether a shape is accepted: 8 rows' values of the dense stack)
size_t dense_lds(const CnnPlan& p) { return (size_t)8 * (p.F0 + 2 * p.F1 + 2 * p.F2 + p.C) * 4; }
size_t dense_group_lds(const CnnPlan& p, int G, int nt) { return ((size_t)G * (p.F0 + 2 * p.F1 + 2 * p.F2 + p.C) + (size_t)nt * G) * 4; }
constexpr size_t kMaxLds = 150 * 1024;
bool bwd_fused(const CnnPlan& p) { return (size_t)bwd_lds(p).total * 4 <= kMaxLds; }
// Threads of a workgroup that has a stacked row to itself.  While a CU has two rows at most, 1024: what counts is how long
// one row takes.  With more rows to do, as few as still fill a CU with the workgroups that its LDS holds: small
// stages are mostly barriers and idle wavefronts at 1024 (8192 rows of 1 x 18 x 18, 4-8 channels: forward 81 us,
// backward 216; with 256 threads 33 and 76; of 3 x 32 x 32, 6-16: 278 -> 204 with 256, 831 -> 669 with 512 and 979 with
// 256; 32-32 channels: forward 655, with 512 threads 710).
int row_threads(int rows, size_t lds, bool with_512) {
  const size_t per_cu = (size_t)160 * 1024 / lds;
  return rows <= 512 ? 1024 : per_cu >= 5 ? 256 : with_512 && per_cu >= 2 ? 512 : 1024;
}
size_t conv_wgrad_lds(const CnnPlan& p, int layer) {
  const int Cin = layer ? p.C1 : p.C0, Cout = layer ? p.C2 : p.C1, Sin = layer ? p.S1 : p.S, Sp = layer ? p.S2 : p.S1;
  return ((size_t)Cin * Sin * Sin + 2 * (size_t)Cout * Sp * Sp) * 4;
}
size_t conv2_bwd_lds(const CnnPlan& p) {
  const size_t Cp = (size_t)((p.C2 + 3) & ~3);
  return (Cp * 4 * p.S2 * p.S2 + (size_t)p.C1 * p.k * p.k * Cp) * 4;
}

void launch_conv_fwd(const CnnDev& d, const RoundDesc& rd, int rows, hipStream_t s) {
  const CnnPlan& p = d.p;
  const size_t fused = (size_t)fwd_lds(p).total * 4;
  if (fused <= kMaxLds) {
#define ABS_FWD(NT)                                                                              \
    switch (p.k) {                                                                               \
      case 3: cnn_fwd_kernel<3, NT><<<dim3(rows), dim3(NT), fused, s>>>(d, rd); break;           \
      case 5: cnn_fwd_kernel<5, NT><<<dim3(rows), dim3(NT), fused, s>>>(d, rd); break;           \
      default: cnn_fwd_kernel<0, NT><<<dim3(rows), dim3(NT), fused, s>>>(d, rd);                 \
    }
    if (row_threads(rows, fused, false) == 256) { ABS_FWD(256) } else { ABS_FWD(1024) }
#undef ABS_FWD
    return;
  }
  // (both convolutions' filters and maps do not fit the LDS together)
  for (int layer = 0; layer < 2; ++layer) {
    const size_t lds = conv_fwd_lds(p, layer);
    switch (p.k) {
      case 3: cnn_conv_pool_fwd_kernel<3><<<dim3(rows), dim3(256), lds, s>>>(d, rd, layer); break;
      case 5: cnn_conv_pool_fwd_kernel<5><<<dim3(rows), dim3(256), lds, s>>>(d, rd, layer); break;
      default: cnn_conv_pool_fwd_kernel<0><<<dim3(rows), dim3(256), lds, s>>>(d, rd, layer);
    }
  }
}

// Rows per workgroup of the dense stack: few while there are CUs without a workgroup (160 rows: 23 us one by one,
// 27 in twos, 34 in fours; every group fetches all dense weights from the L2), and with groups of 8 rows for most CUs
// the form without exchanges, earlier where the sums are short (400-120-84-10, us in fours / eights: 640 rows 34 / 56,
// 2048 64 / 56, 8192 197 / 84; 1152-256-128-10: 86 / 146, 168 / 150, 656 / 401; 72-40-24-10: 20 / 20, 36 / 20, 87 / 23).
void launch_dense(const CnnDev& d, const RoundDesc& rd, int uploads, hipStream_t s, float* eval_loss, float* eval_hit) {
  const CnnPlan& p = d.p;
  auto groups = [&](int G) { return uploads * ((p.B + G - 1) / G); };
#define ABS_DENSE(G, NT, COLS) \
  cnn_dense_kernel<G, NT, COLS><<<dim3(groups(G)), dim3(NT), dense_group_lds(p, G, COLS ? 0 : NT), s>>>(d, rd, eval_loss, eval_hit)
  if (groups(8) >= (p.F0 + p.F1 + p.F2 <= 150 ? 80 : 192)) ABS_DENSE(8, 256, true);
  else if (groups(1) <= 256) ABS_DENSE(1, 1024, false);
  else if (groups(2) <= 256) ABS_DENSE(2, 1024, false);
  else                       ABS_DENSE(4, 1024, false);
#undef ABS_DENSE
}

CnnDev dev_of(const CnnArgs& a) {
  CnnDev d{};
  d.p = a.plan; d.ws = a.ws; d.X = a.X; d.y = a.y;
  d.shard_rows = a.shard_rows; d.batch_key = a.batch_key;
  d.fixed_slot = -1; d.row0 = 0; d.n_rows = 0;
  d.step = -1; d.U = 1;
  return d;
}

}  // namespace

bool cnn_plan(const abs_config& c, CnnPlan& p, const char** why) {
  auto bad = [&](const char* m) { if (why) *why = m; return false; };
  if (c.n_layers != 5) return bad("CNN: n_layers must be 5 (two convolutional + three dense layers)");
  p.C1 = c.dims[1]; p.C2 = c.dims[2]; p.F1 = c.dims[3]; p.F2 = c.dims[4]; p.C = c.dims[5];
  p.C0 = c.dims[6]; p.k = c.dims[7];
  if (p.C0 < 1 || p.C0 > 4 || p.k < 1 || p.k > 7) return bad("CNN: 1 <= C0 <= 4, 1 <= k <= 7");
  if (c.dims[0] < 1 || c.dims[0] % p.C0) return bad("CNN: dims[0] must be C0 * S * S");
  int S = 1;
  while (S * S < c.dims[0] / p.C0) ++S;
  if (S * S * p.C0 != c.dims[0] || S > 64) return bad("CNN: dims[0] must be C0 * S * S with S <= 64");
  p.S = S;
  const int S1c = S - p.k + 1;
  if (S1c < 2 || S1c % 2) return bad("CNN: S - k + 1 must be even and positive");
  p.S1 = S1c / 2;
  const int S2c = p.S1 - p.k + 1;
  if (S2c < 2 || S2c % 2) return bad("CNN: S1 - k + 1 must be even and positive");
  p.S2 = S2c / 2;
  p.F0 = p.C2 * p.S2 * p.S2;
  if (p.C1 < 1 || p.C1 > kMaxCout || p.C2 < 1 || p.C2 > kMaxCout) return bad("CNN: 1 <= C1, C2 <= 32");
  if (p.F1 < 1 || p.F1 > 1024 || p.F2 < 1 || p.F2 > 1024 || p.C < 2 || p.C > 64) return bad("CNN: dense widths out of range");
  if (c.x_dtype != ABS_X_FP32) return bad("CNN: X must be fp32");
  p.B = c.B; p.N = c.N; p.R = c.tau_cap + 3;
  if (conv_fwd_lds(p, 0) > 150 * 1024 || conv_fwd_lds(p, 1) > 150 * 1024 || dense_lds(p) > 150 * 1024 ||
      conv2_bwd_lds(p) > 150 * 1024 || conv_wgrad_lds(p, 0) > 150 * 1024 || conv_wgrad_lds(p, 1) > 150 * 1024)
    return bad("CNN: a stage does not fit the LDS (smaller B, image or layers)");
  const int kk = p.k * p.k;
  const int rows[5] = {p.C0 * kk, p.C1 * kk, p.F0, p.F1, p.F2}, cols[5] = {p.C1, p.C2, p.F1, p.F2, p.C};
  size_t o = 0;
  for (int l = 0; l < 5; ++l) {
    p.w_off[l] = o; o += (size_t)rows[l] * cols[l];
    p.b_off[l] = o; o += (size_t)cols[l];
  }
  p.P = o;
  p.slot_stride = (o + 63) / 64 * 64;
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  const size_t Rm = (size_t)p.N * p.B, n1 = (size_t)p.C1 * p.S1 * p.S1;
  size_t off = 0;
  p.off_ring = off;    off = up(off + (size_t)p.R * p.slot_stride * 4);
  p.off_rowidx = off;  off = up(off + Rm * 4);
  p.off_label = off;   off = up(off + Rm * 4);
  p.off_p1 = off;      off = up(off + Rm * n1 * 4);
  p.off_a1 = off;      off = up(off + Rm * n1);
  p.off_p2 = off;      off = up(off + Rm * p.F0 * 4);
  p.off_a2 = off;      off = up(off + Rm * p.F0);
  p.off_h1 = off;      off = up(off + Rm * p.F1 * 4);
  p.off_h2 = off;      off = up(off + Rm * p.F2 * 4);
  p.off_dz1 = off;     off = up(off + Rm * p.F1 * 4);
  p.off_dz2 = off;     off = up(off + Rm * p.F2 * 4);
  p.off_dz3 = off;     off = up(off + Rm * p.C * 4);
  p.off_dp2 = off;     off = up(off + Rm * p.F0 * 4);
  // (the fused backward half keeps this gradient in LDS)
  p.off_dp1 = off;     if (!bwd_fused(p)) off = up(off + Rm * n1 * 4);
  p.off_lossbuf = off; off = up(off + (size_t)p.N * 4);
  p.off_rowloss = off; off = up(off + Rm * 4);
  p.U = c.U < 1 ? 1 : c.U;
  p.off_priv = off;    off = up(off + (size_t)p.N * p.slot_stride * 4);
  p.off_grow1 = off;   off = up(off + Rm * (p.w_off[1] - p.w_off[0]) * 4);
  p.off_grow2 = off;   off = up(off + Rm * (p.w_off[2] - p.w_off[1]) * 4);
  p.off_eval = off;    off = up(off + eval_scratch_bytes(Rm));
  p.total = off;
  return true;
}

hipError_t launch_cnn_round(const CnnArgs& a, const RoundDesc& rd, hipStream_t s, LaunchHook* hook) {
  const CnnPlan& p = a.plan;
  CnnDev d = dev_of(a);
  const int rows = rd.K * p.B;
  d.n_rows = rows;
  d.U = p.U;
  const bool local = p.U > 1;
  const double ar = (double)rows, kk = (double)p.k * p.k;
  const double f1 = 2.0 * ar * p.C1 * 4.0 * p.S1 * p.S1 * p.C0 * kk, f2 = 2.0 * ar * p.C2 * 4.0 * p.S2 * p.S2 * p.C1 * kk;
  const double fd = 2.0 * ar * ((double)p.F0 * p.F1 + (double)p.F1 * p.F2 + (double)p.F2 * p.C);
  const double n1 = (double)p.C1 * p.S1 * p.S1;
  const long n_dense = (long)p.F0 * p.F1 + p.F1 + (long)p.F1 * p.F2 + p.F2 + (long)p.F2 * p.C + p.C;
  for (int step = 0; step < p.U; ++step) {
    d.step = local ? step : -1;
    hook->begin(KK_CNN_CONV_FWD, f1 + f2, ar * 4.0 * (p.C0 * (double)p.S * p.S + 2.0 * n1 + p.F0));
    launch_conv_fwd(d, rd, rows, s);
    hook->end(KK_CNN_CONV_FWD);
    hook->begin(KK_CNN_DENSE, 2.0 * fd, ar * 4.0 * (2.0 * p.F0 + 2.0 * p.F1 + 2.0 * p.F2 + p.C));
    launch_dense(d, rd, rd.K, s, nullptr, nullptr);
    hook->end(KK_CNN_DENSE);
    // (a private model is stepped in place only where nothing reads it any more: the dense layers here, which the
    // convolutions' backward pass does not read, the filters in the launch behind it)
    const size_t fused = (size_t)bwd_lds(p).total * 4;
    const unsigned dense_blocks = (unsigned)(rd.K * dense_wgrad_blocks(p));
    LossMailbox* box = local ? nullptr : a.mailbox;
    if (bwd_fused(p)) {
      hook->begin(KK_CNN_CONV_BWD, 2.0 * ar * n1 * kk * p.C2 + fd + (f1 + f2) / 4.0,
                  ar * 4.0 * (p.C0 * (double)p.S * p.S + 3.0 * n1 + 3.0 * p.F0 + 2.0 * p.F1 + 2.0 * p.F2 + p.C) + (double)n_dense * 8.0);
      const dim3 grid(rows + dense_blocks);
#define ABS_BWD(NT)                                                                              \
      switch (p.k) {                                                                             \
        case 3: cnn_bwd_kernel<3, NT><<<grid, dim3(NT), fused, s>>>(d, rd, rows, box); break;    \
        case 5: cnn_bwd_kernel<5, NT><<<grid, dim3(NT), fused, s>>>(d, rd, rows, box); break;    \
        default: cnn_bwd_kernel<0, NT><<<grid, dim3(NT), fused, s>>>(d, rd, rows, box);          \
      }
      const int nt = row_threads(rows, fused, true);
      if (nt == 256) { ABS_BWD(256) } else if (nt == 512) { ABS_BWD(512) } else { ABS_BWD(1024) }
#undef ABS_BWD
      hook->end(KK_CNN_CONV_BWD);
    } else {
      hook->begin(KK_CNN_CONV_BWD, 2.0 * ar * n1 * kk * p.C2, ar * 4.0 * (p.F0 + n1));
      switch (p.k) {
        case 3: cnn_conv2_bwd_kernel<3><<<dim3(rows), dim3(256), conv2_bwd_lds(p), s>>>(d, rd); break;
        case 5: cnn_conv2_bwd_kernel<5><<<dim3(rows), dim3(256), conv2_bwd_lds(p), s>>>(d, rd); break;
        default: cnn_conv2_bwd_kernel<0><<<dim3(rows), dim3(256), conv2_bwd_lds(p), s>>>(d, rd);
      }
      hook->end(KK_CNN_CONV_BWD);
      hook->begin(KK_CNN_CONV_WGRAD, (f1 + f2) / 4.0, ar * 4.0 * (p.C0 * (double)p.S * p.S + 2.0 * n1 + p.F0));
      cnn_conv_wgrad_rows_kernel<<<dim3(rows), dim3(256), conv_wgrad_lds(p, 1), s>>>(d, 1);
      cnn_conv_wgrad_rows_kernel<<<dim3(rows), dim3(256), conv_wgrad_lds(p, 0), s>>>(d, 0);
      hook->end(KK_CNN_CONV_WGRAD);
      hook->begin(KK_CNN_DENSE_WGRAD, fd, (double)n_dense * 8.0 + ar * 4.0 * (p.F0 + 2.0 * p.F1 + 2.0 * p.F2 + p.C));
      cnn_dense_wgrad_kernel<<<dim3(dense_blocks), dim3(1024), 0, s>>>(d, rd, box);
      hook->end(KK_CNN_DENSE_WGRAD);
    }
    hook->begin(KK_CNN_COMBINE, (double)p.P * rd.K, 4.0 * (ar * (double)p.w_off[2] + (double)rd.K * n_dense + 2.0 * p.P));
    if (local) {
      cnn_conv_step_kernel<<<dim3((unsigned)((p.w_off[2] + 255) / 256), (unsigned)rd.K), dim3(256), 0, s>>>(d, rd);
    } else {
      const int conv_blocks = (int)((p.w_off[2] + 31) / 32);
      cnn_combine_kernel<<<dim3((unsigned)(conv_blocks + (p.P - p.w_off[2] + 255) / 256)), dim3(256), 0, s>>>(d, rd, conv_blocks);
    }
    hook->end(KK_CNN_COMBINE);
  }
  if (local) {
    hook->begin(KK_DELTA_UPDATE, (double)p.P * rd.K, (double)p.P * 4.0 * (2.0 * rd.K + 2.0));
    cnn_delta_update_kernel<<<dim3((unsigned)((p.P + 255) / 256)), dim3(256), 0, s>>>(d, rd, a.mailbox);
    hook->end(KK_DELTA_UPDATE);
  }
  return hipGetLastError();
}

hipError_t launch_cnn_eval(const CnnArgs& a, uint32_t slot, const EvalArgs& e, hipStream_t s, LaunchHook* hook) {
  const CnnPlan& p = a.plan;
  RoundDesc rd{};
  hipError_t err = launch_eval_clear(e, s);
  const int64_t pass = (int64_t)p.N * p.B;
  for (int64_t row0 = 0; row0 < e.n_rows && err == hipSuccess; row0 += pass) {
    const int n = (int)(e.n_rows - row0 < pass ? e.n_rows - row0 : pass);
    CnnDev d = dev_of(a);
    d.X = (const float*)e.X; d.y = (const int32_t*)e.y;
    d.fixed_slot = (int)slot; d.row0 = row0; d.n_rows = n;
    hook->begin(KK_EVAL, 0.0, 4.0 * n * p.C0 * p.S * p.S);
    launch_conv_fwd(d, rd, n, s);
    launch_dense(d, rd, (n + p.B - 1) / p.B, s, e.rowloss, e.correct);
    hook->end(KK_EVAL);
    err = hipGetLastError();
    if (err == hipSuccess) err = launch_eval_reduce(e, n, s, hook);
  }
  return err;
}

hipError_t cnn_prepare() {
  // stages whose LDS need exceeds the default limit must opt in once per process
  static hipError_t done = [] {
    const void* fns[] = {(const void*)cnn_fwd_kernel<0, 256>, (const void*)cnn_fwd_kernel<3, 256>, (const void*)cnn_fwd_kernel<5, 256>,
                         (const void*)cnn_fwd_kernel<0, 1024>, (const void*)cnn_fwd_kernel<3, 1024>, (const void*)cnn_fwd_kernel<5, 1024>,
                         (const void*)cnn_conv_pool_fwd_kernel<0>, (const void*)cnn_conv_pool_fwd_kernel<3>, (const void*)cnn_conv_pool_fwd_kernel<5>,
                         (const void*)cnn_dense_kernel<1, 1024, false>, (const void*)cnn_dense_kernel<2, 1024, false>,
                         (const void*)cnn_dense_kernel<4, 1024, false>, (const void*)cnn_dense_kernel<8, 256, true>,
                         (const void*)cnn_bwd_kernel<0, 256>, (const void*)cnn_bwd_kernel<3, 256>, (const void*)cnn_bwd_kernel<5, 256>,
                         (const void*)cnn_bwd_kernel<0, 512>, (const void*)cnn_bwd_kernel<3, 512>, (const void*)cnn_bwd_kernel<5, 512>,
                         (const void*)cnn_bwd_kernel<0, 1024>, (const void*)cnn_bwd_kernel<3, 1024>, (const void*)cnn_bwd_kernel<5, 1024>,
                         (const void*)cnn_conv2_bwd_kernel<0>, (const void*)cnn_conv2_bwd_kernel<3>, (const void*)cnn_conv2_bwd_kernel<5>,
                         (const void*)cnn_conv_wgrad_rows_kernel};
    hipError_t e = hipSuccess;
    for (const void* f : fns)
      if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
    return e;
  }();
  return done;
}

}  // namespace abs_impl

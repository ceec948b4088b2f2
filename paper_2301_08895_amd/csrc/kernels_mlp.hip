// MLP rounds: bf16 operands on the matrix cores (MFMA 16x16x32 in the large-tile kernel, 32x32x16
// in the others), fp32 accumulation,
// fp32 master weights.
//
// The K^t uploads of a round are stacked into one batch of K^t * Bp rows (Bp = B padded
// to the 128-row tile, so a row tile never straddles two uploads).  Forward and
// input-gradient products are grouped GEMMs: each 128-row tile multiplies with the bf16
// copy of the model version its upload computed at (Eq. 2 at the stale model
// w^{t - tau_k}).  The weight gradient and the K-of-N reduction of Eq. 3 are ONE
// contraction over all stacked rows, G_l = H_{l-1}^T dZ_l: rows of dZ already carry their
// upload's coefficient c_k = eta_k / (K^t B), so per-upload gradients are never
// materialised.  The contraction is split along the rows into partial sums that are
// combined in a fixed order by the update kernel, which also writes w^{t+1} = w^t - G
// into the next ring slot together with its two bf16 copies.
//
// All three products have the form  C[m][n] = sum_k A[m][k] * Bt[n][k]  with both
// operands contiguous along k, so one main loop serves them:
//   forward    A = H_{l}      [rows][dp_l]      Bt = W_l^T  [dp_{l+1}][dp_l]   (per upload)
//   dgrad      A = dZ_{l+1}   [rows][dp_{l+1}]  Bt = W_l    [dp_l][dp_{l+1}]   (per upload)
//   wgrad      A = H_l^T      [dp_l][rows]      Bt = dZ_{l+1}^T [dp_{l+1}][rows]
// which is why activations and output gradients are stored in both orientations and
// the weights' bf16 copies in both orientations.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <string>

#include "kernels.h"

namespace abs_impl {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int TM = 128;   // rows of C per workgroup
constexpr int BK = 64;    // contraction elements per main-loop step
constexpr int kMaxSplit = 16;
// Row pitches of the bf16 operand arrays are the padded width plus this many elements (128 B):
// with a pitch that is a multiple of 4 KB the same 128-byte column of every row of a tile maps
// to one L2 channel, and all workgroups walk the k dimension in step.  The pad behind a row of a weight copy is
// also read as data: gathered rows fetch the 64 elements behind the first row where a k-step reaches beyond d_0, so
// it must be a k-step long and stays zero in every shadow slot (mlp_prepare clears them; mlp_step_kernel's tiles that are wider
// than the class width store zeros there, nothing else writes to it).
#ifndef ABS_PITCH_PAD
#define ABS_PITCH_PAD 64
#endif
constexpr int kPitchPad = ABS_PITCH_PAD;
static_assert(kPitchPad >= BK && kPitchPad % 8 == 0, "the pad of a row is a gathered k-step's zeros");
constexpr int kPartialPad = 32;         // the same for the fp32 weight-gradient partials (floats)

size_t round_up(size_t x, size_t m) { return (x + m - 1) / m * m; }

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  // round to nearest, ties to even (finite values)
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// 16-byte store that, on request, does not keep its line in the cache.  The activations and
// gradients of a large round are hundreds of megabytes that another kernel reads next; kept out of
// the L2 they no longer evict the operand panels the other workgroups of the XCD still share
// (a 32768 x 2048 x 2048 forward product 250 -> 230 us).  A small round's outputs fit the caches and
// are better left there for their reader (8192 rows: the products that follow got 4 % slower).
#ifndef ABS_STREAM_MIN_BYTES
#define ABS_STREAM_MIN_BYTES (64u << 20)
#endif
__device__ __forceinline__ void store16_stream(uint16_t* p, const uint4& v, bool stream) {
  // (written out by hand: when both forms of the store sit in the two arms of a branch the optimiser
  // merges them into one plain store)
  if (stream) asm volatile("global_store_dwordx4 %0, %1, off nt" : : "v"(p), "v"(u32x4_t{v.x, v.y, v.z, v.w}) : "memory");
  else        *(uint4*)p = v;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ------------------------------------------------------------------ gather + transpose of X
// XgT[k][m] = X[rowidx[m]][k]  (zero for k >= d0): the A operand of the first layer's
// weight-gradient contraction.  64 x 64 tiles through LDS.
__global__ __launch_bounds__(256) void mlp_gather_t_kernel(const uint16_t* X, int d0, const uint32_t* rowidx,
                                                          uint16_t* XgT, size_t ldt) {
  __shared__ uint16_t tile[64][72];
  const int m0 = blockIdx.x * 64, k0 = blockIdx.y * 64;
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = t + 256 * i;
    const int r = q >> 3, c = q & 7;
    const int k = k0 + c * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (k < d0) v = *(const uint4*)(X + (size_t)rowidx[m0 + r] * d0 + k);
    *(uint4*)&tile[r][c * 8] = v;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = t + 256 * i;
    const int kk = q >> 3, c = q & 7;      // output row kk, 8 consecutive m
    uint16_t v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = tile[c * 8 + j][kk];
    uint4 o;
    o.x = v[0] | ((uint32_t)v[1] << 16); o.y = v[2] | ((uint32_t)v[3] << 16);
    o.z = v[4] | ((uint32_t)v[5] << 16); o.w = v[6] | ((uint32_t)v[7] << 16);
    *(uint4*)(XgT + (size_t)(k0 + kk) * ldt + m0 + c * 8) = o;
  }
}

// The same by the last workgroups of the output-layer kernel's launch: it needs nothing but the drawn rows,
// and that launch's own workgroups (ce_rows()) leave CUs idle.  Blocks of 64 rows x 256 columns,
// all of a thread's loads in flight together.  The kernel's LDS lets a CU hold one workgroup (98, 131 or 147 KB for
// up to 64, 128 or 256 classes), so beyond kGatherRide blocks (two waves) the launch of its own is the faster one.
// Sum of a round's kernels, us, own launch / riding, by blocks and classes: 1000-520-C, 64 blocks 46 / 42 (10), 52 / 47
// (100), 60 / 55 (256), 512 blocks 84 / 80, 96 / 90, 101 / 95; 200-1024-C, 128 blocks 77 / 69, 83 / 84, 105 / 97; 3000-2048-C,
// 768 blocks 205 / 201, 217 / 216, 238 / 238, 1536 blocks 307 / 323, 321 / 323, 357 / 362.  With a second hidden layer
// the copy waits longer for its reader: 1000-1024-1024-10, 512 blocks 202 / 198, but 1000-2048-2048-10, 256 blocks 277 / 280,
// 512-1920-1920-50, 512 blocks 75 / 82 (the copy, the output layer and the first weight gradient).
// The 32-row form of that kernel leaves a CU room for a second workgroup up to 96 classes (up to 80 KB; 91 and 101 KB beyond):
// there 768 ride (3072-512-10, 768 blocks, a round 80 / 78.6 us, with split weight gradients 79 / 74; 3072-256-10, 384 blocks
// each way the same; six simulations side by side, 10 classes 410 / 411, 96 classes 417 / 418).  Beyond 96 classes 512 as above
// (3072-512-100, 768 blocks, 83.3 / 84.2, six side by side 451 / 483, 576 blocks 75.1 / 72.5 and 344 / 367; 3072-1024-100, 768
// blocks 106.8 / 106.3 and 560 / 606).
constexpr int kGatherRide = 512, kGatherRideFew = 768, kFewPairClasses = 96;
constexpr int kGatherPitch = 256 + 2;      // the 8 blocks of 8 rows a wavefront reads start 8 banks apart
struct GatherT {
  int blocks;                              // row blocks x column blocks that ride; 0: none
  const uint16_t* X; int d0, dp0;
  const uint32_t* rowidx;
  uint16_t* XgT; size_t ldt;
};
__device__ __forceinline__ void gather_t_block(const GatherT& a, int b, uint16_t* tile) {
  const int nk = (a.dp0 + 255) / 256;
  const int m0 = (b / nk) * 64, k0 = (b % nk) * 256;
  const int t = threadIdx.x;
  uint4 v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = (t >> 5) + 8 * i, k = k0 + (t & 31) * 8;
    v[i] = make_uint4(0, 0, 0, 0);
    if (k < a.d0) v[i] = *(const uint4*)(a.X + (size_t)a.rowidx[m0 + r] * a.d0 + k);     // d0 % 8 == 0
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    uint32_t* q = (uint32_t*)&tile[((t >> 5) + 8 * i) * kGatherPitch + (t & 31) * 8];
    q[0] = v[i].x; q[1] = v[i].y; q[2] = v[i].z; q[3] = v[i].w;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int kk = (t >> 3) + 32 * i, c = t & 7;      // output row kk, 8 consecutive m
    uint16_t h[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) h[j] = tile[(c * 8 + j) * kGatherPitch + kk];
    uint4 o;
    o.x = h[0] | ((uint32_t)h[1] << 16); o.y = h[2] | ((uint32_t)h[3] << 16);
    o.z = h[4] | ((uint32_t)h[5] << 16); o.w = h[6] | ((uint32_t)h[7] << 16);
    if (k0 + kk < a.dp0) *(uint4*)(a.XgT + (size_t)(k0 + kk) * a.ldt + m0 + c * 8) = o;
  }
}

// ------------------------------------------------------------------ Eq. 3 on a block of a weight matrix
// w^{t+1} = w^t - sum_z partial[z] (fixed order) for one weight matrix, written as fp32 into the next
// ring slot and as bf16 in both orientations into the next shadow slot.
struct TileUpdate {
  const float* partial; size_t split_stride; size_t ldp; int nsplit;
  const float* w_cur; float* w_next;   // [d_in][d_out] fp32, pitch d_out
  int d_in, d_out;
  uint16_t* wn; size_t ldwn;           // bf16 [dp_in][dp_out] (may be null)
  uint16_t* wt; size_t ldwt;           // bf16 [dp_out][dp_in]
  // sk_q > 0: the partials come from a weight-gradient launch that cut the contraction into equal
  // runs of sk_q k-steps across the 256 x 256 output tiles (see GemmArgs::sk_q); tile T then has as
  // many partials as runs touch its sk_ksteps k-steps, in slots 0 .. count - 1.
  int sk_q, sk_ksteps, sk_nt;
};
__device__ __forceinline__ int partial_count(const TileUpdate& u, int i0, int j0) {
  if (!u.sk_q) return u.nsplit;
  const int tile = (i0 >> 8) * u.sk_nt + (j0 >> 8);
  return ((tile + 1) * u.sk_ksteps - 1) / u.sk_q - tile * u.sk_ksteps / u.sk_q + 1;
}
// Tiled version for 16-byte aligned rows (d_out % 4 == 0).  One block of 64 rows x TJ columns at
// (i0, j0), by all NT threads of the workgroup (uniform call): a thread moves 4 consecutive columns at
// a time, TJ / 4 threads cover a row (TJ = 256: 1 KB of a model row per row of the tile, so that the
// rows of a tile - a whole number of 4 KB apart for the usual widths - do not all fall on one memory
// channel).  `tile` is 64 x (TJ + 2) bf16 of LDS: with a row pitch of 129 / 33 words the transposed
// copy's 8 blocks of 8 rows start 8 banks apart and no two lanes of a wavefront collide.
template <int NT, int TJ>
__device__ __forceinline__ void update_block64(const TileUpdate& u, int i0, int j0, uint16_t* tile) {
  constexpr int TPR = TJ / 4;            // threads per row
  constexpr int RPP = NT / TPR;          // rows per pass
  constexpr int NPASS = 64 / RPP;        // passes
  constexpr int PT = TJ + 2;             // pitch of the LDS tile
  static_assert(NPASS >= 2 && NPASS % 2 == 0, "two rows of a thread at a time");
  const int jq = ((int)threadIdx.x % TPR) * 4, ir = (int)threadIdx.x / TPR;
  const int nsplit = partial_count(u, i0, j0);
  // two of the thread's rows at a time, with the model row and up to 8 partials of both in
  // flight together (a partial beyond the 8th, rare, is fetched afterwards); summed in split order
#pragma unroll 1
  for (int r2 = 0; r2 < NPASS / 2; ++r2) {
    float4 wc[2], v[2][8];
    bool ok[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = i0 + ir + RPP * (2 * r2 + h), j = j0 + jq;
      ok[h] = i < u.d_in && j < u.d_out;
      if (ok[h]) {
        const float* pp = u.partial + (size_t)i * u.ldp + j;
        wc[h] = *(const float4*)(u.w_cur + (size_t)i * u.d_out + j);
#pragma unroll
        for (int z = 0; z < 8; ++z)
          if (z < nsplit) v[h][z] = *(const float4*)(pp + (size_t)z * u.split_stride);
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int il = ir + RPP * (2 * r2 + h), i = i0 + il, j = j0 + jq;
      uint2 hh = make_uint2(0, 0);
      if (ok[h]) {
        float4 G = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int z = 0; z < 8; ++z)
          if (z < nsplit) { G.x += v[h][z].x; G.y += v[h][z].y; G.z += v[h][z].z; G.w += v[h][z].w; }
        for (int z = 8; z < nsplit; ++z) {
          const float4 t = *(const float4*)(u.partial + (size_t)i * u.ldp + j + (size_t)z * u.split_stride);
          G.x += t.x; G.y += t.y; G.z += t.z; G.w += t.w;
        }
        float4 w = wc[h];
        w.x -= G.x; w.y -= G.y; w.z -= G.z; w.w -= G.w;
        *(float4*)(u.w_next + (size_t)i * u.d_out + j) = w;
        hh.x = f32_to_bf16(w.x) | ((uint32_t)f32_to_bf16(w.y) << 16);
        hh.y = f32_to_bf16(w.z) | ((uint32_t)f32_to_bf16(w.w) << 16);
        if (u.wn) *(uint2*)(u.wn + (size_t)i * u.ldwn + j) = hh;
      }
      *(uint32_t*)&tile[il * PT + jq] = hh.x;
      *(uint32_t*)&tile[il * PT + jq + 2] = hh.y;
    }
  }
  __syncthreads();
  // transposed bf16 copy: thread -> column j, 8 consecutive rows i (the padded pitch of wt makes
  // the 16-byte store safe; rows beyond d_in hold zeros, which is what the padding must be)
  for (int q = threadIdx.x; q < TJ * 8; q += NT) {
    const int jl = q >> 3, ib = (q & 7) * 8;
    const int j = j0 + jl;
    if (j < u.d_out) {
      uint16_t v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = tile[(ib + e) * PT + jl];
      uint4 o;
      o.x = v[0] | ((uint32_t)v[1] << 16); o.y = v[2] | ((uint32_t)v[3] << 16);
      o.z = v[4] | ((uint32_t)v[5] << 16); o.w = v[6] | ((uint32_t)v[7] << 16);
      *(uint4*)(u.wt + (size_t)j * u.ldwt + i0 + ib) = o;
    }
  }
}

// ------------------------------------------------------------------ the GEMM
enum { EPI_RELU = 0, EPI_LOGITS = 1, EPI_DGRAD = 2, EPI_WGRAD = 3 };

// ------------------------------------------------------------------ bias update
// b_j <- b_j - sum over the rows of dZ_l[.][j] (Eq. 2 / Eq. 3 for the biases).  The producers of
// dZ_l leave the column sums of every block of 64 rows (the output layer: ce_rows()); 16 threads per entry
// add them (partial row g, g + 16, ... each, then the 16 shares in order).  A block of 256 threads
// takes 16 consecutive entries of the concatenated bias vectors.
struct BiasCore {
  int L;
  int col_begin[ABS_MAX_LAYERS + 1];       // prefix of valid columns over the layers
  const float* colsum[ABS_MAX_LAYERS]; size_t ldcs[ABS_MAX_LAYERS];
  size_t b_off[ABS_MAX_LAYERS];
  const float* w_cur; float* w_next;
  int prow[ABS_MAX_LAYERS];                // row blocks of colsum[l] (per upload in the per-upload form)
};
// blk: which 16 entries; first_row_block(l): where the sum over layer l's row blocks starts; cur / nxt:
// the model read and written.  Threads 0 .. 255 of the workgroup work, all of them meet the barrier.
template <typename FirstRow>
__device__ __forceinline__ void bias_block(const BiasCore& a, int blk, FirstRow first_row_block, const float* cur,
                                           float* nxt, float* lds) {
  float (*s_part)[17] = (float (*)[17])lds;
  const int t = threadIdx.x, cl = t & 15, grp = (t >> 4) & 15;
  const int w = blk * 16 + cl;
  const int ncol = a.col_begin[a.L];
  float s = 0.f;
  int l = 0, j = 0;
  if (w < ncol && t < 256) {
    while (w >= a.col_begin[l + 1]) ++l;
    j = w - a.col_begin[l];
    const int prow = a.prow[l];
    const float* src = a.colsum[l] + (size_t)first_row_block(l) * a.ldcs[l] + j;
    int r = grp;
    for (; r + 48 < prow; r += 64) {         // four loads in flight
      const float v0 = src[(size_t)r * a.ldcs[l]], v1 = src[(size_t)(r + 16) * a.ldcs[l]];
      const float v2 = src[(size_t)(r + 32) * a.ldcs[l]], v3 = src[(size_t)(r + 48) * a.ldcs[l]];
      s += v0; s += v1; s += v2; s += v3;
    }
    for (; r < prow; r += 16) s += src[(size_t)r * a.ldcs[l]];
  }
  if (t < 256) s_part[grp][cl] = s;
  __syncthreads();
  if (t < 16 && w < ncol) {
    float sum = 0.f;
#pragma unroll
    for (int g = 0; g < 16; ++g) sum += s_part[g][cl];
    nxt[a.b_off[l] + j] = cur[a.b_off[l] + j] - sum;
  }
}

// Local SGD (Eq. 2) with more rows an upload than mlp_step_kernel takes (local_step_tiles): the weight gradient of one step of
// upload z, W_l of its private model and the two bf16 copies.  The contraction is not split (range z = the rows of upload z), so
// the accumulators hold the whole gradient and the epilogue takes the step itself: no partial is written and read back, and the
// update needs no launch (the bias update and the losses ride in this and in the input gradient's launch).
// `own`: the model is private copy z of `cur`, else ring slot rd.w[z].slot.
struct LocalUpdate {
  int own;
  const float* cur; float* next; size_t stride;      // fp32 [d_in][d_out] at the layer's place in a model; models `stride` apart
  uint16_t* wn; size_t ldwn; uint16_t* wt; size_t ldwt; size_t shadow_stride;   // bf16 copies of the private models (wn may be null)
  int d_in, d_out;
};

struct GemmArgs {
  const uint16_t* A;  size_t lda;     // [Mdim][lda], k contiguous
  const uint32_t* a_rowidx;           // GATHER: row m of A is A + a_rowidx[m] * lda
  int a_kvalid;                       // GATHER: k >= a_kvalid reads as zero
  const uint16_t* Bt; size_t ldb;     // [Ndim][ldb], k contiguous
  size_t bt_slot_stride;              // PER_UPLOAD: Bt += slot(upload of the row tile) * stride
  int rows_per_upload;                // Bp
  int by_upload;                      // PER_UPLOAD: the slot is the upload's position (private models) instead of its ring slot
  int ksteps_total;                   // BK-steps of the whole contraction
  int ksteps_per_split;               // BK-steps per blockIdx.z
  const float* bias; size_t bias_slot_stride; int n_valid;   // EPI_RELU / EPI_LOGITS
  uint16_t* out;  size_t ldo;         // bf16 [Mdim][ldo]   (may be null)
  uint16_t* outT; size_t ldoT;        // bf16 [Ndim][ldoT]  (may be null)
  float* outf;    size_t ldof;        // fp32 [Mdim][ldof]; EPI_WGRAD: + z * split_stride
  size_t split_stride;
  int mt, nt, nsplit, rows_per_xcd;   // tile grid (see the block -> tile mapping in the kernel)
  const uint16_t* maskT; size_t ldmaskT; // EPI_DGRAD: H_l^T [Ndim][ldmaskT]; the gradient passes where H_l > 0
  float* colsum; size_t ldcs;         // EPI_DGRAD: column sums of the bf16 results per block of 64 rows, [Mdim / 64][ldcs]
  // 256 x 256 tile kernel only: the ReLU mask as one bit per element in the kernel's own accumulator
  // order (16 bytes per lane and tile: [tile][wavefront][lane][4 words], word a / 2, bit (a & 1) 16 + 4 b + r
  // for the 16 x 16 block (a, b) of the wavefront's sub-tile and accumulator register r).
  // EPI_RELU writes it when set; EPI_DGRAD reads it instead of maskT when set.
  uint32_t* maskbits;
  // 256 x 256 tile kernel, bf16 outputs: store them without keeping their lines in the L2 (set by the
  // launcher for outputs much larger than the L2s: see store16_stream)
  int stream_out;
  // GATHER with gen_rows set: the kernel draws the minibatch rows itself (stacked row m = upload
  // m / rows_per_upload, sample m % rows_per_upload; Section II-A: independent uniform draws from the
  // worker's shard) instead of reading a_rowidx, and the workgroups of the first column tile leave
  // them, with their labels, in gen_rowidx / gen_label for the kernels that follow.
  int gen_rows;
  int gen_B;                          // samples per upload (rows beyond are padding: label -1)
  uint64_t gen_shard_rows, gen_batch_key;
  uint32_t gen_draw0;                 // first draw index of this step (local step u: u B)
  const int32_t* gen_y;
  uint32_t* gen_rowidx; int32_t* gen_label;
  // EPI_WGRAD on the 256 x 256 tile kernel with sk_q > 0: instead of nsplit equal row ranges per
  // output tile, the mt nt ksteps_total (tile, k-step) pairs, tile after tile, are cut into runs of
  // sk_q and workgroup w takes run w - a run may end in one tile and begin the next.  Every workgroup
  // then does the same number of k-steps whatever the tile count (96 tiles on 256 CUs: two splits
  // each leave a quarter of the CUs idle, runs of 48 k-steps none); a tile's partials are the pieces
  // of the runs that touch it, in order, slot = piece number.
  int sk_q;
  // EPI_WGRAD with pig_blocks > 0: the launch's first pig_blocks workgroups do not belong to this
  // product at all - each applies Eq. 3 to one 64 x pig_tj block of ANOTHER layer's weight matrix,
  // whose split partials the previous launch completed (pig_upd).  The update is bound by memory, the
  // product by the matrix cores, and a weight-gradient launch rarely has a whole number of waves of
  // tiles: sharing a launch lets the two overlap without streams, events or fences.
  int pig_blocks, pig_tj;
  TileUpdate pig_upd;
  // ... and its very last bias_blocks workgroups the round's bias update (every dZ_l and its column
  // sums are complete before the first weight-gradient launch).
  int bias_blocks;
  BiasCore bias_upd;
  // (local SGD, TAG 4 / 5: bias_per blocks for each upload, on the upload's own model as local_upd says)
  int bias_per;
  LocalUpdate local_upd;
  // EPI_DGRAD with pub_rowloss set: the first workgroup forms the uploads' mean minibatch losses
  // (sums of pub_nb row blocks each, left by the output-layer kernel) before it starts on its tile and
  // publishes them if pub_mailbox is set.  Local SGD: pub_lossacc carries the sum over the job's pub_U
  // steps, and what the last step publishes is the job's average local loss.
  LossMailbox* pub_mailbox; const float* pub_rowloss; int pub_nb; int pub_B;
  float* pub_lossacc; int pub_first, pub_U;
};

// Dataset row of stacked row m (and whether it carries a sample).
__device__ __forceinline__ uint32_t gen_row_of(const GemmArgs& g, const RoundDesc& rd, int m, bool* real) {
  const int up = m / g.rows_per_upload, b = m - up * g.rows_per_upload;
  const WorkerDesc w = rd.w[up];
  uint64_t row = (uint64_t)w.id * g.gen_shard_rows;
  *real = b < g.gen_B;
  if (b < g.gen_B) row += draw(job_key(g.gen_batch_key, w.id, w.job), g.gen_draw0 + (uint32_t)b) % g.gen_shard_rows;
  return (uint32_t)row;
}
__device__ __forceinline__ void gen_row_store(const GemmArgs& g, int m, uint32_t row, bool real) {
  g.gen_rowidx[m] = row;
  g.gen_label[m] = real ? g.gen_y[row] : -1;
}

// The uploads' mean minibatch losses (what each worker reports next to its gradient) into the
// mailbox: thread a < K adds the loss sums of upload a's row blocks in order.
__device__ __forceinline__ void publish_upload_losses(const GemmArgs& g, int K, uint32_t stamp) {
  const int up = threadIdx.x;
  if (up < K) {
    float sum = 0.f;
    for (int q = 0; q < g.pub_nb; ++q) sum += g.pub_rowloss[(size_t)up * g.pub_nb + q];
    float mean = sum / (float)g.pub_B;
    if (g.pub_lossacc) {
      if (!g.pub_first) mean += g.pub_lossacc[up];
      g.pub_lossacc[up] = mean;
      mean /= (float)g.pub_U;
    }
    if (g.pub_mailbox) post_loss(g.pub_mailbox, up, mean, stamp);
  }
}

// Block b of the bias blocks at the end of a weight-gradient launch: 16 bias entries, of the global model
// or (LOCAL) of upload b / bias_per's private one, over the row blocks of that upload.
template <bool LOCAL>
__device__ __forceinline__ void rider_bias(const GemmArgs& g, const RoundDesc& rd, int b, float* lds) {
  const BiasCore& u = g.bias_upd;
  if (!LOCAL) { bias_block(u, b, [](int) { return 0; }, u.w_cur, u.w_next, lds); return; }
  const int up = b / g.bias_per;
  const size_t from = g.local_upd.own ? (size_t)up : (size_t)rd.w[up].slot;
  bias_block(u, b - up * g.bias_per, [&](int l) { return up * u.prow[l]; }, u.w_cur + from * g.local_upd.stride,
             u.w_next + (size_t)up * g.local_upd.stride, lds);
}

// A piggybacked update block (see GemmArgs::pig_blocks): block b of the other layer's matrix, 64 rows
// x pig_tj columns, by the NT threads of this workgroup.  Blocks beyond the matrix (the count is
// rounded up to a multiple of 8 to keep the product's block -> XCD mapping) do nothing.
template <int NT, bool WIDE_OK>
__device__ __forceinline__ void piggy_update(const GemmArgs& g, int b, uint16_t* lds) {
  const TileUpdate& u = g.pig_upd;
  const int rows = (u.d_in + 63) / 64;
  if (WIDE_OK && g.pig_tj == 256) {
    const int nbx = (u.d_out + 255) / 256;
    if (b < nbx * rows) update_block64<NT, 256>(u, (b / nbx) * 64, (b % nbx) * 256, lds);
  } else {
    const int nbx = (u.d_out + 63) / 64;
    if (b < nbx * rows) update_block64<NT, 64>(u, (b / nbx) * 64, (b % nbx) * 64, lds);
  }
}

// A global -> LDS request, written out by hand: the compiler makes every LDS read that it cannot tell
// apart from a pending request of its own wait for all of them, and it cannot for the
// transposing read: a k-step would then start by waiting for the tile it has just requested.
// Requests issued this way are invisible to that bookkeeping; the loops' own counted waits and
// barriers order them against the reads.  The LDS base travels in m0, which the register
// allocator hands over through the "{m0}" constraint (it knows the register is written).
__device__ __forceinline__ void lds_dma16_raw(const uint16_t* gsrc, uint16_t* lds_block) {
  const uint32_t lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds_block);
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(gsrc), "{m0}"(lds)
               : "memory");
}

// ... to a byte offset in LDS (uniform: scalar arithmetic only, so that m0 is never written by a vector instruction
// right before the request, which needs more wait states than the one here), 16 or 4 bytes per lane.
__device__ __forceinline__ uint32_t lds_offset(const void* p) { return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p; }
__device__ __forceinline__ void lds_dma16_at(const uint16_t* gsrc, uint32_t lds) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(gsrc), "{m0}"(lds) : "memory");
}
__device__ __forceinline__ void lds_dma4_at(const uint32_t* gsrc, uint32_t lds) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dword %0, off" : : "v"(gsrc), "{m0}"(lds) : "memory");
}

// A ring's hand-over: at most N of this wavefront's requests are still on their way (the later stages'),
// its own LDS reads are done, and everybody has got here.
template <int N>
__device__ __forceinline__ void ring_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

// ------------------------------------------------------------------ the GEMM on tiles of 64 and 128
// What a round of few or narrow rows waits for is not arithmetic but the trip of a k-step's tiles from
// memory into LDS and, behind it, the fixed cost of a step (barrier, first fragment reads).  So
//  * tiles travel global -> LDS by DMA through a ring of RING k-steps, RING - 1 of them on
//    their way at any time (one wait, one barrier and one batch of requests per stage);
//  * a wavefront owns a 64 x 64 sub-tile (2 x 2 blocks of MFMA 32x32x16, the fewest fragment bytes per
//    flop that 64 accumulator registers allow), and the KG wavefront groups of a workgroup (1, 2 or 4) share the
//    CONTRACTION of a step, not its columns: two wavefronts per SIMD cover each other's fragment reads
//    without staging a byte more.  At the end the groups exchange blocks through LDS, every group adds
//    and finishes OWN of its sub-tile's four blocks (always in group order);
//  * both orientations of a bf16 result leave through LDS as 16-byte pieces.
// Measured against the same products with one wavefront group, a ring that every barrier drained
// (__syncthreads waits for all of a wavefront's requests when the compiler knows of them) and 2-byte
// row-major stores: first-layer forward 1024 x 512 x 3072 32.0 -> 18.3 us, 4096 x 1024 x 3072 55 -> 39,
// hidden forward / input gradient 4096 x 1024 x 1024 22 -> 18.5.  What bounds it now: a CU draws 23-32 bytes
// per clock from beyond its L1 whatever the ring's depth, about 30 KB in flight over the latency of a miss.
// A tile row is 128 bytes; its 16-byte chunk c is stored at position c ^ ((row >> 1) & 7): the 16 lanes
// that one cycle of a 128-bit LDS read serves (16 consecutive rows of a fragment) then cover all 64 banks.
template <int T, int KG_>
struct TileCfg {
  static constexpr int WS = T / 64;                      // 64 x 64 sub-tiles along each side
  static constexpr int KG = KG_;                         // wavefront groups along the contraction
  static constexpr int NW = WS * WS * KG, NT = NW * 64;  // wavefronts, threads
  static constexpr int OWN = 4 / KG;                     // blocks a wavefront finishes
  static constexpr int kStage = 2 * T * BK;              // elements of a k-step's tiles
  static constexpr int kRed = WS * WS * 4 * (KG - 1) * 1024 * 2;   // exchanged blocks (in elements of 2 bytes)
  static constexpr int kPitch = T + 8;                   // of the staged results
  static constexpr int kOut = 2 * T * kPitch + (T / 32) * T * 2;   // both orientations, column sums per 32 rows
};

template <int T, int KGS, int EPI, bool GATHER, bool PER_UPLOAD, int TAG, int RING>
__global__ __launch_bounds__((TileCfg<T, KGS>::NT), 2) void mlp_tile_kernel(GemmArgs g, RoundDesc rd) {
  using Cfg = TileCfg<T, KGS>;
  constexpr int NW = Cfg::NW, NT = Cfg::NT, KG = Cfg::KG, OWN = Cfg::OWN;
  constexpr bool kLocal = EPI == EPI_WGRAD && TAG >= 4;  // local SGD: the epilogue takes the step (LocalUpdate)
  constexpr bool kStageT = (EPI == EPI_RELU || EPI == EPI_DGRAD || kLocal);
  constexpr int kEpi = Cfg::kRed + (kStageT ? Cfg::kOut : 0);
  constexpr int kSmem = RING * Cfg::kStage > kEpi ? RING * Cfg::kStage : kEpi;
  static_assert(kSmem * 2 <= 160 * 1024 - 1024, "LDS budget");
  __shared__ __attribute__((aligned(16))) uint16_t smem[kSmem];
  __shared__ uint32_t s_row[GATHER ? T : 1];

  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int kg = wave / (Cfg::WS * Cfg::WS), wsub = wave % (Cfg::WS * Cfg::WS);
  const int wm = wsub / Cfg::WS, wn = wsub % Cfg::WS;
  const int bx = blockIdx.x;
  if (EPI == EPI_WGRAD && (g.pig_blocks | g.bias_blocks)) {
    // The update's blocks come last in the grid: they take the CUs that the product's last wave of
    // tiles leaves idle and the tail.  (Dealt out evenly between the tiles they slowed every tile
    // down: 260 -> 400 us for the hidden layer's product at K = 128.)  Behind them the bias blocks.
    const int own = (int)gridDim.x - g.pig_blocks - g.bias_blocks;
    if (bx >= own + g.pig_blocks) {
      rider_bias<kLocal>(g, rd, bx - own - g.pig_blocks, (float*)smem);
      return;
    }
    if (bx >= own) { piggy_update<NT, false>(g, bx - own, smem); return; }
  }
  // Block -> tile mapping.  Workgroups are handed to the 8 XCDs round-robin and every XCD has
  // its own L2, so block b works for XCD b % 8.  The (split, row-tile) pairs are cut into 8
  // contiguous ranges, one per XCD, and inside a range consecutive blocks sweep the column
  // tiles of one row tile: the blocks resident on an XCD then share their A rows (and, for
  // neighbouring row tiles of the same upload, their B rows) through that XCD's L2.
  const int xcd = bx & 7, jx = bx >> 3;
  const int trow = xcd * g.rows_per_xcd + jx / g.nt;
  if (trow >= g.mt * g.nsplit) return;
  const int zsplit = trow / g.mt;
  const int m0 = (trow - zsplit * g.mt) * T, n0 = (jx % g.nt) * T;
  const int ks0 = zsplit * g.ksteps_per_split;
  const int ks1 = min(g.ksteps_total, ks0 + g.ksteps_per_split);

  if (EPI == EPI_DGRAD && g.pub_rowloss && blockIdx.x == 0) publish_upload_losses(g, rd.K, rd.stamp);

  const uint16_t* Bt = g.Bt;
  uint32_t slot = 0;
  if (PER_UPLOAD) {
    slot = g.by_upload ? (uint32_t)(m0 / g.rows_per_upload) : rd.w[m0 / g.rows_per_upload].slot;
    Bt += (size_t)slot * g.bt_slot_stride;
  }

  // Requests: one fills 8 rows of 128 bytes; wavefront w takes rows 8 (w + NW i) .. of A and of B, lane l
  // row (l >> 3) of them at chunk position l & 7, fetching logical chunk (l & 7) ^ ((row >> 1) & 7), and
  // (row >> 1) & 7 is (l >> 4) + 4 (w & 1).
  constexpr int NI = T / (8 * NW);
  const int c8 = ((lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7)) * 8;
  const int rq = 8 * wave + (lane >> 3);
  const uint16_t* pa[NI]; const uint16_t* pb[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) pb[i] = Bt + (size_t)(n0 + rq + 8 * NW * i) * g.ldb + c8;
  if (GATHER) {
    // one draw per row of the tile, shared through LDS
    if (t < T) {
      uint32_t row;
      if (g.gen_rows) {
        bool real;
        row = gen_row_of(g, rd, m0 + t, &real);
        if (n0 == 0) gen_row_store(g, m0 + t, row, real);
      } else {
        row = g.a_rowidx[m0 + t];
      }
      s_row[t] = row;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i) pa[i] = g.A + (size_t)s_row[rq + 8 * NW * i] * g.lda + c8;
  } else {
#pragma unroll
    for (int i = 0; i < NI; ++i) pa[i] = g.A + (size_t)(m0 + rq + 8 * NW * i) * g.lda + c8;
  }
  // GATHER: elements beyond a_kvalid (the padding of the contraction) must read as zero.  The lanes that
  // would fetch them are pointed at the zero pad behind the first row of B (see kPitchPad).
  const int kpad = GATHER ? g.a_kvalid - c8 : 0;
  const uint16_t* const zpad = Bt + (size_t)g.ksteps_total * BK + (lane & 7) * 8;

#define ABS_TILE_DMA(ks_, st_)                                                            \
  {                                                                                       \
    const int k0_ = (ks_) * BK;                                                           \
    uint16_t* a_ = smem + (st_) * Cfg::kStage + wave * 512;                               \
    _Pragma("unroll") for (int i = 0; i < NI; ++i)                                        \
      lds_dma16_raw(GATHER && k0_ >= kpad ? zpad : pa[i] + k0_, a_ + i * NW * 512);       \
    _Pragma("unroll") for (int i = 0; i < NI; ++i)                                        \
      lds_dma16_raw(pb[i] + k0_, a_ + T * BK + i * NW * 512);                             \
  }

  f32x16_t acc[4];                       // block 2 mi + ni of the 64 x 64 sub-tile
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;

  const int lr = lane & 31, lk = lane >> 5;
  const int fa = (wm * 64 + lr) * BK, fb = T * BK + (wn * 64 + lr) * BK;
  const int sw = (lr >> 1) & 7;
  constexpr int SUB = 4 / KG;            // 16-wide sub-steps of a k-step per wavefront group
#pragma unroll
  for (int j = 0; j < RING - 1; ++j)
    if (ks0 + j < ks1) ABS_TILE_DMA(ks0 + j, j);
  int stage = 0;
  for (int ks = ks0; ks < ks1; ++ks) {
    // step ks has landed when at most the RING - 2 steps behind it are outstanding
    if (ks + RING - 1 <= ks1) ring_wait_barrier<(RING - 2) * 2 * NI>();   // ... for every wavefront; and everybody
    else                      ring_wait_barrier<0>();                     // is done with step ks - 1
    if (ks + RING - 1 < ks1) ABS_TILE_DMA(ks + RING - 1, stage == 0 ? RING - 1 : stage - 1);
    const uint16_t* sS = smem + stage * Cfg::kStage;
    stage = stage + 1 == RING ? 0 : stage + 1;
    bf16x8_t va[SUB][2], vb[SUB][2];
#pragma unroll
    for (int s = 0; s < SUB; ++s) {
      const int ch = ((((kg * SUB + s) << 1) | lk) ^ sw) << 3;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        va[s][i] = *(const bf16x8_t*)&sS[fa + i * 32 * BK + ch];
        vb[s][i] = *(const bf16x8_t*)&sS[fb + i * 32 * BK + ch];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[2 * i + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[s][i], vb[s][j], acc[2 * i + j], 0, 0, 0);
    }
    if (KG == 1) {
      // issue order: the first fragments, then one read behind each MFMA (left to the compiler: first-layer
      // weight gradient 2048 x 1152 over 8192 rows 50.6 instead of 46.2 us)
      __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
      for (int i = 0; i < 12; ++i) { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); }
      __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
    }
  }
#undef ABS_TILE_DMA

  // ---- epilogue.  Accumulator register r of lane l holds C[8 (r/4) + 4 (l/32) + r%4][l%32] of its block.
  float* const red = (float*)smem;
  uint16_t* const sT = smem + Cfg::kRed;                 // results [n][kPitch]
  uint16_t* const sN = sT + T * Cfg::kPitch;              // results [m][kPitch]
  float* const sC = (float*)(sN + T * Cfg::kPitch);       // column sums per 32 rows
  u32x4_t mk[EPI == EPI_DGRAD ? T * T / 8 / NT : 1];
  if (EPI == EPI_DGRAD) {
    // the ReLU mask, H_l^T [n][m], as whole rows of the tile
#pragma unroll
    for (int i = 0; i < T * T / 8 / NT; ++i) {
      const int q = t + NT * i, nl = q / (T / 8), ch = (q % (T / 8)) * 8;
      mk[i] = *(const u32x4_t*)(g.maskT + (size_t)(n0 + nl) * g.ldmaskT + m0 + ch);
    }
  }
  __syncthreads();                                       // all fragment reads done before LDS is reused
  // blocks of other groups to their owners: [sub-tile][block][source group][quarter][lane]
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int owner = b / OWN;
    if (owner != kg) {
      float4* q = (float4*)(red + ((wsub * 4 + b) * (KG - 1) + (kg < owner ? kg : kg - 1)) * 1024) + lane;
#pragma unroll
      for (int r = 0; r < 4; ++r) q[r * 64] = make_float4(acc[b][4 * r], acc[b][4 * r + 1], acc[b][4 * r + 2], acc[b][4 * r + 3]);
    }
  }
  if (EPI == EPI_DGRAD) {
#pragma unroll
    for (int i = 0; i < T * T / 8 / NT; ++i) {
      const int q = t + NT * i, nl = q / (T / 8), ch = (q % (T / 8)) * 8;
      *(u32x4_t*)&sT[nl * Cfg::kPitch + ch] = mk[i];
    }
  }
  f32x16_t fin[OWN];
#pragma unroll
  for (int b = 0; b < 4; ++b)
    if (b / OWN == kg) fin[b % OWN] = acc[b];
  __syncthreads();
  const int lcol = lane & 31, lrow4 = lk * 4;
  const float* bias = nullptr;
  if (EPI == EPI_RELU || EPI == EPI_LOGITS) bias = g.bias + (size_t)slot * g.bias_slot_stride;
  float* outf = g.outf;
  if (EPI == EPI_WGRAD && !kLocal) outf += (size_t)zsplit * g.split_stride;
  const LocalUpdate& lu = g.local_upd;
  const float* lcur = nullptr; float* lnext = nullptr;
  if (kLocal) {
    lcur = lu.cur + (size_t)(lu.own ? (uint32_t)zsplit : rd.w[zsplit].slot) * lu.stride;
    lnext = lu.next + (size_t)zsplit * lu.stride;
  }
  const bool row_major = kLocal ? lu.wn != nullptr : g.out != nullptr;
#pragma unroll
  for (int j = 0; j < OWN; ++j) {
    const int b = kg * OWN + j;
    float wv[kLocal ? 16 : 1];             // the block's 16 model elements of this lane, asked for together
    if (kLocal) {
      const int i0 = m0 + wm * 64 + (b >> 1) * 32 + lrow4, jn = n0 + wn * 64 + (b & 1) * 32 + lcol;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = i0 + (r >> 2) * 8 + (r & 3);
        wv[r] = i < lu.d_in && jn < lu.d_out ? lcur[(size_t)i * lu.d_out + jn] : 0.f;
      }
    }
    const float4* q = (const float4*)(red + (wsub * 4 + b) * (KG - 1) * 1024) + lane;
#pragma unroll
    for (int o = 0; o < KG - 1; ++o)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float4 v = q[o * 256 + r * 64];
        fin[j][4 * r] += v.x; fin[j][4 * r + 1] += v.y; fin[j][4 * r + 2] += v.z; fin[j][4 * r + 3] += v.w;
      }
    const int bm = wm * 64 + (b >> 1) * 32, nl = wn * 64 + (b & 1) * 32 + lcol;
    const int n = n0 + nl;
    float bv = 0.f, cs = 0.f;
    if (EPI == EPI_RELU || EPI == EPI_LOGITS) bv = n < g.n_valid ? bias[n] : 0.f;
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      const int ml = bm + rg * 8 + lrow4;
      uint16_t h[4];
      uint2 hm = make_uint2(0, 0);     // H_l of the 4 consecutive rows this lane holds
      if (EPI == EPI_DGRAD) hm = *(const uint2*)&sT[nl * Cfg::kPitch + ml];
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        float v = fin[j][rg * 4 + rr];
        if (EPI == EPI_RELU) {
          v = fmaxf(v + bv, 0.f);
        } else if (EPI == EPI_LOGITS) {
          outf[(size_t)(m0 + ml + rr) * g.ldof + n] = v + bv;
        } else if (EPI == EPI_DGRAD) {
          const uint32_t pair = rr < 2 ? hm.x : hm.y;
          v = ((pair >> ((rr & 1) * 16)) & 0x7FFFu) ? v : 0.f;
        } else if (kLocal) {
          const int i = m0 + ml + rr;
          const bool ok = i < lu.d_in && n < lu.d_out;      // padding stays zero in both copies
          v = ok ? wv[rg * 4 + rr] - v : 0.f;
          if (ok) lnext[(size_t)i * lu.d_out + n] = v;
        } else {
          outf[(size_t)(m0 + ml + rr) * g.ldof + n] = v;
        }
        if (kStageT) {
          h[rr] = f32_to_bf16(v);
          if (EPI == EPI_DGRAD) cs += __uint_as_float((uint32_t)h[rr] << 16);
          if (row_major) sN[(ml + rr) * Cfg::kPitch + nl] = h[rr];
        }
      }
      if (kStageT) {
        uint2 o;
        o.x = h[0] | ((uint32_t)h[1] << 16);
        o.y = h[2] | ((uint32_t)h[3] << 16);
        *(uint2*)&sT[nl * Cfg::kPitch + ml] = o;
      }
    }
    if (EPI == EPI_DGRAD) {
      // (the two half-wavefronts hold alternate groups of 4 rows)
      cs += __shfl_xor(cs, 32, 64);
      if (lane < 32) sC[(bm >> 5) * T + nl] = cs;
    }
  }
  if (kLocal) {
    __syncthreads();
    uint16_t* const wt = lu.wt + (size_t)zsplit * lu.shadow_stride;
#pragma unroll
    for (int i = 0; i < T * T / 8 / NT; ++i) {
      const int q = t + NT * i, nl = q / (T / 8), ch = (q % (T / 8)) * 8;
      if (n0 + nl < lu.d_out) *(uint4*)(wt + (size_t)(n0 + nl) * lu.ldwt + m0 + ch) = *(const uint4*)&sT[nl * Cfg::kPitch + ch];
    }
    if (row_major) {
      uint16_t* const wr = lu.wn + (size_t)zsplit * lu.shadow_stride;
#pragma unroll
      for (int i = 0; i < T * T / 8 / NT; ++i) {
        const int q = t + NT * i, ml = q / (T / 8), ch = (q % (T / 8)) * 8;
        if (m0 + ml < lu.d_in) *(uint4*)(wr + (size_t)(m0 + ml) * lu.ldwn + n0 + ch) = *(const uint4*)&sN[ml * Cfg::kPitch + ch];
      }
    }
  } else if (kStageT) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < T * T / 8 / NT; ++i) {
      const int q = t + NT * i, nl = q / (T / 8), ch = (q % (T / 8)) * 8;
      *(uint4*)(g.outT + (size_t)(n0 + nl) * g.ldoT + m0 + ch) = *(const uint4*)&sT[nl * Cfg::kPitch + ch];
    }
    if (g.out) {
#pragma unroll
      for (int i = 0; i < T * T / 8 / NT; ++i) {
        const int q = t + NT * i, ml = q / (T / 8), ch = (q % (T / 8)) * 8;
        *(uint4*)(g.out + (size_t)(m0 + ml) * g.ldo + n0 + ch) = *(const uint4*)&sN[ml * Cfg::kPitch + ch];
      }
    }
    if (EPI == EPI_DGRAD) {
      // the bias gradient's share of every 64 rows
      for (int q = t; q < (T / 64) * T; q += NT) {
        const int rb = q / T, nl = q % T;
        g.colsum[(size_t)((m0 >> 6) + rb) * g.ldcs + n0 + nl] = sC[2 * rb * T + nl] + sC[(2 * rb + 1) * T + nl];
      }
    }
  }
}

// ------------------------------------------------------------------ the GEMM on tiles of 128 x 256
// Products of uploads whose padded rows are not whole 256-row tiles (or whose gathered rows are not whole
// k-steps), once they are many: half of the bytes per flop of a 128 x 128 tile's columns, and two workgroups per
// CU, so that one's multiplications cover the other's barriers and epilogue.  One LDS stage; the next
// k-step's tiles are on their way in registers (two stages would leave room for one workgroup).
// 256 threads = 2 x 2 wavefronts of 64 x 128 (2 x 4 blocks of MFMA 32x32x16, 128 accumulator registers).  LDS layout
// as in mlp_tile_kernel.
constexpr int TNW = 256;
constexpr int kWideMain = (TM + TNW) * BK;               // elements of a k-step's tiles (48 KB)
constexpr int kWidePitch = 64 + 8;                       // of a wavefront's staged results [128 n][64 m]
constexpr int kWideEpi = 4 * 128 * kWidePitch;
template <int EPI, bool GATHER, bool PER_UPLOAD, int TAG>
__global__ __launch_bounds__(256, 2) void mlp_wide_kernel(GemmArgs g, RoundDesc rd) {
  constexpr bool kStageT = EPI == EPI_RELU || EPI == EPI_DGRAD;
  __shared__ __attribute__((aligned(16))) uint16_t smem[kStageT ? kWideEpi : kWideMain];
  __shared__ uint32_t s_row[GATHER ? TM : 1];
  static_assert(kWideEpi >= kWideMain && kWideEpi * 2 + TM * 4 <= 80 * 1024, "two workgroups per CU");

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int bx = blockIdx.x;
  if (EPI == EPI_WGRAD && (g.pig_blocks | g.bias_blocks)) {      // (see mlp_tile_kernel)
    const int own = (int)gridDim.x - g.pig_blocks - g.bias_blocks;
    if (bx >= own + g.pig_blocks) {
      rider_bias<false>(g, rd, bx - own - g.pig_blocks, (float*)smem);
      return;
    }
    if (bx >= own) { piggy_update<256, false>(g, bx - own, smem); return; }
  }
  const int xcd = bx & 7, jx = bx >> 3;                          // block -> tile as in mlp_tile_kernel
  const int trow = xcd * g.rows_per_xcd + jx / g.nt;
  if (trow >= g.mt * g.nsplit) return;
  const int zsplit = trow / g.mt;
  const int m0 = (trow - zsplit * g.mt) * TM, n0 = (jx % g.nt) * TNW;
  const int ks0 = zsplit * g.ksteps_per_split;
  const int ks1 = min(g.ksteps_total, ks0 + g.ksteps_per_split);

  if (EPI == EPI_DGRAD && g.pub_rowloss && blockIdx.x == 0) publish_upload_losses(g, rd.K, rd.stamp);

  const uint16_t* Bt = g.Bt;
  uint32_t slot = 0;
  if (PER_UPLOAD) {
    slot = g.by_upload ? (uint32_t)(m0 / g.rows_per_upload) : rd.w[m0 / g.rows_per_upload].slot;
    Bt += (size_t)slot * g.bt_slot_stride;
  }
  // thread t moves the 16-byte column t & 7 of rows (t >> 3) + 32 i of both tiles
  const int r0 = t >> 3, c8 = (t & 7) * 8;
  const int st_off = r0 * BK + (((t & 7) ^ ((r0 >> 1) & 7)) << 3);
  const uint16_t* pa[4];
  if (GATHER) {
    if (t < TM) {
      uint32_t row;
      if (g.gen_rows) {
        bool real;
        row = gen_row_of(g, rd, m0 + t, &real);
        if (n0 == 0) gen_row_store(g, m0 + t, row, real);
      } else {
        row = g.a_rowidx[m0 + t];
      }
      s_row[t] = row;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) pa[i] = g.A + (size_t)s_row[r0 + 32 * i] * g.lda + c8;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) pa[i] = g.A + (size_t)(m0 + r0 + 32 * i) * g.lda + c8;
  }
  const uint16_t* const pb = Bt + (size_t)(n0 + r0) * g.ldb + c8;
  const size_t b_step = 32 * g.ldb;

  f32x16_t acc[2][4];
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 4; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

  u32x4_t ra[4], rb[8];
#define ABS_FETCH(ks_)                                                                                      \
  {                                                                                                         \
    const int k0_ = (ks_) * BK;                                                                             \
    const bool in_ = !GATHER || k0_ + c8 < g.a_kvalid;      /* padding of gathered rows reads as zero */    \
    _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                           \
      ra[i] = in_ ? *(const u32x4_t*)(pa[i] + k0_) : u32x4_t{0, 0, 0, 0};                                   \
    _Pragma("unroll") for (int i = 0; i < 8; ++i) rb[i] = *(const u32x4_t*)(pb + i * b_step + k0_);         \
  }
  const int lr = lane & 31, lk = lane >> 5;
  const int fa_row = (wm * 64 + lr) * BK, fb_row = TM * BK + (wn * 128 + lr) * BK;
  const int sw = (lr >> 1) & 7;
  if (ks0 < ks1) ABS_FETCH(ks0);
  for (int ks = ks0; ks < ks1; ++ks) {
#pragma unroll
    for (int i = 0; i < 4; ++i) *(u32x4_t*)&smem[st_off + 32 * i * BK] = ra[i];
#pragma unroll
    for (int i = 0; i < 8; ++i) *(u32x4_t*)&smem[TM * BK + st_off + 32 * i * BK] = rb[i];
    __syncthreads();
    if (ks + 1 < ks1) ABS_FETCH(ks + 1);
    // fragments of sub-step s + 1 are read while the MFMAs of sub-step s run
    bf16x8_t fa[2][2], fb[2][4];
#define ABS_FRAGS(set, s_)                                                                                            \
  {                                                                                                                   \
    const int ch_ = ((((s_) << 1) | lk) ^ sw) << 3;                                                                   \
    _Pragma("unroll") for (int i = 0; i < 2; ++i) fa[set][i] = *(const bf16x8_t*)&smem[fa_row + i * 32 * BK + ch_];   \
    _Pragma("unroll") for (int i = 0; i < 4; ++i) fb[set][i] = *(const bf16x8_t*)&smem[fb_row + i * 32 * BK + ch_];   \
  }
    ABS_FRAGS(0, 0);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (s < 3) ABS_FRAGS((s + 1) & 1, s + 1);
#pragma unroll
      for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s & 1][mi], fb[s & 1][ni], acc[mi][ni], 0, 0, 0);
    }
#undef ABS_FRAGS
    // issue order: the first fragments, then one read behind each of a sub-step's first six MFMAs
    __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
    for (int s = 0; s < 3; ++s) {
#pragma unroll
      for (int i = 0; i < 6; ++i) { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); }
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
    __syncthreads();
  }
#undef ABS_FETCH

  // ---- epilogue: a wavefront's own 64 x 128 block (accumulator layout as in mlp_tile_kernel)
  const int lrow4 = lk * 4, mrow = m0 + wm * 64, ncol = n0 + wn * 128;
  const float* bias = nullptr;
  if (EPI == EPI_RELU || EPI == EPI_LOGITS) bias = g.bias + (size_t)slot * g.bias_slot_stride;
  float* outf = g.outf;
  if (EPI == EPI_WGRAD) outf += (size_t)zsplit * g.split_stride;
  uint16_t* const sE = smem + wave * (128 * kWidePitch);
  if (EPI == EPI_DGRAD) {
    // the ReLU mask, H_l^T, as whole 128-byte rows; a lane later replaces the 4 entries it read by its 4 results
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int q = lane + 64 * i, nl = q >> 3, ch = (q & 7) * 8;
      *(uint4*)&sE[nl * kWidePitch + ch] = *(const uint4*)(g.maskT + (size_t)(ncol + nl) * g.ldmaskT + mrow + ch);
    }
  }
  float cs[4] = {0.f, 0.f, 0.f, 0.f};     // EPI_DGRAD: column sums over the 64 rows
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 4; ++ni) {
      const int nl = ni * 32 + lr, n = ncol + nl;
      float bv = 0.f;
      if (EPI == EPI_RELU || EPI == EPI_LOGITS) bv = n < g.n_valid ? bias[n] : 0.f;
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        const int ml = mi * 32 + rg * 8 + lrow4;
        uint16_t h[4];
        uint2 hm = make_uint2(0, 0);
        if (EPI == EPI_DGRAD) hm = *(const uint2*)&sE[nl * kWidePitch + ml];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const size_t m = (size_t)(mrow + ml + rr);
          float v = acc[mi][ni][rg * 4 + rr];
          if (EPI == EPI_RELU) {
            v = fmaxf(v + bv, 0.f);
          } else if (EPI == EPI_LOGITS) {
            outf[m * g.ldof + n] = v + bv;
          } else if (EPI == EPI_DGRAD) {
            const uint32_t pair = rr < 2 ? hm.x : hm.y;
            v = ((pair >> ((rr & 1) * 16)) & 0x7FFFu) ? v : 0.f;
          } else {
            outf[m * g.ldof + n] = v;
          }
          if (kStageT) {
            h[rr] = f32_to_bf16(v);
            if (EPI == EPI_DGRAD) cs[ni] += __uint_as_float((uint32_t)h[rr] << 16);
            if (g.out) g.out[m * g.ldo + n] = h[rr];
          }
        }
        if (kStageT) {
          uint2 o;
          o.x = h[0] | ((uint32_t)h[1] << 16);
          o.y = h[2] | ((uint32_t)h[3] << 16);
          *(uint2*)&sE[nl * kWidePitch + ml] = o;
        }
      }
    }
  if (EPI == EPI_DGRAD) {
    // (the two half-wavefronts hold alternate groups of 4 rows)
#pragma unroll
    for (int ni = 0; ni < 4; ++ni) {
      const float c = cs[ni] + __shfl_xor(cs[ni], 32, 64);
      if (lane < 32) g.colsum[(size_t)(mrow >> 6) * g.ldcs + ncol + ni * 32 + lr] = c;
    }
  }
  if (kStageT) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int q = lane + 64 * i, nl = q >> 3, ch = (q & 7) * 8;
      *(uint4*)(g.outT + (size_t)(ncol + nl) * g.ldoT + mrow + ch) = *(const uint4*)&sE[nl * kWidePitch + ch];
    }
  }
}

// ------------------------------------------------------------------ the large-tile GEMM
// 256 x 256 tile, 512 threads = 2 x 4 wavefronts of 128 x 64 (8 x 4 blocks of MFMA 16x16x32, 128
// accumulator registers), BK = 64.  On gfx950 the LDS accepts about 64 B/clk of writes
// against 256 B/clk of reads and the L1 delivers 64 B/clk, so what bounds a bf16 GEMM
// tile is the bytes staged per flop: a 256 x 256 tile stages 64 KB per 8.4 MFLOP, two
// thirds of what the 128 x 256 tile needs.  Tiles go from global memory straight into
// LDS (global_load_lds_dwordx4: lane l of a wavefront fills bytes [16 l, 16 l + 16) of a
// 1 KB LDS block, i.e. 8 rows of 128 B).  The XOR swizzle is
// applied on the global side: the lane that fills chunk position p of row r fetches
// logical chunk p ^ ((r >> 1) & 7).
// A k-step is four turns of 16 MFMAs per wavefront (half of A times half of B).  The two wavefronts of a SIMD are one
// half-turn apart (the second one's extra barrier before the loop): while one multiplies, the other reads its next
// fragments and requests, so the matrix pipes do not wait for a k-step's first fragments, nor for the address
// unit to take 64 requests in a row.  A half of A or B is requested again as soon as both groups have it in registers,
// for the k-step after the next: a request is seven turns in flight (1.75 k-steps; with two stages filled and
// drained whole it was one), counted (vmcnt) and never drained inside the loop.
// us, the loop with one barrier and a drained stage per k-step / this one, same box, 32768 rows (outputs bit for bit the same):
// weight gradient 2048 x 2048 222 / 201, 3072 x 2048 from gathered rows 381 / 344, forward 2048 x 2048 with one output 240 / 220
// (row-major A) and 246 / 230 (transposed A), first layer from 3072 gathered features 358 / 326.  Without its requests the loop takes
// 161 us (1.70 PFLOP/s), with all of them hitting the L2 183.  Tried on it: requests in front of the fragment reads (+3 to
// +9 %), between the MFMAs (+6 to +9 %), requests of the next-but-one turn so that no read is waited for in front of a barrier
// (+1 %), s_setprio around the MFMAs (nothing: kept out).
// Needs: row count and column count multiples of 256, GATHER with d_0 equal to the padded
// k extent (d_0 % 128 == 0: a gathered row is read over the whole k range).
constexpr int TM3 = 256, TN3 = 256;
constexpr int kStage3 = (TM3 + TN3) * BK;            // elements per LDS stage (64 KB)
constexpr int kHalf3 = 128 * BK;                     // elements of a half of a k-step's A or B (16 KB)
constexpr int kEpiPitch3 = 64 + 8;                   // per wavefront: staging [64 n][72] and [64 m][72]
constexpr int kEpiElems3 = 8 * 2 * 64 * kEpiPitch3;   // 147456 B
constexpr int kSmem3 = 2 * kStage3 > kEpiElems3 ? 2 * kStage3 : kEpiElems3;
static_assert(kSmem3 * 2 + 8 * 1024 <= 160 * 1024, "LDS budget");

template <int EPI, bool GATHER, bool PER_UPLOAD, int TAG>
__global__ __launch_bounds__(512, 1) void mlp_gemm256_kernel(GemmArgs g, RoundDesc rd) {
  // TAG 2 (first-layer weight gradient): the A operand is the dataset itself, rows gathered by
  // a_rowidx and the contraction running over those rows, i.e. A arrives as [k][m] instead of
  // [m][k]; its fragments are read with the transposing LDS read, so no transposed copy of
  // the minibatch is ever written.
  // TAG 3 (forward / input gradient of a hidden layer): the A operand is the TRANSPOSED copy of the
  // activations / output gradients, [k = features][m = stacked rows], read the same way - the layer
  // that produced it then writes no row-major copy at all.
  // TAG 4 / 5 (weight gradients of local SGD): TAG 2 / 0 whose epilogue takes the step (LocalUpdate).
  constexpr bool kLocal = EPI == EPI_WGRAD && TAG >= 4;
  constexpr bool kATR = (EPI == EPI_WGRAD && (TAG == 2 || TAG == 4)) || ((EPI == EPI_RELU || EPI == EPI_DGRAD) && TAG == 3);
  constexpr bool kARows = kATR && EPI == EPI_WGRAD;      // the k rows of A are gathered through a_rowidx
  // TAG 1 (the output layer's input gradient): the contraction runs over the classes, one to four k-steps.
  constexpr bool kShort = EPI == EPI_DGRAD && TAG == 1;
  __shared__ __attribute__((aligned(16))) uint16_t smem[kSmem3 + (kARows ? 4 * 1024 : 0)];

  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int bx = blockIdx.x;
  if (EPI == EPI_WGRAD && (g.pig_blocks | g.bias_blocks)) {
    // The update's blocks come last in the grid: they take the CUs that the product's last wave of
    // tiles leaves idle and the tail.  (Dealt out evenly between the tiles they slowed every tile
    // down: 260 -> 400 us for the hidden layer's product at K = 128.)  Behind them the bias blocks.
    const int own = (int)gridDim.x - g.pig_blocks - g.bias_blocks;
    if (bx >= own + g.pig_blocks) {
      rider_bias<kLocal>(g, rd, bx - own - g.pig_blocks, (float*)smem);
      return;
    }
    if (bx >= own) { piggy_update<512, true>(g, bx - own, smem); return; }
  }
  int m0, n0, zsplit, ks0, ks1;
  // runs of k-steps across tiles (sk_q > 0): this workgroup's next (tile, k-step) pair and the end of
  // its run.
  const bool kRuns = EPI == EPI_WGRAD && g.sk_q > 0;
  int sk_u = 0, sk_end = 0;
  if (kRuns) {
    const int own = (int)gridDim.x - g.pig_blocks - g.bias_blocks;
    // Block b runs on XCD b % 8.  When eight runs span a whole number of tiles' k ranges
    // (8 q = 0 mod k-steps), runs b, b + 8, b + 16, ... start at the same k-step of their tiles: handing
    // run b to block b puts workgroups on one XCD that walk the same k range in step and share their
    // A and B panels in that XCD's L2.  Otherwise an XCD takes neighbouring runs (neighbouring tiles).
    const int lw = (8 * g.sk_q) % g.ksteps_total == 0 ? bx : (bx & 7) * (own >> 3) + (bx >> 3);
    sk_u = lw * g.sk_q;
    sk_end = min(sk_u + g.sk_q, g.mt * g.nt * g.ksteps_total);
    if (sk_u >= sk_end) return;
  } else {
    const int xcd = bx & 7, jx = bx >> 3;
    const int trow = xcd * g.rows_per_xcd + jx / g.nt;
    if (trow >= g.mt * g.nsplit) return;
    zsplit = trow / g.mt;
    m0 = (trow - zsplit * g.mt) * TM3; n0 = (jx % g.nt) * TN3;
    ks0 = zsplit * g.ksteps_per_split;
    ks1 = min(g.ksteps_total, ks0 + g.ksteps_per_split);
  }

  if (EPI == EPI_DGRAD && g.pub_rowloss && blockIdx.x == 0) publish_upload_losses(g, rd.K, rd.stamp);

  for (;;) {       // one pass per piece of the run (a single pass without runs)
  if (kRuns) {
    const int tile = sk_u / g.ksteps_total;
    ks0 = sk_u - tile * g.ksteps_total;
    ks1 = min(g.ksteps_total, ks0 + (sk_end - sk_u));
    m0 = (tile / g.nt) * TM3; n0 = (tile % g.nt) * TN3;
    zsplit = sk_u / g.sk_q - tile * g.ksteps_total / g.sk_q;     // pieces of earlier runs in this tile
    sk_u += ks1 - ks0;
  }

  const uint16_t* Bt = g.Bt;
  uint32_t slot = 0;
  if (PER_UPLOAD) {
    slot = g.by_upload ? (uint32_t)(m0 / g.rows_per_upload) : rd.w[m0 / g.rows_per_upload].slot;
    Bt += (size_t)slot * g.bt_slot_stride;
  }

  // Requests.  A half of A (h = 0, 1) is rows h 64 .. + 64 of both wavefront rows' 128, a half of B columns
  // h 32 .. + 32 of the four wavefront columns' 64: 16 KB each, two 1 KB requests per wavefront.  A request fills 8
  // rows of 128 bytes, lane l chunk position l & 7 of row l >> 3 (chunk swizzle (row >> 1) & 7).  kATR: a half of A is k rows
  // h 32 .. + 32 of all 256 columns; a request fills two rows of 512 bytes, lane l 16 bytes of row l >> 5; the 64-byte
  // blocks of a row are stored at position b ^ (row & 3), so that the four rows one transposing read touches cover all banks.
  const int pc = lane & 7;
  const int c_even = (pc ^ (((lane >> 4)) & 7)) * 8;        // (row >> 1) & 7 for request 0
  const int c_odd = (pc ^ ((4 + (lane >> 4)) & 7)) * 8;     //                for request 1
  const int dr = (wave >> 2) * 128 + (wave & 3) * 16 + (lane >> 3);         // A row of request 0, half 0
  const uint16_t* pa[4] = {nullptr, nullptr, nullptr, nullptr};              // (GATHER) [2 half + request]
  const uint16_t *va0 = nullptr, *va1 = nullptr;                             // a lane's pieces of A at k-step 0, else
  const int atr_row = wave * 4 + (lane >> 5);                                // k row of request 0, half 0 (kATR)
  const int atr_c = lane & 31;
  const int atr_col0 = m0 + (((((atr_c >> 2) ^ (lane >> 5)) << 2) | (atr_c & 3)) << 3);          // request 0
  const int atr_col1 = m0 + (((((atr_c >> 2) ^ (2 + (lane >> 5))) << 2) | (atr_c & 3)) << 3);    // request 1
  if (kATR) {
    if (!kARows) {
      va0 = g.A + ((size_t)ks0 * BK + atr_row) * g.lda + atr_col0;
      va1 = g.A + ((size_t)ks0 * BK + atr_row + 2) * g.lda + atr_col1;
    }
  } else if (GATHER) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int m = m0 + dr + (q >> 1) * 64 + (q & 1) * 8;
      uint32_t row;
      if (g.gen_rows) {
        bool real;
        row = gen_row_of(g, rd, m, &real);
        if (n0 == 0 && pc == 0) gen_row_store(g, m, row, real);
      } else {
        row = g.a_rowidx[m];
      }
      pa[q] = g.A + (size_t)row * g.lda + (size_t)ks0 * BK + ((q & 1) ? c_odd : c_even);
    }
  } else {
    va0 = g.A + (size_t)(m0 + dr) * g.lda + (size_t)ks0 * BK + c_even;
    va1 = g.A + (size_t)(m0 + dr + 8) * g.lda + (size_t)ks0 * BK + c_odd;
  }
  const int br = (wave >> 1) * 64 + (wave & 1) * 16 + (lane >> 3);          // B row of request 0, half 0
  const uint16_t* const vb0 = Bt + (size_t)(n0 + br) * g.ldb + (size_t)ks0 * BK + c_even;
  const uint16_t* const vb1 = Bt + (size_t)(n0 + br + 8) * g.ldb + (size_t)ks0 * BK + c_odd;
  const uint32_t dmaA = lds_offset(smem) + (uint32_t)wave * 2048u;           // this wavefront's 2 KB of a half
  const uint32_t dmaB = dmaA + 4 * kHalf3 * 2;
  const int nks = ks1 - ks0;
  // (kARows) The dataset rows of a k-step travel through a ring of four steps in LDS as well, each wavefront's 8 (16
  // bytes per parity of lane >> 5) as a request of its own: a register load would be counted with the tile requests,
  // and the wait for it would empty the pipeline.
  u32x4_t aidx = {0, 0, 0, 0};                                               // [2 half + request] of the k-step to request next
  const uint16_t* const idx_ring = smem + (kARows ? kSmem3 + wave * 128 : 0);   // 256 bytes per wavefront, 2 KB per step
  const uint32_t idx_dma = lds_offset(smem) + kSmem3 * 2 + (uint32_t)wave * 256u;
  const uint32_t* const idx_src = kARows ? g.a_rowidx + (size_t)ks0 * BK + ((lane >> 1) & 1) * 32 + wave * 4 + (lane & 1) * 2 + ((lane >> 2) & 1) : nullptr;
#define ABS_DMA_IDX(j_) if (kARows) lds_dma4_at(idx_src + (size_t)min(j_, nks - 1) * BK, idx_dma + (uint32_t)((j_) & 3) * 2048u);
#define ABS_DMA_A(j_, st_, h_)                                                                                \
  {                                                                                                           \
    const uint32_t a_ = dmaA + ((st_) * 2 + (h_)) * kHalf3 * 2;                                               \
    if (kARows) {                                                                                             \
      lds_dma16_at(g.A + (size_t)aidx[2 * (h_)] * g.lda + atr_col0, a_);                                      \
      lds_dma16_at(g.A + (size_t)aidx[2 * (h_) + 1] * g.lda + atr_col1, a_ + 1024);                           \
    } else if (kATR) {                                                                                        \
      const size_t o_ = (size_t)((j_) * BK + (h_) * 32) * g.lda;                                              \
      lds_dma16_at(va0 + o_, a_); lds_dma16_at(va1 + o_, a_ + 1024);                                          \
    } else if (GATHER) {                                                                                      \
      lds_dma16_at(pa[2 * (h_)] + (j_) * BK, a_); lds_dma16_at(pa[2 * (h_) + 1] + (j_) * BK, a_ + 1024);      \
    } else {                                                                                                  \
      const size_t o_ = (size_t)(j_) * BK + (size_t)(h_) * 64 * g.lda;                                        \
      lds_dma16_at(va0 + o_, a_); lds_dma16_at(va1 + o_, a_ + 1024);                                          \
    }                                                                                                         \
  }
#define ABS_DMA_B(j_, st_, h_)                                                                                \
  {                                                                                                           \
    const uint32_t b_ = dmaB + ((st_) * 2 + (h_)) * kHalf3 * 2;                                               \
    const size_t o_ = (size_t)(j_) * BK + (size_t)(h_) * 32 * g.ldb;                                          \
    lds_dma16_at(vb0 + o_, b_); lds_dma16_at(vb1 + o_, b_ + 1024);                                            \
  }

  // ---- main loop on MFMA 16x16x32.  A wavefront's 128 x 64 sub-tile is 8 x 4 blocks of 16 x 16
  // (128 accumulator registers); lane l holds row l & 15 and the 8 k values 8 (l >> 4) .. of an
  // operand block, and accumulator register r of a block is row 4 (l >> 4) + r, column l & 15.
  // Per flop this form moves a quarter of the accumulator registers in and out of the matrix pipe
  // that the 32x32x16 form does: on random operands the pipes alone sustain 2.18 instead of
  // 1.86 PFLOP/s before the chip lowers its clock.
  f32x4_t acc[8][4];
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[a][b][r] = 0.f;
  const int lr = lane & 15, lk = lane >> 4;
  const int sw = (lr >> 1) & 7;
  const int ch0 = (lk ^ sw) << 3, ch1 = ((4 | lk) ^ sw) << 3;
  const int fa_row = (wm * 64 + lr) * BK, fb_row = 4 * kHalf3 + (wn * 32 + lr) * BK;
  // kATR (A stored [k][m]): a block's fragment is two transposing reads.  Such a read works on groups
  // of 16 lanes: lane s of a group points at 4 consecutive columns of row s / 4 of a 4 x 16 piece and
  // receives column s of its 4 rows.  Quarter-wavefront q takes k rows 8 q .. 8 q + 7 of the 32-row
  // sub-step (pieces at rows + 0 and + 4), all quarters the same 16 columns; the block position is
  // XORed with the row's low bits (= s / 4) as stored.
  const int t16s = lane & 15, t16r = t16s >> 2;
  int fa_tr[4];                                              // blocks 2 i, 2 i + 1 of the wavefront's eight
#pragma unroll
  for (int i = 0; i < 4; ++i) fa_tr[i] = (t16r + 8 * lk) * TM3 + (wm * 4 + (i ^ t16r)) * 32 + 4 * (t16s & 3);
  // fragments of a half of A: four blocks of rows, both 32-wide sub-steps [2 block + sub-step]; kATR: eight blocks, one sub-step
  bf16x8_t fa[8], fbx[2][2], fby[2][2];
#define ABS_LOAD_A(st_, h_)                                                                                           \
  _Pragma("unroll") for (int q_ = 0; q_ < 8; ++q_) {                                                                  \
    if (kATR) {                                                                                                       \
      typedef short s16x4_ __attribute__((ext_vector_type(4)));                                                       \
      const uint16_t* p_ = smem + fa_tr[q_ >> 1] + ((st_) * 2 + (h_)) * kHalf3 + (q_ & 1) * 16;                       \
      union { s16x4_ h[2]; bf16x8_t v; } u_;                                                                          \
      u_.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_*)(p_));             \
      u_.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_*)(p_ + 4 * TM3));   \
      fa[q_] = u_.v;                                                                                                  \
    } else {                                                                                                          \
      fa[q_] = *(const bf16x8_t*)&smem[fa_row + ((q_ & 1) ? ch1 : ch0) + ((st_) * 2 + (h_)) * kHalf3 + (q_ >> 1) * 16 * BK]; \
    }                                                                                                                 \
  }
#define ABS_LOAD_B(dst_, st_, h_)                                                                                     \
  _Pragma("unroll") for (int s_ = 0; s_ < 2; ++s_) _Pragma("unroll") for (int j_ = 0; j_ < 2; ++j_)                   \
    dst_[j_][s_] = *(const bf16x8_t*)&smem[fb_row + (s_ ? ch1 : ch0) + ((st_) * 2 + (h_)) * kHalf3 + j_ * 16 * BK];
  // multiply the halves in the registers, between two barriers
#define ABS_MMA(ha_, hb_, b_)                                                                                         \
  __builtin_amdgcn_sched_barrier(0);                                                                                  \
  if (kATR) {                                                                                                         \
    _Pragma("unroll") for (int i_ = 0; i_ < 8; ++i_) _Pragma("unroll") for (int j_ = 0; j_ < 2; ++j_)                 \
      acc[i_][(hb_) * 2 + j_] =                                                                                       \
          __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i_], b_[j_][ha_], acc[i_][(hb_) * 2 + j_], 0, 0, 0);             \
  } else {                                                                                                            \
    _Pragma("unroll") for (int s_ = 0; s_ < 2; ++s_) _Pragma("unroll") for (int i_ = 0; i_ < 4; ++i_)                 \
      _Pragma("unroll") for (int j_ = 0; j_ < 2; ++j_)                                                                \
        acc[(ha_) * 4 + i_][(hb_) * 2 + j_] =                                                                         \
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[2 * i_ + s_], b_[j_][s_], acc[(ha_) * 4 + i_][(hb_) * 2 + j_], 0, 0, 0); \
  }                                                                                                                   \
  __builtin_amdgcn_sched_barrier(0);                                                                                  \
  asm volatile("s_barrier" ::: "memory");
#define ABS_TURN(i_)                                                                                                  \
  if (left >= 2)      ring_wait_barrier<kARows ? 13 : 12>();       /* (kARows: one request of indices among them) */  \
  else if (left == 1) ring_wait_barrier<10 - 2 * (i_)>();                                                             \
  else                ring_wait_barrier<(i_) == 0 ? 2 : 0>();
#define ABS_STEP(X_, Y_, st_)                                                                                         \
  {                                                                                                                   \
    const int left = nks - 1 - j;                                                                                     \
    ABS_LOAD_A(st_, 0);                                                                                               \
    if (kARows) aidx = *(const u32x4_t*)(idx_ring + ((j + 2) & 3) * 1024 + (lane >> 5) * 8);                          \
    if (left >= 2) { ABS_DMA_IDX(j + 4); ABS_DMA_B(j + 2, st_, 0); }                                                  \
    ABS_TURN(0); ABS_MMA(0, 0, X_);                                                                                   \
    ABS_LOAD_B(Y_, st_, 1);                                                                                           \
    if (left >= 2) ABS_DMA_A(j + 2, st_, 0);                                                                          \
    ABS_TURN(1); ABS_MMA(0, 1, Y_);                                                                                   \
    ABS_LOAD_A(st_, 1);                                                                                               \
    if (left >= 2) ABS_DMA_B(j + 2, st_, 1);                                                                          \
    ABS_TURN(2); ABS_MMA(1, 1, Y_);                                                                                   \
    if (left >= 1) ABS_LOAD_B(Y_, (st_) ^ 1, 0);                                                                      \
    if (left >= 2) ABS_DMA_A(j + 2, st_, 1);                                                                          \
    ABS_TURN(3); ABS_MMA(1, 0, X_);                                                                                   \
  }
  if constexpr (kShort) {
    // A start, two k-steps and an end: turns have nothing to overlap, and with both stages requested at once the first one arrives
    // later.  So a stage is drained whole and the next one asked for behind that; the fragments of a 32-wide sub-step are read in
    // halves, one half ahead of the MFMAs that use them (us, the loop below / both stages at once / this, 100 classes: 8192 x 2048
    // 21.1 / 19.7 / 18.8, 32768 x 2048 61.0 / 59.5 / 55.4; 64 classes, 16384 x 1024 16.4 / 15.6 / 14.5).
#define ABS_DMA_STEP(j_, st_) { ABS_DMA_B(j_, st_, 0); ABS_DMA_A(j_, st_, 0); ABS_DMA_B(j_, st_, 1); ABS_DMA_A(j_, st_, 1); }
#define ABS_SUB_A(set_, s_, h_)                                                                                       \
  _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                                       \
    sa[set_][i] = *(const bf16x8_t*)&stage[fa_row + ((s_) ? ch1 : ch0) + (h_) * kHalf3 + i * 16 * BK];
#define ABS_SUB_B(set_)                                                                                               \
  _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                                       \
    sb[set_][i] = *(const bf16x8_t*)&stage[fb_row + ((set_) ? ch1 : ch0) + (i >> 1) * kHalf3 + (i & 1) * 16 * BK];
#define ABS_SUB_MMA(h_, aset_, bset_)                                                                                 \
  _Pragma("unroll") for (int i = 0; i < 4; ++i) _Pragma("unroll") for (int b = 0; b < 4; ++b)                         \
    acc[(h_) * 4 + i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sa[aset_][i], sb[bset_][b], acc[(h_) * 4 + i][b], 0, 0, 0);
    if (nks > 0) ABS_DMA_STEP(0, 0);
    for (int j = 0; j < nks; ++j) {
      const int st = j & 1;
      ring_wait_barrier<0>();            // step j is in LDS, and everybody is done with step j - 1
      if (j + 1 < nks) ABS_DMA_STEP(j + 1, st ^ 1);
      const uint16_t* const stage = smem + st * 2 * kHalf3;
      bf16x8_t sa[2][4], sb[2][4];
      ABS_SUB_B(0); ABS_SUB_A(0, 0, 0);
      ABS_SUB_A(1, 0, 1);                ABS_SUB_MMA(0, 0, 0);
      ABS_SUB_B(1); ABS_SUB_A(0, 1, 0);  ABS_SUB_MMA(1, 1, 0);
      ABS_SUB_A(1, 1, 1);                ABS_SUB_MMA(0, 0, 1);
                                         ABS_SUB_MMA(1, 1, 1);
      // issue order: the first fragments, then the reads of the next half spread between the 16 MFMAs of the current one
      __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) { __builtin_amdgcn_sched_group_barrier(0x008, 2, 0); __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); }
      __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
#pragma unroll
      for (int i = 0; i < 8; ++i) { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); }
      __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) { __builtin_amdgcn_sched_group_barrier(0x008, 2, 0); __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); }
      __builtin_amdgcn_sched_group_barrier(0x008, 24, 0);
    }
#undef ABS_SUB_MMA
#undef ABS_SUB_B
#undef ABS_SUB_A
#undef ABS_DMA_STEP
  } else if (nks > 0) {
    if (kARows) {
      const uint32_t* r0 = g.a_rowidx + (size_t)ks0 * BK + atr_row;
      const uint32_t* r1 = r0 + (nks > 1 ? BK : 0);
      ABS_DMA_IDX(2); ABS_DMA_IDX(3);
      aidx = u32x4_t{r0[0], r0[2], r0[32], r0[34]};
      const u32x4_t a1 = {r1[0], r1[2], r1[32], r1[34]};
      ABS_DMA_B(0, 0, 0); ABS_DMA_A(0, 0, 0); ABS_DMA_B(0, 0, 1); ABS_DMA_A(0, 0, 1);
      aidx = a1;
    } else {
      ABS_DMA_B(0, 0, 0); ABS_DMA_A(0, 0, 0); ABS_DMA_B(0, 0, 1); ABS_DMA_A(0, 0, 1);
    }
    if (nks > 1) {
      ABS_DMA_B(1, 1, 0); ABS_DMA_A(1, 1, 0); ABS_DMA_B(1, 1, 1); ABS_DMA_A(1, 1, 1);
      ring_wait_barrier<12>();
    } else {
      ring_wait_barrier<4>();
    }
    ABS_LOAD_B(fbx, 0, 0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // (requested again in the first turn)
    if (wm) asm volatile("s_barrier" ::: "memory");
    for (int j = 0;;) {
      ABS_STEP(fbx, fby, 0);
      if (++j >= nks) break;
      ABS_STEP(fby, fbx, 1);
      if (++j >= nks) break;
    }
    if (!wm) asm volatile("s_barrier" ::: "memory");
  }
#undef ABS_STEP
#undef ABS_TURN
#undef ABS_MMA
#undef ABS_LOAD_B
#undef ABS_LOAD_A
#undef ABS_DMA_B
#undef ABS_DMA_A
#undef ABS_DMA_IDX
  __syncthreads();      // all fragment reads done before the staging area is reused

  // ---- epilogue: bf16 outputs leave through this wavefront's private LDS staging, half of the
  // wavefront's tile (64 x 64) at a time, staged as [n][m] for the transposed copy and as [m][n]
  // for the row-major one, so that every global store is 16 bytes per lane and 128 contiguous
  // bytes per row.  The ReLU mask of the tile is one bit per element in accumulator order:
  // word a / 2 of a lane, bit (a & 1) 16 + 4 b + r for block (a, b), register r.
  const int lcol = lane & 15, lrow4 = (lane >> 4) * 4;
  if constexpr (kLocal) {
    // half of the wavefront's tile at a time: the 64 model elements of a lane are asked for together
    // (they may be where the results go, so the compiler cannot move them ahead of a store)
    const LocalUpdate& lu = g.local_upd;
    const float* const cur = lu.cur + (size_t)(lu.own ? (uint32_t)zsplit : rd.w[zsplit].slot) * lu.stride;
    float* const next = lu.next + (size_t)zsplit * lu.stride;
    uint16_t* const wt = lu.wt + (size_t)zsplit * lu.shadow_stride;
    uint16_t* const wr = lu.wn ? lu.wn + (size_t)zsplit * lu.shadow_stride : nullptr;
    uint16_t* const sT = smem + wave * (2 * 64 * kEpiPitch3);     // [64 n][72]
    uint16_t* const sN = sT + 64 * kEpiPitch3;                    // [64 m][72]
    const int ncol = n0 + wn * 64;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int mrow = m0 + wm * 128 + half * 64;
      float wv[4][4][4];
#pragma unroll
      for (int ah = 0; ah < 4; ++ah)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const int i = mrow + ah * 16 + lrow4 + rr, n = ncol + b * 16 + lcol;
            wv[ah][b][rr] = i < lu.d_in && n < lu.d_out ? cur[(size_t)i * lu.d_out + n] : 0.f;
          }
#pragma unroll
      for (int ah = 0; ah < 4; ++ah) {
        const int ml = ah * 16 + lrow4;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int nl = b * 16 + lcol, n = ncol + nl;
          uint16_t h[4];
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) {
            const int i = mrow + ml + rr;
            const bool ok = i < lu.d_in && n < lu.d_out;         // padding stays zero in both copies
            const float v = ok ? wv[ah][b][rr] - acc[half * 4 + ah][b][rr] : 0.f;
            if (ok) next[(size_t)i * lu.d_out + n] = v;
            h[rr] = f32_to_bf16(v);
            if (wr) sN[(ml + rr) * kEpiPitch3 + nl] = h[rr];
          }
          uint2 o;
          o.x = h[0] | ((uint32_t)h[1] << 16);
          o.y = h[2] | ((uint32_t)h[3] << 16);
          *(uint2*)&sT[nl * kEpiPitch3 + ml] = o;
        }
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int q = lane + 64 * i, r = q >> 3, ch = (q & 7) * 8;
        if (ncol + r < lu.d_out) *(uint4*)(wt + (size_t)(ncol + r) * lu.ldwt + mrow + ch) = *(const uint4*)&sT[r * kEpiPitch3 + ch];
        if (wr && mrow + r < lu.d_in) *(uint4*)(wr + (size_t)(mrow + r) * lu.ldwn + ncol + ch) = *(const uint4*)&sN[r * kEpiPitch3 + ch];
      }
    }
    break;
  }
  if constexpr (EPI == EPI_WGRAD || EPI == EPI_LOGITS) {
    // fp32 results straight from the accumulators (64 contiguous bytes per row and quarter-wavefront):
    // this piece's partial of the tile, or the logits with their bias
    float* const outf = g.outf + (EPI == EPI_WGRAD ? (size_t)zsplit * g.split_stride : (size_t)0) +
                        (size_t)(m0 + wm * 128 + lrow4) * g.ldof + n0 + wn * 64 + lcol;
    float bv[4] = {0.f, 0.f, 0.f, 0.f};
    if (EPI == EPI_LOGITS) {
      const float* bias = g.bias + (size_t)slot * g.bias_slot_stride;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int n = n0 + wn * 64 + b * 16 + lcol;
        bv[b] = n < g.n_valid ? bias[n] : 0.f;
      }
    }
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr)
#pragma unroll
        for (int b = 0; b < 4; ++b) outf[(size_t)(a * 16 + rr) * g.ldof + b * 16] = acc[a][b][rr] + bv[b];
    if (!kRuns || sk_u >= sk_end) break;
    continue;
  }
  const float* bias = nullptr;
  if (EPI == EPI_RELU) bias = g.bias + (size_t)slot * g.bias_slot_stride;
  uint32_t mbits[4] = {0u, 0u, 0u, 0u};
  uint32_t* const mbits_at =
      g.maskbits ? g.maskbits + ((((size_t)(m0 / TM3) * g.nt + n0 / TN3) * 8 + wave) * 64 + lane) * 4 : nullptr;
  if (EPI == EPI_DGRAD && mbits_at) {
    const uint4 q = *(const uint4*)mbits_at;
    mbits[0] = q.x; mbits[1] = q.y; mbits[2] = q.z; mbits[3] = q.w;
  }
  uint16_t* const sT = smem + wave * (2 * 64 * kEpiPitch3);     // [64 n][72]
  uint16_t* const sN = sT + 64 * kEpiPitch3;                    // [64 m][72]
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    float cs[4] = {0.f, 0.f, 0.f, 0.f};   // EPI_DGRAD: column sums over this half's 64 rows
    if (EPI == EPI_DGRAD && !mbits_at) {
      // the ReLU mask of this half, H_l^T [64 n][64 m], fetched as whole 128-byte rows into sT;
      // every lane later replaces the 4 entries it read by its 4 results
      const int mrow = m0 + wm * 128 + half * 64, ncol = n0 + wn * 64;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int q = lane + 64 * i, r = q >> 3, ch = (q & 7) * 8;
        *(uint4*)&sT[r * kEpiPitch3 + ch] = *(const uint4*)(g.maskT + (size_t)(ncol + r) * g.ldmaskT + mrow + ch);
      }
    }
#pragma unroll
    for (int ah = 0; ah < 4; ++ah) {
      const int a = half * 4 + ah;
      const int ml = ah * 16 + lrow4;                           // first of this lane's 4 rows inside the half
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int nl = b * 16 + lcol;
        const int n = n0 + wn * 64 + nl;
        float bv = 0.f;
        if (EPI == EPI_RELU) bv = n < g.n_valid ? bias[n] : 0.f;
        uint2 hm = make_uint2(0, 0);
        if (EPI == EPI_DGRAD && !mbits_at) hm = *(const uint2*)&sT[nl * kEpiPitch3 + ml];
        uint16_t h[4];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int bit = (a & 1) * 16 + b * 4 + rr;
          float v = acc[a][b][rr];
          if (EPI == EPI_RELU) {
            v = fmaxf(v + bv, 0.f);
            // (the mask is taken from the narrowed value, as the transposed copy would give it)
            if ((f32_to_bf16(v) & 0x7FFFu) != 0) mbits[a >> 1] |= 1u << bit;
          } else {
            const uint32_t pair = rr < 2 ? hm.x : hm.y;
            const bool pass = mbits_at ? ((mbits[a >> 1] >> bit) & 1u) != 0
                                       : ((pair >> ((rr & 1) * 16)) & 0x7FFFu) != 0;
            v = pass ? v : 0.f;
          }
          h[rr] = f32_to_bf16(v);
          if (EPI == EPI_DGRAD) cs[b] += __uint_as_float((uint32_t)h[rr] << 16);
        }
        uint2 o;
        o.x = h[0] | ((uint32_t)h[1] << 16);
        o.y = h[2] | ((uint32_t)h[3] << 16);
        *(uint2*)&sT[nl * kEpiPitch3 + ml] = o;
        if (g.out) {
          // row-major staging in 4-byte pieces: neighbouring lanes hold neighbouring columns of the same
          // 4 rows; the even lane takes rows 0-1 of the pair of columns, the odd lane rows 2-3 (half the
          // LDS writes of one 2-byte write per element: a round 0.7 % faster)
          const bool odd = lane & 1;
          const uint32_t send = odd ? o.x : o.y;
          const uint32_t recv = (uint32_t)__builtin_amdgcn_mov_dpp((int)send, 0xB1, 0xF, 0xF, true);   // lane ^ 1
          const uint32_t w0 = odd ? ((recv & 0xFFFFu) | (o.y << 16)) : ((o.x & 0xFFFFu) | (recv << 16));
          const uint32_t w1 = odd ? ((recv >> 16) | (o.y & 0xFFFF0000u)) : ((o.x >> 16) | (recv & 0xFFFF0000u));
          uint16_t* const q = &sN[(ml + (odd ? 2 : 0)) * kEpiPitch3 + (nl & ~1)];
          *(uint32_t*)q = w0;
          *(uint32_t*)(q + kEpiPitch3) = w1;
        }
      }
    }
    if (EPI == EPI_DGRAD) {
      // the bias gradient's share of these 64 rows (the four quarter-wavefronts hold rows 4 q .. 4 q + 3 of every 16)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        float c = cs[b] + __shfl_xor(cs[b], 16, 64);
        c += __shfl_xor(c, 32, 64);
        if (lane < 16)
          g.colsum[(size_t)((m0 + wm * 128 + half * 64) >> 6) * g.ldcs + n0 + wn * 64 + b * 16 + lcol] = c;
      }
    }
    {
      const int mrow = m0 + wm * 128 + half * 64, ncol = n0 + wn * 64;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int q = lane + 64 * i, r = q >> 3, ch = (q & 7) * 8;
        const uint4 vt = *(const uint4*)&sT[r * kEpiPitch3 + ch];
        store16_stream(g.outT + (size_t)(ncol + r) * g.ldoT + mrow + ch, vt, g.stream_out != 0);
        if (g.out) {
          const uint4 vn = *(const uint4*)&sN[r * kEpiPitch3 + ch];
          store16_stream(g.out + (size_t)(mrow + r) * g.ldo + ncol + ch, vn, g.stream_out != 0);
        }
      }
    }
  }
  if (EPI == EPI_RELU && mbits_at) *(uint4*)mbits_at = make_uint4(mbits[0], mbits[1], mbits[2], mbits[3]);
  break;
  }
}

// ------------------------------------------------------------------ weight gradients that take the step themselves
// Eq. 2 / Eq. 3 for ALL weight matrices of a round (or of a local step) in one launch.  Where the contraction of a
// weight gradient is not split - a round of few rows, or one upload's rows in local SGD - a workgroup's accumulators
// hold the whole gradient of its tile, so its epilogue reads the model, takes the step and writes the fp32 model and both
// bf16 copies: no partial goes to memory and back, no update needs a launch, and the layers' products, which depend
// on nothing but the backward pass, fill the CUs side by side.  The biases ride as the last workgroups.
//   uploads = 1, sel 0:  w^{t+1} = w^t - sum over all stacked rows (Eq. 3)
//   uploads = K, sel 1:  a local step on the private models; sel 2: the first one, from the uploads' ring slots (Eq. 2)
// DIRECT: layer 0's A operand is the dataset as it lies in memory, [k = gathered rows][m], read through the
// transposing LDS read (see mlp_gemm256_kernel), instead of a transposed copy of the minibatch.
// What bounds it: the bytes a CU draws from beyond its L1 (a 128 x 128 tile 0.65 us a k-step, 64 x 64 0.2 us), then 2 us of start
// (arguments, first tiles) and 2-4 us of epilogue.  us of the launches it replaces / its own: 3072-512-10, 1024 rows
// 22.1 (three launches) / 11.3, 1000-520-300-26, 1152 rows 23.4 (four) / 8.9, 3072-1024-1024-10, 4096 rows 89 (four) / 73.
struct StepLayer {
  const uint16_t* A; size_t lda;         // H_l^T [dp_in][lda]; layer 0: the transposed minibatch or, DIRECT, the dataset
  const uint16_t* Bt; size_t ldb;        // dZ_{l+1}^T [dp_out][ldb]
  int mt, nt;                            // tiles
  int d_in, d_out, dp_out;
  const float* cur; float* next;         // fp32 [d_in][d_out]; models `stride` floats apart
  uint16_t* wn; size_t ldwn; uint16_t* wt; size_t ldwt;     // bf16 copies (wn may be null)
};
struct StepArgs {
  int L, uploads, sel, ksteps;           // k-steps of an upload's (uploads = 1: all) rows
  const uint32_t* rowidx;
  size_t stride, shadow_stride;
  int first[8];                          // first workgroup of each layer, then (from [L]) of the biases
  int bias_per;
  StepLayer l[ABS_MAX_LAYERS];
  BiasCore bias;
};

// Tiles of TMx x TNx, NW wavefronts in 64 x 64 sub-tiles (2 x 2 blocks of MFMA 32x32x16) and KG groups along the
// contraction of a k-step, as in mlp_tile_kernel.
template <int TMx, int TNx, int NW_>
struct StepCfg {
  static constexpr int WSM = TMx / 64, WSN = TNx / 64, NW = NW_, NT = NW * 64, KG = NW / (WSM * WSN), OWN = 4 / KG;
  static constexpr int NIA = TMx / (8 * NW), NIB = TNx / (8 * NW);             // requests per wavefront and k-step
  static constexpr int kStage = (TMx + TNx) * BK;
  static constexpr int kRed = WSM * WSN * 4 * (KG - 1) * 1024 * 2;             // exchanged blocks (in elements of 2 bytes) ...
  static constexpr int kPitchT = TMx + 8, kPitchN = TNx + 8;
  static constexpr int kOut = TNx * kPitchT + TMx * kPitchN;                   // ... and, after them, both orientations
  static constexpr int smem(int ring) {
    const int a = ring * kStage, b = kRed > kOut ? kRed : kOut;
    return a > b ? a : b;
  }
  static constexpr int kIdx = 4 * NW * 128;                                    // ring of row indices: 4 steps x 256 bytes per wavefront
};

template <int TMx, int TNx, int NW_, int RING, bool ATR>
__device__ __forceinline__ void step_tile(const StepArgs& g, const StepLayer& ly, const RoundDesc& rd, int z, int m0, int n0, uint16_t* smem) {
  using Cfg = StepCfg<TMx, TNx, NW_>;
  constexpr int NW = Cfg::NW, NT = Cfg::NT, KG = Cfg::KG, OWN = Cfg::OWN, NIA = Cfg::NIA, NIB = Cfg::NIB;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int kg = wave / (Cfg::WSM * Cfg::WSN), wsub = wave % (Cfg::WSM * Cfg::WSN);
  const int wm = wsub / Cfg::WSN, wn = wsub % Cfg::WSN;
  const int nks = g.ksteps;
  const size_t kbase = (size_t)z * nks * BK;               // first stacked row of this contraction

  // requests, k contiguous: 8 rows of 128 bytes (see mlp_tile_kernel)
  const int c8 = ((lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7)) * 8;
  const int rq = 8 * wave + (lane >> 3);
  const uint16_t* pa[NIA]; const uint16_t* pb[NIB];
#pragma unroll
  for (int i = 0; i < NIB; ++i)          // (a tile may be wider than the layer: the columns beyond are dropped)
    pb[i] = ly.Bt + (size_t)min(n0 + rq + 8 * NW * i, ly.dp_out - 1) * ly.ldb + kbase + c8;
  // layer 0: RPR gathered rows of TMx columns each; their 64-byte blocks are stored at position b ^ f(row), so that
  // the four rows one transposing read touches cover all banks.  Columns beyond d_0 re-read the row's first ones (dropped).
  constexpr int RPR = 512 / TMx, LPR = 64 / RPR;           // rows of a request, lanes per row
  const int ar = RPR * wave + lane / LPR;                  // k row of request 0 (+ RPR NW i)
  const int asw = TMx == 128 ? (ar & 3) : ((ar >> 1) & 1);
  int acol = m0 + ((((lane % LPR) >> 2) ^ asw) * 4 + (lane & 3)) * 8;
  if (ATR && acol >= ly.d_in) acol = 0;
  const uint32_t* const idx = g.rowidx + kbase;
  uint32_t ai[NIA];
  uint16_t* const idx_ring = smem + Cfg::smem(RING) + wave * 128;
  const uint32_t idx_dma = lds_offset(idx_ring);
  const int ip = lane % (RPR * NIA);                       // this lane's entry of a request of indices: request ip / RPR, row ip % RPR
  const uint32_t* const idx_src = idx + RPR * (wave + NW * (ip / RPR)) + ip % RPR;
  const int idx_at = (lane / LPR) * 2;                     // (in elements of 2 bytes)
  if (!ATR) {
#pragma unroll
    for (int i = 0; i < NIA; ++i) pa[i] = ly.A + (size_t)(m0 + rq + 8 * NW * i) * ly.lda + kbase + c8;
  }
  const uint32_t dma = lds_offset(smem) + (uint32_t)wave * 1024u;
#define ABS_STEP_DMA(ks_, st_)                                                                                        \
  {                                                                                                                   \
    const uint32_t a_ = dma + (uint32_t)(st_) * (Cfg::kStage * 2);                                                    \
    _Pragma("unroll") for (int i = 0; i < NIA; ++i)                                                                   \
      lds_dma16_at(ATR ? ly.A + (size_t)ai[i] * ly.lda + acol : pa[i] + (ks_) * BK, a_ + i * NW * 1024);              \
    _Pragma("unroll") for (int i = 0; i < NIB; ++i)                                                                   \
      lds_dma16_at(pb[i] + (ks_) * BK, a_ + TMx * BK * 2 + i * NW * 1024);                                            \
  }
#define ABS_STEP_IDX(ks_) if (ATR) lds_dma4_at(idx_src + (size_t)min(ks_, nks - 1) * BK, idx_dma + (uint32_t)((ks_) & 3) * (NW * 256));

  // The model elements of the lane's own blocks, asked for before everything else where there are registers for them.
  constexpr bool kEarly = OWN == 1;
  const float* const cur = ly.cur + (g.sel == 0 ? (size_t)0 : (size_t)(g.sel == 1 ? (uint32_t)z : rd.w[z].slot) * g.stride);
  float* const next = ly.next + (size_t)z * g.stride;
  const int lk = lane >> 5, lcol = lane & 31, lrow4 = lk * 4;
  float wv[OWN][16];
  auto load_model = [&]() {
#pragma unroll
    for (int j = 0; j < OWN; ++j) {
      const int b = kg * OWN + j;
      const int i0 = m0 + wm * 64 + (b >> 1) * 32 + lrow4, n = n0 + wn * 64 + (b & 1) * 32 + lcol;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = i0 + (r >> 2) * 8 + (r & 3);
        wv[j][r] = i < ly.d_in && n < ly.d_out ? cur[(size_t)i * ly.d_out + n] : 0.f;
      }
    }
  };
  if (kEarly) load_model();
  f32x16_t acc[4];                       // block 2 mi + ni of the 64 x 64 sub-tile
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
  const int lr = lane & 31;
  const int fa = (wm * 64 + lr) * BK, fb = TMx * BK + (wn * 64 + lr) * BK;
  const int sw = (lr >> 1) & 7;
  // transposing reads: 16 lanes take 4 k rows x 16 columns; lanes 0-15 / 16-31 the block's columns 0-15 / 16-31 of k rows
  // 0 .. 7 of a 16-wide sub-step, lanes 32-63 of rows 8 .. 15 (two reads of 4 rows each)
  const int t16 = lane & 15, tr = t16 >> 2, th = (lane >> 4) & 1;
  constexpr int SUB = 4 / KG;            // 16-wide sub-steps of a k-step per wavefront group
  if (ATR) {
    uint32_t a0[RING - 1][NIA];
#pragma unroll
    for (int j = 0; j < RING - 1; ++j)
#pragma unroll
      for (int i = 0; i < NIA; ++i) a0[j][i] = idx[(size_t)min(j, nks - 1) * BK + ar + RPR * NW * i];
    uint32_t an[NIA];
#pragma unroll
    for (int i = 0; i < NIA; ++i) an[i] = idx[(size_t)min(RING - 1, nks - 1) * BK + ar + RPR * NW * i];
    ABS_STEP_IDX(RING); ABS_STEP_IDX(RING + 1); ABS_STEP_IDX(RING + 2);
#pragma unroll
    for (int j = 0; j < RING - 1; ++j) {
#pragma unroll
      for (int i = 0; i < NIA; ++i) ai[i] = a0[j][i];
      if (j < nks) ABS_STEP_DMA(j, j);
    }
#pragma unroll
    for (int i = 0; i < NIA; ++i) ai[i] = an[i];
  } else {
#pragma unroll
    for (int j = 0; j < RING - 1; ++j)
      if (j < nks) ABS_STEP_DMA(j, j);
  }
  int stage = 0;
  for (int ks = 0; ks < nks; ++ks) {
    if (ks + RING - 1 <= nks) ring_wait_barrier<(RING - 2) * (NIA + NIB)>();   // step ks has landed for every wavefront; and
    else                      ring_wait_barrier<0>();                          // everybody is done with step ks - 1
    if (ks + RING - 1 < nks) {
      ABS_STEP_IDX(ks + RING + 3);
      ABS_STEP_DMA(ks + RING - 1, stage == 0 ? RING - 1 : stage - 1);
      if (ATR) {
#pragma unroll
        for (int i = 0; i < NIA; ++i) ai[i] = *(const uint32_t*)(idx_ring + ((ks + RING) & 3) * (NW * 128) + i * RPR * 2 + idx_at);
      }
    }
    const uint16_t* sS = smem + stage * Cfg::kStage;
    stage = stage + 1 == RING ? 0 : stage + 1;
    bf16x8_t va[SUB][2], vb[SUB][2];
#pragma unroll
    for (int s = 0; s < SUB; ++s) {
      const int sub = kg * SUB + s;
      const int ch = (((sub << 1) | lk) ^ sw) << 3;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (ATR) {
          typedef short s16x4_ __attribute__((ext_vector_type(4)));
          const int row = sub * 16 + lk * 8 + tr;
          const int f0 = TMx == 128 ? (row & 3) : ((row >> 1) & 1);            // (rows 4 apart: the same swizzle)
          const uint16_t* q = sS + row * TMx + ((wm * 2 + i) ^ f0) * 32 + th * 16 + (t16 & 3) * 4;
          union { s16x4_ h[2]; bf16x8_t v; } u;
          u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_*)(q));
          u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_*)(q + 4 * TMx));
          va[s][i] = u.v;
        } else {
          va[s][i] = *(const bf16x8_t*)&sS[fa + i * 32 * BK + ch];
        }
        vb[s][i] = *(const bf16x8_t*)&sS[fb + i * 32 * BK + ch];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[2 * i + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[s][i], vb[s][j], acc[2 * i + j], 0, 0, 0);
    }
  }
#undef ABS_STEP_DMA
#undef ABS_STEP_IDX

  // ---- epilogue.  Accumulator register r of lane l holds C[8 (r/4) + 4 (l/32) + r%4][l%32] of its block.
  if (!kEarly) load_model();
  float* const red = (float*)smem;
  uint16_t* const sT = smem;                               // results [n][kPitchT]
  uint16_t* const sN = smem + TNx * Cfg::kPitchT;          // results [m][kPitchN]
  __syncthreads();                                         // all fragment reads done before LDS is reused
  // blocks of other groups to their owners: [sub-tile][block][source group][quarter][lane]
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int owner = b / OWN;
    if (owner != kg) {
      float4* q = (float4*)(red + ((wsub * 4 + b) * (KG - 1) + (kg < owner ? kg : kg - 1)) * 1024) + lane;
#pragma unroll
      for (int r = 0; r < 4; ++r) q[r * 64] = make_float4(acc[b][4 * r], acc[b][4 * r + 1], acc[b][4 * r + 2], acc[b][4 * r + 3]);
    }
  }
  f32x16_t fin[OWN];
#pragma unroll
  for (int b = 0; b < 4; ++b)
    if (b / OWN == kg) fin[b % OWN] = acc[b];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < OWN; ++j) {
    const float4* q = (const float4*)(red + (wsub * 4 + kg * OWN + j) * (KG - 1) * 1024) + lane;
#pragma unroll
    for (int o = 0; o < KG - 1; ++o)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float4 v = q[o * 256 + r * 64];
        fin[j][4 * r] += v.x; fin[j][4 * r + 1] += v.y; fin[j][4 * r + 2] += v.z; fin[j][4 * r + 3] += v.w;
      }
  }
  __syncthreads();                                         // the exchanged blocks have been read
#pragma unroll
  for (int j = 0; j < OWN; ++j) {
    const int b = kg * OWN + j;
    const int bm = wm * 64 + (b >> 1) * 32, nl = wn * 64 + (b & 1) * 32 + lcol, n = n0 + nl;
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      const int ml = bm + rg * 8 + lrow4;
      uint16_t h[4];
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int i = m0 + ml + rr;
        const bool ok = i < ly.d_in && n < ly.d_out;       // padding stays zero in both copies
        const float v = ok ? wv[j][rg * 4 + rr] - fin[j][rg * 4 + rr] : 0.f;
        if (ok) next[(size_t)i * ly.d_out + n] = v;
        h[rr] = f32_to_bf16(v);
        if (ly.wn) sN[(ml + rr) * Cfg::kPitchN + nl] = h[rr];
      }
      uint2 o;
      o.x = h[0] | ((uint32_t)h[1] << 16);
      o.y = h[2] | ((uint32_t)h[3] << 16);
      *(uint2*)&sT[nl * Cfg::kPitchT + ml] = o;
    }
  }
  __syncthreads();
  uint16_t* const wt = ly.wt + (size_t)z * g.shadow_stride;
#pragma unroll
  for (int i = 0; i < TMx * TNx / 8 / NT; ++i) {
    const int q = t + NT * i, nl = q / (TMx / 8), ch = (q % (TMx / 8)) * 8;
    if (n0 + nl < ly.d_out) *(uint4*)(wt + (size_t)(n0 + nl) * ly.ldwt + m0 + ch) = *(const uint4*)&sT[nl * Cfg::kPitchT + ch];
  }
  if (ly.wn) {
    uint16_t* const wr = ly.wn + (size_t)z * g.shadow_stride;
#pragma unroll
    for (int i = 0; i < TMx * TNx / 8 / NT; ++i) {
      const int q = t + NT * i, ml = q / (TNx / 8), ch = (q % (TNx / 8)) * 8;
      // (a tile may be wider than dp_out, by up to half: zeros into the rows' pad)
      static_assert(TNx - 64 <= kPitchPad, "the pad holds what a tile has beyond the narrowest layer");
      if (m0 + ml < ly.d_in) *(uint4*)(wr + (size_t)(m0 + ml) * ly.ldwn + n0 + ch) = *(const uint4*)&sN[ml * Cfg::kPitchN + ch];
    }
  }
}

template <int TMx, int TNx, int NW, int RING, int PER_SIMD, bool DIRECT>
__global__ __launch_bounds__(NW * 64, PER_SIMD) void mlp_step_kernel(StepArgs g, RoundDesc rd) {
  using Cfg = StepCfg<TMx, TNx, NW>;
  __shared__ __attribute__((aligned(16))) uint16_t smem[Cfg::smem(RING) + (DIRECT ? Cfg::kIdx : 0)];
  static_assert((Cfg::smem(RING) + Cfg::kIdx) * 2 * (PER_SIMD * 4 / NW) <= 160 * 1024, "LDS budget");
  const int bx = blockIdx.x;
  int l = 0, first = 0;
#pragma unroll
  for (int q = 1; q < 8; ++q)
    if (q <= g.L && bx >= g.first[q]) { l = q; first = g.first[q]; }
  if (l == g.L) {
    const int b = bx - first, up = b / g.bias_per;
    const BiasCore& u = g.bias;
    const size_t from = g.sel == 0 ? (size_t)0 : (size_t)(g.sel == 1 ? (uint32_t)up : rd.w[up].slot) * g.stride;
    bias_block(u, b - up * g.bias_per, [&](int l) { return up * u.prow[l]; }, u.w_cur + from, u.w_next + (size_t)up * g.stride, (float*)smem);
    return;
  }
  const StepLayer ly = g.l[l];
  // the tiles (upload, row, column: columns fastest) in eight contiguous ranges, one per XCD
  const int b = bx - first, tiles = g.uploads * ly.mt * ly.nt, per = (tiles + 7) >> 3;
  const int idx = (b & 7) * per + (b >> 3);
  if ((b >> 3) >= per || idx >= tiles) return;
  const int n0 = (idx % ly.nt) * TNx, row = idx / ly.nt, m0 = (row % ly.mt) * TMx, z = row / ly.mt;
  if constexpr (DIRECT) {
    if (l == 0) { step_tile<TMx, TNx, NW, RING, true>(g, ly, rd, z, m0, n0, smem); return; }
  }
  step_tile<TMx, TNx, NW, RING, false>(g, ly, rd, z, m0, n0, smem);
}

// ------------------------------------------------------------------ output layer: logits, loss, dZ_L
// The last layer's product, the softmax cross-entropy and the output gradient in one kernel: the
// class count is at most 256, so a workgroup that owns 128 stacked rows owns their whole logit rows
// and nothing of Z_L ever goes to memory.  The product is narrow (few classes) and long (the last
// hidden width): what bounds it is how many bytes a CU keeps in flight, so the 64-wide k-steps of
// the A tile (128 rows of H_{L-1}) and the B tile (all classes of W_L^T) go from global memory
// straight into a ring of LDS stages (global_load_lds_dwordx4, swizzled on the global side as in the
// large-tile GEMM), kStages - 1 steps ahead of their use, one barrier per step.  Wavefront w owns
// rows 32 w .. 32 w + 31 and all classes, and multiplies the other way round - W_L^T is the
// MFMA's row operand, the activations its column operand - so that the 32x32 blocks hold Z_L^T:
// accumulator register r of lane l is class 32 b + 8 (r / 4) + 4 (l / 32) + r % 4 of row l % 32.
// All classes of a row then sit in the registers of two lanes (l and l + 32), and its softmax is
// arithmetic inside a lane plus one exchange, instead of a 32-lane reduction per row and class.
// Outputs: dZ_L = c_k (softmax - onehot) narrowed to bf16 (zero in padding rows and classes) in
// both orientations, the 128 rows' loss sum, and the column sums of the narrowed dZ_L (the bias
// gradient's share of these rows).
constexpr int kCeRows = 128;             // stacked rows per workgroup of the output-layer kernel

struct LogitsCeArgs {
  const uint16_t* H; size_t ldh;         // H_{L-1} [rows][ldh]
  int ksteps;                            // dp_{L-1} / 64
  const uint16_t* Wt; size_t ldw;        // W_L^T [dp_L][ldw] inside a shadow slot
  size_t w_slot_stride;
  const float* bias; size_t bias_slot_stride;
  int C;                                 // classes (columns >= C are padding)
  int rows_per_upload, by_upload;
  const int32_t* label;                  // -1: padding row
  uint16_t* dZ; size_t lddz;             // [rows][lddz]
  uint16_t* dZT; size_t lddzt;           // [dp_L][lddzt]
  float* rowloss;                        // [rows / 128]
  float* colsum; size_t ldcs;            // [rows / 128][ldcs]
  GatherT gt;                            // its blocks are the launch's last workgroups
};

template <int NB>                        // dp_L = 32 NB: 2, 4 or 8
__global__ __launch_bounds__(256, 1) void mlp_logits_ce_kernel(LogitsCeArgs a, RoundDesc rd) {
  constexpr int NP = 32 * NB;            // padded class count
  constexpr int kStageElems = (kCeRows + NP) * BK;
  constexpr int kStages = NB == 8 ? 3 : 4;
  constexpr int kPitchD = NP + 8;        // narrowed dZ tile, bf16 [128][kPitchD], after the main loop ...
  constexpr int kPitchT = kCeRows + 8;   // ... and its transpose, bf16 [NP][kPitchT], behind it
  static_assert(kStages * kStageElems >= kCeRows * kPitchD + NP * kPitchT, "staging fits the ring");
  static_assert(kStages * kStageElems * 2 <= 150 * 1024, "LDS budget");
  constexpr int kDmaPerWave = 4 + NB;    // requests per wavefront and stage (8 rows of 128 bytes each)
  __shared__ __attribute__((aligned(16))) uint16_t smem[kStages * kStageElems];
  __shared__ float s_l[4];
  __shared__ __attribute__((aligned(16))) float s_bias[NP];
  static_assert(kStages * kStageElems >= 64 * kGatherPitch, "a gather block fits the ring");
  if (const int own = (int)gridDim.x - a.gt.blocks; (int)blockIdx.x >= own) {
    gather_t_block(a.gt, (int)blockIdx.x - own, smem);
    return;
  }
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int m0 = blockIdx.x * kCeRows;
  const int up = m0 / a.rows_per_upload;
  const uint32_t slot = a.by_upload ? (uint32_t)up : rd.w[up].slot;
  const float coef = rd.w[up].c;
  const uint16_t* Wt = a.Wt + (size_t)slot * a.w_slot_stride;

  // requests of this wavefront: its own 32 rows of A (4 requests) and NP / 4 rows of B (NB requests);
  // lane l of a request fills position l & 7 of row r8 + (l >> 3) with chunk (l & 7) ^ ((row >> 1) & 7)
  const int lr = lane >> 3, lp = lane & 7;
  const uint16_t* ga[4]; const uint16_t* gb[NB];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = wave * 32 + 8 * i + lr;
    ga[i] = a.H + (size_t)(m0 + row) * a.ldh + ((lp ^ ((row >> 1) & 7)) << 3);
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int row = wave * (NP / 4) + 8 * i + lr;
    gb[i] = Wt + (size_t)row * a.ldw + ((lp ^ ((row >> 1) & 7)) << 3);
  }
  uint16_t* const dmaA = smem + (wave * 32) * BK;
  uint16_t* const dmaB = smem + kCeRows * BK + (wave * (NP / 4)) * BK;
#define ABS_CE_DMA(ks_)                                                            \
  {                                                                                \
    const int k0_ = (ks_) * BK;                                                    \
    uint16_t* st_ = smem + ((ks_) % kStages) * kStageElems;                        \
    _Pragma("unroll") for (int i = 0; i < 4; ++i)                                  \
      lds_dma16_raw(ga[i] + k0_, st_ + (dmaA - smem) + i * 512);                   \
    _Pragma("unroll") for (int i = 0; i < NB; ++i)                                 \
      lds_dma16_raw(gb[i] + k0_, st_ + (dmaB - smem) + i * 512);                   \
  }
  f32x16_t acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
  const int l32 = lane & 31, lk = lane >> 5;
  const int sw = (l32 >> 1) & 7;
  const int fa_row = (wave * 32 + l32) * BK, fb_row = kCeRows * BK + l32 * BK;
  const int nk = a.ksteps;
  // what the epilogue needs from memory is requested before the main loop: the label of the lane's
  // row, and the biases, which wait in LDS (padding classes: -inf, so they drop out of max and sum)
  const int lab = a.label[m0 + wave * 32 + l32];
  if (t < NP) s_bias[t] = t < a.C ? (a.bias + (size_t)slot * a.bias_slot_stride)[t] : -INFINITY;
#pragma unroll
  for (int st = 0; st < kStages - 1; ++st)
    if (st < nk) ABS_CE_DMA(st);
  for (int ks = 0; ks < nk; ++ks) {
    // this wavefront's requests of step ks have landed once at most those of the steps behind it
    // (kStages - 2 of them, kDmaPerWave requests each) are still in flight; near the end: all
    if (ks + kStages - 2 < nk) __builtin_amdgcn_s_waitcnt(0x0F70 | (((kStages - 2) * kDmaPerWave) & 15) |
                                                          ((((kStages - 2) * kDmaPerWave) >> 4) << 14));
    else                       __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();                     // everybody's part of step ks is in LDS; everybody is done with step ks - 1
    if (ks + kStages - 1 < nk) ABS_CE_DMA(ks + kStages - 1);
    const uint16_t* sS = smem + (ks % kStages) * kStageElems;
    // fragments of sub-step s + 1 are read while the MFMAs of sub-step s run
    bf16x8_t fa[2], fb[2][NB];
#define ABS_CE_FRAGS(set, s_)                                                      \
  {                                                                                \
    const int ch_ = ((((s_) << 1) | lk) ^ sw) << 3;                                \
    fa[set] = *(const bf16x8_t*)&sS[fa_row + ch_];                                 \
    _Pragma("unroll") for (int b = 0; b < NB; ++b)                                 \
      fb[set][b] = *(const bf16x8_t*)&sS[fb_row + b * 32 * BK + ch_];              \
  }
    ABS_CE_FRAGS(0, 0);
#pragma unroll
    for (int sub = 0; sub < 4; ++sub) {
      if (sub < 3) ABS_CE_FRAGS((sub + 1) & 1, sub + 1);
#pragma unroll
      for (int b = 0; b < NB; ++b)
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[sub & 1][b], fa[sub & 1], acc[b], 0, 0, 0);
    }
#undef ABS_CE_FRAGS
    // issue order: the first fragment set, then per sub-step one read ahead and one read behind each MFMA
    __builtin_amdgcn_sched_group_barrier(0x100, 1 + NB, 0);
#pragma unroll
    for (int sub = 0; sub < 3; ++sub) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    }
    __builtin_amdgcn_sched_group_barrier(0x008, NB, 0);
  }
#undef ABS_CE_DMA
  __syncthreads();                       // all fragment reads done before the ring is reused for staging

  // ---- softmax cross-entropy: the lane's 16 NB classes of row l % 32, its partner holds the rest
  uint16_t* const sD = smem;             // [128][kPitchD]
  uint16_t* const sT = smem + kCeRows * kPitchD;       // [NP][kPitchT]
  const int ml = wave * 32 + l32;
  float zmax = -INFINITY;
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 bq = *(const float4*)&s_bias[b * 32 + q * 8 + lk * 4];
      acc[b][q * 4 + 0] += bq.x; acc[b][q * 4 + 1] += bq.y; acc[b][q * 4 + 2] += bq.z; acc[b][q * 4 + 3] += bq.w;
#pragma unroll
      for (int e = 0; e < 4; ++e) zmax = fmaxf(zmax, acc[b][q * 4 + e]);
    }
  zmax = fmaxf(zmax, __shfl_xor(zmax, 32, 64));
  const int lrel = lab - lk * 4;         // the label relative to this half's class offset
  float ssum = 0.f, zy = 0.f;
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float dz = acc[b][r] - zmax;
      zy = (b * 32 + (r >> 2) * 8 + (r & 3) == lrel) ? dz : zy;
      acc[b][r] = __expf(dz);
      ssum += acc[b][r];
    }
  ssum += __shfl_xor(ssum, 32, 64);
  zy += __shfl_xor(zy, 32, 64);
  float lsum = lab >= 0 ? logf(ssum) - zy : 0.f;       // this row's loss (same in both of its lanes)
  const float cr = lab >= 0 ? coef : 0.f;              // c_k (softmax - onehot), zero for padding rows
  const float scale = cr / ssum;
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint16_t h[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = acc[b][q * 4 + e] * scale - ((b * 32 + q * 8 + e == lrel) ? cr : 0.f);
        h[e] = __builtin_bit_cast(uint16_t, (__bf16)v);
        sT[(b * 32 + q * 8 + lk * 4 + e) * kPitchT + ml] = h[e];       // (32 lanes: 64 contiguous bytes)
      }
      uint2 o;
      o.x = h[0] | ((uint32_t)h[1] << 16);
      o.y = h[2] | ((uint32_t)h[3] << 16);
      *(uint2*)&sD[ml * kPitchD + b * 32 + q * 8 + lk * 4] = o;
    }
  // the 32 rows of the wavefront (lanes of a half), then the four wavefronts, always in this order
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o, 64);
  if (lane == 0) s_l[wave] = lsum;
  __syncthreads();
  if (t == 0) a.rowloss[blockIdx.x] = (s_l[0] + s_l[1]) + (s_l[2] + s_l[3]);
  // row-major copy: 16-byte pieces, NP / 8 per row
  for (int q = t; q < kCeRows * (NP / 8); q += 256) {
    const int row = q / (NP / 8), ch = q % (NP / 8);
    *(uint4*)(a.dZ + (size_t)(m0 + row) * a.lddz + ch * 8) = *(const uint4*)&sD[row * kPitchD + ch * 8];
  }
  // transposed copy: class n, 16-byte pieces of 8 consecutive rows
  for (int q = t; q < NP * (kCeRows / 8); q += 256) {
    const int n = q / (kCeRows / 8), rb8 = (q % (kCeRows / 8)) * 8;
    *(uint4*)(a.dZT + (size_t)n * a.lddzt + m0 + rb8) = *(const uint4*)&sT[n * kPitchT + rb8];
  }
  // the bias gradient's share of these 128 rows: class n's narrowed values added in row order
  for (int n = t; n < NP; n += 256) {
    float c = 0.f;
#pragma unroll 4
    for (int p8 = 0; p8 < kCeRows / 8; ++p8) {
      const uint4 v = *(const uint4*)&sT[n * kPitchT + p8 * 8];
      c += __uint_as_float(v.x << 16); c += __uint_as_float(v.x & 0xFFFF0000u);
      c += __uint_as_float(v.y << 16); c += __uint_as_float(v.y & 0xFFFF0000u);
      c += __uint_as_float(v.z << 16); c += __uint_as_float(v.z & 0xFFFF0000u);
      c += __uint_as_float(v.w << 16); c += __uint_as_float(v.w & 0xFFFF0000u);
    }
    a.colsum[(size_t)blockIdx.x * a.ldcs + n] = c;
  }
}

// The same for rounds of few rows (ce_rows), where the kernel above leaves most CUs idle and each busy one waits for its own
// long stream of tiles (0.9 us a k-step of 64, bound by what one CU has in flight: some 32 KB).  A workgroup owns 32 rows,
// its four wavefronts share the CONTRACTION (pairs of 32-wide sub-steps p, p + 4, ...), and operands go from memory straight
// into registers, the next pair's on their way under this one's products.  The four partial logits meet in LDS, summed in
// wavefront order; then a wavefront has 8 whole rows, 16 lanes to a row.
// us, 128-row / 32-row workgroups: 1024 x 512, 10 classes 9.0 / 6.7, 4096 x 1024 12.9 / 7.8, 1152 x 300, 26 classes 8.2 / 6.5,
// 8192 x 2048, 100 classes 33 / 25.  Eight wavefronts to the contraction: 7.3 instead of 7.8 for 4096 x 1024, but 46
// for the last one (more lines asked for than the L1 can hold until their other half is).
constexpr int kCeFewRows = 32;
template <int CB>                        // blocks of 16 classes that are computed: 16 CB >= C, at most 8
__global__ __launch_bounds__(256, 1) void mlp_logits_ce_few_kernel(LogitsCeArgs a, RoundDesc rd) {
  constexpr int kBlk = 320;              // floats of a block of partial logits: 64 x 4, quarter-wavefronts 16 further apart
  constexpr int kRedFloats = 4 * 2 * CB * kBlk;
  constexpr int NP = CB <= 4 ? 64 : 128; // padded class count dp_L
  constexpr int kPitchD = NP + 8, kPitchT = kCeFewRows + 8;
  constexpr int kSmemBytes = kRedFloats * 4 > 64 * kGatherPitch * 2 ? kRedFloats * 4 : 64 * kGatherPitch * 2;
  __shared__ __attribute__((aligned(16))) unsigned char smem_raw[kSmemBytes];
  __shared__ __attribute__((aligned(16))) uint16_t sD[kCeFewRows * kPitchD], sT[NP * kPitchT];
  __shared__ float s_loss[kCeFewRows];
  if (const int own = (int)gridDim.x - a.gt.blocks; (int)blockIdx.x >= own) {
    gather_t_block(a.gt, (int)blockIdx.x - own, (uint16_t*)smem_raw);
    return;
  }
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int m0 = blockIdx.x * kCeFewRows;
  const int up = m0 / a.rows_per_upload;
  const uint32_t slot = a.by_upload ? (uint32_t)up : rd.w[up].slot;
  const float coef = rd.w[up].c;
  const int l16 = lane & 15, lq = lane >> 4;
  const uint16_t* const ph = a.H + (size_t)(m0 + l16) * a.ldh + lq * 8;
  const uint16_t* const pw = a.Wt + (size_t)slot * a.w_slot_stride + (size_t)l16 * a.ldw + lq * 8;
  f32x4_t acc[2][CB];
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[0][b][r] = acc[1][b][r] = 0.f;
  struct Frags { bf16x8_t h[2][2], w[CB][2]; };
  auto load = [&](Frags& f, int p) {
    const size_t k0 = (size_t)p * BK;    // (the two halves of a 128-byte line one after the other: the second finds it in the L1)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) f.h[i][s] = *(const bf16x8_t*)(ph + (size_t)(16 * i) * a.ldh + k0 + 32 * s);
#pragma unroll
    for (int b = 0; b < CB; ++b)
#pragma unroll
      for (int s = 0; s < 2; ++s) f.w[b][s] = *(const bf16x8_t*)(pw + (size_t)(16 * b) * a.ldw + k0 + 32 * s);
  };
  auto multiply = [&](const Frags& f) {  // block (i, b): class 16 b + 4 (l / 16) + r of row 16 i + l % 16
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int b = 0; b < CB; ++b)
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[b][s], f.h[i][s], acc[i][b], 0, 0, 0);
  };
  Frags f0, f1;
  int p = wave;
  if (p < a.ksteps) load(f0, p);
  // what the epilogue needs from memory: labels and biases (padding classes -inf: they drop out of max and sum)
  int lab[2]; float bias[CB];
#pragma unroll
  for (int q = 0; q < 2; ++q) lab[q] = a.label[m0 + wave * 8 + q * 4 + lq];
#pragma unroll
  for (int b = 0; b < CB; ++b) bias[b] = b * 16 + l16 < a.C ? (a.bias + (size_t)slot * a.bias_slot_stride)[b * 16 + l16] : -INFINITY;
  while (p < a.ksteps) {
    if (p + 4 < a.ksteps) load(f1, p + 4);
    multiply(f0);
    p += 4;
    if (p >= a.ksteps) break;
    if (p + 4 < a.ksteps) load(f0, p + 4);
    multiply(f1);
    p += 4;
  }
  float* const red = (float*)smem_raw;   // [wavefront][i][b][kBlk]
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int b = 0; b < CB; ++b)
      *(f32x4_t*)&red[((wave * 2 + i) * CB + b) * kBlk + lane * 4 + lq * 16] = acc[i][b];
  __syncthreads();
  // row 8 wave + 4 q + lq of the workgroup, classes l16, l16 + 16, ...
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int ml = wave * 8 + q * 4 + lq;
    const float* const at_row = red + (size_t)(ml >> 4) * CB * kBlk + (l16 >> 2) * 80 + (ml & 15) * 4 + (l16 & 3);
    float z[CB], zmax = -INFINITY;
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      float v = at_row[b * kBlk];
#pragma unroll
      for (int w = 1; w < 4; ++w) v += at_row[(w * 2 * CB + b) * kBlk];
      z[b] = v + bias[b];
      zmax = fmaxf(zmax, z[b]);
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, o, 64));
    float ssum = 0.f, zy = 0.f;
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const float dz = z[b] - zmax;
      zy = b * 16 + l16 == lab[q] ? dz : zy;
      z[b] = __expf(dz);
      ssum += z[b];
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) { ssum += __shfl_xor(ssum, o, 64); zy += __shfl_xor(zy, o, 64); }
    const float cr = lab[q] >= 0 ? coef : 0.f;             // c_k (softmax - onehot), zero for padding rows
    const float scale = cr / ssum;
    if (l16 == 0) s_loss[ml] = lab[q] >= 0 ? logf(ssum) - zy : 0.f;
#pragma unroll
    for (int b = 0; b < NP / 16; ++b) {
      const float v = b < CB ? z[b < CB ? b : 0] * scale - (b * 16 + l16 == lab[q] ? cr : 0.f) : 0.f;
      const uint16_t h = __builtin_bit_cast(uint16_t, (__bf16)v);
      sD[ml * kPitchD + b * 16 + l16] = h;
      sT[(b * 16 + l16) * kPitchT + ml] = h;
    }
  }
  __syncthreads();
  if (t == 0) {
    float l = 0.f;
#pragma unroll
    for (int r = 0; r < kCeFewRows; ++r) l += s_loss[r];
    a.rowloss[blockIdx.x] = l;
  }
  for (int q = t; q < kCeFewRows * (NP / 8); q += 256) {
    const int row = q / (NP / 8), ch = q % (NP / 8);
    *(uint4*)(a.dZ + (size_t)(m0 + row) * a.lddz + ch * 8) = *(const uint4*)&sD[row * kPitchD + ch * 8];
  }
  for (int q = t; q < NP * (kCeFewRows / 8); q += 256) {
    const int n = q / (kCeFewRows / 8), rb8 = (q % (kCeFewRows / 8)) * 8;
    *(uint4*)(a.dZT + (size_t)n * a.lddzt + m0 + rb8) = *(const uint4*)&sT[n * kPitchT + rb8];
  }
  if (t < NP) {                          // the bias gradient's share of these rows, in row order
    float c = 0.f;
#pragma unroll
    for (int p8 = 0; p8 < kCeFewRows / 8; ++p8) {
      const uint4 v = *(const uint4*)&sT[t * kPitchT + p8 * 8];
      c += __uint_as_float(v.x << 16); c += __uint_as_float(v.x & 0xFFFF0000u);
      c += __uint_as_float(v.y << 16); c += __uint_as_float(v.y & 0xFFFF0000u);
      c += __uint_as_float(v.z << 16); c += __uint_as_float(v.z & 0xFFFF0000u);
      c += __uint_as_float(v.w << 16); c += __uint_as_float(v.w & 0xFFFF0000u);
    }
    a.colsum[(size_t)blockIdx.x * a.ldcs + t] = c;
  }
}

// ------------------------------------------------------------------ update + snapshot
// The update as a kernel of its own (a TileUpdate for a whole matrix): the averaged change of the uploads
// of local SGD, matrices whose rows are not 16-byte aligned, a round's last layer, the bf16 copies of w^0.
// (With a per-upload form that moved its argument's pointers the whole argument lived in scratch memory: a
// 512 x 10 layer 7.5 us instead of 3.3.)
template <int TJ>
__global__ __launch_bounds__(256) void mlp_update_kernel(TileUpdate u) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[64 * (TJ + 2)];
  update_block64<256, TJ>(u, blockIdx.y * 64, blockIdx.x * TJ, tile);
}

// Element-wise version for narrow or odd output widths (e.g. the 10-class output layer):
// one thread per weight, four partial loads in flight.
__global__ __launch_bounds__(256) void mlp_update_small_kernel(TileUpdate u) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= u.d_in * u.d_out) return;
  const int i = e / u.d_out, j = e - i * u.d_out;
  const float* pp = u.partial + (size_t)i * u.ldp + j;
  float G = 0.f;
  int z = 0;
  for (; z + 4 <= u.nsplit; z += 4) {
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = pp[(size_t)(z + q) * u.split_stride];
#pragma unroll
    for (int q = 0; q < 4; ++q) G += v[q];
  }
  for (; z < u.nsplit; ++z) G += pp[(size_t)z * u.split_stride];
  const float wnew = u.w_cur[e] - G;
  u.w_next[e] = wnew;
  const uint16_t h = f32_to_bf16(wnew);
  if (u.wn) u.wn[(size_t)i * u.ldwn + j] = h;
  u.wt[(size_t)j * u.ldwt + i] = h;
}

// ------------------------------------------------------------------ local SGD helpers
// Eq. 3 over the uploads: D = (1/K) sum_a (w^{t - tau_a} - w_a^{U}) in arrival order, for every
// parameter; bias entries are applied right away, weight matrices go through the update kernels
// (which also refresh the bf16 copies).
struct DeltaArgs {
  const float* ring; size_t slot_stride;
  const float* priv;
  float* D;
  size_t P;
  int L;
  size_t b_off[ABS_MAX_LAYERS]; int b_len[ABS_MAX_LAYERS];
  const float* w_cur; float* w_next;
};
__global__ __launch_bounds__(256) void mlp_delta_kernel(DeltaArgs a, RoundDesc rd) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.P) return;
  float s = 0.f;
  for (int up = 0; up < rd.K; ++up)
    s += a.ring[(size_t)rd.w[up].slot * a.slot_stride + i] - a.priv[(size_t)up * a.slot_stride + i];
  const float d = s / (float)rd.K;
  a.D[i] = d;
  for (int l = 0; l < a.L; ++l)
    if (i >= a.b_off[l] && i < a.b_off[l] + (size_t)a.b_len[l]) a.w_next[i] = a.w_cur[i] - d;
}

__global__ void mlp_fill_zero_kernel(uint4* p, size_t n16) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t step = (size_t)gridDim.x * blockDim.x;
  for (; i < n16; i += step) p[i] = make_uint4(0, 0, 0, 0);
}

// ------------------------------------------------------------------ held-out evaluation
// Sequential evaluation rows row0 .. row0 + n in the index arrays of the forward pass (x_row0: where row row0 is in
// the matrix that pass reads); the padding rows read a valid row and carry label -1.
__global__ void mlp_eval_index_kernel(uint32_t* rowidx, int32_t* label, const int32_t* y, int64_t row0, int64_t x_row0, int n,
                                      int rows) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= rows) return;
  rowidx[m] = (uint32_t)(x_row0 + (m < n ? m : 0));
  label[m] = m < n ? y[row0 + m] : -1;
}

// A pass's rows from a caller's matrix that is not 16-byte aligned (a view into a larger buffer): the forward pass
// requests 16-byte pieces straight into LDS, which need the alignment, so the rows go through the workspace.
__global__ void mlp_eval_align_kernel(const uint16_t* X, uint4* out, size_t n8) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n8) return;
  const uint16_t* v = X + i * 8;
  uint4 o;
  o.x = v[0] | ((uint32_t)v[1] << 16); o.y = v[2] | ((uint32_t)v[3] << 16);
  o.z = v[4] | ((uint32_t)v[5] << 16); o.w = v[6] | ((uint32_t)v[7] << 16);
  out[i] = o;
}

// One wavefront per row of the logits: -log softmax(z)_y and whether the first largest logit
// is the label.  NC = logits width / 64.
template <int NC>
__global__ __launch_bounds__(256) void mlp_eval_rows_kernel(const float* Z, size_t ldz, int C, const int32_t* label,
                                                            int n, float* rowloss, float* correct) {
  const int lane = threadIdx.x & 63;
  const int m = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (m >= n) return;
  const int lab = label[m];
  float z[NC], zmax = -INFINITY;
  int best = 0;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c = lane + 64 * q;
    z[q] = c < C ? Z[(size_t)m * ldz + c] : -INFINITY;
    if (z[q] > zmax) { zmax = z[q]; best = c; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {            // largest value, lowest class among equals
    const float ov = __shfl_xor(zmax, o, 64);
    const int ob = __shfl_xor(best, o, 64);
    if (ov > zmax || (ov == zmax && ob < best)) { zmax = ov; best = ob; }
  }
  float ssum = 0.f, zy = 0.f;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c = lane + 64 * q;
    if (c == lab) zy = z[q] - zmax;
    ssum += c < C ? expf(z[q] - zmax) : 0.f;
  }
  ssum = wave_sum(ssum);
  zy = wave_sum(zy);
  if (lane == 0) { rowloss[m] = logf(ssum) - zy; correct[m] = best == lab ? 1.f : 0.f; }
}

template <typename T>
T* at(const MlpArgs& a, size_t off) { return (T*)(a.ws + off); }

// Number of row-range splits of a weight-gradient contraction.  `slots` workgroups run at
// once; a split costs `step_us` per k-step of its range and `fixed_us` per wave of workgroups, and every
// extra split adds a partial tile to write and read back.  Picks the cheapest under that model.
int pick_split(int tiles, int ksteps, int slots, double tile_bytes, double step_us, double fixed_us) {
  const double bytes_per_us = 3.0e6;
  int best = 1;
  double best_cost = 1e300;
  for (int z = 1; z <= std::min(ksteps, kMaxSplit); ++z) {
    const int rounds = (tiles * z + slots - 1) / slots;
    const int steps = (ksteps + z - 1) / z;
    const double cost = rounds * (steps * step_us + fixed_us) + (double)z * tiles * tile_bytes * 2.0 / bytes_per_us;
    if (cost < best_cost) { best_cost = cost; best = z; }
  }
  return best;
}

// Whether a weight gradient off the large-tile kernel takes 128-wide tiles: a long contraction that can
// still be cut into a workgroup per CU (cfg 5's output layer, 2048 x 128 over 8192 / 32768 rows: 33 / 62 us
// against 39 / 71 with 64-wide tiles, which read the activations twice; short ones are faster with 64).  Local steps are
// cut into the uploads and no further (us with 64 / 128-wide tiles, 2048 x 128: 2 uploads of 4096 rows, 32 workgroups
// of 128, 22 / 46, 64 of 128 rows 51 / 43; 512 x 2048, 2 of 4096 rows, 128 workgroups, 38 / 53; 1152 x 640, 8 of 128 rows,
// 360 workgroups, 18.7 / 14.6).
bool wgrad_wide_tiles(int Mdim, int Ndim, int ksteps, int uploads) {
  return Ndim % 128 == 0 && (Mdim / 128) * (Ndim / 128) * (uploads ? uploads : std::min(ksteps / 8, kMaxSplit)) >= 256;
}
// ... or tiles of 128 x 256: two workgroups per CU with at least 25 k-steps each, in few splits (us of this product
// and the next, which carries its update, with 128 x 128 / 128 x 256 tiles: 3200 x 2048 over 4096 rows 96 / 89, 8192:
// 185 / 147; 1920 x 2048 over 8192: 96 / 97, 16384: 181 / 161; 3200 x 512 over 16384: 77 / 86).
bool wgrad_256_columns(int Mdim, int Ndim, int ksteps) {
  const int tiles = (Mdim / 128) * (Ndim / 256);
  return Ndim % 256 == 0 && tiles >= 100 && tiles * ksteps >= 12800;
}
// Row-range splits of layer l's weight-gradient contraction over `rows` stacked rows
// (per_upload > 0: local SGD, one split per upload).
int wgrad_split(const MlpPlan& p, int l, int rows, int per_upload) {
  if (per_upload > 0) return per_upload;
  const int ksteps = rows / BK;
  if (p.dp[l] % TM3 == 0 && p.dp[l + 1] % TN3 == 0)
    return pick_split((p.dp[l] / TM3) * (p.dp[l + 1] / TN3), ksteps, 256, 256.0 * 256 * 4, 2.0, 0.0);
  if (wgrad_256_columns(p.dp[l], p.dp[l + 1], ksteps))
    return pick_split((p.dp[l] / 128) * (p.dp[l + 1] / 256), ksteps, 512, 128.0 * 256 * 4, 1.5, 0.0);
  if (wgrad_wide_tiles(p.dp[l], p.dp[l + 1], ksteps, 0))
    return pick_split((p.dp[l] / 128) * (p.dp[l + 1] / 128), ksteps, 512, 128.0 * 128 * 4, 0.5, 0.0);
  return pick_split((p.dp[l] / 64) * (p.dp[l + 1] / 64), ksteps, 512, 64.0 * 64 * 4, 0.25, 0.0);
}

}  // namespace

// ------------------------------------------------------------------ planning
bool mlp_plan(const abs_config& c, MlpPlan& p, const char** why) {
  p = MlpPlan{};
  const int L = c.n_layers;
  if (c.dims[0] % 8) { *why = "MLP: d_0 must be a multiple of 8"; return false; }
  if (c.dims[L] < 2 || c.dims[L] > 256) { *why = "MLP: 2 <= d_L <= 256"; return false; }
  for (int l = 0; l <= L; ++l)
    if (c.dims[l] < 1 || c.dims[l] > 16384) { *why = "MLP: layer widths must be in [1, 16384]"; return false; }
  p.L = L;
  for (int l = 0; l <= L; ++l) {
    p.d[l] = c.dims[l];
    p.dp[l] = (int)round_up((size_t)c.dims[l], 128);
  }
  if (c.dims[L] <= 64) p.dp[L] = 64;
  for (int l = 0; l <= L; ++l) p.ld[l] = p.dp[l] + kPitchPad;
  p.U = c.U > 1 ? c.U : 1;
  p.B = c.B;
  p.Bp = (int)round_up((size_t)c.B, TM);
  p.N = c.N;
  p.Mp = c.N * p.Bp;
  p.ldm = (size_t)p.Mp + kPitchPad;
  p.R = c.tau_cap + 3;
  size_t o = 0;
  for (int l = 0; l < L; ++l) {
    p.w_off[l] = o; o += (size_t)p.d[l] * p.d[l + 1];
    p.b_off[l] = o; o += (size_t)p.d[l + 1];
  }
  p.P = o;
  p.slot_stride = round_up(p.P, 64);
  o = 0;
  for (int l = 0; l < L; ++l) {
    p.wt_off[l] = o; o += (size_t)p.dp[l + 1] * p.ld[l];
    p.wn_off[l] = o; if (l >= 1) o += (size_t)p.dp[l] * p.ld[l + 1];
  }
  p.shadow_stride = round_up(o, 128);
  size_t b = 0;
  auto take = [&](size_t bytes) { size_t at = b; b = round_up(b + bytes, 256); return at; };
  const size_t Mp = (size_t)p.Mp;
  p.off_ring = take((size_t)p.R * p.slot_stride * 4);
  p.off_shadow = take((size_t)p.R * p.shadow_stride * 2);
  p.off_rowidx = take(Mp * 4);
  p.off_label = take(Mp * 4);
  p.off_xgt = take((size_t)p.dp[0] * p.ldm * 2);
  for (int l = 1; l < L; ++l) {
    p.off_h[l] = take(Mp * p.ld[l] * 2);
    p.off_ht[l] = take(p.ldm * p.dp[l] * 2);
  }
  p.off_z = take(Mp * p.dp[L] * 4);
  for (int l = 1; l <= L; ++l) {
    p.off_dz[l] = take(Mp * p.ld[l] * 2);
    p.off_dzt[l] = take(p.ldm * p.dp[l] * 2);
  }
  p.off_rowloss = take(Mp * 4);
  for (int l = 1; l <= L; ++l) p.off_colsum[l] = take(Mp / (l == L ? kCeFewRows : 64) * p.dp[l] * 4);
  for (int l = 1; l < L; ++l) p.off_maskbits[l] = take(round_up(Mp, 256) * round_up((size_t)p.dp[l], 256) / 8);
  if (p.U == 1) {          // (a local step is taken in the weight gradient's epilogue: no partials)
    for (int l = 0; l < L; ++l) p.off_partial[l] = take((size_t)p.dp[l] * (p.dp[l + 1] + kPartialPad) * 4 * kMaxSplit);
  } else {
    p.off_priv = take((size_t)c.N * p.slot_stride * 4);
    p.off_priv_shadow = take((size_t)c.N * p.shadow_stride * 2);
    p.off_lossacc = take((size_t)c.N * 4);
    p.off_delta = take(p.slot_stride * 4);
  }
  p.off_eval = take(eval_scratch_bytes((size_t)p.Mp));
  p.total = b;
  return true;
}

// ------------------------------------------------------------------ launches
namespace {

// Plan recording: with t_plan set, the launch functions below append what they would launch
// (kernel, tile shape, split count) and launch nothing; mlp_round_plan() uses it so that the
// description of a round's launches comes from the very code that issues them.
thread_local std::string* t_plan = nullptr;
#define ABS_LAUNCH(...) do { if (!t_plan) { __VA_ARGS__; } } while (0)
// A round's kernels carry their own start / stop events when the round is timed: kbegin() asks the
// hook for the pair, the next ABS_LAUNCH_K attaches it to its dispatch (null events: a plain launch).
thread_local hipEvent_t t_ev0 = nullptr, t_ev1 = nullptr;
void kbegin(LaunchHook* hook, int kind, double flops, double bytes) { hook->begin_kernel(kind, flops, bytes, &t_ev0, &t_ev1); }
void kend(LaunchHook* hook, int kind) { hook->end_kernel(kind); t_ev0 = t_ev1 = nullptr; }
#define ABS_LAUNCH_K(kernel, grid, block, stream, ...)                                                    \
  do {                                                                                                    \
    if (!t_plan) hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, t_ev0, t_ev1, 0, __VA_ARGS__);     \
  } while (0)
void plan_note(const char* what, int a, int b, int c) {
  if (t_plan) *t_plan += std::string(what) + ":" + std::to_string(a) + "x" + std::to_string(b) + "/" + std::to_string(c) + " ";
}

struct NullHook : LaunchHook {
  void begin(int, double, double) override {}
  void end(int) override {}
};

// The two uses of the update kernels:
//   UPD_GLOBAL  w^{t+1} = w^t - sum of the split partials                    (U = 1, Eq. 3)
//   UPD_DELTA   w^{t+1} = w^t - D, D = the averaged change of the uploads    (U > 1, Eq. 3)
// each also writes the bf16 copies of what it produced.
enum { UPD_GLOBAL = 0, UPD_DELTA = 1 };
// Weight gradient of layer l over `rows` stacked rows on the 256 x 256 tile kernel: k-steps per run if
// the contraction should be cut into equal runs across the tiles (GemmArgs::sk_q), else 0.  Runs pay
// when equal row ranges per tile leave a good part of the CUs idle in the launch's last wave and a
// run is still long enough to amortise a tile's epilogue; a tile then gets up to *max_parts partials.
int wgrad_runs(const MlpPlan& p, int l, int rows, int nsplit, int* max_parts) {
  constexpr int kCUs = 256, kMinRun = 24;
  if (p.dp[l] % TM3 || p.dp[l + 1] % TN3 || p.d[l + 1] % 4 || p.w_off[l] % 4) return 0;   // (the tiled update kernels read the per-tile counts)
  const int tiles = (p.dp[l] / TM3) * (p.dp[l + 1] / TN3), ksteps = rows / BK;
  const int wgs = tiles * nsplit;
  if (wgs < 128) return 0;                                   // (not a launch of the large-tile kernel)
  const int waves = (wgs + kCUs - 1) / kCUs;
  if ((double)wgs / (waves * kCUs) >= 0.9) return 0;         // equal ranges already fill the CUs
  const long units = (long)tiles * ksteps;
  const int q = (int)((units + kCUs - 1) / kCUs);            // one run per CU
  if (q < kMinRun) return 0;
  const int parts = (ksteps + q - 1) / q + 1;
  if (parts > kMaxSplit) return 0;
  *max_parts = parts;
  return q;
}

// Eq. 3 for layer l's weight matrix from the split partials of its weight gradient (U = 1).
TileUpdate global_update_args(const MlpArgs& a, int l, const RoundDesc& rd, int nsplit) {
  const MlpPlan& p = a.plan;
  float* ring = at<float>(a, p.off_ring);
  uint16_t* shadow = at<uint16_t>(a, p.off_shadow) + (size_t)rd.slot_next * p.shadow_stride;
  TileUpdate u{};
  u.partial = at<float>(a, p.off_partial[l]);
  u.split_stride = (size_t)p.dp[l] * (p.dp[l + 1] + kPartialPad);
  u.ldp = (size_t)p.dp[l + 1] + kPartialPad;
  u.nsplit = nsplit;
  u.w_cur = ring + (size_t)rd.slot_cur * p.slot_stride + p.w_off[l];
  u.w_next = ring + (size_t)rd.slot_next * p.slot_stride + p.w_off[l];
  u.d_in = p.d[l];
  u.d_out = p.d[l + 1];
  u.wn = l >= 1 ? shadow + p.wn_off[l] : nullptr; u.ldwn = (size_t)p.ld[l + 1];
  u.wt = shadow + p.wt_off[l]; u.ldwt = (size_t)p.ld[l];
  return u;
}
// Whether the rows of layer l's fp32 weight matrix can be moved 16 bytes at a time.
bool update_rows_aligned(const MlpPlan& p, int l) { return p.d[l + 1] % 4 == 0 && p.w_off[l] % 4 == 0; }

void launch_update(const MlpArgs& a, int l, const RoundDesc& rd, int mode, int nsplit,
                   hipStream_t s, LaunchHook* hook, int run_q = 0, int run_ksteps = 0) {
  const MlpPlan& p = a.plan;
  float* ring = at<float>(a, p.off_ring);
  TileUpdate u{};
  u.d_in = p.d[l];
  u.d_out = p.d[l + 1];
  u.ldwn = (size_t)p.ld[l + 1];
  u.ldwt = (size_t)p.ld[l];
  {
    uint16_t* shadow = at<uint16_t>(a, p.off_shadow) + (size_t)rd.slot_next * p.shadow_stride;
    if (mode == UPD_GLOBAL) {
      u.partial = at<float>(a, p.off_partial[l]);
      u.split_stride = (size_t)p.dp[l] * (p.dp[l + 1] + kPartialPad);
      u.ldp = (size_t)p.dp[l + 1] + kPartialPad;
      u.nsplit = nsplit;
    } else {
      u.partial = at<float>(a, p.off_delta) + p.w_off[l];
      u.split_stride = 0;
      u.ldp = (size_t)p.d[l + 1];
      u.nsplit = 1;
    }
    u.w_cur = ring + (size_t)rd.slot_cur * p.slot_stride + p.w_off[l];
    u.w_next = ring + (size_t)rd.slot_next * p.slot_stride + p.w_off[l];
    u.wn = l >= 1 ? shadow + p.wn_off[l] : nullptr;
    u.wt = shadow + p.wt_off[l];
  }
  if (run_q) { u.sk_q = run_q; u.sk_ksteps = run_ksteps; u.sk_nt = p.dp[l + 1] / TN3; }
  const double n = (double)p.d[l] * p.d[l + 1];
  kbegin(hook, KK_MLP_UPDATE, n * (u.nsplit + 1), n * (4.0 * (u.nsplit + 2) + (l >= 1 ? 4.0 : 2.0)));
  const dim3 block(256);
  const bool vec = update_rows_aligned(p, l);
  // wide tiles (fewer, longer stores) only where they still give every CU a workgroup
  const bool wide = p.d[l + 1] >= 256 && ((p.d[l + 1] + 255) / 256) * ((p.d[l] + 63) / 64) >= 256;
  plan_note("update", 64, vec && wide ? 256 : vec ? 64 : 1, u.nsplit);
  if (vec && wide) ABS_LAUNCH_K((mlp_update_kernel<256>), dim3((p.d[l + 1] + 255) / 256, (p.d[l] + 63) / 64), block, s, u);
  else if (vec) ABS_LAUNCH_K((mlp_update_kernel<64>), dim3((p.d[l + 1] + 63) / 64, (p.d[l] + 63) / 64), block, s, u);
  else     ABS_LAUNCH_K(mlp_update_small_kernel, dim3((p.d[l] * p.d[l + 1] + 255) / 256), block, s, u);
  kend(hook, KK_MLP_UPDATE);
}

// Whether a product goes to the 256 x 256 tile kernel.
inline bool gemm_is_big(bool gather, bool per_upload, const GemmArgs& g, int Mdim, int Ndim, int nsplit) {
  return Mdim % TM3 == 0 && Ndim % TN3 == 0 && (!per_upload || g.rows_per_upload % TM3 == 0) &&
         (!gather || g.a_kvalid == g.ksteps_total * BK) && (Mdim / TM3) * (Ndim / TN3) * nsplit >= 128;
}

// Returns whether the product went to the 256 x 256 tile kernel (only that one knows maskbits).
template <int EPI, bool GATHER, bool PER_UPLOAD, int TAG = 0>
bool launch_gemm(GemmArgs g, const RoundDesc& rd, int Mdim, int Ndim, int nsplit, hipStream_t s) {
  g.nsplit = nsplit;
  // (TAG 2, 3 and 4: the caller picks them with this very test, only the large-tile kernel reads such an A)
  constexpr bool kBigOnly = TAG >= 2 && TAG <= 4;
  const bool big = g.sk_q > 0 || gemm_is_big(GATHER, PER_UPLOAD, g, Mdim, Ndim, nsplit);
  if constexpr (kBigOnly) {
    if (!big) {
      std::fprintf(stderr, "libabs: gathered or transposed A outside the large-tile kernel\n");
      std::abort();
    }
  }
  if (big && g.sk_q > 0) {
    // runs of sk_q k-steps across the tiles: one workgroup per run
    g.mt = Mdim / TM3;
    g.nt = Ndim / TN3;
    g.rows_per_xcd = 0;
    const int runs = (g.mt * g.nt * g.ksteps_total + g.sk_q - 1) / g.sk_q;
    plan_note(TAG == 2 ? "wgrad_x_runs" : "wgrad_runs", TM3, TN3, g.sk_q);
    ABS_LAUNCH_K((mlp_gemm256_kernel<EPI, GATHER, PER_UPLOAD, TAG>), dim3((runs + 7) / 8 * 8 + g.pig_blocks + g.bias_blocks), dim3(512), s, g, rd);
    return true;
  }
  if (big) {
    g.mt = Mdim / TM3;
    g.nt = Ndim / TN3;
    g.rows_per_xcd = (g.mt * nsplit + 7) / 8;
    // long products with outputs beyond the caches stream them out (short ones are bound by these very
    // stores and were slower for it: the output layer's input gradient 75 -> 79 us at 32768 rows; so was
    // the first layer's forward product, whose gathered rows come from memory anyway: 368 -> 374 us)
    g.stream_out = (EPI == EPI_RELU || EPI == EPI_DGRAD) && !GATHER && g.ksteps_total >= 16 &&
                   (size_t)Mdim * (size_t)Ndim * 2 >= ABS_STREAM_MIN_BYTES;
    plan_note(EPI == EPI_RELU ? (TAG == 3 ? "fwd_t" : "fwd") : EPI == EPI_LOGITS ? "logits" : EPI == EPI_DGRAD ? (TAG == 3 ? "dgrad_t" : "dgrad")
              : TAG == 4 ? "wgrad_x_step" : TAG == 5 ? "wgrad_step" : TAG == 2 ? "wgrad_x" : "wgrad", TM3, TN3, nsplit);
    ABS_LAUNCH_K((mlp_gemm256_kernel<EPI, GATHER, PER_UPLOAD, TAG>), dim3(8 * g.rows_per_xcd * g.nt + g.pig_blocks + g.bias_blocks), dim3(512), s, g, rd);
    return true;
  }
  if constexpr (!kBigOnly) {
    // 128 x 256 tiles once they are two workgroups for every CU (below, 128 x 128 tiles in two workgroups per CU; us at
    // uploads of 128 rows with 128 x 128 / 128 x 256: first layer 8192 x 2048 x 1024 57 / 49.5, 16384 x 2048 x 3072
    // 258 / 217, hidden 8192 x 2048 x 2048 91 / 77, 16384 x 1024 x 1024 49 / 46; at half of that, 8192 x 1024 x 1024,
    // 27 / 33).
    if constexpr (TAG < 2) {
      if (EPI == EPI_WGRAD ? wgrad_256_columns(Mdim, Ndim, g.ksteps_total)
                           : Ndim % TNW == 0 && (Mdim / TM) * (Ndim / TNW) * nsplit >= 512) {
        g.mt = Mdim / TM;
        g.nt = Ndim / TNW;
        g.rows_per_xcd = (g.mt * nsplit + 7) / 8;
        plan_note(EPI == EPI_RELU ? "fwd_wide" : EPI == EPI_LOGITS ? "logits_wide" : EPI == EPI_DGRAD ? "dgrad_wide" : "wgrad_wide", TM, TNW, nsplit);
        ABS_LAUNCH_K((mlp_wide_kernel<EPI, GATHER, PER_UPLOAD, TAG>), dim3(8 * g.rows_per_xcd * g.nt + g.pig_blocks + g.bias_blocks), dim3(256), s, g, rd);
        return false;
      }
    }
    // 128-wide tiles once 64-wide ones would be more than the two workgroups a CU holds (a 64-wide workgroup
    // stages twice the bytes per flop, but a CU draws at most 23-32 bytes per clock from beyond the L1, so
    // a product spread over twice the CUs or in two workgroups per CU is the faster one; 3072 x 1024, us with
    // 64 / 128 wide tiles at 2048 rows: 31.5 / 35.1, 2560: 44.8 / 36.5, 3072: 46.3 / 37.0, 4608: 70.1 / 69.3).
    // Up to one 128-wide tile per CU the two wavefront groups of a workgroup share the contraction (KG = 2); with
    // more tiles than CUs each takes four wavefronts and a ring of two, so that two fit a CU and the second
    // covers the first one's barriers and epilogue (us with KG = 2 / 1: 8192 x 1024 x 1024 31.4 / 26.9, first layer
    // 8192 x 1024 x 3072 48 / 44, 8192 x 2048 x 2048 102 / 91).
    const bool wide = EPI == EPI_WGRAD ? wgrad_wide_tiles(Mdim, Ndim, g.ksteps_total, TAG >= 4 ? nsplit : 0)
                                       : Ndim % 128 == 0 && (Mdim / 128) * (Ndim / 128) * nsplit > 128;
    const int tile = wide ? 128 : 64;
    g.mt = Mdim / tile;
    g.nt = Ndim / tile;
    g.rows_per_xcd = (g.mt * nsplit + 7) / 8;
    const bool pairs = wide && g.mt * g.nt * nsplit > 256;
    const dim3 grid(8 * g.rows_per_xcd * g.nt + g.pig_blocks + g.bias_blocks);
    plan_note((std::string(EPI == EPI_RELU ? "fwd" : EPI == EPI_LOGITS ? "logits" : EPI == EPI_DGRAD ? "dgrad" : TAG >= 4 ? "wgrad_step" : "wgrad") +
               (pairs ? "_tile2" : "_tile")).c_str(), tile, tile, nsplit);
    // Ring depths: forward and input-gradient products keep three steps on their way (64-wide: 64 KB, two
    // workgroups per CU; 8 steps and one workgroup: the evaluation's logits 22.5 instead of 16.8 us; 3 steps: cfg 3's
    // first layer 22.4 instead of 18.4).  A weight gradient carries the previous layer's update as extra
    // workgroups and leaves LDS for several of them per CU (128-wide, ring of 4 and one workgroup:
    // cfg 5's output layer 39 instead of 33 us).
    constexpr int kRing128 = EPI == EPI_WGRAD ? 2 : 4, kRing64 = EPI == EPI_WGRAD ? 3 : 4;
    if (pairs)     ABS_LAUNCH_K((mlp_tile_kernel<128, 1, EPI, GATHER, PER_UPLOAD, TAG, 2>), grid, dim3(TileCfg<128, 1>::NT), s, g, rd);
    else if (wide) ABS_LAUNCH_K((mlp_tile_kernel<128, 2, EPI, GATHER, PER_UPLOAD, TAG, kRing128>), grid, dim3(TileCfg<128, 2>::NT), s, g, rd);
    else           ABS_LAUNCH_K((mlp_tile_kernel<64, 4, EPI, GATHER, PER_UPLOAD, TAG, kRing64>), grid, dim3(TileCfg<64, 4>::NT), s, g, rd);
  }
  return false;
}

// Forward pass over `rows` stacked rows: H_l and H_l^T for the hidden layers; the model of the rows
// of upload a is slot rd.w[a].slot of the ring given by wbase / sbase (own: slot a of the private
// models).  draw0 >= 0 (training): the first layer draws the minibatch rows itself (draw index
// draw0 + sample) and leaves them in rowidx / label, and the pass stops before the output layer
// (launch_logits_ce takes over); draw0 < 0 (evaluation): rowidx holds the rows of Xsrc and the fp32
// logits are written.
// Returns the set of hidden layers l (bit l) whose ReLU mask bits were written (want_bits and the
// layer's product ran on the 256 x 256 tile kernel).
unsigned mlp_forward(const MlpArgs& a, const uint16_t* Xsrc, const RoundDesc& rd, int rows, double arows,
                     const float* wbase, const uint16_t* sbase, bool own, bool want_bits, long draw0,
                     hipStream_t s, LaunchHook* hook) {
  unsigned have_bits = 0;
  const MlpPlan& p = a.plan;
  const int L = p.L;
  uint32_t* rowidx = at<uint32_t>(a, p.off_rowidx);
  const bool train = draw0 >= 0;
  // H_l is read row-major by the next layer's product and transposed by its weight gradient and mask.
  // When both the product that writes H_l and the one that reads it run on the 256 x 256 tile kernel,
  // the reader takes the transposed copy (transposing LDS reads, TAG 3) and the row-major copy is never
  // written: half of the writer's output bytes (cfg 5's first-layer forward at 32768 rows: 134 MB, 368 -> 351 us;
  // the reader pays 7 us for the two LDS reads per fragment; a round at K = 128 -1.4 %, at K = 40 -2 %).
  // The last hidden layer keeps both: the output-layer kernels read it row-major.
  bool a_transposed = false;           // this layer reads H_l^T
  for (int l = 0; l < (train ? L - 1 : L); ++l) {
    GemmArgs g{};
    if (l == 0) {
      g.A = Xsrc; g.lda = (size_t)p.d[0]; g.a_rowidx = rowidx; g.a_kvalid = p.d[0];
      if (train) {
        g.gen_rows = 1; g.gen_B = p.B; g.gen_shard_rows = a.shard_rows; g.gen_batch_key = a.batch_key;
        g.gen_draw0 = (uint32_t)draw0; g.gen_y = a.y; g.gen_rowidx = rowidx; g.gen_label = at<int32_t>(a, p.off_label);
      }
    } else if (a_transposed) {
      g.A = at<uint16_t>(a, p.off_ht[l]); g.lda = p.ldm;
    } else {
      g.A = at<uint16_t>(a, p.off_h[l]); g.lda = (size_t)p.ld[l];
    }
    g.Bt = sbase + p.wt_off[l]; g.ldb = (size_t)p.ld[l];
    g.bt_slot_stride = p.shadow_stride;
    g.by_upload = own;
    g.rows_per_upload = p.Bp;
    g.ksteps_total = g.ksteps_per_split = p.dp[l] / BK;
    g.bias = wbase + p.b_off[l]; g.bias_slot_stride = p.slot_stride; g.n_valid = p.d[l + 1];
    const double fl = 2.0 * arows * p.d[l] * p.d[l + 1];
    if (l < L - 1) {
      g.out = at<uint16_t>(a, p.off_h[l + 1]); g.ldo = (size_t)p.ld[l + 1];
      g.outT = at<uint16_t>(a, p.off_ht[l + 1]); g.ldoT = p.ldm;
      const int kind = l == 0 ? KK_MLP_FWD_L1 : KK_MLP_FWD_HIDDEN;
      kbegin(hook, kind, fl, arows * (p.d[l] * 2.0 + p.d[l + 1] * 4.0));
      if (want_bits) g.maskbits = at<uint32_t>(a, p.off_maskbits[l + 1]);
      // does the next layer's product read H_{l+1} transposed?  (both on the large-tile kernel)
      bool next_transposed = false;
      if (l + 1 <= L - 2) {
        GemmArgs nx{};
        nx.rows_per_upload = p.Bp;
        next_transposed = gemm_is_big(l == 0, true, g, rows, p.dp[l + 1], 1) && gemm_is_big(false, true, nx, rows, p.dp[l + 2], 1);
      }
      if (next_transposed) g.out = nullptr;
      const bool big = l == 0        ? launch_gemm<EPI_RELU, true, true>(g, rd, rows, p.dp[l + 1], 1, s)
                       : a_transposed ? launch_gemm<EPI_RELU, false, true, 3>(g, rd, rows, p.dp[l + 1], 1, s)
                                      : launch_gemm<EPI_RELU, false, true>(g, rd, rows, p.dp[l + 1], 1, s);
      a_transposed = next_transposed;
      if (big && want_bits) have_bits |= 1u << (l + 1);
      kend(hook, kind);
    } else {
      g.outf = at<float>(a, p.off_z); g.ldof = (size_t)p.dp[L];
      kbegin(hook, KK_MLP_FWD_LOGITS, fl, arows * (p.d[l] * 2.0 + p.d[l + 1] * 4.0));
      launch_gemm<EPI_LOGITS, false, true>(g, rd, rows, p.dp[L], 1, s);
      kend(hook, KK_MLP_FWD_LOGITS);
    }
  }
  return have_bits;
}

// Rows per workgroup of the output-layer kernel.  32-row workgroups each read all of W_L^T, 128-row ones a quarter as
// often, so the line lies where their number outweighs what they read: up to 32 classes at three 32-row workgroups
// per CU, beyond (a workgroup's W_L^T is the larger operand) at half a one, or at one where the contraction is
// long.  us of a round with 32 / 128 rows: 512-256-10, 16384 rows 65 / 70, 24576: 79.7 / 80.6, 32768: 103.9 / 103.5;
// 512-2048-30, 16384: 205 / 208, 32768: 369 / 358; 512-256-100, 4096: 59.0 / 61.5, 6144: 68.1 / 66.6, 8192: 69.6 / 68.0;
// 512-1536-100, 8192: 115.6 / 114.3; 512-2048-100, 8192: 133 / 138, 9216: 183 / 169; 512-4096-100, 8192: 230 / 240, 9216: 297 / 276.
// Beyond 96 classes a CU holds one 32-row workgroup.  A short contraction, which gives the four wavefronts little to share, then
// stays with 128 rows where blocks of the transposed minibatch ride (`gather` of them are there) and make it more than a workgroup
// per CU, alone / six simulations side by side: 880-73-100, 2048 rows (192 workgroups) 35.8 / 37.8 and 88.0 / 88.6, 3072 (288)
// 42.8 / 42.1 and 110 / 105, 4096 (384) 48.3 / 47.5 and 124 / 121; 2048-256-100, 3072 (480) 48.1 / 46.6 and 171 / 164; up to a
// workgroup per CU, 512-200-100, 4096 (256) 42.9 / 45.3 and 132 / 126; long ones, 1000-300-100, 4096 (384) 49.3 / 50.1 and 188 / 178.
int ce_rows(const MlpPlan& p, int rows, int gather) {
  bool few = p.d[p.L] <= 32 ? rows <= 24576
           : p.dp[p.L] <= 128 && (rows <= 4096 || (rows <= 8192 && p.dp[p.L - 1] >= 2048));
  if (p.d[p.L] > kFewPairClasses && p.dp[p.L - 1] <= 256 && gather <= kGatherRide && rows / kCeFewRows + gather > 256) few = false;
  return few ? kCeFewRows : kCeRows;
}
// ... and how many blocks of the transposed minibatch ride in its launch.
int gather_ride(const MlpPlan& p, int block_rows) { return block_rows == kCeFewRows && p.d[p.L] <= kFewPairClasses ? kGatherRideFew : kGatherRide; }

// Output layer of a training pass: logits, loss sums per `block_rows` rows (ce_rows()), dZ_L in both orientations and its
// column sums, in one kernel (mlp_logits_ce_kernel).
void launch_logits_ce(const MlpArgs& a, const RoundDesc& rd, int rows, double arows, const float* wbase,
                      const uint16_t* sbase, bool own, int block_rows, int gather_blocks, hipStream_t s, LaunchHook* hook) {
  const MlpPlan& p = a.plan;
  const int L = p.L;
  LogitsCeArgs c{};
  if (gather_blocks) {
    c.gt.X = a.X; c.gt.d0 = p.d[0]; c.gt.dp0 = p.dp[0];
    c.gt.rowidx = at<uint32_t>(a, p.off_rowidx);
    c.gt.XgT = at<uint16_t>(a, p.off_xgt); c.gt.ldt = p.ldm;
    c.gt.blocks = gather_blocks;
    plan_note("with_gather_t", 64, 256, 1);
  }
  c.H = at<uint16_t>(a, p.off_h[L - 1]); c.ldh = (size_t)p.ld[L - 1];
  c.ksteps = p.dp[L - 1] / BK;
  c.Wt = sbase + p.wt_off[L - 1]; c.ldw = (size_t)p.ld[L - 1];
  c.w_slot_stride = p.shadow_stride;
  c.bias = wbase + p.b_off[L - 1]; c.bias_slot_stride = p.slot_stride;
  c.C = p.d[L];
  c.rows_per_upload = p.Bp; c.by_upload = own;
  c.label = at<int32_t>(a, p.off_label);
  c.dZ = at<uint16_t>(a, p.off_dz[L]); c.lddz = (size_t)p.ld[L];
  c.dZT = at<uint16_t>(a, p.off_dzt[L]); c.lddzt = p.ldm;
  c.rowloss = at<float>(a, p.off_rowloss);
  c.colsum = at<float>(a, p.off_colsum[L]); c.ldcs = (size_t)p.dp[L];
  kbegin(hook, KK_MLP_LOGITS_CE, 2.0 * arows * p.d[L - 1] * p.d[L] + arows * p.d[L] * 8.0,
              arows * (p.d[L - 1] * 2.0 + p.d[L] * 4.0 + (c.gt.blocks ? p.d[0] * 4.0 : 0.0)));
  plan_note("logits_ce", block_rows, p.dp[L], 1);
  const dim3 grid(rows / block_rows + c.gt.blocks), block(256);
  if (block_rows == kCeFewRows) {
    switch ((p.d[L] + 15) / 16) {
#define ABS_CASE(cb) case cb: ABS_LAUNCH_K((mlp_logits_ce_few_kernel<cb>), grid, block, s, c, rd); break;
      ABS_CASE(1) ABS_CASE(2) ABS_CASE(3) ABS_CASE(4) ABS_CASE(5) ABS_CASE(6) ABS_CASE(7) ABS_CASE(8)
#undef ABS_CASE
    }
    kend(hook, KK_MLP_LOGITS_CE);
    return;
  }
  switch (p.dp[L] / 64) {
    case 1: ABS_LAUNCH_K((mlp_logits_ce_kernel<2>), grid, block, s, c, rd); break;
    case 2: ABS_LAUNCH_K((mlp_logits_ce_kernel<4>), grid, block, s, c, rd); break;
    default: ABS_LAUNCH_K((mlp_logits_ce_kernel<8>), grid, block, s, c, rd); break;
  }
  kend(hook, KK_MLP_LOGITS_CE);
}

// Whether a round of `rows` stacked rows at U = 1 takes its steps in mlp_step_kernel, and with which tiles (0: split
// weight gradients, partials and updates).  Unsplit, the contraction may have at most 64 k-steps: up to there it wins in every
// shape measured that the limits below leave in, beyond it turns at another length for each (us of a round, split / unsplit with
// the better tiles, at 64, 68, 72, 80 and 96 k-steps: 3072-512-10 82 / 75, 93 / 88, 86 / 89, 97 / 93, 93 / 101; 2048-1024-10 86 / 83,
// 101 / 96, 102 / 98, 104 / 105, 109 / 117; 3072-2048-2048-100 361 / 339, 465 / 439, 461 / 452, 477 / 478, 497 / 520; 512-512-100
// 54 / 45, 65 / 54, 61 / 54, 68 / 55, 72 / 59).  With tiles of 128 x 128 there is a limit to the work too, beyond which the 256 x 256
// kernel's fewer bytes per flop win over its partials.  128 x 128 from 128 such tiles on, 64 x 64 below; where even these
// are few, the split ones win earlier (us of a round, split / 64 x 64: 512-128-10, 18 tiles, 3072 rows 36.8 / 36.8, 4096: 37.4 / 40.7;
// 880-73-100, 32 tiles, 3072: 44.9 / 44.6, 4096: 45.7 / 47.5; 1024-128-100, 36 tiles, 4096: 55.4 / 47.8).
// us of a round with split weight gradients / 64 x 64 / 128 x 128 tiles, by rows:
//   3072-512-10   1024: 53.5 / 46.3 / 48.4   4096: 80 / 75 / 81       1000-520-300-26  512: 59 / 45 / 49   3072: 61 / 50 / 55
//   512-256-10    4096: 50 / 44 / 59         8192: 53 / 59 / 89       2048-1024-10    1024: 52 / 49 / 45   4096: 90 / 93 / 87
//   3072-1024-1024-10  512: 84 / 72 / 67     2048: 132 / 121 / 112    4096: 177 / 186 / 164   8192: 265 / 314 / 280
//   3072-2048-2048-100 512: 147 / 136 / 122  1024: 198 / 186 / 165    4096: 400 / 470 / 376
//   3072-4096-4096-100 1024: 392 / 400 / 342 2048: 570 / 641 / 534    4096: 691 / 965 / 743
int step_tiles(const MlpPlan& p, int rows) {
  const long ksteps = rows / BK;
  if (ksteps > 64) return 0;
  long tiles = 0, small = 0;
  for (int l = 0; l < p.L; ++l) {
    tiles += (long)(p.dp[l] / 128) * ((p.dp[l + 1] + 127) / 128);
    small += (long)(p.dp[l] / 64) * (p.dp[l + 1] / 64);
  }
  if (small <= 32 && ksteps > 48) return 0;
  if (tiles < 128) return 64;
  return tiles * ksteps <= 60000 ? 128 : 0;
}
// Blocks of the transposed minibatch (64 rows x 256 columns).
int gather_t_blocks(const MlpPlan& p, int rows) { return (rows / 64) * ((p.dp[0] + 255) / 256); }
// 128 x 128 tiles: one workgroup per CU with three k-steps on their way while the tiles do not outnumber the CUs (us, one /
// two workgroups: 2048-1024-10, 136 tiles, 4096 rows 87 / 95; 3072-1024-1024-10, 264 tiles, 2048 rows 119 / 114) ...
bool step_pairs(const MlpPlan& p) {
  int tiles = 0;
  for (int l = 0; l < p.L; ++l) tiles += (p.dp[l] / 128) * ((p.dp[l + 1] + 127) / 128);
  return tiles > 256;
}
// ... and the pairs read the first layer's minibatch rows where they lie if its transposed copy is beyond what rides for
// nothing (a k-step then touches 64 rows all over the dataset: 0.86 instead of 0.65 us; 3072-1024-1024-10, 4096 rows, 768
// blocks, 164 us a round against 174 with the copy, 2048 rows, 384 blocks 113.6 / 112.2, 3072-2048-2048-100, 384 blocks 224 / 216).
bool step_direct(const MlpPlan& p, int rows) { return step_tiles(p, rows) == 128 && step_pairs(p) && gather_t_blocks(p, rows) > 512; }

// The same for a local step of K uploads: their rows are contractions of their own, so it is the private models' bytes that
// count, and one launch for all layers, with tiles of half the models' rows, moves them faster than the products one by one
// (256 x 256 tiles with an epilogue of 4 us and nothing beside it); up to 32 k-steps an upload, 64 x 64 tiles while the wider
// ones would be few.  us of a round, a launch per layer / 64 x 64 / 128 x 128: 3072-512-10, U = 10, 128 rows: K = 2 510 / 456 /
// 431, 8 669 / 646 / 591, 32 1878 / 1902 / 1778; 3072-1024-1024-10, K = 8, U = 5 879 / 786 / 711; 3072-2048-2048-100, K = 8, U = 3, 256
// rows 1383 / 1426 / 1242; 512-512-10, K = 8, U = 10, 1024 rows 556 / 481 / 494, U = 4, 2048: 259 / 233 / 251, 4096: 431 / 403 / 446;
// 512-2048-100, U = 4: K = 2, 1024 rows (160 tiles of 128) 302 / 269 / 278, K = 4, 1536 rows (320) 477 / 454 / 435.
int local_step_tiles(const MlpPlan& p, int K) {
  if (p.Bp / BK > 32) return 0;
  long tiles = 0;
  for (int l = 0; l < p.L; ++l) tiles += (long)(p.dp[l] / 128) * ((p.dp[l + 1] + 127) / 128);
  return tiles * K <= 192 ? 64 : 128;
}

// All weight matrices and biases in one launch (mlp_step_kernel): w^t -> w^{t+1} of a round at U = 1, or a local step of
// the uploads' private models (own: from themselves, else from the uploads' ring slots).
void launch_steps(const MlpArgs& a, const RoundDesc& rd, int rows, double arows, int tile, bool direct, const BiasCore& bias, int bias_cols,
                  bool own, hipStream_t s, LaunchHook* hook) {
  const MlpPlan& p = a.plan;
  float* ring = at<float>(a, p.off_ring);
  uint16_t* shadow = p.U > 1 ? at<uint16_t>(a, p.off_priv_shadow) : at<uint16_t>(a, p.off_shadow) + (size_t)rd.slot_next * p.shadow_stride;
  float* const priv = at<float>(a, p.off_priv);
  StepArgs g{};
  const bool local = p.U > 1;
  const int up = local ? rd.K : 1;
  g.L = p.L; g.uploads = up; g.sel = local ? (own ? 1 : 2) : 0; g.ksteps = rows / up / BK;
  g.stride = p.slot_stride; g.shadow_stride = p.shadow_stride;
  g.rowidx = at<uint32_t>(a, p.off_rowidx);
  g.bias = bias; g.bias_per = (bias_cols + 15) / 16;
  int first = 0;
  double flops = 0.0, bytes = 0.0;
  for (int l = 0; l < p.L; ++l) {
    StepLayer& y = g.l[l];
    y.A = l > 0 ? at<uint16_t>(a, p.off_ht[l]) : direct ? a.X : at<uint16_t>(a, p.off_xgt); y.lda = l == 0 && direct ? (size_t)p.d[0] : p.ldm;
    y.Bt = at<uint16_t>(a, p.off_dzt[l + 1]); y.ldb = p.ldm;
    g.first[l] = first; y.mt = p.dp[l] / tile; y.nt = (p.dp[l + 1] + tile - 1) / tile;
    first += (up * y.mt * y.nt + 7) / 8 * 8;
    y.d_in = p.d[l]; y.d_out = p.d[l + 1]; y.dp_out = p.dp[l + 1];
    y.cur = (!local ? ring + (size_t)rd.slot_cur * p.slot_stride : own ? priv : ring) + p.w_off[l];
    y.next = (local ? priv : ring + (size_t)rd.slot_next * p.slot_stride) + p.w_off[l];
    y.wn = l >= 1 ? shadow + p.wn_off[l] : nullptr; y.ldwn = (size_t)p.ld[l + 1];
    y.wt = shadow + p.wt_off[l]; y.ldwt = (size_t)p.ld[l];
    flops += 2.0 * arows * p.d[l] * p.d[l + 1];
    bytes += arows * (p.d[l] + p.d[l + 1]) * 2.0 + (double)up * p.d[l] * p.d[l + 1] * (l >= 1 ? 12.0 : 10.0);
  }
  for (int l = p.L; l < 8; ++l) g.first[l] = first;
  kbegin(hook, KK_MLP_WGRAD_L1, flops, bytes);
  const bool pairs = tile == 128 && (local || step_pairs(p));
  if (local) { for (int l = 0; l < p.L; ++l) plan_note(pairs ? "wgrad_step_tile2" : "wgrad_step_tile", tile, tile, up); }
  else       plan_note(direct ? "steps_x" : pairs ? "steps2" : "steps", tile, tile, 1);
  const dim3 grid(first + up * g.bias_per);
  if (tile == 64 && local) ABS_LAUNCH_K((mlp_step_kernel<64, 64, 4, 2, 3, false>), grid, dim3(256), s, g, rd);
  else if (tile == 64)     ABS_LAUNCH_K((mlp_step_kernel<64, 64, 4, 4, 2, false>), grid, dim3(256), s, g, rd);
  else if (direct)         ABS_LAUNCH_K((mlp_step_kernel<128, 128, 8, 2, 4, true>), grid, dim3(512), s, g, rd);
  else if (pairs)          ABS_LAUNCH_K((mlp_step_kernel<128, 128, 8, 2, 4, false>), grid, dim3(512), s, g, rd);
  else                     ABS_LAUNCH_K((mlp_step_kernel<128, 128, 8, 4, 2, false>), grid, dim3(512), s, g, rd);
  kend(hook, KK_MLP_WGRAD_L1);
}

}  // namespace

hipError_t mlp_prepare(const MlpArgs& a, hipStream_t s) {
  const MlpPlan& p = a.plan;
  // padding of every bf16 weight copy must read as zero
  const size_t n16 = (size_t)p.R * p.shadow_stride * 2 / 16;
  mlp_fill_zero_kernel<<<dim3(1024), dim3(256), 0, s>>>(at<uint4>(a, p.off_shadow), n16);
  if (p.U > 1)
    mlp_fill_zero_kernel<<<dim3(1024), dim3(256), 0, s>>>(at<uint4>(a, p.off_priv_shadow),
                                                          (size_t)p.N * p.shadow_stride * 2 / 16);
  NullHook nh;
  RoundDesc rd0{};                       // slot_cur = slot_next = 0, no partials: w^0 onto itself
  for (int l = 0; l < p.L; ++l) launch_update(a, l, rd0, UPD_GLOBAL, 0, s, &nh);   // bf16 copies of w^0
  return hipGetLastError();
}

// One pass of minibatch gradients for the K uploads of the round: U = 1 runs it once and folds
// the K-of-N reduction into the weight-gradient contraction (Eq. 3); U > 1 runs it U times on
// the uploads' private models (Eq. 2), each upload's weight gradient being its own range of
// the stacked rows, and then averages the uploads' changes into w^{t+1}.
hipError_t launch_mlp_round(const MlpArgs& a, const RoundDesc& rd, hipStream_t s, LaunchHook* hook) {
  const MlpPlan& p = a.plan;
  const int L = p.L, K = rd.K, U = p.U;
  const bool local = U > 1;
  const int rows = K * p.Bp;                 // stacked rows incl. padding (multiple of 128)
  const double arows = (double)K * p.B;      // rows that carry samples
  float* ring = at<float>(a, p.off_ring);
  const uint16_t* shadow = at<uint16_t>(a, p.off_shadow);
  float* priv = local ? at<float>(a, p.off_priv) : nullptr;
  const uint16_t* pshadow = local ? at<uint16_t>(a, p.off_priv_shadow) : nullptr;
  uint32_t* rowidx = at<uint32_t>(a, p.off_rowidx);

  for (int step = 0; step < U; ++step) {
    // where the uploads' models live during this step: the ring (by slot) or the private copies
    const bool own = local && step > 0;
    const float* wbase = own ? priv : ring;
    const uint16_t* sbase = own ? pshadow : shadow;

    // The first layer's weight gradient reads the minibatch rows straight from the dataset when
    // it runs on the 256 x 256 tile kernel and the rows are whole tiles wide; otherwise it needs
    // the transposed bf16 copy of the gathered rows.
    const bool wg0_direct = p.d[0] % TM3 == 0 && gemm_is_big(false, false, GemmArgs{}, p.dp[0], p.dp[1],
                                                               wgrad_split(p, 0, rows, local ? K : 0));

    // ---- forward at the uploads' model versions; the first layer draws the minibatch rows
    const unsigned have_bits = mlp_forward(a, a.X, rd, rows, arows, wbase, sbase, own, true,
                                           (long)step * (long)p.B, s, hook);

    // ---- output layer: loss and output gradient, already scaled by the uploads' coefficients
    const int stile = local ? local_step_tiles(p, K) : step_tiles(p, rows);
    const bool sdirect = !local && stile && step_direct(p, rows);
    const int gather_blocks = (stile ? sdirect : wg0_direct) ? 0 : gather_t_blocks(p, rows);
    const int ce_block = ce_rows(p, rows, gather_blocks);
    const bool gather_rides = gather_blocks <= gather_ride(p, ce_block);
    launch_logits_ce(a, rd, rows, arows, wbase, sbase, own, ce_block, gather_rides ? gather_blocks : 0, s, hook);
    const int loss_blocks = p.Bp / ce_block;               // row blocks of the loss sums per upload

    // ---- input gradients back through W_{L-1} .. W_1 (none is needed for the first layer)
    // (dZ_l likewise: read row-major only by the next product down; when writer and reader both run on
    // the large-tile kernel the reader takes dZ_l^T and the row-major copy is not written)
    bool dz_transposed = false;          // this product reads dZ_{l+1}^T
    for (int l = L - 1; l >= 1; --l) {
      GemmArgs g{};
      if (dz_transposed) { g.A = at<uint16_t>(a, p.off_dzt[l + 1]); g.lda = p.ldm; }
      else               { g.A = at<uint16_t>(a, p.off_dz[l + 1]); g.lda = (size_t)p.ld[l + 1]; }
      g.Bt = sbase + p.wn_off[l]; g.ldb = (size_t)p.ld[l + 1];
      g.bt_slot_stride = p.shadow_stride;
      g.by_upload = own;
      g.rows_per_upload = p.Bp;
      g.ksteps_total = g.ksteps_per_split = p.dp[l + 1] / BK;
      g.maskT = at<uint16_t>(a, p.off_ht[l]); g.ldmaskT = p.ldm;
      if ((have_bits >> l) & 1u) g.maskbits = at<uint32_t>(a, p.off_maskbits[l]);   // the tile kernel ignores it
      g.out = l >= 2 ? at<uint16_t>(a, p.off_dz[l]) : nullptr; g.ldo = (size_t)p.ld[l];
      g.outT = at<uint16_t>(a, p.off_dzt[l]); g.ldoT = p.ldm;
      g.colsum = at<float>(a, p.off_colsum[l]); g.ldcs = (size_t)p.dp[l];
      if (l == L - 1) {
        // the losses reach the host as the backward pass starts: it selects and enqueues the next
        // round while the device is still in this one
        // (local SGD: every step adds its losses, the job's last one publishes)
        g.pub_mailbox = step == U - 1 ? a.mailbox : nullptr; g.pub_rowloss = at<float>(a, p.off_rowloss);
        g.pub_nb = loss_blocks; g.pub_B = p.B;
        if (local) { g.pub_lossacc = at<float>(a, p.off_lossacc); g.pub_first = step == 0; g.pub_U = U; }
      }
      // the product through the output layer contracts over the classes only: bandwidth-bound
      const int kind = l == L - 1 ? KK_MLP_DGRAD_OUT : KK_MLP_DGRAD;
      kbegin(hook, kind, 2.0 * arows * p.d[l] * p.d[l + 1], arows * (p.d[l + 1] * 2.0 + p.d[l] * 6.0));
      bool next_transposed = false;      // the product for layer l - 1 reads dZ_l^T
      if (l >= 2)
        next_transposed = gemm_is_big(false, true, g, rows, p.dp[l], 1) && gemm_is_big(false, true, g, rows, p.dp[l - 1], 1);
      if (next_transposed) g.out = nullptr;
      if (l == L - 1)         launch_gemm<EPI_DGRAD, false, true, 1>(g, rd, rows, p.dp[l], 1, s);
      else if (dz_transposed) launch_gemm<EPI_DGRAD, false, true, 3>(g, rd, rows, p.dp[l], 1, s);
      else                    launch_gemm<EPI_DGRAD, false, true, 0>(g, rd, rows, p.dp[l], 1, s);
      dz_transposed = next_transposed;
      kend(hook, kind);
    }

    if (!gather_rides) {
      // (right before its reader, which then finds it in the caches; ahead of the output layer the first layer's
      // weight gradient took 73 instead of 59 us at 16384 x 1024)
      kbegin(hook, KK_MLP_GATHER_T, 0, arows * p.d[0] * 4.0);
      plan_note("gather_t", 64, 64, 1);
      ABS_LAUNCH_K(mlp_gather_t_kernel, dim3(rows / 64, p.dp[0] / 64), dim3(256), s, a.X, p.d[0], (const uint32_t*)rowidx,
                   at<uint16_t>(a, p.off_xgt), p.ldm);
      kend(hook, KK_MLP_GATHER_T);
    }

    // ---- weight gradients.  U = 1: one contraction over all stacked rows = the K-of-N
    //      reduction, split over row ranges for occupancy, then update + snapshot per layer.
    //      U > 1: split a = the rows of upload a, applied to that upload's private model.
    // U = 1: first layer first.  The update of a layer (Eq. 3: bound by memory) does not get a launch of
    // its own but rides along in the NEXT layer's weight-gradient launch (bound by the matrix cores) as
    // that launch's last workgroups: they take the CUs its last wave of tiles leaves idle and its tail,
    // and there is no gap between two launches.  Only the last layer's update, small, is launched by
    // itself.  (cfg 5, same box, microseconds per round at K = 32 / K = 128: 680 / 1838 with an update
    // launch per layer, 650 / 1811 this way.  Hiding the second layer's update under the first layer's
    // product instead - order 1, 0, 2, no runs: a quarter of the CUs is idle there at K = 32 - gave
    // 631 / 1807, but the product that bounds the round then carries another layer's traffic and its
    // own figure, 0.31 of the matrix peak instead of 0.37 with runs, says little about it.)
    // The bias update (column sums of every dZ_l, complete since the backward pass) rides along in the
    // same way: as the very last workgroups of the last layer's weight-gradient launch.
    BiasCore bias{};
    bias.L = L;
    int bias_cols = 0;
    for (int l = 0; l < L; ++l) {
      bias.col_begin[l] = bias_cols; bias_cols += p.d[l + 1];
      bias.colsum[l] = at<float>(a, p.off_colsum[l + 1]); bias.ldcs[l] = (size_t)p.dp[l + 1];
      bias.b_off[l] = p.b_off[l];
      bias.prow[l] = (local ? p.Bp : rows) / (l == L - 1 ? ce_block : 64);
    }
    bias.col_begin[L] = bias_cols;
    bias.w_cur = local ? wbase : ring + (size_t)rd.slot_cur * p.slot_stride;
    bias.w_next = local ? priv : ring + (size_t)rd.slot_next * p.slot_stride;
    if (stile) {
      launch_steps(a, rd, rows, arows, stile, sdirect, bias, bias_cols, own, s, hook);
      continue;
    }
    int pend = -1, pend_split = 0, pend_q = 0;   // layer whose partials are complete and whose update is still due (its splits or run length)
    for (int li = 0; li < L; ++li) {
      const int l = local ? L - 1 - li : li;
      GemmArgs g{};
      if (li == L - 1) {
        g.bias_per = (bias_cols + 15) / 16;
        g.bias_blocks = g.bias_per * (local ? K : 1);
        g.bias_upd = bias;
        plan_note("with_biases", 16, 1, 1);
      }
      g.A = l == 0 ? at<uint16_t>(a, p.off_xgt) : at<uint16_t>(a, p.off_ht[l]); g.lda = p.ldm;
      g.Bt = at<uint16_t>(a, p.off_dzt[l + 1]); g.ldb = p.ldm;
      const int ksteps = rows / BK;
      const int nsplit = wgrad_split(p, l, rows, local ? K : 0);
      g.ksteps_total = ksteps;
      g.ksteps_per_split = local ? p.Bp / BK : (ksteps + nsplit - 1) / nsplit;
      if (!local) {
        g.outf = at<float>(a, p.off_partial[l]); g.ldof = (size_t)p.dp[l + 1] + kPartialPad;
        g.split_stride = (size_t)p.dp[l] * (p.dp[l + 1] + kPartialPad);
      }
      int run_parts = 0;
      const int run_q = local ? 0 : wgrad_runs(p, l, rows, nsplit, &run_parts);
      if (run_q) { g.sk_q = run_q; }
      double upd_bytes = 0.0;
      if (pend >= 0) {
        g.nsplit = nsplit;
        const bool big = gemm_is_big(false, false, g, p.dp[l], p.dp[l + 1], nsplit);
        g.pig_upd = global_update_args(a, pend, rd, pend_split);
        if (pend_q) { g.pig_upd.sk_q = pend_q; g.pig_upd.sk_ksteps = ksteps; g.pig_upd.sk_nt = p.dp[pend + 1] / TN3; }
        g.pig_tj = big && p.d[pend + 1] >= 256 ? 256 : 64;
        g.pig_blocks = (((p.d[pend + 1] + g.pig_tj - 1) / g.pig_tj) * ((p.d[pend] + 63) / 64) + 7) / 8 * 8;
        upd_bytes = (double)p.d[pend] * p.d[pend + 1] * (4.0 * (pend_split + 2) + (pend >= 1 ? 4.0 : 2.0));
        plan_note("with_update_of_previous", 64, g.pig_tj, pend_split);
        pend = -1;
      }
      const int kind = l == 0 ? KK_MLP_WGRAD_L1 : l == L - 1 ? KK_MLP_WGRAD_OUT : KK_MLP_WGRAD;
      kbegin(hook, kind, 2.0 * arows * p.d[l] * p.d[l + 1],
             arows * (p.d[l] + p.d[l + 1]) * 2.0 +
                 (double)nsplit * p.d[l] * p.d[l + 1] * (local ? l >= 1 ? 12.0 : 10.0 : 4.0) + upd_bytes);
      if (l == 0 && wg0_direct) { g.A = a.X; g.lda = (size_t)p.d[0]; g.a_rowidx = rowidx; }
      if (local) {
        LocalUpdate& lu = g.local_upd;
        uint16_t* pw = at<uint16_t>(a, p.off_priv_shadow);
        lu.own = own; lu.cur = wbase + p.w_off[l]; lu.next = priv + p.w_off[l]; lu.stride = p.slot_stride;
        lu.wn = l >= 1 ? pw + p.wn_off[l] : nullptr; lu.ldwn = (size_t)p.ld[l + 1];
        lu.wt = pw + p.wt_off[l]; lu.ldwt = (size_t)p.ld[l]; lu.shadow_stride = p.shadow_stride;
        lu.d_in = p.d[l]; lu.d_out = p.d[l + 1];
        if (l == 0 && wg0_direct) launch_gemm<EPI_WGRAD, false, false, 4>(g, rd, p.dp[l], p.dp[l + 1], nsplit, s);
        else                      launch_gemm<EPI_WGRAD, false, false, 5>(g, rd, p.dp[l], p.dp[l + 1], nsplit, s);
      } else if (l == 0 && wg0_direct) {
        launch_gemm<EPI_WGRAD, false, false, 2>(g, rd, p.dp[l], p.dp[l + 1], nsplit, s);
      } else if (l == 0) {
        launch_gemm<EPI_WGRAD, false, false, 1>(g, rd, p.dp[l], p.dp[l + 1], nsplit, s);
      } else {
        launch_gemm<EPI_WGRAD, false, false, 0>(g, rd, p.dp[l], p.dp[l + 1], nsplit, s);
      }
      kend(hook, kind);
      const int parts = run_q ? run_parts : nsplit;          // partials per tile (at most, with runs)
      if (!local && update_rows_aligned(p, l) && li + 1 < L) { pend = l; pend_split = parts; pend_q = run_q; }
      else if (!local) launch_update(a, l, rd, UPD_GLOBAL, parts, s, hook, run_q, ksteps);
    }
  }

  if (local) {
    // ---- Eq. 3 over the uploads' changes, then update + snapshot per layer
    DeltaArgs d{};
    d.ring = ring; d.slot_stride = p.slot_stride;
    d.priv = priv;
    d.D = at<float>(a, p.off_delta);
    d.P = p.P;
    d.L = L;
    for (int l = 0; l < L; ++l) { d.b_off[l] = p.b_off[l]; d.b_len[l] = p.d[l + 1]; }
    d.w_cur = ring + (size_t)rd.slot_cur * p.slot_stride;
    d.w_next = ring + (size_t)rd.slot_next * p.slot_stride;
    kbegin(hook, KK_DELTA_UPDATE, 2.0 * K * p.P, (2.0 * K + 1.0) * p.P * 4.0);
    ABS_LAUNCH_K(mlp_delta_kernel, dim3((unsigned)((p.P + 255) / 256)), dim3(256), s, d, rd);
    kend(hook, KK_DELTA_UPDATE);
    for (int l = L - 1; l >= 0; --l) launch_update(a, l, rd, UPD_DELTA, 1, s, hook);
  }
  return t_plan ? hipSuccess : hipGetLastError();
}

std::string mlp_round_plan(const abs_config& cfg, int K) {
  MlpArgs a{};
  const char* why = nullptr;
  if (K < 1 || K > cfg.N || !mlp_plan(cfg, a.plan, &why)) return std::string();
  RoundDesc rd{};
  rd.K = K;
  NullHook nh;
  std::string out;
  t_plan = &out;
  (void)launch_mlp_round(a, rd, nullptr, &nh);   // records, launches nothing, touches no memory
  t_plan = nullptr;
  if (!out.empty() && out.back() == ' ') out.pop_back();
  return out;
}

hipError_t launch_mlp_eval(const MlpArgs& a, uint32_t slot, const EvalArgs& e, hipStream_t s, LaunchHook* hook) {
  const MlpPlan& p = a.plan;
  if (e.cap < p.Mp) return hipErrorInvalidValue;
  uint32_t* rowidx = at<uint32_t>(a, p.off_rowidx);
  int32_t* label = at<int32_t>(a, p.off_label);
  hipError_t err = launch_eval_clear(e, s);
  const bool aligned = ((uintptr_t)e.X & 15) == 0;
  for (int64_t row0 = 0; row0 < e.n_rows && err == hipSuccess; row0 += p.Mp) {
    const int n = (int)(e.n_rows - row0 < p.Mp ? e.n_rows - row0 : p.Mp);
    const uint16_t* X = (const uint16_t*)e.X;
    if (!aligned) {
      // (the transposed minibatch's place, dp_0 x ldm elements: every round that reads it writes it first)
      uint16_t* const staged = at<uint16_t>(a, p.off_xgt);
      const size_t n8 = (size_t)n * p.d[0] / 8;
      hook->begin(KK_EVAL, 0, 4.0 * n * p.d[0]);
      mlp_eval_align_kernel<<<dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, s>>>(X + (size_t)row0 * p.d[0], (uint4*)staged, n8);
      hook->end(KK_EVAL);
      X = staged;
    }
    RoundDesc rd{};                               // every block of Bp rows uses the same version
    rd.K = (n + p.Bp - 1) / p.Bp;
    for (int k = 0; k < rd.K; ++k) rd.w[k].slot = slot;
    const int rows = rd.K * p.Bp;
    hook->begin(KK_EVAL, 0, 12.0 * n);
    mlp_eval_index_kernel<<<dim3((rows + 255) / 256), dim3(256), 0, s>>>(rowidx, label, (const int32_t*)e.y, row0,
                                                                              aligned ? row0 : 0, n, rows);
    hook->end(KK_EVAL);
    mlp_forward(a, X, rd, rows, (double)n, at<float>(a, p.off_ring), at<uint16_t>(a, p.off_shadow),
                false, false, -1, s, hook);
    hook->begin(KK_EVAL, 8.0 * n * p.d[p.L], 4.0 * n * p.d[p.L]);
    const dim3 grid((n + 3) / 4), block(256);
    const float* Z = at<float>(a, p.off_z);
    const size_t ld = (size_t)p.dp[p.L];
    switch (p.dp[p.L] / 64) {
      case 1: mlp_eval_rows_kernel<1><<<grid, block, 0, s>>>(Z, ld, p.d[p.L], label, n, e.rowloss, e.correct); break;
      case 2: mlp_eval_rows_kernel<2><<<grid, block, 0, s>>>(Z, ld, p.d[p.L], label, n, e.rowloss, e.correct); break;
      default: mlp_eval_rows_kernel<4><<<grid, block, 0, s>>>(Z, ld, p.d[p.L], label, n, e.rowloss, e.correct); break;
    }
    hook->end(KK_EVAL);
    err = hipGetLastError();
    if (err == hipSuccess) err = launch_eval_reduce(e, n, s, hook);
  }
  return err;
}

}  // namespace abs_impl

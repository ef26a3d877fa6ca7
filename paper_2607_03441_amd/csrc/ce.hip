// Token-weighted cross-entropy through a frozen LM head (Sec. 3.3, Eq. 10) on gfx950: the
// forward of both dtypes, the float32 backward, and the row and episode kernels around the bf16
// backward, whose two contractions run fused in one persistent kernel (ce_fused.hip).
//
// Forward (logits never leave the chip): one GEMM z = h W^T over (vocab tile, row tile) whose
// epilogue reduces every row of the tile to (max, sum exp(z - max)). A row kernel merges the
// partials into lse and w * CE; an episode kernel sums those in a fixed order into
// loss_e = (1/L_e) sum w_t CE_t.
//
// bf16 forward + backward: every row takes its own label logit r_t = z_{t,y_t} (ce_label_logit,
// one dot product per row) as the exponent reference, so the fused kernel forms
// e_tv = exp(z_tv - r_t) without knowing lse:
//     sigma_t = sum_{v != y_t} e_tv,   lse_t = r_t + log1p(sigma_t),   CE_t = log1p(sigma_t)
//     dL/dh_t = (w_t / L_e) (U_t - sigma_t W_{y_t}) / (1 + sigma_t),  U_t = sum_{v != y_t} e_tv W_v
// which is (w_t / L_e)(softmax(z_t) - onehot(y_t)) W rewritten; the label term is kept out of
// the sums, so nothing cancels when p_y is close to 1. ce_row_final turns the fused kernel's
// per-(row, vocab tile) sums into sigma, lse and the row losses. r_t is one of the row's logits,
// so sigma never underflows; a logit more than 64 above r_t (a label with probability below
// e^-64) could overflow e and raises a flag, on which the exact path (forward lse, then the fused
// kernel on coef exp(z - lse)) reruns in full, overwriting the outputs. Its kernels read the flag
// first and return at once when it is clear.
//
// bf16 GEMMs: MFMA v_mfma_f32_32x32x16_bf16 through the core in gemm_core.hpp (256x256 tiles on 8
// waves, 128x128 on 4 for small problems; XCD-aware tile order).
// f32 path: 64x64 tiles on the float32 MFMA running the three-GEMM algorithm (forward,
// dZ = coef (softmax - onehot) staged per block of rows and vocabulary, dH = dZ W, its vocabulary
// range split over workgroups when there are few tiles); it serves the float32 configuration.
#include "common.hpp"
#include "gemm_core.hpp"
#include "internal.hpp"
#include "lds_limit.hpp"

namespace attt {


// ------------------------------------------------------------------------------------------
// bf16 forward. The GEMM runs transposed, z^T = W h^T, so a workgroup tile is 256 vocab rows x
// 256 token columns and every lane holds, for one token, 64 of the tile's vocab logits in its
// registers: the per-token (max, sum exp) needs one cross-lane step (lanes l and l+32) and a
// two-wave merge in LDS, instead of a 32-lane shuffle tree per row.
// ------------------------------------------------------------------------------------------
template <class C>
__device__ __forceinline__ void ce_fwd_bf16_body(
    const bf16_t* __restrict__ h, const bf16_t* __restrict__ W, int N, int d, int V, int tiles_v,
    int tiles_t, float2* __restrict__ partials, int n_vb) {
  extern __shared__ __align__(16) uint8_t smem[];
  int tv, tt;
  tile_of(blockIdx.x, tiles_v, tiles_t, tv, tt);
  const int v0 = tv * C::BM, t0 = tt * C::BN;
  f32x16 acc[C::TM][C::TN];
  mfma_mainloop<C>(W + (int64_t)v0 * d, d, V - v0, h + (int64_t)t0 * d, d, N - t0, d,
                   reinterpret_cast<bf16_t*>(smem), acc);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / C::WGN, wn = wave % C::WGN;
  float* red_m = reinterpret_cast<float*>(smem);  // [WGM][BN]
  float* red_s = red_m + C::WGM * C::BN;
  const int vbase = v0 + wm * C::WTM;
#pragma unroll
  for (int j = 0; j < C::TN; ++j) {
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (vbase + i * 32 + mfma_row(r, lane) < V) mx = fmaxf(mx, acc[i][j][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    float s = 0.0f;
    if (mx != -INFINITY) {
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (vbase + i * 32 + mfma_row(r, lane) < V) s += __expf(acc[i][j][r] - mx);
    }
    s += __shfl_xor(s, 32, 64);
    if (lane < 32) {
      const int tl = wn * C::WTN + j * 32 + lane;
      red_m[wm * C::BN + tl] = mx;
      red_s[wm * C::BN + tl] = s;
    }
  }
  __syncthreads();
  for (int tl = threadIdx.x; tl < C::BN; tl += C::NT) {
    const int t = t0 + tl;
    if (t >= N) continue;
    float m = red_m[tl], s = red_s[tl];
#pragma unroll
    for (int w = 1; w < C::WGM; ++w) lse_merge(m, s, red_m[w * C::BN + tl], red_s[w * C::BN + tl]);
    partials[(int64_t)t * n_vb + tv] = make_float2(m, s);
  }
}

template <class C>
__global__ __launch_bounds__(C::NT) void ce_fwd_bf16_kernel(
    const bf16_t* __restrict__ h, const bf16_t* __restrict__ W, int N, int d, int V, int tiles_v,
    int tiles_t, float2* __restrict__ partials, int n_vb) {
  ce_fwd_bf16_body<C>(h, W, N, d, V, tiles_v, tiles_t, partials, n_vb);
}

// The same kernel launched by the overflow guard: returns at once unless *gate != 0.
template <class C>
__global__ __launch_bounds__(C::NT) void ce_guard_fwd_bf16_kernel(
    const bf16_t* __restrict__ h, const bf16_t* __restrict__ W, int N, int d, int V, int tiles_v,
    int tiles_t, float2* __restrict__ partials, int n_vb, const int* __restrict__ gate) {
  if (*gate == 0) return;
  ce_fwd_bf16_body<C>(h, W, N, d, V, tiles_v, tiles_t, partials, n_vb);
}

// Label logit z_{t, y_t} = h_t . W_{y_t} (float32 accumulation), one wave per row.
__global__ __launch_bounds__(256) void ce_label_logit_bf16_kernel(const bf16_t* __restrict__ h,
                                                                  const bf16_t* __restrict__ W,
                                                                  const int32_t* __restrict__ labels,
                                                                  int N, int d, int V,
                                                                  float* __restrict__ label_logit,
                                                                  int* __restrict__ flag) {
  const int lane = threadIdx.x & 63;
  if (flag && blockIdx.x == 0 && threadIdx.x == 0) *flag = 0;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= N) return;
  const int y = labels[row];
  if (y < 0 || y >= V) {  // outside the contract: make the loss NaN instead of reading out of bounds
    if (lane == 0) label_logit[row] = __int_as_float(0x7FC00000);
    return;
  }
  const bf16_t* hr = h + (int64_t)row * d;
  const bf16_t* wr = W + (int64_t)y * d;
  float s = 0.0f;
  for (int k = lane * 8; k < d; k += 64 * 8) {
    const u32x4 a = *reinterpret_cast<const u32x4*>(hr + k);
    const u32x4 b = *reinterpret_cast<const u32x4*>(wr + k);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s = fmaf(bf16_bits_to_f32(a[e] & 0xFFFFu), bf16_bits_to_f32(b[e] & 0xFFFFu), s);
      s = fmaf(bf16_bits_to_f32(a[e] >> 16), bf16_bits_to_f32(b[e] >> 16), s);
    }
  }
  s = group_sum<64>(s);
  if (lane == 0) label_logit[row] = s;
}

// Rows [r0, r0 + R) after the fused backward: sigma_t = sum of the vocab-tile partials (fixed
// order), lse_t = r_t + log1p(sigma_t), row loss w_t log1p(sigma_t), and (when sa, sb are given)
// the row scales coef / (1 + sigma), coef sigma / (1 + sigma). One wave per row.
__global__ __launch_bounds__(256) void ce_row_final_kernel(int r0, int R, const float* __restrict__ sig_part,
                                                           int n_vb, const float* __restrict__ label_logit,
                                                           const float* __restrict__ weights,
                                                           const float* __restrict__ coef,
                                                           float* __restrict__ lse,
                                                           float* __restrict__ rowloss,
                                                           float* __restrict__ sa, float* __restrict__ sb) {
  const int lane = threadIdx.x & 63;
  const int local = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (local >= R) return;
  const int64_t row = (int64_t)r0 + local;
  float sum = 0.0f;
  for (int i = lane; i < n_vb; i += 64) sum += sig_part[row * n_vb + i];
  sum = group_sum<64>(sum);
  if (lane == 0) {
    const float ce = log1pf(sum);
    const float inv = __fdiv_rn(1.0f, 1.0f + sum);
    const float c = coef[row];
    lse[row] = label_logit[row] + ce;
    rowloss[row] = weights[row] * ce;
    if (sa) sa[row] = c * inv;
    if (sb) sb[row] = c * (sum * inv);
  }
}

// coef_t = w_t / L_e for every row of the batch's episodes, 256 rows per block.
__global__ __launch_bounds__(256) void ce_coef_kernel(CeEpBatch b, const float* __restrict__ weights,
                                                      float* __restrict__ coef) {
  int ei = 0;
  while (ei + 1 < b.count && b.e[ei + 1].block_begin <= (int)blockIdx.x) ++ei;
  const CeEp E = b.e[ei];
  const int local = ((int)blockIdx.x - E.block_begin) * 256 + threadIdx.x;
  if (local >= E.L) return;
  const int64_t row = E.row0 + local;
  coef[row] = __fdiv_rn(weights[row], (float)E.L);
}

// ------------------------------------------------------------------------------------------
// f32 path: 64x64 tiles on v_mfma_f32_32x32x2_f32 (float32 products and sums), 4 waves with one
// 32x32 block each. K advances 32 per step through two LDS buffers; the next step's global loads
// are in flight while the current one computes, and a step costs one barrier. These GEMMs are
// small (1 GFLOP at 512 x 256 x 4096) and bound by the latency of their K walk and by how many
// tiles there are, not by the matrix cores. At that size forward and dZ take 17 us each (25 with
// VALU tiles and no prefetch) and dH 16 us plus 4 for its split sums (290 us unsplit, 32 workgroups).
// ------------------------------------------------------------------------------------------
constexpr int kVT = 64, kVK = 32;
constexpr int kVP = kVK + 4;   // LDS pitch (floats) of a row-major [64][32] operand tile
constexpr int kVPn = kVT + 8;  // LDS pitch of a [32][64] tile (rows 4 apart fall in other banks)
constexpr int kVTile = kVT * kVP > kVK * kVPn ? kVT * kVP : kVK * kVPn;

// acc = A[0:64, 0:K] * op(B) of this wave's 32x32 block: NT reads B as [64, K] (K-contiguous), NN
// as [K, 64]. Rows at or past mval (nval columns) and K past kval_a (A) or kval_b (B, NN) read as
// zero. The k slots of an MFMA pair follow the 16-byte reads of a row-major tile (slot i of lane
// half h is k = 8 j + 4 h + i), the same order for both operands.
template <bool NN>
__device__ __forceinline__ void f32_mainloop(const float* __restrict__ A, int64_t lda, int mval,
                                             const float* __restrict__ B, int64_t ldb, int nval, int k_begin,
                                             int k_end, int kval_b, float (&lds)[2][2][kVTile], f32x16& acc) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, hi = lane >> 5;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  const int lr = tid >> 3, lk = (tid & 7) * 4;   // row-major tiles: rows lr and lr + 32, k lk .. +3
  const int kr = tid >> 4, nc = (tid & 15) * 4;  // [k][64] tiles: k kr and kr + 16, columns nc .. +3
  f32x4 ra[2], rb[2];
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  auto load = [&](int k0) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = lr + 32 * u;
      ra[u] = row < mval && k0 + lk < k_end ? *reinterpret_cast<const f32x4*>(A + (int64_t)row * lda + k0 + lk) : zero;
      if (!NN) {
        rb[u] = row < nval && k0 + lk < k_end ? *reinterpret_cast<const f32x4*>(B + (int64_t)row * ldb + k0 + lk) : zero;
      } else {
        const int k = k0 + kr + 16 * u;
        rb[u] = k < k_end && k < kval_b && nc < nval ? *reinterpret_cast<const f32x4*>(B + (int64_t)k * ldb + nc) : zero;
      }
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      *reinterpret_cast<f32x4*>(&lds[buf][0][(lr + 32 * u) * kVP + lk]) = ra[u];
      if (!NN)
        *reinterpret_cast<f32x4*>(&lds[buf][1][(lr + 32 * u) * kVP + lk]) = rb[u];
      else
        *reinterpret_cast<f32x4*>(&lds[buf][1][(kr + 16 * u) * kVPn + nc]) = rb[u];
    }
  };
  load(k_begin);
  store(0);
  int buf = 0;
  for (int k0 = k_begin; k0 < k_end; k0 += kVK, buf ^= 1) {
    // this step's tiles are stored, and every wave is done with the other buffer
    __syncthreads();
    const bool more = k0 + kVK < k_end;
    if (more) load(k0 + kVK);
    const float* As = &lds[buf][0][(wm * 32 + l32) * kVP + 4 * hi];
    const float* Bs = &lds[buf][1][NN ? 4 * hi * kVPn + wn * 32 + l32 : (wn * 32 + l32) * kVP + 4 * hi];
#pragma unroll
    for (int j = 0; j < kVK / 8; ++j) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(As + 8 * j);
      f32x4 b;
      if (!NN) {
        b = *reinterpret_cast<const f32x4*>(Bs + 8 * j);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = Bs[(8 * j + i) * kVPn];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], acc, 0, 0, 0);
    }
    if (more) store(buf ^ 1);
  }
}

// Forward, transposed like the bf16 form (z^T = W h^T): each lane holds 16 logits of one token, and
// a token's (max, sum exp) meets across the lane pair and the two waves of its columns.
__global__ __launch_bounds__(256) void ce_fwd_f32_kernel(const float* __restrict__ h,
                                                         const float* __restrict__ W,
                                                         const int32_t* __restrict__ labels, int N,
                                                         int d, int V, int tiles_m,
                                                         float2* __restrict__ partials, int n_vb,
                                                         float* __restrict__ label_logit) {
  __shared__ __align__(16) float lds[2][2][kVTile];
  __shared__ float red[2][2][kVT];  // (max, sum) of each wave row's half of the tile
  const int tm = blockIdx.x % tiles_m, tn = blockIdx.x / tiles_m;
  const int t0 = tm * kVT, v0 = tn * kVT;
  f32x16 acc;
  f32_mainloop<false>(W + (int64_t)v0 * d, d, V - v0, h + (int64_t)t0 * d, d, N - t0, 0, d, 0, lds, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int tl = wn * 32 + (lane & 31), row = t0 + tl;
  const int vb = v0 + wm * 32;
  const int y = row < N ? labels[row] : -1;
  float mx = -INFINITY;
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (vb + mfma_row(r, lane) < V) mx = fmaxf(mx, acc[r]);
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  const float m0 = mx != -INFINITY ? mx : 0.0f;  // no finite maximum: -inf adds exp(-inf) = 0, a NaN itself
  float s = 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int v = vb + mfma_row(r, lane);
    if (v < V) {
      s += expf(acc[r] - m0);
      if (v == y) label_logit[row] = acc[r];
    }
  }
  s += __shfl_xor(s, 32, 64);
  if (s != s) mx = s;  // the maxima and merges pass NaNs over: without a finite logit beside it, one would be lost
  if (lane < 32) {
    red[0][wm][tl] = mx;
    red[1][wm][tl] = s;
  }
  __syncthreads();
  if (threadIdx.x < kVT && t0 + (int)threadIdx.x < N) {
    const int t = t0 + threadIdx.x;
    float m = red[0][0][threadIdx.x], sum = red[1][0][threadIdx.x];
    lse_merge(m, sum, red[0][1][threadIdx.x], red[1][1][threadIdx.x]);
    partials[(int64_t)t * n_vb + tn] = make_float2(m, sum);
    // outside the contract: the row's loss term becomes NaN instead of reading stale memory
    const int yt = labels[t];
    if (tn == 0 && (yt < 0 || yt >= V)) label_logit[t] = __int_as_float(0x7FC00000);
  }
}

__global__ __launch_bounds__(256) void ce_dz_f32_kernel(const float* __restrict__ h,
                                                        const float* __restrict__ W,
                                                        const int32_t* __restrict__ labels,
                                                        const float* __restrict__ lse,
                                                        const float* __restrict__ coef, int r0,
                                                        int R, int d, int c0, int cend, int V,
                                                        int tiles_m, float* __restrict__ dz,
                                                        int ldz) {
  __shared__ __align__(16) float lds[2][2][kVTile];
  const int tm = blockIdx.x % tiles_m, tn = blockIdx.x / tiles_m;
  const int m0 = tm * kVT, n0 = tn * kVT;
  f32x16 acc;  // transposed: vocabulary entries on the rows, tokens on the columns
  f32_mainloop<false>(W + (int64_t)(c0 + n0) * d, d, cend - (c0 + n0), h + (int64_t)(r0 + m0) * d, d, R - m0, 0, d, 0,
                      lds, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rl = m0 + (wave & 1) * 32 + (lane & 31);
  if (rl >= R) return;
  const int row = r0 + rl;
  const float l = lse[row], c = coef[row];
  const int y = labels[row];
  const bool bad = y < 0 || y >= V;  // outside the contract: NaN gradient row
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int cl = n0 + (wave >> 1) * 32 + mfma_row(4 * q, lane);
    f32x4 g;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int col = c0 + cl + e;
      g[e] = 0.0f;
      if (col < V) g[e] = bad ? __int_as_float(0x7FC00000) : c * (expf(acc[4 * q + e] - l) - (col == y ? 1.0f : 0.0f));
    }
    *reinterpret_cast<f32x4*>(dz + (int64_t)rl * ldz + cl) = g;
  }
}

// dH rows [r0, r0 + R) (+)= dZ chunk . W[c0 : c0 + K]. With `splits` > 1 the K range of a tile is cut
// into splits of `kper` (a multiple of kVK) whose sums go to `part` [splits][R][d]; a second kernel
// adds them in order.
__global__ __launch_bounds__(256) void ce_dh_f32_kernel(const float* __restrict__ dz, int ldz,
                                                        const float* __restrict__ W, int r0, int R,
                                                        int d, int c0, int K, int kval,
                                                        int tiles_m, int tiles, int kper,
                                                        float* __restrict__ part, float* __restrict__ grad,
                                                        int first) {
  __shared__ __align__(16) float lds[2][2][kVTile];
  const int sp = blockIdx.x / tiles, tile = blockIdx.x - sp * tiles;
  const int tm = tile % tiles_m, tn = tile / tiles_m;
  const int m0 = tm * kVT, n0 = tn * kVT;
  f32x16 acc;
  f32_mainloop<true>(dz + (int64_t)m0 * ldz, ldz, R - m0, W + (int64_t)c0 * d + n0, d, d - n0, sp * kper,
                     min(K, sp * kper + kper), kval, lds, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = n0 + (wave & 1) * 32 + (lane & 31);
  if (col >= d) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int rl = m0 + (wave >> 1) * 32 + mfma_row(r, lane);
    if (rl >= R) continue;
    if (part) {
      part[((int64_t)sp * R + rl) * d + col] = acc[r];
    } else {
      const int64_t o = (int64_t)(r0 + rl) * d + col;
      grad[o] = first ? acc[r] : grad[o] + acc[r];
    }
  }
}

// grad [n] (+)= sum over the splits of part [splits][n], in split order; n is a multiple of 8.
__global__ __launch_bounds__(256) void ce_dh_reduce_kernel(const float* __restrict__ part, int splits, int64_t n,
                                                           float* __restrict__ grad, int first) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n) return;
  f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int sp = 0; sp < splits; ++sp) s += *reinterpret_cast<const f32x4*>(part + sp * n + i);
  if (!first) s += *reinterpret_cast<const f32x4*>(grad + i);
  *reinterpret_cast<f32x4*>(grad + i) = s;
}

// ------------------------------------------------------------------------------------------
// Row and episode reductions, LM-head transpose.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void ce_row_reduce_body(
    CeEpBatch b, const float2* __restrict__ partials, int n_vb,
    const float* __restrict__ label_logit, const float* __restrict__ weights,
    float* __restrict__ lse, float* __restrict__ coef, float* __restrict__ rowloss) {
  int ei = 0;
  while (ei + 1 < b.count && b.e[ei + 1].block_begin <= (int)blockIdx.x) ++ei;
  const CeEp E = b.e[ei];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int local = ((int)blockIdx.x - E.block_begin) * 4 + wave;
  if (local >= E.L) return;
  const int64_t row = E.row0 + local;
  float m = -INFINITY, s = 0.0f;
  for (int i = lane; i < n_vb; i += 64) {
    const float2 p = partials[row * n_vb + i];
    lse_merge(m, s, p.x, p.y);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float m2 = __shfl_xor(m, o, 64), s2 = __shfl_xor(s, o, 64);
    lse_merge(m, s, m2, s2);
  }
  if (lane == 0) {
    const float l = m + logf(s);
    const float w = weights[row];
    lse[row] = l;
    coef[row] = __fdiv_rn(w, (float)E.L);
    rowloss[row] = w * (l - label_logit[row]);
  }
}

__global__ __launch_bounds__(256) void ce_row_reduce_kernel(
    CeEpBatch b, const float2* __restrict__ partials, int n_vb,
    const float* __restrict__ label_logit, const float* __restrict__ weights,
    float* __restrict__ lse, float* __restrict__ coef, float* __restrict__ rowloss) {
  ce_row_reduce_body(b, partials, n_vb, label_logit, weights, lse, coef, rowloss);
}

// The same kernel launched by the overflow guard: returns at once unless *gate != 0.
__global__ __launch_bounds__(256) void ce_guard_row_reduce_kernel(
    CeEpBatch b, const float2* __restrict__ partials, int n_vb,
    const float* __restrict__ label_logit, const float* __restrict__ weights,
    float* __restrict__ lse, float* __restrict__ coef, float* __restrict__ rowloss,
    const int* __restrict__ gate) {
  if (*gate == 0) return;
  ce_row_reduce_body(b, partials, n_vb, label_logit, weights, lse, coef, rowloss);
}

// One 1024-thread workgroup per episode: every thread sums its rows in order (loads issued
// eight at a time), then the waves' sums meet in a fixed order.
constexpr int kLossThreads = 1024;
__device__ __forceinline__ void ce_loss_body(
    CeEpBatch b, const float* __restrict__ rowloss, float* __restrict__ loss) {
  const CeEp E = b.e[blockIdx.x];
  double acc = 0.0;
#pragma unroll 8
  for (int i = threadIdx.x; i < E.L; i += kLossThreads) acc += (double)rowloss[E.row0 + i];
  acc = wave_sum_f64(acc);
  constexpr int kWaves = kLossThreads / 64;
  __shared__ double part[kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) part[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kWaves; ++w) t += part[w];
    loss[b.first + blockIdx.x] = E.L > 0 ? (float)(t / (double)E.L) : 0.0f;
  }
}

__global__ __launch_bounds__(kLossThreads) void ce_loss_kernel(
    CeEpBatch b, const float* __restrict__ rowloss, float* __restrict__ loss) {
  ce_loss_body(b, rowloss, loss);
}

// The same kernel launched by the overflow guard: returns at once unless *gate != 0.
__global__ __launch_bounds__(kLossThreads) void ce_guard_loss_kernel(
    CeEpBatch b, const float* __restrict__ rowloss, float* __restrict__ loss,
    const int* __restrict__ gate) {
  if (*gate == 0) return;
  ce_loss_body(b, rowloss, loss);
}

// W [V, d] -> WT [d, Vp] in 64 x 64 tiles: 16-byte global reads along d, 16-byte global writes
// along V, through an LDS tile whose padded pitch (66) keeps the column reads conflict-free.
__global__ __launch_bounds__(256) void ce_head_transpose_kernel(const bf16_t* __restrict__ W, int V,
                                                                int d, int Vp,
                                                                bf16_t* __restrict__ WT) {
  constexpr int P = 66;
  __shared__ __align__(16) bf16_t t[64 * P];
  const int v0 = blockIdx.x * 64, j0 = blockIdx.y * 64;
  const int r = threadIdx.x >> 2, c = threadIdx.x & 3;  // row r, 16 columns from 16c
  {
    const int v = v0 + r, j = j0 + 16 * c;
    u32x4 x0 = u32x4{0u, 0u, 0u, 0u}, x1 = u32x4{0u, 0u, 0u, 0u};
    if (v < V && j < d) {
      const u32x4* src = reinterpret_cast<const u32x4*>(W + (int64_t)v * d + j);
      x0 = src[0];
      if (j + 8 < d) x1 = src[1];
    }
    uint32_t* dst = reinterpret_cast<uint32_t*>(t + r * P + 16 * c);  // 4-byte aligned: P even
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      dst[e] = x0[e];
      dst[4 + e] = x1[e];
    }
  }
  __syncthreads();
  const int j = j0 + r, v = v0 + 16 * c;  // output row j, 16 vocab entries from v
  if (j < d && v < Vp) {
    uint32_t w[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      w[e] = (uint32_t)t[(16 * c + 2 * e) * P + r] | ((uint32_t)t[(16 * c + 2 * e + 1) * P + r] << 16);
    u32x4* out = reinterpret_cast<u32x4*>(WT + (int64_t)j * Vp + v);
    out[0] = u32x4{w[0], w[1], w[2], w[3]};
    out[1] = u32x4{w[4], w[5], w[6], w[7]};
  }
}

// ------------------------------------------------------------------------------------------
// Launchers
// ------------------------------------------------------------------------------------------
template <class C>
static hipError_t fwd_bf16(const bf16_t* h, const bf16_t* W, int N, int d, int V, float2* partials,
                           int n_vb, const int* gate, hipStream_t s) {
  static LdsLimit plain, guard;
  if (hipError_t e = plain.raise((const void*)ce_fwd_bf16_kernel<C>, 160 * 1024)) return e;
  if (hipError_t e = guard.raise((const void*)ce_guard_fwd_bf16_kernel<C>, 160 * 1024)) return e;
  const int tv = (V + C::BM - 1) / C::BM, tt = (N + C::BN - 1) / C::BN;
  KernelTimer t(gate ? K_CE_GUARD : K_CE_FWD, s);
  if (gate)
    hipLaunchKernelGGL(ce_guard_fwd_bf16_kernel<C>, dim3(tv * tt), dim3(C::NT), C::LDS, s, h, W, N, d, V,
                       tv, tt, partials, n_vb, gate);
  else
    hipLaunchKernelGGL(ce_fwd_bf16_kernel<C>, dim3(tv * tt), dim3(C::NT), C::LDS, s, h, W, N, d, V, tv,
                       tt, partials, n_vb);
  return hipGetLastError();
}

hipError_t launch_ce_fwd(int dtype, CeGemmShape t, const void* h, const void* W,
                         const int32_t* labels, int N, int d, int V, float2* partials, int n_vb,
                         float* label_logit, const int* gate, hipStream_t s) {
  if (N == 0) return hipSuccess;
  if (dtype == 1) {
    const bf16_t* hb = static_cast<const bf16_t*>(h);
    const bf16_t* Wb = static_cast<const bf16_t*>(W);
    if (t.bm == 256) return fwd_bf16<CfgBig>(hb, Wb, N, d, V, partials, n_vb, gate, s);
    return fwd_bf16<CfgSmall>(hb, Wb, N, d, V, partials, n_vb, gate, s);
  }
  const int tm = (N + kVT - 1) / kVT, tn = (V + kVT - 1) / kVT;
  KernelTimer tt(K_CE_FWD, s);
  hipLaunchKernelGGL(ce_fwd_f32_kernel, dim3(tm * tn), dim3(256), 0, s,
                     static_cast<const float*>(h), static_cast<const float*>(W), labels, N, d, V, tm,
                     partials, n_vb, label_logit);
  return hipGetLastError();
}

hipError_t launch_ce_label(const void* h, const void* W, const int32_t* labels, int N, int d, int V,
                           float* label_logit, int* flag, hipStream_t s) {
  if (N == 0) return hipSuccess;
  KernelTimer t(K_CE_LABEL, s);
  hipLaunchKernelGGL(ce_label_logit_bf16_kernel, dim3((N + 3) / 4), dim3(256), 0, s,
                     static_cast<const bf16_t*>(h), static_cast<const bf16_t*>(W), labels, N, d, V,
                     label_logit, flag);
  return hipGetLastError();
}

hipError_t launch_ce_row_reduce(const CeEpBatch& b, int total_blocks, const float2* partials,
                                int n_vb, const float* label_logit, const float* weights,
                                float* lse, float* coef, float* rowloss, const int* gate,
                                hipStream_t s) {
  if (total_blocks <= 0) return hipSuccess;
  KernelTimer t(gate ? K_CE_GUARD : K_CE_ROW_REDUCE, s);
  if (gate)
    hipLaunchKernelGGL(ce_guard_row_reduce_kernel, dim3(total_blocks), dim3(256), 0, s, b, partials, n_vb,
                       label_logit, weights, lse, coef, rowloss, gate);
  else
    hipLaunchKernelGGL(ce_row_reduce_kernel, dim3(total_blocks), dim3(256), 0, s, b, partials, n_vb,
                       label_logit, weights, lse, coef, rowloss);
  return hipGetLastError();
}

hipError_t launch_ce_loss(const CeEpBatch& b, const float* rowloss, float* loss, const int* gate,
                          hipStream_t s) {
  if (b.count <= 0) return hipSuccess;
  KernelTimer t(gate ? K_CE_GUARD : K_CE_LOSS, s);
  if (gate)
    hipLaunchKernelGGL(ce_guard_loss_kernel, dim3(b.count), dim3(kLossThreads), 0, s, b, rowloss, loss, gate);
  else
    hipLaunchKernelGGL(ce_loss_kernel, dim3(b.count), dim3(kLossThreads), 0, s, b, rowloss, loss);
  return hipGetLastError();
}

hipError_t launch_ce_coef(const CeEpBatch& b, int total_blocks, const float* weights, float* coef,
                          hipStream_t s) {
  if (total_blocks <= 0) return hipSuccess;
  KernelTimer t(K_CE_ROW_REDUCE, s);
  hipLaunchKernelGGL(ce_coef_kernel, dim3(total_blocks), dim3(256), 0, s, b, weights, coef);
  return hipGetLastError();
}

hipError_t launch_ce_head_transpose(const void* W, int V, int d, int Vp, void* WT, hipStream_t s) {
  KernelTimer t(K_CE_HEAD_T, s);
  hipLaunchKernelGGL(ce_head_transpose_kernel, dim3((Vp + 63) / 64, (d + 63) / 64), dim3(256), 0, s,
                     static_cast<const bf16_t*>(W), V, d, Vp, static_cast<bf16_t*>(WT));
  return hipGetLastError();
}

hipError_t launch_ce_row_final(int r0, int R, const float* sig_part, int n_vb, const float* label_logit,
                               const float* weights, const float* coef, float* lse, float* rowloss,
                               float* sa, float* sb, hipStream_t s) {
  if (R == 0) return hipSuccess;
  KernelTimer t(K_CE_ROW_REDUCE, s);
  hipLaunchKernelGGL(ce_row_final_kernel, dim3((R + 3) / 4), dim3(256), 0, s, r0, R, sig_part, n_vb,
                     label_logit, weights, coef, lse, rowloss, sa, sb);
  return hipGetLastError();
}

hipError_t launch_ce_bwd_dz(const float* h, const float* W, const int32_t* labels, const float* lse,
                            const float* coef, int r0, int R, int d, int c0, int Vc, int V, float* dz, int ldz,
                            hipStream_t s) {
  if (R == 0) return hipSuccess;
  const int tm = (R + kVT - 1) / kVT, tn = (Vc + kVT - 1) / kVT;
  const int cend = min(c0 + Vc, V);
  KernelTimer tt(K_CE_BWD_DZ, s);
  hipLaunchKernelGGL(ce_dz_f32_kernel, dim3(tm * tn), dim3(256), 0, s, h, W, labels, lse, coef, r0, R, d, c0, cend,
                     V, tm, dz, ldz);
  return hipGetLastError();
}

hipError_t launch_ce_bwd_dh(const float* dz, int ldz, const float* W, int r0, int R, int d, int c0, int K, int V,
                            int splits, float* part, float* grad, bool first, hipStream_t s) {
  if (R == 0) return hipSuccess;
  const int tm = (R + kVT - 1) / kVT, tn = (d + kVT - 1) / kVT;
  const int kper = ((K + splits - 1) / splits + kVK - 1) / kVK * kVK;
  KernelTimer tt(K_CE_BWD_DH, s);
  hipLaunchKernelGGL(ce_dh_f32_kernel, dim3(tm * tn * splits), dim3(256), 0, s, dz, ldz, W, r0, R, d, c0, K, V - c0,
                     tm, tm * tn, kper, splits > 1 ? part : nullptr, grad, first ? 1 : 0);
  if (splits > 1) {
    const int64_t n = (int64_t)R * d;
    hipLaunchKernelGGL(ce_dh_reduce_kernel, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, s, part, splits, n,
                       grad + (int64_t)r0 * d, first ? 1 : 0);
  }
  return hipGetLastError();
}

}  // namespace attt

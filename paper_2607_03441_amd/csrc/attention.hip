// Backward of one adapted attention block (the step before the LoRA gradient: dY_q, dY_k, dY_v
// are the adapter's upstream gradients; Sec. 3.1, Appendix C). Causal attention with grouped
// key/value heads, per episode; head dimension 128; bf16 inputs and outputs, float32
// accumulation. With S = scale Q K^T, P = softmax(S) over the allowed keys, O = P V:
//   D = rowsum(dO * O),  dP = dO V^T,  dS = P * (dP - D),
//   dQ = scale dS K,  dK = scale dS^T Q,  dV = P^T dO.
// Three passes, each recomputing S from Q and K on v_mfma_f32_16x16x32_bf16 over blocks of 64
// keys, 256 threads (four waves of 16 rows, or of 32 query rows), blocks in the causal order with
// the longest rows first, the next block's global loads in flight while the current one computes:
//   attn_fwd_stats_kernel  per (query head, 64- or 128-query block): lse and D (online softmax; D as
//                          the softmax-weighted sum of dP = dO V^T, so O is never formed)
//   attn_dkdv_kernel       per (key/value head, 64- or 128-key block, part of its queries): dK and dV
//                          accumulated in registers over every query head of the group and every
//                          later query block, in a fixed order (no atomics), 512 threads
//   attn_dkdv_short_kernel the same for a 64-key block with half the threads and LDS, where walks are short
//   attn_dq_kernel         per (query head, 64- or 128-query block): dQ over the allowed key blocks
// The operand that stays (a wave's 16 or 32 queries, or its keys) is held in registers, or for
// attn_dkdv_kernel in LDS, as the B operand of the score products, so each lane ends up with scores
// of its own rows. The probabilities (or dS) of those rows then enter the second product (P^T dO,
// dS^T Q, dS K) directly as the A operand: the contraction index is the one the lane's registers run
// over, in the order they hold it, and the B operand is read in the same order from the row-major LDS
// tile with transposing reads (ds_read_tr16_b64). Every block goes to LDS once, row-major, with
// 16-byte stores, into one of two buffers (one barrier per block). Blocks strictly below the
// diagonal skip the causal and ragged-row masks.
// P and dS enter their second products as bf16 pairs hi + lo (two MFMA passes, about 16
// significant bits): those sums mix signs (dS even sums to zero over each row), and a single
// bf16 rounding of P or dS would show in their small elements. The final bf16 rounding of the
// outputs is then the main error.
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"
#include "lds_limit.hpp"

namespace attt {

namespace {
constexpr int DH = 128;     // head dimension
constexpr int BLK = 64;     // query / key rows per block
constexpr int KBLK = kAttnKeyBlock;  // keys per block of a split dK / dV walk
constexpr int PR = DH + 8;  // LDS pitch of a [64][128] tile (bf16): 272 B, conflict-free b128 reads
constexpr float kLog2e = 1.4426950408889634f;

// LDS: two buffers, so that the next block is stored while the current one is read and a step
// needs one barrier. A buffer of the per-query kernels holds the K and V tiles; one of the
// per-key kernels holds the Q and dO tiles, then lse and D of the block's 64 queries.
constexpr int kTileBytes = BLK * PR * 2;
constexpr int kKvBuf = 2 * kTileBytes;
constexpr int kQoBuf = 2 * kTileBytes + 2 * BLK * 4;

__device__ __forceinline__ bf16_t* kv_tile(uint8_t* smem, int buf, int t) {
  return reinterpret_cast<bf16_t*>(smem + buf * kKvBuf + t * kTileBytes);
}
__device__ __forceinline__ bf16_t* qo_tile(uint8_t* smem, int buf, int t) {
  return reinterpret_cast<bf16_t*>(smem + buf * kQoBuf + t * kTileBytes);
}
__device__ __forceinline__ float* qo_stats(uint8_t* smem, int buf) {  // lse [64], then D [64]
  return reinterpret_cast<float*>(smem + buf * kQoBuf + 2 * kTileBytes);
}

__device__ __forceinline__ bf16_t f2bf(float x) { return (bf16_t)(pack_bf16x2(x, 0.0f) & 0xFFFFu); }

// The block a workgroup works on: episode, head, block index. Workgroups start in launch
// order, so the long causal rows go first: the last query blocks for the per-query kernels
// (`late_first`), the first key blocks for the per-key kernel.
__device__ __forceinline__ void attn_locate(const AttnBatch& b, int heads, bool late_first, int& ei, int& head,
                                            int& blk) {
  ei = 0;
  while (ei + 1 < b.count && b.e[ei + 1].wg_begin <= (int)blockIdx.x) ++ei;
  const int local = (int)blockIdx.x - b.e[ei].wg_begin;
  const int nb = b.e[ei].blocks;
  head = local % heads;
  blk = late_first ? nb - 1 - local / heads : local / heads;
}

}  // namespace

// This wave's 16 queries (or keys) as MFMA B operands over the head dimension: lane (l16, q4) holds row
// `row` (its own) at columns 32 s + 8 q4 .. +7 for s = 0..3. Rows at or past nvalid read as zero.
__device__ __forceinline__ void load_row_frags(bf16x8 (&f)[4], const bf16_t* src, int64_t stride, int row,
                                               int nvalid, int q4) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    if (row < nvalid) v = *reinterpret_cast<const u32x4*>(src + (int64_t)row * stride + 32 * s + 8 * q4);
    f[s] = __builtin_bit_cast(bf16x8, v);
  }
}

// Rows [0, BLK) of a [rows][DH] block, staged in LDS row-major (pitch PR). Thread tid takes rows
// 4 (tid / 16) .. +3 and columns 8 (tid % 16) .. +7: fetch_block issues its four 16-byte loads
// (rows >= nvalid read as zero), store_block writes them with four 16-byte stores.
// The loads go through one buffer descriptor over the block's valid rows (base and range in
// scalar registers, 32-bit offsets per lane): rows at or past nvalid fall outside its range and
// read as zero. A 64-row block spans less than 2^30 bytes (heads < 2^16, checked on the host).
__device__ __forceinline__ void fetch_block(u32x4 (&v)[4], const bf16_t* src, int64_t stride, int nvalid, int tid) {
  const int r0 = (tid >> 4) * 4, c0 = (tid & 15) * 8;
  const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(src, nvalid > 0 ? (int)(((int64_t)(nvalid - 1) * stride + DH) * 2) : 0);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    v[i] = __builtin_bit_cast(
        u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (uint32_t)(((int64_t)(r0 + i) * stride + c0) * 2), 0, 0));
}

__device__ __forceinline__ void store_block(const u32x4 (&v)[4], bf16_t* dst, int tid) {
  const int r0 = (tid >> 4) * 4, c0 = (tid & 15) * 8;
#pragma unroll
  for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4*>(dst + (r0 + i) * PR + c0) = v[i];
}

// hi = RN(x), lo = RN(x - hi) of the eight values of an MFMA operand, as bf16x8 pairs.
__device__ __forceinline__ void split_frag(const float (&x)[8], bf16x8& hi, bf16x8& lo) {
  u32x4 h, l;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = pack_bf16x2(x[2 * i], x[2 * i + 1]);
    l[i] = pack_bf16x2(x[2 * i] - bf16_bits_to_f32(h[i] & 0xFFFFu), x[2 * i + 1] - bf16_bits_to_f32(h[i] >> 16));
  }
  hi = __builtin_bit_cast(bf16x8, h);
  lo = __builtin_bit_cast(bf16x8, l);
}

// B operand of the second products over the 32 rows (queries, or keys) of chunk u, from a
// row-major [64][DH] tile (pitch PR) through transposing LDS reads: lane (l16, q4) receives
// column c0 + l16 at rows 32 u + 4 q4 .. +3 and 32 u + 16 + 4 q4 .. +3, the order in which the
// P / dS fragments hold them. ds_read_tr16_b64 hands, within each group of 16 lanes, lane i the
// element i mod 4 of lanes 4e + i/4 (e = 0..3), so lane 4e + c of group q4 addresses row
// 32 u + 4 q4 + e (then 16 rows further) at columns c0 + 4c .. +3.
__device__ __forceinline__ bf16x8 trfrag(const bf16_t* R, int c0, int u, int lane) {
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) v4s* lds_v4s;
  const int q4 = lane >> 4, e = (lane >> 2) & 3, c = lane & 3;
  const bf16_t* p = R + (32 * u + 4 * q4 + e) * PR + c0 + 4 * c;
  const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p));
  const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p + 16 * PR));
  const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
  return __builtin_bit_cast(bf16x8, u32x4{a.x, a.y, b.x, b.y});
}

// lse and D = rowsum(dO * O) of one (query head, 64 QT-query block). Wave w owns queries 16 QT w ..
// + 16 QT - 1 as QT tiles of 16; their Q and dO fragments stay in registers. Per key block: S^T =
// K Q^T and dP^T = V dO^T with the keys on the MFMA rows, each K and V fragment read from LDS once
// for all tiles, so each lane holds 16 scores of each of its QT queries and the online softmax
// of a query is a reduction over the lane's registers and its three partner lanes (lanes l,
// l + 16, l + 32, l + 48 hold the same queries). O = P V is never formed: since
// O = sum_k P_k V_k, D = sum_k P_k (dO . V_k) = sum_k P_k dP_k, so each lane keeps, beside the
// running softmax sum, the running sum of p dP over its keys, both rescaled by the same factor
// when the running max grows; the four partial sums of a query are added at the end.
template <int QT>
__global__ __launch_bounds__(256, 2) void attn_fwd_stats_kernel(AttnArgs a, AttnBatch b) {
  constexpr int QBLK = 64 * QT;
  int ei, h, qb;
  attn_locate(b, a.heads, true, ei, h, qb);
  const AttnEp E = b.e[ei];
  const int kh = h / (a.heads / a.kv_heads);
  const int q0 = qb * QBLK, nq = min(QBLK, E.L - q0);
  extern __shared__ __align__(16) uint8_t smem[];  // two buffers of [K tile][V tile], [64][PR] each
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l16 = lane & 15, q4 = lane >> 4;
  const int64_t qs = (int64_t)a.heads * DH, ks = (int64_t)a.kv_heads * DH;
  bf16x8 qf[QT][4], of[QT][4];
#pragma unroll
  for (int c = 0; c < QT; ++c) {
    const int qry = 16 * QT * w + 16 * c + l16;
    load_row_frags(qf[c], a.q + ((int64_t)(E.row0 + q0) * a.heads + h) * DH, qs, qry, nq, q4);
    load_row_frags(of[c], a.dout + ((int64_t)(E.row0 + q0) * a.heads + h) * DH, qs, qry, nq, q4);
  }
  const float sl = a.scale * kLog2e;
  // per query tile: running max (base 2, the same in the query's four lanes), and this lane's
  // running sums of p and of p dP over its keys
  float m[QT], l[QT], dacc[QT];
#pragma unroll
  for (int c = 0; c < QT; ++c) m[c] = -INFINITY, l[c] = 0.0f, dacc[c] = 0.0f;
  u32x4 fk[4], fv[4];
  auto fetch = [&](int kb) {
    const int k0 = kb * BLK, nk = min(BLK, E.L - k0);
    fetch_block(fk, a.k + ((int64_t)(E.row0 + k0) * a.kv_heads + kh) * DH, ks, nk, tid);
    fetch_block(fv, a.v + ((int64_t)(E.row0 + k0) * a.kv_heads + kh) * DH, ks, nk, tid);
  };
  const int kb_last = (q0 + nq - 1) / BLK;  // the key block of the block's last query
  const int wq0 = q0 + 16 * QT * w;              // this wave's first query
  fetch(0);
  store_block(fk, kv_tile(smem, 0, 0), tid);
  store_block(fv, kv_tile(smem, 0, 1), tid);
  for (int kb = 0; kb <= kb_last; ++kb) {
    const int k0 = kb * BLK, nk = min(BLK, E.L - k0);
    // This block's tiles are stored, and every wave is done with the other buffer.
    __syncthreads();
    if (kb < kb_last) fetch(kb + 1);  // the next key block loads while this one computes
    // A wave whose queries all precede the block has nothing to add (it still takes part in
    // the barriers and the stores).
    if (k0 <= wq0 + 16 * QT - 1) {
      const bf16_t* Ks = kv_tile(smem, kb & 1, 0);
      const bf16_t* Vs = kv_tile(smem, kb & 1, 1);
      // S^T[16 tt + 4 q4 + r][query] and dP^T likewise, for both query tiles
      f32x4 st[QT][4], dp[QT][4];
#pragma unroll
      for (int c = 0; c < QT; ++c)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) st[c][tt] = f32x4{0, 0, 0, 0}, dp[c][tt] = f32x4{0, 0, 0, 0};
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
          const bf16x8 ak = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const u32x4*>(Ks + (16 * tt + l16) * PR + 32 * s4 + 8 * q4));
          const bf16x8 av = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const u32x4*>(Vs + (16 * tt + l16) * PR + 32 * s4 + 8 * q4));
#pragma unroll
          for (int c = 0; c < QT; ++c) {
            st[c][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ak, qf[c][s4], st[c][tt], 0, 0, 0);
            dp[c][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, of[c][s4], dp[c][tt], 0, 0, 0);
          }
        }
      // each K and V fragment pair is read just ahead of its four products, which bounds the
      // registers held by reads in flight
#pragma unroll
      for (int n = 0; n < 16; ++n) {
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 2 * QT, 0);
      }
      // online softmax (base-2 exponent of scale * S) over this block's keys 16 tt + 4 q4 + r.
      // A whole key block that ends at or before the wave's first query is entirely allowed:
      // no mask there.
      auto softmax = [&](auto masked) {
#pragma unroll
        for (int c = 0; c < QT; ++c) {
          const int qry = 16 * QT * w + 16 * c + l16;
          float mx = -INFINITY, sum = 0.0f, dsum = 0.0f;
#pragma unroll
          for (int tt = 0; tt < 4; ++tt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int kl = 16 * tt + 4 * q4 + r;
              float v = st[c][tt][r] * sl;
              if constexpr (decltype(masked)::value) v = (k0 + kl <= q0 + qry && kl < nk) ? v : -INFINITY;
              st[c][tt][r] = v;
              mx = fmaxf(mx, v);
            }
          mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
          mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
          const float mn = fmaxf(m[c], mx);
#pragma unroll
          for (int tt = 0; tt < 4; ++tt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              float p = __builtin_amdgcn_exp2f(st[c][tt][r] - mn);
              if constexpr (decltype(masked)::value) p = (st[c][tt][r] == -INFINITY) ? 0.0f : p;
              sum += p;
              dsum += p * dp[c][tt][r];
            }
          const float alpha = (m[c] == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(m[c] - mn);
          l[c] = l[c] * alpha + sum;
          dacc[c] = dacc[c] * alpha + dsum;
          m[c] = mn;
        }
      };
      if (k0 + BLK - 1 <= wq0 && nk == BLK)
        softmax(std::false_type{});
      else
        softmax(std::true_type{});
    }
    if (kb < kb_last) {
      store_block(fk, kv_tile(smem, (kb + 1) & 1, 0), tid);
      store_block(fv, kv_tile(smem, (kb + 1) & 1, 1), tid);
    }
  }
#pragma unroll
  for (int c = 0; c < QT; ++c) {
    const int qry = 16 * QT * w + 16 * c + l16;
    float lc = l[c], dc = dacc[c];
    lc += __shfl_xor(lc, 16, 64);
    lc += __shfl_xor(lc, 32, 64);
    dc += __shfl_xor(dc, 16, 64);
    dc += __shfl_xor(dc, 32, 64);
    if (q4 == 0 && qry < nq) {
      const int64_t t = (int64_t)h * a.N + E.row0 + q0 + qry;
      a.lse[t] = m[c] / kLog2e + logf(lc);
      a.dsum[t] = dc / lc;
    }
  }
}

// Key blocks of an episode (64 KT keys each) whose walk of g steps per query block has a whole piece
// number `split`: the first ones, since a block's walk is KT g steps shorter than that of the one before.
template <int KT>
__host__ __device__ __forceinline__ int whole_pieces(int L, int g, int split, int chunk) {
  const int64_t left = (int64_t)g * ((L + BLK - 1) / BLK) - (int64_t)(split + 1) * chunk;
  return left >= 0 ? (int)(left / (KT * g)) + 1 : 0;
}

// dK, dV of one (key/value head, 64 KT-key block) over a range of its (query block, query head) steps.
// Eight waves: wave (kw, qw) owns keys 16 KT kw .. + 16 KT - 1, as KT tiles of 16, and half qw (32
// queries) of every 64-query step. S = Q K^T and dP = dO V^T with the queries on the MFMA rows (two tiles
// of 16) and the wave's keys on the columns; K and V come from LDS tiles kept for the whole walk. Each
// lane holds 8 (query, key) values of its own key of a tile. P and dS = P (dP - D) then feed dV += P^T dO
// and dK += dS^T Q straight from those registers as the A operand: the contraction runs over the 32
// queries, whose 8 values a lane holds (tile rows 4 q4 .. +3 of two tiles) are its k slots; the B operand
// reads the dO and Q tiles through transposing reads in the same query order. At the end the two halves
// of the queries are added through LDS (one order, no atomics).
// LDS reads bound the layout of 16 keys and 64 queries per wave (2304 of 3312 cycles a 64-key step against
// 1536 of MFMA): here a wave's 96 products read 48 KiB instead of 64 per 32. K in registers spilled 34
// of them (1935 us); the matrix phases at raised wave priority, so that one wave's products run under the
// other's softmax, took 1594 -> 1558 us. 8192 rows, 32 heads over 8: 1726 -> 1558 us.
template <int KT>
__global__ __launch_bounds__(512, 2) void attn_dkdv_kernel(AttnArgs a, AttnBatch b) {
  constexpr int KEYS = 64 * KT;
  int ei = 0;
  while (ei + 1 < b.count && b.e[ei + 1].wg_begin <= (int)blockIdx.x) ++ei;
  const AttnEp E = b.e[ei];
  const int g = a.heads / a.kv_heads;
  // The pieces of `chunk` steps first, then the rests of the walks, the longest first, so that the last
  // round is filled by short ones. Where `chunk` is m times the KT g steps by which the walks of
  // neighbouring blocks differ, blocks c, c + m, ... leave the same rest; otherwise the launch is one round
  // and the order does not matter. (By block, with
  // workgroups past a walk's end that left at once, and rests in the blocks' order: 2048 rows, 16 heads over
  // 4, 6 pieces 120 us, here 81; 8192 rows, 8 over 2, 4 pieces 686 us, here 455.)
  int local = (int)blockIdx.x - E.wg_begin, split = 0;
  for (int n; split < b.splits && local >= (n = whole_pieces<KT>(E.L, g, split, b.chunk) * a.kv_heads); ++split)
    local -= n;
  const int kh = local % a.kv_heads;
  int kb = local / a.kv_heads;
  if (split == b.splits && b.splits > 1 && b.chunk % (KT * g) == 0) {
    const int m = b.chunk / (KT * g), q = E.blocks / m, r = E.blocks % m;
    int c = g * ((E.L + BLK - 1) / BLK) % b.chunk / (KT * g) + 1;  // the longest rests
    for (int n;; ++c) {
      if (c == m) c = 0;
      n = q + (c < r);
      if (kb < n) break;  // the classes hold all E.blocks blocks
      kb -= n;
    }
    kb = c + m * kb;
  }
  const int k0 = kb * KEYS, nk = min(KEYS, E.L - k0);
  const int nqb = (E.L + BLK - 1) / BLK;
  // (query block, query head) steps: query blocks from the last down to the key block's first, the
  // group's query heads inside. Every workgroup of a key/value head walks the same blocks in the same
  // order, so those running together on an XCD read each Q and dO block from its L2.
  const int steps = g * (nqb - kb * KT);
  if (split == b.splits) split = steps / b.chunk;
  const int i0 = split * b.chunk, i1 = min(steps, i0 + b.chunk);
  if (i0 >= i1) return;  // a walk of whole pieces has no rest
  extern __shared__ __align__(16) uint8_t smem[];  // two buffers of [Q tile][dO tile][lse][D], the V tile
  bf16_t* Vs = reinterpret_cast<bf16_t*>(smem + 2 * kQoBuf);
  bf16_t* Ks = Vs + KEYS * PR;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = w & 3, qw = w >> 2;
  const int l16 = lane & 15, q4 = lane >> 4;
  const int64_t qs = (int64_t)a.heads * DH, ks = (int64_t)a.kv_heads * DH;
  const int64_t krow = ((int64_t)(E.row0 + k0) * a.kv_heads + kh) * DH;
  const int r0 = (tid >> 4) * 2, c0 = (tid & 15) * 8;  // a thread's two rows of a 64-row block, and columns
  {
    const int bytes = (int)(((int64_t)(nk - 1) * ks + DH) * 2);
    const __amdgpu_buffer_rsrc_t rk = buffer_rsrc(a.k + krow, bytes), rv = buffer_rsrc(a.v + krow, bytes);
#pragma unroll
    for (int i = 0; i < 2 * KT; ++i) {
      const int r = (i >> 1) * BLK + r0 + (i & 1);
      const uint32_t off = (uint32_t)(((int64_t)r * ks + c0) * 2);
      *reinterpret_cast<u32x4*>(Ks + r * PR + c0) =
          __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, off, 0, 0));
      *reinterpret_cast<u32x4*>(Vs + r * PR + c0) =
          __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rv, off, 0, 0));
    }
  }
  f32x4 dk[KT][8], dv[KT][8];
#pragma unroll
  for (int c = 0; c < KT; ++c)
#pragma unroll
    for (int j = 0; j < 8; ++j) dk[c][j] = f32x4{0, 0, 0, 0}, dv[c][j] = f32x4{0, 0, 0, 0};
  const float sl = a.scale * kLog2e;
  u32x4 fq[2], fo[2];
  float fs = 0.0f;
  auto fetch = [&](int i) {
    const int h = kh * g + i % g, q0 = (nqb - 1 - i / g) * BLK, nq = min(BLK, E.L - q0);
    const int64_t row = ((int64_t)(E.row0 + q0) * a.heads + h) * DH;
    const int bytes = (int)(((int64_t)(nq - 1) * qs + DH) * 2);
    const __amdgpu_buffer_rsrc_t rq = buffer_rsrc(a.q + row, bytes), ro = buffer_rsrc(a.dout + row, bytes);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const uint32_t off = (uint32_t)(((int64_t)(r0 + r) * qs + c0) * 2);
      fq[r] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rq, off, 0, 0));
      fo[r] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ro, off, 0, 0));
    }
    if (tid < 2 * BLK) {
      const int ql = tid & (BLK - 1);
      const int64_t t = (int64_t)h * a.N + E.row0 + q0 + ql;
      if (tid < BLK)
        fs = ql < nq ? a.lse[t] * kLog2e : INFINITY;  // absent rows: P = 0
      else
        fs = ql < nq ? a.dsum[t] : 0.0f;
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      *reinterpret_cast<u32x4*>(qo_tile(smem, buf, 0) + (r0 + r) * PR + c0) = fq[r];
      *reinterpret_cast<u32x4*>(qo_tile(smem, buf, 1) + (r0 + r) * PR + c0) = fo[r];
    }
    if (tid < 2 * BLK) qo_stats(smem, buf)[tid] = fs;
  };
  fetch(i0);
  stage(0);
  for (int i = i0; i < i1; ++i) {
    const int buf = (i - i0) & 1;
    const int qw0 = (nqb - 1 - i / g) * BLK + 32 * qw;  // this wave's first query
    // This step's tiles are stored, and every wave is done with the other buffer.
    __syncthreads();
    if (i + 1 < i1) fetch(i + 1);  // the next step's blocks load while this one computes
    // A wave whose queries all precede its keys has nothing to add.
    if (qw0 + 31 >= k0 + 16 * KT * kw) {
      const bf16_t* Qs = qo_tile(smem, buf, 0);
      const bf16_t* dOs = qo_tile(smem, buf, 1);
      const float* lse_s = qo_stats(smem, buf) + 32 * qw;
      const float* d_s = lse_s + BLK;
      __builtin_amdgcn_s_setprio(1);
      // S[16 t + 4 q4 + r][key] and dP likewise, for both key tiles
      f32x4 st[KT][2], dp[KT][2];
#pragma unroll
      for (int c = 0; c < KT; ++c)
#pragma unroll
        for (int t = 0; t < 2; ++t) st[c][t] = f32x4{0, 0, 0, 0}, dp[c][t] = f32x4{0, 0, 0, 0};
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) {
        bf16x8 bk[KT], bv[KT];
#pragma unroll
        for (int c = 0; c < KT; ++c) {
          bk[c] = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const u32x4*>(Ks + (16 * KT * kw + 16 * c + l16) * PR + 32 * s4 + 8 * q4));
          bv[c] = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const u32x4*>(Vs + (16 * KT * kw + 16 * c + l16) * PR + 32 * s4 + 8 * q4));
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const bf16x8 aq = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const u32x4*>(Qs + (32 * qw + 16 * t + l16) * PR + 32 * s4 + 8 * q4));
          const bf16x8 ao = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const u32x4*>(dOs + (32 * qw + 16 * t + l16) * PR + 32 * s4 + 8 * q4));
#pragma unroll
          for (int c = 0; c < KT; ++c) {
            st[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, bk[c], st[c][t], 0, 0, 0);
            dp[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ao, bv[c], dp[c][t], 0, 0, 0);
          }
        }
      }
      // P and dS of this lane's 8 (query, key) pairs of each key tile, in fragment order: slot i is
      // query 4 q4 + i (i < 4) or 16 + 4 q4 + i - 4. Queries at or after the wave's last key see all of
      // its keys: no mask there. (Keys past the episode only reach rows that are not written.)
      bf16x8 ph[KT], pl[KT], sh[KT], slo[KT];
      auto probs = [&](auto masked) {
#pragma unroll
        for (int c = 0; c < KT; ++c) {
          float pv[8], dsv[8];
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const f32x4 ls = *reinterpret_cast<const f32x4*>(lse_s + 16 * t + 4 * q4);
            const f32x4 dd = *reinterpret_cast<const f32x4*>(d_s + 16 * t + 4 * q4);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              float p = __builtin_amdgcn_exp2f(st[c][t][r] * sl - ls[r]);
              if constexpr (decltype(masked)::value)
                p = (k0 + 16 * KT * kw + 16 * c + l16 <= qw0 + 16 * t + 4 * q4 + r) ? p : 0.0f;
              pv[4 * t + r] = p;
              dsv[4 * t + r] = p * (dp[c][t][r] - dd[r]);
            }
          }
          split_frag(pv, ph[c], pl[c]);
          split_frag(dsv, sh[c], slo[c]);
        }
      };
      __builtin_amdgcn_s_setprio(0);
      if (qw0 >= k0 + 16 * KT * kw + 16 * KT - 1)
        probs(std::false_type{});
      else
        probs(std::true_type{});
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const bf16x8 bo = trfrag(dOs, 16 * j, qw, lane), bq = trfrag(Qs, 16 * j, qw, lane);
#pragma unroll
        for (int c = 0; c < KT; ++c) {
          dv[c][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph[c], bo, dv[c][j], 0, 0, 0);
          dv[c][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl[c], bo, dv[c][j], 0, 0, 0);
          dk[c][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sh[c], bq, dk[c][j], 0, 0, 0);
          dk[c][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(slo[c], bq, dk[c][j], 0, 0, 0);
        }
      }
    }
    __builtin_amdgcn_s_setprio(0);
    if (i + 1 < i1) stage(buf ^ 1);
  }
  // Both query halves: per key tile the waves of the second half hand over dK, those of the first dV,
  // and each adds the other's to its own. 64 KiB of the tiles' LDS.
  f32x4* ex = reinterpret_cast<f32x4*>(smem);
#pragma unroll
  for (int c = 0; c < KT; ++c) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) ex[(w * 8 + j) * 64 + lane] = qw ? dk[c][j] : dv[c][j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const f32x4 o = ex[((w ^ 4) * 8 + j) * 64 + lane];
      if (qw)
        dv[c][j] += o;
      else
        dk[c][j] += o;
    }
  }
  // D of tile (c, j): lane (l16, q4), register r -> key 32 kw + 16 c + 4 q4 + r, column 16 j + l16
  const float os = qw ? 1.0f : a.scale;
  float* part = b.part + (((int64_t)(E.blocks0 + kb) * a.kv_heads + kh) * b.splits + split) * (2 * KEYS * DH) +
                qw * KEYS * DH;
  bf16_t* outp = qw ? a.dv : a.dk;
#pragma unroll
  for (int c = 0; c < KT; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int kr = 16 * KT * kw + 16 * c + 4 * q4 + r;
      if (kr >= nk) continue;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float v = (qw ? dv[c][j][r] : dk[c][j][r]) * os;
        if (b.splits > 1)
          part[kr * DH + 16 * j + l16] = v;
        else
          outp[krow + (int64_t)kr * ks + 16 * j + l16] = f2bf(v);
      }
    }
}

// dK, dV of one (key/value head, 64-key block) by four waves and 68 KiB of LDS, so that two workgroups share
// a CU and one's start and end run under the other's steps: for walks that are short, or many and even. Wave
// w owns keys 16 w .. 16 w + 15; their K and V fragments stay in registers. Per query block: S = Q K^T and dP = dO V^T with the queries on
// the MFMA rows (four tiles of 16) and this wave's keys on the columns, so each lane holds 16
// (query, key) values of its own key. P and dS = P (dP - D) then feed dV += P^T dO and
// dK += dS^T Q straight from those registers as the A operand: the contraction runs over the
// queries, and the 8 values a lane holds per 32-query chunk (tile rows 4 q4 .. +3 of two tiles)
// are its k slots; the B operand reads the transposed dO and Q tiles in the same query order.
// A step takes a CU 1.42 us (1.40 per 64 keys of the 128-key kernel) and a workgroup's start and end 3.4
// (7.3): 64 episodes of 64 rows, 32 heads over 32: 46 us against 70 and 87 for the kernel above on 64 and on
// 128 keys; 3 episodes of 1000 rows, 40 over 40: 124, 159 and 127; 8192 rows, 32 over 8: 1726 against 1509.
__global__ __launch_bounds__(256, 2) void attn_dkdv_short_kernel(AttnArgs a, AttnBatch b) {
  int ei, kh, kb;
  attn_locate(b, a.kv_heads, false, ei, kh, kb);
  const AttnEp E = b.e[ei];
  const int g = a.heads / a.kv_heads;
  const int k0 = kb * BLK, nk = min(BLK, E.L - k0);
  extern __shared__ __align__(16) uint8_t smem[];  // two buffers of [Q tile][dO tile][lse][D]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l16 = lane & 15, q4 = lane >> 4;
  const int key = 16 * w + l16;  // this lane's key in the block
  const int64_t qs = (int64_t)a.heads * DH, ks = (int64_t)a.kv_heads * DH;
  bf16x8 kf[4], vf[4];
  load_row_frags(kf, a.k + ((int64_t)(E.row0 + k0) * a.kv_heads + kh) * DH, ks, key, nk, q4);
  load_row_frags(vf, a.v + ((int64_t)(E.row0 + k0) * a.kv_heads + kh) * DH, ks, key, nk, q4);
  f32x4 dk[8], dv[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) dk[j] = f32x4{0, 0, 0, 0}, dv[j] = f32x4{0, 0, 0, 0};
  const float sl = a.scale * kLog2e;
  const int nqb = (E.L + BLK - 1) / BLK;
  // (query block, query head) steps: query blocks from the last down to kb, the group's query
  // heads inside. Every workgroup of a key/value head walks the same blocks in the same order
  // (starting at the last, stopping at its own key block), so those running together on an XCD
  // read each Q and dO block from its L2.
  const int steps = g * (nqb - kb);
  u32x4 fq[4], fo[4];
  float fl = INFINITY, fd = 0.0f;
  auto fetch = [&](int i) {
    const int h = kh * g + i % g, q0 = (nqb - 1 - i / g) * BLK, nq = min(BLK, E.L - q0);
    fetch_block(fq, a.q + ((int64_t)(E.row0 + q0) * a.heads + h) * DH, qs, nq, tid);
    fetch_block(fo, a.dout + ((int64_t)(E.row0 + q0) * a.heads + h) * DH, qs, nq, tid);
    if (tid < BLK) {
      const int64_t t = (int64_t)h * a.N + E.row0 + q0 + tid;
      fl = tid < nq ? a.lse[t] * kLog2e : INFINITY;  // absent rows: P = 0
      fd = tid < nq ? a.dsum[t] : 0.0f;
    }
  };
  auto stage = [&](int buf) {
    store_block(fq, qo_tile(smem, buf, 0), tid);
    store_block(fo, qo_tile(smem, buf, 1), tid);
    if (tid < BLK) qo_stats(smem, buf)[tid] = fl, qo_stats(smem, buf)[BLK + tid] = fd;
  };
  fetch(0);
  stage(0);
  for (int i = 0; i < steps; ++i) {
    const int q0 = (nqb - 1 - i / g) * BLK;
    // This step's tiles are stored, and every wave is done with the other buffer.
    __syncthreads();
    if (i + 1 < steps) fetch(i + 1);  // the next step's blocks load while this one computes
    const bf16_t* Qs = qo_tile(smem, i & 1, 0);
    const bf16_t* dOs = qo_tile(smem, i & 1, 1);
    const float* lse_s = qo_stats(smem, i & 1);
    const float* d_s = lse_s + BLK;
    {
      // S[16 t + 4 q4 + r][key] and dP likewise
      f32x4 st[4], dp[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) st[t] = f32x4{0, 0, 0, 0}, dp[t] = f32x4{0, 0, 0, 0};
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const bf16x8 aq = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const u32x4*>(Qs + (16 * t + l16) * PR + 32 * s4 + 8 * q4));
          const bf16x8 ao = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const u32x4*>(dOs + (16 * t + l16) * PR + 32 * s4 + 8 * q4));
          st[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, kf[s4], st[t], 0, 0, 0);
          dp[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ao, vf[s4], dp[t], 0, 0, 0);
        }
      // P and dS of this lane's 16 (query, key) pairs, in fragment order: chunk u, slot i is
      // query 32 u + 4 q4 + i (i < 4) or 32 u + 16 + 4 q4 + i - 4. A query block after the key
      // block sees every key, and the key block is then not the last, so it is whole: no mask.
      float pv[2][8], dsv[2][8];
      auto probs = [&](auto masked) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const f32x4 ls = *reinterpret_cast<const f32x4*>(lse_s + 16 * t + 4 * q4);
          const f32x4 dd = *reinterpret_cast<const f32x4*>(d_s + 16 * t + 4 * q4);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int ql = 16 * t + 4 * q4 + r;
            float p = __builtin_amdgcn_exp2f(st[t][r] * sl - ls[r]);
            if constexpr (decltype(masked)::value) p = (k0 + key <= q0 + ql && key < nk) ? p : 0.0f;
            pv[t >> 1][4 * (t & 1) + r] = p;
            dsv[t >> 1][4 * (t & 1) + r] = p * (dp[t][r] - dd[r]);
          }
        }
      };
      if (q0 > k0)
        probs(std::false_type{});
      else
        probs(std::true_type{});
      bf16x8 ph[2], pl[2], sh[2], slo[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        split_frag(pv[u], ph[u], pl[u]);
        split_frag(dsv[u], sh[u], slo[u]);
      }
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const bf16x8 bo = trfrag(dOs, 16 * j, u, lane);
          dv[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph[u], bo, dv[j], 0, 0, 0);
          dv[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl[u], bo, dv[j], 0, 0, 0);
          const bf16x8 bq = trfrag(Qs, 16 * j, u, lane);
          dk[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sh[u], bq, dk[j], 0, 0, 0);
          dk[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(slo[u], bq, dk[j], 0, 0, 0);
        }
    }
    if (i + 1 < steps) stage((i + 1) & 1);
  }
  // D of dV / dK tile j: lane (l16, q4), register r -> key 16 w + 4 q4 + r, column 16 j + l16
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int kr = 16 * w + 4 * q4 + r;
    if (kr >= nk) continue;
    bf16_t* dkr = a.dk + ((int64_t)(E.row0 + k0 + kr) * a.kv_heads + kh) * DH;
    bf16_t* dvr = a.dv + ((int64_t)(E.row0 + k0 + kr) * a.kv_heads + kh) * DH;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      dkr[16 * j + l16] = f2bf(dk[j][r] * a.scale);
      dvr[16 * j + l16] = f2bf(dv[j][r]);
    }
  }
}

// Sums the float32 partials of a key block's step ranges in their order and rounds once. One thread per
// 8 columns of a key's dK or dV row.
__global__ __launch_bounds__(256) void attn_dkdv_reduce_kernel(AttnArgs a, AttnBatch b) {
  int ei = 0;
  const int blk = (int)blockIdx.x / 16;  // (key block, key/value head) of the launch
  while (ei + 1 < b.count && b.e[ei + 1].blocks0 * a.kv_heads <= blk) ++ei;
  const AttnEp E = b.e[ei];
  const int kh = blk % a.kv_heads, kb = blk / a.kv_heads - E.blocks0;
  const int id = ((int)blockIdx.x & 15) * 256 + threadIdx.x;
  const int which = id >> 11, kr = (id >> 4) & (KBLK - 1), c0 = (id & 15) * 8;
  if (kb * KBLK + kr >= E.L) return;
  const int steps = (a.heads / a.kv_heads) * ((E.L + BLK - 1) / BLK - kb * (KBLK / BLK));
  const int ns = (steps + b.chunk - 1) / b.chunk;
  const float* p = b.part + (int64_t)blk * b.splits * (2 * KBLK * DH) + (which * KBLK + kr) * DH + c0;
  f32x4 s0 = *reinterpret_cast<const f32x4*>(p), s1 = *reinterpret_cast<const f32x4*>(p + 4);
  for (int i = 1; i < ns; ++i) {
    p += 2 * KBLK * DH;
    s0 += *reinterpret_cast<const f32x4*>(p);
    s1 += *reinterpret_cast<const f32x4*>(p + 4);
  }
  bf16_t* o = (which ? a.dv : a.dk) + ((int64_t)(E.row0 + kb * KBLK + kr) * a.kv_heads + kh) * DH + c0;
  *reinterpret_cast<u32x4*>(o) = u32x4{pack_bf16x2(s0[0], s0[1]), pack_bf16x2(s0[2], s0[3]),
                                       pack_bf16x2(s1[0], s1[1]), pack_bf16x2(s1[2], s1[3])};
}

// dQ of one (query head, 64 QT-query block). Wave w owns queries 16 QT w .. + 16 QT - 1 as QT tiles of
// 16; their Q and dO fragments stay in registers. Per half of a key block (32 keys): S^T = K Q^T and
// dP^T = V dO^T with the keys on the MFMA rows and this wave's queries on the columns, so each lane
// holds 8 (key, query) values of its own query of a tile; dS then feeds dQ += dS K as the A operand
// (the contraction runs over the keys in the order the lane holds them), with the B operand from the
// row-major K tile through transposing reads. With one tile per wave the LDS reads bound it (1792 of
// 2140 cycles a block and workgroup at 8192 rows, 32 heads); two tiles halve them per product, and
// halves of 32 keys, K's next block fetched in the first and V's in the second, keep that within 248
// VGPRs without spills: 1118 -> 867 us.
template <int QT>
__global__ __launch_bounds__(256, 2) void attn_dq_kernel(AttnArgs a, AttnBatch b) {
  constexpr int QBLK = 64 * QT;
  int ei, h, qb;
  attn_locate(b, a.heads, true, ei, h, qb);
  const AttnEp E = b.e[ei];
  const int kh = h / (a.heads / a.kv_heads);
  const int q0 = qb * QBLK, nq = min(QBLK, E.L - q0);
  extern __shared__ __align__(16) uint8_t smem[];  // two buffers of [K tile][V tile], [64][PR] each
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l16 = lane & 15, q4 = lane >> 4;
  const int64_t qs = (int64_t)a.heads * DH, ks = (int64_t)a.kv_heads * DH;
  const int wq = 16 * QT * w;  // this wave's first query in the block
  bf16x8 qf[QT][4], of[QT][4];
  float ls[QT], dd[QT];
#pragma unroll
  for (int c = 0; c < QT; ++c) {
    const int qry = wq + 16 * c + l16;
    load_row_frags(qf[c], a.q + ((int64_t)(E.row0 + q0) * a.heads + h) * DH, qs, qry, nq, q4);
    load_row_frags(of[c], a.dout + ((int64_t)(E.row0 + q0) * a.heads + h) * DH, qs, qry, nq, q4);
    const int64_t t = (int64_t)h * a.N + E.row0 + q0 + qry;
    ls[c] = qry < nq ? a.lse[t] * kLog2e : INFINITY;  // absent queries: P = 0
    dd[c] = qry < nq ? a.dsum[t] : 0.0f;
  }
  f32x4 dq[QT][8];
#pragma unroll
  for (int c = 0; c < QT; ++c)
#pragma unroll
    for (int j = 0; j < 8; ++j) dq[c][j] = f32x4{0, 0, 0, 0};
  const float sl = a.scale * kLog2e;
  u32x4 f[4];
  auto fetch = [&](const bf16_t* src, int kb) {
    const int k0 = kb * BLK, nk = min(BLK, E.L - k0);
    fetch_block(f, src + ((int64_t)(E.row0 + k0) * a.kv_heads + kh) * DH, ks, nk, tid);
  };
  const int kb_last = (q0 + nq - 1) / BLK;  // the key block of the block's last query
  fetch(a.k, 0);
  store_block(f, kv_tile(smem, 0, 0), tid);
  fetch(a.v, 0);
  store_block(f, kv_tile(smem, 0, 1), tid);
  for (int kb = 0; kb <= kb_last; ++kb) {
    const int k0 = kb * BLK;
    // This block's tiles are stored, and every wave is done with the other buffer.
    __syncthreads();
    if (kb < kb_last) fetch(a.k, kb + 1);  // the next K block loads during the first half, V during the second
    const bf16_t* Ks = kv_tile(smem, kb & 1, 0);
    const bf16_t* Vs = kv_tile(smem, kb & 1, 1);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int ku = k0 + 32 * u;
      // A wave whose queries all precede the half has nothing to add.
      if (ku <= q0 + wq + 16 * QT - 1) {
        // S^T[16 t + 4 q4 + r][query] and dP^T likewise
        f32x4 st[QT][2], dp[QT][2];
#pragma unroll
        for (int c = 0; c < QT; ++c)
#pragma unroll
          for (int t = 0; t < 2; ++t) st[c][t] = f32x4{0, 0, 0, 0}, dp[c][t] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const bf16x8 ak = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const u32x4*>(Ks + (32 * u + 16 * t + l16) * PR + 32 * s4 + 8 * q4));
            const bf16x8 av = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const u32x4*>(Vs + (32 * u + 16 * t + l16) * PR + 32 * s4 + 8 * q4));
#pragma unroll
            for (int c = 0; c < QT; ++c) {
              st[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ak, qf[c][s4], st[c][t], 0, 0, 0);
              dp[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, of[c][s4], dp[c][t], 0, 0, 0);
            }
          }
        // dS of this lane's queries against 8 keys, in fragment order: slot i is key 32 u + 4 q4 + i
        // (i < 4) or 32 u + 16 + 4 q4 + i - 4. A half that ends at or before the wave's first query is
        // whole and entirely allowed: no mask there. (Keys past the episode come after every query.)
        bf16x8 sh[QT], slo[QT];
        auto grad = [&](auto masked) {
#pragma unroll
          for (int c = 0; c < QT; ++c) {
            float dsv[8];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                float p = __builtin_amdgcn_exp2f(st[c][t][r] * sl - ls[c]);
                if constexpr (decltype(masked)::value)
                  p = (ku + 16 * t + 4 * q4 + r <= q0 + wq + 16 * c + l16) ? p : 0.0f;
                dsv[4 * t + r] = p * (dp[c][t][r] - dd[c]);
              }
            split_frag(dsv, sh[c], slo[c]);
          }
        };
        if (ku + 31 <= q0 + wq)
          grad(std::false_type{});
        else
          grad(std::true_type{});
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const bf16x8 bk = trfrag(Ks, 16 * j, u, lane);
#pragma unroll
          for (int c = 0; c < QT; ++c) {
            dq[c][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sh[c], bk, dq[c][j], 0, 0, 0);
            dq[c][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(slo[c], bk, dq[c][j], 0, 0, 0);
          }
        }
      }
      if (kb < kb_last) {
        store_block(f, kv_tile(smem, (kb + 1) & 1, u), tid);
        if (u == 0) fetch(a.v, kb + 1);
      }
    }
  }
  // D of dQ tile j: lane (l16, q4), register r -> query 16 c + 4 q4 + r of the wave's, column 16 j + l16
#pragma unroll
  for (int c = 0; c < QT; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int qi = wq + 16 * c + 4 * q4 + r;
      if (qi >= nq) continue;
      bf16_t* dqr = a.dq + ((int64_t)(E.row0 + q0 + qi) * a.heads + h) * DH;
#pragma unroll
      for (int j = 0; j < 8; ++j) dqr[16 * j + l16] = f2bf(dq[c][j][r] * a.scale);
    }
}

// A kernel whose 256-thread workgroups take blocks of `rows` queries or keys of one of `heads`.
template <class K>
static hipError_t launch_blocks(K kernel, LdsLimit& limit, int rows, int heads, size_t lds, const AttnArgs& a, AttnBatch b,
                                int id, hipStream_t s) {
  if (hipError_t e = limit.raise((const void*)kernel, lds)) return e;
  int n = 0;
  for (int i = 0; i < b.count; ++i) {
    b.e[i].blocks = (b.e[i].L + rows - 1) / rows;
    b.e[i].wg_begin = n;
    n += b.e[i].blocks * heads;
  }
  if (n <= 0) return hipSuccess;
  KernelTimer t(id, s);
  hipLaunchKernelGGL(kernel, dim3(n), dim3(256), lds, s, a, b);
  return hipGetLastError();
}

template <int KT>
static hipError_t launch_keys(LdsLimit& limit, const AttnArgs& a, AttnBatch b, hipStream_t s) {
  constexpr int KEYS = 64 * KT;
  constexpr size_t lds = 2 * (size_t)kQoBuf + 2 * KEYS * PR * 2;
  static_assert(2 * kQoBuf >= 65536 && lds <= 160 * 1024, "the exchange at the end needs 64 KiB");
  if (hipError_t e = limit.raise((const void*)attn_dkdv_kernel<KT>, lds)) return e;
  int n = 0, blocks = 0;
  for (int i = 0; i < b.count; ++i) {
    b.e[i].blocks = (b.e[i].L + KEYS - 1) / KEYS;
    b.e[i].blocks0 = blocks;
    b.e[i].wg_begin = n;
    blocks += b.e[i].blocks;
    for (int p = 0; p < b.splits; ++p)
      n += whole_pieces<KT>(b.e[i].L, a.heads / a.kv_heads, p, b.chunk) * a.kv_heads;
    n += b.e[i].blocks * a.kv_heads;
  }
  if (n <= 0) return hipSuccess;
  KernelTimer t(K_ATTN_DKDV, s);
  hipLaunchKernelGGL(attn_dkdv_kernel<KT>, dim3(n), dim3(512), lds, s, a, b);
  if (b.splits > 1)
    hipLaunchKernelGGL(attn_dkdv_reduce_kernel, dim3(blocks * a.kv_heads * 16), dim3(256), 0, s, a, b);
  return hipGetLastError();
}

hipError_t launch_attn(int kernel, const AttnArgs& a, const AttnBatch& b, hipStream_t s) {
  static LdsLimit limits[7];
  if (kernel == 1 && b.tiles == 0)
    return launch_blocks(attn_dkdv_short_kernel, limits[6], BLK, a.kv_heads, 2 * (size_t)kQoBuf, a, b, K_ATTN_DKDV, s);
  if (kernel == 1) return b.tiles == 1 ? launch_keys<1>(limits[4], a, b, s) : launch_keys<2>(limits[5], a, b, s);
  constexpr size_t lds = 2 * (size_t)kKvBuf;
  // Two query tiles per wave where their workgroups nearly fill the chip's two per CU; below that the longest
  // chain of key blocks is the time, and a step of one tile is the shorter one. One tile too where blocks of
  // 128 queries are hardly fewer than those of 64 (short episodes). Statistics + dQ, one tile / two, by the
  // two-tile workgroups: 256 (2048 rows x 16 heads) 51 + 61 / 63 + 71 us; 416 (6636 x 8) 169 + 220 / 203 + 244; 456
  // (6540 x 8 and three short ones) 151 + 195 / 190 + 225; 504 (9 of 781 x 8) 42 + 50 / 36 + 44; 720 (4518 x 20)
  // 190 + 237 / 143 + 190; 768 (3 of 3970 x 8) 196 + 241 / 157 + 216; 2048 of either (64 of 64 x 32) 32 + 39 / 35 + 41.
  int n1 = 0, n2 = 0;
  for (int i = 0; i < b.count; ++i) n1 += (b.e[i].L + 63) / 64, n2 += (b.e[i].L + 127) / 128;
  const bool wide = (int64_t)n2 * a.heads > 480 && 8 * (int64_t)n1 > 9 * (int64_t)n2;
  if (kernel == 0)
    return wide ? launch_blocks(attn_fwd_stats_kernel<2>, limits[0], 128, a.heads, lds, a, b, K_ATTN_FWD, s)
                : launch_blocks(attn_fwd_stats_kernel<1>, limits[1], 64, a.heads, lds, a, b, K_ATTN_FWD, s);
  return wide ? launch_blocks(attn_dq_kernel<2>, limits[2], 128, a.heads, lds, a, b, K_ATTN_DQ, s)
              : launch_blocks(attn_dq_kernel<1>, limits[3], 64, a.heads, lds, a, b, K_ATTN_DQ, s);
}

}  // namespace attt

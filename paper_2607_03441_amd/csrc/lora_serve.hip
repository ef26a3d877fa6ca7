// Serving side of the episode adapters on gfx950: concurrent episodes decode through the
// shared base model, each with its own LoRA adapter, and the adapter trained by an update is
// swapped into serving (Appendix A; adapter of Sec. 3.1, rank and alpha in Appendix C).
//
// lora_fwd_kernel: grouped multi-adapter forward. The base product x W0^T is a plain GEMM the
// caller has written into y; this adds y <- RN(y + scale (x A^T) B^T) for every (episode,
// projection), in one launch for all of them. A job is one x (an episode's rows) with up to
// four projections reading it (q, k, v of a layer): x is read once for all their ranks.
//   Phase 1: U = x A^T on v_mfma_f32_16x16x32_bf16 for 16 rows per workgroup; its waves split d_in
//     and their partial U meet in LDS in a fixed order. Rows of x and A lie 2 d_in bytes apart, so an
//     MFMA's own operand order (16 rows x 64 bytes per load) would touch 16 half lines of one cache set
//     and one L2 channel; each wave loads 8 rows x 128 bytes instead (whole lines), two steps of 64 in
//     flight, and turns them into operands through 9 KiB of LDS of its own. (Operand-order loads ran at
//     20 GB/s per CU: 21 us for a decoding step's 15 MB, 165 us at prefill.) scale U (float32) stays in
//     LDS: nothing goes through HBM between the phases.
//   Phase 2: y's columns in blocks of 64, dealt to the waves. U B^T runs on the
//     float32 MFMA (v_mfma_f32_16x16x4_f32 on U and the widened B: the products and sums of float32
//     arithmetic); MFMA column n of tile q is column 4 n + q of the block, so a lane ends up with 4
//     consecutive columns of 4 rows: an 8-byte load and store of y each, 128 contiguous bytes per row.
//   The rank product is a sixth of the float32 matrix rate at prefill, where the bytes of x and y
//   bound the kernel.
//   A row block's outputs are split over `ncs` workgroups (each recomputing phase 1) only where row
//   blocks are too few to fill the chip; logical workgroups are mapped so that consecutive ones
//   (the splits of one row block, the row blocks of one episode) run on one XCD and share its L2.
// lora_swap_kernel: the swap. float32 adapter tensors -> their bf16 serving copies, rounded to
// nearest even, every tensor of an adapter in one launch.
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"

namespace attt {

namespace {
constexpr uint32_t kOOBF = 0x7FFFFFF0u;  // offset past every descriptor's range: loads return 0
constexpr int kUP = 65;                  // LDS pitch (floats) of a row of U
constexpr int kSP = 144;                 // LDS pitch (bytes) of a staged row's 64 elements: conflict-free b128 reads

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// A lane's SPL consecutive elements of a row of B, from byte offset `off`; of 16, zero from `valid` on (8 or 16).
template <int SPL>
struct BRow {
  uint32_t w[(SPL + 1) / 2];
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off, int valid) {
    if constexpr (SPL == 2) {
      w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
    } else if constexpr (SPL == 4) {
      const uint2 v = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
      w[0] = v.x, w[1] = v.y;
    } else {
#pragma unroll
      for (int q = 0; q < SPL / 8; ++q) {
        const u32x4 v = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, 8 * q < valid ? off + 16u * q : kOOBF, 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) w[4 * q + e] = v[e];
      }
    }
  }
  __device__ __forceinline__ float get(int i) const { return (i & 1) ? bf_hi(w[i >> 1]) : bf_lo(w[i >> 1]); }
};
// Any rank: a lane's elements are k = g, g + 4, ... of the row, loaded one by one, zero from `rank` on.
template <int SPL>
struct BRowAny {
  uint32_t w[(SPL + 1) / 2];
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off, int g, int rank) {
    auto one = [&](int i) {
      return (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, i < SPL && 4 * i + g < rank ? off + 2u * (4 * i + g) : kOOBF, 0, 0) & 0xFFFFu;
    };
#pragma unroll
    for (int i = 0; i < (SPL + 1) / 2; ++i) w[i] = SPL == 1 ? one(0) : one(2 * i) | (one(2 * i + 1) << 16);
  }
  __device__ __forceinline__ float get(int i) const { return (i & 1) ? bf_hi(w[i >> 1]) : bf_lo(w[i >> 1]); }
};

// Phase 2 of one projection: blocks first, first + stride, ... < nb of 64 columns from o_lo. Lane
// (l16, g) holds row l16 of U and, for column tile q, column TQ l16 + q of B, at k = g SPL .. +SPL-1 (R = 0:
// the rank is 4 SPL; R = 1: a multiple of min(SPL, 8) below it) or at k = g, g + 4, ... (R = 2: any); it ends up with columns TQ l16 .. + TQ - 1 of rows 4 g .. 4 g + 3. kDepth blocks have their loads in
// flight.
template <int SPL, int R, int kDepth>
__device__ __forceinline__ void add_columns(const LoraFwdOut& O, const float* Uf, int row0, int nrows, int o_lo,
                                            int o_hi, int first, int stride, int nb, int lane) {
  constexpr int TQ = 4;
  typedef uint32_t YVec __attribute__((ext_vector_type(2)));  // 4 bf16 of a row of y
  const int l16 = lane & 15, g = lane >> 4;
  const int d_out = O.d_out, rank = O.rank;
  float u[SPL];
#pragma unroll
  for (int i = 0; i < SPL; ++i) {
    const int k = R == 2 ? 4 * i + g : g * SPL + i;
    u[i] = R == 0 || k < rank ? Uf[l16 * kUP + 16 * O.u0 + k] : 0.0f;
  }
  const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(O.B, d_out * rank * 2);
  const __amdgpu_buffer_rsrc_t ry = buffer_rsrc(static_cast<bf16_t*>(O.y) + (int64_t)row0 * d_out, nrows * d_out * 2);
  using Row = std::conditional_t<R == 2, BRowAny<SPL>, BRow<SPL>>;
  YVec yv[kDepth][4];
  Row br[kDepth][TQ];
  // column of the lane's first element of y in a block, and its byte offset in row 4 g + v; rows at or
  // past nrows fall outside the descriptor's range
  auto ycol = [&](int blk) { return o_lo + blk * 16 * TQ + TQ * l16; };
  auto yoff = [&](int yc, int v) { return yc < o_hi ? (uint32_t)((4 * g + v) * d_out + yc) * 2u : kOOBF; };
  auto load = [&](int d, int blk) {
    const int yc = ycol(blk);
#pragma unroll
    for (int v = 0; v < 4; ++v)
      yv[d][v] = __builtin_bit_cast(YVec, __builtin_amdgcn_raw_buffer_load_b64(ry, yoff(yc, v), 0, 0));
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
      if constexpr (R == 2)
        br[d][q].load(rb, (uint32_t)((yc + q) * rank) * 2u, g, yc < o_hi ? rank : 0);
      else
        br[d][q].load(rb, yc < o_hi && (R == 0 || g * SPL < rank) ? (uint32_t)((yc + q) * rank + g * SPL) * 2u : kOOBF,
                      R == 0 ? SPL : rank - g * SPL);
    }
  };
  // Loads past the last block fall outside the descriptors' ranges; they are issued all the same, so that
  // the number of loads in flight is the same on every path and each wait names only what it needs.
#pragma unroll
  for (int d = 0; d < kDepth; ++d) load(d, first + d * stride);
  for (int b0 = first; b0 < nb; b0 += kDepth * stride) {
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
      const int blk = b0 + d * stride;
      if (blk >= nb) break;
      f32x4 acc[TQ];
#pragma unroll
      for (int q = 0; q < TQ; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < SPL; ++i)
#pragma unroll
        for (int q = 0; q < TQ; ++q)
          acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(u[i], br[d][q].get(i), acc[q], 0, 0, 0);
      const int yc = ycol(blk);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        YVec out;
#pragma unroll
        for (int e = 0; e < TQ / 2; ++e)
          out[e] = pack_bf16x2(bf_lo(yv[d][v][e]) + acc[2 * e][v], bf_hi(yv[d][v][e]) + acc[2 * e + 1][v]);
        __builtin_amdgcn_raw_buffer_store_b64(out, ry, yoff(yc, v), 0, 0);
      }
      // this slot's next block: the loads of the other slots stay in flight behind it
      load(d, blk + kDepth * stride);
    }
  }
}
}  // namespace

template <int N>
using I = std::integral_constant<int, N>;

// W = 8 or 4 waves, blocks of 64 columns. Without kHigh every rank of the launch is at most 16, which keeps
// the kernel at 99 registers (four waves per SIMD); higher ranks hold up to 16 k values per lane. kAny: ranks
// other than 8, 16, 32 and 64 too. They take the products of the next of 4, 8, 16, 32 and 64, and 12 and the
// multiples of 8 its loads. (In the products of 64, loaded one by one, rank 4 took 239 us at the prefill
// below and rank 24 398, here 110 and 161; 187 and 500 with the kernel before.) Ranks of 32 and 64 alone need
// 112 registers, but four waves per SIMD are one too many for them: 173 us at rank 32 there, 166 with three.
// 16 x 512 rows of q, k, v and o (483 MB): 279 us with 64-row workgroups that recomputed U in eight
// column splits and walked the rank per thread, 132 us now (3.7 TB/s); the decoding step of 16 episodes
// 42 us in two launches, 15 in one.
template <int NU, bool kHigh, bool kAny, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2, kHigh && !kAny ? 3 : 8))) void lora_fwd_kernel(
    LoraFwdBatch b, int grid) {
  constexpr int NT = 64 * W, TQ = 4;
  constexpr int kWaveStage = 16 * (1 + NU) * kSP;  // bytes: 16 rows of x, then the units' rows of A
  static_assert(kWaveStage >= 16 * kUP * 4, "the partial U reuses the stage");
  // hardware places workgroup i on XCD i % 8: give each XCD a contiguous range of logical ids
  const int per = grid >> 3;
  const int li = (int)(blockIdx.x & 7u) * per + (int)(blockIdx.x >> 3);
  if (li >= b.total) return;
  const LoraFwdJob& J = b.j[find_job(b, li)];
  const int ncs = b.ncs;
  const int local = li - J.b_begin;
  const int rblk = local / ncs, cs = local - rblk * ncs;
  const int row0 = rblk * kLoraFwdRows;
  const int nrows = min(kLoraFwdRows, J.rows - row0);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  __shared__ __align__(16) float Uf[16 * kUP];
  __shared__ __align__(16) uint8_t scr[W * kWaveStage];
  uint8_t* mine = scr + w * kWaveStage;
  const int no = J.no, nu = J.nu;
  const LoraFwdOut* outs = b.o + J.o_begin;

  // ---- phase 1 ------------------------------------------------------------------------
  const int d_in = J.d_in;
  const bf16_t* xs = static_cast<const bf16_t*>(J.x) + (int64_t)row0 * d_in;
  const __amdgpu_buffer_rsrc_t rx = buffer_rsrc(xs, nrows * d_in * 2);
  // unit t: 16 ranks (the last of a projection may have fewer; the rest read as zero)
  __amdgpu_buffer_rsrc_t ra[NU];
  float usc[NU];
#pragma unroll
  for (int t = 0; t < NU; ++t) {
    int p = 0;
    while (p + 1 < no && outs[p + 1].u0 <= t) ++p;
    const LoraFwdOut& O = outs[p];
    const int sub = t - O.u0;
    ra[t] = buffer_rsrc(static_cast<const bf16_t*>(O.A) + (int64_t)16 * sub * d_in,
                        t < nu ? max(0, min(16, O.rank - 16 * sub)) * d_in * 2 : 0);
    usc[t] = O.scale;
  }
  const int ns = (d_in + 63) / 64;
  const int spw = (ns + W - 1) / W;
  const int s_begin = w * spw, s_end = min(ns, s_begin + spw);
  f32x4 acc[NU];
#pragma unroll
  for (int t = 0; t < NU; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  // step s of 64: a load instruction takes rows sr (+ 8) at 16-byte chunk sc of the step
  const int sr = lane >> 3, sc = lane & 7;
  auto load = [&](int s, u32x4 (&v)[1 + NU][2]) {
    const int k = s * 64 + sc * 8;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t off = s < s_end && k < d_in ? (uint32_t)((sr + 8 * h) * d_in + k) * 2u : kOOBF;
      v[0][h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, 0));
#pragma unroll
      for (int t = 0; t < NU; ++t)
        v[1 + t][h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ra[t], off, 0, 0));
    }
  };
  // The stage is this wave's own and its LDS operations run in order: no barrier.
  auto mma = [&](const u32x4 (&v)[1 + NU][2]) {
#pragma unroll
    for (int t = 0; t < 1 + NU; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *reinterpret_cast<u32x4*>(mine + (16 * t + sr + 8 * h) * kSP + 16 * sc) = v[t][h];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const uint8_t* f = mine + l16 * kSP + (32 * q + 8 * g) * 2;
      const bf16x8 x = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(f));
#pragma unroll
      for (int t = 0; t < NU; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            x, __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(f + 16 * (1 + t) * kSP)), acc[t], 0, 0, 0);
    }
  };
  {
    u32x4 v0[1 + NU][2], v1[1 + NU][2];
    // steps at or past s_end and absent units load zeros (no memory access), on every path alike
    load(s_begin, v0);
    load(s_begin + 1, v1);
    for (int s = s_begin; s < s_end; s += 2) {
      mma(v0);
      load(s + 2, v0);
      mma(v1);
      load(s + 3, v1);
    }
  }
  // D of a 16x16 tile: lane l, register v -> row 4 (l / 16) + v, rank l % 16
  float* Up = reinterpret_cast<float*>(mine);
#pragma unroll
  for (int t = 0; t < NU; ++t) {
    if (t >= nu) break;
#pragma unroll
    for (int v = 0; v < 4; ++v) Up[(4 * g + v) * kUP + 16 * t + l16] = acc[t][v];
  }
  __syncthreads();
  for (int i = tid; i < 16 * 64; i += NT) {
    const int row = i >> 6, c = i & 63, t = c >> 4;
    if (t >= nu) continue;
    float sc2 = usc[0];
#pragma unroll
    for (int k = 1; k < NU; ++k)
      if (t == k) sc2 = usc[k];
    const float* part = reinterpret_cast<const float*>(scr) + row * kUP + c;
    float v = part[0];
#pragma unroll
    for (int k = 1; k < W; ++k) v += part[k * (kWaveStage / 4)];  // fixed order
    Uf[row * kUP + c] = sc2 * v;
  }
  __syncthreads();

  // ---- phase 2: the blocks of all projections in one sequence, dealt to the waves in turn ------
  int base = 0;
#pragma unroll 1
  for (int p = 0; p < no; ++p) {
    const LoraFwdOut& O = outs[p];
    constexpr int CB = 16 * TQ;
    const int cw = (((O.d_out + ncs - 1) / ncs) + CB - 1) & ~(CB - 1);
    const int o_lo = min(O.d_out, cs * cw), o_hi = min(O.d_out, o_lo + cw);
    const int nb = (o_hi - o_lo + CB - 1) / CB;
    const int first = (w - base) & (W - 1);
    base += nb;
    auto add = [&](auto spl, auto ranks, auto depth) {
      add_columns<decltype(spl)::value, decltype(ranks)::value, decltype(depth)::value>(O, Uf, row0, nrows, o_lo, o_hi,
                                                                                         first, W, nb, lane);
    };
    if (O.rank == 16) {
      add(I<4>{}, I<0>{}, I<2>{});
    } else if (O.rank == 8) {
      add(I<2>{}, I<0>{}, I<2>{});
    } else if (kHigh && O.rank == 32) {
      add(I<8>{}, I<0>{}, I<1>{});
    } else if (kHigh && O.rank == 64) {
      add(I<16>{}, I<0>{}, I<1>{});
    } else if constexpr (kAny) {
      if (O.rank == 12)
        add(I<4>{}, I<1>{}, I<2>{});
      else if (O.rank <= 4)
        add(I<1>{}, I<2>{}, I<2>{});
      else if (O.rank < 8)
        add(I<2>{}, I<2>{}, I<2>{});
      else if (O.rank < 16)
        add(I<4>{}, I<2>{}, I<1>{});
      else if constexpr (kHigh) {
        if (O.rank == 24)
          add(I<8>{}, I<1>{}, I<1>{});
        else if (O.rank % 8 == 0)
          add(I<16>{}, I<1>{}, I<1>{});
        else if (O.rank < 32)
          add(I<8>{}, I<2>{}, I<1>{});
        else
          add(I<16>{}, I<2>{}, I<1>{});
      }
    }
  }
}

__global__ __launch_bounds__(256) void lora_swap_kernel(LoraSwapBatch b) {
  const int ji = find_job(b, (int)blockIdx.x);
  const LoraSwapJob J = b.j[ji];
  const int64_t i0 = ((int64_t)((int)blockIdx.x - J.b_begin) * 256 + threadIdx.x) * 8;
  if (i0 >= J.n) return;
  if (J.vec && i0 + 8 <= J.n) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(J.src + i0);
    const f32x4 c = *reinterpret_cast<const f32x4*>(J.src + i0 + 4);
    u32x4 o;
    o[0] = pack_bf16x2(a[0], a[1]);
    o[1] = pack_bf16x2(a[2], a[3]);
    o[2] = pack_bf16x2(c[0], c[1]);
    o[3] = pack_bf16x2(c[2], c[3]);
    *reinterpret_cast<u32x4*>(J.dst + i0) = o;
  } else {
    for (int64_t i = i0; i < J.n && i < i0 + 8; ++i) J.dst[i] = (uint16_t)f32_to_bf16_bits(J.src[i]);
  }
}

template <bool kHigh, bool kAny>
static void launch_fwd(int nu, bool four, const LoraFwdBatch& b, int grid, hipStream_t s) {
  auto launch = [&](auto n) {
    constexpr int NU = decltype(n)::value;
    if (four)
      hipLaunchKernelGGL((lora_fwd_kernel<NU, kHigh, kAny, 4>), dim3(grid), dim3(256), 0, s, b, grid);
    else
      hipLaunchKernelGGL((lora_fwd_kernel<NU, kHigh, kAny, 8>), dim3(grid), dim3(512), 0, s, b, grid);
  };
  switch (nu) {
    case 1: launch(I<1>{}); break;
    case 2: launch(I<2>{}); break;
    case 3: launch(I<3>{}); break;
    default: launch(I<4>{}); break;
  }
}

hipError_t launch_lora_fwd(int nu, const LoraFwdBatch& b, hipStream_t s) {
  if (b.total <= 0) return hipSuccess;
  const int grid = (b.total + 7) & ~7;
  bool high = false, any = false;
  for (int i = 0; i < b.outs; ++i) {
    const int r = b.o[i].rank;
    high = high || r > 16;
    any = any || !(r == 8 || r == 16 || r == 32 || r == 64);
  }
  // Four waves where d_in leaves eight too little each to start with and two workgroups per CU are there to
  // fill it (8 / 4 waves, rank 16: 4 x 5000 rows of 256 55 / 40 us, 8 x 2000 of 1024 72 / 61, 16 x 700 of 2048
  // 78 / 69, 16 x 512 of 4096 131 / 136; 100 x 3 of 2048, 200 workgroups, 109 / 117).
  bool four = b.total >= 512;
  for (int i = 0; i < b.count; ++i) four = four && b.j[i].d_in <= 2048;
  KernelTimer t(K_LORA_FWD, s);
  if (high)
    any ? launch_fwd<true, true>(nu, four, b, grid, s) : launch_fwd<true, false>(nu, four, b, grid, s);
  else
    any ? launch_fwd<false, true>(nu, four, b, grid, s) : launch_fwd<false, false>(nu, four, b, grid, s);
  return hipGetLastError();
}

hipError_t launch_lora_swap(const LoraSwapBatch& b, int blocks, hipStream_t s) {
  if (blocks <= 0) return hipSuccess;
  KernelTimer t(K_LORA_SWAP, s);
  hipLaunchKernelGGL(lora_swap_kernel, dim3(blocks), dim3(256), 0, s, b);
  return hipGetLastError();
}

}  // namespace attt

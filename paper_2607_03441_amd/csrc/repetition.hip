// Update-text repetition (Sec. 3.2, Eq. 6-7): rho(x_k) = max over the previous update texts x'
// of the episode of the Jaccard similarity of the word sets W(x_k) and W(x'), nu = 1 - rho, and
// the sequence-level filter that skips an update when nu < tau.
//
//   rep_count_kernel   one workgroup per (previous text, hash partition). Words are
//                      split into `parts` partitions by the high bits of a 32-bit hash (the
//                      MurmurHash3 finalizer), so |A|, |B| and |A & B| are sums over partitions
//                      and a partition's sets fit LDS whatever the text lengths. The workgroup
//                      inserts its partition's words of the candidate into one LDS hash set and
//                      those of the previous text into another; a new entry of the second set
//                      that is also in the first counts towards the intersection.
//   rep_reduce_kernel  one wave per episode: sums the partitions, takes the maximum Jaccard
//                      over the previous texts by exact cross-multiplication (the first maximum
//                      wins a tie), rho = the nearest float64 to |A & B| / |A | B|,
//                      nu = RN(1 - rho), skip = nu < tau.
// Integer counts throughout, so the result is bit-reproducible.
#include "common.hpp"
#include "internal.hpp"
#include "lds_limit.hpp"

namespace attt {

constexpr uint32_t kRepEmpty = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t word_hash(int32_t w) {
  uint32_t h = (uint32_t)w;
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  h *= 0xC2B2AE35u;
  h ^= h >> 16;
  return h;
}
// partition of a hash: multiply-shift range reduction of its high 24 bits
__device__ __forceinline__ int part_of(uint32_t h, int parts) { return (int)(((h >> 8) * (uint32_t)parts) >> 24); }

// A set is an array of buckets of four words (bmask + 1 of them), searched bucket by bucket from the
// hash's low bits; kRepEmpty marks a free slot. A word takes the first free slot of a bucket in an order that
// begins at its own slot and goes round, and nothing leaves a set: a bucket with a free slot ends every
// search. Dense sets (up to half full and beyond) read the bucket first, 16 bytes that settle nearly all
// searches (a wave walks on for as long as any of its lanes does); their own slot is the first. In sparse
// ones (a quarter full) the own slot comes from two more bits of the hash and is nearly always free or the
// word's, so that an exchange on it settles the insertion by itself; a free own slot means that the word is
// not there.
template <bool kSparse>
__device__ __forceinline__ uint32_t own_slot(uint32_t h) { return kSparse ? (h >> 12) & 3u : 0u; }
static_assert(kRepSlots / 4 <= 1 << 12, "the bucket comes from the hash bits below the own slot's");

// set_insert returns 1 if w was new, 0 if present, -1 if the set is full (the caller flags the call).
template <bool kSparse>
__device__ __forceinline__ int set_insert(uint32_t* tab, uint32_t bmask, uint32_t h, uint32_t w) {
  const uint32_t own = own_slot<kSparse>(h);
  uint32_t b = h & bmask;
  if constexpr (kSparse) {
    const uint32_t cur = atomicCAS(tab + 4 * b + own, kRepEmpty, w);
    if (cur == kRepEmpty) return 1;
    if (cur == w) return 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  for (uint32_t probe = 0; probe <= bmask;) {
    const u32x4 e = *reinterpret_cast<const u32x4*>(tab + 4 * b);
    if (e[0] == w || e[1] == w || e[2] == w || e[3] == w) return 0;
    uint32_t free;
    if constexpr (kSparse) {
      const uint32_t m = (e[0] == kRepEmpty ? 1u : 0u) | (e[1] == kRepEmpty ? 2u : 0u) | (e[2] == kRepEmpty ? 4u : 0u) |
                         (e[3] == kRepEmpty ? 8u : 0u);
      free = m ? (own + __builtin_ctz((m | m << 4) >> own)) & 3u : 4u;
    } else {
      free = e[0] == kRepEmpty ? 0 : e[1] == kRepEmpty ? 1 : e[2] == kRepEmpty ? 2 : e[3] == kRepEmpty ? 3 : 4;
    }
    if (free == 4) {
      b = (b + 1u) & bmask;
      ++probe;
      continue;
    }
    const uint32_t cur = atomicCAS(tab + 4 * b + free, kRepEmpty, w);
    if (cur == kRepEmpty) return 1;
    if (cur == w) return 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");  // another word took the slot: read the bucket again
  }
  return -1;
}
template <bool kSparse>
__device__ __forceinline__ bool set_contains(const uint32_t* tab, uint32_t bmask, uint32_t h, uint32_t w) {
  uint32_t b = h & bmask;
  for (uint32_t probe = 0; probe <= bmask; ++probe) {
    const u32x4 e = *reinterpret_cast<const u32x4*>(tab + 4 * b);
    if (e[0] == w || e[1] == w || e[2] == w || e[3] == w) return true;
    if (e[3] == kRepEmpty || (kSparse && (e[0] == kRepEmpty || e[1] == kRepEmpty || e[2] == kRepEmpty))) return false;
    b = (b + 1u) & bmask;
  }
  return false;
}

// Bound by latency: the words of both texts, then their probes of the LDS sets. A thread takes kRepAhead
// words at a time; the first of both texts are loaded before the sets are cleared, the next ones while a
// block is inserted. Sparse sets are the largest LDS holds, dense ones as small as the texts allow (64 KiB for
// texts of 4096 words, so two workgroups share a CU). 512 such pairs took 32 us with 128 KiB sets probed word by
// word, 26 with dense ones; the one pair of two texts of 100000 words 112 us with words loaded one by one, 104 now
// (both kernels).
constexpr int kRepAhead = 4;

template <bool kSparse>
__global__ __launch_bounds__(1024) void rep_count_kernel(RepBatch batch, const int32_t* __restrict__ words,
                                                         const int64_t* __restrict__ toff,
                                                         int32_t* __restrict__ counts) {
  // the last episode whose first workgroup is at most this one (kEpBatch = 64: one per lane)
  const int ln = threadIdx.x & 63;
  const int ei = __builtin_amdgcn_readfirstlane(
      __popcll(__ballot(ln < batch.count && batch.e[ln < batch.count ? ln : 0].wg_begin <= (int)blockIdx.x)) - 1);
  const RepEp E = batch.e[ei];
  const int local = (int)blockIdx.x - E.wg_begin;
  const int pair = local / E.parts, part = local % E.parts;
  const int64_t ct = E.text0 + E.ntexts - 1, bt = E.text0 + pair;
  const int64_t a0 = toff[ct], a1 = toff[ct + 1], b0 = toff[bt], b1 = toff[bt + 1];

  extern __shared__ __align__(16) uint8_t smem[];
  uint32_t* ta = reinterpret_cast<uint32_t*>(smem);  // [slots] candidate words of the partition
  uint32_t* tb = ta + E.slots;                       // [slots] previous text's words
  const uint32_t mask = (uint32_t)(E.slots >> 2) - 1u;  // of the buckets
  __shared__ int cnt[4];                             // |A|, |B|, |A & B|, full
  const int tid = threadIdx.x, nt = blockDim.x;
  const int na_words = max(0, (int)(a1 - a0)), nb_words = max(0, (int)(b1 - b0));  // at most 2^20 each
  const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(words + a0, na_words * 4), rb = buffer_rsrc(words + b0, nb_words * 4);
  // words i, i + nt, ... of a text; zero past its end
  auto load = [&](uint32_t (&w)[kRepAhead], __amdgpu_buffer_rsrc_t r, int i) {
#pragma unroll
    for (int u = 0; u < kRepAhead; ++u) w[u] = __builtin_amdgcn_raw_buffer_load_b32(r, (uint32_t)(i + u * nt) * 4u, 0, 0);
  };
  uint32_t wa[kRepAhead], wb[kRepAhead];
  load(wa, ra, tid);
  load(wb, rb, tid);
  {
    u32x4* t4 = reinterpret_cast<u32x4*>(smem);
    for (int i = tid; i < E.slots / 2; i += nt) t4[i] = u32x4{kRepEmpty, kRepEmpty, kRepEmpty, kRepEmpty};
    if (tid < 4) cnt[tid] = 0;
  }
  __syncthreads();
  int na = 0, nb = 0, ni = 0, full = 0;
  // Inserts the partition's words of a text of n, the thread's first of them in `next`, into `tab`;
  // added(h, w) for every new one.
  auto insert_text = [&](uint32_t* tab, __amdgpu_buffer_rsrc_t r, int n, uint32_t (&next)[kRepAhead], auto added) {
    for (int i = tid; i < n; i += kRepAhead * nt) {
      uint32_t w[kRepAhead];
#pragma unroll
      for (int u = 0; u < kRepAhead; ++u) w[u] = next[u];
      if (n > kRepAhead * nt) load(next, r, i + kRepAhead * nt);
#pragma unroll
      for (int u = 0; u < kRepAhead; ++u) {
        const uint32_t h = word_hash((int32_t)w[u]);
        if (i + u * nt >= n || part_of(h, E.parts) != part) continue;
        const int got = set_insert<kSparse>(tab, mask, h, w[u]);
        if (got > 0) added(h, w[u]);
        full |= got < 0;
      }
    }
  };
  insert_text(ta, ra, na_words, wa, [&](uint32_t, uint32_t) { ++na; });
  __syncthreads();
  insert_text(tb, rb, nb_words, wb, [&](uint32_t h, uint32_t w) {
    ++nb;
    ni += set_contains<kSparse>(ta, mask, h, w);
  });
  // per-thread counts, then one LDS atomic each
  if (na) atomicAdd(cnt + 0, na);
  if (nb) atomicAdd(cnt + 1, nb);
  if (ni) atomicAdd(cnt + 2, ni);
  if (full) atomicOr(cnt + 3, 1);
  __syncthreads();
  if (tid < 4) counts[(E.wg_global + local) * 4 + tid] = cnt[tid];
}

// One wave per episode: lane k takes the previous texts k, k + 64, ..., then the lanes' best fractions
// meet (a single thread walking an episode's texts took 11 us for 32 of them).
__global__ __launch_bounds__(64) void rep_reduce_kernel(RepBatch batch, const int32_t* __restrict__ counts, double tau,
                                                        double* __restrict__ rho, double* __restrict__ nu,
                                                        int32_t* __restrict__ skip, int32_t* __restrict__ best,
                                                        int32_t* __restrict__ pair_counts) {
  const RepEp E = batch.e[blockIdx.x];
  const int lane = threadIdx.x;
  int64_t bi = 0, bu = 1;  // this lane's best fraction bi / bu and its text; none yet
  int bk = -1;
  bool bad = false;
  for (int k = lane; k + 1 < E.ntexts; k += 64) {
    int64_t a = 0, b = 0, in = 0;
#pragma unroll 4
    for (int p = 0; p < E.parts; ++p) {
      const int4 c = *reinterpret_cast<const int4*>(counts + (E.wg_global + (int64_t)k * E.parts + p) * 4);
      a += c.x;
      b += c.y;
      in += c.z;
      bad |= c.w != 0;
    }
    const int64_t un = a + b - in;
    if (pair_counts) {
      pair_counts[(E.pair_base + k) * 2] = (int32_t)in;
      pair_counts[(E.pair_base + k) * 2 + 1] = (int32_t)un;
    }
    // J = in / un (0 when un = 0); J > best  <=>  in * bu > bi * un (the first maximum stays)
    const int64_t ju = un > 0 ? un : 1;
    if (bk < 0 || in * bu > bi * ju) {
      bk = k;
      bi = in;
      bu = ju;
    }
  }
  // the larger fraction wins, the earlier text among equals
  for (int o = 32; o > 0; o >>= 1) {
    const int64_t oi = __shfl_xor(bi, o, 64), ou = __shfl_xor(bu, o, 64);
    const int ok = __shfl_xor(bk, o, 64);
    const bool take = ok >= 0 && (bk < 0 || oi * bu > bi * ou || (oi * bu == bi * ou && ok < bk));
    if (take) bi = oi, bu = ou, bk = ok;
  }
  bad = __ballot(bad) != 0;
  if (lane != 0) return;
  double r = 0.0;
  if (bk >= 0) r = __ddiv_rn((double)bi, (double)bu);
  const double v = __dsub_rn(1.0, r);
  const int e = E.ep;
  if (bad) {
    rho[e] = __longlong_as_double(0x7FF8000000000000ll);
    nu[e] = __longlong_as_double(0x7FF8000000000000ll);
    skip[e] = 0;
    best[e] = -1;
    return;
  }
  rho[e] = r;
  nu[e] = v;
  skip[e] = v < tau ? 1 : 0;
  best[e] = bk;
}

template <bool kSparse>
static hipError_t rep_count(const RepBatch& b, int total_wgs, int slots, int threads, const int32_t* words,
                            const int64_t* toff, int32_t* counts, hipStream_t s) {
  static LdsLimit limit;
  if (hipError_t e = limit.raise((const void*)rep_count_kernel<kSparse>, 2 * kRepSlots * 4)) return e;
  KernelTimer t(K_REP_COUNT, s);
  hipLaunchKernelGGL(rep_count_kernel<kSparse>, dim3(total_wgs), dim3(threads), (size_t)2 * slots * 4, s, b, words, toff,
                     counts);
  return hipGetLastError();
}

hipError_t launch_rep_count(const RepBatch& b, int total_wgs, int slots, const int32_t* words, const int64_t* toff,
                            int32_t* counts, hipStream_t s) {
  if (total_wgs <= 0) return hipSuccess;
  // Where there is a CU for every workgroup the latency of one counts, and sparse sets cost nothing. Dense /
  // sparse, both kernels: one pair of 1000 words 26.0 / 20.2 us, of 4096 31.3 / 27.4, of 100000 (25 workgroups)
  // 129 / 104; 512 pairs of 4096 words 45 / 57.
  if (total_wgs <= 256) {
    RepBatch big = b;
    for (int i = 0; i < big.count; ++i) big.e[i].slots = kRepSlots;
    return rep_count<true>(big, total_wgs, kRepSlots, 1024, words, toff, counts, s);
  }
  // four words of each text per thread up to 1024 threads, so that CUs share small sets
  const int threads = slots <= 2048 ? 256 : slots <= 4096 ? 512 : 1024;
  return rep_count<false>(b, total_wgs, slots, threads, words, toff, counts, s);
}

hipError_t launch_rep_reduce(const RepBatch& b, const int32_t* counts, double tau, double* rho, double* nu,
                             int32_t* skip, int32_t* best, int32_t* pair_counts, hipStream_t s) {
  if (b.count <= 0) return hipSuccess;
  KernelTimer t(K_REP_REDUCE, s);
  hipLaunchKernelGGL(rep_reduce_kernel, dim3(b.count), dim3(64), 0, s, b, counts, tau, rho, nu, skip, best, pair_counts);
  return hipGetLastError();
}

}  // namespace attt

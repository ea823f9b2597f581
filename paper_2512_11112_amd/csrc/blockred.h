// Block-level sums of residues: wave shuffles, then LDS across waves.
#pragma once
#include "ctx.h"

namespace spdz {

// --------------------------------------------------------------------------
// block-level reduction of K residues per thread
// --------------------------------------------------------------------------
template <class F>
__device__ __forceinline__ typename F::E shfl_xor_e(typename F::E a, int mask) {
  u32 w[F::WORDS32];
#pragma unroll
  for (int k = 0; k < F::WORDS32; k++) w[k] = (u32)__shfl_xor((int)F::word32(a, k), mask, 64);
  return F::from32(w);
}

// v of the lane's neighbour in its pair
template <class F>
__device__ __forceinline__ typename F::E lane_xor1(typename F::E v) {
  u32 w[F::WORDS32];
#pragma unroll
  for (int k = 0; k < F::WORDS32; k++)
    w[k] = (u32)__builtin_amdgcn_update_dpp(0, (int)F::word32(v, k), 0xB1, 15, 15, false);  // quad_perm [1, 0, 3, 2]
  return F::from32(w);
}

// sum of v over aligned groups of R lanes (R = 4, 8, 16), in every lane of the group: lane exchanges
// within a row of 16 lanes are operand modifiers, without the LDS's round trip that a shuffle takes
template <class F, int R>
__device__ __forceinline__ typename F::E group_sum(typename F::E v) {
  auto step = [&](auto ctrl) {
    u32 w[F::WORDS32];
#pragma unroll
    for (int k = 0; k < F::WORDS32; k++)
      w[k] = (u32)__builtin_amdgcn_update_dpp(0, (int)F::word32(v, k), decltype(ctrl)::value, 15, 15, false);
    v = F::add(v, F::from32(w));
  };
  step(std::integral_constant<int, 0xB1>{});                      // quad_perm [1, 0, 3, 2]
  step(std::integral_constant<int, 0x4E>{});                      // quad_perm [2, 3, 0, 1]
  if constexpr (R >= 8) step(std::integral_constant<int, 0x141>{});   // row_half_mirror: the other quad of 8
  if constexpr (R >= 16) step(std::integral_constant<int, 0x140>{});  // row_mirror: the other half of 16
  return v;
}

// sum of v over the wave, in every lane
template <class F>
__device__ __forceinline__ typename F::E wave_sum(typename F::E v) {
  v = group_sum<F, 16>(v);
  v = F::add(v, shfl_xor_e<F>(v, 16));
  return F::add(v, shfl_xor_e<F>(v, 32));
}

// Sum v[k] over the block; the total of component k is returned in thread k
// (k < K), other threads get zero.  Contains __syncthreads(): call from every
// thread of the block.
template <class F, int K>
__device__ typename F::E block_sum(typename F::E (&v)[K]) {
  using E = typename F::E;
  __shared__ E sh[WAVES][K];
#pragma unroll
  for (int k = 0; k < K; k++) v[k] = wave_sum<F>(v[k]);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();  // sh may be in use by a previous call
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < K; k++) sh[wave][k] = v[k];
  }
  __syncthreads();
  E s = F::zero();
  if (threadIdx.x < K) {
#pragma unroll
    for (int w = 0; w < WAVES; w++) s = F::add(s, sh[w][threadIdx.x]);
  }
  return s;
}

// add the block total of v into slot (K residues of L words)
template <class F, int K>
__device__ __forceinline__ void block_add_to_slot(typename F::E (&v)[K], u64 *slot) {
  typename F::E s = block_sum<F, K>(v);
  if (threadIdx.x < K) {
    u64 *p = slot + threadIdx.x * F::L;
    F::to_words(F::add(F::from_words(p), s), p);
  }
}

// store the block total of v into slot (K residues of L words) for the last block of the launch
// (last_block) to read: stores and loads of device scope go past the caches that XCDs do not share, so no
// cache is written back or invalidated (a device-wide fence in every block took a ReduceAdd of 2048
// blocks from 17 to 240 us)
template <class F, int K>
__device__ __forceinline__ void block_store_slot(typename F::E (&v)[K], u64 *slot) {
  typename F::E s = block_sum<F, K>(v);
  if (threadIdx.x < K) {
    u64 w[F::L];
    F::to_words(s, w);
#pragma unroll
    for (int l = 0; l < F::L; l++)
      __hip_atomic_store(slot + threadIdx.x * F::L + l, w[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// True in every thread of the last block of the launch to call this: every wave's device-scope stores
// have arrived before its block counts itself.  Blocks count in COUNT_GROUPS groups, each on a line of its
// own, and the last of a group counts the group: additions to one word follow each other at about 10 ns,
// which 768 blocks on a single word waited 8 us for.  The counts are reset for the next launch.
// Contains __syncthreads().
__device__ __forceinline__ bool last_block(unsigned *count) {
  __shared__ int last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    auto full = [](unsigned *c, unsigned n) {  // counts one; true (and the count reset) for the nth
      const bool f = __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
      if (f) __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return f;
    };
    const unsigned g = blockIdx.x % COUNT_GROUPS, members = (gridDim.x - g + COUNT_GROUPS - 1) / COUNT_GROUPS;
    last = full(count + (1 + g) * COUNT_STRIDE, members) && full(count, min(gridDim.x, (unsigned)COUNT_GROUPS));
  }
  __syncthreads();
  return last;
}

// Sum of slots [0, nslots) ([slot][K] residues) by one block of TH threads; the total of component k is
// returned in thread k (k < K), other threads get zero.  A thread takes one component of every
// (TH / K)th slot, so consecutive threads read consecutive words, eight requests at a time; then 16
// threads per component join the rest.  COHERENT: slots of block_store_slot in the same launch.
// Contains __syncthreads(): call from every thread.
template <class F, int K, int TH, bool COHERENT>
__device__ typename F::E slots_sum(const u64 *slots, int nslots) {
  using E = typename F::E;
  constexpr int A = TH / K * K, PER = 8;
  static_assert(TH >= 16 * K, "16 threads per component");
  __shared__ E sh[TH], tot[K];
  const int t = threadIdx.x, total = nslots * K;
  E s = F::zero();
  if (t < A) {
    for (int i = t; i < total; i += PER * A) {
      u64 w[PER][F::L];
#pragma unroll
      for (int u = 0; u < PER; u++)
#pragma unroll
        for (int l = 0; l < F::L; l++) {
          const u64 *p = slots + (size_t)(i + u * A) * F::L + l;
          w[u][l] = i + u * A >= total ? 0
                    : COHERENT         ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                       : *p;
        }
#pragma unroll
      for (int u = 0; u < PER; u++) s = F::add(s, F::from_words(w[u]));
    }
  }
  __syncthreads();  // sh may be in use by a previous call
  sh[t] = s;
  __syncthreads();
  if (t < 16 * K) {
    const int k = t >> 4;
    E r = F::zero();
    for (int j = t & 15; j < A / K; j += 16) r = F::add(r, sh[j * K + k]);
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) r = F::add(r, shfl_xor_e<F>(r, off));
    if ((t & 15) == 0) tot[k] = r;
  }
  __syncthreads();
  return t < K ? tot[t] : F::zero();
}

// ReduceAdd finalisation by the launch's last block: sums slots [0, nslots) of red ([slot][2 N][L], the
// values then the MAC shares of the N parties, stored by block_store_slot) and writes the width-1
// result to out.  With s_pub the result is also opened: s_pub receives sum_i s_i, and the MAC-check
// terms r s and r m(s)_i of log index js are added to acc_slot ([N + 1][L], a slot this block
// owns).  Contains __syncthreads(): call from every thread of the block.
template <class F, int N>
__device__ void reduce_finalize_block(const u64 *red, int nslots, SV out, u64 *s_pub, u64 coef_state, int64_t js,
                                      u64 *acc_slot) {
  using E = typename F::E;
  const E t = slots_sum<F, 2 * N, BLOCK, true>(red, nslots);
  __shared__ E tot[2 * N];
  if (threadIdx.x < 2 * N) {
    const int i = threadIdx.x % N;
    u64 *base = (threadIdx.x < N ? out.val : out.mac) + i * out.ps;
    u64 w[F::L];
    F::to_words(t, w);
#pragma unroll
    for (int l = 0; l < F::L; l++) base[l * out.ls] = w[l];
    tot[threadIdx.x] = t;
  }
  if (!s_pub) return;
  __syncthreads();
  if (threadIdx.x == 0) {
    E v = F::zero();
#pragma unroll
    for (int i = 0; i < N; i++) v = F::add(v, tot[i]);
    u64 w[F::L];
    F::to_words(v, w);
#pragma unroll
    for (int l = 0; l < F::L; l++) s_pub[l] = w[l];
    const E r = uniform_elem<F>(coef_state, (u64)js);
    F::to_words(F::add(F::from_words(acc_slot), F::mul(r, v)), acc_slot);
#pragma unroll
    for (int i = 0; i < N; i++) {
      u64 *q = acc_slot + (1 + i) * F::L;
      F::to_words(F::add(F::from_words(q), F::mul(r, tot[N + i])), q);
    }
  }
}

}  // namespace spdz

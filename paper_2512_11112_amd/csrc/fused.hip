// Fused element-wise groups of the control-flow runtime.
//
// A basic block's consecutive secret element-wise nodes of one width (Beaver
// products, share additions and subtractions, additions and products with public
// values; Sec. II-A "Secure operations") run as one kernel: every thread walks
// the group's instruction list for its elements, keeping intermediate secret
// values in its own column of LDS ("slots"), so a value produced and consumed
// inside the group never travels through HBM.  Each Beaver product opens d and e
// and adds them to the MAC-check sums at its node's log positions, exactly as the
// per-node product kernel does, so shares, opened values and sigma are the same
// bits whether a block runs fused or node by node.
#include <type_traits>

#include "blockred.h"
#include "coef.h"
#include "ctx.h"

namespace spdz {

template <class F, int N>
struct FusedArgs {
  FusedIns ins[FUSED_MAX_INS];
  int nins;
  int64_t W;
  typename F::E alpha[N];
  u64 coef_state;
  u64 *acc;
};

template <class F, int N>
__global__ __launch_bounds__(BLOCK) void k_fused(const FusedArgs<F, N> A) {
  using E = typename F::E;
  constexpr int L = F::L;
  // [slot][2 N][L][BLOCK] words (4 bytes for residues below 2^32): thread t owns column t
  using WordT = typename std::conditional<sizeof(E) == 4, uint32_t, u64>::type;
  extern __shared__ u64 lds_raw[];
  WordT *lds = reinterpret_cast<WordT *>(lds_raw);
  const int t = threadIdx.x;
  auto put = [&](int slot, int k, E x) {
    u64 w[2] = {0, 0};
    F::to_words(x, w);
#pragma unroll
    for (int l = 0; l < L; l++) lds[((slot * 2 * N + k) * L + l) * BLOCK + t] = (WordT)w[l];
  };
  auto get = [&](int slot, int k) -> E {
    u64 w[2] = {0, 0};
#pragma unroll
    for (int l = 0; l < L; l++) w[l] = lds[((slot * 2 * N + k) * L + l) * BLOCK + t];
    return F::from_words(w);
  };
  E mc[N + 1];
#pragma unroll
  for (int k = 0; k <= N; k++) mc[k] = F::zero();
  const int64_t W = A.W, plane = (int64_t)L * W, half = (int64_t)N * L * W;  // party plane, MAC offset
  for (int64_t e = (int64_t)blockIdx.x * BLOCK + t; e < W; e += (int64_t)gridDim.x * BLOCK) {
    for (int q = 0; q < A.nins; q++) {
      const FusedIns &I = A.ins[q];
      if (I.kind == FK_LOAD) {
#pragma unroll
        for (int i = 0; i < N; i++) {
          put(I.dst, i, F::load(I.p0 + i * plane, W, e));
          put(I.dst, N + i, F::load(I.p0 + half + i * plane, W, e));
        }
        continue;
      }
      if constexpr (2 * N * L <= 12) {  // (the runtime merges loads only while they fit 24 words)
      if (I.kind == FK_LOADS) {  // two or three operands, every word requested before any store
        constexpr int MJ = 24 / (2 * N * L) < 3 ? 24 / (2 * N * L) : 3;  // the runtime's most per step
        E v[MJ][2 * N];
        const u64 *src[3] = {I.p0, I.p1, I.p2};
#pragma unroll
        for (int j = 0; j < MJ; j++)
          if (j < I.flags)
#pragma unroll
            for (int i = 0; i < N; i++) {
              v[j][i] = F::load(src[j] + i * plane, W, e);
              v[j][N + i] = F::load(src[j] + half + i * plane, W, e);
            }
        const int dst[3] = {I.dst, I.a, I.b};
#pragma unroll
        for (int j = 0; j < MJ; j++)
          if (j < I.flags)
#pragma unroll
            for (int k = 0; k < 2 * N; k++) put(dst[j], k, v[j][k]);
        continue;
      }
      }
      if (I.kind == FK_BEAVER) {
        E av[N], bv[N];
        E d = F::zero(), ee = F::zero();
#pragma unroll
        for (int i = 0; i < N; i++) {
          av[i] = F::load(I.p0 + i * plane, W, e);
          bv[i] = F::load(I.p1 + i * plane, W, e);
          d = F::add(d, F::sub(get(I.a, i), av[i]));
          ee = F::add(ee, F::sub(get(I.b, i), bv[i]));
        }
        const E de = F::mul(d, ee);
        const E rd = uniform_elem<F>(A.coef_state, (u64)(I.j + e));
        const E re = uniform_elem<F>(A.coef_state, (u64)(I.j + W + e));
        mc[0] = F::add(mc[0], F::add(F::mul(rd, d), F::mul(re, ee)));
        // the destination slot never holds an operand of the same instruction
#pragma unroll
        for (int i = 0; i < N; i++) {
          const E am = F::load(I.p0 + half + i * plane, W, e), bm = F::load(I.p1 + half + i * plane, W, e);
          const E cv = F::load(I.p2 + i * plane, W, e), cm = F::load(I.p2 + half + i * plane, W, e);
          E z = F::add(cv, F::add(F::mul(d, bv[i]), F::mul(ee, av[i])));
          if (i == 0) z = F::add(z, de);
          const E mz = F::add(F::add(cm, F::mul(d, bm)), F::add(F::mul(ee, am), F::mul(A.alpha[i], de)));
          mc[1 + i] = F::add(mc[1 + i], F::add(F::mul(rd, F::sub(get(I.a, N + i), am)),
                                               F::mul(re, F::sub(get(I.b, N + i), bm))));
          put(I.dst, i, z);
          put(I.dst, N + i, mz);
        }
      } else if (I.kind == FK_LIN) {
#pragma unroll
        for (int k = 0; k < 2 * N; k++) {
          const E x = get(I.a, k), y = get(I.b, k);
          put(I.dst, k, (I.flags & FF_SUB) ? F::sub(x, y) : F::add(x, y));
        }
      } else {  // public operand [L][W] or a scalar [L][1]
        const bool vec = I.flags & FF_PUB_VEC;
        const E v = F::load(I.p0, vec ? W : 1, vec ? e : 0);
        if (I.kind == FK_PUBMUL) {
#pragma unroll
          for (int k = 0; k < 2 * N; k++) put(I.dst, k, F::mul(get(I.a, k), v));
        } else {  // (-)secret (+/-) public: party 0 adds to its value, party i adds alpha_i v to its MAC
          const E pv = (I.flags & FF_NEG_P) ? F::sub(F::zero(), v) : v;
#pragma unroll
          for (int i = 0; i < N; i++) {
            E x = get(I.a, i), m = get(I.a, N + i);
            if (I.flags & FF_NEG_A) {
              x = F::sub(F::zero(), x);
              m = F::sub(F::zero(), m);
            }
            put(I.dst, i, i == 0 ? F::add(x, pv) : x);
            put(I.dst, N + i, F::add(m, F::mul(A.alpha[i], pv)));
          }
        }
      }
      if (I.flags & FF_STORE) {
#pragma unroll
        for (int i = 0; i < N; i++) {
          F::store(I.out + i * plane, W, e, get(I.dst, i));
          F::store(I.out + half + i * plane, W, e, get(I.dst, N + i));
        }
      }
    }
  }
  block_add_to_slot<F, N + 1>(mc, A.acc + (size_t)blockIdx.x * (N + 1) * L);
}

// --------------------------------------------------------------------------
// The same list for few elements, where one element's chain of round trips and instructions is what a run
// waits for.  A lane takes one of the 2 N residues of an element (LANES per element), so the parties' and
// MAC shares' arithmetic runs side by side and only d and e are summed across lanes; every word the list
// reads, operands and triples, is requested up front straight into LDS, one round trip for the whole
// list.  LDS: [slot, then operand in list order][words of a residue][thread], each thread its own column.
// --------------------------------------------------------------------------
// the byte fields of an instruction from one 8-byte word, which the scalar unit can load (bytes and
// half-words it cannot: each would be a vector load's round trip on the list's way)
struct FusedOp {
  int kind, dst, a, b, flags;
};
__device__ __forceinline__ FusedOp fused_op(const FusedIns &I) {
  u64 w;
  __builtin_memcpy(&w, &I, 8);
  return FusedOp{(int)(w & 255), (int)(w >> 8 & 255), (int)(w >> 16 & 255), (int)(w >> 24 & 255), (int)(w >> 32 & 255)};
}

// buffers an instruction reads through p0, p1, p2 (public operands apart)
__host__ __device__ __forceinline__ int fused_operands(int kind, int flags) {
  return kind == FK_BEAVER ? 3 : kind == FK_LOADS ? flags : kind == FK_LOAD ? 1 : 0;
}

// lanes per element: a power of two of at least 2 n
__host__ __device__ constexpr int narrow_lanes(int n) { return n <= 2 ? 4 : n <= 4 ? 8 : 16; }

struct NarrowOps {
  const u64 *base[3 * FUSED_MAX_INS];  // the operands' buffers in list order
  int n, nslots;
};

template <class F, int N>
__global__ __launch_bounds__(BLOCK) void k_fused_narrow(const FusedArgs<F, N> A, const NarrowOps O) {
  using E = typename F::E;
  using Wd = typename F::Wide;
  constexpr int L = F::L, D = F::WORDS32, R = narrow_lanes(N), EPB = BLOCK / R;
  extern __shared__ u32 lds32[];
  const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), r = t & (R - 1);
  const int64_t W = A.W, e0 = (int64_t)blockIdx.x * EPB + t / R, e = min(e0, W - 1);
  const bool live = e0 < W && r < 2 * N;   // (other lanes follow along on words in bounds)
  const int k = r < 2 * N ? r : 0;         // residue: value share of party k, or MAC share of party k - N
  const bool mac = k >= N;
  const int64_t at_k = (int64_t)k * L * W + e;
  for (int o = 0; o < O.n; o++) {
    const u64 *src = O.base[o] + at_k;
#pragma unroll
    for (int d = 0; d < D; d++)
      __builtin_amdgcn_global_load_lds((const u32 *)(src + (d >> 1) * W) + (d & 1),
                                       (__attribute__((address_space(3))) void *)(lds32 + ((O.nslots + o) * D + d) * BLOCK + wave * 64),
                                       4, 0, 0);
  }
  // the block's MAC-check slot (its own: no other block of the launch touches it)
  u64 *slot = A.acc + (size_t)blockIdx.x * (N + 1) * L;
  const E prev = t < N + 1 ? F::from_words(slot + t * L) : F::zero();
  E alpha = F::zero();
#pragma unroll
  for (int i = 0; i < N; i++)
    if (k == N + i) alpha = A.alpha[i];
  auto get = [&](int op) -> E {
    u32 w[D];
#pragma unroll
    for (int d = 0; d < D; d++) w[d] = lds32[(op * D + d) * BLOCK + t];
    return F::from32(w);
  };
  auto put = [&](int op, E x) {
    x = F::canon(x);
#pragma unroll
    for (int d = 0; d < D; d++) lds32[(op * D + d) * BLOCK + t] = F::word32(x, d);
  };
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // a wave reads only what it requested itself
  E mc = F::zero();  // residue 0: sum r a; MAC share of party i: sum r gamma_i
  for (int q = 0, at = O.nslots; q < A.nins; q++) {
    const FusedIns &I = A.ins[q];
    const FusedOp op = fused_op(I);
    const int no = fused_operands(op.kind, op.flags);
    if (op.kind == FK_LOAD || op.kind == FK_LOADS) {
      for (int o = 0; o < no; o++) put(o == 0 ? op.dst : o == 1 ? op.a : op.b, get(at + o));
      at += no;
      continue;
    }
    const E x = get(op.a);
    E out;
    if (op.kind == FK_BEAVER) {
      const E y = get(op.b), a = get(at), b = get(at + 1), c = get(at + 2);
      const E rd = uniform_elem<F>(A.coef_state, (u64)(I.j + e));
      const E re = uniform_elem<F>(A.coef_state, (u64)(I.j + W + e));
      const E dx = F::sub(x, a), dy = F::sub(y, b);
      const bool value = r < N;
      const E d = group_sum<F, R>(value ? dx : F::zero()), ee = group_sum<F, R>(value ? dy : F::zero());
      const E de = F::mul(d, ee);
      Wd w = F::wzero();
      F::wadd(w, c);
      F::wmac(w, d, b);
      F::wmac(w, ee, a);
      // party 0's value share takes d e, a MAC share alpha_i d e
      if (mac) F::wmac(w, alpha, de);
      else if (k == 0) F::wadd(w, de);
      out = F::wreduce(w);
      Wd g = F::wzero();
      F::wmac(g, rd, mac ? dx : d);
      F::wmac(g, re, mac ? dy : ee);
      mc = F::add(mc, F::wreduce(g));
    } else if (op.kind == FK_LIN) {
      const E y = get(op.b);
      out = (op.flags & FF_SUB) ? F::sub(x, y) : F::add(x, y);
    } else {  // public operand [L][W] or a scalar [L][1]
      const bool vec = op.flags & FF_PUB_VEC;
      const E v = F::load(I.p0, vec ? W : 1, vec ? e : 0);
      if (op.kind == FK_PUBMUL) {
        out = F::mul(x, v);
      } else {  // (-)secret (+/-) public: party 0 adds to its value, party i adds alpha_i v to its MAC
        const E pv = (op.flags & FF_NEG_P) ? F::sub(F::zero(), v) : v;
        out = (op.flags & FF_NEG_A) ? F::sub(F::zero(), x) : x;
        if (mac) out = F::add(out, F::mul(alpha, pv));
        else if (k == 0) out = F::add(out, pv);
      }
    }
    put(op.dst, out);
    if ((op.flags & FF_STORE) && live) F::store(I.out + (int64_t)k * L * W, W, e, out);
    at += no;
  }
  // the MAC-check sums of residue 0 and the MAC shares: over the wave's elements, then over the waves
  if (!live) mc = F::zero();
#pragma unroll
  for (int off = 32; off >= R; off >>= 1) mc = F::add(mc, shfl_xor_e<F>(mc, off));
  __shared__ E sh[WAVES][N + 1];
  if ((t & 63) < 2 * N && (k == 0 || mac)) sh[wave][k == 0 ? 0 : 1 + k - N] = mc;
  __syncthreads();
  if (t < N + 1) {
    E s = prev;
#pragma unroll
    for (int w = 0; w < WAVES; w++) s = F::add(s, sh[w][t]);
    F::to_words(s, slot + t * L);
  }
}

spdz_status launch_fused(spdz_ctx *c, const FusedIns *ins, int nins, int nslots, int64_t W) {
  if (nins < 1 || nins > FUSED_MAX_INS || nslots < 1 || nslots > fused_max_slots(c->n, c->L, c->fid) || W < 1)
    return SPDZ_E_INVAL;
  for (int q = 0; q < nins; q++)
    if (ins[q].dst >= nslots || ins[q].a >= nslots || ins[q].b >= nslots) return SPDZ_E_INVAL;
  return visit(c, [&](auto f, auto nn) -> spdz_status {
    using F = decltype(f);
    constexpr int N = decltype(nn)::value;
    FusedArgs<F, N> A;
    for (int q = 0; q < nins; q++) A.ins[q] = ins[q];
    A.nins = nins;
    A.W = W;
    alpha_of<F, N>(c, A.alpha);
    A.coef_state = coef_state(c);
    A.acc = c->d_acc;
    // narrow: at most four blocks per CU (of BLOCK / LANES elements), and everything the list reads in LDS.
    // A loop of three products and two additions, us per trip, narrow / wide: 2^32 - 5, 2 parties, width 64
    // 7.0 / 9.0, 4096 7.5 / 13.1, 65536 (four blocks) 12.6 / 14.2, 131072 18.6 / 16.7; 2^61 - 1, 3 parties,
    // width 1000 9.0 / 17.1, 32768 (four) 14.8 / 18.5, 65536 23.9 / 19.4.
    NarrowOps O;
    O.n = 0;
    O.nslots = nslots;
    for (int q = 0; q < nins; q++) {
      const u64 *p[3] = {ins[q].p0, ins[q].p1, ins[q].p2};
      for (int o = 0; o < fused_operands(ins[q].kind, ins[q].flags); o++) O.base[O.n++] = p[o];
    }
    constexpr int EPB = BLOCK / narrow_lanes(N);
    const int64_t narrow_lds = (int64_t)(nslots + O.n) * F::WORDS32 * BLOCK * 4, blocks = (W + EPB - 1) / EPB;
    if (blocks <= 4 * c->num_cus && blocks <= MAX_SLOTS && narrow_lds <= FUSED_LDS_BYTES) {
      KTimer tm(c, "fused");
      hipLaunchKernelGGL((k_fused_narrow<F, N>), dim3((unsigned)blocks), dim3(BLOCK), (size_t)narrow_lds, c->stream, A, O);
      spdz_status s = hip_status(hipGetLastError());
      if (s == SPDZ_OK && blocks > c->slots) c->slots = (int)blocks;
      return s;
    }
    const size_t lds = (size_t)nslots * 2 * N * F::L * fused_word_bytes(c->fid) * BLOCK;
    const void *k = (const void *)k_fused<F, N>;
    const int g = grid_for(c, k, W);
    KTimer tm(c, "fused");
    hipLaunchKernelGGL((k_fused<F, N>), dim3(g), dim3(BLOCK), lds, c->stream, A);
    spdz_status s = hip_status(hipGetLastError());
    if (s == SPDZ_OK && g > c->slots) c->slots = g;
    return s;
  });
}

}  // namespace spdz

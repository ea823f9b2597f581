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
#include <algorithm>
#include <cstring>
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
        E av[N], bv[N], tm[N][4];
        // every word of the triple requested before any is used, while the registers leave the blocks in flight
        // that the loop needs (the loop of launch_fused over 2^19 elements of 2^61 - 1: 2 parties 52.8 -> 47.5 us
        // per iteration; 2^20 of 2^32 - 5, 3 parties 95 -> 100)
        constexpr bool AHEAD = N * L <= 2;
        auto rest = [&](int i) {
          tm[i][0] = F::load(I.p0 + half + i * plane, W, e);
          tm[i][1] = F::load(I.p1 + half + i * plane, W, e);
          tm[i][2] = F::load(I.p2 + i * plane, W, e);
          tm[i][3] = F::load(I.p2 + half + i * plane, W, e);
        };
#pragma unroll
        for (int i = 0; i < N; i++) {
          av[i] = F::load(I.p0 + i * plane, W, e);
          bv[i] = F::load(I.p1 + i * plane, W, e);
        }
        if constexpr (AHEAD)
#pragma unroll
          for (int i = 0; i < N; i++) rest(i);
        const E rd = uniform_elem<F>(A.coef_state, (u64)(I.j + e));
        const E re = uniform_elem<F>(A.coef_state, (u64)(I.j + W + e));
        E d = F::zero(), ee = F::zero();
#pragma unroll
        for (int i = 0; i < N; i++) {
          d = F::add(d, F::sub(get(I.a, i), av[i]));
          ee = F::add(ee, F::sub(get(I.b, i), bv[i]));
        }
        const E de = F::mul(d, ee);
        mc[0] = F::add(mc[0], F::add(F::mul(rd, d), F::mul(re, ee)));
        // the destination slot never holds an operand of the same instruction
#pragma unroll
        for (int i = 0; i < N; i++) {
          if constexpr (!AHEAD) rest(i);
          const E am = tm[i][0], bm = tm[i][1], cv = tm[i][2], cm = tm[i][3];
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
// MAC shares' arithmetic runs side by side and only d and e are summed across lanes.  The list itself comes
// into LDS in one round trip (walked through the scalar cache, each line of the kernel arguments was one,
// 0.45 us an instruction), then every word it reads, operands, triples and public operands, straight into LDS
// in a second.  After that an addition takes 0.18 us and a product 0.65 (2^32 - 5, 2 parties; 0.8 at 3 parties
// over 2^61 - 1, 2.3 over 2^127 - 1): a wave's own chain of dependent instructions.
// LDS: [slot, then operand in list order][words of a residue][thread], each thread its own column.
// --------------------------------------------------------------------------
// lanes per element: a power of two of at least 2 n
__host__ __device__ constexpr int narrow_lanes(int n) { return n <= 2 ? 4 : n <= 4 ? 8 : 16; }

struct NarrowIns {
  u64 fields;  // the first 8 bytes of a FusedIns
  u64 *out;
  int64_t j;
};
// what the list reads, in list order: buffers of shares, and public operands marked in the low bits
enum : u64 { NB_PUB = 1, NB_VEC = 2 };
template <class F, int N>
struct NarrowArgs {
  NarrowIns ins[FUSED_MAX_INS];
  u64 base[3 * FUSED_MAX_INS];
  int nins, nbase, nslots;
  int64_t W;
  typename F::E alpha[N];
  u64 coef_state;
  u64 *acc;
};

template <class F, int N>
__global__ __launch_bounds__(BLOCK) void k_fused_narrow(const NarrowArgs<F, N> A) {
  using E = typename F::E;
  using Wd = typename F::Wide;
  constexpr int L = F::L, D = F::WORDS32, R = narrow_lanes(N), EPB = BLOCK / R;
  extern __shared__ u32 lds32[];
  __shared__ NarrowIns list[FUSED_MAX_INS + 1];  // (the last is read ahead, never run)
  __shared__ u64 base[3 * FUSED_MAX_INS];
  const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), r = t & (R - 1);
  const int64_t W = A.W, e0 = (int64_t)blockIdx.x * EPB + t / R, e = min(e0, W - 1);
  const bool live = e0 < W && r < 2 * N;   // (other lanes follow along on words in bounds)
  const int k = r < 2 * N ? r : 0;         // residue: value share of party k, or MAC share of party k - N
  const bool mac = k >= N;
  const int64_t at_k = (int64_t)k * L * W + e;
  for (int i = t; i < A.nbase; i += BLOCK) base[i] = A.base[i];
  for (int i = t; i < A.nins * (int)(sizeof(NarrowIns) / 8); i += BLOCK)
    reinterpret_cast<u64 *>(list)[i] = reinterpret_cast<const u64 *>(A.ins)[i];
  __syncthreads();
#pragma unroll 4
  for (int o = 0; o < A.nbase; o++) {
    const u64 b = base[o];
    const bool pub = b & NB_PUB, vec = b & NB_VEC;
    const u64 *src = reinterpret_cast<const u64 *>(b & ~(u64)(NB_PUB | NB_VEC)) + (!pub ? at_k : vec ? e : 0);
    const int64_t limb = pub && !vec ? 1 : W;
#pragma unroll
    for (int d = 0; d < D; d++)
      __builtin_amdgcn_global_load_lds((const u32 *)(src + (d >> 1) * limb) + (d & 1),
                                       (__attribute__((address_space(3))) void *)(lds32 + ((A.nslots + o) * D + d) * BLOCK + wave * 64),
                                       4, 0, 0);
  }
  // the block's MAC-check slot (its own: no other block of the launch touches it)
  u64 *slot = A.acc + (size_t)blockIdx.x * (N + 1) * L;
  const E prev = t < N + 1 ? F::from_words(slot + t * L) : F::zero();
  // what a public value v adds to this lane's residue, times v: 1 for party 0's value, alpha_i for party i's
  // MAC share, 0 for the other values
  u64 one[2] = {k == 0, 0};
  E alpha = F::from_words(one);
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
  constexpr int TERMS = [] {  // products of two residues that Wide holds
    if constexpr (L == 1) return F::WIDE_TERMS;
    else return 2;
  }();
  Wd g = F::wzero();
  int terms = 0;  // Beaver products in g, two terms each
  const u32 *fields = reinterpret_cast<const u32 *>(list);
  constexpr int STEP = sizeof(NarrowIns) / 4;
  u32 f0 = fields[0], f1 = fields[1];
  for (int q = 0, at = A.nslots; q < A.nins; q++) {
    // the instruction's byte fields, uniform over the wave; the next one's are requested meanwhile
    const u32 w0 = __builtin_amdgcn_readfirstlane(f0), w1 = __builtin_amdgcn_readfirstlane(f1);
    const int kind = w0 & 255, dst = w0 >> 8 & 255, ia = w0 >> 16 & 255, ib = w0 >> 24, flags = w1 & 255, reads = w1 >> 8 & 255;
    f0 = fields[(q + 1) * STEP];
    f1 = fields[(q + 1) * STEP + 1];
    const NarrowIns &I = list[q];
    const E x = get(ia), y = get(ib);  // (slots in range for every kind; each uses what it needs)
    E out;
    if (kind == FK_BEAVER) {
      const E a = get(at), b = get(at + 1), c = get(at + 2);
      // the coefficients of d (even lanes) and e (odd lanes), exchanged
      const E own = uniform_elem<F>(A.coef_state, (u64)(I.j + e + ((t & 1) ? W : 0))), other = lane_xor1<F>(own);
      const E rd = (t & 1) ? other : own, re = (t & 1) ? own : other;
      const E dx = F::sub(x, a), dy = F::sub(y, b);
      const bool value = r < N;
      const E d = group_sum<F, R>(value ? dx : F::zero()), ee = group_sum<F, R>(value ? dy : F::zero());
      const E de = F::mul(d, ee);
      Wd w = F::wzero();
      F::wadd(w, c);
      F::wmac(w, d, b);
      F::wmac(w, ee, a);
      F::wmac(w, alpha, de);
      out = F::wreduce(w);
      F::wmac(g, rd, mac ? dx : d);
      F::wmac(g, re, mac ? dy : ee);
      if (++terms == TERMS / 2) {
        mc = F::add(mc, F::wreduce(g));
        g = F::wzero();
        terms = 0;
      }
    } else if (kind == FK_LIN) {
      out = F::add(x, (flags & FF_SUB) ? F::sub(F::zero(), y) : y);
    } else if (kind == FK_LOAD || kind == FK_LOADS) {
      put(dst, get(at));
      if (reads > 1) put(ia, get(at + 1));
      if (reads > 2) put(ib, get(at + 2));
      at += reads;
      continue;
    } else {  // public operand [L][W] or a scalar [L][1]
      const E v = get(at);
      if (kind == FK_PUBMUL) {
        out = F::mul(x, v);
      } else {  // (-)secret (+/-) public
        const E pv = (flags & FF_NEG_P) ? F::sub(F::zero(), v) : v;
        out = F::add((flags & FF_NEG_A) ? F::sub(F::zero(), x) : x, F::mul(alpha, pv));
      }
    }
    put(dst, out);
    if ((flags & FF_STORE) && live) F::store(I.out + (int64_t)k * L * W, W, e, out);
    at += reads;
  }
  mc = F::add(mc, F::wreduce(g));
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

// blocks of the narrow kernel over W elements, or 0 if there are too many for it (rule in launch_fused)
static int64_t narrow_blocks(const spdz_ctx *c, int64_t W) {
  const int64_t per = BLOCK / narrow_lanes(c->n), blocks = (W + per - 1) / per;
  return blocks <= 2 * c->num_cus && blocks <= MAX_SLOTS ? blocks : 0;
}

static int64_t narrow_bytes(const spdz_ctx *c, int nslots, int operands) {
  return (int64_t)(nslots + operands) * (c->fid == FID_32 ? 1 : 2 * c->L) * BLOCK * 4;
}

// the CU's LDS less what the kernel itself declares
constexpr int64_t NARROW_LDS_BYTES = 163840 - 6144;
static bool narrow_fits(const spdz_ctx *c, int nslots, int operands, int64_t blocks) {
  const int64_t bytes = narrow_bytes(c, nslots, operands);
  return bytes <= FUSED_LDS_BYTES || bytes * ((blocks + c->num_cus - 1) / c->num_cus) <= NARROW_LDS_BYTES;
}

// The narrow kernel's slots cost a lane one residue, the wide one's a thread all 2 N: 12 hold a loop body
// whole where three split it (2^127 - 1, 2 parties, width 64, the loop of launch_fused: 25.7 -> 9.2 us).
int fused_slots(const spdz_ctx *c, int64_t W) {
  const int wide = fused_max_slots(c->n, c->L, c->fid);
  return wide >= FUSED_MIN_SLOTS && narrow_blocks(c, W) > 0 ? std::max(wide, 12) : wide;
}

bool fused_runs(const spdz_ctx *c, int nslots, int operands, int64_t W, bool joined) {
  const int64_t blocks = narrow_blocks(c, W);
  if (blocks > 0 && narrow_fits(c, nslots, operands, blocks)) return true;
  return nslots <= fused_max_slots(c->n, c->L, c->fid) && !(joined && blocks > 0);
}

template <class F, int N>
static spdz_status launch_list(spdz_ctx *c, const FusedIns *ins, int nins, int nslots, int64_t W) {
  // narrow: at most two blocks per CU (of BLOCK / LANES elements), and everything the list reads in LDS.
  // A loop of three products and two additions, joined, us per iteration, narrow / wide: 2^32 - 5, 2 parties,
  // width 64 2.8 / 7.4, 32768 (two blocks) 4.9 / 7.6, 50000 8.6 / 7.7, 65536 (four) 9.6 / 8.2; 2^61 - 1,
  // 2 parties, 32768 6.9 / 9.0, 65536 13.7 / 9.9, 3 parties, 16384 (two) 7.5 / 12.6, 32768 13.8 / 12.9.
  int operands = 0;
  for (int q = 0; q < nins; q++) operands += fused_operands(ins[q].kind, ins[q].flags);
  const int64_t blocks = narrow_blocks(c, W);
  if (blocks > 0 && narrow_fits(c, nslots, operands, blocks)) {
    NarrowArgs<F, N> A;
    A.nins = nins;
    A.nbase = 0;
    A.nslots = nslots;
    for (int q = 0; q < nins; q++) {
      FusedIns I = ins[q];
      const u64 *p[3] = {I.p0, I.p1, I.p2};
      const bool pub = I.kind == FK_PUBADD || I.kind == FK_PUBMUL;
      const u64 mark = !pub ? 0 : (I.flags & FF_PUB_VEC) ? NB_PUB | NB_VEC : NB_PUB;
      I.reads = (uint8_t)fused_operands(I.kind, I.flags);
      for (int o = 0; o < I.reads; o++) A.base[A.nbase++] = (u64)(uintptr_t)p[o] | mark;
      std::memcpy(&A.ins[q].fields, &I, 8);
      A.ins[q].out = I.out;
      A.ins[q].j = I.j;
    }
    A.W = W;
    alpha_of<F, N>(c, A.alpha);
    A.coef_state = coef_state(c);
    A.acc = c->d_acc;
    KTimer tm(c, "fused");
    hipLaunchKernelGGL((k_fused_narrow<F, N>), dim3((unsigned)blocks), dim3(BLOCK),
                       (size_t)narrow_bytes(c, nslots, operands), c->stream, A);
    spdz_status s = hip_status(hipGetLastError());
    if (s == SPDZ_OK && blocks > c->slots) c->slots = (int)blocks;
    return s;
  }
  if (nslots > fused_max_slots(c->n, c->L, c->fid)) return SPDZ_E_INVAL;
  FusedArgs<F, N> A;
  for (int q = 0; q < nins; q++) A.ins[q] = ins[q];
  A.nins = nins;
  A.W = W;
  alpha_of<F, N>(c, A.alpha);
  A.coef_state = coef_state(c);
  A.acc = c->d_acc;
  const size_t lds = (size_t)nslots * 2 * N * F::L * fused_word_bytes(c->fid) * BLOCK;
  const void *k = (const void *)k_fused<F, N>;
  const int g = grid_for(c, k, W);
  KTimer tm(c, "fused");
  hipLaunchKernelGGL((k_fused<F, N>), dim3(g), dim3(BLOCK), lds, c->stream, A);
  spdz_status s = hip_status(hipGetLastError());
  if (s == SPDZ_OK && g > c->slots) c->slots = g;
  return s;
}

spdz_status launch_fused(spdz_ctx *c, const FusedIns *ins, int nins, int nslots, int64_t W) {
  if (nins < 1 || nins > FUSED_MAX_INS || nslots < 1 || nslots > FUSED_MAX_SLOTS || W < 1)
    return SPDZ_E_INVAL;
  for (int q = 0; q < nins; q++)
    if (ins[q].dst >= nslots || ins[q].a >= nslots || ins[q].b >= nslots) return SPDZ_E_INVAL;
  return visit(c, [&](auto f, auto nn) -> spdz_status {
    using F = decltype(f);
    constexpr int N = decltype(nn)::value;
    // (no list is made where a thread's slots are too few, so no kernel either)
    constexpr int word = sizeof(typename F::E) == 4 ? 4 : 8;
    if constexpr (FUSED_LDS_BYTES / (2 * N * F::L * word * BLOCK) < FUSED_MIN_SLOTS) return SPDZ_E_UNSUPPORTED;
    else return launch_list<F, N>(c, ins, nins, nslots, W);
  });
}

}  // namespace spdz

// Matrix-triple product over p = 2^61 - 1 (the tile-level Beaver identity
// Z = C + D B + A E + D E of Sec. III-D, "MPC-specific optimization"; here the
// opened matrices are called E = X - A and F = Y - B).
//
// For n parties every output is one product over a concatenated inner dimension
// 2K, with C added at the end.  The VALU engine computes P = E F once and then
//   Z_i    = C_i    + [i = 0] P   + [E | A_i]    [B_i; F]
//   M(Z)_i = M(C)_i + alpha_i P   + [E | M(A)_i] [M(B)_i; F]
// (4n + 1 products); the matrix engine folds P into the right operands,
//   Z_i    = C_i    + [E | A_i]    [B_i + [i = 0] F; F]
//   M(Z)_i = M(C)_i + [E | M(A)_i] [M(B)_i + alpha_i F; F]
// (4n products).
//
// Two engines compute the same exact integers mod p:
//   * VALU: 64 x 64 output tiles staged through LDS, 64 x 64 -> 128-bit
//     products accumulated exactly in 128 bits and folded every 32 steps;
//   * matrix cores: the operands' residues modulo 17 or 18 coprime byte-sized
//     moduli (rns.h), one exact int8 product per modulus with
//     v_mfma_i32_32x32x32_i8, whose entries mod m_t are stored as bytes and
//     joined by the Chinese remainder theorem.
#include <string.h>

#include <algorithm>

#include "ctx.h"
#include "panels.h"
#include "rns.h"

namespace spdz {

static_assert(2 * MAX_MFMA_K <= rns::MAX_TERMS, "the concatenated inner dimension of two operand pairs");

constexpr int MAXOUT = 2 * MAX_PARTIES;
constexpr int TILE = 64;

struct GemmJob {
  int npairs;
  const void *L[2];  // u64 [rows][K] (ld K)
  const void *R[2];  // u64 [K][cols] (ld cols)
  const u64 *init;   // [M][N] canonical or null
  const u64 *pmat;   // [M][N] canonical or null, added times pscale
  u64 pscale;
  u64 *out;          // [M][N]
};

struct GemmArgs {
  GemmJob job[MAXOUT];
  int64_t M, N, K;   // K of each pair
};

__device__ __forceinline__ u64 epilogue_add(u64 v, const GemmJob &j, int64_t idx) {
  F61::E x{v};
  if (j.init) x = F61::add(x, F61::E{j.init[idx]});
  if (j.pmat) x = F61::add(x, F61::mul(F61::E{j.pscale}, F61::E{j.pmat[idx]}));
  return F61::canon(x).v;
}

// --------------------------------------------------------------------------
// VALU engine
// --------------------------------------------------------------------------
constexpr int VK = 16;  // inner-dimension step staged in LDS

__global__ __launch_bounds__(256) void k_gemm_valu(const GemmArgs A) {
  const GemmJob &J = A.job[blockIdx.z];
  const int64_t r0 = (int64_t)blockIdx.y * TILE, c0 = (int64_t)blockIdx.x * TILE;
  __shared__ u64 As[VK][TILE + 1];  // [k][row]
  __shared__ u64 Bs[VK][TILE + 1];  // [k][col]
  const int t = threadIdx.x, tr = t / 16, tc = t % 16;
  u128 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 4; j++) acc[i][j] = 0;
  int since_fold = 0;
  const int64_t M = A.M, N = A.N, K = A.K;
  for (int pr = 0; pr < J.npairs; pr++) {
    const u64 *Lm = (const u64 *)J.L[pr];
    const u64 *Rm = (const u64 *)J.R[pr];
    for (int64_t k0 = 0; k0 < K; k0 += VK) {
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int idx = t + q * 256;
        const int rr = idx / VK, kk = idx % VK;
        const int64_t gr = r0 + rr, gk = k0 + kk;
        As[kk][rr] = (gr < M && gk < K) ? Lm[gr * K + gk] : 0;
        const int kb = idx / TILE, cc = idx % TILE;
        const int64_t gk2 = k0 + kb, gc = c0 + cc;
        Bs[kb][cc] = (gk2 < K && gc < N) ? Rm[gk2 * N + gc] : 0;
      }
      __syncthreads();
#pragma unroll 4
      for (int kk = 0; kk < VK; kk++) {
        u64 a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; i++) a[i] = As[kk][tr + 16 * i];
#pragma unroll
        for (int j = 0; j < 4; j++) b[j] = Bs[kk][tc + 16 * j];
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
          for (int j = 0; j < 4; j++) acc[i][j] += (u128)a[i] * b[j];
      }
      __syncthreads();
      // each product is < 2^122; after a fold the sum is < 2^67, so 32 more products fit
      since_fold += VK;
      if (since_fold >= 32) {
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
          for (int j = 0; j < 4; j++) acc[i][j] = (acc[i][j] & F61::P) + (acc[i][j] >> 61);
        since_fold = 0;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int64_t r = r0 + tr + 16 * i, c = c0 + tc + 16 * j;
      if (r < M && c < N) J.out[r * N + c] = epilogue_add(F61::reduce(acc[i][j]).v, J, r * N + c);
    }
}

// --------------------------------------------------------------------------
// matrix engine: residue planes
//
// Planes of one operand panel: per modulus, per block of 64 plane rows (rows of a
// left operand, columns of a right one) and per 64 inner indices one contiguous 4 KB
// block [chunk 4][row 64][16 bytes].  A tile's operand stage is a few such blocks, moved to
// LDS as they lie; zeros outside the matrix.  Which inner indices a chunk holds is free as long as
// both operands agree: chunk c holds c, c + 4, ..., c + 60 of its 64, so that the four lanes with one
// row of a left operand read along it.
// --------------------------------------------------------------------------
constexpr int PB = 4096;                          // bytes of one plane block
constexpr int MAXSRC = 2 * (2 * MAX_PARTIES + 1); // planes kernel: operands of one launch

__device__ __forceinline__ u32 pack4(int a, int b, int c, int d) {  // the low bytes of four ints
  return __builtin_amdgcn_perm((u32)b, (u32)a, 0x0c0c0400u) | __builtin_amdgcn_perm((u32)d, (u32)c, 0x04000c0cu);
}

struct PlaneSrc {
  const u64 *src;   // LEFT: [rows][K]; RIGHT: [K][cols]; row-major
  const u64 *add;   // nullable: scale * add joins src (same shape)
  u64 scale;
  int8_t *out;
  int64_t ld;       // columns of src
  int64_t r0, nrow; // first plane row of the panel, plane rows of the whole operand
  int64_t rb;       // 64-row blocks of the panel
  int right;
};

struct PlaneArgs {
  PlaneSrc s[MAXSRC];
  int64_t K, ks;    // inner dimension, 64-deep blocks of it
};

// One work item of 256 threads makes one plane block of every modulus: 64 plane rows x 64 inner
// indices, a thread 16 of them of one row.  Left operands: lanes 4 chunks x 16 rows; right operands: a
// wave one chunk of 64 consecutive columns.  blockIdx.y takes one operand, blockIdx.z one of gridDim.z
// parts of the moduli.  Bound by memory: 8 bytes read and T written per element (10 operands of 1024^2,
// 17 moduli: 61 -> 54 us when the loads lost their conditions, 4.9 TB/s).  The loop over the
// moduli is not unrolled: small products wait for the code itself.
template <int T>
__global__ __launch_bounds__(256) void k_planes(const PlaneArgs A) {
  const PlaneSrc &S = A.s[blockIdx.y];
  constexpr const rns::Tables &B = rns::tab<T>();
  const int t256 = threadIdx.x, left = !S.right;
  const int pr = left ? t256 >> 2 : t256 & 63, c = left ? t256 & 3 : t256 >> 6;
  const int64_t step = S.rb * A.ks * PB;
  const int per = (T + gridDim.z - 1) / gridDim.z, t0 = blockIdx.z * per, t1 = min(T, t0 + per);
  for (int64_t item = blockIdx.x; item < S.rb * A.ks; item += gridDim.x) {
    const int64_t rb = item % S.rb, kb = item / S.rb;
    const int64_t row = S.r0 + rb * 64 + pr, k = kb * 64 + c;
    // loads unconditional, at addresses kept inside (behind conditions each would be waited for by itself)
    const u64 *src = S.src + (left ? min(row, S.nrow - 1) * S.ld : min(row, S.nrow - 1));
    const u64 *add = S.add ? S.add + (src - S.src) : src;
    const int64_t dk = left ? 1 : S.ld;
    u64 d[16];
#pragma unroll
    for (int j = 0; j < 16; j++) d[j] = src[min(k + 4 * j, A.K - 1) * dk];
    if (S.add) {
      u64 y[16];
#pragma unroll
      for (int j = 0; j < 16; j++) y[j] = add[min(k + 4 * j, A.K - 1) * dk];
#pragma unroll
      for (int j = 0; j < 16; j++) d[j] = F61::canon(F61::add(F61::E{d[j]}, F61::mul(F61::E{S.scale}, F61::E{y[j]}))).v;
    }
#pragma unroll
    for (int j = 0; j < 16; j++) d[j] = row < S.nrow && k + 4 * j < A.K ? rns::digits(d[j]) : 0;
    int8_t *out = S.out + t0 * step + (rb * A.ks + kb) * PB + c * 1024 + pr * 16;
    rns::Digits next = B.digits[left][t0];
#pragma unroll 1
    for (int t = t0; t < t1; t++) {
      const rns::Digits D = next;
      next = B.digits[left][t + 1];
      u32 pk[4];
#pragma unroll
      for (int q = 0; q < 4; q++) {
        int r[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const int j = 4 * q + i;
          const int s = __builtin_amdgcn_sdot4((int)d[j], D.c0,
                                               __builtin_amdgcn_sdot4((int)(d[j] >> 32), D.c1, D.bias, false), false);
          r[i] = rns::round_mod((u32)s, D.inv, D.neg);
        }
        pk[q] = pack4(r[0], r[1], r[2], r[3]);
      }
      *reinterpret_cast<uint4 *>(out) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
      out += step;
    }
  }
}

// --------------------------------------------------------------------------
// matrix engine: the int8 products
//
// 2 x 2 waves per block, each WM x WN subtiles of 32 x 32: a block's tile is 64 WM rows by
// 64 WN columns of one output modulo one m_t.  Persistent blocks take tiles in turn; a ring of
// NB stage buffers (64 inner indices of both operands) is filled straight from global memory
// NB - 1 stages ahead, across tile ends too, so the next tile's operands arrive while the
// last one's sums are reduced.  One barrier a stage: in its first half the waves multiply
// operands read in the half before and read the second half's; then every wave waits for its
// loads of the next stage and its LDS reads, so past the barrier the next stage is whole and
// this stage's buffer is free; the second half multiplies, reads the next stage's first half
// and refills the buffer.
//
// Bound by the matrix cores at the clock the chip's power allows.  M = K = N = 4096 at 2 parties (72
// products of 4096 x 4096 x 8192): 7.7-7.9 ms, 2.5-2.6 POPS, matrix cores 78 % busy at 1.57 GHz; the
// same kernel without its loads takes 6.6 ms and with products alone 6.2-6.3.  64 products of
// base-256 digits, 64 x 64 outputs a block, took 27.5 ms for the same result.  Half-size tiles (two
// blocks a CU, 1.5 times the operand traffic) take 8.3 ms, a quarter 11.9.
// --------------------------------------------------------------------------
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void *lds_ptr;

// 16 bytes per lane from base + uoff + loff straight into LDS: a wave's 64 lanes fill the 1 KB at
// `wave_dst` (wave-uniform), lane l at wave_dst + 16 l.  The buffer form takes the uniform part of
// the address from scalar registers, so a load costs no vector instruction beside itself.
__device__ __forceinline__ void to_lds(const int8_t *base, u32 loff, u32 uoff, int8_t *wave_dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void *)base, 0, -1, 0x00027000),
                                           (lds_ptr)wave_dst, 16, (int)loff, (int)uoff, 0, 0);
}

// waits until at most V of the wave's vector-memory operations are outstanding (they end in order)
// and none of its LDS reads, then for the block
template <int V>
__device__ __forceinline__ void stage_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt((V & 15) | (V >> 4 << 14) | 0x70);  // vmcnt(V) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_lds() {
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_sched_barrier(0);
}

struct RnsArgs {
  const int8_t *L, *R;              // planes of the panel's left / right operands, source by source
  int8_t *res;                      // bytes: [z][tile][t][wave][WM][WN][lane][16]
  int lsrc[MAXOUT][2], rsrc[MAXOUT][2];  // operand pair q of output z
  int nz, T, npairs, ks;
  int64_t rbl, rbr;                 // 64-row blocks of the left / right panel
  int tx, ty;                       // tiles of the panel
};

// Tile of rank w among tx x ty: groups of four tile rows, column by column within a group, so a
// run of consecutive ranks (the tiles one XCD works on at a time) is a compact patch.
__device__ __forceinline__ void tile_of(int w, int tx, int ty, int &bx, int &by) {
  const int g = w / (4 * tx), r = w - g * 4 * tx, rows = min(4, ty - 4 * g);
  bx = r / rows;
  by = 4 * g + r - bx * rows;
}

template <int WM, int WN, int NB>
__global__ __launch_bounds__(256, WM * WN >= 16 ? 1 : 2) void k_rns_gemm(const RnsArgs A) {
  constexpr int NQ = WM + WN, SB = NQ * PB;  // plane blocks and bytes of a stage
  __shared__ __attribute__((aligned(16))) int8_t S[NB * SB];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave >> 1, wc = wave & 1;
  const int G = gridDim.x, total = A.nz * A.T * A.tx * A.ty, nst = A.npairs * A.ks;
  // blocks are dealt to the 8 XCDs in turn: XCD x takes a run of G / 8 consecutive tiles of each G
  int idx = G % 8 == 0 ? (int)(blockIdx.x % 8) * (G / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
  const u32 lrow = (u32)A.ks * PB;  // bytes of one 64-row block (<= 128 * 4096)
  const int8_t *lp, *rp;
  int lidx = idx, pair = 0, left = A.ks;  // tile, operand pair and stages left of it of the next load
  const u32 loff = threadIdx.x * 16;
  auto point = [&](int id, int pr) {
    const int per = A.tx * A.ty, gz = id / per, t = gz / A.nz, z = gz - t * A.nz;
    int bx, by;
    tile_of(id - gz * per, A.tx, A.ty, bx, by);
    lp = A.L + (((int64_t)A.lsrc[z][pr] * A.T + t) * A.rbl + (int64_t)by * WM) * (int64_t)lrow;
    rp = A.R + (((int64_t)A.rsrc[z][pr] * A.T + t) * A.rbr + (int64_t)bx * WN) * (int64_t)lrow;
  };
  // load q of the stage (blocks 0 .. WM - 1 left, then right) into the stage buffer at `buf`
  auto load = [&](int q, int8_t *buf) {
    to_lds(q < WM ? lp : rp, loff, (q < WM ? q : q - WM) * lrow, buf + q * PB + wave * 1024);
  };
  auto advance = [&]() {
    if (__builtin_expect(--left == 0, 0)) {  // the second operand pair, or the next tile's first
      left = A.ks;
      if (++pair == A.npairs) {  // past the last tile its first stages are read again (unused)
        pair = 0;
        if (lidx + G < total) lidx += G;
      }
      point(lidx, pair);
    } else {
      lp += PB;
      rp += PB;
    }
  };
  point(idx, 0);
#pragma unroll
  for (int b = 0; b < NB - 1; b++) {
#pragma unroll
    for (int q = 0; q < NQ; q++) load(q, S + b * SB);
    advance();
  }
#pragma unroll
  for (int q = 0; q < NQ / 2; q++) load(q, S + (NB - 1) * SB);
  stage_barrier<(NB - 2) * NQ + NQ / 2>();
  // MFMA operands: lane supplies row (lane & 31) of a 32-row subtile at chunk 2 kk + (lane >> 5);
  // left and right use the same chunk, so the pairing of inner indices is consistent
  const int lo = (lane >> 5) * 1024 + (lane & 31) * 16;
  const int aoff = wr * (WM / 2) * PB + lo, boff = (WM + wc * (WN / 2)) * PB + lo;
  auto rd = [&](const int8_t *base, int i, int kk) {
    return *reinterpret_cast<const v4i *>(base + (i >> 1) * PB + (i & 1) * 512 + kk * 2048);
  };
  v4i a0[WM], b0[WN], a1[WM], b1[WN];
  int cur = 0, prv = (NB - 1) * SB;  // byte offsets of the current stage's buffer and the one before
#pragma unroll
  for (int i = 0; i < WM; i++) a0[i] = rd(S + aoff, i, 0);
#pragma unroll
  for (int j = 0; j < WN; j++) b0[j] = rd(S + boff, j, 0);
  wait_lds();
  // the load of a half that follows its product k, or -1: spread evenly
  auto load_at = [](int k) constexpr { return (k + 1) * (NQ / 2) % (WM * WN) < NQ / 2 ? (k + 1) * (NQ / 2) / (WM * WN) - 1 : -1; };
  for (; idx < total; idx += G) {
    v16i acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; i++)
#pragma unroll
      for (int j = 0; j < WN; j++) acc[i][j] = (v16i){0};
    for (int st = 0; st < nst; st++) {
      const int nxt = cur + SB == NB * SB ? 0 : cur + SB;
      // behind each product at most one read (of what the next half multiplies) or one load (half a
      // stage in each half): the matrix core takes 32 cycles a product, and a run of other
      // instructions, or of loads in all four waves at once, would outlast it
#pragma unroll
      for (int k = 0; k < WM * WN; k++) {
        acc[k / WN][k % WN] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0[k / WN], b0[k % WN], acc[k / WN][k % WN], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (k < WN) b1[k] = rd(S + cur + boff, k, 1);
        if (k >= WM * WN - WM - WN && k < WM * WN - WN) a1[k - (WM * WN - NQ)] = rd(S + cur + aoff, k - (WM * WN - NQ), 1);
        if (load_at(k) >= 0) load(NQ / 2 + load_at(k), S + prv);
        __builtin_amdgcn_sched_barrier(0);
      }
      advance();
      stage_barrier<(NB - 2) * NQ>();
#pragma unroll
      for (int k = 0; k < WM * WN; k++) {
        acc[k / WN][k % WN] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1[k / WN], b1[k % WN], acc[k / WN][k % WN], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (k < WN) b0[k] = rd(S + nxt + boff, k, 0);
        if (k >= WM * WN - WM - WN && k < WM * WN - WN) a0[k - (WM * WN - NQ)] = rd(S + nxt + aoff, k - (WM * WN - NQ), 0);
        if (load_at(k) >= 0) load(load_at(k), S + cur);
        __builtin_amdgcn_sched_barrier(0);
      }
      wait_lds();
      prv = cur;
      cur = nxt;
    }
    if constexpr (WM * WN >= 16) {  // the sums stay in the accumulation registers until each is read below
#pragma unroll
      for (int i = 0; i < WM; i++)
#pragma unroll
        for (int j = 0; j < WN; j++) asm volatile("" : "+a"(acc[i][j]));
    }
    // the sums mod m_t, a byte each (|sum| <= 16382 * 128^2 < 2^28)
    const int per = A.tx * A.ty, gz = idx / per, t = gz / A.nz, z = gz - t * A.nz;
    const float inv = rns::TAB18.inv[t];
    const int neg = rns::TAB18.neg[t], c14 = rns::TAB18.c14[t];
    const u32 bias14 = rns::TAB18.bias14[t];
    int8_t *out = A.res + (((int64_t)z * per + (idx - gz * per)) * A.T + t) * (64 * 64 * WM * WN) +
                  wave * (WM * WN * 1024) + lane * 16;
#pragma unroll
    for (int i = 0; i < WM; i++)
#pragma unroll
      for (int j = 0; j < WN; j++) {
        u32 pk[4];
#pragma unroll
        for (int q = 0; q < 4; q++) {
          int r[4];
#pragma unroll
          for (int e = 0; e < 4; e++) {
            int x = acc[i][j][4 * q + e];
            asm volatile("" : "+v"(x));  // read the accumulator here, not hoisted across subtiles
            r[e] = rns::round_mod28(x, inv, neg, c14, bias14);
          }
          pk[q] = pack4(r[0], r[1], r[2], r[3]);
        }
        *reinterpret_cast<uint4 *>(out + (i * WN + j) * 1024) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        __builtin_amdgcn_sched_barrier(0);
      }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load of this block lands after its LDS is given away
}

// --------------------------------------------------------------------------
// matrix engine: the T bytes of every output element joined mod p, plus C
//
// One thread per 4 elements of a subtile, in the order the products are stored: every load a
// contiguous 256 bytes per wave, C and Z in runs of 128.  Bound by memory: T bytes, C and Z per
// element, 0.40-0.42 ms for 4 outputs of 4096^2 (5.5 TB/s; 16 elements a thread: 0.46).
struct CrtArgs {
  const int8_t *res;
  const u64 *init[MAXOUT];  // canonical or null
  u64 *out[MAXOUT];
  int64_t M, N, r0, c0;     // output shape, first row and column of the panel
  int tx, ty;
};

template <int T, int WM, int WN>
__global__ __launch_bounds__(256) void k_crt(const CrtArgs A) {
  constexpr const rns::Tables &B = rns::tab<T>();
  constexpr int TB = 64 * 64 * WM * WN, SUBS = 4 * WM * WN;  // bytes of a tile per modulus, its subtiles
  const int z = blockIdx.y, lane = threadIdx.x >> 2, q = threadIdx.x & 3;
  const int64_t nsub = (int64_t)A.tx * A.ty * SUBS;
  const u64 *init = A.init[z];
  u64 *out = A.out[z];
  for (int64_t s = blockIdx.x; s < nsub; s += gridDim.x) {
    const int tile = (int)(s / SUBS), sub = (int)(s % SUBS);
    int bx, by;
    tile_of(tile, A.tx, A.ty, bx, by);
    const int wave = sub / (WM * WN), i = sub / WN % WM, j = sub % WN;
    const int64_t row0 = A.r0 + (int64_t)by * 64 * WM + (wave >> 1) * 32 * WM + i * 32 + 8 * q + 4 * (lane >> 5);
    const int64_t col = A.c0 + (int64_t)bx * 64 * WN + (wave & 1) * 32 * WN + j * 32 + (lane & 31);
    const int8_t *p = A.res + ((int64_t)z * A.tx * A.ty + tile) * T * TB + (int64_t)sub * 1024 + threadIdx.x * 4;
    u64 ini[4];  // requested with the bytes
#pragma unroll
    for (int e = 0; e < 4; e++)  // (addresses kept inside)
      ini[e] = init ? __builtin_nontemporal_load(init + min(row0 + e, A.M - 1) * A.N + min(col, A.N - 1)) : 0;
    u32 by4[5][4];  // bytes of four moduli of one element, offset by 128
    u32 v[20];
#pragma unroll
    for (int t = 0; t < 20; t++) v[t] = t < T ? *reinterpret_cast<const u32 *>(p + (int64_t)t * TB) ^ 0x80808080u : 0u;
#pragma unroll
    for (int g = 0; g < 5; g++) {  // 4 x 4 byte transposes
      const u32 *w = v + 4 * g;
      const u32 a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), b = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
      const u32 c = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u), d = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
      by4[g][0] = __builtin_amdgcn_perm(b, a, 0x05040100u);
      by4[g][1] = __builtin_amdgcn_perm(b, a, 0x07060302u);
      by4[g][2] = __builtin_amdgcn_perm(d, c, 0x05040100u);
      by4[g][3] = __builtin_amdgcn_perm(d, c, 0x07060302u);
    }
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int64_t row = row0 + e;
      u32 D[8] = {0, 0, 0, 0, 0, 0, 0, 0}, f[2] = {0, 0};
#pragma unroll
      for (int g = 0; g < 5; g++) {
#pragma unroll
        for (int k = 0; k < 8; k++) D[k] = __builtin_amdgcn_udot4(by4[g][e], B.w[g][k], D[k], false);
#pragma unroll
        for (int k = 0; k < 2; k++) f[k] = __builtin_amdgcn_udot4(by4[g][e], B.f[g][k], f[k], false);
      }
      const int qq = ((int)(f[0] + (f[1] << 8) - B.fsum) + (1 << (rns::FRAC - 1))) >> rns::FRAC;  // |qq| <= 12
      // each D below 2^21, so either half below 2^46
      const u64 l = (u64)D[0] + ((u64)D[1] << 8) + ((u64)D[2] << 16) + ((u64)D[3] << 24);
      const u64 h = (u64)D[4] + ((u64)D[5] << 8) + ((u64)D[6] << 16) + ((u64)D[7] << 24);
      // h 2^32 = (h mod 2^29) 2^32 + (h >> 29) mod p
      const u64 s61 = F61::fold(((h & ((1ull << 29) - 1)) << 32) + (h >> 29) + l);
      F61::E x = F61::add(F61::E{s61}, F61::mul_small(F61::E{B.mp}, (u32)(16 - qq)));
      x = F61::add(x, F61::E{B.wsum});
      if (row < A.M && col < A.N) F61::store(out, 0, row * A.N + col, F61::add(x, F61::E{ini[e]}));
    }
  }
}

// ==========================================================================
// host side
// ==========================================================================
// takes a workspace of `bytes` in the old one's place, both held together; nothing changes where that fails
static spdz_status swap_ws(spdz_ctx *c, size_t bytes) {
  // (beyond a context's limit: more than any device has, so that the refusal is the runtime's own)
  const size_t ask = c->ws_limit && bytes > c->ws_limit ? (size_t)1 << 60 : bytes;
  void *fresh = nullptr;
  if (dev_alloc(&fresh, ask) != hipSuccess) return SPDZ_E_NOMEM;
  if (c->ws) {
    if (hipStreamSynchronize(c->stream) != hipSuccess) {
      hipFree(fresh);
      return SPDZ_E_HIP;
    }
    hipFree(c->ws);
  }
  c->ws = fresh;
  c->ws_bytes = bytes;
  return SPDZ_OK;
}

spdz_status ensure_ws(spdz_ctx *c, size_t bytes) {
  if (c->ws_bytes >= bytes) return SPDZ_OK;
  spdz_status s = swap_ws(c, bytes);
  if (s == SPDZ_E_NOMEM && c->ws) {
    SPDZ_RET(hip_status(hipStreamSynchronize(c->stream)));
    hipFree(c->ws);
    c->ws = nullptr;
    c->ws_bytes = 0;
    s = swap_ws(c, bytes);
  }
  return s;
}

namespace {

spdz_status valu_gemm(spdz_ctx *c, const GemmArgs &G, int nout) {
  dim3 grid((unsigned)((G.N + TILE - 1) / TILE), (unsigned)((G.M + TILE - 1) / TILE), (unsigned)nout);
  KTimer tm(c, "matmul_valu");
  hipLaunchKernelGGL(k_gemm_valu, grid, dim3(256), 0, c->stream, G);
  return hip_status(hipGetLastError());
}

// one operand of the matrix engine: src + scale add (add nullable), row-major
struct RnsOperand {
  const u64 *src, *add;
  u64 scale;
};

// outputs z < nz: init + sum over pairs q of L[lsrc[z][q]] R[rsrc[z][q]] mod p, of M x N over K
struct RnsProblem {
  int64_t M, K, N;
  int nl, nr, nz, npairs;
  RnsOperand L[2 * MAX_PARTIES + 1], R[2 * MAX_PARTIES + 1];
  int lsrc[MAXOUT][2], rsrc[MAXOUT][2];
  const u64 *init[MAXOUT];
  u64 *out[MAXOUT];
};

// workspace of a panel of pm rows and pn columns (whole tiles of tm x tn)
struct RnsPlan {
  int64_t pm, pn;           // panel size
  size_t lbytes, rbytes, sbytes;
  size_t bytes() const { return lbytes + rbytes + sbytes; }
};

constexpr size_t RNS_WS = (size_t)8 << 30;  // largest workspace taken without trying panels

RnsPlan rns_plan(const RnsProblem &P, int T, int64_t pm, int64_t pn) {
  const int64_t kp = up(P.K, 64);
  return RnsPlan{pm, pn, (size_t)P.nl * T * pm * kp, (size_t)P.nr * T * pn * kp, (size_t)P.nz * T * pm * pn};
}

// the largest panels within RNS_WS, down to one tile
RnsPlan rns_first_plan(const RnsProblem &P, int T, int tm, int tn) {
  int64_t pm = up(P.M, tm), pn = up(P.N, tn);
  while (rns_plan(P, T, pm, pn).bytes() > RNS_WS && smaller_panel(pm, pn, tm, tn)) {
  }
  return rns_plan(P, T, pm, pn);
}

template <int T, int WM, int WN, int NB>
spdz_status rns_panels(spdz_ctx *c, const RnsProblem &P, const RnsPlan &plan, char *ws, int bpc) {
  int8_t *lp = (int8_t *)ws, *rp = lp + plan.lbytes, *res = rp + plan.rbytes;
  const int64_t ks = up(P.K, 64) / 64;
  RnsArgs G;
  memset(&G, 0, sizeof(G));
  G.L = lp;
  G.R = rp;
  G.res = res;
  memcpy(G.lsrc, P.lsrc, sizeof(G.lsrc));
  memcpy(G.rsrc, P.rsrc, sizeof(G.rsrc));
  G.nz = P.nz;
  G.T = T;
  G.npairs = P.npairs;
  G.ks = (int)ks;
  CrtArgs R;
  memset(&R, 0, sizeof(R));
  R.res = res;
  memcpy(R.init, P.init, sizeof(R.init));
  memcpy(R.out, P.out, sizeof(R.out));
  R.M = P.M;
  R.N = P.N;
  for (int64_t c0 = 0; c0 < P.N; c0 += plan.pn) {
    const int64_t wn = up(std::min(plan.pn, P.N - c0), 64 * WN);
    for (int64_t r0 = 0; r0 < P.M; r0 += plan.pm) {
      const int64_t wm = up(std::min(plan.pm, P.M - r0), 64 * WM);
      PlaneArgs A;
      memset(&A, 0, sizeof(A));
      A.K = P.K;
      A.ks = ks;
      int ns = 0;
      for (int i = 0; i < P.nl; i++)
        A.s[ns++] = PlaneSrc{P.L[i].src, P.L[i].add, P.L[i].scale, lp + (size_t)i * T * wm * ks * 64, P.K, r0, P.M,
                             wm / 64, 0};
      if (r0 == 0)  // the right operands' planes serve every row panel of the column panel
        for (int i = 0; i < P.nr; i++)
          A.s[ns++] = PlaneSrc{P.R[i].src, P.R[i].add, P.R[i].scale, rp + (size_t)i * T * wn * ks * 64, P.N, c0, P.N,
                               wn / 64, 1};
      {
        const int64_t items = std::max(wm, wn) / 64 * ks;
        // few work items: the moduli are split, up to six ways, for about four blocks a CU
        const int64_t parts = std::min<int64_t>(6, std::max<int64_t>(1, 4 * (int64_t)c->num_cus / (items * ns)));
        KTimer tm(c, "matmul_planes");
        hipLaunchKernelGGL((k_planes<T>), dim3((unsigned)std::min<int64_t>(items, 65535), (unsigned)ns, (unsigned)parts),
                           dim3(256), 0, c->stream, A);
      }
      SPDZ_RET(hip_status(hipGetLastError()));
      G.rbl = wm / 64;
      G.rbr = wn / 64;
      G.tx = R.tx = (int)(wn / (64 * WN));
      G.ty = R.ty = (int)(wm / (64 * WM));
      R.r0 = r0;
      R.c0 = c0;
      const int64_t tiles = (int64_t)G.tx * G.ty;
      const int64_t grid = std::min<int64_t>(tiles * P.nz * T, (int64_t)c->num_cus * bpc);
      {
        KTimer tm(c, "matmul_mfma");
        hipLaunchKernelGGL((k_rns_gemm<WM, WN, NB>), dim3((unsigned)grid), dim3(256), 0, c->stream, G);
      }
      SPDZ_RET(hip_status(hipGetLastError()));
      {
        KTimer tm(c, "matmul_crt");
        hipLaunchKernelGGL((k_crt<T, WM, WN>),
                           dim3((unsigned)std::min<int64_t>(tiles * WM * WN, 65535), (unsigned)P.nz), dim3(256), 0,
                           c->stream, R);
      }
      SPDZ_RET(hip_status(hipGetLastError()));
    }
  }
  return SPDZ_OK;
}

// Runs the problem behind `head` bytes of the context workspace (grown as needed), after open(ws),
// which enqueues what makes its operands.  A problem whose planes and bytes would take more than
// RNS_WS runs in panels of whole tiles; where even that is not to be had, in smaller ones.
template <int T, int WM, int WN, int NB, class Open>
spdz_status rns_run(spdz_ctx *c, RnsProblem &P, size_t head, int bpc, Open &&open) {
  constexpr int tm = 64 * WM, tn = 64 * WN;
  RnsPlan plan = rns_first_plan(P, T, tm, tn);
  for (;;) {
    const spdz_status s = ensure_ws(c, head + plan.bytes());
    if (s == SPDZ_OK) {
      char *ws = (char *)c->ws;
      SPDZ_RET(open(ws));
      return rns_panels<T, WM, WN, NB>(c, P, plan, ws + head, bpc);
    }
    if (s != SPDZ_E_NOMEM || !smaller_panel(plan.pm, plan.pn, tm, tn)) return s;
    plan = rns_plan(P, T, plan.pm, plan.pn);
  }
}

// fn(moduli, WM, WN, stage buffers, blocks per CU) for the problem's moduli and tiling
template <class Fn>
auto rns_tiling(const spdz_ctx *c, const RnsProblem &P, Fn &&fn) {
  auto go = [&](auto tt) {
    constexpr int T = decltype(tt)::value;
    // Relative time of a tiling: whole rounds of the resident blocks, each as long as its tile's products
    // and the reduction of its sums (in inner indices: 340 where one block a CU leaves the matrix cores
    // idle meanwhile, half where a second one fills them), over the rate the tile reaches (M = N = 2048
    // at 2 parties: 0.99, 1.05 and 1.20 ms; 1800 x 100 x 1800 at 4: 301, 228 and 249 us; 300 x 1362 x 160
    // at 2: 36, 34 and 24 us).
    auto cost = [&](int wm, int wn, int bpc, double idle, double rate) {
      const int64_t tiles = (P.M + 64 * wm - 1) / (64 * wm) * ((P.N + 64 * wn - 1) / (64 * wn)) * P.nz * T;
      const int64_t slots = (int64_t)c->num_cus * bpc, rounds = (tiles + slots - 1) / slots;
      return (double)(rounds * slots) * wm * wn * ((double)P.K * P.npairs + idle) / rate;
    };
    const double c44 = cost(4, 4, 1, 340, 1.0), c42 = cost(4, 2, 2, 170, 0.93), c22 = cost(2, 2, 2, 170, 0.8);
    using std::integral_constant;
    if (c44 <= c42 && c44 <= c22)
      return fn(tt, integral_constant<int, 4>{}, integral_constant<int, 4>{}, integral_constant<int, 4>{}, 1);
    if (c42 <= c22)
      return fn(tt, integral_constant<int, 4>{}, integral_constant<int, 2>{}, integral_constant<int, 3>{}, 2);
    return fn(tt, integral_constant<int, 2>{}, integral_constant<int, 2>{}, integral_constant<int, 4>{}, 2);
  };
  if (P.K * P.npairs <= rns::T17_TERMS) return go(std::integral_constant<int, 17>{});
  return go(std::integral_constant<int, 18>{});
}

template <class Open>
spdz_status rns_product(spdz_ctx *c, RnsProblem &P, size_t head, Open &&open) {
  return rns_tiling(c, P, [&](auto t, auto wm, auto wn, auto nb, int bpc) {
    return rns_run<decltype(t)::value, decltype(wm)::value, decltype(wn)::value, decltype(nb)::value>(c, P, head, bpc,
                                                                                                      open);
  });
}

// the sizes of a matrix triple's product
RnsProblem triple_problem(int n, int64_t M, int64_t K, int64_t N) {
  RnsProblem P;
  memset(&P, 0, sizeof(P));
  P.M = M;
  P.K = K;
  P.N = N;
  P.nl = P.nr = 1 + 2 * n;
  P.nz = 2 * n;
  P.npairs = 2;
  return P;
}

size_t up256(size_t b) { return (b + 255) / 256 * 256; }

}  // namespace

spdz_status launch_matmul_triple(spdz_ctx *c, int64_t M, int64_t K, int64_t N, const spdz_shares *X,
                                 const spdz_shares *Y, const spdz_triple *T, spdz_shares *Z, u64 *E_pub, u64 *F_pub,
                                 int variant) {
  const int n = c->n;
  // workspace: the opened matrices if not supplied and, for the VALU engine, P; then the matrix engine's
  const size_t e_bytes = E_pub ? 0 : up256((size_t)M * K * 8), f_bytes = F_pub ? 0 : up256((size_t)K * N * 8);
  const size_t p_bytes = variant == 1 ? 0 : up256((size_t)M * N * 8), head = e_bytes + f_bytes + p_bytes;
  u64 *E = E_pub, *Fm = F_pub;
  // opens E = X - A (row-major, M K values), then F = Y - B (K N values)
  auto open = [&](char *ws) -> spdz_status {
    if (!E) E = (u64 *)ws;
    if (!Fm) Fm = (u64 *)(ws + e_bytes);
    return launch_open_diffs(c, X, &T->a, E, Y, &T->b, Fm);
  };
  auto a_of = [&](int i, bool mac) { return (mac ? T->a.mac : T->a.val) + i * T->a.party_stride; };
  auto b_of = [&](int i, bool mac) { return (mac ? T->b.mac : T->b.val) + i * T->b.party_stride; };
  auto c_of = [&](int i, bool mac) { return (mac ? T->c.mac : T->c.val) + i * T->c.party_stride; };
  auto z_of = [&](int i, bool mac) { return (mac ? Z->mac : Z->val) + i * Z->party_stride; };
  if (variant == 1) {
    RnsProblem P = triple_problem(n, M, K, N);
    for (int z = 0; z < 2 * n; z++) {
      P.lsrc[z][0] = P.rsrc[z][1] = 0;  // E, F
      P.lsrc[z][1] = P.rsrc[z][0] = 1 + z;
      P.init[z] = c_of(z % n, z >= n);
      P.out[z] = z_of(z % n, z >= n);
    }
    return rns_product(c, P, head, [&](char *ws) -> spdz_status {
      SPDZ_RET(open(ws));
      P.L[0] = RnsOperand{E, nullptr, 0};
      P.R[0] = RnsOperand{Fm, nullptr, 0};
      for (int z = 0; z < 2 * n; z++) {
        const int i = z % n;
        P.L[1 + z] = RnsOperand{a_of(i, z >= n), nullptr, 0};
        P.R[1 + z] = RnsOperand{b_of(i, z >= n), z == 0 || z >= n ? Fm : nullptr,
                                z >= n ? F61::canon(F61::E{c->alpha[i][0]}).v : 1};
      }
      return SPDZ_OK;
    });
  }
  SPDZ_RET(ensure_ws(c, head));
  SPDZ_RET(open((char *)c->ws));
  u64 *P = (u64 *)((char *)c->ws + e_bytes + f_bytes);
  GemmArgs G;
  memset(&G, 0, sizeof(G));
  G.M = M;
  G.N = N;
  G.K = K;
  // P = E F
  G.job[0] = GemmJob{1, {E, nullptr}, {Fm, nullptr}, nullptr, nullptr, 0, P};
  SPDZ_RET(valu_gemm(c, G, 1));
  // Z_i and M(Z)_i
  for (int i = 0; i < n; i++) {
    G.job[i] = GemmJob{2, {E, a_of(i, false)}, {b_of(i, false), Fm}, c_of(i, false), i == 0 ? P : nullptr, 1,
                       z_of(i, false)};
    G.job[n + i] = GemmJob{2, {E, a_of(i, true)}, {b_of(i, true), Fm}, c_of(i, true), P,
                           F61::canon(F61::E{c->alpha[i][0]}).v, z_of(i, true)};
  }
  return valu_gemm(c, G, 2 * n);
}

// C = A B mod p for public matrices (used by the dealer of matrix triples).  Takes room for the product that
// will use the triple, where it is to be had: grown from the dealer's own in the first product, the workspace
// cost that product a wait for the stream and about 300 us of hipFree and hipMalloc (3 parties, 64 x 4000 x 64:
// 685 us where the second took 116).
spdz_status launch_public_matmul(spdz_ctx *c, int64_t M, int64_t K, int64_t N, const u64 *Am, const u64 *Bm, u64 *Cm) {
  const RnsProblem use = triple_problem(c->n, M, K, N);
  const size_t room = rns_tiling(c, use, [&](auto t, auto wm, auto wn, auto, int) {
    return rns_first_plan(use, t, 64 * wm, 64 * wn).bytes();
  }) + up256((size_t)M * K * 8) + up256((size_t)K * N * 8);
  if (c->ws_bytes < room && swap_ws(c, room) == SPDZ_E_HIP) return SPDZ_E_HIP;
  RnsProblem P;
  memset(&P, 0, sizeof(P));
  P.M = M;
  P.K = K;
  P.N = N;
  P.nl = P.nr = P.nz = P.npairs = 1;
  P.L[0] = RnsOperand{Am, nullptr, 0};
  P.R[0] = RnsOperand{Bm, nullptr, 0};
  P.out[0] = Cm;
  return rns_product(c, P, 0, [](char *) { return SPDZ_OK; });
}

}  // namespace spdz

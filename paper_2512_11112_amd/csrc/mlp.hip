// FP32 MLP cost model of the learned dispatcher: 7 -> 64 -> 64 -> 64 -> 2 with
// ReLU on the hidden layers, trained by minibatch Adam on the mean squared
// error.  A wave takes a few samples at a time, one lane per neuron, the
// weights of its neuron in registers; gradients are summed over chunks of the
// batch in a fixed order (no atomics, so they are deterministic).
#include <string.h>

#include <algorithm>
#include <numeric>
#include <random>
#include <vector>

#include "ctx.h"

namespace spdz {

constexpr int IN = SPDZ_MLP_IN, HID = SPDZ_MLP_HID, OUT = SPDZ_MLP_OUT;
// parameter offsets
constexpr int OW1 = 0, OB1 = OW1 + HID * IN, OW2 = OB1 + HID, OB2 = OW2 + HID * HID, OW3 = OB2 + HID,
              OB3 = OW3 + HID * HID, OW4 = OB3 + HID, OB4 = OW4 + OUT * HID, NPARAM = OB4 + OUT;
static_assert(NPARAM == SPDZ_MLP_NPARAM, "parameter count");

constexpr int NS = 4;    // samples a wave works on at a time (independent sums, one set of weights)
constexpr int LD = 68;   // row length of weights in LDS: 16 lanes' 16-byte reads of consecutive rows hit all banks

// sums of NS samples' row . weights over 64 inputs, each in ascending order from s; hs: a wave's [NS][64] in LDS
__device__ __forceinline__ void dot64(const float (&w)[HID], const float *hs, float (&s)[NS]) {
#pragma unroll
  for (int k = 0; k < HID; k += 4) {
    if (k % 16 == 0) __builtin_amdgcn_sched_barrier(0);  // reads run at most 32 inputs ahead: registers
#pragma unroll
    for (int q = 0; q < NS; q++) {
      const float4 h = *reinterpret_cast<const float4 *>(hs + q * HID + k);
      s[q] = fmaf(w[k], h.x, s[q]);
      s[q] = fmaf(w[k + 1], h.y, s[q]);
      s[q] = fmaf(w[k + 2], h.z, s[q]);
      s[q] = fmaf(w[k + 3], h.w, s[q]);
    }
  }
}

// Lane j of a wave is neuron j of each layer; activations pass between layers through the wave's own
// LDS rows, read by all lanes at once.  Bound at small batches by reading the weights and a chain of
// about 210 multiply-adds: 6 us at batch 32, where one thread per sample with its activations in
// scratch memory took 41-45.
__global__ __launch_bounds__(256) void k_mlp_forward(const float *__restrict__ W, const float *__restrict__ X,
                                                     int64_t B, float *__restrict__ Y, float *__restrict__ acts) {
  __shared__ __attribute__((aligned(16))) float w2[HID * LD], w3[HID * LD], w4[OUT * LD], h[4][NS * HID];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
#pragma unroll
  for (int i = 0; i < HID * HID / 256; i++) {
    const int e = t + 256 * i;
    w2[e / HID * LD + e % HID] = W[OW2 + e];
    w3[e / HID * LD + e % HID] = W[OW3 + e];
  }
  if (t < OUT * HID) w4[t / HID * LD + t % HID] = W[OW4 + t];
  float r1[IN], r2[HID], r3[HID];
#pragma unroll
  for (int k = 0; k < IN; k++) r1[k] = W[OW1 + lane * IN + k];
  const float b1 = W[OB1 + lane], b2 = W[OB2 + lane], b3 = W[OB3 + lane], b4 = W[OB4 + (lane & 1)];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < HID; k += 4) {
    *reinterpret_cast<float4 *>(r2 + k) = *reinterpret_cast<const float4 *>(w2 + lane * LD + k);
    *reinterpret_cast<float4 *>(r3 + k) = *reinterpret_cast<const float4 *>(w3 + lane * LD + k);
  }
  float *hs = h[wave];
  for (int64_t s0 = ((int64_t)blockIdx.x * 4 + wave) * NS; s0 < B; s0 += (int64_t)gridDim.x * 4 * NS) {
    const int ns = (int)min((int64_t)NS, B - s0);  // (samples past the batch repeat the last one, unwritten)
    float s[NS];
    auto layer = [&](int l) {  // ReLU, into the wave's rows and the saved activations
#pragma unroll
      for (int q = 0; q < NS; q++) {
        s[q] = fmaxf(s[q], 0.f);
        hs[q * HID + lane] = s[q];
        if (acts && q < ns) acts[((int64_t)l * B + s0 + q) * HID + lane] = s[q];
      }
    };
#pragma unroll
    for (int q = 0; q < NS; q++) {
      const float *x = X + (s0 + min(q, ns - 1)) * IN;
      s[q] = b1;
#pragma unroll
      for (int k = 0; k < IN; k++) s[q] = fmaf(r1[k], x[k], s[q]);
    }
    layer(0);
#pragma unroll
    for (int q = 0; q < NS; q++) s[q] = b2;
    dot64(r2, hs, s);
    layer(1);
#pragma unroll
    for (int q = 0; q < NS; q++) s[q] = b3;
    dot64(r3, hs, s);
    layer(2);
    if (lane < OUT * NS) {  // the head: lane 2 q + o is output o of sample q
      const int q = lane >> 1, o = lane & 1;
      float y = b4;
#pragma unroll
      for (int k = 0; k < HID; k += 4) {
        const float4 a = *reinterpret_cast<const float4 *>(w4 + o * LD + k);
        const float4 v = *reinterpret_cast<const float4 *>(hs + q * HID + k);
        y = fmaf(a.x, v.x, y);
        y = fmaf(a.y, v.y, y);
        y = fmaf(a.z, v.z, y);
        y = fmaf(a.w, v.w, y);
      }
      if (q < ns) Y[(s0 + q) * OUT + o] = y;
    }
  }
}

// one thread per sample, the weights read from LDS by all lanes at once: outputs alone, of batches that
// fill the GPU with samples (the same sums in the same order)
__global__ __launch_bounds__(256) void k_mlp_predict(const float *__restrict__ W, const float *__restrict__ X,
                                                     int64_t B, float *__restrict__ Y) {
  __shared__ float w[NPARAM];
  for (int i = threadIdx.x; i < NPARAM; i += 256) w[i] = W[i];
  __syncthreads();
  const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (b >= B) return;
  float x[IN], h1[HID], h2[HID];
#pragma unroll
  for (int k = 0; k < IN; k++) x[k] = X[b * IN + k];
#pragma unroll 4
  for (int j = 0; j < HID; j++) {
    float s = w[OB1 + j];
#pragma unroll
    for (int k = 0; k < IN; k++) s = fmaf(w[OW1 + j * IN + k], x[k], s);
    h1[j] = fmaxf(s, 0.f);
  }
#pragma unroll 4
  for (int j = 0; j < HID; j++) {
    float s = w[OB2 + j];
#pragma unroll
    for (int k = 0; k < HID; k++) s = fmaf(w[OW2 + j * HID + k], h1[k], s);
    h2[j] = fmaxf(s, 0.f);
  }
  // layer 3 reuses h1 as storage
#pragma unroll 4
  for (int j = 0; j < HID; j++) {
    float s = w[OB3 + j];
#pragma unroll
    for (int k = 0; k < HID; k++) s = fmaf(w[OW3 + j * HID + k], h2[k], s);
    h1[j] = fmaxf(s, 0.f);
  }
#pragma unroll
  for (int o = 0; o < OUT; o++) {
    float s = w[OB4 + o];
#pragma unroll
    for (int k = 0; k < HID; k++) s = fmaf(w[OW4 + o * HID + k], h1[k], s);
    Y[b * OUT + o] = s;
  }
}

// Gradients of one parameter group (blockIdx.y: 0 first layer and head, 1 second, 2 third hidden layer)
// over the chunks of CHUNK samples this block takes, into out + blockIdx.x NPARAM.  Per chunk the 8
// waves form the deltas of the pre-activations they need (lane k sums column k of the weights), the
// block then its group's outer products, a thread eight of them, samples in ascending order.
// A block keeps the deltas on chip: 10 us at batch 32 (12 with the samples' LDS reads one at a time; 25 at 8192, then
// 30 for the sum of the parts), where deltas by one thread per sample (43-47 us) and products by one thread per
// parameter (11; 2300 at 8192) met in memory.
constexpr int CHUNK = 64;
__global__ __launch_bounds__(512) void k_mlp_backward(const float *__restrict__ W, const float *__restrict__ X,
                                                      const float *__restrict__ acts, const float *__restrict__ dY,
                                                      int64_t B, float *__restrict__ out) {
  __shared__ __attribute__((aligned(16))) float D[CHUNK * HID], in[CHUNK * HID], h[8][NS * HID], dy[CHUNK * OUT], xs[CHUNK * IN];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, group = blockIdx.y;
  out += (int64_t)blockIdx.x * NPARAM;
  float c2[HID], c3[HID], c4[OUT];
  if (group < 2)
#pragma unroll
    for (int j = 0; j < HID; j++) c3[j] = W[OW3 + j * HID + lane];
  if (group < 1)
#pragma unroll
    for (int j = 0; j < HID; j++) c2[j] = W[OW2 + j * HID + lane];
#pragma unroll
  for (int o = 0; o < OUT; o++) c4[o] = W[OW4 + o * HID + lane];
  float *hs = h[wave];
  float g[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, ga = 0.f, gb = 0.f;
  for (int64_t c0 = (int64_t)blockIdx.x * CHUNK; c0 < B; c0 += (int64_t)gridDim.x * CHUNK) {
    const int n = (int)min((int64_t)CHUNK, B - c0);
    // the products' other operand: activations of the layer below (of the head's for group 0)
    const float *src = acts + ((group == 0 ? 2 : group - 1) * B + c0) * HID;
    for (int i = t; i < n * HID; i += 512) in[i] = src[i];
    if (group == 0) {
      for (int i = t; i < n * OUT; i += 512) dy[i] = dY[c0 * OUT + i];
      for (int i = t; i < n * IN; i += 512) xs[i] = X[c0 * IN + i];
    }
    for (int q0 = wave * NS; q0 < n; q0 += 8 * NS) {
      float s[NS], m[NS][3];
#pragma unroll
      for (int q = 0; q < NS; q++) {
        const int64_t b = c0 + min(q0 + q, n - 1);
#pragma unroll
        for (int l = 0; l < 3; l++) m[q][l] = l + 1 >= group ? acts[(l * B + b) * HID + lane] : 0.f;
        s[q] = 0.f;
#pragma unroll
        for (int o = 0; o < OUT; o++) s[q] = fmaf(c4[o], dY[b * OUT + o], s[q]);
        s[q] = m[q][2] > 0.f ? s[q] : 0.f;
      }
      auto down = [&](const float (&c)[HID], int l) {  // deltas of the layer below
#pragma unroll
        for (int q = 0; q < NS; q++) {
          hs[q * HID + lane] = s[q];
          s[q] = 0.f;
        }
        dot64(c, hs, s);
#pragma unroll
        for (int q = 0; q < NS; q++) s[q] = m[q][l] > 0.f ? s[q] : 0.f;
      };
      if (group < 2) down(c3, 1);
      if (group < 1) down(c2, 0);
#pragma unroll
      for (int q = 0; q < NS; q++)
        if (q0 + q < n) D[(q0 + q) * HID + lane] = s[q];
    }
    __syncthreads();
    if (group > 0) {  // 2 rows x 4 columns a thread; a bias in each of the first 64
      const int j = t >> 4 << 1, k = (t & 15) << 2;
#pragma unroll 4
      for (int b = 0; b < n; b++) {
        const float2 d = *reinterpret_cast<const float2 *>(D + b * HID + j);
        const float4 v = *reinterpret_cast<const float4 *>(in + b * HID + k);
        g[0] = fmaf(d.x, v.x, g[0]);
        g[1] = fmaf(d.x, v.y, g[1]);
        g[2] = fmaf(d.x, v.z, g[2]);
        g[3] = fmaf(d.x, v.w, g[3]);
        g[4] = fmaf(d.y, v.x, g[4]);
        g[5] = fmaf(d.y, v.y, g[5]);
        g[6] = fmaf(d.y, v.z, g[6]);
        g[7] = fmaf(d.y, v.w, g[7]);
      }
      if (t < HID)
#pragma unroll 8
        for (int b = 0; b < n; b++) ga += D[b * HID + t];
    } else {  // first layer: 448 weights and 64 biases; head: 128 weights and 2 biases
      const int j = t / IN, k = t % IN;
      if (t < HID * IN)
#pragma unroll 8
        for (int b = 0; b < n; b++) ga = fmaf(D[b * HID + j], xs[b * IN + k], ga);
      else
#pragma unroll 8
        for (int b = 0; b < n; b++) ga += D[b * HID + t - HID * IN];
      if (t < OUT * HID)
#pragma unroll 8
        for (int b = 0; b < n; b++) gb = fmaf(dy[b * OUT + t / HID], in[b * HID + t % HID], gb);
      else if (t < OUT * HID + OUT)
#pragma unroll 8
        for (int b = 0; b < n; b++) gb += dy[b * OUT + t - OUT * HID];
    }
    __syncthreads();  // the chunk's rows are reused
  }
  if (group > 0) {
    const int j = t >> 4 << 1, k = (t & 15) << 2;
    float *o = out + (group == 1 ? OW2 : OW3) + j * HID + k;
#pragma unroll
    for (int i = 0; i < 8; i++) o[i / 4 * HID + i % 4] = g[i];
    if (t < HID) out[(group == 1 ? OB2 : OB3) + t] = ga;
  } else {
    out[OW1 + t] = ga;  // W1, then b1
    if (t < OUT * HID + OUT) out[OW4 + t] = gb;  // W4, then b4
  }
}

// dW = the sum of n partial gradients
__global__ __launch_bounds__(256) void k_mlp_sum(const float *__restrict__ part, int n, float *__restrict__ dW) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= NPARAM) return;
  float s = 0.f;
  for (int i = 0; i < n; i++) s += part[(int64_t)i * NPARAM + p];
  dW[p] = s;
}

__global__ __launch_bounds__(256) void k_mlp_adam(float *W, const float *dW, float *m, float *v, float lr, float b1,
                                                  float b2, float eps, float c1, float c2) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= NPARAM) return;
  const float g = dW[p];
  const float mm = b1 * m[p] + (1.f - b1) * g;
  const float vv = b2 * v[p] + (1.f - b2) * g * g;
  m[p] = mm;
  v[p] = vv;
  W[p] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
}

// dY = 2 (Y - T) / (B * OUT): gradient of the mean squared error over the batch
__global__ __launch_bounds__(256) void k_mse_grad(const float *Y, const float *T, int64_t n, float scale, float *dY) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) dY[i] = scale * (Y[i] - T[i]);
}

__global__ __launch_bounds__(256) void k_gather_rows(const float *src, const int32_t *idx, int64_t B, int width,
                                                     float *dst) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < B * width) dst[i] = src[(int64_t)idx[i / width] * width + i % width];
}

static unsigned blocks(int64_t n) { return (unsigned)((n + 255) / 256); }

// blocks of the forward kernel: one per 16 samples, at most what is resident (more samples loop)
spdz_status mlp_forward_launch(hipStream_t st, const float *W, const float *X, int64_t B, float *Y, float *acts) {
  if (B <= 0) return SPDZ_OK;
  // outputs alone: one lane per neuron takes 29 us for 30000 samples and 79 for 100000, one thread per
  // sample 46 and 67; with the activations the first is ahead throughout (96 against 109 at 100000)
  if (!acts && B > 65536) {
    hipLaunchKernelGGL(k_mlp_predict, dim3(blocks(B)), dim3(256), 0, st, W, X, B, Y);
    return hip_status(hipGetLastError());
  }
  const int64_t need = (B + 4 * NS - 1) / (4 * NS);
  hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)std::min<int64_t>(need, 512)), dim3(256), 0, st, W, X, B, Y, acts);
  return hip_status(hipGetLastError());
}

}  // namespace spdz

using namespace spdz;

extern "C" {

spdz_status spdz_mlp_forward(void *stream, const float *W, const float *X, int64_t B, float *Y, float *acts) {
  if (!W || !X || !Y || B < 0) return SPDZ_E_INVAL;
  return mlp_forward_launch((hipStream_t)stream, W, X, B, Y, acts);
}

spdz_status spdz_mlp_backward(void *stream, const float *W, const float *X, const float *acts, const float *dY,
                              int64_t B, float *dW) {
  if (!W || !X || !acts || !dY || !dW || B < 1) return SPDZ_E_INVAL;
  hipStream_t st = (hipStream_t)stream;
  // one chunk writes the gradient itself; more leave partial sums (of up to 256 blocks) for a second pass
  const int64_t parts = std::min<int64_t>((B + CHUNK - 1) / CHUNK, 256);
  float *part = dW;
  if (parts > 1 &&
      no_error(hipMallocAsync((void **)&part, (size_t)parts * NPARAM * sizeof(float), st)) != hipSuccess)
    return SPDZ_E_NOMEM;
  hipLaunchKernelGGL(k_mlp_backward, dim3((unsigned)parts, 3), dim3(512), 0, st, W, X, acts, dY, B, part);
  if (parts > 1) hipLaunchKernelGGL(k_mlp_sum, dim3(blocks(NPARAM)), dim3(256), 0, st, part, (int)parts, dW);
  spdz_status s = hip_status(hipGetLastError());
  if (parts > 1) (void)hipFreeAsync(part, st);
  return s;
}

spdz_status spdz_mlp_adam(void *stream, float *W, const float *dW, float *m, float *v, int64_t t, float lr, float beta1,
                          float beta2, float eps) {
  if (!W || !dW || !m || !v || t < 1) return SPDZ_E_INVAL;
  const float c1 = 1.f - powf(beta1, (float)t), c2 = 1.f - powf(beta2, (float)t);
  hipLaunchKernelGGL(k_mlp_adam, dim3(blocks(NPARAM)), dim3(256), 0, (hipStream_t)stream, W, dW, m, v, lr, beta1, beta2,
                     eps, c1, c2);
  return hip_status(hipGetLastError());
}

spdz_status spdz_mlp_train(void *stream, float *W, const float *X, const float *T, int64_t N, int epochs, int batch,
                           float lr, uint64_t seed, float *loss_per_epoch) {
  if (!W || !X || !T || N < 1 || epochs < 1 || batch < 1) return SPDZ_E_INVAL;
  hipStream_t st = (hipStream_t)stream;
  const int64_t Bm = std::min<int64_t>(batch, N);
  float *buf = nullptr;
  int32_t *d_idx = nullptr;
  const size_t nb = (size_t)Bm * IN + (size_t)Bm * OUT * 3 + (size_t)3 * Bm * HID + 3 * (size_t)NPARAM +
                    (size_t)N * OUT;
  if (dev_alloc(&buf, nb * sizeof(float)) != hipSuccess) return SPDZ_E_NOMEM;
  if (dev_alloc(&d_idx, (size_t)N * sizeof(int32_t)) != hipSuccess) {
    (void)hipFree(buf);
    return SPDZ_E_NOMEM;
  }
  float *xb = buf, *tb = xb + Bm * IN, *yb = tb + Bm * OUT, *dy = yb + Bm * OUT, *acts = dy + Bm * OUT,
        *dW = acts + 3 * Bm * HID, *m = dW + NPARAM, *v = m + NPARAM, *yall = v + NPARAM;
  spdz_status s = hip_status(hipMemsetAsync(m, 0, 2 * NPARAM * sizeof(float), st));
  std::vector<int32_t> order(N);
  std::iota(order.begin(), order.end(), 0);
  std::mt19937_64 rng(seed);
  std::vector<float> yh((size_t)N * OUT), th((size_t)N * OUT);
  if (s == SPDZ_OK && loss_per_epoch)
    s = hip_status(hipMemcpyAsync(th.data(), T, th.size() * sizeof(float), hipMemcpyDeviceToHost, st));
  int64_t step = 0;
  for (int ep = 0; ep < epochs && s == SPDZ_OK; ep++) {
    std::shuffle(order.begin(), order.end(), rng);
    s = hip_status(hipMemcpyAsync(d_idx, order.data(), (size_t)N * sizeof(int32_t), hipMemcpyHostToDevice, st));
    for (int64_t b0 = 0; b0 + Bm <= N && s == SPDZ_OK; b0 += Bm) {
      hipLaunchKernelGGL(k_gather_rows, dim3(blocks(Bm * IN)), dim3(256), 0, st, X, d_idx + b0, Bm, IN, xb);
      hipLaunchKernelGGL(k_gather_rows, dim3(blocks(Bm * OUT)), dim3(256), 0, st, T, d_idx + b0, Bm, OUT, tb);
      s = mlp_forward_launch(st, W, xb, Bm, yb, acts);
      if (s != SPDZ_OK) break;
      hipLaunchKernelGGL(k_mse_grad, dim3(blocks(Bm * OUT)), dim3(256), 0, st, yb, tb, Bm * OUT,
                         2.f / (float)(Bm * OUT), dy);
      s = spdz_mlp_backward(st, W, xb, acts, dy, Bm, dW);
      if (s == SPDZ_OK) s = spdz_mlp_adam(st, W, dW, m, v, ++step, lr, 0.9f, 0.999f, 1e-8f);
    }
    if (s == SPDZ_OK && loss_per_epoch) {
      s = mlp_forward_launch(st, W, X, N, yall, nullptr);
      if (s == SPDZ_OK)
        s = hip_status(hipMemcpyAsync(yh.data(), yall, yh.size() * sizeof(float), hipMemcpyDeviceToHost, st));
      if (s == SPDZ_OK) s = hip_status(hipStreamSynchronize(st));
      double acc = 0;
      for (size_t i = 0; i < yh.size(); i++) acc += (double)(yh[i] - th[i]) * (yh[i] - th[i]);
      loss_per_epoch[ep] = (float)(acc / yh.size());
    }
  }
  if (hipStreamSynchronize(st) != hipSuccess && s == SPDZ_OK) s = SPDZ_E_HIP;
  (void)hipFree(buf);
  (void)hipFree(d_idx);
  return s;
}

}  // extern "C"

// Learned parameter initialiser for the gradient-descent mixing application (paper Sec. 4,
// "Example usage"): a convolutional encoder maps the log-mel features of a dry track and of the
// target mix to the normalised parameters of the track's gain/pan -> EQ -> compressor chain.
//
// Network: six convolution layers (kernel 5, stride 2, zero padding 2, bias, ReLU), 256 -> 64
// channels then 64 -> 64, frames F -> ceil(F/2) per layer; the mean over the remaining frames;
// one linear head 64 -> 11 and a sigmoid. Weights are one flat float32 buffer:
// [W1 (64 x 256 x 5), b1 (64), W2 (64 x 64 x 5), b2, ..., W6, b6, Wh (11 x 64), bh (11)].
//
// Every convolution, forward and backward, is an implicit GEMM on the matrix cores without an
// im2col buffer. Training runs in float32 on v_mfma_f32_16x16x4_f32: the instruction is a chain of
// float32 fused multiply-adds in ascending k (compared bit for bit with fmaf on gfx950), so an
// output has the bits of the plain loop over (channel, tap) whatever tile computes it. Inference
// can run on v_mfma_f32_16x16x16_bf16 with float32 accumulation. The first layer (256 input
// channels, 0.8 of the multiplications) has a tiled kernel; the others are small (a few frames a
// sample), so one block per sample runs all of them, the pooling and the head from LDS, and the
// backward does the same in reverse. The weight gradients of all layers and of the head are one
// launch (sums in a fixed order: runs are bit-reproducible).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "device_common.h"
#include "grafx_internal.h"
#include "kernels.h"

namespace grafx {
namespace {

constexpr int kCin = 256, kCh = 64, kLayers = 6, kKs = 5, kOut = 11;

int frames_after(int f) { return (f + 1) / 2; }

struct EncLayout {
  int B, F[kLayers + 1];
  size_t w[kLayers + 2], b[kLayers + 2];  // weight and bias offsets (layer 1..6, head = 7)
  size_t n_w;
  size_t y[kLayers + 1], h, act;          // activations: y_l [B][64][F_l], pooled h [B][64]
  size_t dy[kLayers + 1], dz, lossp, grad;  // backward scratch
};

int cin_of(int l) { return l == 1 ? kCin : kCh; }

EncLayout enc_layout(int B, int F) {
  EncLayout L{};
  L.B = B;
  L.F[0] = F;
  size_t o = 0;
  for (int l = 1; l <= kLayers; ++l) {
    L.F[l] = frames_after(L.F[l - 1]);
    L.w[l] = o;
    o += (size_t)kCh * cin_of(l) * kKs;
    L.b[l] = o;
    o += kCh;
  }
  L.w[kLayers + 1] = o;
  o += (size_t)kOut * kCh;
  L.b[kLayers + 1] = o;
  o += kOut;
  L.n_w = o;
  size_t a = 0, d = 0;
  for (int l = 1; l <= kLayers; ++l) {
    L.y[l] = a;
    a += (size_t)B * kCh * L.F[l];
    L.dy[l] = d;
    d += (size_t)B * kCh * L.F[l];
  }
  L.h = a;
  a += (size_t)B * kCh;
  L.act = a;
  L.dz = d;
  d += (size_t)B * kOut;
  L.lossp = d;
  d += (size_t)B;
  d += (size_t)B * kCh;  // not used; part of the size callers allocate
  L.grad = d;
  return L;
}

// ---- matrix-core layers -----------------------------------------------------------------------

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // weights: any float address

__device__ __forceinline__ short to_bf16(float f) {  // round to nearest even
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (short)(u >> 16);
}

// Operand layouts, lane l = i + 16 q. v_mfma_f32_16x16x4_f32: A row i, k = q; B column i, k = q.
// v_mfma_f32_16x16x16_bf16: k = 4 q .. 4 q + 3. Both: D column i, rows 4 q .. 4 q + 3.
//
// A row of K operands in LDS, read four steps at a time: in float32 lane q takes k = 4 s + q, so
// the entries of one q are stored together ([q][s]) and one 16-byte read serves four steps; in
// bfloat16 the natural order is already what a lane reads. Rows are padded by 4 entries, which
// spreads the 16-byte reads of eight consecutive rows over distinct banks.
template <bool BF16, int KC>
struct Operand {
  using T = typename std::conditional<BF16, short, float>::type;
  static constexpr int kRow = KC + 4;
  static __device__ __forceinline__ int at(int k) { return BF16 ? k : (k & 3) * (KC / 4) + (k >> 2); }
  static __device__ __forceinline__ T put(float v) {
    if constexpr (BF16) return to_bf16(v);
    else return v;
  }
};

// acc[j] += A(16 rows at a) x B(16 columns at b + j * 16 rows) over KC entries
template <bool BF16, int KC, int NT, typename T>
__device__ __forceinline__ void mma_chunk(const T* a, const T* b, f32x4 (&acc)[NT], int i, int q) {
  constexpr int R = Operand<BF16, KC>::kRow;
  if constexpr (BF16) {
#pragma unroll
    for (int ks = 0; ks < KC; ks += 16) {
      const bf16x4 av = *reinterpret_cast<const bf16x4*>(a + i * R + ks + 4 * q);
#pragma unroll
      for (int j = 0; j < NT; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
            av, *reinterpret_cast<const bf16x4*>(b + (16 * j + i) * R + ks + 4 * q), acc[j], 0, 0,
            0);
    }
  } else {
#pragma unroll
    for (int s = 0; s < KC / 4; s += 4) {
      const f32x4 av = *reinterpret_cast<const f32x4*>(a + i * R + q * (KC / 4) + s);
      f32x4 bv[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j)
        bv[j] = *reinterpret_cast<const f32x4*>(b + (16 * j + i) * R + q * (KC / 4) + s);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], bv[j][e], acc[j], 0, 0, 0);
    }
  }
}

// One layer over columns n = b * Fout + t: y[b][co][t] = ReLU(bias[co] + sum_{ci,k} W[co][ci][k]
// x[b][ci][2t + k - 2]). A block computes all 64 channels of 16 NT columns, wave w the channels
// 16 w .. 16 w + 15. K = Cin x 5 advances in chunks of CI input channels, staged in LDS while the
// next chunk's loads are in flight. Two shapes: NT = 4, CI = 16 fills the CUs from 140 to 190
// blocks on (256 samples x 125 frames, layer 1, 2.6 GFLOP: 44 us, 61 TFLOP/s of the 154 that a
// large float32 matrix product reaches; the six layers took 1105 us with one thread per output);
// below that a chunk's load latency counts, and NT = 1, CI = 64 has four times the blocks and a
// quarter of the chunks (4 samples in bfloat16: 14 us, 27 us with 64 columns and a block per 64).
template <bool BF16, int NT, int CI>
__global__ __launch_bounds__(kBlock) void conv_fwd_kernel(int B, int Cin, int Fin, int Fout,
                                                          const float* x, const float* W,
                                                          const float* bias, float* y) {
  constexpr int KC = CI * kKs, COLS = 16 * NT;
  using Op = Operand<BF16, KC>;
  constexpr int kA = kCh * KC / 4 / kBlock;       // 4-float groups of W staged per thread
  constexpr int kStep = kBlock / COLS, kB = CI / kStep;  // input channels staged per thread
  __shared__ __align__(16) typename Op::T As[kCh * Op::kRow], Bs[COLS * Op::kRow];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = lane & 15, q = lane >> 4;
  const int64_t N = (int64_t)B * Fout, n0 = (int64_t)blockIdx.x * COLS;
  const int K = Cin * kKs;
  // B staging: this thread's column and first input channel; taps outside [0, Fin) read element 0
  // of the row and store zero
  const int col = threadIdx.x % COLS, c0 = threadIdx.x / COLS;
  const int64_t ns = n0 + col < N ? n0 + col : N - 1;
  const int ts = (int)(ns % Fout);
  const float* xcol = x + ((ns / Fout) * Cin + c0) * Fin;
  int src[kKs], dst[kKs];
  bool ok[kKs];
#pragma unroll
  for (int k = 0; k < kKs; ++k) {
    const int f = 2 * ts + k - 2;
    ok[k] = f >= 0 && f < Fin;
    src[k] = ok[k] ? f : 0;
    dst[k] = col * Op::kRow + Op::at(c0 * kKs + k);
  }
  constexpr int kDst = BF16 ? kStep * kKs : kStep * kKs / 4;  // from one staged channel to the next
  f32x4 va[kA];
  float vb[kB][kKs];
  auto load = [&](int ci0) {
#pragma unroll
    for (int e = 0; e < kA; ++e) {
      const int id = threadIdx.x + kBlock * e;
      va[e] = *reinterpret_cast<const f32x4u*>(W + (id / (KC / 4)) * K + ci0 * kKs +
                                               4 * (id % (KC / 4)));
    }
#pragma unroll
    for (int j = 0; j < kB; ++j)
#pragma unroll
      for (int k = 0; k < kKs; ++k) vb[j][k] = xcol[(int64_t)(ci0 + kStep * j) * Fin + src[k]];
  };
  f32x4 acc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[j][e] = BF16 ? 0.f : bias[16 * wave + 4 * q + e];
  load(0);
  for (int ci0 = 0; ci0 < Cin; ci0 += CI) {
    __syncthreads();  // the previous chunk's operands have been read
#pragma unroll
    for (int e = 0; e < kA; ++e) {
      const int id = threadIdx.x + kBlock * e;
      typename Op::T* row = As + (id / (KC / 4)) * Op::kRow;
#pragma unroll
      for (int k = 0; k < 4; ++k) row[Op::at(4 * (id % (KC / 4)) + k)] = Op::put(va[e][k]);
    }
#pragma unroll
    for (int j = 0; j < kB; ++j)
#pragma unroll
      for (int k = 0; k < kKs; ++k) Bs[dst[k] + j * kDst] = Op::put(ok[k] ? vb[j][k] : 0.f);
    __syncthreads();
    if (ci0 + CI < Cin) load(ci0 + CI);
    mma_chunk<BF16, KC, NT>(As + 16 * wave * Op::kRow, Bs, acc, i, q);
  }
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int64_t n = n0 + 16 * j + i;
    if (n >= N) continue;
    float* yc = y + ((n / Fout) * kCh + 16 * wave + 4 * q) * Fout + n % Fout;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      yc[(int64_t)e * Fout] =
          fmaxf(BF16 ? acc[j][e] + bias[16 * wave + 4 * q + e] : acc[j][e], 0.f);
  }
}

// ---- per-sample kernels ------------------------------------------------------------------------

constexpr int kTailF = 128;          // largest layer input, in frames, that a per-sample block takes
constexpr int kK = kCh * kKs;        // 320 entries per row of a 64-channel layer's weights
constexpr int kWRow = kK + 4;
constexpr int kWStage = kCh * kK / 4 / kBlock;  // 4-float groups of W per thread

struct TailLayers {
  int first;                // first layer of the per-sample part (7: none)
  int F[kLayers + 1];
  const float* W[kLayers + 2];
  const float* b[kLayers + 2];
  float* y[kLayers + 1];
  float* dy[kLayers + 1];
};

// Loads of a 64-channel layer's weights, in the order in which the threads store them to LDS.
__device__ __forceinline__ void load_w(const float* W, f32x4 (&w)[kWStage]) {
#pragma unroll
  for (int e = 0; e < kWStage; ++e)
    w[e] = reinterpret_cast<const f32x4u*>(W)[threadIdx.x + kBlock * e];
}

// Layers first .. 6, mean over frames, linear head and sigmoid of one sample per block. A layer's
// input sits in LDS with two zero columns on either side (rows of kTailF + 5 floats), its weights
// are staged as above while the next layer's are already being loaded; wave w computes channels
// 16 w .. 16 w + 15, 16 frames at a time. Few frames a layer (32 .. 2 for 125 frames in), so the
// time is the staging of 82 KB of weights a layer and the chain of 80 dependent matrix
// instructions: 30 us for five layers, pooling and head of 256 samples, 38 us for 4 samples in
// bfloat16 (135 us as six launches).
template <bool BF16>
__global__ __launch_bounds__(kBlock) void tail_fwd_kernel(TailLayers L, float* h, float* out) {
  using Op = Operand<BF16, kK>;
  constexpr int R = kTailF + 5;
  __shared__ __align__(16) typename Op::T Ws[kCh * Op::kRow];
  __shared__ float xs[kCh * R], ys[kCh * (kTailF / 2 + 5)];
  __shared__ float hs[kCh];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = lane & 15, q = lane >> 4;
  const int64_t smp = blockIdx.x;
  f32x4 w[kWStage];
  float* in = xs;
  float* next = ys;
  int rin = R, rout = kTailF / 2 + 5;  // row lengths of `in` and `next`
  if (L.first <= kLayers) {
    load_w(L.W[L.first], w);
    const int F = L.F[L.first - 1];
    const float* src = L.y[L.first - 1] + smp * kCh * F;
    for (int c = wave; c < kCh; c += kBlock / 64)
      for (int f = lane; f < F + 5; f += 64)
        in[c * rin + f] = f >= 2 && f < F + 2 ? src[c * F + f - 2] : 0.f;
  }
  for (int l = L.first; l <= kLayers; ++l) {
    const int Fout = L.F[l];
#pragma unroll
    for (int e = 0; e < kWStage; ++e) {
      const int id = threadIdx.x + kBlock * e;
      typename Op::T* row = Ws + (id / (kK / 4)) * Op::kRow;
#pragma unroll
      for (int k = 0; k < 4; ++k) row[Op::at(4 * (id % (kK / 4)) + k)] = Op::put(w[e][k]);
    }
    __syncthreads();
    if (l < kLayers) load_w(L.W[l + 1], w);
    const typename Op::T* a = Ws + (16 * wave + i) * Op::kRow;
    const float* bias = L.b[l] + 16 * wave + 4 * q;
    float* yg = L.y[l] + (smp * kCh + 16 * wave + 4 * q) * Fout;
    // entry k of a column reads channel k / 5, tap k % 5: the pattern repeats every 4 channels
    // (float32, five steps) or 16 channels (bfloat16, five steps of 16 entries)
    for (int t0 = 0; t0 < Fout; t0 += 16) {
      const int t = t0 + i;
      const float* xc = in + 2 * (t < Fout ? t : Fout - 1);
      f32x4 acc;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = BF16 ? 0.f : bias[e];
      if constexpr (BF16) {
        for (int c = 0; c < kCh; c += 16)
#pragma unroll
          for (int s = 0; s < 5; ++s) {
            bf16x4 bv;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int k = 16 * s + 4 * q + e;
              bv[e] = to_bf16(xc[(c + k / kKs) * rin + k % kKs]);
            }
            const bf16x4 av = *reinterpret_cast<const bf16x4*>(a + c * kKs + 16 * s + 4 * q);
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bv, acc, 0, 0, 0);
          }
      } else {
        int off[5];
#pragma unroll
        for (int s = 0; s < 5; ++s) off[s] = (4 * s + q) / kKs * rin + (4 * s + q) % kKs;
#pragma unroll 1
        for (int c = 0; c < kCh; c += 16) {  // 16 channels: 20 steps
          const f32x4* ap = reinterpret_cast<const f32x4*>(a + q * (kK / 4) + c * kKs / 4);
          const float* xq = xc + c * rin;
          float bv[20];
#pragma unroll
          for (int s = 0; s < 20; ++s) bv[s] = xq[s / 5 * 4 * rin + off[s % 5]];
#pragma unroll
          for (int s = 0; s < 20; s += 4) {
            const f32x4 av = ap[s / 4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], bv[s + e], acc, 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = fmaxf(BF16 ? acc[e] + bias[e] : acc[e], 0.f);
        if (t < Fout) {
          yg[(int64_t)e * Fout + t] = v;
          next[(16 * wave + 4 * q + e) * rout + 2 + t] = v;
        }
      }
    }
    for (int c = threadIdx.x; c < kCh; c += kBlock) {  // the next input's zero columns
      next[c * rout] = next[c * rout + 1] = 0.f;
      for (int f = Fout + 2; f < Fout + 5; ++f) next[c * rout + f] = 0.f;
    }
    __syncthreads();
    float* const p = in;
    in = next;
    next = p;
    const int r = rin;
    rin = rout;
    rout = r;
  }
  const int F6 = L.F[kLayers], c = threadIdx.x;
  if (c < kCh) {
    float acc = 0.f;
    if (L.first <= kLayers)
      for (int t = 0; t < F6; ++t) acc += in[c * rin + 2 + t];
    else
      for (int t = 0; t < F6; ++t) acc += L.y[kLayers][(smp * kCh + c) * F6 + t];
    acc /= (float)F6;
    hs[c] = acc;
    h[smp * kCh + c] = acc;
  }
  __syncthreads();
  if (c < kOut) {
    float z = L.b[kLayers + 1][c];
    for (int k = 0; k < kCh; ++k) z = fmaf(L.W[kLayers + 1][c * kCh + k], hs[k], z);
    out[smp * kOut + c] = 1.f / (1.f + expf(-z));
  }
}

// Input gradient of a 64-channel layer over frames 2 s, 2 s + 1 (s in [s0, s0 + n)) from the
// masked output gradient in LDS: gs row co holds g[co][t] at column t - s0 + 1 (columns
// 0 .. n + 1, zero outside [0, Fout)). dx[ci][f] = sum_{co,k: f = 2t + k - 2} W[co][ci][k] g[co][t]:
// taps 0, 2, 4 (t = s + 1, s, s - 1) for even f, taps 1, 3 (t = s + 1, s) for odd f; both chains
// run over (co, tap) in ascending order. Ws: weights in their natural order, rows of kWRow.
// put(ci, f, value) receives every frame f < Fin.
template <typename Put>
__device__ __forceinline__ void bwd_data(const float* Ws, const float* gs, int grow, int s0, int n,
                                         int Fin, Put&& put) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = lane & 15, q = lane >> 4;
  const float* wc = Ws + (16 * wave + i) * kKs;
  int ea[3], eb[3];  // even f: entries 4 s + q = (co, tap / 2) repeat every 4 channels (3 steps)
  int oa[2], ob[2];  // odd f: every 2 channels (1 step); two steps listed
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int k = 4 * s + q;
    ea[s] = k / 3 * kWRow + 2 * (k % 3);
    eb[s] = k / 3 * grow + 2 - k % 3;
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int k = 4 * s + q;
    oa[s] = k / 2 * kWRow + 2 * (k % 2) + 1;
    ob[s] = k / 2 * grow + 2 - k % 2;
  }
  for (int t0 = 0; t0 < n; t0 += 16) {
    const int t = t0 + i;
    const float* gc = gs + (t < n ? t : n - 1);
    f32x4 ev = {0.f, 0.f, 0.f, 0.f}, od = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int c = 0; c < kCh; c += 4) {
      float a0[3], b0[3], a1[2], b1[2];
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        a0[s] = wc[c * kWRow + ea[s]];
        b0[s] = gc[c * grow + eb[s]];
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        a1[s] = wc[c * kWRow + oa[s]];
        b1[s] = gc[c * grow + ob[s]];
      }
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        ev = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[s], b0[s], ev, 0, 0, 0);
        if (s < 2) od = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[s], b1[s], od, 0, 0, 0);
      }
    }
    if (t < n)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int f = 2 * (s0 + t);
        put(16 * wave + 4 * q + e, f, ev[e]);
        if (f + 1 < Fin) put(16 * wave + 4 * q + e, f + 1, od[e]);
      }
  }
}

__device__ __forceinline__ void store_w(float* Ws, const f32x4 (&w)[kWStage]) {
#pragma unroll
  for (int e = 0; e < kWStage; ++e) {
    const int id = threadIdx.x + kBlock * e;
    *reinterpret_cast<f32x4*>(Ws + (id / (kK / 4)) * kWRow + 4 * (id % (kK / 4))) = w[e];
  }
}

// Loss terms, the head's backward and the input gradients of layers 6 .. first of one sample:
// dz = 2 (s - y) s (1 - s) / (B 11), dh = Wh^T dz, dy6[c][t] = dh[c] / F6. What is written to
// dy[l] is the masked gradient g = dy where y > 0, which is all that the layers below read, with the
// channel as the fastest index ([B][F_l][64]), as the weight gradients read it. 32 us
// for 256 samples x 125 frames (530 us as one launch a layer with one thread per output).
__global__ __launch_bounds__(kBlock) void tail_bwd_kernel(int B, TailLayers L, const float* out,
                                                          const float* labels, float* dz,
                                                          float* lossp) {
  constexpr int R = kTailF / 2 + 2;  // no layer output here is longer than kTailF / 2
  __shared__ __align__(16) float Ws[kCh * kWRow];
  __shared__ float ga[kCh * R], gb[kCh * R];
  __shared__ float dzs[kOut], sq[kOut];
  const int64_t smp = blockIdx.x;
  const int c = threadIdx.x;
  f32x4 w[kWStage];
  if (L.first <= kLayers) load_w(L.W[kLayers], w);
  if (c < kOut) {
    const float sv = out[smp * kOut + c], d = sv - labels[smp * kOut + c];
    const float g = 2.f * d / (float)(B * kOut) * sv * (1.f - sv);
    dzs[c] = g;
    sq[c] = d * d;
    dz[smp * kOut + c] = g;
  }
  __syncthreads();
  const int F6 = L.F[kLayers];
  float *g = ga, *gn = gb;
  if (c < kCh) {
    float dh = 0.f;
    for (int o = 0; o < kOut; ++o) dh = fmaf(L.W[kLayers + 1][o * kCh + c], dzs[o], dh);
    const int64_t row = (smp * kCh + c) * F6;
    for (int t = 0; t < F6; ++t) {
      const float v = L.y[kLayers][row + t] > 0.f ? dh / (float)F6 : 0.f;
      L.dy[kLayers][(smp * F6 + t) * kCh + c] = v;
      if (L.first <= kLayers) g[c * R + 1 + t] = v;
    }
    if (L.first <= kLayers) g[c * R] = g[c * R + 1 + F6] = 0.f;
  }
  if (c == 0) {
    float a = 0.f;
    for (int o = 0; o < kOut; ++o) a += sq[o];
    lossp[smp] = a;
  }
  for (int l = kLayers; l >= L.first; --l) {
    store_w(Ws, w);
    __syncthreads();
    if (l > L.first) load_w(L.W[l - 1], w);
    const int Fin = L.F[l - 1];
    const float* y = L.y[l - 1] + smp * kCh * Fin;
    float* dy = L.dy[l - 1] + smp * kCh * Fin;
    bwd_data(Ws, g, R, 0, L.F[l], Fin, [&](int ci, int f, float v) {
      v = y[ci * Fin + f] > 0.f ? v : 0.f;
      dy[f * kCh + ci] = v;
      if (l > L.first) gn[ci * R + 1 + f] = v;
    });
    if (l > L.first)
      for (int k = threadIdx.x; k < kCh; k += kBlock) gn[k * R] = gn[k * R + 1 + Fin] = 0.f;
    __syncthreads();
    float* const p = g;
    g = gn;
    gn = p;
  }
}

// The same input gradient of one layer with more frames than a per-sample block holds: a block
// takes 64 output frames of one sample.
__global__ __launch_bounds__(kBlock) void conv_bwd_data_kernel(int Fin, int Fout, const float* W,
                                                               const float* g, const float* y,
                                                               float* dy) {
  constexpr int S = 64, R = S + 2;
  __shared__ __align__(16) float Ws[kCh * kWRow];
  __shared__ float gs[kCh * R];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int s0 = blockIdx.x * S, n = min(S, Fout - s0);
  const int64_t smp = blockIdx.y;
  f32x4 w[kWStage];
  load_w(W, w);
  const float* gr = g + smp * kCh * Fout;
  for (int k = wave; k < n + 2; k += kBlock / 64) {
    const int t = s0 + k - 1;
    gs[lane * R + k] = t >= 0 && t < Fout ? gr[(int64_t)t * kCh + lane] : 0.f;
  }
  store_w(Ws, w);
  __syncthreads();
  const float* yr = y + smp * kCh * Fin;
  float* dr = dy + smp * kCh * Fin;
  bwd_data(Ws, gs, R, s0, n, Fin, [&](int ci, int f, float v) {
    dr[(int64_t)f * kCh + ci] = yr[(int64_t)ci * Fin + f] > 0.f ? v : 0.f;
  });
}

// ---- weight gradients --------------------------------------------------------------------------

struct GradLayer {
  const float* x;  // layer input [B][Cin][Fin]
  const float* g;  // masked output gradient [B][Fout][64]
  float* dw;       // weight gradient, followed by the bias gradient
  int Cin, Fin, Fout, blocks;
};
struct GradLayers {
  GradLayer l[kLayers];
};

// Descriptor of n floats from p (wave-uniform), of 2^32 bytes at most; loads past it return 0.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const float* p, int64_t n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0,
                                           (int)(unsigned)min(4 * n, (int64_t)0xFFFFFFF0), 0x00020000);
}

constexpr int kGradWaves = 16, kGradBlock = 64 * kGradWaves;
constexpr int kGradFrames = 16;                    // frames of a unit
constexpr int kGradCols = 2 * kGradFrames + 3;     // input frames of a unit
constexpr int kGradStage = (4 * kGradCols + 63) / 64;
constexpr int kGradRow = 80;  // 4 rows' 11 columns read at a time lie on distinct banks

// dW[co][ci][k] = sum_{b,t} g[b][co][t] x[b][ci][2t + k - 2]: M = co, N = (ci, k), K = (b, t). A
// block owns 32 x 16 weights and all of K, dealt to its 16 waves and summed in double through LDS,
// so no partial sums go to memory and the weights come out of one launch. Consecutive blocks are
// the two halves of co: with blocks dealt to the XCDs in turn, an XCD's L2 holds one half of g.
// A wave's unit is 16 frames of a sample. Lane (i, q) of a matrix instruction holds frame q of four and
// two output channels, g's fastest index, so that a load of g is four whole lines; the 16 columns
// are four rows of x at most, which go through the wave's own piece of LDS (read by lanes, their 16
// columns cost an L1 access per row and instruction: 87 us). A chain of 64 terms is added to double
// sums before the next, which keeps the error of a long float32 chain out. The matrix instructions
// are the bound to work towards (27 us on the 160 blocks of the first layer at 256 samples x 125
// frames). 71 us there for all layers, the head and the loss; units of 32 frames 84 us; blocks of 64
// x 64 channels with the batch split 64 ways and a launch that sums the parts 80 us, with 47 MB of
// scratch.
// The last blocks sum the head's gradients (one output row each) and the loss over the batch.
__global__ __launch_bounds__(kGradBlock) void weight_grad_kernel(GradLayers P, int B,
                                                                const float* dz, const float* h,
                                                                const float* lossp, float* dWh,
                                                                float* dbh, float* loss) {
  __shared__ double red[kGradWaves][8][64];
  __shared__ float xs[kGradWaves][4 * kGradRow];  // each wave's own
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int blk = blockIdx.x, li = 0;
  while (li < kLayers && blk >= P.l[li].blocks) blk -= P.l[li++].blocks;
  if (li == kLayers) {  // wave r sums samples r, r + 16, ...
    double a = 0.0, ab = 0.0;
    if (blk < kOut) {
#pragma unroll 4
      for (int b = wave; b < B; b += kGradWaves) {
        const double d = dz[(int64_t)b * kOut + blk];
        a += d * (double)h[(int64_t)b * kCh + lane];
        ab += d;
      }
    } else {
      for (int b = threadIdx.x; b < B; b += kGradBlock) a += (double)lossp[b];
    }
    red[wave][0][lane] = a;
    red[wave][1][lane] = ab;
    __syncthreads();
    if (wave != 0) return;
    a = ab = 0.0;
    for (int r = 0; r < kGradWaves; ++r) {
      a += red[r][0][lane];
      ab += red[r][1][lane];
    }
    if (blk < kOut) {
      dWh[blk * kCh + lane] = (float)a;
      if (lane == 0) dbh[blk] = (float)ab;
    } else {
      for (int d = 32; d > 0; d >>= 1) a += __shfl_xor(a, d);
      if (lane == 0 && loss) *loss = (float)(a / (double)(B * kOut));
    }
    return;
  }
  const GradLayer& L = P.l[li];
  const int i = lane & 15, q = lane >> 4;
  const int co = (blk & 1) * 32, col = (blk >> 1) * 16 + i;  // this lane's column (ci, k)
  const int ci = col / kKs, k = col - ci * kKs;
  const int Fin = L.Fin, Fout = L.Fout;
  const int tiles = (Fout + kGradFrames - 1) / kGradFrames;
  const int w = __builtin_amdgcn_readfirstlane(wave);
  const int64_t units = (int64_t)B * tiles, u0 = units * w / kGradWaves;
  const int n = (int)(units * (w + 1) / kGradWaves - u0);
  int b = (int)(u0 / tiles), t0 = (int)(u0 - (int64_t)b * tiles) * kGradFrames;
  const int c0 = (blk >> 1) * 16 / kKs;  // first channel of the columns
  struct Unit {
    f32x2 a[kGradFrames / 4];
    float x[kGradStage];
    int nt;  // frames
  };
  auto load = [&](Unit& U) {
    const auto rx = buffer_at(L.x + ((int64_t)b * L.Cin + c0) * Fin, (int64_t)(L.Cin - c0) * Fin);
    const auto rg = buffer_at(L.g + ((int64_t)b * Fout + t0) * kCh, (int64_t)(Fout - t0) * kCh);
    U.nt = Fout - t0;
#pragma unroll
    for (int m = 0; m < kGradStage; ++m) {
      const int e = lane + 64 * m, r = e / kGradCols, f = 2 * t0 - 2 + e - r * kGradCols;
      const unsigned off = (unsigned)f < (unsigned)Fin ? (unsigned)(r * Fin + f) * 4u : ~0u;
      U.x[m] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, off, 0, 0));
    }
#pragma unroll
    for (int j = 0; j < kGradFrames / 4; ++j)
      U.a[j] = __builtin_bit_cast(
          f32x2, __builtin_amdgcn_raw_buffer_load_b64(
                     rg, (unsigned)((4 * j + q) * kCh + co + 2 * i) * 4u, 0, 0));
    t0 += kGradFrames;
    if (t0 >= Fout) {
      t0 = 0;
      ++b;
    }
  };
  float* const xw = xs[wave];
  const float* const xq = xw + (ci - c0) * kGradRow + k + 2 * q;
  double tot[2][4] = {};
  double bias[2] = {0.0, 0.0};
  Unit nx;
  if (n > 0) load(nx);
  for (int s = 0; s < n;) {
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    float bs[2] = {0.f, 0.f};
    const int end = min(s + 64 / kGradFrames, n);
    for (; s < end; ++s) {
      const Unit c = nx;
#pragma unroll
      for (int m = 0; m < kGradStage; ++m) {
        const int e = lane + 64 * m, r = e / kGradCols;
        if (e < 4 * kGradCols) xw[r * kGradRow + e - r * kGradCols] = c.x[m];
      }
      lds_order();
      if (s + 1 < n) load(nx);
      float xv[kGradFrames / 4];
#pragma unroll
      for (int j = 0; j < kGradFrames / 4; ++j) xv[j] = xq[8 * j];
      lds_order();  // read before the next unit's stores
      auto multiply = [&](auto whole) {
#pragma unroll
        for (int j = 0; j < kGradFrames / 4; ++j) {
          if (!whole.value && 4 * j >= c.nt) break;
          const float v = whole.value || 4 * j + q < c.nt ? xv[j] : 0.f;
#pragma unroll
          for (int m = 0; m < 2; ++m) {
            acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(c.a[j][m], v, acc[m], 0, 0, 0);
            bs[m] += c.a[j][m];
          }
        }
      };
      if (c.nt >= kGradFrames)
        multiply(std::true_type{});
      else
        multiply(std::false_type{});
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
#pragma unroll
      for (int e = 0; e < 4; ++e) tot[m][e] += (double)acc[m][e];
      bias[m] += (double)bs[m];
    }
  }
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][4 * m + e][lane] = tot[m][e];
  __syncthreads();
  if (wave < 8) {
    double v = 0.0;
    for (int r = 0; r < kGradWaves; ++r) v += red[r][wave][lane];
    L.dw[(int64_t)(co + 2 * (4 * q + (wave & 3)) + (wave >> 2)) * L.Cin * kKs + col] = (float)v;
  }
  if (blk >= 2) return;  // bias: by the blocks of the first columns
  __syncthreads();
  red[wave][0][lane] = bias[0];
  red[wave][1][lane] = bias[1];
  __syncthreads();
  if (threadIdx.x >= 32) return;
  double v = 0.0;
  for (int r = 0; r < kGradWaves; ++r)
    for (int u = 0; u < 4; ++u) v += red[r][threadIdx.x & 1][16 * u + (threadIdx.x >> 1)];
  L.dw[(int64_t)kCh * L.Cin * kKs + co + threadIdx.x] = (float)v;
}

__global__ __launch_bounds__(kBlock) void adam_kernel(int64_t n, float* p, const float* g,
                                                      float* m, float* v, const float* scale,
                                                      float lr, float b1, float b2, float c1,
                                                      float c2, float eps) {
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kBlock) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= (scale ? lr * scale[i] : lr) * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

// x[b] = [dry_feats[dry[b]]; mix_feats[mix[b]]] ([256][F]); labels[b] = label_table[dry[b]].
__global__ __launch_bounds__(kBlock) void gather_kernel(int B, int F, const float* dry_feats,
                                                        const int32_t* dry,
                                                        const float* mix_feats,
                                                        const int32_t* mix,
                                                        const float* label_table, float* labels,
                                                        float* x) {
  const int64_t n = (int64_t)B * kCin * F;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kBlock) {
    const int f = (int)(i % F), c = (int)((i / F) % kCin), b = (int)(i / F / kCin);
    const bool is_dry = c < kCin / 2;
    const float* table = is_dry ? dry_feats : mix_feats;
    const int src = is_dry ? dry[b] : mix[b];
    x[i] = table[((int64_t)src * (kCin / 2) + (c % (kCin / 2))) * F + f];
  }
  if (label_table)
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < (int64_t)B * kOut;
         i += (int64_t)gridDim.x * kBlock)
      labels[i] = label_table[(int64_t)dry[i / kOut] * kOut + i % kOut];
}

// Normalised outputs -> the chain's parameter rows: gain/pan dB [-12, 6] per channel, six EQ
// band gains [-12, 12] dB spread over 1024 log-magnitudes (linear in log-frequency between band
// centres 20 * 1000^((b + 0.5) / 6) Hz, bin k at k fs / 2047 Hz, constant beyond the outer
// centres), compressor time constant [1, 100] ms, threshold [-30, -10] dB, ratio [2, 8], knee
// 3 dB.
__global__ __launch_bounds__(kBlock) void params_kernel(const float* s, float* gp, float* eq,
                                                        float* comp) {
  const int b = blockIdx.x;
  const float* sb = s + (int64_t)b * kOut;
  const float ln10_20 = 0.11512925464970229f, ln10_10 = 0.23025850929940458f;
  __shared__ float band[6], lc[6];
  if (threadIdx.x < 6) {
    band[threadIdx.x] = -12.f + 24.f * sb[2 + threadIdx.x];
    lc[threadIdx.x] = logf(20.f) + logf(1000.f) * ((float)threadIdx.x + 0.5f) / 6.f;
  }
  if (threadIdx.x < 2) gp[(int64_t)b * 2 + threadIdx.x] = (-12.f + 18.f * sb[threadIdx.x]) * ln10_20;
  if (threadIdx.x == 0) {
    const float tau = 1.f + 99.f * sb[8];
    comp[(int64_t)b * 4 + 0] = expf(-1.f / (tau * 1e-3f * 44100.f));
    comp[(int64_t)b * 4 + 1] = (-30.f + 20.f * sb[9]) * ln10_10;
    comp[(int64_t)b * 4 + 2] = 3.f * ln10_10;
    comp[(int64_t)b * 4 + 3] = 2.f + 6.f * sb[10];
  }
  __syncthreads();
  for (int k = threadIdx.x; k < 1024; k += kBlock) {
    const float lf = logf(fmaxf((float)k * 44100.f / 2047.f, 1e-3f));
    float gdb;
    if (lf <= lc[0]) {
      gdb = band[0];
    } else if (lf >= lc[5]) {
      gdb = band[5];
    } else {
      int i = 0;
      while (lf >= lc[i + 1]) ++i;
      gdb = band[i] + (band[i + 1] - band[i]) * (lf - lc[i]) / (lc[i + 1] - lc[i]);
    }
    eq[(int64_t)b * 1024 + k] = gdb * ln10_20;
  }
}

unsigned grid_for(int64_t n) {
  const int64_t g = (n + kBlock - 1) / kBlock;
  return (unsigned)(g < 65536 ? (g > 0 ? g : 1) : 65536);
}

// The per-sample kernels take the layers from the first whose input fits their LDS; the first
// layer always runs in the tiled kernel.
TailLayers tail_layers(const EncLayout& L, const float* weights, float* acts, float* grads) {
  TailLayers t{};
  t.first = 2;
  while (t.first <= kLayers && L.F[t.first - 1] > kTailF) ++t.first;
  for (int l = 0; l <= kLayers; ++l) t.F[l] = L.F[l];
  for (int l = 1; l <= kLayers + 1; ++l) {
    t.W[l] = weights + L.w[l];
    t.b[l] = weights + L.b[l];
  }
  for (int l = 1; l <= kLayers; ++l) {
    t.y[l] = acts + L.y[l];
    t.dy[l] = grads ? grads + L.dy[l] : nullptr;
  }
  return t;
}

// 64-column tiles where they give enough blocks, 16-column tiles below (same bits). Forward of frames of
// 125, by blocks of 64 columns, us with 64 and with 16 columns: float32 99: 67.7 and 59.0, 148: 70.0 and
// 72.0, 178: 69.9 and 72.7, 200: 70.2 and 84.9; bfloat16 148: 71.4 and 68.3, 178: 71.8 and 67.9, 200:
// 71.4 and 74.2.
template <bool BF16>
void launch_conv_fwd(int B, int Cin, int Fin, int Fout, const float* x, const float* W,
                     const float* bias, float* y, hipStream_t s) {
  const int64_t n = (int64_t)B * Fout;
  if (n >= (BF16 ? 190 : 140) * 64)
    conv_fwd_kernel<BF16, 4, 16><<<(unsigned)((n + 63) / 64), kBlock, 0, s>>>(B, Cin, Fin, Fout, x,
                                                                             W, bias, y);
  else
    conv_fwd_kernel<BF16, 1, 64><<<(unsigned)((n + 15) / 16), kBlock, 0, s>>>(B, Cin, Fin, Fout, x,
                                                                             W, bias, y);
}

grafx_status hip_st(hipError_t e, const char* what) {
  if (e == hipSuccess) return GRAFX_OK;
  return fail(GRAFX_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

grafx_status check_dims(int32_t batch, int32_t frames) {
  if (batch < 1 || batch > (1 << 20)) return fail(GRAFX_E_SHAPE, "batch must be in [1, 2^20]");
  if (frames < 1 || frames > (1 << 20)) return fail(GRAFX_E_SHAPE, "frames must be in [1, 2^20]");
  return GRAFX_OK;
}

}  // namespace
}  // namespace grafx

using namespace grafx;

extern "C" {

grafx_status grafx_encoder_sizes(int32_t batch, int32_t frames, size_t* n_weights,
                                 size_t* act_floats, size_t* grad_floats) {
  clear_error();
  grafx_status st = check_dims(batch, frames);
  if (st != GRAFX_OK) return st;
  const EncLayout L = enc_layout(batch, frames);
  if (n_weights) *n_weights = L.n_w;
  if (act_floats) *act_floats = L.act;
  if (grad_floats) *grad_floats = L.grad;
  return GRAFX_OK;
}

grafx_status grafx_logmel(int32_t n_signals, int64_t T, const float* signals, float* features,
                          hipStream_t stream) {
  clear_error();
  if (n_signals < 1) return fail(GRAFX_E_SHAPE, "n_signals must be >= 1");
  if (T < 1024 || T >= ((int64_t)1 << 29)) return fail(GRAFX_E_SHAPE, "T must be in [1024, 2^29)");
  if (!signals || !features) return fail(GRAFX_E_ARG, "NULL argument");
  return hip_st(launch_logmel(n_signals, T, signals, features, stream), "logmel launch");
}

grafx_status grafx_encoder_gather(int32_t batch, int32_t frames, const float* dry_features,
                                  const int32_t* dry, const float* mix_features,
                                  const int32_t* mix, const float* label_table, float* labels,
                                  float* x, hipStream_t stream) {
  clear_error();
  grafx_status st = check_dims(batch, frames);
  if (st != GRAFX_OK) return st;
  if (!dry_features || !dry || !mix_features || !mix || !x || (label_table && !labels))
    return fail(GRAFX_E_ARG, "NULL argument");
  const int64_t n = (int64_t)batch * kCin * frames;
  gather_kernel<<<grid_for(n), kBlock, 0, stream>>>(batch, frames, dry_features, dry,
                                                    mix_features, mix, label_table, labels, x);
  return hip_st(hipGetLastError(), "encoder_gather launch");
}

grafx_status grafx_encoder_forward(int32_t batch, int32_t frames, const float* x,
                                   const float* weights, int32_t bf16, float* acts, float* out,
                                   hipStream_t stream) {
  clear_error();
  grafx_status st = check_dims(batch, frames);
  if (st != GRAFX_OK) return st;
  if (!x || !weights || !acts || !out) return fail(GRAFX_E_ARG, "NULL argument");
  if (bf16 && (int64_t)batch * kCin * frames >= ((int64_t)1 << 29))
    return fail(GRAFX_E_SHAPE, "bf16 forward: batch x 256 x frames must be below 2^29");
  const EncLayout L = enc_layout(batch, frames);
  TailLayers t = tail_layers(L, weights, acts, nullptr);
  const float* in = x;
  for (int l = 1; l < t.first; ++l) {
    float* y = acts + L.y[l];
    if (bf16)
      launch_conv_fwd<true>(batch, cin_of(l), L.F[l - 1], L.F[l], in, t.W[l], t.b[l], y, stream);
    else
      launch_conv_fwd<false>(batch, cin_of(l), L.F[l - 1], L.F[l], in, t.W[l], t.b[l], y, stream);
    in = y;
  }
  if (bf16)
    tail_fwd_kernel<true><<<batch, kBlock, 0, stream>>>(t, acts + L.h, out);
  else
    tail_fwd_kernel<false><<<batch, kBlock, 0, stream>>>(t, acts + L.h, out);
  return hip_st(hipGetLastError(), "encoder_forward launch");
}

grafx_status grafx_encoder_backward(int32_t batch, int32_t frames, const float* x,
                                    const float* weights, const float* acts, const float* out,
                                    const float* labels, float* loss, float* dweights,
                                    float* grads, hipStream_t stream) {
  clear_error();
  grafx_status st = check_dims(batch, frames);
  if (st != GRAFX_OK) return st;
  if (!x || !weights || !acts || !out || !labels || !dweights || !grads)
    return fail(GRAFX_E_ARG, "NULL argument");
  const EncLayout L = enc_layout(batch, frames);
  const TailLayers t = tail_layers(L, weights, const_cast<float*>(acts), grads);
  tail_bwd_kernel<<<batch, kBlock, 0, stream>>>(batch, t, out, labels, grads + L.dz,
                                                grads + L.lossp);
  for (int l = t.first - 1; l >= 2; --l)
    for (int b0 = 0; b0 < batch; b0 += 65535) {  // samples on the grid's second dimension
      const int64_t in = (int64_t)b0 * kCh * L.F[l - 1], o = (int64_t)b0 * kCh * L.F[l];
      conv_bwd_data_kernel<<<dim3((L.F[l] + 63) / 64, std::min(batch - b0, 65535)), kBlock, 0,
                             stream>>>(L.F[l - 1], L.F[l], t.W[l], t.dy[l] + o, t.y[l - 1] + in,
                                       t.dy[l - 1] + in);
    }
  GradLayers P;
  int blocks = 0;
  for (int l = 1; l <= kLayers; ++l) {
    GradLayer& G = P.l[l - 1];
    G.x = l == 1 ? x : t.y[l - 1];
    G.g = t.dy[l];
    G.dw = dweights + L.w[l];
    G.Cin = cin_of(l);
    G.Fin = L.F[l - 1];
    G.Fout = L.F[l];
    G.blocks = 2 * (G.Cin * kKs / 16);
    blocks += G.blocks;
  }
  weight_grad_kernel<<<blocks + kOut + 1, kGradBlock, 0, stream>>>(
      P, batch, grads + L.dz, acts + L.h, grads + L.lossp, dweights + L.w[kLayers + 1],
      dweights + L.b[kLayers + 1], loss);
  return hip_st(hipGetLastError(), "encoder_backward launch");
}

grafx_status grafx_adam(int64_t n, float* p, const float* g, float* m, float* v,
                        const float* lr_scale, int32_t step, float lr, float beta1, float beta2,
                        float eps, hipStream_t stream) {
  clear_error();
  if (n < 0 || step < 1) return fail(GRAFX_E_ARG, "n must be >= 0 and step >= 1");
  if (n == 0) return GRAFX_OK;
  if (!p || !g || !m || !v) return fail(GRAFX_E_ARG, "NULL argument");
  const float c1 = (float)(1.0 - std::pow((double)beta1, step));
  const float c2 = (float)(1.0 - std::pow((double)beta2, step));
  adam_kernel<<<grid_for(n), kBlock, 0, stream>>>(n, p, g, m, v, lr_scale, lr, beta1, beta2, c1,
                                                  c2, eps);
  return hip_st(hipGetLastError(), "adam launch");
}

grafx_status grafx_encoder_params(int32_t batch, const float* out, float* gain_pan, float* eq,
                                  float* comp, hipStream_t stream) {
  clear_error();
  if (batch < 1) return fail(GRAFX_E_SHAPE, "batch must be >= 1");
  if (!out || !gain_pan || !eq || !comp) return fail(GRAFX_E_ARG, "NULL argument");
  params_kernel<<<batch, kBlock, 0, stream>>>(out, gain_pan, eq, comp);
  return hip_st(hipGetLastError(), "encoder_params launch");
}

}  // extern "C"

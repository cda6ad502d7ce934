// Filtered-noise mid/side reverb (paper Sec. 3 "Reverb", Eqs. 6-7) and its adjoint.
//
// Impulse response (once per render, every reverb node): a fixed noise realisation, one signal
// for mid and one for side, is analysed by an STFT (384-point frames, hop 192, periodic Hann
// window; frame m covers samples [192 m - 192, 192 m + 192), zero outside the noise); its bins are
// scaled by the mask exp(H0[k] + m HD[k]) (Eq. 7, frames counted from 0; the Nyquist bin takes
// bin 191's mask); every frame goes back through a real inverse DFT, and the frames are
// overlap-added without a synthesis window (the periodic Hann window sums to one at half
// overlap). Mid/side become left/right as in the imager: h_l = (h_m + h_s) / 2,
// h_r = (h_m - h_s) / 2. All of this is in double, on a 384-point transform of one wave (mid + i side
// in one complex signal): a hop of h is one inverse transform of the two masked frames that overlap
// there, combined in the frequency domain.
//
// Filtering: y_c[t] = sum_n h_c[n] u_c[t - n], a causal FIR as long as the noise (two seconds in
// the paper), as uniformly partitioned overlap-save. The FIR is cut into partitions of 2048 taps,
// each zero-padded to 4096 and transformed once per render; the input is transformed once per
// block of 2048 outputs (the 4096-sample window that ends with the block); the spectrum of output
// block b is the sum over partitions p of the spectrum of input window b - p times that of
// partition p, and the second half of its inverse transform is the block. Both channels ride in
// one complex transform (left + i right) and are separated into one-sided per-channel spectra
// (bins 0..2048) when stored. The sum over partitions runs bin-major (a lane per bin, a run of
// output blocks summed in registers, the input spectra sliding past them), the products go through
// the workspace, and a second kernel rebuilds each block's packed spectrum and transforms it back.
//
// Adjoint: the input adjoint is the correlation ubar_c[s] = sum_n h_c[n] ybar_c[s + n], the same
// partitioned product with the conjugate partition spectra over forward-looking windows
// [2048 b, 2048 b + 4096), keeping the first half. Only the spectra Y0[b] of single adjoint blocks
// (placed in the second half of a window) are transformed: a window that starts at block b is
// block b shifted by half a window plus block b + 1, so its spectrum is
// Y0[b + 1][k] + (-1)^k Y0[b][k]. The FIR gradient hbar_c[n] = sum_t ybar_c[t] u_c[t - n] is, per
// partition p, the inverse transform of sum_b Y0_c[b][k] conj(X_c[b - p][k]) (X: the forward's
// input-window spectra, kept in the workspace), first half. It goes back through mid/side, the
// overlap-add (each frame reads its own slice of hbar), the inverse DFT and the mask to dH0 and
// dHD, with partials per group of frames summed in a fixed order.
#include "device_common.h"
#include "fft4096.h"
#include "grafx_internal.h"
#include "kernels.h"

namespace grafx {
namespace {

using namespace fft4;

constexpr int kF = kRvFft;      // 384
constexpr int kHop = kRvHop;    // 192
constexpr int kK = kF / 2 + 1;  // 193 one-sided STFT bins
constexpr int kB = kRvBlock;    // 2048
constexpr int kHalfBins = 9;    // bins k = j + 256 r (r < 9, k <= 2048) of thread j

// ---- 384-point transform in double, one wave ----------------------------------------------------
// 384 = 6 x 8 x 8 (Stockham): pass 0 takes 64 lanes x 6 points, passes 1 and 2 take 48 lanes x 8
// points; the exchanges go through the wave's own LDS slice, whose accesses are executed in order.

constexpr int kWaves = kBlock / 64;

// exp(+2 pi i j / 384) in double, j = 0..383.
__device__ __forceinline__ void fill_tw384(double2* tw) {
  for (int j = threadIdx.x; j < kF; j += blockDim.x) {
    double s, c;
    sincospi(2.0 * j / kF, &s, &c);
    tw[j] = make_double2(c, s);
  }
}

__device__ __forceinline__ double2 dadd(double2 a, double2 b) {
  return make_double2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ double2 dsub(double2 a, double2 b) {
  return make_double2(a.x - b.x, a.y - b.y);
}
// a times the table entry w = e^(+i theta): w for the inverse, its conjugate for the forward
template <bool INV>
__device__ __forceinline__ double2 dtw(double2 a, double2 w) {
  return INV ? make_double2(fma(a.x, w.x, -a.y * w.y), fma(a.x, w.y, a.y * w.x))
             : make_double2(fma(a.x, w.x, a.y * w.y), fma(a.y, w.x, -a.x * w.y));
}
template <bool INV>
__device__ __forceinline__ double2 dmul_mi(double2 a) {  // times -i (forward) or +i (inverse)
  return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

template <bool INV>
__device__ __forceinline__ void ddft3(double2& a, double2& b, double2& c) {
  constexpr double h = 0.86602540378443864676;  // sin(pi / 3)
  const double2 s = dadd(b, c), d = dmul_mi<INV>(dsub(b, c));
  const double2 t = make_double2(fma(-0.5, s.x, a.x), fma(-0.5, s.y, a.y));
  a = dadd(a, s);
  b = make_double2(fma(h, d.x, t.x), fma(h, d.y, t.y));
  c = make_double2(fma(-h, d.x, t.x), fma(-h, d.y, t.y));
}

// X[k] = sum_n v[n] e^(-+2 pi i nk / 6), natural order: n = 2 n1 + n2, k = k1 + 3 k2
template <bool INV>
__device__ __forceinline__ void ddft6(double2 (&v)[6]) {
  constexpr double h = 0.86602540378443864676;
  ddft3<INV>(v[0], v[2], v[4]);
  ddft3<INV>(v[1], v[3], v[5]);
  // twiddles e^(-+2 pi i k1 / 6) on the odd part
  v[3] = dtw<INV>(v[3], make_double2(0.5, h));
  v[5] = dtw<INV>(v[5], make_double2(-0.5, h));
  const double2 o[6] = {dadd(v[0], v[1]), dadd(v[2], v[3]), dadd(v[4], v[5]),
                        dsub(v[0], v[1]), dsub(v[2], v[3]), dsub(v[4], v[5])};
#pragma unroll
  for (int i = 0; i < 6; ++i) v[i] = o[i];
}

template <bool INV>
__device__ __forceinline__ void ddft4(double2& a0, double2& a1, double2& a2, double2& a3) {
  const double2 t0 = dadd(a0, a2), t1 = dsub(a0, a2);
  const double2 t2 = dadd(a1, a3), t3 = dmul_mi<INV>(dsub(a1, a3));
  a0 = dadd(t0, t2);
  a2 = dsub(t0, t2);
  a1 = dadd(t1, t3);
  a3 = dsub(t1, t3);
}

template <bool INV>
__device__ __forceinline__ void ddft8(double2 (&v)[8]) {  // as dft8, in double
  constexpr double r2 = 0.70710678118654752440;
  ddft4<INV>(v[0], v[2], v[4], v[6]);
  ddft4<INV>(v[1], v[3], v[5], v[7]);
  v[3] = dtw<INV>(v[3], make_double2(r2, r2));
  v[5] = dmul_mi<INV>(v[5]);
  v[7] = dtw<INV>(v[7], make_double2(-r2, r2));
  const double2 o[8] = {dadd(v[0], v[1]), dadd(v[2], v[3]), dadd(v[4], v[5]), dadd(v[6], v[7]),
                        dsub(v[0], v[1]), dsub(v[2], v[3]), dsub(v[4], v[5]), dsub(v[6], v[7])};
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = o[i];
}

// On entry x[r] holds element j + 64 r (r < 6); on exit v[r] of lane j < 48 holds X[j + 48 r].
// s: the wave's slice of kF entries.
template <bool INV>
__device__ __forceinline__ void fft384(double2 (&x)[6], double2 (&v)[8], double2* s,
                                       const double2* tw, int j) {
  ddft6<INV>(x);
  lds_order();
#pragma unroll
  for (int r = 0; r < 6; ++r) s[6 * j + r] = x[r];
  lds_order();
  const int b = j < 48 ? j : 47;  // idle lanes repeat lane 47's reads
#pragma unroll
  for (int r = 0; r < 8; ++r) v[r] = s[b + 48 * r];
  lds_order();
  const int q = b % 6;
#pragma unroll
  for (int r = 1; r < 8; ++r) v[r] = dtw<INV>(v[r], tw[8 * r * q]);
  ddft8<INV>(v);
  if (j < 48) {
#pragma unroll
    for (int r = 0; r < 8; ++r) s[b / 6 * 48 + q + 6 * r] = v[r];
  }
  lds_order();
#pragma unroll
  for (int r = 0; r < 8; ++r) v[r] = s[b + 48 * r];
  lds_order();
#pragma unroll
  for (int r = 1; r < 8; ++r) v[r] = dtw<INV>(v[r], tw[r * b]);
  ddft8<INV>(v);
}

// Puts the transform's output into the slice, entry k at k.
__device__ __forceinline__ void put384(const double2 (&v)[8], double2* s, int j) {
  if (j < 48) {
#pragma unroll
    for (int r = 0; r < 8; ++r) s[j + 48 * r] = v[r];
  }
  lds_order();
}

__device__ __forceinline__ double hann384(int q) { return 0.5 - 0.5 * cospi(2.0 * q / kF); }

// The mask of Eq. 7 at one-sided bin k of frame m for mid (x = 0) or side (x = 1), and its ratio
// from one frame to the next: runs of frames step the mask by it.
__device__ __forceinline__ double mask_at(const float* p, int x, int k, int m) {
  const int kp = k < kRvBins ? k : kRvBins - 1;  // the Nyquist bin shares bin 191's mask
  return exp((double)p[x * 2 * kRvBins + kp] +
             (double)m * (double)p[x * 2 * kRvBins + kRvBins + kp]);
}
__device__ __forceinline__ double mask_step(const float* p, int x, int k) {
  const int kp = k < kRvBins ? k : kRvBins - 1;
  return exp((double)p[x * 2 * kRvBins + kRvBins + kp]);
}

// After a forward transform of a packed window (left + i right) held as v[r] = W[j + 256 r]:
// store the one-sided per-channel spectra (L[k], R[k]), k = 0..2048, scaled by `scale`, as
// float4 (L re, L im, R re, R im): L = (W[k] + conj W[N - k]) / 2, R = (W[k] - conj W[N - k]) / 2i.
__device__ __forceinline__ void store_separated(const float2 (&v)[16], float2* lds, float4* out,
                                                float scale) {
  const int j = threadIdx.x;
#pragma unroll
  for (int r = 0; r < 16; ++r) lds[pad(j + 256 * r)] = v[r];
  __syncthreads();
  const float h = 0.5f * scale;
#pragma unroll
  for (int r = 0; r < kHalfBins; ++r) {
    const int k = j + 256 * r;
    if (k > kN / 2) break;
    const float2 w = lds[pad(k)], m = lds[pad((kN - k) & (kN - 1))];
    out[k] = make_float4(h * (w.x + m.x), h * (w.y - m.y), h * (w.y + m.y), h * (m.x - w.x));
  }
}

// Inverse of store_separated for a product held per channel at the thread's one-sided bins:
// writes the packed spectrum Y[k] = L[k] + i R[k] and Y[N - k] = conj L[k] + i conj R[k] into
// LDS and reads it back in the transform's layout (v[r] = Y[j + 256 r]).
__device__ __forceinline__ void pack_spectrum(const float2 (&al)[kHalfBins],
                                              const float2 (&ar)[kHalfBins], float2* lds,
                                              float2 (&v)[16]) {
  const int j = threadIdx.x;
#pragma unroll
  for (int r = 0; r < kHalfBins; ++r) {
    const int k = j + 256 * r;
    if (k > kN / 2) break;
    lds[pad(k)] = make_float2(al[r].x - ar[r].y, al[r].y + ar[r].x);
    if (k != 0 && k != kN / 2)
      lds[pad(kN - k)] = make_float2(al[r].x + ar[r].y, ar[r].x - al[r].y);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = lds[pad(j + 256 * r)];
  __syncthreads();  // the transform overwrites the LDS
}

// ---- noise STFT -------------------------------------------------------------------------------
// Un[x][m][k] = sum_q w[q] noise_x[192 m - 192 + q] e^(-2 pi i k q / 384), k = 0..192: one wave per
// frame, mid and side in one transform. 461 frames of 2 s of noise: 11 us, 37 us as
// direct sums.
__global__ __launch_bounds__(kBlock) void rv_noise_stft_kernel(const float* noise, int64_t L,
                                                               int M, double2* Un) {
  __shared__ double2 tw[kF], lds[kWaves][kF];
  fill_tw384(tw);
  __syncthreads();
  const int wave = threadIdx.x >> 6, j = threadIdx.x & 63;
  const int m = blockIdx.x * kWaves + wave;
  if (m >= M) return;  // no block barrier below
  double2* s = lds[wave];
  double2 x[6], v[8];
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    const int q = j + 64 * r;
    const int64_t n = (int64_t)kHop * m - kHop + q;
    const bool in = n >= 0 && n < L;
    const double w = in ? hann384(q) : 0.0;
    x[r] = make_double2(in ? w * (double)noise[n] : 0.0, in ? w * (double)noise[L + n] : 0.0);
  }
  fft384<false>(x, v, s, tw, j);
  put384(v, s, j);
  for (int k = j; k < kK; k += 64) {
    const double2 a = s[k], b = s[k ? kF - k : 0];
    Un[(int64_t)m * kK + k] = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
    Un[((int64_t)M + m) * kK + k] = make_double2(0.5 * (a.y + b.y), 0.5 * (b.x - a.x));
  }
}

// ---- impulse response -------------------------------------------------------------------------
// Sample 192 s + t of h_x (t < 192) is the sum of frame s at q = 192 + t and frame s + 1 at q = t.
// Since e^(2 pi i k (192 + t) / 384) = (-1)^k e^(2 pi i k t / 384), that is one real inverse DFT
// per hop s of the combined spectrum Y_s[k] = (X_{s+1}[k] + (-1)^k X_s[k]) / 384, X_m the masked
// frame spectrum; mid and side ride in one complex inverse transform, whose first 192 outputs are
// the hop. A wave takes kIrHops hops of one reverb slot in a row, so each frame's masked spectrum
// serves two of them and the masks are stepped from frame to frame by multiplication (an exp per
// bin and frame costs more than the transform). Lane j forms the entries q = j + 64 r of the full
// spectrum from bin min(q, 384 - q). 16 slots, 2 s: 17 us, 111 us as direct sums; 2 or 8 hops a wave
// were slower (21 and 22 us).
constexpr int kIrHops = 4;

__global__ __launch_bounds__(kBlock) void rv_ir_kernel(const float* P, const double2* Un,
                                                       int64_t L, int M, float* h) {
  __shared__ double2 tw[kF], lds[kWaves][kF];
  fill_tw384(tw);
  __syncthreads();
  const int wave = threadIdx.x >> 6, j = threadIdx.x & 63;
  const int s0 = (blockIdx.x * kWaves + wave) * kIrHops, slot = blockIdx.y;
  if (s0 >= M - 1) return;  // no block barrier below
  const float* p = P + (int64_t)slot * kRvParams;
  double2* s = lds[wave];
  double mu[2][6], step[2][6];
  double2 prev[2][6];  // masked frame s, times (-1)^k / 384
  auto frame = [&](int m, int r, int x) {
    const int q = j + 64 * r, k = q < kK ? q : kF - q;
    const double2 u = Un[((int64_t)x * M + m) * kK + k];
    const double c = mu[x][r] * (1.0 / kF);
    return make_double2(c * u.x, c * u.y);
  };
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      const int q = j + 64 * r, k = q < kK ? q : kF - q;
      mu[x][r] = mask_at(p, x, k, s0);
      step[x][r] = mask_step(p, x, k);
      prev[x][r] = frame(s0, r, x);
    }
  const bool odd = j & 1;  // parity of q, hence of k
  float* hs = h + (int64_t)slot * 2 * L;
  for (int i = 0; i < kIrHops && s0 + i < M - 1; ++i) {
    double2 z[6], v[8];
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      const bool upper = j + 64 * r >= kK;  // bins above the Nyquist bin are conjugates
      double2 y[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        mu[x][r] *= step[x][r];
        const double2 f = frame(s0 + i + 1, r, x);
        y[x] = odd ? dsub(f, prev[x][r]) : dadd(f, prev[x][r]);
        if (upper) y[x].y = -y[x].y;
        prev[x][r] = f;
      }
      // the DC and Nyquist bins of a real signal's spectrum are taken as real
      const bool real = j == 0 && (r == 0 || r == 3);
      z[r] = make_double2(y[0].x - (real ? 0.0 : y[1].y), (real ? 0.0 : y[0].y) + y[1].x);
    }
    fft384<true>(z, v, s, tw, j);
    if (j < 48)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t n = (int64_t)kHop * (s0 + i) + j + 48 * r;
        if (n < L) {
          hs[n] = (float)(0.5 * (v[r].x + v[r].y));
          hs[L + n] = (float)(0.5 * (v[r].x - v[r].y));
        }
      }
  }
}

// ---- partition spectra ------------------------------------------------------------------------
// Partition p of the stereo FIR (taps 2048 p .. 2048 p + 2047, zero-padded to 4096), scaled by
// 1 / 4096 for the unnormalised inverse transforms of the products.
__global__ __launch_bounds__(kBlock) void rv_partition_kernel(const float* h, int64_t L, int parts,
                                                              float4* Hs) {
  __shared__ float2 lds[kLds];
  __shared__ float2 w1lds[kW1Lds];
  const int p = blockIdx.x, slot = blockIdx.y;
  const int j = threadIdx.x;
  Twiddles tw;
  load_twiddles(tw, w1lds);
  const float* hl = h + (int64_t)slot * 2 * L;
  float2 v[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t n = (int64_t)kB * p + j + 256 * r;
    v[r] = (r < 8 && n < L) ? make_float2(hl[n], hl[L + n]) : make_float2(0.f, 0.f);
  }
  fft4096<false, 0x00FFu>(v, lds, tw);
  store_separated(v, lds, Hs + ((int64_t)slot * parts + p) * kRvStride, 1.0f / kN);
}

// ---- block spectra ----------------------------------------------------------------------------
// ADJ false: input window [2048 b - 2048 + shift, 2048 b + 2048 + shift) of the node's input sum;
// ADJ true: output-adjoint block [2048 b + shift, 2048 b + 2048 + shift) in the second half of a
// zero window. Stored at the node's parameter slot.
template <bool ADJ>
__global__ __launch_bounds__(kBlock) void rv_spectra_kernel(GraphView g, int node_begin, int nb,
                                                            int shift, float4* out,
                                                            int32_t* slot_len) {
  __shared__ float2 lds[kLds];
  __shared__ float2 w1lds[kW1Lds];
  const int b = blockIdx.x, node = node_begin + blockIdx.y;
  const int slot = g.param_row[node];
  Twiddles tw;
  load_twiddles(tw, w1lds);
  float2 v[16];
  if (slot_len && b == 0 && threadIdx.x == 0) slot_len[slot] = (int32_t)node_len(g, node);
  gather_window<ADJ>(g, node, kB * b - kB + shift, v, ADJ ? 8 : 0, 16);
  fft4096<false, ADJ ? 0xFF00u : 0xFFFFu>(v, lds, tw);
  store_separated(v, lds, out + ((int64_t)slot * nb + b) * kRvStride, 1.0f);
}

// ---- partitioned product, bin-major -------------------------------------------------------------
// For one one-sided bin k the partitioned product is a short convolution along the block index:
// forward C[b] = sum_p X[b - p] H[p], adjoint C[b] = sum_p Yf[b + p] conj(H[p]) with
// Yf[c] = Y0[c + 1] + (-1)^k Y0[c] (per channel, complex). A lane owns one bin of one node and
// kConvOut output blocks, summed in registers over every partition, the last one first, so that a
// decaying response adds its large terms at the end (relative errors over five draws of 2 s noise:
// output 2.93e-7 -> 2.43e-7, source adjoint 3.00e-7 -> 2.41e-7; two sums of 22 partitions each, as
// the kernel before this one made, 2.81e-7 and 2.84e-7; 391 -> 387 us a step of 16 reverbs). The
// blocks' spectra slide through a register ring (one enters per partition; the loop is unrolled by
// the ring's size, so the ring is indexed statically) and each partition spectrum is read once per
// kConvOut blocks, so a step of two 16-byte loads, made a step ahead, feeds 8 kConvOut
// multiply-adds. One wave per 64 bins; bin 2048 is left to the inverse kernel, since a 33rd wave for
// it alone would be a thirty-third of the launch. Waves of one node and bin range are neighbours on
// one XCD, whose L2 keeps the spectra that they share. 16 nodes, 128 blocks, 44 partitions: 4096
// waves, three a SIMD (151 and 163 VGPRs), so one round and a third: 60 us (0.1 ms with 22
// partitions in registers, blocks streaming through and the partial products of the tiles written
// apart). Loads further ahead, 14 or 12 blocks a wave, or two waves per SIMD instead of three gained
// nothing.
constexpr int kConvOut = 16;
constexpr int kBinWave = 64;
constexpr int kBinWaves = kN / 2 / kBinWave;  // 32

__device__ __forceinline__ float4 cmac2(float4 acc, float4 a, float4 b) {
  // per channel (x, y) and (z, w): acc += a * b (complex)
  acc.x = fma(a.x, b.x, fma(-a.y, b.y, acc.x));
  acc.y = fma(a.x, b.y, fma(a.y, b.x, acc.y));
  acc.z = fma(a.z, b.z, fma(-a.w, b.w, acc.z));
  acc.w = fma(a.z, b.w, fma(a.w, b.z, acc.w));
  return acc;
}

// Entry c of a node's rows of nb spectra at one bin, zero outside: a load from a clamped, valid
// address and a select on the value.
__device__ __forceinline__ float4 row_entry(const float4* Sk, int c, int nb) {
  const float4 v = Sk[(int64_t)min(max(c, 0), nb - 1) * kRvStride];
  return c >= 0 && c < nb ? v : make_float4(0.f, 0.f, 0.f, 0.f);
}

// The entry that partition p meets at output block b: X[b - p], or Yf[b + p].
template <bool CORR>
__device__ __forceinline__ float4 conv_entry(const float4* Sk, int b, int p, int nb, float sg) {
  if (!CORR) return row_entry(Sk, b - p, nb);
  const float4 y1 = row_entry(Sk, b + p + 1, nb), y0 = row_entry(Sk, b + p, nb);
  return make_float4(fmaf(sg, y0.x, y1.x), fmaf(sg, y0.y, y1.y), fmaf(sg, y0.z, y1.z),
                     fmaf(sg, y0.w, y1.w));
}

template <bool CORR>
__global__ __launch_bounds__(kBinWave, 3) void rv_conv_bins_kernel(GraphView g, int node_begin,
                                                                   int nb, int parts, int groups,
                                                                   const float4* S,
                                                                   const float4* Hs, float4* C) {
  const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
  const int node = node_begin + lb / (kBinWaves * groups);
  const int b0 = lb % groups * kConvOut;
  const int k = lb / groups % kBinWaves * kBinWave + threadIdx.x;
  const int slot = g.param_row[node];
  const float4* Sk = S + (int64_t)slot * nb * kRvStride + k;
  const float4* Hk = Hs + (int64_t)slot * parts * kRvStride + k;
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  const float sg = (k & 1) ? -1.f : 1.f;
  // Step q takes partition pe - 1 - q. Forward: it meets block b0 + i in ring[(i + q) mod kConvOut];
  // X[b0 + kConvOut - pe + 1 + q] enters after it. Adjoint: in ring[(i - q) mod kConvOut];
  // Yf[b0 + pe - 2 - q] enters after it. Partitions from pe on meet zeros only.
  const int pe = min(parts, CORR ? nb - b0 : b0 + kConvOut);
  float4 acc[kConvOut], ring[kConvOut];
  float4 y1 = CORR ? row_entry(Sk, b0 + pe - 1, nb) : zero;
  float4 ya = y1;
#pragma unroll
  for (int i = 0; i < kConvOut; ++i) {
    acc[i] = zero;
    const float4 yb = row_entry(Sk, CORR ? b0 + pe + i : b0 + i - pe + 1, nb);
    ring[i] = CORR ? make_float4(fmaf(sg, ya.x, yb.x), fmaf(sg, ya.y, yb.y), fmaf(sg, ya.z, yb.z),
                                 fmaf(sg, ya.w, yb.w))
                   : yb;
    ya = yb;
  }
  // what enters after step q: X[b0 + kConvOut - pe + 1 + q], or Y0[b0 + pe - 2 - q] (Y0 of the next
  // block before it)
  auto entering = [&](int q) {
    return row_entry(Sk, CORR ? b0 + pe - 2 - q : b0 + kConvOut - pe + 1 + q, nb);
  };
  auto filter = [&](int q) { return Hk[(int64_t)max(pe - 1 - q, 0) * kRvStride]; };
  float4 next_h = filter(0), next_e = entering(0);
  for (int q0 = 0; q0 < pe; q0 += kConvOut) {
#pragma unroll
    for (int j = 0; j < kConvOut; ++j) {
      const int q = q0 + j;
      if (q < pe) {  // uniform
        float4 h = next_h, e = next_e;
        next_h = filter(q + 1);
        next_e = entering(q + 1);
        if (CORR) h = make_float4(h.x, -h.y, h.z, -h.w);
#pragma unroll
        for (int i = 0; i < kConvOut; ++i)
          acc[i] = cmac2(acc[i], ring[(CORR ? i - j + kConvOut : i + j) % kConvOut], h);
        if (CORR) {
          const float4 y0 = e;
          e = make_float4(fmaf(sg, y0.x, y1.x), fmaf(sg, y0.y, y1.y), fmaf(sg, y0.z, y1.z),
                          fmaf(sg, y0.w, y1.w));
          y1 = y0;
        }
        ring[CORR ? kConvOut - 1 - j : j] = e;
      }
    }
  }
  float4* Ck = C + (int64_t)slot * nb * kRvStride + k;
#pragma unroll
  for (int i = 0; i < kConvOut; ++i)
    if (b0 + i < nb) Ck[(int64_t)(b0 + i) * kRvStride] = acc[i];
}

// Output block b: bin 2048 of the product (real per channel; one wave, a lane per partition), the
// packed spectrum rebuilt through LDS, one inverse transform; forward keeps its second half,
// adjoint its first.
template <bool CORR>
__global__ __launch_bounds__(kBlock) void rv_inverse_kernel(GraphView g, float* out, int node_begin,
                                                            int nb, int parts, const float4* S,
                                                            const float4* Hs, const float4* C) {
  __shared__ float2 lds[kLds];
  __shared__ float2 w1lds[kW1Lds];
  const int b = blockIdx.x, node = node_begin + blockIdx.y;
  const int slot = g.param_row[node];
  const int j = threadIdx.x;
  const int64_t T = g.T, Tn = node_len(g, node);
  if ((int64_t)kB * b >= Tn) return;  // block past the node's length (uniform over the block)
  float2 nyquist = make_float2(0.f, 0.f);  // (left, right), valid in wave 0
  if (j < 64) {
    const float4* Sk = S + (int64_t)slot * nb * kRvStride + kN / 2;
    const float4* Hk = Hs + (int64_t)slot * parts * kRvStride + kN / 2;
    for (int p = j; p < parts; p += 64) {
      const float4 e = conv_entry<CORR>(Sk, b, p, nb, 1.f), h = Hk[(int64_t)p * kRvStride];
      nyquist.x = fmaf(e.x, h.x, nyquist.x);
      nyquist.y = fmaf(e.z, h.z, nyquist.y);
    }
    nyquist.x = wave_sum(nyquist.x);
    nyquist.y = wave_sum(nyquist.y);
  }
  Twiddles tw;
  load_twiddles(tw, w1lds);
  const float4* Cb = C + ((int64_t)slot * nb + b) * kRvStride;
  float2 al[kHalfBins], ar[kHalfBins];
#pragma unroll
  for (int r = 0; r < kHalfBins - 1; ++r) {
    const float4 v = Cb[j + 256 * r];
    al[r] = make_float2(v.x, v.y);
    ar[r] = make_float2(v.z, v.w);
  }
  al[kHalfBins - 1] = make_float2(nyquist.x, 0.f);  // bin 2048, on thread 0
  ar[kHalfBins - 1] = make_float2(nyquist.y, 0.f);
  float2 v[16];
  pack_spectrum(al, ar, lds, v);
  fft4096<true>(v, lds, tw);
  float* y = out + (int64_t)node * 2 * T;
  float* ds = CORR ? source_row(g, node) : nullptr;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int64_t t = (int64_t)kB * b + j + 256 * r;
    if (t < Tn) {
      const float2 o = v[CORR ? r : r + 8];
      store_nt(y + t, o.x);
      store_nt(y + T + t, o.y);
      if (CORR && ds) {
        store_nt(ds + t, 0.f + o.x);
        store_nt(ds + T + t, 0.f + o.y);
      }
    }
  }
}

// ---- FIR gradient (the partitioned cross-correlation), bin-major ---------------------------------
// Cross-spectrum of partition p per channel, one-sided bins: G_c[k] = sum_{b >= p} Y0_c[b][k]
// conj(X_c[b - p][k]), scaled by 1 / 4096. A thread owns one bin of one slot and kCrossTile
// partitions: the input spectra enter a register ring one block per step (as in the product),
// the block's Y0 is read once for the whole tile. Each group of kCrossTile consecutive blocks is
// summed in float (at most kCrossTile terms), the groups in double, in block order. Bin 2048 is
// left to the next kernel: 16 nodes, 128 blocks, 44 partitions are 2048 waves, two a SIMD (203
// VGPRs), one round, which a 33rd wave per node and tile would make two: 67 us (139 us with it).
constexpr int kCrossTile = 11;

__global__ __launch_bounds__(kBinWave) void rv_cross_kernel(int nb, int parts, const float4* Y0,
                                                            const float4* X, float4* Gs) {
  const int k = blockIdx.x * kBinWave + threadIdx.x;
  const int p0 = blockIdx.y * kCrossTile, slot = blockIdx.z;
  const float4* ys = Y0 + (int64_t)slot * nb * kRvStride + k;
  const float4* xs = X + (int64_t)slot * nb * kRvStride + k;
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  float4 ring[kCrossTile];
  double acc[kCrossTile][4];
#pragma unroll
  for (int i = 0; i < kCrossTile; ++i) {
    ring[i] = zero;
    acc[i][0] = acc[i][1] = acc[i][2] = acc[i][3] = 0.0;
  }
  // blocks before p0 meet no input; Y0[b] and X[b - p0] are loaded a block ahead
  float4 next_x = row_entry(xs, 0, nb), next_y = row_entry(ys, p0, nb);
  for (int b0 = p0; b0 < nb; b0 += kCrossTile) {
    float4 part[kCrossTile];
#pragma unroll
    for (int i = 0; i < kCrossTile; ++i) part[i] = zero;
#pragma unroll
    for (int j = 0; j < kCrossTile; ++j) {
      const int b = b0 + j;
      if (b < nb) {  // uniform
        ring[j] = next_x;  // X[b - p0]
        const float4 y = next_y;
        next_x = row_entry(xs, b - p0 + 1, nb);
        next_y = row_entry(ys, b + 1, nb);
#pragma unroll
        for (int i = 0; i < kCrossTile; ++i) {  // partition p0 + i: X[b - p0 - i]
          const float4 x = ring[(j - i + kCrossTile) % kCrossTile];
          part[i].x = fma(y.x, x.x, fma(y.y, x.y, part[i].x));
          part[i].y = fma(y.y, x.x, fma(-y.x, x.y, part[i].y));
          part[i].z = fma(y.z, x.z, fma(y.w, x.w, part[i].z));
          part[i].w = fma(y.w, x.z, fma(-y.z, x.w, part[i].w));
        }
      }
    }
#pragma unroll
    for (int i = 0; i < kCrossTile; ++i) {
      acc[i][0] += part[i].x;
      acc[i][1] += part[i].y;
      acc[i][2] += part[i].z;
      acc[i][3] += part[i].w;
    }
  }
  constexpr double s = 1.0 / kN;
#pragma unroll
  for (int i = 0; i < kCrossTile; ++i)
    if (p0 + i < parts)
      Gs[((int64_t)slot * parts + p0 + i) * kRvStride + k] =
          make_float4((float)(s * acc[i][0]), (float)(s * acc[i][1]), (float)(s * acc[i][2]),
                      (float)(s * acc[i][3]));
}

// hbar_c[2048 p + i] = first half of the inverse transform of G (left: real part, right:
// imaginary part of the packed transform G_l + i G_r). Lags from valid_len[slot] + valid_shift on
// have no term (the shifted signals no longer overlap) and are written as exact zeros, not as
// rounding residue; valid_len is the node's own length, so a node of a merged batch gets the
// bits it gets alone.
// Bin 2048 of the cross-spectrum (real per channel) is summed here, in double over the blocks.
__global__ __launch_bounds__(kBlock) void rv_hbar_kernel(const float4* Gs, int nb, int parts,
                                                         int64_t L, const float4* Y0,
                                                         const float4* X,
                                                         const int32_t* valid_len, int valid_shift,
                                                         float* hbar) {
  __shared__ float2 lds[kLds];
  __shared__ float2 w1lds[kW1Lds];
  __shared__ double red[4];
  const int p = blockIdx.x, slot = blockIdx.y;
  const int j = threadIdx.x;
  double nl = 0.0, nr = 0.0;
  {
    const float4* ys = Y0 + (int64_t)slot * nb * kRvStride + kN / 2;
    const float4* xs = X + (int64_t)slot * nb * kRvStride + kN / 2;
    for (int b = p + j; b < nb; b += kBlock) {
      const float4 y = ys[(int64_t)b * kRvStride], x = xs[(int64_t)(b - p) * kRvStride];
      nl = fma((double)y.x, (double)x.x, nl);
      nr = fma((double)y.z, (double)x.z, nr);
    }
    nl = block_sum<double>(nl, red);
    nr = block_sum<double>(nr, red);
  }
  Twiddles tw;
  load_twiddles(tw, w1lds);
  const float4* G = Gs + ((int64_t)slot * parts + p) * kRvStride;
  float2 al[kHalfBins], ar[kHalfBins];
#pragma unroll
  for (int r = 0; r < kHalfBins - 1; ++r) {
    const float4 q = G[j + 256 * r];
    al[r] = make_float2(q.x, q.y);
    ar[r] = make_float2(q.z, q.w);
  }
  al[kHalfBins - 1] = make_float2((float)(nl * (1.0 / kN)), 0.f);  // bin 2048, on thread 0
  ar[kHalfBins - 1] = make_float2((float)(nr * (1.0 / kN)), 0.f);
  float2 v[16];
  pack_spectrum(al, ar, lds, v);
  fft4096<true>(v, lds, tw);
  float* hb = hbar + (int64_t)slot * 2 * L;
  const int64_t valid = (int64_t)valid_len[slot] + valid_shift;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int64_t n = (int64_t)kB * p + j + 256 * r;
    if (n < L) {
      hb[n] = n < valid ? v[r].x : 0.f;
      hb[L + n] = n < valid ? v[r].y : 0.f;
    }
  }
}

// Mask gradient. Frame m of channel x (mid, side) reads fbar[q] = hbar_x[192 m - 192 + q]
// (hbar_m = (hbar_l + hbar_r) / 2, hbar_s = (hbar_l - hbar_r) / 2), and the gradient with respect
// to the log-mask entry (k, m) is (c_k / 384) Re(Un[k] V_m[k]) mu[k] with c_k = 1 at k = 0, 192,
// else 2, and V_m[k] = sum_q fbar[q] e^(2 pi i k q / 384) = D_{m-1}[k] + (-1)^k D_m[k], where
// D_s[k] = sum_{t<192} hbar_x[192 s + t] e^(2 pi i k t / 384) is the DFT of one hop segment. A wave
// takes kGradFrames frames of one reverb slot: the segment of each is transformed (mid and side in
// one transform, zero-padded) and shared with the next frame, the masks are stepped as for the
// impulse response, and (sum_m G, sum_m m G) is summed per bin in frame order. Per-wave partials:
// part[slot][wave][x][k] = (a, d). 16 slots, 2 s: 29 us,
// 102 us as direct sums (4 frames a wave: 24 us, but 8 us more in the sum of the partials).
constexpr int kGradFrames = 8;

__global__ __launch_bounds__(kBlock) void rv_mask_grad_kernel(const float* P, const double2* Un,
                                                              const float* hbar, int64_t L, int M,
                                                              int nblk, double2* part) {
  constexpr int NK = (kK + 63) / 64;  // bins j + 64 r of lane j (the last on lane 0 only)
  __shared__ double2 tw[kF], lds[kWaves][kF];
  fill_tw384(tw);
  __syncthreads();
  const int wave = threadIdx.x >> 6, j = threadIdx.x & 63;
  const int blk = blockIdx.x * kWaves + wave, slot = blockIdx.y;
  if (blk >= nblk) return;  // no block barrier below
  const int m0 = blk * kGradFrames;
  const float* hb = hbar + (int64_t)slot * 2 * L;
  const float* p = P + (int64_t)slot * kRvParams;
  double2* s = lds[wave];
  double2 D[2][NK];  // the previous frame's segment (mid, side)
  auto segment = [&](int seg, double2 (&d)[2][NK]) {
    double2 x[6], v[8];
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      const int64_t n = (int64_t)kHop * seg + j + 64 * r;
      x[r] = make_double2(0.0, 0.0);
      if (r < 3 && n >= 0 && n < L) {
        const double a = hb[n], b = hb[L + n];
        x[r] = make_double2(0.5 * (a + b), 0.5 * (a - b));
      }
    }
    fft384<true>(x, v, s, tw, j);
    put384(v, s, j);
#pragma unroll
    for (int r = 0; r < NK; ++r) {
      const int k = min(j + 64 * r, kK - 1);
      const double2 a = s[k], b = s[k ? kF - k : 0];
      d[0][r] = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
      d[1][r] = make_double2(0.5 * (a.y + b.y), 0.5 * (b.x - a.x));
    }
    lds_order();
  };
  double mu[2][NK], step[2][NK], sa[2][NK], sd[2][NK];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int r = 0; r < NK; ++r) {
      const int k = min(j + 64 * r, kK - 1);
      mu[x][r] = mask_at(p, x, k, m0);
      step[x][r] = mask_step(p, x, k);
      sa[x][r] = sd[x][r] = 0.0;
    }
  segment(m0 - 1, D);
  const double sg = (j & 1) ? -1.0 : 1.0;
  for (int i = 0; i < kGradFrames && m0 + i < M; ++i) {
    const int m = m0 + i;
    double2 E[2][NK];
    segment(m, E);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int r = 0; r < NK; ++r) {
        const int k = min(j + 64 * r, kK - 1);
        const double2 u = Un[((int64_t)x * M + m) * kK + k];
        const double vr = fma(sg, E[x][r].x, D[x][r].x), vi = fma(sg, E[x][r].y, D[x][r].y);
        const double ck = (k == 0 || k == kK - 1) ? 1.0 / kF : 2.0 / kF;
        const double g = ck * (u.x * vr - u.y * vi) * mu[x][r];
        sa[x][r] += g;
        sd[x][r] = fma((double)m, g, sd[x][r]);
        mu[x][r] *= step[x][r];
        D[x][r] = E[x][r];
      }
  }
  double2* out = part + ((int64_t)slot * nblk + blk) * 2 * kK;
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int r = 0; r < NK; ++r)
      if (j + 64 * r < kK) out[x * kK + j + 64 * r] = make_double2(sa[x][r], sd[x][r]);
}

// dH0[k] = sum_m G[m][k], dHD[k] = sum_m m G[m][k]: the partials in order, four runs of them at a
// time (bin 191 adds the Nyquist bin, which shares its mask).
__global__ __launch_bounds__(kBlock) void rv_param_grad_kernel(const double2* part, int nblk,
                                                               float* dP) {
  __shared__ double2 red[kWaves][64];
  const int slot = blockIdx.x, x = blockIdx.y, w = threadIdx.x >> 6, j = threadIdx.x & 63;
  const int k = blockIdx.z * 64 + j;
  const int per = (nblk + kWaves - 1) / kWaves, b1 = min(nblk, (w + 1) * per);
  double a = 0.0, d = 0.0;
#pragma unroll 4
  for (int b = w * per; b < b1; ++b) {
    const double2* pb = part + (((int64_t)slot * nblk + b) * 2 + x) * kK;
    double2 v = pb[k];
    if (k == kRvBins - 1) {
      const double2 n = pb[kK - 1];
      v.x += n.x;
      v.y += n.y;
    }
    a += v.x;
    d += v.y;
  }
  red[w][j] = make_double2(a, d);
  __syncthreads();
  if (w != 0) return;
  const double2 t = dadd(dadd(dadd(red[0][j], red[1][j]), red[2][j]), red[3][j]);
  float* out = dP + (int64_t)slot * kRvParams + x * 2 * kRvBins;
  out[k] = (float)t.x;
  out[kRvBins + k] = (float)t.y;
}

}  // namespace

int rv_frames(int64_t L) { return (int)((L + kHop - 1) / kHop) + 1; }
int rv_parts(int64_t L) { return (int)((L + kB - 1) / kB); }
int rv_blocks(int64_t T) { return (int)((T + kB - 1) / kB); }
int rv_grad_blocks(int64_t L) { return (rv_frames(L) + kGradFrames - 1) / kGradFrames; }

hipError_t launch_rv_design(const float* P, int n, const float* noise, int64_t L, double2* Un,
                            float* h, float4* Hs, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int M = rv_frames(L), parts = rv_parts(L);
  rv_noise_stft_kernel<<<(M + kWaves - 1) / kWaves, kBlock, 0, s>>>(noise, L, M, Un);
  constexpr int kPerBlock = kWaves * kIrHops;
  rv_ir_kernel<<<dim3((M - 1 + kPerBlock - 1) / kPerBlock, n), kBlock, 0, s>>>(P, Un, L, M, h);
  rv_partition_kernel<<<dim3(parts, n), kBlock, 0, s>>>(h, L, parts, Hs);
  return hipGetLastError();
}

hipError_t launch_xcorr_spectra(const GraphView& g, int node_begin, int n_nodes, bool adj,
                                int shift, int nb, float4* out, int32_t* slot_len, hipStream_t s) {
  if (adj)
    rv_spectra_kernel<true><<<dim3(nb, n_nodes), kBlock, 0, s>>>(g, node_begin, nb, shift, out,
                                                                 slot_len);
  else
    rv_spectra_kernel<false><<<dim3(nb, n_nodes), kBlock, 0, s>>>(g, node_begin, nb, shift, out,
                                                                  slot_len);
  return hipGetLastError();
}

hipError_t launch_xcorr(int n, int nb, int parts, int64_t len, const int32_t* valid_len,
                        int valid_shift, const float4* Y0, const float4* X, float4* Gs, float* R,
                        hipStream_t s) {
  if (n <= 0) return hipSuccess;
  rv_cross_kernel<<<dim3(kBinWaves, (parts + kCrossTile - 1) / kCrossTile, n), kBinWave, 0, s>>>(
      nb, parts, Y0, X, Gs);
  rv_hbar_kernel<<<dim3(parts, n), kBlock, 0, s>>>(Gs, nb, parts, len, Y0, X, valid_len,
                                                   valid_shift, R);
  return hipGetLastError();
}

hipError_t launch_rv_fwd(const GraphView& g, float* U, int node_begin, int n_nodes, int64_t L,
                         const float4* Hs, float4* Z, float4* C, hipStream_t s) {
  const int nb = rv_blocks(g.T), parts = rv_parts(L), groups = (nb + kConvOut - 1) / kConvOut;
  rv_spectra_kernel<false><<<dim3(nb, n_nodes), kBlock, 0, s>>>(g, node_begin, nb, 0, Z, nullptr);
  rv_conv_bins_kernel<false><<<(unsigned)(kBinWaves * groups * n_nodes), kBinWave, 0, s>>>(
      g, node_begin, nb, parts, groups, Z, Hs, C);
  rv_inverse_kernel<false><<<dim3(nb, n_nodes), kBlock, 0, s>>>(g, U, node_begin, nb, parts, Z, Hs,
                                                                C);
  return hipGetLastError();
}

hipError_t launch_rv_bwd(const GraphView& g, float* dU, int node_begin, int n_nodes, int64_t L,
                         const float4* Hs, float4* Y0, float4* C, int32_t* slot_len,
                         hipStream_t s) {
  const int nb = rv_blocks(g.T), parts = rv_parts(L), groups = (nb + kConvOut - 1) / kConvOut;
  rv_spectra_kernel<true><<<dim3(nb, n_nodes), kBlock, 0, s>>>(g, node_begin, nb, 0, Y0, slot_len);
  rv_conv_bins_kernel<true><<<(unsigned)(kBinWaves * groups * n_nodes), kBinWave, 0, s>>>(
      g, node_begin, nb, parts, groups, Y0, Hs, C);
  rv_inverse_kernel<true><<<dim3(nb, n_nodes), kBlock, 0, s>>>(g, dU, node_begin, nb, parts, Y0, Hs,
                                                               C);
  return hipGetLastError();
}

hipError_t launch_rv_grad(int n, int64_t T, int64_t L, const float* P, const double2* Un,
                          const float4* Z, const float4* Y0, const int32_t* slot_len, float4* Gs,
                          float* hbar, double* part, float* dP, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int nb = rv_blocks(T), parts = rv_parts(L), M = rv_frames(L);
  // hbar[n] = sum_t ybar[t] u[t - n] has no term for n >= the node's length
  const hipError_t e = launch_xcorr(n, nb, parts, L, slot_len, 0, Y0, Z, Gs, hbar, s);
  if (e != hipSuccess) return e;
  const int nblk = rv_grad_blocks(L);
  rv_mask_grad_kernel<<<dim3((nblk + kWaves - 1) / kWaves, n), kBlock, 0, s>>>(
      P, Un, hbar, L, M, nblk, reinterpret_cast<double2*>(part));
  rv_param_grad_kernel<<<dim3(n, 2, kRvBins / 64), kBlock, 0, s>>>(
      reinterpret_cast<const double2*>(part), nblk, dP);
  return hipGetLastError();
}

}  // namespace grafx

// Zero-phase FIR equaliser (paper Sec. 3 "Equalizer", Eqs. 4-5): 2047 taps designed from 1024
// log-magnitudes, applied to both channels.
//
// Design (once per render, all EQ nodes): h[n] = v[n] (A_0 + 2 sum_k A_k cos(2 pi k n / 2047)) /
// 2047 with A_k = exp(p_k) and a symmetric Hann window v, accumulated in double; then the real
// spectrum of h on the 4096-point grid, H[k] = h[0] + 2 sum_n h[n] cos(2 pi k n / 4096), scaled
// by 1/4096 for the inverse transform.
//
// Filtering: overlap-save, one 4096-point complex FFT per tile of 2048 outputs. The two
// channels ride in one complex signal (left + i right); the filter is real and even, so
// multiplying the spectrum by real H filters both channels at once. A tile's window starts 1024
// samples before its first output, so the 2047-tap kernel never wraps. The FFT is a radix-16
// Stockham transform with 256 threads x 16 points held in registers: the forward transform ends
// and the inverse begins in the same register layout, so only the two inner passes of each
// transform touch LDS; each thread keeps the 15 twiddles of the last pass in registers for all
// transforms of the block and reads those of the middle pass, which take only 16 x 16 values,
// from LDS. Window gathers use raw buffer loads whose range check supplies the zero padding. Tiles
// of one node are mapped onto one XCD (neighbouring tiles share the halo through its L2); the
// EQ block-order setting can keep the hardware order instead (same arithmetic).
//
// Adjoint: the input adjoint is the same filter applied to the output adjoint (h is even). The
// FIR gradient hbar[n] = sum_{c,t} ybar_c[t] u_c[t - n] is the real part of a complex
// correlation, accumulated per tile as C[k] = W'[k] conj(U_tile[k]) (ybar window spectrum times
// the conjugate spectrum of the zero-padded input tile). The design is even in n, so only
// hbar[n] + hbar[-n] matters: the inverse transform of the real, even sequence
// F[k] = Re C[k] + Re C[N - k], of which N/2 + 1 values are kept. Each block handles one tile
// and writes its folded F into its node's own region; after the last step the tiles' F are summed
// per node in a fixed order, by a launch of its own or (rows of few tiles) by the blocks of the
// transform that follows. The order does not depend on how nodes are grouped into steps, so
// results do not depend on the schedule. Then one inverse FFT per node gives
// hbar[n] + hbar[-n], and the chain rule through the design gives
// dL/dp_k = (kappa_k / 2047) A_k sum_n hbar[n] v[n] cos(2 pi k n / 2047).
#include <type_traits>

#include "device_common.h"
#include "grafx_internal.h"
#include "kernels.h"
#include "fft4096.h"
#include "reduce_partials.h"
#include "tables.inc"

namespace grafx {
namespace {

using namespace fft4;

// ---- design ----------------------------------------------------------------------------------
// The three cosine sums (A -> h, h -> H and, in the adjoint, hbar -> dL/dp) are products of a
// [nodes x 1024] matrix with a cosine matrix, in double on the matrix cores: a block computes 16
// outputs of 16 nodes, its 4 waves taking 256 terms each. Lane (i, q) supplies node i and output i at
// the wave's terms 64 q, 64 q + 1, ..., so a row is read 16 bytes at a time; the cosines follow the
// Chebyshev recurrence c_{m+1} = 2 cos(theta) c_m - c_{m-1} over 64 terms from correctly rounded table
// values (every angle is 2 pi s / M for an integer s). The sums over even and odd terms are kept
// apart: their difference is the sum at M / 2 - s, so H needs half the products. 48 nodes: h 11.2 ->
// 7.6 us, H 18.5 -> 8.5 us, dL/dp 11.4 -> 7.8 us, bound by the matrix rate in double (twice the waves
// with half the terms each take as long); 4 nodes: 5.9, 5.4, 5.7 -> 5.3, 4.9, 4.9 us (launch and load
// latency). Before, eight lanes an output read every term from LDS, and each of 32 blocks a node
// formed all 1024 exponentials, which are now part of the launch that prepares the pass.

typedef double f64x4 __attribute__((ext_vector_type(4)));

// w [rows][stride] -> the 16 x 16 sums of this block: thread (r, n) of 16 x 16 receives
// sum_m w[16 blockIdx.y + r][m] cos(2 pi m s / M), s = 16 blockIdx.x + n, 0 <= s <= M, as the sums over
// even and over odd m (added: the sum at s; subtracted, for even M: at M / 2 - s); the term m = 0
// counts half if HALF. Rows past the last repeat it.
template <int M, bool HALF>
__device__ __forceinline__ double2 cos_sums(const double* w, int rows, int stride,
                                            const double* tab) {
  __shared__ double2 red[4][256];
  const int wave = threadIdx.x >> 6, i = threadIdx.x & 15, q = (threadIdx.x >> 4) & 3;
  const int row = min((int)blockIdx.y * 16 + i, rows - 1), s = (int)blockIdx.x * 16 + i;
  const int m0 = 256 * wave + 64 * q;
  const double2* wr = reinterpret_cast<const double2*>(w + (int64_t)row * stride + m0);
  double2 a[32];
#pragma unroll
  for (int m = 0; m < 32; ++m) a[m] = wr[m];
  double c = tab[m0 * s % M], cm = tab[(m0 + M - 1) * s % M];
  const double two_c = 2.0 * tab[s % M];
  if (HALF && m0 == 0) a[0].x *= 0.5;
  f64x4 acc[2] = {f64x4{0.0, 0.0, 0.0, 0.0}, f64x4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
  for (int m = 0; m < 32; ++m) {
    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m].x, c, acc[0], 0, 0, 0);
    cm = fma(two_c, c, -cm);
    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m].y, cm, acc[1], 0, 0, 0);
    c = fma(two_c, cm, -c);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) red[wave][(q + 4 * e) * 16 + i] = make_double2(acc[0][e], acc[1][e]);
  __syncthreads();
  const int t = threadIdx.x;
  return make_double2(((red[0][t].x + red[1][t].x) + red[2][t].x) + red[3][t].x,
                      ((red[0][t].y + red[1][t].y) + red[2][t].y) + red[3][t].y);
}

constexpr int kAStride = kN / 2;  // A = exp(p) waits in the first half of the node's row of H

__global__ __launch_bounds__(kBlock) void eq_design_h_kernel(const double* A, int n_eq,
                                                             double* h) {
  const double2 sum = cos_sums<2047, true>(A, n_eq, kAStride, kCos2047);
  const int slot = blockIdx.y * 16 + (threadIdx.x >> 4), n = blockIdx.x * 16 + (threadIdx.x & 15);
  if (slot >= n_eq) return;
  const double win = 0.5 + 0.5 * cospi((double)n / 1023.0);
  h[(int64_t)slot * 1024 + n] = win * (2.0 * (sum.x + sum.y) / 2047.0);
}

__global__ __launch_bounds__(kBlock) void eq_design_H_kernel(const double* h, int n_eq, float* H) {
  const double2 sum = cos_sums<kN, true>(h, n_eq, 1024, kCos4096);
  const int slot = blockIdx.y * 16 + (threadIdx.x >> 4), k = blockIdx.x * 16 + (threadIdx.x & 15);
  if (slot >= n_eq || k > kN / 4) return;
  float* Hn = H + (int64_t)slot * kN;
  auto put = [&](int bin, double v) {
    const float Hk = (float)(2.0 * v / (double)kN);
    Hn[bin] = Hk;
    if (bin > 0 && bin < kN / 2) Hn[kN - bin] = Hk;
  };
  put(k, sum.x + sum.y);
  if (k < kN / 4) put(kN / 2 - k, sum.x - sum.y);
}

// ---- forward ----------------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void eq_fwd_kernel(GraphView g, float* U, const float* H,
                                                        int node_begin, int tiles) {
  __shared__ float2 lds[kLds];
  __shared__ float2 w1lds[kW1Lds];
  const int lb = g.eq_order ? (int)blockIdx.x : xcd_logical_block(blockIdx.x, gridDim.x);
  const int tile = lb % tiles, node = node_begin + lb / tiles;
  const int j = threadIdx.x;
  const int64_t T = g.T, Tn = node_len(g, node);
  const int t0 = tile * kEqHop;
  if (t0 >= Tn) return;  // tile past the node's length
  Twiddles tw;
  load_twiddles(tw, w1lds);
  float2 v[16];
  gather_window<false>(g, node, t0 - kN / 4, v, 0, 16);  // window: 1024 samples of history
  fft4096<false>(v, lds, tw);
  const float* Hn = H + (int64_t)g.param_row[node] * kN;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float hk = Hn[j + 256 * r];
    v[r].x *= hk;
    v[r].y *= hk;
  }
  fft4096<true>(v, lds, tw);
  float* y = U + (int64_t)node * 2 * T;
  const auto yl = row_rsrc(y, Tn), yr = row_rsrc(y + T, Tn);  // stores past Tn are dropped
#pragma unroll
  for (int r = 4; r < 12; ++r) {
    const int t = t0 + j + 256 * (r - 4);
    bstore_nt(yl, t, v[r].x);
    bstore_nt(yr, t, v[r].y);
  }
}

// ---- adjoint ----------------------------------------------------------------------------------
// Per tile: FFT of the output-adjoint window (its spectrum kept in registers), times H and
// inverse FFT for the input adjoint, FFT of the zero-padded input tile, real part of the
// cross-spectrum through LDS, folded and written per tile.
__global__ __launch_bounds__(kBlock) void eq_bwd_kernel(GraphView g, float* dU, const float* H,
                                                        int node_begin, int tiles, float* Fpart) {
  __shared__ float2 lds[kLds];
  __shared__ float2 w1lds[kW1Lds];
  const int lb = g.eq_order ? (int)blockIdx.x : xcd_logical_block(blockIdx.x, gridDim.x);
  const int tile = lb % tiles, node = node_begin + lb / tiles;
  const int j = threadIdx.x;
  const int64_t T = g.T, Tn = node_len(g, node);
  const int slot = g.param_row[node];
  const float* Hn = H + (int64_t)slot * kN;
  float* d = dU + (int64_t)node * 2 * T;
  float* out = Fpart + ((int64_t)slot * tiles + tile) * kEqFoldStride;
  const int t0 = tile * kEqHop;
  if (t0 >= Tn) {  // tile past the node's length: contributes nothing to the gradient
    for (int k = j; k <= kN / 2; k += kBlock) out[k] = 0.f;
    return;
  }
  Twiddles tw;
  load_twiddles(tw, w1lds);
  float2 v[16], keep[16];
  gather_window<true>(g, node, t0 - kN / 4, v, 0, 16);
  fft4096<false>(v, lds, tw);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    keep[r] = v[r];
    const float hk = Hn[j + 256 * r];
    v[r].x *= hk;
    v[r].y *= hk;
  }
  fft4096<true>(v, lds, tw);
  {
    const auto dl = row_rsrc(d, Tn), dr = row_rsrc(d + T, Tn);  // stores past Tn are dropped
#pragma unroll
    for (int r = 4; r < 12; ++r) {
      const int t = t0 + j + 256 * (r - 4);
      bstore_nt(dl, t, v[r].x);
      bstore_nt(dr, t, v[r].y);
    }
    if (float* ds = source_row(g, node)) {
      const auto sl = row_rsrc(ds, Tn), sr = row_rsrc(ds + T, Tn);
#pragma unroll
      for (int r = 4; r < 12; ++r) {
        const int t = t0 + j + 256 * (r - 4);
        bstore_nt(sl, t, 0.f + v[r].x);
        bstore_nt(sr, t, 0.f + v[r].y);
      }
    }
  }
  gather_window<false>(g, node, t0 - kN / 4, v, 4, 12);  // input tile, zero-padded
  fft4096<false, 0x0FF0u>(v, lds, tw);
  // Re C[k] = Re(W'[k] conj(U[k])); fold F[k] = Re C[k] + Re C[N - k], k = 0..N/2 (bins of other
  // threads: through the transform's LDS, free again after its last barrier)
  float* cre = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int r = 0; r < 16; ++r) cre[j + 256 * r] = keep[r].x * v[r].x + keep[r].y * v[r].y;
  __syncthreads();
  for (int k = j; k <= kN / 2; k += kBlock) out[k] = cre[k] + cre[(kN - k) & (kN - 1)];
}

// Sum the folded cross-spectra of the tiles of every EQ node per bin, in double and in a fixed
// order: tiles w, w + 4, w + 8, ... for w = 0..3, then the four sums in order. Each node has its own
// region of partials, so one launch after the last adjoint step serves every step, and the order
// does not depend on how nodes form steps. Long rows: blocks of 64 bins, wave w taking sum w; the
// blocks after them are reduction jobs of other types.
__global__ __launch_bounds__(kBlock) void eq_fold_reduce_kernel(const float* Fpart, int tiles,
                                                                float* F, int n_eq,
                                                                ReduceJobs jobs) {
  __shared__ double part[4][64];
  constexpr int kBinBlocks = (kN / 2 + 64) / 64;
  const int slot = blockIdx.x / kBinBlocks, bin = blockIdx.x % kBinBlocks;
  if (slot >= n_eq) return reduce_partials(jobs, (int)blockIdx.x - n_eq * kBinBlocks);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int k = bin * 64 + lane;
  const bool live = k <= kN / 2;
  double s = 0.0;
  if (live) {
    const float* p = Fpart + (int64_t)slot * tiles * kEqFoldStride + k;
#pragma unroll 8
    for (int t = w; t < tiles; t += 4) s += p[(int64_t)t * kEqFoldStride];
  }
  part[w][lane] = s;
  __syncthreads();
  if (w == 0 && live)
    F[(int64_t)slot * kEqFoldStride + k] =
        (float)(((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane]);
}

// The inverse FFT of the folded cross-spectrum gives hbar[n] + hbar[-n]; with the window,
// s[0] = hbar[0] and s[n] = v[n] (hbar[n] + hbar[-n]). FOLD (short rows, up to kFoldTiles tiles): the
// block first forms the folded spectrum itself, in the order above, and the blocks after the nodes'
// are the reduction jobs: one launch instead of three (4 nodes of 2^15 samples: 7.4 us, 3.3 + 4.8
// + 4.3 us apart). One block a node then sums all tiles, against 33 blocks in a launch of its own, so
// the line lies at 16 tiles. Adjoint of 1, 4, 17, 48 EQ strips folded here and apart, us: 8 tiles 23.4,
// 24.0, 26.8, 31.0 and 23.8, 24.6, 27.4, 31.9; 16 tiles 24.7, 25.4, 30.3, 38.3 and 24.8, 25.4, 30.3,
// 39.1; 24 tiles 25.8, 26.9, 32.5, 47.0 and 25.6, 26.3, 32.2, 46.7; 32 tiles 26.9, 28.4, 38.2, 52.4
// and 24.0, 25.4, 35.5, 51.4.
constexpr int kFoldTiles = 16;
template <bool FOLD>
__global__ __launch_bounds__(kBlock) void eq_grad_ifft_kernel(const float* F, int tiles, int n_eq,
                                                              double* sbuf, ReduceJobs jobs) {
  __shared__ float2 lds[kLds];
  __shared__ float2 w1lds[kW1Lds];
  const int slot = blockIdx.x;
  if (FOLD && slot >= n_eq) return reduce_partials(jobs, slot - n_eq);
  const int j = threadIdx.x;
  Twiddles tw;
  load_twiddles(tw, w1lds);
  const float* f = F + (int64_t)slot * (FOLD ? tiles : 1) * kEqFoldStride;
  if constexpr (FOLD) {
    float* folded = reinterpret_cast<float*>(lds);
    double p[4][9] = {};  // bins j + 256 r, and N / 2
    auto add = [&](int t, auto count) {  // all loads of a group of tiles before any sum
      float q[4][9];
#pragma unroll
      for (int w = 0; w < count.value; ++w)
#pragma unroll
        for (int r = 0; r < 9; ++r)
          q[w][r] = f[(int64_t)(t + w) * kEqFoldStride + (r < 8 ? j + 256 * r : kN / 2)];
#pragma unroll
      for (int w = 0; w < count.value; ++w)
#pragma unroll
        for (int r = 0; r < 9; ++r) p[w][r] += (double)q[w][r];
    };
    int t = 0;
    for (; t + 4 <= tiles; t += 4) add(t, std::integral_constant<int, 4>{});
    switch (tiles - t) {
      case 1: add(t, std::integral_constant<int, 1>{}); break;
      case 2: add(t, std::integral_constant<int, 2>{}); break;
      case 3: add(t, std::integral_constant<int, 3>{}); break;
    }
#pragma unroll
    for (int r = 0; r < 9; ++r)
      if (r < 8 || j == 0)
        folded[j + 256 * r] = (float)(((p[0][r] + p[1][r]) + p[2][r]) + p[3][r]);
    __syncthreads();
    f = folded;
  }
  float2 v[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int k = j + 256 * r;
    v[r] = make_float2(f[k <= kN / 2 ? k : kN - k], 0.f);
  }
  if (FOLD) __syncthreads();  // the transform reuses the folded spectrum's LDS
  fft4096<true>(v, lds, tw);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int n = j + 256 * r;
    const float hb = v[r].x * (1.0f / kN);
    double s;
    if (n == 0) {
      s = 0.5 * (double)hb;
    } else {
      const double win = 0.5 + 0.5 * cospi((double)n / 1023.0);
      s = win * (double)hb;
    }
    sbuf[(int64_t)slot * 1024 + n] = s;
  }
}

// dL/dp_k = (kappa_k / 2047) A_k (s[0] + sum_{n>=1} s[n] cos(2 pi k n / 2047)).
__global__ __launch_bounds__(kBlock) void eq_grad_p_kernel(const float* P, const double* sbuf,
                                                           int n_eq, float* dP) {
  const double2 sum = cos_sums<2047, false>(sbuf, n_eq, 1024, kCos2047);
  const int slot = blockIdx.y * 16 + (threadIdx.x >> 4), k = blockIdx.x * 16 + (threadIdx.x & 15);
  if (slot >= n_eq) return;
  const double A = exp((double)P[(int64_t)slot * 1024 + k]);
  const double kappa = k == 0 ? 1.0 : 2.0;
  dP[(int64_t)slot * 1024 + k] = (float)(kappa / 2047.0 * A * (sum.x + sum.y));
}

}  // namespace

int eq_tiles(int64_t T) { return (int)((T + kEqHop - 1) / kEqHop); }

hipError_t launch_eq_design(int n_eq, double* h, float* H, hipStream_t s) {
  if (n_eq <= 0) return hipSuccess;
  const int rows = (n_eq + 15) / 16;
  eq_design_h_kernel<<<dim3(1024 / 16, rows), kBlock, 0, s>>>(reinterpret_cast<double*>(H), n_eq,
                                                             h);
  eq_design_H_kernel<<<dim3(kN / 4 / 16 + 1, rows), kBlock, 0, s>>>(h, n_eq, H);
  return hipGetLastError();
}

hipError_t launch_eq_fwd(const GraphView& g, float* U, const float* H, int node_begin,
                         int n_nodes, hipStream_t s) {
  const int tiles = eq_tiles(g.T);
  eq_fwd_kernel<<<(unsigned)(tiles * n_nodes), kBlock, 0, s>>>(g, U, H, node_begin, tiles);
  return hipGetLastError();
}

hipError_t launch_eq_bwd(const GraphView& g, float* dU, const float* H, int node_begin,
                         int n_nodes, float* Fpart, hipStream_t s) {
  const int tiles = eq_tiles(g.T);
  eq_bwd_kernel<<<(unsigned)(tiles * n_nodes), kBlock, 0, s>>>(g, dU, H, node_begin, tiles,
                                                               Fpart);
  return hipGetLastError();
}

hipError_t launch_eq_grad(const float* P, const float* Fpart, int tiles, float* F, int n_eq,
                          double* sbuf, float* dP, const ReduceJobs& jobs, hipStream_t s) {
  if (n_eq <= 0) return hipSuccess;
  if (tiles <= kFoldTiles) {
    eq_grad_ifft_kernel<true><<<n_eq + jobs.blocks(), kBlock, 0, s>>>(Fpart, tiles, n_eq, sbuf,
                                                                      jobs);
  } else {
    eq_fold_reduce_kernel<<<n_eq * ((kN / 2 + 64) / 64) + jobs.blocks(), kBlock, 0, s>>>(
        Fpart, tiles, F, n_eq, jobs);
    eq_grad_ifft_kernel<false><<<n_eq, kBlock, 0, s>>>(F, tiles, n_eq, sbuf, ReduceJobs());
  }
  eq_grad_p_kernel<<<dim3(1024 / 16, (n_eq + 15) / 16), kBlock, 0, s>>>(P, sbuf, n_eq, dP);
  return hipGetLastError();
}

}  // namespace grafx

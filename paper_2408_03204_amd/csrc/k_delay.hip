// Multitap delay (paper Sec. 3 "Multitap delay", Eq. 14) with M 100 ms slots per channel:
// y_c[t] = sum_m sum_{j=-19}^{19} c_{c,m}[j] u_c[t - d_{c,m} - j]. Two node types share these
// kernels, templated on M: the 2 s delay of the paper (M = 20, 880 parameters) and a 500 ms one
// (M = 5, 220 parameters).
//
// Design (once per render): the integer delay of slot m is (m * 4410) plus
// rint(-arg(z) * 4410 / 2 pi) mod 4410, decided in float32; each slot's 39-tap zero-phase FIR is
// built from its 20 log-magnitudes like the EQ (N = 39, symmetric Hann), in double, and so is its
// spectrum on 512 points, which is real and even.
//
// Filtering: overlap-save on 512-point transforms, 474 outputs a tile, one wave per tile. A slot's
// window (the input read at the slot's delay, left + i right, each channel at its own delay) is
// transformed, its bins 0 .. 256 are separated into the two channels (bins k and -k: one exchange)
// and multiplied by the slot's two real spectra; the slots' products are summed in registers, and
// one inverse transform gives the tile. M + 1 transforms of 512 points replace 78 M multiply-adds
// per stereo sample. Bound by instruction issue: 24 nodes, T = 2^17, M = 5: 34 us, 47 us as a
// direct form.
// Adjoint: the input adjoint is the same sum over windows of the output adjoint read at plus the
// delays. The same windows' spectra Y give the tap gradients: with U the spectrum of the
// zero-padded input tile, sum_s ybar_c[s + d + j] u_c[s] is the inverse transform of Y conj U per
// channel, and since the filters are even only its even part enters, whose spectrum is
// Re(Y conj U). That is summed over a wave's tiles in registers and inverted once per group. One
// launch (M + 2 transforms a tile) replaces 156 M multiply-adds per stereo sample: 60 us, 101 us
// as two direct-form launches.
// The partial lags (0 .. 19 of the even part) are summed over the groups in double and mapped back
// to the log-magnitudes through the design. By default the delay times are not differentiated
// (their phasor gradients are 0).
//
// Delay-time surrogate (Sec. 3 "Multitap delay", Eq. 15), an option of the schedule: the phasor z
// of slot m gets the straight-through gradient of the surrogate impulse
// s[n] = Re (1/N) sum_{k<N} z^k e^(2 pi i k n / N) (N = 4410 lags from the slot's start), which is
// the unit impulse at the slot's integer delay when z lies on the unit circle at that delay. With
// G[n] = dL/ds[n] = sum_j c[j] R[4410 m + n + j - 19] (R[l] = sum_t ybar[t] u[t - l], the
// cross-correlation of the output adjoint and the input, from the partitioned correlation of the
// reverb's FIR gradient with the output adjoint delayed by 19 samples so that lags start at -19),
// dL/dRe z = Re Q and dL/dIm z = -Im Q with Q = sum_n G[n] s'(z)[n]
// = (1/N) sum_{k>=1} k z^(k-1) sum_n G[n] e^(2 pi i k n / N), all in double.
#include <type_traits>

#include "device_common.h"
#include "grafx_internal.h"
#include "kernels.h"
#include "tables.inc"

namespace grafx {
namespace {

constexpr int kHalf = 19;                   // taps j = -19..19
constexpr int kN = kDelayFFT;               // 512-point transforms
constexpr int kHop = kN - 2 * kHalf;        // 474 outputs per tile
constexpr int kWaves = kBlock / 64;
constexpr int kSlotsPerWave = 5;            // adjoint: slots whose gradients a wave accumulates
constexpr int kSlice = kN + kN / 8 + 2;     // LDS entries per wave (one pad per 8, element 512 = 0)

// Tiles of one tap-gradient group: half of the schedule's setting, not a function of T, so a node's
// partial sums are grouped the same way whatever the row stride (a graph merged with longer ones
// gets the same bits as alone). More tiles amortise the five inverse transforms and the partial
// lags of a group; fewer give short steps more waves.
__host__ __device__ constexpr int group_tiles(int tap_tiles) { return tap_tiles / 2; }

// ---- 512-point transform of one wave -----------------------------------------------------------
// 64 lanes x 8 points, radix 8 three times (Stockham); the two exchanges go through the wave's own
// LDS slice. A wave's LDS accesses are executed in order, so they need no barrier, only that the
// compiler keeps their order.

// Twiddles of lane j: w2[r] = exp(-2 pi i r j / 512) differ in every lane and stay in registers;
// w1[r] = exp(-2 pi i r (j mod 8) / 64) take 8 x 8 values, in LDS (rows of 9, distinct banks).
struct Twiddles512 {
  float2 w2[8];
  const float2* w1;
};
constexpr int kW1 = 8 * 9;

// Every wave of the block fills its own copy of the table.
__device__ __forceinline__ void load_twiddles512(Twiddles512& tw, float2* w1, int j) {
  w1[(j >> 3) * 9 + (j & 7)] = kTw4096[64 * (j >> 3) * (j & 7)];
#pragma unroll
  for (int r = 1; r < 8; ++r) tw.w2[r] = kTwRows512[64 * r + j];
  tw.w1 = w1 + (j & 7) * 9;
}

__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

// On entry v[r] = x[j + 64 r], on exit X[j + 64 r] (forward exp(-2 pi i nk/N), inverse exp(+...),
// unnormalised). Element e of an exchange sits at e + e / 8: the writes at 8 j + r and
// 64 (j / 8) + j mod 8 + 8 r and the reads at j + 64 r fall on distinct banks (but for a wrap of
// three lanes of the reads), and all are a lane base plus a constant.
template <bool INV>
__device__ __forceinline__ void fft512(float2 (&v)[8], float2* s, const Twiddles512& tw, int j) {
  float2* const s0 = s + 9 * j;
  float2* const s1 = s + j + (j >> 3);
  float2* const s2 = s + (j >> 3) * 72 + (j & 7);
  dft8<INV>(v);
  lds_order();
#pragma unroll
  for (int r = 0; r < 8; ++r) s0[r] = v[r];
  lds_order();
#pragma unroll
  for (int r = 0; r < 8; ++r) v[r] = s1[72 * r];
  lds_order();
#pragma unroll
  for (int r = 1; r < 8; ++r) v[r] = INV ? cmulc(v[r], tw.w1[r]) : cmul(v[r], tw.w1[r]);
  dft8<INV>(v);
#pragma unroll
  for (int r = 0; r < 8; ++r) s2[9 * r] = v[r];
  lds_order();
#pragma unroll
  for (int r = 0; r < 8; ++r) v[r] = s1[72 * r];
  lds_order();
#pragma unroll
  for (int r = 1; r < 8; ++r) v[r] = INV ? cmulc(v[r], tw.w2[r]) : cmul(v[r], tw.w2[r]);
  dft8<INV>(v);
}

// Bins 0 .. 256 of the two real channels of a window, doubled: lane j holds k = j + 64 r (r < 4),
// and lane 0 also bin 256 (both channels real there; the other lanes' value is not used).
struct Bins {
  float2 l[4], r[4];
  float nl, nr;
};

// Element e of a spectrum in a slice sits at e + e / 8; element 512 stands for element 0.
__device__ __forceinline__ float2* at(float2* s, int j) { return s + j + (j >> 3); }  // j + 64 r: [72 r]
__device__ __forceinline__ float2* at_mirror(float2* s, int j) {  // 512 - j - 64 r: [-72 r]
  return s + (kN - j) + ((kN - j) >> 3);
}

// From Z = FFT(left + i right): 2 L[k] = Z[k] + conj Z[-k], 2 R[k] = -i (Z[k] - conj Z[-k]).
__device__ __forceinline__ void separate(const float2 (&z)[8], Bins& b, float2* s, int j) {
  lds_order();
#pragma unroll
  for (int r = 4; r < 8; ++r) at(s, j)[72 * r] = z[r];
  if (j == 0) s[kN + kN / 8] = z[0];
  lds_order();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float2 m = at_mirror(s, j)[-72 * r];
    b.l[r] = make_float2(z[r].x + m.x, z[r].y - m.y);
    b.r[r] = make_float2(z[r].y + m.y, m.x - z[r].x);
  }
  b.nl = 2.f * z[4].x;
  b.nr = 2.f * z[4].y;
  lds_order();
}

// The spectrum of left + i right from bins 0 .. 256 of the channels: v[k] = L + i R and
// v[-k] = conj L + i conj R.
__device__ __forceinline__ void join(const Bins& b, float2 (&v)[8], float2* s, int j) {
  lds_order();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    v[r] = make_float2(b.l[r].x - b.r[r].y, b.l[r].y + b.r[r].x);
    at_mirror(s, j)[-72 * r] = make_float2(b.l[r].x + b.r[r].y, b.r[r].x - b.l[r].y);
  }
  if (j == 0) s[kN / 2 + kN / 16] = make_float2(b.nl, b.nr);
  lds_order();
#pragma unroll
  for (int r = 4; r < 8; ++r) v[r] = at(s, j)[72 * r];
  lds_order();
}

// Keeps the compiler from moving the computation of a value past this point (sunk to their next
// use, the sums of a slot would keep the slot's whole spectrum in registers until then).
__device__ __forceinline__ void pin(float& x) { asm volatile("" : "+v"(x)); }

// acc += spectra x bins; sp: this lane's bin j of the slot's (left, right) spectra, n: its bin 256
__device__ __forceinline__ void multiply_add(const Bins& b, const float2* sp, float2 n, Bins& acc) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float2 c = sp[64 * r];
    acc.l[r] = make_float2(fmaf(c.x, b.l[r].x, acc.l[r].x), fmaf(c.x, b.l[r].y, acc.l[r].y));
    acc.r[r] = make_float2(fmaf(c.y, b.r[r].x, acc.r[r].x), fmaf(c.y, b.r[r].y, acc.r[r].y));
  }
  acc.nl = fmaf(n.x, b.nl, acc.nl);
  acc.nr = fmaf(n.y, b.nr, acc.nr);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    pin(acc.l[r].x);
    pin(acc.l[r].y);
    pin(acc.r[r].x);
    pin(acc.r[r].y);
  }
}

__device__ __forceinline__ void clear(Bins& b) {
#pragma unroll
  for (int r = 0; r < 4; ++r) b.l[r] = b.r[r] = make_float2(0.f, 0.f);
  b.nl = b.nr = 0.f;
}

// row[t + j + 64 r], zero outside [0, L). Each address is formed by itself: where a window starts
// before the row, a negative base and a constant offset must not meet in one instruction, whose
// range check adds them without wrapping.
__device__ __forceinline__ void load_channel(const float* row, int L, int t, int j,
                                             float (&x)[8]) {
  const auto rs = row_rsrc(row, L);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    int i = t + j + 64 * r;
    asm volatile("" : "+v"(i));
    x[r] = bload(rs, i);
  }
}

// z[r] = sum over the node's rows of (left[tl + j + 64 r], right[tr + j + 64 r]); zero outside the
// rows (buffer loads with the hardware range check). The first row is loaded in place.
template <bool ADJ>
__device__ __forceinline__ void load_window(const GraphView& g, int e0, int e1, int tl, int tr,
                                            int j, float2 (&z)[8]) {
  auto row = [&](int e, int& L) {
    const int other = __builtin_amdgcn_readfirstlane(ADJ ? g.out_dst[e] : g.in_src[e]);
    L = __builtin_amdgcn_readfirstlane((int)node_len(g, other));
    return ADJ ? adj_row(g, other) : out_row(g, other);
  };
  if (e0 == e1) {
#pragma unroll
    for (int r = 0; r < 8; ++r) z[r] = make_float2(0.f, 0.f);
    return;
  }
  float x[8], y[8];
  int L;
  const float* p = row(e0, L);
  load_channel(p, L, tl, j, x);
  load_channel(p + g.T, L, tr, j, y);
#pragma unroll
  for (int r = 0; r < 8; ++r) z[r] = make_float2(x[r], y[r]);
  for (int e = e0 + 1; e < e1; ++e) {
    p = row(e, L);
    load_channel(p, L, tl, j, x);
#pragma unroll
    for (int r = 0; r < 8; ++r) z[r].x += x[r];
    load_channel(p + g.T, L, tr, j, x);
#pragma unroll
    for (int r = 0; r < 8; ++r) z[r].y += x[r];
  }
}

__device__ __forceinline__ void store_tile(const GraphView& g, float* y, int Tn, int t0, int j,
                                           const float2 (&v)[8]) {
  // a tile's outputs are elements 19 .. 492 of the transform, those past Tn are dropped
  const int n = min(kHop, Tn - t0);
  const auto yl = row_rsrc(y + t0, n), yr = row_rsrc(y + g.T + t0, n);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    bstore_nt(yl, j + 64 * r - kHalf, v[r].x);
    bstore_nt(yr, j + 64 * r - kHalf, v[r].y);
  }
}

// ---- design ------------------------------------------------------------------------------------

// One block per (node, slot): the taps of both channels, the integer delays and the spectra.
template <int M>
__global__ __launch_bounds__(kBlock) void delay_design_kernel(const float* P, float* taps,
                                                              float2* spec, int32_t* offs) {
  __shared__ double cn[kN], c39[kDelayFir], A[2][20], h[2][20];
  const int node = blockIdx.x, m = blockIdx.y, tid = threadIdx.x;
  const float* p = P + (int64_t)node * delay_row(M);
  for (int i = tid; i < kN; i += kBlock) cn[i] = cospi((double)i / (kN / 2));
  if (tid < kDelayFir) c39[tid] = cospi(2.0 * tid / 39.0);
  if (tid < 40) A[tid / 20][tid % 20] = exp((double)p[(tid / 20 * M + m) * 22 + 2 + tid % 20]);
  __syncthreads();
  if (tid < 40) {
    const int c = tid / 20, j = tid % 20;
    double acc = A[c][0];
    for (int k = 1; k <= kHalf; ++k) acc += 2.0 * A[c][k] * c39[k * j % kDelayFir];
    const double t = (0.5 + 0.5 * cospi((double)j / kHalf)) * (acc / 39.0);
    h[c][j] = t;
    float* out = taps + (int64_t)node * delay_coef(M) + (c * M + m) * kDelayFir + kHalf;
    out[j] = out[-j] = (float)t;
  }
  if (tid < 2) {
    const float* q = p + (tid * M + m) * 22;
    const float kScale = (float)(4410.0 / (2.0 * 3.14159265358979323846));
    const float ph = atan2f(q[1], q[0]);
    const int r = (int)rintf(-ph * kScale);
    const int d = ((r % kDelaySlot) + kDelaySlot) % kDelaySlot;
    offs[(int64_t)node * 2 * M + tid * M + m] = m * kDelaySlot + d;
  }
  __syncthreads();
  float2* sp = spec + (int64_t)node * delay_spec(M) + m * kDelayBins;
  for (int k = tid; k <= kN / 2; k += kBlock) {
    double l = h[0][0], r = h[1][0];
    for (int j = 1; j <= kHalf; ++j) {
      const double c = 2.0 * cn[j * k & (kN - 1)];
      l = fma(h[0][j], c, l);
      r = fma(h[1][j], c, r);
    }
    sp[k] = make_float2((float)(l * (0.5 / kN)), (float)(r * (0.5 / kN)));
  }
}

// ---- forward -----------------------------------------------------------------------------------

// Logical blocks (four neighbouring tiles each) are spread XCD-contiguously, so the slot windows
// of a node's tiles, which overlap over the M x 100 ms of its delays, are read from one L2. Five
// waves per SIMD hide the loads; loading the next slot's window ahead gained nothing.
template <int M>
__global__ __launch_bounds__(kBlock, 4) void delay_fwd_kernel(GraphView g, float* U,
                                                           const float2* spec,
                                                           const int32_t* offs, int node_begin,
                                                           int per_node) {
  __shared__ float2 lds[kWaves][kSlice], w1[kWaves][kW1];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), j = threadIdx.x & 63;
  const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
  const int node = node_begin + lb / per_node;
  const int t0 = (lb % per_node * kWaves + wave) * kHop;
  const int Tn = __builtin_amdgcn_readfirstlane((int)node_len(g, node));
  if (t0 >= Tn) return;  // no block barrier below
  float2* s = lds[wave];
  const int slot = __builtin_amdgcn_readfirstlane(g.param_row[node]);
  const int32_t* d = offs + (int64_t)slot * 2 * M;
  const float2* sp = spec + (int64_t)slot * delay_spec(M);
  const int e0 = __builtin_amdgcn_readfirstlane(g.in_ptr[node]);
  const int e1 = __builtin_amdgcn_readfirstlane(g.in_ptr[node + 1]);
  Twiddles512 tw;
  load_twiddles512(tw, w1[wave], j);
  Bins acc;
  clear(acc);
  float2 z[8];
  for (int m = 0; m < M; ++m) {
    load_window<false>(g, e0, e1, t0 - d[m] - kHalf, t0 - d[M + m] - kHalf, j, z);
    fft512<false>(z, s, tw, j);
    Bins b;
    separate(z, b, s, j);
    multiply_add(b, sp + m * kDelayBins + j, sp[m * kDelayBins + kN / 2], acc);
  }
  join(acc, z, s, j);
  fft512<true>(z, s, tw, j);
  store_tile(g, U + (int64_t)node * 2 * g.T, Tn, t0, j, z);
}

// ---- adjoint -----------------------------------------------------------------------------------

// A block takes one group of tiles of a node. M = 5: its waves take the tiles in turn, all five
// slots each, and their sums are added at the end of the group. M = 20: every wave takes five
// slots of every tile, and the waves add up their parts of the input adjoint (one of them, by
// turns, inverts and stores it). The registers hold the gradient sums of five slots (50), the
// input adjoint's sums (18), the tile's bins (18), the transform, its twiddles and the next
// window (46): 210 with the addresses, two waves per SIMD. A cap at 168 for three waves spilled 34
// of them and took 85 us instead of 60.
template <int M>
__global__ __launch_bounds__(kBlock, 2) void delay_bwd_kernel(GraphView g, float* dU,
                                                              const float2* spec,
                                                              const int32_t* offs, int node_begin,
                                                              int groups, float* part) {
  constexpr int MS = kSlotsPerWave;
  constexpr bool kSplit = M > MS;  // slots dealt to the waves, not tiles
  static_assert(M == MS || M == MS * kWaves, "one wave per tile, or the block's waves");
  __shared__ float2 lds[kWaves][kSlice], other[kWaves][kSlice], w1[kWaves][kW1];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), j = threadIdx.x & 63;
  const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
  const int node = node_begin + lb / groups, group = lb % groups;
  const int m0 = kSplit ? wave * MS : 0;
  float2* const s = lds[wave];
  const int Tn = __builtin_amdgcn_readfirstlane((int)node_len(g, node));
  const int slot = __builtin_amdgcn_readfirstlane(g.param_row[node]);
  const int32_t* d = offs + (int64_t)slot * 2 * M + m0;
  const float2* sp = spec + (int64_t)slot * delay_spec(M) + m0 * kDelayBins;
  const int i0 = __builtin_amdgcn_readfirstlane(g.in_ptr[node]);
  const int i1 = __builtin_amdgcn_readfirstlane(g.in_ptr[node + 1]);
  const int o0 = __builtin_amdgcn_readfirstlane(g.out_ptr[node]);
  const int o1 = __builtin_amdgcn_readfirstlane(g.out_ptr[node + 1]);
  const int tiles = (Tn + kHop - 1) / kHop;  // the node's own
  const int first = group * group_tiles(g.tap_tiles);
  const int last = min(tiles, first + group_tiles(g.tap_tiles));
  Twiddles512 tw;
  load_twiddles512(tw, w1[wave], j);
  float El[MS][5], Er[MS][5];  // 4 Re(Y conj U) of bins j + 64 r, and bin 256 on lane 0
#pragma unroll
  for (int m = 0; m < MS; ++m)
#pragma unroll
    for (int r = 0; r < 5; ++r) El[m][r] = Er[m][r] = 0.f;
  for (int tile = first + (kSplit ? 0 : wave); tile < last; tile += kSplit ? 1 : kWaves) {
    const int t0 = tile * kHop, tw0 = t0 - kHalf;
    Bins u, acc;
    float2 z[8], next[8];
    load_window<false>(g, i0, i1, tw0, tw0, j, z);
    load_window<true>(g, o0, o1, tw0 + d[0], tw0 + d[M], j, next);
    // the tile alone: elements 19 .. 492
    if (j < kHalf) z[0] = make_float2(0.f, 0.f);
    if (j + 64 * 7 >= kHalf + kHop) z[7] = make_float2(0.f, 0.f);
    fft512<false>(z, s, tw, j);
    separate(z, u, s, j);
    clear(acc);
#pragma unroll
    for (int m = 0; m < MS; ++m) {
#pragma unroll
      for (int r = 0; r < 8; ++r) z[r] = next[r];
      if (m + 1 < MS) load_window<true>(g, o0, o1, tw0 + d[m + 1], tw0 + d[M + m + 1], j, next);
      fft512<false>(z, s, tw, j);
      Bins b;
      separate(z, b, s, j);
      multiply_add(b, sp + m * kDelayBins + j, sp[m * kDelayBins + kN / 2], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        El[m][r] = fmaf(b.l[r].x, u.l[r].x, fmaf(b.l[r].y, u.l[r].y, El[m][r]));
        Er[m][r] = fmaf(b.r[r].x, u.r[r].x, fmaf(b.r[r].y, u.r[r].y, Er[m][r]));
      }
      El[m][4] = fmaf(b.nl, u.nl, El[m][4]);
      Er[m][4] = fmaf(b.nr, u.nr, Er[m][4]);
#pragma unroll
      for (int r = 0; r < 5; ++r) {
        pin(El[m][r]);
        pin(Er[m][r]);
      }
    }
    join(acc, z, s, j);
    if constexpr (kSplit) {
#pragma unroll
      for (int r = 0; r < 8; ++r) s[j + 64 * r] = z[r];
      __syncthreads();
      const bool mine = wave == tile % kWaves;
      if (mine) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
          z[r] = cadd(cadd(cadd(lds[0][j + 64 * r], lds[1][j + 64 * r]), lds[2][j + 64 * r]),
                      lds[3][j + 64 * r]);
      }
      __syncthreads();
      if (!mine) continue;
    }
    fft512<true>(z, s, tw, j);
    store_tile(g, dU + (int64_t)node * 2 * g.T, Tn, t0, j, z);
    if (float* ds = source_row(g, node)) {
#pragma unroll
      for (int r = 0; r < 8; ++r) z[r] = make_float2(0.f + z[r].x, 0.f + z[r].y);
      store_tile(g, ds, Tn, t0, j, z);
    }
  }
  // lags of the even parts of the correlations (zeros for a group past the node's end)
  float* out = part + ((int64_t)slot * groups + group) * delay_lags(M);
#pragma unroll
  for (int m = 0; m < MS; ++m) {
    float2 c[5];
#pragma unroll
    for (int r = 0; r < 5; ++r) c[r] = make_float2(El[m][r], Er[m][r]);
    float2(*const buf)[kSlice] = m & 1 ? other : lds;  // the next slot's sum may overlap these reads
    if constexpr (!kSplit) {  // sum over the waves' tiles, one slot at a time
#pragma unroll
      for (int r = 0; r < 5; ++r) buf[wave][j + 64 * r] = c[r];
      __syncthreads();
      if (wave != m % kWaves) continue;
#pragma unroll
      for (int r = 0; r < 5; ++r)
        c[r] = cadd(cadd(cadd(buf[0][j + 64 * r], buf[1][j + 64 * r]), buf[2][j + 64 * r]),
                    buf[3][j + 64 * r]);
    }
    // E_l + i E_r, both real and even
    float2* const own = buf[wave];
    float2 v[8];
    lds_order();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[r] = make_float2(c[r].x * (0.25f / kN), c[r].y * (0.25f / kN));
      at_mirror(own, j)[-72 * r] = v[r];
    }
    if (j == 0)
      own[kN / 2 + kN / 16] = make_float2(c[4].x * (0.25f / kN), c[4].y * (0.25f / kN));
    lds_order();
#pragma unroll
    for (int r = 4; r < 8; ++r) v[r] = at(own, j)[72 * r];
    fft512<true>(v, own, tw, j);
    // A delay past the node's end leaves only lags j <= Tn - 1 - d: where no term exists on either
    // side the sum is exactly 0, not the transform's rounding (which would outweigh the few terms
    // left, whose taps the Hann window has almost closed).
    if (j < 20) {
      out[(m0 + m) * 20 + j] = j > d[m] - Tn ? v[0].x : 0.f;
      out[(M + m0 + m) * 20 + j] = j > d[M + m] - Tn ? v[0].y : 0.f;
    }
  }
}

// Sum the partial lags of one (node, channel-slot) over the groups, in double and in a fixed order
// (12 threads per lag), and map them to the log-magnitudes:
// dL/dlogmag_k = A_k (kappa_k / 39) sum_j cbar[j] v[j] cos(2 pi k j / 39).
template <int M>
__global__ __launch_bounds__(kBlock) void delay_grad_kernel(const float* P, const float* part,
                                                            int groups, float* dP) {
  constexpr int kParts = 12;
  __shared__ double c39[kDelayFir], sums[kParts][20], cb[20];
  const int slot = blockIdx.x, cm = blockIdx.y, tid = threadIdx.x;
  const int j = tid % 20, q = tid / 20;
  if (tid < kDelayFir) c39[tid] = cospi(2.0 * tid / 39.0);
  if (q < kParts) {
    const float* p = part + (int64_t)slot * groups * delay_lags(M) + cm * 20 + j;
    double a = 0.0;
#pragma unroll 4
    for (int gi = q; gi < groups; gi += kParts) a += (double)p[(int64_t)gi * delay_lags(M)];
    sums[q][j] = a;
  }
  __syncthreads();
  if (tid < 20) {
    double a = 0.0;
    for (int i = 0; i < kParts; ++i) a += sums[i][tid];
    // lags j and -j together
    cb[tid] = (tid == 0 ? 1.0 : 2.0) * a * (0.5 + 0.5 * cospi((double)tid / kHalf));
  }
  __syncthreads();
  const float* p = P + (int64_t)slot * delay_row(M) + cm * 22;
  float* d = dP + (int64_t)slot * delay_row(M) + cm * 22;
  if (tid < 2) d[tid] = 0.f;
  if (tid < 20) {
    double acc = 0.0;
    for (int i = 0; i < 20; ++i) acc += cb[i] * c39[tid * i % kDelayFir];
    const double kappa = tid == 0 ? 1.0 : 2.0;
    d[2 + tid] = (float)(exp((double)p[2 + tid]) * kappa / 39.0 * acc);
  }
}

// Straight-through phasor gradient of one (node slot, channel x slot) pair: G into LDS, then Q as
// above, each thread taking the k = 1 + thread, 1 + thread + 256, ... terms; the inner sum over n
// steps the phasor e^(2 pi i k n / N) by multiplication, restarting from an exact value every 256
// steps; per-thread partials are added in a fixed order.
template <int M>
__global__ __launch_bounds__(kBlock) void delay_phasor_grad_kernel(const float* P,
                                                                   const float* taps,
                                                                   const float* R, int64_t Lr,
                                                                   float* dP) {
  constexpr int kRow = delay_row(M);
  __shared__ double G[kDelaySlot];
  __shared__ double2 red[kBlock / 64];
  const int slot = blockIdx.x, cm = blockIdx.y;  // cm = channel * M + slot
  const int c = cm / M, m = cm % M;
  const float* tp = taps + (int64_t)slot * delay_coef(M) + cm * kDelayFir;
  const float* Rc = R + ((int64_t)slot * 2 + c) * Lr + (int64_t)m * kDelaySlot;
  for (int n = threadIdx.x; n < kDelaySlot; n += kBlock) {
    double acc = 0.0;
    for (int j = 0; j < kDelayFir; ++j) acc = fma((double)tp[j], (double)Rc[n + j], acc);
    G[n] = acc;
  }
  __syncthreads();
  const float* q = P + (int64_t)slot * kRow + cm * 22;
  const double zr = q[0], zi = q[1];
  const double lr = 0.5 * log(zr * zr + zi * zi), th = atan2(zi, zr);  // principal log z
  double qr = 0.0, qi = 0.0;
  for (int k = 1 + threadIdx.x; k < kDelaySlot; k += kBlock) {
    double gr = 0.0, gi = 0.0, sr, si;  // the step e^(2 pi i k / N)
    sincospi(2.0 * (double)k / kDelaySlot, &si, &sr);
    for (int n0 = 0; n0 < kDelaySlot; n0 += 256) {
      double wr, wi;  // e^(2 pi i k n0 / N), exactly
      sincospi(2.0 * (double)(((int64_t)k * n0) % kDelaySlot) / kDelaySlot, &wi, &wr);
      const int n1 = min(n0 + 256, kDelaySlot);
      for (int n = n0; n < n1; ++n) {
        gr = fma(G[n], wr, gr);
        gi = fma(G[n], wi, gi);
        const double t = wr * sr - wi * si;
        wi = fma(wr, si, wi * sr);
        wr = t;
      }
    }
    // k z^(k - 1) = k exp((k - 1) log z)
    double sn, cs;
    sincos((double)(k - 1) * th, &sn, &cs);
    const double mag = (double)k * exp((double)(k - 1) * lr);
    const double ar = mag * cs, ai = mag * sn;
    qr += ar * gr - ai * gi;
    qi += ar * gi + ai * gr;
  }
  qr = wave_sum(qr);
  qi = wave_sum(qi);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = make_double2(qr, qi);
  __syncthreads();
  if (threadIdx.x == 0) {
    double sr = 0.0, si = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) {
      sr += red[w].x;
      si += red[w].y;
    }
    float* d = dP + (int64_t)slot * kRow + cm * 22;
    d[0] = (float)(sr / kDelaySlot);
    d[1] = (float)(-si / kDelaySlot);
  }
}

// Optimiser-side treatment of the phasor gradients (the paper normalises each delay's gradient and
// pulls z towards the unit circle, without constants): every (re z, im z) gradient pair is scaled
// to unit length (a zero pair stays zero), then the gradient of weight * (|z| - 1)^2,
// 2 weight (|z| - 1) z / |z| (zero at z = 0), is added. One thread per phasor.
__global__ __launch_bounds__(kBlock) void delay_phasor_regularise_kernel(int M, int n,
                                                                         const float* P, float* dP,
                                                                         float weight) {
  const int i = blockIdx.x * kBlock + threadIdx.x;  // phasor index: node * 2 M + c * M + m
  if (i >= n * 2 * M) return;
  const int64_t o = (int64_t)i * 22;  // rows are [channel][slot][22], contiguous per node
  const double gr = dP[o], gi = dP[o + 1];
  const double gn = sqrt(gr * gr + gi * gi);
  const double zr = P[o], zi = P[o + 1];
  const double r = sqrt(zr * zr + zi * zi);
  const double s = r > 0.0 ? 2.0 * (double)weight * (r - 1.0) / r : 0.0;
  dP[o] = (float)((gn > 0.0 ? gr / gn : 0.0) + s * zr);
  dP[o + 1] = (float)((gn > 0.0 ? gi / gn : 0.0) + s * zi);
}

}  // namespace

int delay_groups(int64_t T, int tap_tiles) {
  const int64_t span = (int64_t)kHop * group_tiles(tap_tiles);
  return (int)((T + span - 1) / span);
}

// Calls body(std::integral_constant<int, M>) for the slot counts the library supports.
template <typename F>
hipError_t with_slots(int M, F&& body) {
  if (M == kDelayTaps) return body(std::integral_constant<int, kDelayTaps>{});
  if (M == kDelayTapsLong) return body(std::integral_constant<int, kDelayTapsLong>{});
  return hipErrorInvalidValue;
}

hipError_t launch_delay_design(int M, const float* P, int n, float* taps, float2* spec,
                               int32_t* offs, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  return with_slots(M, [&](auto m) {
    delay_design_kernel<decltype(m)::value><<<dim3(n, M), kBlock, 0, s>>>(P, taps, spec, offs);
    return hipGetLastError();
  });
}

hipError_t launch_delay_fwd(int M, const GraphView& g, float* U, const float2* spec,
                            const int32_t* offs, int node_begin, int n_nodes, hipStream_t s) {
  const int tiles = (int)((g.T + kHop - 1) / kHop), per_node = (tiles + kWaves - 1) / kWaves;
  return with_slots(M, [&](auto m) {
    delay_fwd_kernel<decltype(m)::value><<<(unsigned)(per_node * n_nodes), kBlock, 0, s>>>(
        g, U, spec, offs, node_begin, per_node);
    return hipGetLastError();
  });
}

hipError_t launch_delay_bwd(int M, const GraphView& g, float* dU, const float2* spec,
                            const int32_t* offs, int node_begin, int n_nodes, float* part,
                            hipStream_t s) {
  const int groups = delay_groups(g.T, g.tap_tiles);
  return with_slots(M, [&](auto m) {
    delay_bwd_kernel<decltype(m)::value><<<(unsigned)(groups * n_nodes), kBlock, 0, s>>>(
        g, dU, spec, offs, node_begin, groups, part);
    return hipGetLastError();
  });
}

hipError_t launch_delay_grad(int M, const float* P, const float* part, int n, int groups,
                             float* dP, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  return with_slots(M, [&](auto m) {
    constexpr int kM = decltype(m)::value;
    delay_grad_kernel<kM><<<dim3(n, 2 * kM), kBlock, 0, s>>>(P, part, groups, dP);
    return hipGetLastError();
  });
}

hipError_t launch_delay_phasor_regularise(int M, int n, const float* P, float* dP, float weight,
                                          hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int phasors = n * 2 * M;
  delay_phasor_regularise_kernel<<<(phasors + kBlock - 1) / kBlock, kBlock, 0, s>>>(M, n, P, dP,
                                                                                   weight);
  return hipGetLastError();
}

hipError_t launch_delay_phasor_grad(int M, const float* P, const float* taps, const float* R,
                                    int n, float* dP, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  return with_slots(M, [&](auto m) {
    constexpr int kM = decltype(m)::value;
    delay_phasor_grad_kernel<kM><<<dim3(n, 2 * kM), kBlock, 0, s>>>(P, taps, R,
                                                                    delay_sur_len(kM), dP);
    return hipGetLastError();
  });
}

}  // namespace grafx

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
// Filtering: overlap-save on 512-point transforms, 474 outputs a tile. A wave takes two neighbouring
// tiles of one channel, which ride in one complex transform (tile + i next tile): a slot's windows
// (the input read at the slot's delay) are transformed, their bins 0 .. 256 separated into the two
// tiles (bins k and -k: one exchange) and multiplied by the slot's real spectrum; the slots'
// products are summed in registers, and one inverse transform gives both tiles. M + 1 transforms of
// 512 points replace 39 M multiply-adds a sample. Bound by instruction issue: 24 nodes, T = 2^17,
// M = 5: 33 us, 47 us as a direct form.
// The two channels must not share a transform: its rounding is relative to the larger of the
// signals that ride in it, so a channel 60 dB below the other would keep 4 digits, one 120 dB below
// it none, and a silent one would receive the other's rounding (34 us forward and 60 us backward,
// packed that way; with each channel scaled by a power of two of its own 35 and 84 us). With
// neighbouring tiles an output's rounding is relative to the samples of its own channel within
// 22 ms, about 2e-7 of the largest of them.
// Adjoint: the input adjoint is the same sum over windows of the output adjoint read at plus the
// delays. The same windows' spectra Y give the tap gradients: with U the spectrum of the
// zero-padded input tile, sum_s ybar_c[s + d + j] u_c[s] is the inverse transform of Y conj U,
// and since the filters are even only its even part enters, whose spectrum is Re(Y conj U). That is
// summed over a wave's tiles in registers and inverted once per group. One launch (M + 2 transforms
// for two tiles of a channel) replaces 156 M multiply-adds per stereo sample: 65 us, 101 us as two
// direct-form launches.
// What only a direct sum gives is kept: an output that depends on zeros alone is an exact zero, and
// where a transform meets an infinity, a NaN or an overflow, its two tiles are summed directly.
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
constexpr int kReach = kHalf - 1;           // farthest tap that is not 0 (the Hann window's ends are)
constexpr int kWaves = kBlock / 64;
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

// Bins 0 .. 256 of the two tiles a and b of a window, doubled: lane j holds k = j + 64 r (r < 4), and
// lane 0 also bin 256 (real for both; the other lanes' value is not used).
struct Bins {
  float2 a[4], b[4];
  float na, nb;
};

// Element e of a spectrum in a slice sits at e + e / 8; element 512 stands for element 0.
__device__ __forceinline__ float2* at(float2* s, int j) { return s + j + (j >> 3); }  // + 64 r: [72 r]
__device__ __forceinline__ float2* at_mirror(float2* s, int j) {  // 512 - j - 64 r: [-72 r]
  return s + (kN - j) + ((kN - j) >> 3);
}

// From Z = FFT(a + i b): 2 A[k] = Z[k] + conj Z[-k], 2 B[k] = -i (Z[k] - conj Z[-k]).
__device__ __forceinline__ void separate(const float2 (&z)[8], Bins& b, float2* s, int j) {
  lds_order();
#pragma unroll
  for (int r = 4; r < 8; ++r) at(s, j)[72 * r] = z[r];
  if (j == 0) s[kN + kN / 8] = z[0];
  lds_order();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float2 m = at_mirror(s, j)[-72 * r];
    b.a[r] = make_float2(z[r].x + m.x, z[r].y - m.y);
    b.b[r] = make_float2(z[r].y + m.y, m.x - z[r].x);
  }
  b.na = 2.f * z[4].x;
  b.nb = 2.f * z[4].y;
  lds_order();
}

// The spectrum of a + i b from bins 0 .. 256 of both: v[k] = A + i B and v[-k] = conj A + i conj B.
__device__ __forceinline__ void join(const Bins& b, float2 (&v)[8], float2* s, int j) {
  lds_order();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    v[r] = make_float2(b.a[r].x - b.b[r].y, b.a[r].y + b.b[r].x);
    at_mirror(s, j)[-72 * r] = make_float2(b.a[r].x + b.b[r].y, b.b[r].x - b.a[r].y);
  }
  if (j == 0) s[kN / 2 + kN / 16] = make_float2(b.na, b.nb);
  lds_order();
#pragma unroll
  for (int r = 4; r < 8; ++r) v[r] = at(s, j)[72 * r];
  lds_order();
}

// Keeps the compiler from moving the computation of a value past this point (sunk to their next
// use, the sums of a slot would keep the slot's whole spectrum in registers until then).
__device__ __forceinline__ void pin(float& x) { asm volatile("" : "+v"(x)); }

// acc += spectrum x bins; sp: the slot's spectrum for the channel, this lane's bin j and on, n: bin 256
__device__ __forceinline__ void multiply_add(const Bins& b, const float* sp, float n, Bins& acc) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float c = sp[64 * r];
    acc.a[r] = make_float2(fmaf(c, b.a[r].x, acc.a[r].x), fmaf(c, b.a[r].y, acc.a[r].y));
    acc.b[r] = make_float2(fmaf(c, b.b[r].x, acc.b[r].x), fmaf(c, b.b[r].y, acc.b[r].y));
  }
  acc.na = fmaf(n, b.na, acc.na);
  acc.nb = fmaf(n, b.nb, acc.nb);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    pin(acc.a[r].x);
    pin(acc.a[r].y);
    pin(acc.b[r].x);
    pin(acc.b[r].y);
  }
}

__device__ __forceinline__ void clear(Bins& b) {
#pragma unroll
  for (int r = 0; r < 4; ++r) b.a[r] = b.b[r] = make_float2(0.f, 0.f);
  b.na = b.nb = 0.f;
}

// row[t + j + 64 r], zero outside [0, L). Each address is formed by itself: where a window starts
// before the row, a negative base and a constant offset must not meet in one instruction, whose
// range check adds them without wrapping.
__device__ __forceinline__ void load_row(const float* row, int L, int t, int j, float (&x)[8]) {
  const auto rs = row_rsrc(row, L);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    int i = t + j + 64 * r;
    asm volatile("" : "+v"(i));
    x[r] = bload(rs, i);
  }
}

// z[r] = sum over the node's rows, in channel c, of (x[t + j + 64 r], x[t + kHop + j + 64 r]); zero
// outside the rows (buffer loads with the hardware range check). The first row is loaded in place.
template <bool ADJ>
__device__ __forceinline__ void load_window(const GraphView& g, int e0, int e1, int c, int t, int j,
                                            float2 (&z)[8]) {
  auto row = [&](int e, int& L) {
    const int other = __builtin_amdgcn_readfirstlane(ADJ ? g.out_dst[e] : g.in_src[e]);
    L = __builtin_amdgcn_readfirstlane((int)node_len(g, other));
    return (ADJ ? adj_row(g, other) : out_row(g, other)) + c * g.T;
  };
  if (e0 == e1) {
#pragma unroll
    for (int r = 0; r < 8; ++r) z[r] = make_float2(0.f, 0.f);
    return;
  }
  float x[8], y[8];
  int L;
  const float* p = row(e0, L);
  load_row(p, L, t, j, x);
  load_row(p, L, t + kHop, j, y);
#pragma unroll
  for (int r = 0; r < 8; ++r) z[r] = make_float2(x[r], y[r]);
  for (int e = e0 + 1; e < e1; ++e) {
    p = row(e, L);
    load_row(p, L, t, j, x);
#pragma unroll
    for (int r = 0; r < 8; ++r) z[r].x += x[r];
    load_row(p, L, t + kHop, j, x);
#pragma unroll
    for (int r = 0; r < 8; ++r) z[r].y += x[r];
  }
}

// The tiles at t0 and t0 + kHop into a channel's row: elements 19 .. 492 of each, those past Tn are
// dropped.
__device__ __forceinline__ void store_tiles(float* y, int Tn, int t0, int j, const float2 (&v)[8]) {
  y = scalar_ptr(y + t0);  // kept scalar, or a store would loop over the lanes' descriptors
  const int n = __builtin_amdgcn_readfirstlane(Tn - t0);
  const auto ya = row_rsrc(y, min(kHop, n));
  const auto yb = row_rsrc(y + kHop, min(kHop, max(0, n - kHop)));
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    bstore_nt(ya, j + 64 * r - kHalf, v[r].x);
    bstore_nt(yb, j + 64 * r - kHalf, v[r].y);
  }
}

// ---- what a direct sum gives -------------------------------------------------------------------

// Whether the two tiles' parts of a window hold anything but zeros.
struct Live {
  bool a, b;
};
__device__ __forceinline__ Live live(const float2 (&z)[8]) {
  unsigned a = 0, b = 0;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    a |= __float_as_uint(z[r].x);
    b |= __float_as_uint(z[r].y);
  }
  return {__any(a << 1) != 0, __any(b << 1) != 0};
}

// The bins of a part that is all zero are zero, not the other part's rounding (times a signal of any
// level, that would be a gradient where there is none).
__device__ __forceinline__ void clear_dead(const Live& l, Bins& b) {
  if (!l.a) {
#pragma unroll
    for (int r = 0; r < 4; ++r) b.a[r] = make_float2(0.f, 0.f);
    b.na = 0.f;
  }
  if (!l.b) {
#pragma unroll
    for (int r = 0; r < 4; ++r) b.b[r] = make_float2(0.f, 0.f);
    b.nb = 0.f;
  }
}

// What is known of the zeros in the windows of two tiles. reached: in some slot's windows they are too
// few for a run as long as the filter (37, of which 19 would lie in one of the 64-sample words), so
// every output depends on something else, as nearly always. odd: some window holds zeros inside the
// signal of Tn samples; if not, its zeros are the samples before the start or past the end. live: some
// window holds anything else.
struct Zeros {
  bool reached = false, odd = false, live = false;
  // z: the window whose first tile starts at sample t. False if it is all zero.
  __device__ __forceinline__ bool add(const float2 (&z)[8], int t, int Tn) {
    if (reached) return true;
    float m = INFINITY;
#pragma unroll
    for (int i = 0; i < 8; ++i) m = fminf(fminf(fabsf(z[i].x), fabsf(z[i].y)), m);
    if (__all(m > 0.f)) return reached = live = true;
    int n = 0, most = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int a = __popcll(__ballot(z[i].x == 0.f)), b = __popcll(__ballot(z[i].y == 0.f));
      n += a + b;
      most = max(most, max(a, b));
    }
    reached = most <= kReach;
    auto outside = [&](int a) { return min(max(-a, 0), kN) + min(max(a + kN - Tn, 0), kN); };
    odd = odd || n != outside(t) + outside(t + kHop);
    const bool any = n != 2 * kN;
    live = live || any;
    return any;
  }
};

// Which samples of the windows of two tiles are not zero, over all slots: words 0 .. 7 for the first
// tile, 8 .. 15 for the second, bit j of word r for element j + 64 r. Reads the windows again.
template <bool ADJ, int M>
__device__ __forceinline__ void see(const GraphView& g, int e0, int e1, int c, int t0, int j,
                                    const int32_t* d, uint64_t* words) {
  uint64_t mine = 0;
#pragma unroll 1
  for (int m = 0; m < M; ++m) {
    const int lag = d[c * M + m];
    float2 x[8];
    load_window<ADJ>(g, e0, e1, c, t0 - kHalf + (ADJ ? lag : -lag), j, x);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint64_t a = __ballot(x[i].x != 0.f), b = __ballot(x[i].y != 0.f);
      mine |= j == i ? a : j == 8 + i ? b : 0;
    }
  }
  lds_order();
  if (j < 16) words[j] = mine;
  lds_order();
}

// Whether any of the elements e - 18 .. e + 18 that output e = j + 64 r depends on was seen.
__device__ __forceinline__ bool reached(const uint64_t* w, int r, int j) {
  const int i = r - (j < kReach), sh = (j + 64 - kReach) & 63;  // of element e - 18
  const uint64_t lo = i >= 0 ? w[i >= 0 ? i : 0] : 0, hi = i < 7 ? w[i < 7 ? i + 1 : 7] : 0;
  return (((lo >> sh) | (hi << 1 << (63 - sh))) & ((1ull << (2 * kReach + 1)) - 1)) != 0;
}

// The tiles' samples as direct sums over a channel c: taps and d (delays) of the node, both channels.
// Rare, so plain.
template <bool ADJ, int M>
__device__ __forceinline__ void direct_samples(const GraphView& g, int e0, int e1, int c, int t0,
                                               int j, const float* taps, const int32_t* d,
                                               float2 (&z)[8]) {
#pragma unroll
  for (int r = 0; r < 8; ++r) z[r] = make_float2(0.f, 0.f);
#pragma unroll 1
  for (int q = 0; q < M * kDelayFir; ++q) {
    const int m = q / kDelayFir, i = q - m * kDelayFir, lag = d[c * M + m] + i - kHalf;
    float2 x[8];
    load_window<ADJ>(g, e0, e1, c, t0 - kHalf + (ADJ ? lag : -lag), j, x);
    const float k = taps[(c * M + m) * kDelayFir + i];
#pragma unroll
    for (int r = 0; r < 8; ++r) z[r] = make_float2(fmaf(k, x[r].x, z[r].x), fmaf(k, x[r].y, z[r].y));
  }
}

// What the tiles' samples in the wave's slice (element e at e) still need: direct sums if the transform
// met an infinity or NaN or overflowed, exact zeros where only zeros are reached. A function of its own
// and not inlined: the few waves that come here would otherwise cost every wave scalar registers (72
// spilled; the adjoint 73 instead of 65 us at the sizes above). kernarg: the kernel's arguments, of which
// the graph is the first.
using Slice = __attribute__((address_space(3))) float2;

template <bool ADJ, int M>
__device__ __attribute__((noinline, cold)) void rare_samples(const GraphView* kernarg, int node,
                                                             int c, int t0, const float* taps,
                                                             const int32_t* d, bool direct,
                                                             Slice* slice) {
  GraphView g = *kernarg;  // the same in every lane, like all arguments: kept scalar
  auto scalar = [](auto& p) { p = scalar_ptr(p); };
  scalar(g.in_ptr), scalar(g.in_src), scalar(g.out_ptr), scalar(g.out_dst), scalar(g.len);
  scalar(g.S), scalar(g.U), scalar(g.dY), scalar(g.dU);
  g.T = __builtin_amdgcn_readfirstlane((int)g.T);
  g.K = __builtin_amdgcn_readfirstlane(g.K);
  g.out_begin = __builtin_amdgcn_readfirstlane(g.out_begin);
  node = __builtin_amdgcn_readfirstlane(node);
  c = __builtin_amdgcn_readfirstlane(c);
  t0 = __builtin_amdgcn_readfirstlane(t0);
  taps = scalar_ptr(taps);
  d = scalar_ptr(d);
  const int j = threadIdx.x & 63;
  const int32_t* ptr = ADJ ? g.out_ptr : g.in_ptr;
  const int e0 = __builtin_amdgcn_readfirstlane(ptr[node]);
  const int e1 = __builtin_amdgcn_readfirstlane(ptr[node + 1]);
  float2* const s = (float2*)slice;
  if (direct) {
    float2 z[8];
    direct_samples<ADJ, M>(g, e0, e1, c, t0, j, taps, d, z);
#pragma unroll
    for (int r = 0; r < 8; ++r) s[j + 64 * r] = z[r];
  } else {
    uint64_t* const words = reinterpret_cast<uint64_t*>(s + kN);
    see<ADJ, M>(g, e0, e1, c, t0, j, d, words);
#pragma unroll 1
    for (int r = 0; r < 8; ++r) {
      if (!reached(words, r, j)) s[j + 64 * r].x = 0.f;
      if (!reached(words + 8, r, j)) s[j + 64 * r].y = 0.f;
    }
  }
  lds_order();
}

// The tiles' samples from their bins. Outputs that depend on zeros only are exact zeros; a transform
// that met an infinity or NaN, or overflowed, gives way to the direct sums.
template <bool ADJ, int M>
__device__ __forceinline__ void tile_samples(int node, int c, int t0, int Tn, int j, const float* taps,
                                             const int32_t* d, const Bins& acc, const Zeros& zeros,
                                             float2* s, const Twiddles512& tw, float2 (&z)[8]) {
  join(acc, z, s, j);
  fft512<true>(z, s, tw, j);
  float t = 0.f;
#pragma unroll
  for (int r = 0; r < 8; ++r) t = fmaf(z[r].x, 0.f, fmaf(z[r].y, 0.f, t));
  const bool direct = __any(t != t);
  if (!direct && zeros.reached) return;
  if (!direct && !zeros.live) {
#pragma unroll
    for (int r = 0; r < 8; ++r) z[r] = make_float2(0.f, 0.f);
    return;
  }
  if (!direct && !zeros.odd) {  // reached from the signal's start or end on
    int nearest = d[c * M];
    for (int m = 1; m < M; ++m) nearest = min(nearest, d[c * M + m]);
    // the first element that is not reached (adjoint), or the first that is
    const int e = ADJ ? Tn - t0 + kHalf + kReach - nearest : nearest - t0 + kHalf - kReach;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int i = j + 64 * r;
      if (ADJ ? i >= e : i < e) z[r].x = 0.f;
      if (ADJ ? i + kHop >= e : i + kHop < e) z[r].y = 0.f;
    }
    return;
  }
  lds_order();
#pragma unroll
  for (int r = 0; r < 8; ++r) s[j + 64 * r] = z[r];
  lds_order();
  rare_samples<ADJ, M>((const GraphView*)__builtin_amdgcn_kernarg_segment_ptr(), node, c, t0, taps, d,
                       direct, (Slice*)s);
#pragma unroll
  for (int r = 0; r < 8; ++r) z[r] = s[j + 64 * r];
  lds_order();
}

// ---- balance of the cross-spectra --------------------------------------------------------------
// The cross-spectra of the two channels, real and even, do ride in one inverse transform. The smaller
// one is brought up to the exponent of the larger by a power of two, which is exact, and taken back
// afterwards; one that is all zero, or was cleared for an infinity or NaN, is left out.

constexpr unsigned kInfinity = 0x7F800000u, kOne = 127u << 23;

// Largest magnitude over the wave, as the bits of the float without its sign (uniform).
__device__ __forceinline__ unsigned level(const float (&x)[5]) {
  unsigned v = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i) v = max(v, __float_as_uint(x[i]) & 0x7FFFFFFFu);
  // rows of 16 lanes by DPP moves (lane ^ 1, ^ 2, mirrored within 8 and 16), then the four rows
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));
  auto row = [&](int i) { return (unsigned)__builtin_amdgcn_readlane((int)v, i); };
  return max(max(row(0), row(16)), max(row(32), row(48)));
}

struct Balance {
  float up, down;  // before and after the transform
  bool finite;
  __device__ __forceinline__ Balance(unsigned own, unsigned other)
      : up(0.f), down(0.f), finite(own < kInfinity) {
    if (!own || !finite) return;
    const int d = other < kInfinity ? (int)(other >> 23) - (int)(own >> 23) : 0;
    const unsigned k = (unsigned)min(max(d, 0), 126) << 23;
    up = __uint_as_float(kOne + k);
    down = __uint_as_float(kOne - k);
  }
  __device__ __forceinline__ float before(float x) const { return up == 0.f ? 0.f : x * up; }
  __device__ __forceinline__ float after(float x) const { return finite ? x * down : NAN; }
};

// ---- design ------------------------------------------------------------------------------------

// One block per (node, slot): the taps of both channels, the integer delays and the spectra.
template <int M>
__global__ __launch_bounds__(kBlock) void delay_design_kernel(const float* P, const int32_t* rows,
                                                              float* taps, float* spec,
                                                              int32_t* offs) {
  __shared__ double cn[kN], c39[kDelayFir], A[2][20], h[2][20];
  const int node = rows ? rows[blockIdx.x] : (int)blockIdx.x, m = blockIdx.y, tid = threadIdx.x;
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
  float* sp = spec + (int64_t)blockIdx.x * delay_spec(M) + 2 * m * kDelayBins;
  for (int k = tid; k <= kN / 2; k += kBlock) {
    double l = h[0][0], r = h[1][0];
    for (int j = 1; j <= kHalf; ++j) {
      const double c = 2.0 * cn[j * k & (kN - 1)];
      l = fma(h[0][j], c, l);
      r = fma(h[1][j], c, r);
    }
    sp[k] = (float)(l * (0.5 / kN));
    sp[kDelayBins + k] = (float)(r * (0.5 / kN));
  }
}

// ---- forward -----------------------------------------------------------------------------------

// Logical blocks (four neighbouring tiles each, wave w takes channel w & 1) are spread XCD-contiguously,
// so the slot windows of a node's tiles, which overlap over the M x 100 ms of its delays, are read from
// one L2. Five waves per SIMD hide the loads; loading the next slot's window ahead gained nothing.
template <int M>
__global__ __launch_bounds__(kBlock, 4) void delay_fwd_kernel(GraphView g, float* U,
                                                              const float* taps, const float* spec,
                                                              bool spec_by_node,
                                                              const int32_t* offs, int node_begin,
                                                              int per_node) {
  __shared__ float2 lds[kWaves][kSlice], w1[kWaves][kW1];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), j = threadIdx.x & 63;
  const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
  const int node = node_begin + lb / per_node, c = wave & 1;
  const int t0 = (lb % per_node * kWaves + (wave & ~1)) * kHop;
  const int Tn = __builtin_amdgcn_readfirstlane((int)node_len(g, node));
  if (t0 >= Tn) return;  // no block barrier below
  float2* s = lds[wave];
  const int slot = __builtin_amdgcn_readfirstlane(g.param_row[node]);
  const int32_t* d = offs + (int64_t)slot * 2 * M;
  const float* sp =
      spec + (int64_t)(spec_by_node ? node - node_begin : slot) * delay_spec(M) + c * kDelayBins;
  const int e0 = __builtin_amdgcn_readfirstlane(g.in_ptr[node]);
  const int e1 = __builtin_amdgcn_readfirstlane(g.in_ptr[node + 1]);
  Twiddles512 tw;
  load_twiddles512(tw, w1[wave], j);
  Bins acc;
  clear(acc);
  Zeros zeros;
  float2 z[8];
  for (int m = 0; m < M; ++m) {
    const int t = t0 - d[c * M + m] - kHalf;
    load_window<false>(g, e0, e1, c, t, j, z);
    if (!zeros.add(z, t, Tn)) continue;
    fft512<false>(z, s, tw, j);
    Bins b;
    separate(z, b, s, j);
    multiply_add(b, sp + 2 * m * kDelayBins + j, sp[2 * m * kDelayBins + kN / 2], acc);
  }
  tile_samples<false, M>(node, c, t0, Tn, j, taps + (int64_t)slot * delay_coef(M), d, acc, zeros,
                         s, tw, z);
  store_tiles(U + ((int64_t)node * 2 + c) * g.T, Tn, t0, j, z);
}

// ---- adjoint -----------------------------------------------------------------------------------

// A block takes one group of tiles of a node, wave w channel w & 1 of it. M = 5: the two waves of a
// channel take the pairs of tiles in turn, all five slots each, and their sums are added at the end of
// the group. M = 20: each of them takes ten slots of every pair, and they add up their parts of the
// input adjoint (one of them, by turns, inverts and stores it). The registers hold the gradient sums of
// the slots (25 or 50), the input adjoint's sums (18), the tiles' bins (18), the transform, its twiddles
// and the next window (46): 194 or 222 with the addresses, two waves per SIMD. Three spill.
template <int M>
__global__ __launch_bounds__(kBlock, 2) void delay_bwd_kernel(GraphView g, float* dU,
                                                              const float* taps, const float* spec,
                                                              const int32_t* offs, int node_begin,
                                                              int groups, float* part) {
  constexpr bool kSplit = M > 5;  // slots dealt to the two waves of a channel, not pairs of tiles
  constexpr int MS = kSplit ? M / 2 : M;
  static_assert(kWaves == 4, "two waves a channel");
  __shared__ float2 lds[kWaves][kSlice], other[kWaves][kSlice], w1[kWaves][kW1];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), j = threadIdx.x & 63;
  const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
  const int node = node_begin + lb / groups, group = lb % groups;
  const int c = wave & 1, half = wave >> 1, m0 = kSplit ? half * MS : 0;
  float2* const s = lds[wave];
  const int Tn = __builtin_amdgcn_readfirstlane((int)node_len(g, node));
  const int slot = __builtin_amdgcn_readfirstlane(g.param_row[node]);
  const int32_t* nd = offs + (int64_t)slot * 2 * M;  // the node's delays, and this wave's
  const int32_t* d = nd + c * M + m0;
  const float* sp = spec + (int64_t)slot * delay_spec(M) + (2 * m0 + c) * kDelayBins;
  const int i0 = __builtin_amdgcn_readfirstlane(g.in_ptr[node]);
  const int i1 = __builtin_amdgcn_readfirstlane(g.in_ptr[node + 1]);
  const int o0 = __builtin_amdgcn_readfirstlane(g.out_ptr[node]);
  const int o1 = __builtin_amdgcn_readfirstlane(g.out_ptr[node + 1]);
  const int tiles = (Tn + kHop - 1) / kHop;  // the node's own
  const int first = group * group_tiles(g.tap_tiles);
  const int last = min(tiles, first + group_tiles(g.tap_tiles));
  Twiddles512 tw;
  load_twiddles512(tw, w1[wave], j);
  float E[MS][5];  // 4 Re(Y conj U) of bins j + 64 r, and bin 256 on lane 0
#pragma unroll
  for (int m = 0; m < MS; ++m)
#pragma unroll
    for (int r = 0; r < 5; ++r) E[m][r] = 0.f;
  for (int tile = first + (kSplit ? 0 : 2 * half); tile < last; tile += kSplit ? 2 : kWaves) {
    const int t0 = tile * kHop, tw0 = t0 - kHalf;
    Bins u, acc;
    float2 z[8], next[8];
    load_window<false>(g, i0, i1, c, tw0, j, z);
    load_window<true>(g, o0, o1, c, tw0 + d[0], j, next);
    // the tiles alone: elements 19 .. 492
    if (j < kHalf) z[0] = make_float2(0.f, 0.f);
    if (j + 64 * 7 >= kHalf + kHop) z[7] = make_float2(0.f, 0.f);
    const Live ul = live(z);
    fft512<false>(z, s, tw, j);
    separate(z, u, s, j);
    clear_dead(ul, u);
    clear(acc);
    Zeros zeros;
#pragma unroll
    for (int m = 0; m < MS; ++m) {
#pragma unroll
      for (int r = 0; r < 8; ++r) z[r] = next[r];
      if (m + 1 < MS) load_window<true>(g, o0, o1, c, tw0 + d[m + 1], j, next);
      zeros.add(z, tw0 + d[m], Tn);
      const Live yl = live(z);
      if (!yl.a && !yl.b) continue;
      fft512<false>(z, s, tw, j);
      Bins b;
      separate(z, b, s, j);
      clear_dead(yl, b);
      multiply_add(b, sp + 2 * m * kDelayBins + j, sp[2 * m * kDelayBins + kN / 2], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        E[m][r] = fmaf(b.a[r].x, u.a[r].x, fmaf(b.a[r].y, u.a[r].y, E[m][r]));
        E[m][r] = fmaf(b.b[r].x, u.b[r].x, fmaf(b.b[r].y, u.b[r].y, E[m][r]));
      }
      E[m][4] = fmaf(b.na, u.na, fmaf(b.nb, u.nb, E[m][4]));
#pragma unroll
      for (int r = 0; r < 5; ++r) pin(E[m][r]);
    }
    if constexpr (kSplit) {  // sums and zeros over both waves' slots
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[j + 64 * r] = acc.a[r];
        s[kN / 2 + j + 64 * r] = acc.b[r];
      }
      if (j == 0) {
        s[kN] = make_float2(acc.na, acc.nb);
        s[kN + 1] = make_float2(zeros.reached ? 1.f : 0.f, zeros.odd ? 1.f : 0.f);
        s[kN + 2] = make_float2(zeros.live ? 1.f : 0.f, 0.f);
      }
      __syncthreads();
      const bool mine = half == (tile >> 1 & 1);
      if (mine) {
        auto sum = [&](int e) { return cadd(lds[c][e], lds[c + 2][e]); };
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc.a[r] = sum(j + 64 * r);
          acc.b[r] = sum(kN / 2 + j + 64 * r);
        }
        const float2 n = sum(kN), f = sum(kN + 1);
        acc.na = n.x;
        acc.nb = n.y;
        zeros.reached = __builtin_amdgcn_readfirstlane((int)f.x) != 0;
        zeros.odd = __builtin_amdgcn_readfirstlane((int)f.y) != 0;
        zeros.live = __builtin_amdgcn_readfirstlane((int)sum(kN + 2).x) != 0;
      }
      __syncthreads();
      if (!mine) continue;
    }
    tile_samples<true, M>(node, c, t0, Tn, j, taps + (int64_t)slot * delay_coef(M), nd, acc, zeros,
                          s, tw, z);
    store_tiles(dU + ((int64_t)node * 2 + c) * g.T, Tn, t0, j, z);
    if (float* ds = source_row(g, node)) {
#pragma unroll
      for (int r = 0; r < 8; ++r) z[r] = make_float2(0.f + z[r].x, 0.f + z[r].y);
      store_tiles(ds + c * g.T, Tn, t0, j, z);
    }
  }
  // lags of the even parts of the correlations (zeros for a group past the node's end)
  float* out = part + ((int64_t)slot * groups + group) * delay_lags(M);
#pragma unroll
  for (int m = 0; m < MS; ++m) {
    float2(*const buf)[kSlice] = m & 1 ? other : lds;  // the next slot's sums may overlap these reads
#pragma unroll
    for (int r = 0; r < 5; ++r) reinterpret_cast<float*>(buf[wave])[j + 64 * r] = E[m][r];
    __syncthreads();
    // M = 5: one wave adds up all; M = 20: either wave of the two that hold the slot
    if (kSplit ? c != (m & 1) : wave != m % kWaves) continue;
    float l[5], r[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      auto of = [&](int w) { return reinterpret_cast<const float*>(buf[w])[j + 64 * i]; };
      l[i] = kSplit ? of(wave & ~1) : of(0) + of(2);
      r[i] = kSplit ? of(wave | 1) : of(1) + of(3);
    }
    if (j != 0) l[4] = r[4] = 0.f;
    const unsigned ll = level(l), lr = level(r);
    const Balance kl(ll, lr), kr(lr, ll);
    // E_l + i E_r, both real and even
    float2* const own = buf[wave];
    float2 v[8];
    lds_order();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = make_float2(kl.before(l[i]) * (0.25f / kN), kr.before(r[i]) * (0.25f / kN));
      at_mirror(own, j)[-72 * i] = v[i];
    }
    if (j == 0)
      own[kN / 2 + kN / 16] =
          make_float2(kl.before(l[4]) * (0.25f / kN), kr.before(r[4]) * (0.25f / kN));
    lds_order();
#pragma unroll
    for (int i = 4; i < 8; ++i) v[i] = at(own, j)[72 * i];
    fft512<true>(v, own, tw, j);
    // A delay past the node's end leaves only lags j <= Tn - 1 - d: where no term exists on either
    // side the sum is exactly 0, not the transform's rounding (which would outweigh the few terms
    // left, whose taps the Hann window has almost closed).
    if (j < 20) {
      const int sl = m0 + m;
      out[sl * 20 + j] = j > nd[sl] - Tn ? kl.after(v[0].x) : 0.f;
      out[(M + sl) * 20 + j] = j > nd[M + sl] - Tn ? kr.after(v[0].y) : 0.f;
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

hipError_t launch_delay_design(int M, const float* P, const int32_t* rows, int n, float* taps,
                               float* spec, int32_t* offs, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  return with_slots(M, [&](auto m) {
    delay_design_kernel<decltype(m)::value><<<dim3(n, M), kBlock, 0, s>>>(P, rows, taps, spec,
                                                                            offs);
    return hipGetLastError();
  });
}

hipError_t launch_delay_fwd(int M, const GraphView& g, float* U, const float* taps,
                            const float* spec, bool spec_by_node, const int32_t* offs,
                            int node_begin, int n_nodes, hipStream_t s) {
  const int tiles = (int)((g.T + kHop - 1) / kHop), per_node = (tiles + kWaves - 1) / kWaves;
  return with_slots(M, [&](auto m) {
    delay_fwd_kernel<decltype(m)::value><<<(unsigned)(per_node * n_nodes), kBlock, 0, s>>>(
        g, U, taps, spec, spec_by_node, offs, node_begin, per_node);
    return hipGetLastError();
  });
}

hipError_t launch_delay_bwd(int M, const GraphView& g, float* dU, const float* taps,
                            const float* spec, const int32_t* offs, int node_begin, int n_nodes,
                            float* part, hipStream_t s) {
  const int groups = delay_groups(g.T, g.tap_tiles);
  return with_slots(M, [&](auto m) {
    delay_bwd_kernel<decltype(m)::value><<<(unsigned)(groups * n_nodes), kBlock, 0, s>>>(
        g, dU, taps, spec, offs, node_begin, groups, part);
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

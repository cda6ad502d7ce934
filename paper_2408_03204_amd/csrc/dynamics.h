// Device helpers shared by the dynamics kernels (compressor and noisegate with one ballistics
// constant, k_comp.hip; compressor with attack/release ballistics, k_comp_ar.hip): chunk geometry,
// the static gain curves (paper Eqs. 10-11 and the noisegate of Sec. 3), the chunk ticket and
// publication protocol, and the gather-sum staging of a chunk into LDS.
#pragma once

#include "device_common.h"
#include "kernels.h"

namespace grafx {
namespace dyn {

constexpr int kPer = 12;
constexpr int kChunk = kCompChunk;  // 256 x kPer

// LDS layout of a chunk: element x sits at x + x / 96, one padding word after every 8 threads'
// segments of kPer samples. Thread j's segment is then contiguous from seg_base(j), and the 32
// lanes that one LDS cycle serves, reading element i of their own segments (a 12-word stride
// that would put 4 lanes on each of 8 banks), fall on 32 distinct banks; the coalesced staging
// writes and the stores stay conflict-free.
constexpr int kLdsChunk = kChunk + kChunk / 96;
__device__ __forceinline__ int lpos(int x) { return x + x / 96; }
__device__ __forceinline__ int seg_base(int j) { return kPer * j + (j >> 3); }
static_assert(kPer * 8 == 96, "one padding word per 8 segments");
constexpr double kEps = 1e-8;
constexpr uint64_t kNotReady = ~0ull;

// ---- gain curves ------------------------------------------------------------------------------
// Both curves (Eqs. 10-11 and the noisegate's) are a coefficient times one ramp function of the
// distance d between the log-envelope and the threshold (compressor: d = G_u - T, c = 1/R - 1;
// noisegate: d = T - G_u, c = 1 - R), G_y - G_u = c f(d):
//   f(d) = m^2 / (4 W) + max(d - W, 0),  m = clamp(d + W, 0, 2 W),
// which is 0 below the knee, (d + W)^2 / (4 W) inside it and d above it, with f'(d) = m / (2 W) and
// df/dW = f' (1 - f') in all three regions, so no region is selected per sample. A hard knee
// (W <= 0) is W = 0 with f' a step. Logarithms are base 2 throughout: what is stored is in those
// units, the threshold as a sum of two floats.
struct CurveCoef {
  float thr_hi, thr_lo;  // T
  float thr_n, thr_r;    // T: nearest whole number, rest
  float w, w_2;          // W (0 for a hard knee), 2 W
  float inv2w, inv4w;    // 1/(2W), 1/(4W) (0 for a hard knee)
  float c;               // 1/R - 1 (compressor) or 1 - R (noisegate)
  float kR;              // -dc/dR in natural-log units: ln 2 / R^2 or ln 2
};

// An infinite coefficient (a noise gate of infinite ratio) as the largest float, so that its product
// with a ramp of 0 is 0 where the curve has no effect, not NaN; elsewhere the gain is 0 all the same.
__device__ __forceinline__ float finite_coef(float c) {
  constexpr float most = 3.402823466e38f;
  return c > most ? most : c < -most ? -most : c;
}

__device__ __forceinline__ CurveCoef make_curve(double thr, double knee, double ratio, bool gate) {
  constexpr double log2e = 1.4426950408889634074, ln2 = 0.69314718055994530942;
  CurveCoef k;
  const double t = thr * log2e, w = knee > 1e-30 ? knee * log2e : 0.0;  // 1/(4W) in float's range
  k.thr_hi = (float)t;
  k.thr_lo = fabsf(k.thr_hi) < INFINITY ? (float)(t - (double)k.thr_hi) : 0.f;
  k.thr_n = (float)rint(t);
  k.thr_r = fabsf(k.thr_n) < INFINITY ? (float)(t - (double)k.thr_n) : 0.f;
  k.w = (float)w;
  k.w_2 = (float)(2.0 * w);
  k.inv2w = w > 0.0 ? (float)(0.5 / w) : 0.f;
  k.inv4w = w > 0.0 ? (float)(0.25 / w) : 0.f;
  k.c = finite_coef((float)(gate ? 1.0 - ratio : 1.0 / ratio - 1.0));
  k.kR = finite_coef((float)(gate ? ln2 : ln2 / (ratio * ratio)));
  return k;
}

struct Ramp {
  float f, fp, fq;  // f(d), f'(d) and 1 - f'(d) inside the knee (0 where f' = 1)
};

// The ramp at an envelope value gs > 0 (normal: the envelope plus 1e-8), through the hardware base-2
// logarithm. For derivatives exponent and mantissa are taken apart before it, so that the distance d
// is a difference of whole numbers plus a part below 2 and carries an absolute error near 1e-7; the
// logarithm of gs itself, up to 27 in size, would carry ten times that into the knee's derivatives
// and the sums over all samples (parameter gradients against float64: 1.3-7.9e-7 -> 0.7-1.6e-7 for
// 1 us of 82 on 48 compressors of 2^18 samples). A render keeps the one logarithm: there the error
// moves one sample's gain by a millionth. NaN stays NaN (v_med3 and v_max alone would drop it).
template <bool GATE, bool GRAD>
__device__ __forceinline__ Ramp ramp(float gs, const CurveCoef& k) {
  float d;
  if (GRAD) {
    const float e = (float)__builtin_amdgcn_frexp_expf(gs);
    const float L = __builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(gs));
    d = GATE ? (k.thr_n - e) + (k.thr_r - L) : (e - k.thr_n) + (L - k.thr_r);
  } else {
    const float L = __builtin_amdgcn_logf(gs);
    d = GATE ? (k.thr_hi - L) + k.thr_lo : (L - k.thr_hi) - k.thr_lo;
  }
  const float m = __builtin_amdgcn_fmed3f(d + k.w, 0.f, k.w_2);
  Ramp r;
  r.f = fmaf(m * k.inv4w, m, fmaxf(d - k.w, 0.f));
  r.f = d == d ? r.f : d;
  r.fp = GRAD ? m * k.inv2w : 0.f;
  r.fq = GRAD ? (k.w_2 - m) * k.inv2w : 0.f;
  if (GRAD && k.w_2 == 0.f) r.fp = (GATE ? d > 0.f : d >= 0.f) ? 1.f : 0.f;  // uniform condition
  return r;
}

// exp(c f): the gain, through the hardware base-2 exponential (relative error about 2e-6 where the
// exponent is 30)
__device__ __forceinline__ float gain(float f, const CurveCoef& k) {
  return __builtin_amdgcn_exp2f(k.c * f);
}

// ---- wave exchanges without LDS ----------------------------------------------------------------

// The value of another lane of the same row of 16 (a DPP control); lanes without a source get `old`.
template <int CTRL>
__device__ __forceinline__ double row_move(double x, double old = 0.0) {
  const int2 v = __builtin_bit_cast(int2, x), o = __builtin_bit_cast(int2, old);
  return __builtin_bit_cast(
      double, make_int2(__builtin_amdgcn_update_dpp(o.x, v.x, CTRL, 0xF, 0xF, false),
                        __builtin_amdgcn_update_dpp(o.y, v.y, CTRL, 0xF, 0xF, false)));
}
// From the lane N below (forward) or above (REV) in the row.
template <bool REV, int N>
__device__ __forceinline__ double row_before(double x, double old = 0.0) {
  return row_move<(REV ? 0x100 : 0x110) + N>(x, old);
}
__device__ __forceinline__ double lane_value(double x, int lane) {
  const int2 v = __builtin_bit_cast(int2, x);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(v.x, lane),
                                              __builtin_amdgcn_readlane(v.y, lane)));
}

// Sum over the wave, in every lane: a butterfly inside the rows, then the four rows in order.
__device__ __forceinline__ double wave_total(double v) {
  v += row_move<0xB1>(v);   // lane ^ 1
  v += row_move<0x4E>(v);   // lane ^ 2
  v += row_move<0x141>(v);  // mirrored within 8
  v += row_move<0x140>(v);  // mirrored within 16
  return ((lane_value(v, 0) + lane_value(v, 16)) + lane_value(v, 32)) + lane_value(v, 48);
}

// Sums of N values over the block (kBlock threads) with one exchange through LDS; the results are
// valid on every thread. `scratch` holds 4 N doubles.
template <int N>
__device__ __forceinline__ void block_totals(double (&v)[N], double* scratch) {
  const int w = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = wave_total(v[i]);
  __syncthreads();
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int i = 0; i < N; ++i) scratch[4 * i + w] = v[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i)
    v[i] = ((scratch[4 * i] + scratch[4 * i + 1]) + scratch[4 * i + 2]) + scratch[4 * i + 3];
}

// ---- per-node coefficients ---------------------------------------------------------------------
// Computed once per pass by the kernel that resets the chaining state and kept next to the node's
// ticket (second half of its 256-byte line), so a block reads them as scalars instead of forming
// them in every thread.

struct DynCoef {
  double a, b;   // alpha, 1 - alpha
  double logA;   // ln(a^kChunk), -inf for a = 0
  double pw[8];  // pw[d] = (a^kPer)^(2^d)
  CurveCoef cv;
};
struct DynCoefAR {
  double aa, ar, ba, br;  // alpha_a, alpha_r, 1 - alpha_a, 1 - alpha_r
  CurveCoef cv;
};
constexpr int kCoefOffset = 128;  // bytes into a ticket line
static_assert(sizeof(DynCoef) <= 128 && sizeof(DynCoefAR) <= 128 &&
                  kCompTicketStride * sizeof(unsigned) == 256,
              "coefficients fit the second half of a ticket line");

inline const char* dyn_coefs(const unsigned* tickets) {  // of row 0
  return reinterpret_cast<const char*>(tickets) + kCoefOffset;
}

template <class C>
__device__ __forceinline__ C load_coef(const char* __restrict__ coefs, int row) {
  return *reinterpret_cast<const C*>(coefs + (int64_t)row * kCompTicketStride * sizeof(unsigned));
}

__device__ __forceinline__ int comp_chunks_of(int64_t n) { return (int)((n + kChunk - 1) / kChunk); }

// Node of a block within its step: a node's `chunks` blocks contiguous (order 0) or the step's
// nodes interleaved block by block (order 1). A block's chunk comes from its node's ticket, so
// the order decides only when a node's chunks are issued, not what they compute.
__device__ __forceinline__ int block_node(const GraphView& g, int n_nodes, int chunks) {
  return g.dyn_order ? (int)blockIdx.x % n_nodes : (int)blockIdx.x / chunks;
}

// ---- chunk chaining ---------------------------------------------------------------------------

__device__ __forceinline__ int take_ticket(unsigned* counter, int* sh) {
  __syncthreads();
  if (threadIdx.x == 0)
    *sh = (int)__hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  return *sh;
}

__device__ __forceinline__ void publish(uint64_t* slot, double v) {
  __hip_atomic_store(slot, (uint64_t)__double_as_longlong(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

// Wait for a published total: at most `polls` reads of the slot (0: give up at once). A wait
// that gives up sets bit 0 of the error word and returns NaN, so the kernel still ends normally.
__device__ __forceinline__ double await_total(uint64_t* slot, unsigned* err, int polls) {
  for (int spin = 0; spin < polls; ++spin) {
    const uint64_t x = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (x != kNotReady) return __longlong_as_double((long long)x);
    __builtin_amdgcn_s_sleep(1);
  }
  atomicOr(err, 1u);
  return __longlong_as_double(0x7FF8000000000001ll);
}

// ---- staging -----------------------------------------------------------------------------------

// Gather-sum of a chunk (both channels) into LDS (padded layout): ADJ = false sums the input
// edges over U/S, ADJ = true the output edges over dU/dY. Zero beyond T.
template <bool ADJ, bool RAGGED>
__device__ __forceinline__ void stage(const GraphView& g, int node, int t0, float* sl, float* sr) {
  const int64_t T = g.T;
  // the edges, their rows and lengths are the same in every lane: kept scalar, or a load would loop
  // over the lanes' descriptors
  const int e0 = __builtin_amdgcn_readfirstlane(ADJ ? g.out_ptr[node] : g.in_ptr[node]);
  const int e1 = __builtin_amdgcn_readfirstlane(ADJ ? g.out_ptr[node + 1] : g.in_ptr[node + 1]);
  float l[kPer], r[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) l[q] = r[q] = 0.f;
  for (int e = e0; e < e1; ++e) {  // all loads of a row issued before any is consumed
    const int other = __builtin_amdgcn_readfirstlane(ADJ ? g.out_dst[e] : g.in_src[e]);
    const float* row = ADJ ? adj_row(g, other) : out_row(g, other);
    const int64_t L = RAGGED ? (int64_t)__builtin_amdgcn_readfirstlane(g.len[other]) : T;
    const auto rl = row_rsrc(row, L), rr = row_rsrc(row + T, L);
    float xl[kPer], xr[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int t = t0 + (int)threadIdx.x + kBlock * q;
      xl[q] = bload_nt(rl, t);
      xr[q] = bload_nt(rr, t);
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      l[q] += xl[q];
      r[q] += xr[q];
    }
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    sl[lpos(threadIdx.x + kBlock * q)] = l[q];
    sr[lpos(threadIdx.x + kBlock * q)] = r[q];
  }
}

// x = (u_l + u_r)^2 at LDS position idx, formed in float and fed to the double envelope
// recursion.
__device__ __forceinline__ double energy(const float* sl, const float* sr, int idx) {
  const float m = sl[idx] + sr[idx];
  return (double)(m * m);
}

// Chunk store (from the padded layout) into a row of stride T; samples at or beyond the node's
// length Tn are dropped. SUM: as the sum over one consumer (a zero's sign).
template <bool SUM = false>
__device__ __forceinline__ void store_chunk(float* row, int64_t T, int64_t Tn, int t0,
                                            const float* sl, const float* sr) {
  const int n = __builtin_amdgcn_readfirstlane((int)Tn);
  row = scalar_ptr(row);
  const auto rl = row_rsrc(row, n), rr = row_rsrc(row + T, n);
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    // an opaque copy of the thread index keeps the compiler from holding the staging
    // addresses, which are the same, in registers from the staging to here
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int idx = tid + kBlock * q;
    const float l = sl[lpos(idx)], r = sr[lpos(idx)];
    bstore_nt(rl, t0 + idx, SUM ? 0.f + l : l);
    bstore_nt(rr, t0 + idx, SUM ? 0.f + r : r);
  }
}

}  // namespace dyn
}  // namespace grafx

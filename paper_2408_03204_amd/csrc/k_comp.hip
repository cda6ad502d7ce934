// Feed-forward compressor (paper Sec. 3 "Compressor", Eqs. 8-12) and noisegate (Sec. 3
// "Noisegate": the same envelope with a downward-expander curve), parallel across nodes and
// time chunks, one pass over the signal per direction.
//
// With equal attack and release the energy envelope g[t] = a g[t-1] + (1-a) x[t],
// x = (u_l + u_r)^2, is a linear one-pole recursion (the untruncated FIR of Eq. 9). It is computed
// in double as a chunked scan: a block owns a chunk of 3072 samples (256 threads x 12 consecutive
// samples); a thread folds its samples, a scan inside the rows of 16 lanes and folds over the rows
// and the 4 waves give every thread its state relative to the chunk start. The chunk then publishes its
// total (the state it would leave from a zero start) and folds the totals of all earlier chunks
// of its node, c_k = sum_{j<k} total_j A^(k-1-j), A = a^3072, as one block-wide sum in a fixed
// order. Folding totals (never partially folded prefixes) keeps the arithmetic independent of
// timing, so results are deterministic and do not depend on the schedule. A block lives through
// several dependent memory round trips (ticket, loads, publish and wait, stores); the chunk size
// is chosen so that a 17-node step of 2^18 samples is resident in one round of blocks (24 KB of
// LDS and at most 80 VGPRs per thread give 6 blocks per CU), since a second round costs a whole
// block lifetime.
//
// Instructions bound the adjoint as much as memory does (1.4k float and 0.5k double instructions
// per wave left the vector units busy 64 of 98 us on 48 compressors of 2^18 samples), so: what
// depends only on the node (powers of a, curve constants) is formed once per pass by
// prepare_kernel and read as scalars; lanes exchange by DPP moves and readlane, not through
// LDS; both gain curves are one branch-free ramp in base-2 units (dynamics.h); the curve's
// derivatives are scaled once per chunk instead of per sample; and a thread's first read of an
// earlier total is under way during the parameter sums. The same strips: adjoint 94 -> 82 us,
// forward 51 us before and after (there memory, 3.9 of 4.8 TB/s, is the bound).
//
// A block's node comes from its block id; its chunk within the node comes from an atomic ticket
// on that node's counter (one cache line per counter), taken when the block starts, so every
// chunk a block waits for belongs to a block that started earlier and publishes without waiting:
// the waits always end. A total is published as one 64-bit atomic store at device scope over a
// "not ready" sentinel and read back by 64-bit atomic loads at device scope (the XCDs do not
// share an L2; device-scope atomics bypass the non-coherent caches). The reader consumes only
// that word, so no ordering with other data is needed: the accesses are relaxed, which avoids L2
// write-back and invalidation. Every wait is bounded; a wait that runs out records an error word
// and poisons its result instead of spinning forever.
//
// The gain curve (log of g + 1e-8, quadratic knee, gain) is evaluated in float.
//
// Adjoint (rho = sum_c ybar_c y_c, e = G_y - G_u):
//   gbar = rho de/dG_u / (g + 1e-8);  lambda[t] = gbar[t] + a lambda[t+1]  (reverse scan);
//   ubar_c = gamma ybar_c + 2 (u_l + u_r)(1 - a) lambda;
//   dL/da = sum lambda[t] (g[t-1] - x[t]);  dL/d(T, W, R) = sum rho de/d(T, W, R).
// The adjoint takes chunks from the end of each node backwards and runs the same scan on
// reversed thread order; the envelope entering each chunk is kept from the forward call.
#include <algorithm>

#include "device_common.h"
#include "dynamics.h"
#include "grafx_internal.h"
#include "kernels.h"

namespace grafx {
namespace {

using namespace dyn;

using Coef = DynCoef;

// Powers (a^kPer)^n of this thread's place: n its lane's position in the row of 16 and in the wave,
// counted from the end of the chunk when REV.
struct Powers {
  double row, wave;
};
template <bool REV>
__device__ __forceinline__ Powers lane_powers(const Coef& k) {
  const int lane0 = threadIdx.x & 63, n = REV ? 63 - lane0 : lane0;
  Powers p;
  double r = (n & 1) ? k.pw[0] : 1.0;
  if (n & 2) r *= k.pw[1];
  if (n & 4) r *= k.pw[2];
  if (n & 8) r *= k.pw[3];
  p.row = r;
  if (n & 16) r *= k.pw[4];
  if (n & 32) r *= k.pw[5];
  p.wave = r;
  return p;
}

// (a^kPer)^J' of this thread's place J' in the chunk, from its place in the wave
template <bool REV>
__device__ __forceinline__ double chunk_power(const Coef& k, double wave) {
  const int w0 = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), w = REV ? 3 - w0 : w0;
  if (w & 1) wave *= k.pw[6];
  if (w & 2) wave *= k.pw[7];
  return wave;
}

// Chunk scan of s_out = a^kPer s_in + B over the block's 256 threads (reversed thread order when
// REV), from a zero state entering the chunk: inside the rows of 16 lanes by DPP moves, then over
// the four rows and the four waves. Returns the state entering this thread's samples; `total`
// receives the state leaving the chunk (every thread). The thread's state for a non-zero entering
// state c is the returned value plus chunk_power c.
template <bool REV>
__device__ __forceinline__ double chunk_scan(double B, const Coef& k, const Powers& p, double* wtot,
                                             double& total) {
  const int lane0 = threadIdx.x & 63, w0 = threadIdx.x >> 6;
  const int row = REV ? 3 - (lane0 >> 4) : lane0 >> 4;
  const int w = REV ? 3 - w0 : w0;
  double S = B;
  S = fma(k.pw[0], row_before<REV, 1>(S), S);
  S = fma(k.pw[1], row_before<REV, 2>(S), S);
  S = fma(k.pw[2], row_before<REV, 4>(S), S);
  S = fma(k.pw[3], row_before<REV, 8>(S), S);
  double C = 0.0, Ci = 0.0;  // states leaving the rows before this lane's, and row i
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (row == i) C = Ci;
    Ci = fma(k.pw[4], Ci, lane_value(S, REV ? 48 - 16 * i : 16 * i + 15));
  }
  const double ex = fma(p.row, C, row_before<REV, 1>(S));
  __syncthreads();
  if (lane0 == 0) wtot[w] = Ci;
  __syncthreads();
  double P = 0.0, end = 0.0;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    if (v < w) P = fma(k.pw[6], P, wtot[v]);
    end = fma(k.pw[6], end, wtot[v]);
  }
  total = end;
  return fma(p.wave, P, ex);
}

// Entering state of chunk k: fixed-order block-wide sum over the published totals of the
// chunks before it (REV: after it), weighted by A^(distance - 1). The adjacent chunk's weight is
// exactly 1, so a = 0 (A = 0, logA = -inf) gives the plain recursion's carry without 0 * inf.
__device__ __forceinline__ double carry_weight(int dist, const Coef& c) {
  return dist == 0 ? 1.0 : exp((double)dist * c.logA);
}

// A thread's first total is read as soon as the chunk's own is published, and its weight (and, in
// the adjoint, the parameter sums) formed while that read is under way.
template <bool REV>
struct Carry {
  uint64_t* tot;
  int n;  // totals to fold: distances 0 .. n - 1 at tot[-dist] (forward) or tot[dist]
  uint64_t first;

  __device__ __forceinline__ uint64_t* at(int dist) const { return REV ? tot + dist : tot - dist; }
  __device__ __forceinline__ Carry(uint64_t* tots, int k, int chunks)
      : tot(REV ? tots + k + 1 : tots + k - 1), n(REV ? chunks - 1 - k : k), first(kNotReady) {
    const int d = threadIdx.x;
    if (d < n) first = __hip_atomic_load(at(d), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // This thread's part of the sum.
  __device__ __forceinline__ double part(const Coef& c, unsigned* err, int polls) const {
    double s = 0.0;
    int d = threadIdx.x;
    if (d < n) {
      const double w = carry_weight(d, c);
      s = (first != kNotReady && polls > 0 ? __longlong_as_double((long long)first)
                                           : await_total(at(d), err, polls)) * w;
    }
    for (d += kBlock; d < n; d += kBlock) s += await_total(at(d), err, polls) * carry_weight(d, c);
    return s;
  }
};

// ---- forward ----------------------------------------------------------------------------------

template <bool RAGGED, bool GATE>
__global__ __launch_bounds__(kBlock) void comp_fwd_kernel(GraphView g, float* U, int node_begin,
                                                          int n_nodes, int chunks, int ws_off,
                                                          const char* __restrict__ coefs,
                                                          uint64_t* agg, double* carry,
                                                          unsigned* ticket, unsigned* err) {
  __shared__ float sl[kLdsChunk], sr[kLdsChunk];
  __shared__ double wtot[4], red[4];
  __shared__ int sh_ticket;
  const int node = node_begin + block_node(g, n_nodes, chunks);
  const int ws = g.param_row[node] + ws_off;  // row of the dynamics workspace (compressors, then gates)
  const Coef k = load_coef<Coef>(coefs, ws);
  const int chunk = take_ticket(ticket + (int64_t)ws * kCompTicketStride, &sh_ticket);
  if (chunk >= chunks) {  // tickets not reset before the launch: do nothing
    if (threadIdx.x == 0) atomicOr(err, 2u);
    return;
  }
  const int64_t Tn = RAGGED ? (int64_t)g.len[node] : g.T;
  if (RAGGED && chunk >= comp_chunks_of(Tn)) return;  // past the node's length
  const int t0 = chunk * kChunk;
  stage<false, RAGGED>(g, node, t0, sl, sr);
  __syncthreads();
  const int i0 = seg_base(threadIdx.x);  // this thread's kPer samples
  double B = 0.0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) B = fma(k.a, B, k.b * energy(sl, sr, i0 + i));
  const Powers p = lane_powers<false>(k);
  double total;
  const double E0 = chunk_scan<false>(B, k, p, wtot, total);
  uint64_t* tots = agg + (int64_t)ws * chunks;
  if (threadIdx.x == 0) publish(tots + chunk, total);
  const Carry<false> from(tots, chunk, chunks);
  const double pj = chunk_power<false>(k, p.wave);
  double cin[1] = {from.part(k, err, g.wait_polls)};
  block_totals(cin, red);
  if (threadIdx.x == 0) carry[(int64_t)ws * chunks + chunk] = cin[0];
  double s = fma(pj, cin[0], E0);
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    s = fma(k.a, s, k.b * energy(sl, sr, i0 + i));
    const float gam = gain(ramp<GATE, false>((float)(s + kEps), k.cv).f, k.cv);
    sl[i0 + i] = gam * sl[i0 + i];
    sr[i0 + i] = gam * sr[i0 + i];
  }
  __syncthreads();
  store_chunk(U + (int64_t)node * 2 * g.T, g.T, Tn, t0, sl, sr);
}

// ---- adjoint ----------------------------------------------------------------------------------

template <bool RAGGED, bool GATE>
__global__ __launch_bounds__(kBlock) void comp_bwd_kernel(GraphView g, float* dU, int node_begin,
                                                          int n_nodes, int chunks, int ws_off,
                                                          const char* __restrict__ coefs,
                                                          const double* carry, uint64_t* ragg,
                                                          double* part, unsigned* ticket,
                                                          unsigned* err) {
  __shared__ float ul[kLdsChunk], ur[kLdsChunk], yl[kLdsChunk], yr[kLdsChunk];
  __shared__ double wtot[4], red[16];
  __shared__ int sh_ticket;
  const int node = node_begin + block_node(g, n_nodes, chunks);
  const int ws = g.param_row[node] + ws_off;  // row of the dynamics workspace (compressors, then gates)
  const Coef k = load_coef<Coef>(coefs, ws);
  const int tk = take_ticket(ticket + (int64_t)ws * kCompTicketStride, &sh_ticket);
  if (tk >= chunks) {  // tickets not reset before the launch: do nothing
    if (threadIdx.x == 0) atomicOr(err, 2u);
    return;
  }
  const int64_t Tn = RAGGED ? (int64_t)g.len[node] : g.T;
  const int chunks_n = RAGGED ? comp_chunks_of(Tn) : chunks;
  if (RAGGED && tk >= chunks_n) {  // past the node's length: this ticket zeroes one unused partial slot
    if (threadIdx.x < 4) part[((int64_t)ws * chunks + tk) * 4 + threadIdx.x] = 0.0;
    return;
  }
  const int chunk = chunks_n - 1 - tk;
  const int t0 = chunk * kChunk;
  stage<false, RAGGED>(g, node, t0, ul, ur);
  stage<true, RAGGED>(g, node, t0, yl, yr);
  __syncthreads();
  const int i0 = seg_base(threadIdx.x);  // this thread's kPer samples
  // envelope rebuilt from the forward carry
  double B = 0.0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) B = fma(k.a, B, k.b * energy(ul, ur, i0 + i));
  double total, E;
  {
    const Powers p = lane_powers<false>(k);
    const double E0 = chunk_scan<false>(B, k, p, wtot, total);
    E = fma(chunk_power<false>(k, p.wave), carry[(int64_t)ws * chunks + chunk], E0);
  }
  // First pass (forward over the thread's samples): envelope, gain and the local adjoint terms.
  // What the reverse pass needs is written back over the thread's own LDS slots: ul <- g[t-1] -
  // x[t], ur <- u_l + u_r, yl/yr <- gain * ybar. With de/dG_u = dg f': gbar = rho dg f' / (g + eps).
  const float dg = GATE ? -k.cv.c : k.cv.c;
  float gbar[kPer];
  double sum_fp = 0.0, sum_w = 0.0, sum_f = 0.0;  // of rho f', rho f' (1 - f') and rho f
  {
    double s = E;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int idx = i0 + i;
      const float u_l = ul[idx], u_r = ur[idx];
      const float m = u_l + u_r;
      const double x = (double)(m * m);  // as in energy()
      const double sprev = s;
      s = fma(k.a, s, k.b * x);
      const float gs = (float)(s + kEps);
      const Ramp r = ramp<GATE, true>(gs, k.cv);
      const float gam = gain(r.f, k.cv);
      const float y_l = gam * yl[idx], y_r = gam * yr[idx];
      const float rho = fmaf(y_l, u_l, y_r * u_r);
      const float rfp = rho * r.fp;
      gbar[i] = dg * rfp / gs;
      sum_fp += (double)rfp;
      sum_w += (double)(rfp * r.fq);
      sum_f += (double)(rho * r.f);
      ul[idx] = (float)(sprev - x);
      ur[idx] = m;
      yl[idx] = y_l;
      yr[idx] = y_r;
    }
  }
  // reverse recursion lambda[t] = gbar[t] + a lambda[t+1]
  double R = 0.0;
#pragma unroll
  for (int i = kPer - 1; i >= 0; --i) R = fma(k.a, R, (double)gbar[i]);
  const Powers p = lane_powers<true>(k);
  double rtotal;
  const double L0 = chunk_scan<true>(R, k, p, wtot, rtotal);
  uint64_t* rtots = ragg + (int64_t)ws * chunks;
  if (threadIdx.x == 0) publish(rtots + chunk, rtotal);
  const Carry<true> from(rtots, chunk, chunks_n);  // own chunks
  const double pj = chunk_power<true>(k, p.wave);
  double sums[4] = {sum_fp, sum_w, sum_f, 0.0};
#pragma unroll
  for (int i = 0; i < 3; ++i) sums[i] = wave_total(sums[i]);
  double rin[1] = {from.part(k, err, g.wait_polls)};
  block_totals(rin, red);
  double lam = fma(pj, rin[0], L0);
  double accA = 0.0;
#pragma unroll
  for (int i = kPer - 1; i >= 0; --i) {
    const int idx = i0 + i;
    lam = fma(k.a, lam, (double)gbar[i]);
    accA += lam * (double)ul[idx];
    const float mid = (float)(2.0 * k.b * lam) * ur[idx];
    yl[idx] += mid;
    yr[idx] += mid;
  }
  sums[3] = wave_total(accA);
  __syncthreads();
  store_chunk(dU + (int64_t)node * 2 * g.T, g.T, Tn, t0, yl, yr);
  if (float* ds = source_row(g, node)) store_chunk<true>(ds, g.T, Tn, t0, yl, yr);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[4 * i + (threadIdx.x >> 6)] = sums[i];
  __syncthreads();
  if (threadIdx.x < 4) {  // dL/da, dL/dT, dL/dW, dL/dR
    const double* q = red + 4 * ((threadIdx.x + 3) & 3);
    const double v = ((q[0] + q[1]) + q[2]) + q[3];
    const double f = threadIdx.x == 0   ? 1.0
                     : threadIdx.x == 1 ? -(double)dg
                     : threadIdx.x == 2 ? (double)k.cv.c
                                        : -(double)k.cv.kR;
    part[((int64_t)ws * chunks + chunk) * 4 + threadIdx.x] = f * v;
  }
}

__device__ __forceinline__ void* reset_line(unsigned* tickets, int64_t row) {
  unsigned* line = tickets + row * kCompTicketStride;
  *line = 0u;
  return reinterpret_cast<char*>(line) + kCoefOffset;
}

// Before a pass: published totals set to "not ready", tickets and the error word to 0, the nodes'
// coefficients and the EQ nodes' exp(p) formed. One thread an item of every kind.
__global__ __launch_bounds__(kBlock) void prepare_kernel(PrepareJobs j) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i == 0 && j.err) *j.err = 0u;
  if (i < j.comp.n_tot) j.comp.tot[i] = kNotReady;
  if (i < j.ar.n_tot) j.ar.tot[i] = kNotReady;
  if (i < (int64_t)j.n_eq * 1024)
    reinterpret_cast<double*>(j.eq_H + (i >> 10) * kEqFFT)[i & 1023] = exp((double)j.eq_P[i]);
  if (i < j.ar.n) {
    const float* p = j.ar.P + i * kArParams;
    DynCoefAR k;
    k.aa = (double)p[0];
    k.ar = (double)p[1];
    k.ba = 1.0 - k.aa;
    k.br = 1.0 - k.ar;
    k.cv = make_curve(p[2], p[3], p[4], false);
    *reinterpret_cast<DynCoefAR*>(reset_line(j.ar.tickets, i)) = k;
  }
  if (i < j.comp.n + j.comp.n_gate) {
    const bool gate = i >= j.comp.n;
    const float* p = gate ? j.comp.Pg + (i - j.comp.n) * 4 : j.comp.P + i * 4;
    DynCoef k;
    k.a = (double)p[0];
    k.b = 1.0 - k.a;
    k.logA = (double)kChunk * log(fabs(k.a));  // a^kChunk = |a|^kChunk: kChunk is even
    double q = 1.0, b = k.a;  // a^kPer by binary powering
    for (int e = kPer; e > 0; e >>= 1) {
      if (e & 1) q *= b;
      b *= b;
    }
    k.pw[0] = q;
#pragma unroll
    for (int d = 1; d < 8; ++d) k.pw[d] = k.pw[d - 1] * k.pw[d - 1];
    k.cv = make_curve(p[1], p[2], p[3], gate);
    *reinterpret_cast<DynCoef*>(reset_line(j.comp.tickets, i)) = k;
  }
}

}  // namespace

int comp_chunks(int64_t T) { return (int)((T + kChunk - 1) / kChunk); }

hipError_t launch_prepare(const PrepareJobs& j, hipStream_t s) {
  const int64_t m = std::max({j.comp.n_tot, j.ar.n_tot, (int64_t)j.n_eq * 1024, (int64_t)j.ar.n,
                              (int64_t)j.comp.n + j.comp.n_gate, (int64_t)(j.err ? 1 : 0)});
  if (m <= 0) return hipSuccess;
  prepare_kernel<<<(unsigned)((m + kBlock - 1) / kBlock), kBlock, 0, s>>>(j);
  return hipGetLastError();
}

template <bool RAGGED, bool GATE>
static void launch_fwd_t(const GraphView& g, float* U, int node_begin, int n_nodes, int chunks,
                         int ws_off, uint64_t* agg, double* carry, unsigned* ticket, unsigned* err,
                         hipStream_t s) {
  comp_fwd_kernel<RAGGED, GATE><<<(unsigned)(chunks * n_nodes), kBlock, 0, s>>>(
      g, U, node_begin, n_nodes, chunks, ws_off, dyn_coefs(ticket), agg, carry, ticket, err);
}

template <bool RAGGED, bool GATE>
static void launch_bwd_t(const GraphView& g, float* dU, int node_begin, int n_nodes, int chunks,
                         int ws_off, const double* carry, uint64_t* ragg, double* part,
                         unsigned* ticket, unsigned* err, hipStream_t s) {
  comp_bwd_kernel<RAGGED, GATE><<<(unsigned)(chunks * n_nodes), kBlock, 0, s>>>(
      g, dU, node_begin, n_nodes, chunks, ws_off, dyn_coefs(ticket), carry, ragg, part, ticket,
      err);
}

// Per-node lengths and the noisegate curve get their own instantiations, so the uniform
// compressor carries no code for either.
hipError_t launch_comp_fwd(const GraphView& g, float* U, int node_begin, int n_nodes, int ws_off,
                           bool gate, uint64_t* agg, double* carry, unsigned* ticket,
                           unsigned* err, hipStream_t s) {
  const int chunks = comp_chunks(g.T);
  if (g.len)
    (gate ? launch_fwd_t<true, true> : launch_fwd_t<true, false>)(
        g, U, node_begin, n_nodes, chunks, ws_off, agg, carry, ticket, err, s);
  else
    (gate ? launch_fwd_t<false, true> : launch_fwd_t<false, false>)(
        g, U, node_begin, n_nodes, chunks, ws_off, agg, carry, ticket, err, s);
  return hipGetLastError();
}

hipError_t launch_comp_bwd(const GraphView& g, float* dU, int node_begin, int n_nodes, int ws_off,
                           bool gate, const double* carry, uint64_t* ragg, double* part,
                           unsigned* ticket, unsigned* err, hipStream_t s) {
  const int chunks = comp_chunks(g.T);
  if (g.len)
    (gate ? launch_bwd_t<true, true> : launch_bwd_t<true, false>)(
        g, dU, node_begin, n_nodes, chunks, ws_off, carry, ragg, part, ticket, err, s);
  else
    (gate ? launch_bwd_t<false, true> : launch_bwd_t<false, false>)(
        g, dU, node_begin, n_nodes, chunks, ws_off, carry, ragg, part, ticket, err, s);
  return hipGetLastError();
}

}  // namespace grafx

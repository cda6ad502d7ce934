// Fused gather-sum -> pointwise processors -> store, for one schedule step (paper Algorithm 1:
// Gather, Aggregate, Process, Store of one iteration) or a chain of up to four, and the matching
// adjoint steps.
//
// Types: mix / out (identity, Eq. 1b only), gain_pan (Eq. 2), imager (Eq. 3), tanh distortion. A
// chain is a run of pointwise steps whose i-th nodes form paths: node i of a step has one input,
// node i of the step before, which has no other consumer. A pointwise node needs only the sample it
// writes, so a thread carries a path's sample through the chain in registers: every node's row is
// stored as before (the adjoint and callers read them) but not read back by the next step, and a
// chain is one launch. What bounds these kernels is HBM: a chain of n single-input nodes moves n + 1
// rows instead of 2 n forward. The arithmetic is that of the steps one by one, to the bit.
// One block of 256 threads covers 1024 x UN samples of one node (both channels), UN = 1, 2 or 4
// being a tuning setting of the schedule; blockIdx.y picks the node inside the step. Thread j
// covers samples 4j..4j+3 of each 1024-sample part of the tile and moves them as one 16-byte
// access per channel and input. The hardware takes such an access at any 4-byte boundary, so rows
// of odd lengths (whose starts are not 16-byte aligned) use it too; only the last tile of a node
// whose length is not a multiple of 4 moves the samples one by one, because a group of four there
// may cross the row's end. (64 tracks of gain_pan -> imager -> tanh at T = 250,007, render and
// adjoint: 908 us with one-by-one moves, 424 us with these, 5.7 TB/s, 302 us with the three
// nodes as a chain.) Inputs are read through raw buffer resources
// sized to their node's length, so samples past an input's length read as zero without a branch,
// and are summed in original edge order, so a node's arithmetic does not depend on the step it was
// batched into. A node's own samples past its length are neither computed nor stored.
#include "device_common.h"
#include "grafx_internal.h"
#include "kernels.h"
#include "reduce_partials.h"

namespace grafx {
namespace {

constexpr int kTile = 1024;

struct Gains {
  float e0, e1;
};

__device__ __forceinline__ Gains load_gains(int type, const float* P, int row) {
  Gains g{1.f, 1.f};
  if (type == GRAFX_GAIN_PAN) {
    g.e0 = expf(P[2 * row]);
    g.e1 = expf(P[2 * row + 1]);
  } else if (type == GRAFX_IMAGER || type == GRAFX_TANH) {
    g.e0 = expf(P[row]);
  }
  return g;
}

// A value as it is stored: keeps the compiler from contracting one link's product into the next
// link's sum, which a step on its own would not see.
__device__ __forceinline__ float stored(float x) {
  asm volatile("" : "+v"(x));
  return x;
}

// One link on N samples per channel. `type` is uniform.
template <int N>
__device__ __forceinline__ void fwd_op(int type, float (&l)[N], float (&r)[N], Gains k) {
  if (type == GRAFX_GAIN_PAN) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      l[i] *= k.e0;
      r[i] *= k.e1;
    }
  } else if (type == GRAFX_IMAGER) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float m = l[i] + r[i], s = k.e0 * (l[i] - r[i]);
      l[i] = 0.5f * (m + s);
      r[i] = 0.5f * (m - s);
    }
  } else if (type == GRAFX_TANH) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      l[i] = tanhf(k.e0 * l[i]);
      r[i] = tanhf(k.e0 * r[i]);
    }
  }
}

constexpr int kAnyType = -1;
template <int TYPE>
__device__ __forceinline__ int type_of(const PointwiseChain& c, int n) {
  return TYPE == kAnyType ? c.link[n].type : TYPE;
}

// Streaming store of 4 floats (any 4-byte boundary): marked non-temporal, since a step's output rows
// are read back only by later steps, long after the caches have turned over.
typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void nt_store4(float* p, float a, float b, float c, float d) {
  __builtin_nontemporal_store(v4f{a, b, c, d}, reinterpret_cast<v4f*>(p));
}

// n (4 or 1) consecutive floats of a row through a length-bounded buffer resource. NT (cache policy
// bit 1, non-temporal): for the forward pass over rows that start on 16-byte boundaries, which are
// read once, a whole line at a time (108 imagers of 2^20 samples: 191 us, 197 us without). In rows
// that do not, neighbouring threads' groups share lines, which the policy drops between them (64
// gain_pan -> imager -> tanh paths at T = 250,007: 100 us with it, 88 us without). In the adjoint it
// costs at either alignment (imagers 291 us with, 280 us without), but copies (mix, inputs) keep it:
// they gain nothing and would turn over the cache that the next kernels read from (the reverb's
// cross-spectra after the copy to the sources' adjoints: 67 us with, 81 us without).
template <bool V4, bool NT = false>
__device__ __forceinline__ void bload_n(__amdgpu_buffer_rsrc_t r, int idx, float* out) {
  if constexpr (V4) {
    const v4f a = __builtin_bit_cast(
        v4f, __builtin_amdgcn_raw_buffer_load_b128(r, idx * 4, 0, NT ? 2 : 0));
    out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
  } else {
    out[0] = bload(r, idx);
  }
}

// Whether the groups of four samples of the tile at `base` are each wholly inside or wholly outside
// a row of Tn samples (uniform over the block).
__device__ __forceinline__ bool whole_groups(int64_t base, int tile, int64_t Tn) {
  return (Tn & 3) == 0 || base + tile <= Tn;
}

// An edge's row and length are the same in every lane; said so, they stay scalar and a load needs no
// loop over the lanes' descriptors.
struct InputRow {
  const float* row;
  int len;
};
__device__ __forceinline__ InputRow input_row(const GraphView& g, int edge) {
  const int s = __builtin_amdgcn_readfirstlane(edge);
  return {out_row(g, s), __builtin_amdgcn_readfirstlane((int)node_len(g, s))};
}
__device__ __forceinline__ InputRow adjoint_row(const GraphView& g, int edge) {
  const int d = __builtin_amdgcn_readfirstlane(edge);
  return {adj_row(g, d), __builtin_amdgcn_readfirstlane((int)node_len(g, d))};
}

// l, r += the rows of input edges e .. e + R - 1, in order. All loads are issued before any is
// summed: a mix of one long row has one block a CU, so what it keeps in flight is what it reaches
// (48 rows of 2^18 samples and the output node: 32.6 us with four rows ahead, 35.8 us with one).
template <bool V4, bool NT, int UN, int R>
__device__ __forceinline__ void add_rows(const GraphView& g, int e, int64_t base,
                                         float (&l)[4 * UN], float (&r)[4 * UN]) {
  float a[R][4 * UN], b[R][4 * UN];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const InputRow in = input_row(g, g.in_src[e + i]);
    const auto rl = row_rsrc(in.row, in.len), rr = row_rsrc(in.row + g.T, in.len);
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int t = (int)(base + kTile * u + 4 * threadIdx.x);
      if constexpr (V4) {
        bload_n<true, NT>(rl, t, a[i] + 4 * u);
        bload_n<true, NT>(rr, t, b[i] + 4 * u);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          a[i][4 * u + q] = bload(rl, t + q);
          b[i][4 * u + q] = bload(rr, t + q);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int q = 0; q < 4 * UN; ++q) {
      l[q] += a[i][q];
      r[q] += b[i][q];
    }
}

template <int TYPE, bool V4, bool NT, int UN, int kMax>
__device__ __forceinline__ void fwd_tile(const GraphView& g, float* U, const PointwiseChain& c,
                                         int i, int64_t Tn, int64_t base) {
  const int64_t T = g.T;
  const int node = c.link[0].node_begin + i;
  constexpr int kRows = UN >= 4 ? 1 : 4 / UN;  // input rows ahead
  const int e0 = g.in_ptr[node], e1 = g.in_ptr[node + 1];
  Gains k[kMax];
#pragma unroll
  for (int n = 0; n < kMax; ++n)
    if (n < c.n)
      k[n] = load_gains(type_of<TYPE>(c, n), c.link[n].P, g.param_row[c.link[n].node_begin + i]);
  // thread j covers samples base + kTile u + 4 j .. + 3 for u < UN (samples past an input's length
  // read as zero)
  float l[4 * UN], r[4 * UN];
#pragma unroll
  for (int q = 0; q < 4 * UN; ++q) l[q] = r[q] = 0.f;
  int e = e0;
  for (; e + kRows <= e1; e += kRows) add_rows<V4, NT, UN, kRows>(g, e, base, l, r);
  for (; e < e1; ++e) add_rows<V4, NT, UN, 1>(g, e, base, l, r);
#pragma unroll
  for (int n = 0; n < kMax; ++n) {
    if (n >= c.n) break;
    if (n > 0)
#pragma unroll
      for (int q = 0; q < 4 * UN; ++q) {  // the sum over the link's one input
        l[q] = 0.f + stored(l[q]);
        r[q] = 0.f + stored(r[q]);
      }
    fwd_op(type_of<TYPE>(c, n), l, r, k[n]);
    float* y = U + (int64_t)(c.link[n].node_begin + i) * 2 * T;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t t = base + kTile * u + 4 * threadIdx.x;
      const float *yl = l + 4 * u, *yr = r + 4 * u;
      if constexpr (V4) {
        if (t < Tn) {
          nt_store4(y + t, yl[0], yl[1], yl[2], yl[3]);
          nt_store4(y + T + t, yr[0], yr[1], yr[2], yr[3]);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (t + q < Tn) {
            y[t + q] = yl[q];
            y[T + t + q] = yr[q];
          }
      }
    }
  }
}

// TYPE and kMax = 1 for a single step (fewer registers, more blocks in flight), kAnyType and the
// longest chain's length otherwise.
template <int TYPE, int UN, int kMax>
__global__ __launch_bounds__(kBlock) void pointwise_fwd_kernel(GraphView g, float* U,
                                                               PointwiseChain c) {
  const int i = blockIdx.y;
  const int64_t Tn = node_len(g, c.link[0].node_begin + i);
  const int64_t base = (int64_t)blockIdx.x * (kTile * UN);
  if (base >= Tn) return;  // tile past the node's length (uniform over the block)
  if (!whole_groups(base, kTile * UN, Tn))
    fwd_tile<TYPE, false, false, UN, kMax>(g, U, c, i, Tn, base);
  else if ((g.T & 3) == 0)
    fwd_tile<TYPE, true, true, UN, kMax>(g, U, c, i, Tn, base);
  else
    fwd_tile<TYPE, true, false, UN, kMax>(g, U, c, i, Tn, base);
}

// Adjoint of a chain. dst receives the links' input adjoints (dU, or dS for the input step, whose
// rows are indexed the same way). Parameter-gradient partials (one per block and parameter, double)
// go to the link's part[(slot * tiles + tile) * NP + j].
template <bool V4>
__device__ __forceinline__ void load_n(const float* p, float* out) {
  if constexpr (V4) {
    const v4f a = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p));
    out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
  } else {
    out[0] = *p;
  }
}

template <bool V4>
__device__ __forceinline__ void store_n(float* p, const float* v) {
  if constexpr (V4) nt_store4(p, v[0], v[1], v[2], v[3]);
  else *p = v[0];
}

// yl, yr: node output (gain_pan, imager) or input (tanh); gl, gr: output adjoint in, input adjoint
// out.
template <int N>
__device__ __forceinline__ void adj_op(int type, const float (&yl)[N], const float (&yr)[N],
                                       float (&gl)[N], float (&gr)[N], Gains k, float (&acc)[2]) {
  if (type == GRAFX_GAIN_PAN) {
#pragma unroll
    for (int v = 0; v < N; ++v) {
      acc[0] += gl[v] * yl[v];
      acc[1] += gr[v] * yr[v];
      gl[v] *= k.e0;
      gr[v] *= k.e1;
    }
  } else if (type == GRAFX_IMAGER) {
#pragma unroll
    for (int v = 0; v < N; ++v) {
      const float mb = 0.5f * (gl[v] + gr[v]), sb = 0.5f * (gl[v] - gr[v]);
      acc[0] += sb * (yl[v] - yr[v]);
      gl[v] = mb + k.e0 * sb;
      gr[v] = mb - k.e0 * sb;
    }
  } else if (type == GRAFX_TANH) {
#pragma unroll
    for (int v = 0; v < N; ++v) {
      const float al = tanhf(k.e0 * yl[v]), ar = tanhf(k.e0 * yr[v]);
      gl[v] = gl[v] * k.e0 * (1.f - al * al);
      gr[v] = gr[v] * k.e0 * (1.f - ar * ar);
      acc[0] += gl[v] * yl[v] + gr[v] * yr[v];
    }
  }
}

__host__ __device__ __forceinline__ int params_of(int type) {
  return type == GRAFX_GAIN_PAN ? 2 : type == GRAFX_IMAGER || type == GRAFX_TANH ? 1 : 0;
}

template <int TYPE, bool V4, int UN, int kMax>
__device__ __forceinline__ void bwd_tile(const GraphView& g, const PointwiseChain& c, int i,
                                         int64_t Tn, int64_t base, const Gains* k,
                                         float (*acc)[2]) {
  constexpr int NV = V4 ? 4 : 1;
  constexpr bool kNt = TYPE == GRAFX_MIX;  // copies only
  const int64_t T = g.T;
  const int last = c.link[c.n - 1].node_begin + i, first = c.link[0].node_begin + i;
  const int o0 = g.out_ptr[last], o1 = g.out_ptr[last + 1];
  const int i0 = g.in_ptr[first], i1 = g.in_ptr[first + 1];
  float* const ds = first >= g.K ? source_row(g, first) : nullptr;
  // Thread j covers samples base + kTile u + 4j .. + 3 (u < UN) in both paths, in the same order,
  // so the gradient partials are accumulated identically whichever path a launch takes. Blocks
  // past the node's length still write their (zero) partials.
#pragma unroll
  for (int u = 0; u < UN; ++u) {
    const int64_t t_first = base + kTile * u + 4 * threadIdx.x;
#pragma unroll
    for (int q = 0; q < (V4 ? 1 : 4); ++q) {
      const int64_t t = t_first + q;
      if (t >= Tn) break;
      // every link's output row, where it or the tanh that reads it needs it
      float yl[kMax][NV], yr[kMax][NV];
#pragma unroll
      for (int n = 0; n < kMax; ++n) {
        if (n >= c.n) break;
        const int type = type_of<TYPE>(c, n);
        if (type == GRAFX_GAIN_PAN || type == GRAFX_IMAGER ||
            (n + 1 < c.n && type_of<TYPE>(c, n + 1 < kMax ? n + 1 : n) == GRAFX_TANH)) {
          const float* y = out_row(g, c.link[n].node_begin + i);
          load_n<V4>(y + t, yl[n]);
          load_n<V4>(y + T + t, yr[n]);
        }
      }
      float gl[NV], gr[NV], ul[NV], ur[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) gl[v] = gr[v] = ul[v] = ur[v] = 0.f;
      for (int e = o0; e < o1; ++e) {
        const InputRow in = adjoint_row(g, g.out_dst[e]);
        float a[NV], b[NV];
        bload_n<V4, kNt>(row_rsrc(in.row, in.len), (int)t, a);
        bload_n<V4, kNt>(row_rsrc(in.row + T, in.len), (int)t, b);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          gl[v] += a[v];
          gr[v] += b[v];
        }
      }
      if (type_of<TYPE>(c, 0) == GRAFX_TANH)
        for (int e = i0; e < i1; ++e) {
          const InputRow in = input_row(g, g.in_src[e]);
          float a[NV], b[NV];
          bload_n<V4>(row_rsrc(in.row, in.len), (int)t, a);
          bload_n<V4>(row_rsrc(in.row + T, in.len), (int)t, b);
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            ul[v] += a[v];
            ur[v] += b[v];
          }
        }
#pragma unroll
      for (int n = kMax - 1; n >= 0; --n) {
        if (n >= c.n) continue;
        if (n < c.n - 1)
#pragma unroll
          for (int v = 0; v < NV; ++v) {  // the sum over the link's one consumer
            gl[v] = 0.f + stored(gl[v]);
            gr[v] = 0.f + stored(gr[v]);
          }
        const int type = type_of<TYPE>(c, n);
        if (type == GRAFX_TANH && n > 0) {
          float xl[NV], xr[NV];
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            xl[v] = 0.f + yl[n > 0 ? n - 1 : 0][v];
            xr[v] = 0.f + yr[n > 0 ? n - 1 : 0][v];
          }
          adj_op(type, xl, xr, gl, gr, k[n], acc[n]);
        } else if (type == GRAFX_TANH) {
          adj_op(type, ul, ur, gl, gr, k[n], acc[n]);
        } else {
          adj_op(type, yl[n], yr[n], gl, gr, k[n], acc[n]);
        }
        float* d = c.dst + (int64_t)(c.link[n].node_begin + i) * 2 * T;
        store_n<V4>(d + t, gl);
        store_n<V4>(d + T + t, gr);
        if (n == 0 && ds) {
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            gl[v] = 0.f + stored(gl[v]);
            gr[v] = 0.f + stored(gr[v]);
          }
          store_n<V4>(ds + t, gl);
          store_n<V4>(ds + T + t, gr);
        }
      }
    }
  }
}

template <int TYPE, int UN, int kMax>
__global__ __launch_bounds__(kBlock) void pointwise_bwd_kernel(GraphView g, PointwiseChain c,
                                                               int tiles) {
  const int i = blockIdx.y;
  const int64_t Tn = node_len(g, c.link[0].node_begin + i);
  Gains k[kMax];
  int slot[kMax];
  float acc[kMax][2];
#pragma unroll
  for (int n = 0; n < kMax; ++n) {
    acc[n][0] = acc[n][1] = 0.f;
    if (n >= c.n) continue;
    slot[n] = g.param_row[c.link[n].node_begin + i];
    k[n] = load_gains(type_of<TYPE>(c, n), c.link[n].P, slot[n]);
  }
  const int64_t base = (int64_t)blockIdx.x * (kTile * UN);
  if (whole_groups(base, kTile * UN, Tn))
    bwd_tile<TYPE, true, UN, kMax>(g, c, i, Tn, base, k, acc);
  else
    bwd_tile<TYPE, false, UN, kMax>(g, c, i, Tn, base, k, acc);
  __shared__ double red[4];
#pragma unroll
  for (int n = 0; n < kMax; ++n) {
    if (n >= c.n) break;
    const int np = params_of(type_of<TYPE>(c, n));
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (j >= np) break;
      const double s = block_sum<double>((double)acc[n][j], red);
      if (threadIdx.x == 0)
        c.link[n].part[((int64_t)slot[n] * tiles + blockIdx.x) * np + j] = s;
    }
  }
}

__global__ __launch_bounds__(kBlock) void reduce_partials_kernel(ReduceJobs J) {
  reduce_partials(J, blockIdx.x);
}

}  // namespace

int pointwise_tiles(int64_t T, int unroll) {
  const int64_t tile = (int64_t)kTile * (unroll > 0 ? unroll : 1);
  return (int)((T + tile - 1) / tile);
}

// Single steps and chains of mix and output nodes alone have their type at compile time.
template <int UN>
static void fwd_un(const PointwiseChain& c, const GraphView& g, float* U, dim3 grid,
                   hipStream_t s) {
  constexpr int kMax = PointwiseChain::kMax;
  bool copies = true;
  for (int n = 0; n < c.n; ++n) copies = copies && params_of(c.link[n].type) == 0;
  const int type = c.n == 1 || copies ? c.link[0].type : kAnyType;
  if (type == kAnyType)
    pointwise_fwd_kernel<kAnyType, UN, kMax><<<grid, kBlock, 0, s>>>(g, U, c);
  else if (c.n > 1)
    pointwise_fwd_kernel<GRAFX_MIX, UN, kMax><<<grid, kBlock, 0, s>>>(g, U, c);
  else if (type == GRAFX_GAIN_PAN)
    pointwise_fwd_kernel<GRAFX_GAIN_PAN, UN, 1><<<grid, kBlock, 0, s>>>(g, U, c);
  else if (type == GRAFX_IMAGER)
    pointwise_fwd_kernel<GRAFX_IMAGER, UN, 1><<<grid, kBlock, 0, s>>>(g, U, c);
  else if (type == GRAFX_TANH)
    pointwise_fwd_kernel<GRAFX_TANH, UN, 1><<<grid, kBlock, 0, s>>>(g, U, c);
  else
    pointwise_fwd_kernel<GRAFX_MIX, UN, 1><<<grid, kBlock, 0, s>>>(g, U, c);
}

hipError_t launch_pointwise_fwd(const PointwiseChain& c, const GraphView& g, float* U, int n_nodes,
                                hipStream_t s) {
  const dim3 grid((unsigned)pointwise_tiles(g.T, g.pw_unroll), (unsigned)n_nodes);
  switch (g.pw_unroll) {
    case 2: fwd_un<2>(c, g, U, grid, s); break;
    case 4: fwd_un<4>(c, g, U, grid, s); break;
    default: fwd_un<1>(c, g, U, grid, s); break;
  }
  return hipGetLastError();
}

// Single steps and chains of mix and output nodes alone have their type at compile time.
template <int UN>
static void bwd_un(const PointwiseChain& c, const GraphView& g, dim3 grid, hipStream_t s) {
  constexpr int kMax = PointwiseChain::kMax;
  bool copies = true;
  for (int n = 0; n < c.n; ++n) copies = copies && params_of(c.link[n].type) == 0;
  const int type = c.n == 1 || copies ? c.link[0].type : kAnyType;
  if (type == kAnyType)
    pointwise_bwd_kernel<kAnyType, UN, kMax><<<grid, kBlock, 0, s>>>(g, c, (int)grid.x);
  else if (c.n > 1)
    pointwise_bwd_kernel<GRAFX_MIX, UN, kMax><<<grid, kBlock, 0, s>>>(g, c, (int)grid.x);
  else if (type == GRAFX_GAIN_PAN)
    pointwise_bwd_kernel<GRAFX_GAIN_PAN, UN, 1><<<grid, kBlock, 0, s>>>(g, c, (int)grid.x);
  else if (type == GRAFX_IMAGER)
    pointwise_bwd_kernel<GRAFX_IMAGER, UN, 1><<<grid, kBlock, 0, s>>>(g, c, (int)grid.x);
  else if (type == GRAFX_TANH)
    pointwise_bwd_kernel<GRAFX_TANH, UN, 1><<<grid, kBlock, 0, s>>>(g, c, (int)grid.x);
  else
    pointwise_bwd_kernel<GRAFX_MIX, UN, 1><<<grid, kBlock, 0, s>>>(g, c, (int)grid.x);
}

hipError_t launch_pointwise_bwd(const PointwiseChain& c, const GraphView& g, int n_nodes,
                                hipStream_t s) {
  const dim3 grid((unsigned)pointwise_tiles(g.T, g.pw_unroll), (unsigned)n_nodes);
  switch (g.pw_unroll) {
    case 2: bwd_un<2>(c, g, grid, s); break;
    case 4: bwd_un<4>(c, g, grid, s); break;
    default: bwd_un<1>(c, g, grid, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_reduce_partials(const ReduceJobs& jobs, hipStream_t s) {
  if (jobs.blocks() <= 0) return hipSuccess;
  reduce_partials_kernel<<<jobs.blocks(), kBlock, 0, s>>>(jobs);
  return hipGetLastError();
}

}  // namespace grafx

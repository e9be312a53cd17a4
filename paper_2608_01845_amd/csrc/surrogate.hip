// HBM-bound kernels of the surrogate and the risk controller (Sec. 4.2-4.3).
//
// The latent [C, F, H, W] is processed as C*8 contiguous segments: segment
// (c, g) holds the flat spatial indices j of channel c with floor(8j/T) = g,
// which is the finest chunking the 256-d summary pools over (coarser chunks
// nest: floor(4j/T) = floor(floor(8j/T)/2)). Each block streams one slice of
// one segment, so every per-chunk sum is a plain per-block sum and the grid
// needs no atomics. The blocks write their partial sums (6 to 10 doubles each)
// straight into the state's pinned host memory, and the host, which waits for
// them anyway, adds the slices of a segment in a fixed order in float64
// (deterministic, bit-reproducible run to run): no reduction launch and no copy
// between the kernel and the decision. That needs few blocks: up to four slices of
// 4,096 elements and 256 threads per segment, then slices of 16,384 elements and 1,024
// threads, at most 64 (make_seg_plan). The candidate step on 16 x 7 x 32 x 48
// (two such waits): 51 -> 37 us; a rollout step on 16 x 33 x 90 x 160: 74 -> 56
// us, the combine of four latents at 6.2 TB/s (the 256 MB cache holds most of them).
//
// Slices are read as 16-byte vectors when every buffer of the launch is
// 16-byte aligned: a slice is split into a scalar head (< 4 elements up to
// the first multiple of 4), a float4 body and a scalar tail.
//
// The observation and exact-step kernels also emit the pass-1 statistics of
// the latent they produce, under the anchor the next step will use, so a
// rollout reads each latent once per step (Eq. (2), (5), (6)).
#include "common.h"

namespace wdc {

namespace {
constexpr int kThreads = 1024;   // most threads per block

struct SegRange {
  int64_t a, b;  // flat element range [a, b) of this block
};

__device__ __forceinline__ SegRange seg_range(int64_t t, int g, int splits) {
  const int blk = blockIdx.x;
  const int seg = blk / splits, sp = blk % splits;
  const int c = seg / g, gi = seg % g;
  const int64_t s0 = (gi * t + g - 1) / g;        // ceil(gi*T/G)
  const int64_t s1 = ((gi + 1) * t + g - 1) / g;  // ceil((gi+1)*T/G)
  const int64_t len = s1 - s0;
  SegRange r;
  r.a = (int64_t)c * t + s0 + (len * sp) / splits;
  r.b = (int64_t)c * t + s0 + (len * (sp + 1)) / splits;
  return r;
}

template <int W>
struct Vf {
  float x[W];
};

template <int W>
__device__ __forceinline__ Vf<W> ldv(const float *__restrict__ p, int64_t i) {
  Vf<W> o;
  if constexpr (W == 4) {
    const float4 t = *reinterpret_cast<const float4 *>(p + i);
    o.x[0] = t.x;
    o.x[1] = t.y;
    o.x[2] = t.z;
    o.x[3] = t.w;
  } else {
    o.x[0] = p[i];
  }
  return o;
}

template <int W>
__device__ __forceinline__ void stv(float *__restrict__ p, int64_t i, const Vf<W> &v) {
  if constexpr (W == 4) {
    *reinterpret_cast<float4 *>(p + i) = make_float4(v.x[0], v.x[1], v.x[2], v.x[3]);
  } else {
    p[i] = v.x[0];
  }
}

template <int W>
__device__ __forceinline__ Vf<W> zeros() {
  Vf<W> o;
#pragma unroll
  for (int e = 0; e < W; ++e) o.x[e] = 0.f;
  return o;
}

// Streams [a, b) through op.template step<W>(i, acc): W = 4 on aligned
// indices when vec, else W = 1.
template <int NV, class Op>
__device__ __forceinline__ void stream_range(const Op &op, SegRange r, bool vec, float (&acc)[NV]) {
  if (vec) {
    const int64_t a4 = min(r.b, (r.a + 3) & ~(int64_t)3);
    const int64_t b4 = max(a4, r.b & ~(int64_t)3);
    if (r.a + threadIdx.x < a4) op.template step<1>(r.a + threadIdx.x, acc);
#pragma unroll 2
    for (int64_t i = a4 + 4 * (int64_t)threadIdx.x; i < b4; i += 4 * (int64_t)blockDim.x) op.template step<4>(i, acc);
    if (b4 + threadIdx.x < r.b) op.template step<1>(b4 + threadIdx.x, acc);
  } else {
    for (int64_t i = r.a + threadIdx.x; i < r.b; i += blockDim.x) op.template step<1>(i, acc);
  }
}

// The block's sums, one store by NV neighbouring lanes (part: pinned host memory).
// The wave sums are added in float64, as the host goes on, so that a block of 16
// waves loses no more than one of 4.
template <int NV>
__device__ __forceinline__ void write_partials(float (&v)[NV], float *lds, double *__restrict__ part) {
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = wave_sum_fast(v[i]);
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < NV; ++i) lds[(threadIdx.x >> 6) * NV + i] = v[i];
  __syncthreads();
  if (threadIdx.x < NV) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += (double)lds[w * NV + threadIdx.x];
    part[(int64_t)blockIdx.x * NV + threadIdx.x] = s;
  }
}

// pass-1 statistics of z against the anchor za (0 without one):
// [sum z, sum d, sum z^2, sum d^2, sum |d|, sum |za|], d = z - za
template <int W>
__device__ __forceinline__ void acc_pre(const Vf<W> &z, const Vf<W> &za, float (&v)[PRE_NV]) {
#pragma unroll
  for (int e = 0; e < W; ++e) {
    const float x = z.x[e], a = za.x[e], d = x - a;
    v[0] += x;
    v[1] += d;
    v[2] += x * x;
    v[3] += d * d;
    v[4] += fabsf(d);
    v[5] += fabsf(a);
  }
}

struct PreOp {
  const float *z, *za;
  template <int W>
  __device__ __forceinline__ void step(int64_t i, float (&v)[PRE_NV]) const {
    const Vf<W> x = ldv<W>(z, i);
    const Vf<W> a = za ? ldv<W>(za, i) : zeros<W>();
    acc_pre<W>(x, a, v);
  }
};

__global__ __launch_bounds__(kThreads) void k_stats_pre(SegPlan pl, PreOp op, double *__restrict__ part) {
  __shared__ float lds[16 * PRE_NV];
  float v[PRE_NV] = {};
  stream_range<PRE_NV>(op, seg_range(pl.t, pl.g, pl.splits), pl.vec, v);
  write_partials<PRE_NV>(v, lds, part);
}

// M: number of combined latents, 0 = m (read four at a time, so that their
// loads travel together)
template <int M>
struct ObsOp {
  const float *outs[WDC_MAXB];
  float kappa[WDC_MAXB];
  int m;
  const float *za;
  float *zhat;
  template <int W>
  __device__ __forceinline__ void step(int64_t i, float (&v)[OBS_NV]) const {
    const Vf<W> a = za ? ldv<W>(za, i) : zeros<W>();
    Vf<W> acc = zeros<W>();
    auto add = [&](int j, const Vf<W> &o) {
#pragma unroll
      for (int e = 0; e < W; ++e) acc.x[e] += kappa[j] * o.x[e];
    };
    if constexpr (M > 0) {
      Vf<W> o[M];
#pragma unroll
      for (int j = 0; j < M; ++j) o[j] = ldv<W>(outs[j], i);
#pragma unroll
      for (int j = 0; j < M; ++j) add(j, o[j]);
    } else {
      int j = 0;
      for (; j + 4 <= m; j += 4) {
        Vf<W> o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = ldv<W>(outs[j + q], i);
#pragma unroll
        for (int q = 0; q < 4; ++q) add(j + q, o[q]);
      }
      for (; j < m; ++j) add(j, ldv<W>(outs[j], i));
    }
    stv<W>(zhat, i, acc);
    float pre[PRE_NV] = {};
    acc_pre<W>(acc, a, pre);
#pragma unroll
    for (int q = 0; q < PRE_NV; ++q) v[q] += pre[q];
#pragma unroll
    for (int e = 0; e < W; ++e) v[PRE_NV] += isfinite(acc.x[e]) ? 0.f : 1.f;
  }
};

template <int M>
__global__ __launch_bounds__(kThreads) void k_observe(SegPlan pl, ObsOp<M> op, double *__restrict__ part) {
  __shared__ float lds[16 * OBS_NV];
  float v[OBS_NV] = {};
  stream_range<OBS_NV>(op, seg_range(pl.t, pl.g, pl.splits), pl.vec, v);
  write_partials<OBS_NV>(v, lds, part);
}

struct PostOp {
  PostArgs a;
  template <int W>
  __device__ __forceinline__ void step(int64_t i, float (&v)[POST_NV]) const {
    const Vf<W> x = ldv<W>(a.z, i);
    Vf<W> xn;
    if (a.v) {
      const Vf<W> vv = ldv<W>(a.v, i);
#pragma unroll
      for (int e = 0; e < W; ++e) xn.x[e] = x.x[e] + a.dt * vv.x[e];
      stv<W>(a.zn_out, i, xn);
    } else {
      xn = ldv<W>(a.zn_in, i);
    }
    if (a.bank_slot) stv<W>(a.bank_slot, i, xn);
    if (a.anchor_out) stv<W>(a.anchor_out, i, x);
    if (a.in_slot) stv<W>(a.in_slot, i, x);
    const Vf<W> za = a.has_anchor ? ldv<W>(a.za, i) : zeros<W>();
    const Vf<W> zh = a.has_zhat ? ldv<W>(a.zhat, i) : zeros<W>();
#pragma unroll
    for (int e = 0; e < W; ++e) {
      const float n = xn.x[e], dn = n - za.x[e], dx = n - x.x[e];
      v[0] += n;
      v[1] += dn;
      v[2] += dx;
      v[3] += n * n;
      v[4] += dn * dn;
      v[5] += dx * dx;
      v[6] += a.has_zhat ? fabsf(n - zh.x[e]) : 0.f;
      v[7] += fabsf(n);
      v[8] += fabsf(dx);
      v[9] += fabsf(x.x[e]);
    }
  }
};

__global__ __launch_bounds__(kThreads) void k_exact_post(SegPlan pl, PostOp op, double *__restrict__ part) {
  __shared__ float lds[16 * POST_NV];
  float v[POST_NV] = {};
  stream_range<POST_NV>(op, seg_range(pl.t, pl.g, pl.splits), pl.vec, v);
  write_partials<POST_NV>(v, lds, part);
}

template <int W>
__global__ __launch_bounds__(256) void k_psi(const float *__restrict__ z, const float *__restrict__ v, float dt,
                                             float *__restrict__ zn, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x * W;
  for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * W; i < n; i += stride) {
    if (W == 4 && i + 4 <= n) {
      const Vf<4> a = ldv<4>(z, i), b = ldv<4>(v, i);
      Vf<4> o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o.x[e] = a.x[e] + dt * b.x[e];
      stv<4>(zn, i, o);
    } else {
      for (int64_t j = i; j < i + W && j < n; ++j) zn[j] = z[j] + dt * v[j];
    }
  }
}

bool al16(const void *p) { return ((uintptr_t)p & 15) == 0; }
}  // namespace

// Slices of at most 4,096 elements and 256 threads while at most 4 of them make a
// segment; longer segments in slices of at most 16,384 elements and 1,024 threads
// (longer ones from 64 slices on, 1,048,576 elements): as many threads in flight, a quarter of the partial sums (16 x
// 33 x 90 x 160, exact-step epilogue 44 -> 36 us with the wave sums by lane moves).
SegPlan make_seg_plan(int c, int64_t t, int g) {
  SegPlan p;
  p.c = c;
  p.t = t;
  p.g = g;
  p.vec = 1;
  const int64_t seglen = (t + g - 1) / g;
  int64_t sp = (seglen + 4095) / 4096;
  p.threads = 256;
  if (sp > 4) {
    sp = (seglen + 16383) / 16384;
    p.threads = kThreads;
  }
  p.splits = (int)(sp < 1 ? 1 : (sp > 64 ? 64 : sp));
  return p;
}

void reduce_partials(const SegPlan &pl, const double *part, int nv, double *out) {
  const int nseg = pl.nseg();
  for (int seg = 0; seg < nseg; ++seg) {
    double *o = out + (size_t)seg * nv;
    for (int v = 0; v < nv; ++v) o[v] = 0.0;
    for (int sp = 0; sp < pl.splits; ++sp, part += nv)
      for (int v = 0; v < nv; ++v) o[v] += part[v];
  }
}

hipError_t launch_stats_pre(const SegPlan &pl, const float *z, const float *za, double *partials, hipStream_t s) {
  SegPlan p = pl;
  p.vec = al16(z) && al16(za);
  hipLaunchKernelGGL(k_stats_pre, dim3(p.nblocks()), dim3(p.threads), 0, s, p, PreOp{z, za}, partials);
  return hipGetLastError();
}

namespace {
template <int M>
hipError_t run_observe(const SegPlan &p, const ObsOp<0> &o, double *partials, hipStream_t s) {
  ObsOp<M> op;
  for (int j = 0; j < WDC_MAXB; ++j) {
    op.outs[j] = o.outs[j];
    op.kappa[j] = o.kappa[j];
  }
  op.m = o.m;
  op.za = o.za;
  op.zhat = o.zhat;
  hipLaunchKernelGGL(k_observe<M>, dim3(p.nblocks()), dim3(p.threads), 0, s, p, op, partials);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_observe(const SegPlan &pl, const float *const *outs, const float *kappa, int m, const float *za,
                          float *zhat, double *partials, hipStream_t s) {
  if (m < 1 || m > WDC_MAXB) return hipErrorInvalidValue;
  ObsOp<0> op;
  bool vec = al16(zhat) && al16(za);
  for (int j = 0; j < WDC_MAXB; ++j) {
    op.outs[j] = j < m ? outs[j] : nullptr;
    op.kappa[j] = j < m ? kappa[j] : 0.f;
    if (j < m) vec = vec && al16(outs[j]);
  }
  op.m = m;
  op.za = za;
  op.zhat = zhat;
  SegPlan p = pl;
  p.vec = vec;
  // the bank's default capacity and its filling, and the secant's three latents
  switch (m) {
    case 1: return run_observe<1>(p, op, partials, s);
    case 2: return run_observe<2>(p, op, partials, s);
    case 3: return run_observe<3>(p, op, partials, s);
    case 4: return run_observe<4>(p, op, partials, s);
    default: return run_observe<0>(p, op, partials, s);
  }
}

hipError_t launch_exact_post(const SegPlan &pl, const PostArgs &a, double *partials, hipStream_t s) {
  SegPlan p = pl;
  p.vec = al16(a.z) && al16(a.v) && al16(a.zn_in) && al16(a.za) && al16(a.zhat) && al16(a.zn_out) &&
          al16(a.bank_slot) && al16(a.anchor_out) && al16(a.in_slot);
  hipLaunchKernelGGL(k_exact_post, dim3(p.nblocks()), dim3(p.threads), 0, s, p, PostOp{a}, partials);
  return hipGetLastError();
}

hipError_t launch_psi(const float *z, const float *v, float dt, float *zn, int64_t n, hipStream_t s) {
  const bool vec = al16(z) && al16(v) && al16(zn);
  const int w = vec ? 4 : 1;
  int64_t blocks = (n + 256 * w - 1) / (256 * w);
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  if (vec)
    hipLaunchKernelGGL(k_psi<4>, dim3((unsigned)blocks), dim3(256), 0, s, z, v, dt, zn, n);
  else
    hipLaunchKernelGGL(k_psi<1>, dim3((unsigned)blocks), dim3(256), 0, s, z, v, dt, zn, n);
  return hipGetLastError();
}

}  // namespace wdc

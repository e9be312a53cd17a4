// Memory-bound kernels of the denoiser: LayerNorm + adaLN modulation, q/k/v
// preparation (per-head RMSNorm, 3D rotary embedding, attention layouts),
// conditioning products, patch (un)folding and seeded initialisation.
#include "common.h"

namespace wdc {

namespace {

// ---------------------------------------------------------------- LayerNorm + modulate
// One 256-thread block per row; the row stays in registers between the two
// passes (mean, then variance of the centred values).
template <typename T, int MAXV>
__global__ __launch_bounds__(256) void k_ln_mod(const float *__restrict__ x, int64_t ldx, T *__restrict__ h,
                                               int64_t ldh, LnRows lr, int d, const float *__restrict__ shift,
                                               const float *__restrict__ scale) {
  __shared__ float red[8];
  const int64_t i = blockIdx.x;
  const int64_t smp = i / lr.rps;
  const int64_t r = smp * lr.sstride + i % lr.rps;
  shift += smp * lr.mstride;
  scale += smp * lr.mstride;
  const float *xr = x + r * ldx;
  float v[MAXV];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    int c = threadIdx.x + i * 256;
    v[i] = c < d ? xr[c] : 0.f;
    s += v[i];
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  s = warp_sum(s);
  if (lane == 0) red[w] = s;
  __syncthreads();
  const float mean = (red[0] + red[1] + red[2] + red[3]) / (float)d;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    int c = threadIdx.x + i * 256;
    float t = c < d ? v[i] - mean : 0.f;
    q += t * t;
  }
  q = warp_sum(q);
  if (lane == 0) red[4 + w] = q;
  __syncthreads();
  const float var = (red[4] + red[5] + red[6] + red[7]) / (float)d;
  const float rstd = rsqrtf(var + 1e-6f);
  T *hr = h + r * ldh;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    int c = threadIdx.x + i * 256;
    if (c < d) st<T>(hr + c, (v[i] - mean) * rstd * (1.f + scale[c]) + shift[c]);
  }
}

// ---------------------------------------------------------------- q/k preparation
// Sample blockIdx.z of a batched preparation: shifted source and destinations
template <typename T>
__device__ __forceinline__ void prep_sample(QKVPrepArgs &a) {
  const int64_t z = blockIdx.z;
  a.src = (const T *)a.src + z * a.src_bs;
  a.q = (T *)a.q + z * a.dst_bs;
  a.k = (T *)a.k + z * a.dst_bs;
  a.v = (T *)a.v + z * a.dst_bs;
}

// One thread per rotary pair (2p, 2p+1) of one head of one row. The hd/2
// threads of a head sit in one wavefront, so the RMS reduction is a shuffle.
// float32: v, whose layout is the same, goes along.
template <typename T, int HALF>
__global__ __launch_bounds__(256) void k_qk_prep(QKVPrepArgs a) {
  prep_sample<T>(a);
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int p = (int)(gid % HALF);
  const int64_t rh = gid / HALF;
  const int h = (int)(rh % a.heads);
  const int64_t r = rh / a.heads;
  const bool live = r < a.rows;
  const int64_t rr = live ? r : 0;
  const T *src = (const T *)a.src + rr * a.ld + (int64_t)h * a.hd + 2 * p;
  float q0 = ld<T>(src), q1 = ld<T>(src + 1);
  float k0 = ld<T>(src + a.d), k1 = ld<T>(src + a.d + 1);
  if (a.qk_norm) {
    float sq = q0 * q0 + q1 * q1, sk = k0 * k0 + k1 * k1;
#pragma unroll
    for (int o = HALF / 2; o > 0; o >>= 1) {
      sq += __shfl_xor(sq, o, 64);
      sk += __shfl_xor(sk, o, 64);
    }
    const float rq = rsqrtf(sq / (float)a.hd + 1e-6f), rk = rsqrtf(sk / (float)a.hd + 1e-6f);
    q0 *= rq;
    q1 *= rq;
    k0 *= rk;
    k1 *= rk;
  }
  const int64_t j = a.row0 + rr;  // joint-sequence index
  if (a.rope && j < a.n_video) {
    float2 cs = a.rope[j * HALF + p];
    float t0 = q0 * cs.x - q1 * cs.y, t1 = q0 * cs.y + q1 * cs.x;
    q0 = t0;
    q1 = t1;
    t0 = k0 * cs.x - k1 * cs.y;
    t1 = k0 * cs.y + k1 * cs.x;
    k0 = t0;
    k1 = t1;
  }
  if (!live) return;
  const int64_t o = ((int64_t)h * a.n_pad + j) * a.hd + 2 * p;
  st<T>((T *)a.q + o, q0);
  st<T>((T *)a.q + o + 1, q1);
  st<T>((T *)a.k + o, k0);
  st<T>((T *)a.k + o + 1, k1);
  if constexpr (sizeof(T) == 4) {
    ((T *)a.v)[o] = src[2 * a.d];
    ((T *)a.v)[o + 1] = src[2 * a.d + 1];
  }
}

// Position of key j in a V^T row: inside each aligned group of 16 keys the
// order is 0-3, 8-11, 4-7, 12-15 (bits 2 and 3 of j swapped), which makes the 8
// keys one lane feeds to an O^T = V^T P^T step one 16-byte chunk.
__device__ __forceinline__ int64_t vt_pos(int64_t j) { return (j & ~(int64_t)12) | ((j & 4) << 1) | ((j & 8) >> 1); }

// v rows -> transposed [H, hd, n_pad] through a 64-row LDS tile, so that both
// the reads (rows of the projection output) and the writes (runs of 64 tokens)
// are coalesced.
__global__ __launch_bounds__(256) void k_v_transpose(QKVPrepArgs a) {
  prep_sample<bf16_t>(a);
  __shared__ bf16_t tile[64][128 + 2];
  const int h = blockIdx.y;
  const int64_t r0 = (int64_t)blockIdx.x * 64;
  for (int idx = threadIdx.x; idx < 64 * a.hd; idx += 256) {
    int rr = idx / a.hd, e = idx % a.hd;
    int64_t r = r0 + rr;
    bf16_t val = 0;
    if (r < a.rows) val = ((const bf16_t *)a.src)[r * a.ld + 2 * a.d + (int64_t)h * a.hd + e];
    tile[rr][e] = val;
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < 64 * a.hd; idx += 256) {
    int e = idx / 64, rr = idx % 64;
    int64_t r = r0 + rr;
    if (r < a.rows) ((bf16_t *)a.v)[((int64_t)h * a.hd + e) * a.n_pad + vt_pos(a.row0 + r)] = tile[rr][e];
  }
}

// bf16 forms of the two kernels above with 16-byte accesses.
// q/k: one thread per 8 consecutive elements (4 rotary pairs) of one head row;
// the HD/8 threads of a head row are consecutive lanes of one wavefront, so the
// RMS reduction is a butterfly over them. Same arithmetic per element as
// k_qk_prep (float32, RMS scale, then rotation, one bf16 rounding).
__device__ __forceinline__ void unpack8(const uint4 &u, float (&x)[8]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] = __uint_as_float(w[i] << 16);
    x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
// eight floats -> bf16 (round to nearest even, four v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint4 pack8(const float (&x)[8]) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_v;
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    bf16x2_v p;
    p[0] = (__bf16)x[2 * i];
    p[1] = (__bf16)x[2 * i + 1];
    w[i] = __builtin_bit_cast(uint32_t, p);
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// (No fused multiply-adds in the norm and rotation arithmetic, here and in the
// GEMM's fused q/k epilogue, so both give the same bits.)
template <int HD>
__device__ __forceinline__ void qk_prep8(const QKVPrepArgs &a, int64_t block) {
#pragma clang fp contract(off)
  constexpr int TPH = HD / 8;              // threads per head row
  const int64_t gid = block * 256 + threadIdx.x;
  const int c = (int)(gid % TPH);
  const int64_t rh = gid / TPH;
  const int h = (int)(rh % a.heads);
  const int64_t r = rh / a.heads;
  const bool live = r < a.rows;
  const int64_t rr = live ? r : 0;
  const bf16_t *src = (const bf16_t *)a.src + rr * a.ld + (int64_t)h * HD + 8 * c;
  float q[8], k[8];
  unpack8(*(const uint4 *)src, q);
  unpack8(*(const uint4 *)(src + a.d), k);
  if (a.qk_norm) {
    float sq = 0.f, sk = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      sq += q[e] * q[e];
      sk += k[e] * k[e];
    }
    sq = group_sum<TPH>(sq);
    sk = group_sum<TPH>(sk);
    const float rq = rsqrtf(sq / (float)HD + 1e-6f), rk = rsqrtf(sk / (float)HD + 1e-6f);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      q[e] *= rq;
      k[e] *= rk;
    }
  }
  const int64_t j = a.row0 + rr;           // joint-sequence index
  if (a.rope && j < a.n_video) {
    const float4 *cs4 = (const float4 *)(a.rope + j * (HD / 2) + 4 * c);
    const float4 c01 = cs4[0], c23 = cs4[1];
    const float cs[8] = {c01.x, c01.y, c01.z, c01.w, c23.x, c23.y, c23.z, c23.w};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const float co = cs[2 * p], si = cs[2 * p + 1];
      float t0 = q[2 * p] * co - q[2 * p + 1] * si, t1 = q[2 * p] * si + q[2 * p + 1] * co;
      q[2 * p] = t0;
      q[2 * p + 1] = t1;
      t0 = k[2 * p] * co - k[2 * p + 1] * si;
      t1 = k[2 * p] * si + k[2 * p + 1] * co;
      k[2 * p] = t0;
      k[2 * p + 1] = t1;
    }
  }
  if (!live) return;
  const int64_t o = ((int64_t)h * a.n_pad + j) * HD + 8 * c;
  *(uint4 *)((bf16_t *)a.q + o) = pack8(q);
  *(uint4 *)((bf16_t *)a.k + o) = pack8(k);
}

// V^T through a 64-row LDS tile with 16-byte row reads and 16-byte writes of 8
// consecutive V^T positions. Needs row0 % 16 == 0: then the key order of
// vt_pos permutes tokens only inside each aligned group of 16 of this tile, and
// output position p holds token vt_pos(p) (the permutation is its own
// inverse). Groups of 16 with rows missing are written element by element,
// valid tokens only (their other positions are padding, zeroed separately).
template <int HD>
__device__ __forceinline__ void v_transpose8(const QKVPrepArgs &a, int64_t r0, int h) {
  __shared__ __attribute__((aligned(16))) bf16_t tile[64][HD + 8];
  for (int idx = threadIdx.x; idx < 64 * (HD / 8); idx += 256) {
    const int rr = idx / (HD / 8), c = idx % (HD / 8);
    const int64_t r = r0 + rr;
    uint4 val = make_uint4(0, 0, 0, 0);
    if (r < a.rows) val = *(const uint4 *)((const bf16_t *)a.src + r * a.ld + 2 * a.d + (int64_t)h * HD + 8 * c);
    *(uint4 *)&tile[rr][8 * c] = val;
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < HD * 8; idx += 256) {
    const int e = idx / 8, c = idx % 8;    // feature row, 8-position chunk of the tile
    int tok[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) tok[i] = (int)vt_pos(8 * c + i);
    bf16_t *dst = (bf16_t *)a.v + ((int64_t)h * HD + e) * a.n_pad + a.row0 + r0 + 8 * c;
    const int64_t group_end = r0 + (8 * c / 16) * 16 + 16;   // rows this chunk's group needs
    if (group_end <= a.rows) {
      uint32_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w[i] = (uint32_t)tile[tok[2 * i]][e] | ((uint32_t)tile[tok[2 * i + 1]][e] << 16);
      *(uint4 *)dst = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (r0 + tok[i] < a.rows) dst[i] = tile[tok[i]][e];
    }
  }
}

// q, k and v of all samples in one launch: the first qk_blocks blocks of a
// sample take q and k, the others one 64-row tile of one head of v each.
template <int HD>
__global__ __launch_bounds__(256) void k_qkv_prep8(QKVPrepArgs a, int qk_blocks) {
  prep_sample<bf16_t>(a);
  if ((int)blockIdx.x < qk_blocks) {
    qk_prep8<HD>(a, blockIdx.x);
  } else {
    const int b = (int)blockIdx.x - qk_blocks;
    v_transpose8<HD>(a, (int64_t)(b / a.heads) * 64, b % a.heads);
  }
}

// Zero rows (keys) [n, n_pad) of head blockIdx.x of q (blockIdx.y 0), k (1) or v
// (2). Rows of q, k and a row-major v are one contiguous run per head; of V^T
// each feature row has the keys of the group of 16 that n falls in, at their
// permuted positions, then a contiguous run.
template <typename T, bool VT>
__global__ __launch_bounds__(256) void k_qkv_pad(T *q, T *k, T *v, int hd, int64_t n, int64_t n_pad) {
  T *p = (blockIdx.y == 0 ? q : blockIdx.y == 1 ? k : v) + (int64_t)blockIdx.x * n_pad * hd;
  constexpr int V = 16 / sizeof(T);
  const uint4 zero = make_uint4(0, 0, 0, 0);
  if (!VT || blockIdx.y < 2) {
    uint4 *p4 = (uint4 *)(p + n * hd);     // hd is a multiple of V
    for (int64_t i = threadIdx.x; i < (n_pad - n) * hd / V; i += 256) p4[i] = zero;
    return;
  }
  const int64_t g = min((n + 15) / 16 * 16, n_pad);
  for (int e = threadIdx.x >> 4; e < hd; e += 16) {
    T *row = p + e * n_pad;
    const int64_t j = g - 16 + (threadIdx.x & 15);
    if (j >= n) row[vt_pos(j)] = 0;
    for (int64_t i = g + V * (threadIdx.x & 15); i < n_pad; i += 16 * V) *(uint4 *)(row + i) = zero;
  }
}

// ---------------------------------------------------------------- conditioning products
// Matrix-vector products of the conditioning path, bound by the weight stream
// (each weight is read once for up to four samples). The input vectors are
// staged in LDS once per block, activation applied there: computing SiLU in
// every wave cost more than its weights' loads (a 18,432 x 3,072 modulation
// 57 us, 2.0 TB/s; 35 us here). Sums run in one fixed order (explicit fused
// multiply-adds, lane by lane, then the butterfly), so a sample's result does
// not depend on how many share the launch. The 8 (float32: 4) products of a
// 16-byte load are summed before they meet the lane's sum: one rounding at its
// size per load and not per product.
// CH input elements per sample are in LDS at a time; a chunk's weights are
// requested before the barriers of its staging, so they travel under it.

// acc[r][b] += the lane's part of sum_j w[r][j] x_b[j]; fill(b, j) gives x_b[j]
template <typename T, int R, int NB, int CH, class Fill>
__device__ __forceinline__ void gv_dot(const T *const (&w)[R], int k, bool vec, float *xs, const Fill &fill,
                                       float (&acc)[R][NB]) {
  constexpr int V = 16 / sizeof(T), IT = CH / (64 * V);
  static_assert(IT >= 1 && CH % (64 * V) == 0, "whole 16-byte loads of a wave");
  const int lane = threadIdx.x & 63;
  for (int c0 = 0; c0 < k; c0 += CH) {
    const int n = min(CH, k - c0);
    uint4 u[IT][R];
    if (vec)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int j = (it * 64 + lane) * V;
#pragma unroll
        for (int r = 0; r < R; ++r) u[it][r] = j < n ? *(const uint4 *)(w[r] + c0 + j) : make_uint4(0, 0, 0, 0);
      }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b)
      for (int i = threadIdx.x; i < n; i += 256) xs[b * CH + i] = fill(b, c0 + i);
    __syncthreads();
    if (vec) {
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int j = (it * 64 + lane) * V;
        if (j >= n) break;
        float x[NB][V];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int e = 0; e < V; e += 4) *(float4 *)&x[b][e] = *(const float4 *)&xs[b * CH + j + e];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const uint32_t uu[4] = {u[it][r].x, u[it][r].y, u[it][r].z, u[it][r].w};
          float t[NB];
#pragma unroll
          for (int e = 0; e < V; ++e) {
            const float wv = sizeof(T) == 4 ? __uint_as_float(uu[e % 4])
                                            : __uint_as_float(e & 1 ? uu[e / 2] & 0xffff0000u : uu[e / 2] << 16);
#pragma unroll
            for (int b = 0; b < NB; ++b) t[b] = e == 0 ? wv * x[b][0] : fmaf(wv, x[b][e], t[b]);
          }
#pragma unroll
          for (int b = 0; b < NB; ++b) acc[r][b] += t[b];
        }
      }
    } else {
      for (int j = lane; j < n; j += 64)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float wv = ld<T>(w[r] + c0 + j);
#pragma unroll
          for (int b = 0; b < NB; ++b) acc[r][b] = fmaf(wv, xs[b * CH + j], acc[r][b]);
        }
    }
  }
}

template <typename T>
__device__ __forceinline__ bool gv_vec(const void *w, int k) {
  return k % (16 / (int)sizeof(T)) == 0 && (uintptr_t)w % 16 == 0;
}

// Modulation vectors of the listed weights for NB samples: y_b[i] = W[i, :] SiLU(x_b) + bias[i]
// R rows per wave: 8 where the rows are many and long (each staged input then
// serves 32 of them: 18,432 x 3,072 35 us against 42 with 2), else 2 (51,200 x
// 1,024: 26 us against 28 with 8)
template <typename T, int NB, int R>
__global__ __launch_bounds__(256) void k_mod(ModArgs a) {
  constexpr int CH = 1024;
  __shared__ __attribute__((aligned(16))) float xs[NB * CH];
  // the block's rows lie in one entry of one section (rows % 32 == 0)
  int64_t row = (int64_t)blockIdx.x * 4 * R;
  int s = 0;
  while (s + 1 < a.nsec && row >= (int64_t)a.sec[s].rows * a.sec[s].count) {
    row -= (int64_t)a.sec[s].rows * a.sec[s].count;
    ++s;
  }
  const ModSec sec = a.sec[s];
  const int64_t entry = row / sec.rows;
  const int r0 = (int)(row - entry * sec.rows) + R * (threadIdx.x >> 6), b0 = blockIdx.y * NB;
  const T *w0 = (const T *)((const char *)sec.w + entry * sec.stride);
  const T *bias = (const T *)((const char *)sec.b + entry * sec.stride);
  const T *w[R];
#pragma unroll
  for (int r = 0; r < R; ++r) w[r] = w0 + (int64_t)(r0 + r) * a.k;
  float acc[R][NB] = {};
  gv_dot<T, R, NB, CH>(w, a.k, gv_vec<T>(sec.w, a.k) && sec.stride % 16 == 0, xs,
                   [&](int b, int j) { return silu(a.x[(int64_t)min(b0 + b, a.nb - 1) * a.k + j]); }, acc);
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float v = warp_sum(acc[r][b]);
      if ((threadIdx.x & 63) == 0 && b0 + b < a.nb)
        a.y[(b0 + b) * a.ys + sec.yoff + entry * sec.ystep + r0 + r] = v + ld<T>(bias + r0 + r);
    }
}

// y = SiLU(fc1 * sinusoid(1000 t) + bias): 128 frequencies 1e4^(-j/128), cosines then
// sines, in float64 by every block (a separate launch cost more)
template <typename T>
__global__ __launch_bounds__(256) void k_cond1(const T *w, const T *bias, double t, float *y, int n) {
  __shared__ __attribute__((aligned(16))) float xs[512];
  __shared__ float feat[256];
  const int j = threadIdx.x & 127;
  const double arg = 1000.0 * t * exp(-log(10000.0) * (double)j / 128.0);
  feat[threadIdx.x] = threadIdx.x < 128 ? (float)cos(arg) : (float)sin(arg);
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const T *wr[1] = {w + (int64_t)min(row, n - 1) * 256};
  float acc[1][1] = {};
  gv_dot<T, 1, 1, 512>(wr, 256, true, xs, [&](int, int i) { return feat[i]; }, acc);
  const float v = warp_sum(acc[0][0]);
  if ((threadIdx.x & 63) == 0 && row < n) y[row] = silu(v + ld<T>(bias + row));
}

// out_b = fc2 tmp + bias2 (+ Wc cond_b + bias_c) (+ Wm cam_b + bias_m): the
// three products of the conditioning vector in one launch, one row per wave so
// that 3,072 rows keep 3,072 waves loading
template <typename T, int NB>
__global__ __launch_bounds__(256) void k_cond2(CondArgs a) {
  constexpr int CH = NB == 1 ? 4096 : 2048;
  __shared__ __attribute__((aligned(16))) float xs[NB * CH];
  const int rw = blockIdx.x * 4 + (threadIdx.x >> 6), row = min(rw, a.n - 1), b0 = blockIdx.y * NB;
  float out[NB] = {};
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int k = s == 0 ? a.n : s == 1 ? a.cond_dim : a.cam_dim;
    if (k == 0) continue;
    const T *w = (const T *)a.w[s], *bias = (const T *)a.b[s];
    const T *wr[1] = {w + (int64_t)row * k};
    float acc[1][NB] = {};
    if (s == 0) {
      // the same input for every sample
      float one[1][1] = {};
      gv_dot<T, 1, 1, CH>(wr, k, gv_vec<T>(w, k), xs, [&](int, int j) { return a.tmp[j]; }, one);
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[0][b] = one[0][0];
    } else {
      const void *const *xp = s == 1 ? a.cond : a.cam;
      gv_dot<T, 1, NB, CH>(wr, k, gv_vec<T>(w, k), xs,
                       [&](int b, int j) { return ld<T>((const T *)xp[min(b0 + b, a.nb - 1)] + j); }, acc);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) out[b] += warp_sum(acc[0][b]) + ld<T>(bias + row);
  }
  if ((threadIdx.x & 63) == 0 && rw < a.n)
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (b0 + b < a.nb) a.y[(int64_t)(b0 + b) * a.n + row] = out[b];
}

template <typename T>
__global__ void k_to_f32(const T *src, float *dst, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = ld<T>(src + i);
}

// ---------------------------------------------------------------- patches
// Sample blockIdx.y of the launch; I: index type (32-bit divisions where a
// sample's elements allow it: 8 samples of 172,032 elements 8.2 us against 10.7).
template <typename T, typename I>
__global__ void k_patchify(SamplePtrs zs, T *__restrict__ out, int c, int f, int h, int w, int pt, int ph, int pw) {
  const float *__restrict__ z = (const float *)zs.p[blockIdx.y];
  const unsigned hp = h / ph, wp = w / pw, P = c * pt * ph * pw;
  const I total = (I)(f / pt) * hp * wp * P;
  const I i = (I)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  out += (int64_t)blockIdx.y * total;
  const unsigned feat = (unsigned)(i % P);
  const I n = i / P;
  const unsigned wq = (unsigned)(n % wp), hq = (unsigned)(n / wp % hp), fq = (unsigned)(n / wp / hp);
  const unsigned jj = feat % pw, ii = feat / pw % ph, aa = feat / pw / ph % pt, cc = feat / pw / ph / pt;
  const I src = (((I)cc * f + (fq * pt + aa)) * h + (hq * ph + ii)) * w + (wq * pw + jj);
  st<T>(out + i, z[src]);
}

template <typename I>
__global__ void k_unpatchify(const float *__restrict__ tok, SamplePtrs vs, int c, int f, int h, int w, int pt, int ph,
                             int pw) {
  float *__restrict__ v = (float *)vs.p[blockIdx.y];
  const I total = (I)c * f * h * w;
  const I i = (I)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  tok += (int64_t)blockIdx.y * total;
  const unsigned x = (unsigned)(i % w), y = (unsigned)(i / w % h), fr = (unsigned)(i / w / h % f), cc = (unsigned)(i / w / h / f);
  const unsigned hp = h / ph, wp = w / pw;
  const I n = ((I)(fr / pt) * hp + (y / ph)) * wp + (x / pw);
  const unsigned feat = ((cc * pt + fr % pt) * ph + y % ph) * pw + x % pw;
  v[i] = tok[n * (I)(c * pt * ph * pw) + feat];
}

// ---------------------------------------------------------------- seeded normal fill
// splitmix64 of (seed, counter) -> two 32-bit uniforms -> Box-Muller.
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  x += 0x9e3779b97f4a7c15ull;
  x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
  x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
  return x ^ (x >> 31);
}

template <typename T>
__global__ void k_fill_normal(T *dst, int64_t n, uint64_t seed, uint64_t offset, float std) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    uint64_t r = splitmix64(seed * 0x632be59bd9b4e019ull + offset + (uint64_t)i);
    float u1 = ((uint32_t)(r >> 32) + 1.0f) * 2.3283064365386963e-10f;  // (0, 1]
    float u2 = (uint32_t)r * 2.3283064365386963e-10f;
    float g = sqrtf(-2.f * logf(u1)) * cosf(6.283185307179586f * u2);
    st<T>(dst + i, g * std);
  }
}

inline unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }
}  // namespace

// Vector form (d % 4 == 0, 16-byte aligned rows): thread t owns the float4
// groups t, t + 256, ... of the row; bf16 output goes out as 8-byte groups.
template <typename T>
__device__ __forceinline__ void st4(T *p, float a, float b, float c, float d);
template <>
__device__ __forceinline__ void st4<bf16_t>(bf16_t *p, float a, float b, float c, float d) {
  *(uint2 *)p = make_uint2((uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16), (uint32_t)f2bf(c) | ((uint32_t)f2bf(d) << 16));
}
template <>
__device__ __forceinline__ void st4<float>(float *p, float a, float b, float c, float d) {
  *(float4 *)p = make_float4(a, b, c, d);
}

template <typename T, int NV4>
__global__ __launch_bounds__(256) void k_ln_mod4(const float *__restrict__ x, int64_t ldx, T *__restrict__ h,
                                                int64_t ldh, LnRows lr, int d, const float *__restrict__ shift,
                                                const float *__restrict__ scale) {
  __shared__ float red[8];
  const int64_t i = blockIdx.x;
  const int64_t smp = i / lr.rps;
  const int64_t r = smp * lr.sstride + i % lr.rps;
  shift += smp * lr.mstride;
  scale += smp * lr.mstride;
  const float4 *xr = (const float4 *)(x + r * ldx);
  const int d4 = d >> 2;
  float4 v[NV4];
  float s = 0.f;
#pragma unroll
  for (int k = 0; k < NV4; ++k) {
    const int c = threadIdx.x + k * 256;
    v[k] = c < d4 ? xr[c] : make_float4(0.f, 0.f, 0.f, 0.f);
    s += (v[k].x + v[k].y) + (v[k].z + v[k].w);
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  s = warp_sum(s);
  if (lane == 0) red[w] = s;
  __syncthreads();
  const float mean = (red[0] + red[1] + red[2] + red[3]) / (float)d;
  float q = 0.f;
#pragma unroll
  for (int k = 0; k < NV4; ++k) {
    const int c = threadIdx.x + k * 256;
    if (c < d4) {
      const float a = v[k].x - mean, b = v[k].y - mean, e = v[k].z - mean, f = v[k].w - mean;
      q += (a * a + b * b) + (e * e + f * f);
    }
  }
  q = warp_sum(q);
  if (lane == 0) red[4 + w] = q;
  __syncthreads();
  const float var = (red[4] + red[5] + red[6] + red[7]) / (float)d;
  const float rstd = rsqrtf(var + 1e-6f);
  T *hr = h + r * ldh;
#pragma unroll
  for (int k = 0; k < NV4; ++k) {
    const int c = threadIdx.x + k * 256;
    if (c < d4) {
      const float4 sh = ((const float4 *)shift)[c], sc = ((const float4 *)scale)[c];
      st4<T>(hr + 4 * c, (v[k].x - mean) * rstd * (1.f + sc.x) + sh.x, (v[k].y - mean) * rstd * (1.f + sc.y) + sh.y,
             (v[k].z - mean) * rstd * (1.f + sc.z) + sh.z, (v[k].w - mean) * rstd * (1.f + sc.w) + sh.w);
    }
  }
}

hipError_t launch_ln_mod(int dtype, const float *x, int64_t ldx, void *h, int64_t ldh, const LnRows &r, int d,
                         const float *shift, const float *scale, hipStream_t s) {
  if (r.rows <= 0) return hipSuccess;
  if (d > 16 * 256 || r.rps <= 0 || r.sstride < r.rps) return hipErrorInvalidValue;
  dim3 g((unsigned)r.rows), b(256);
  const bool vec = d % 4 == 0 && ldx % 4 == 0 && ldh % 4 == 0 && r.mstride % 4 == 0 && (uintptr_t)x % 16 == 0 &&
                   (uintptr_t)h % 16 == 0 && (uintptr_t)shift % 16 == 0 && (uintptr_t)scale % 16 == 0;
  if (vec) {
    if (dtype == 1) {
      if (d <= 4 * 256)
        hipLaunchKernelGGL((k_ln_mod4<bf16_t, 1>), g, b, 0, s, x, ldx, (bf16_t *)h, ldh, r, d, shift, scale);
      else
        hipLaunchKernelGGL((k_ln_mod4<bf16_t, 4>), g, b, 0, s, x, ldx, (bf16_t *)h, ldh, r, d, shift, scale);
    } else {
      if (d <= 4 * 256)
        hipLaunchKernelGGL((k_ln_mod4<float, 1>), g, b, 0, s, x, ldx, (float *)h, ldh, r, d, shift, scale);
      else
        hipLaunchKernelGGL((k_ln_mod4<float, 4>), g, b, 0, s, x, ldx, (float *)h, ldh, r, d, shift, scale);
    }
    return hipGetLastError();
  }
  if (dtype == 1) {
    if (d <= 4 * 256)
      hipLaunchKernelGGL((k_ln_mod<bf16_t, 4>), g, b, 0, s, x, ldx, (bf16_t *)h, ldh, r, d, shift, scale);
    else
      hipLaunchKernelGGL((k_ln_mod<bf16_t, 16>), g, b, 0, s, x, ldx, (bf16_t *)h, ldh, r, d, shift, scale);
  } else {
    if (d <= 4 * 256)
      hipLaunchKernelGGL((k_ln_mod<float, 4>), g, b, 0, s, x, ldx, (float *)h, ldh, r, d, shift, scale);
    else
      hipLaunchKernelGGL((k_ln_mod<float, 16>), g, b, 0, s, x, ldx, (float *)h, ldh, r, d, shift, scale);
  }
  return hipGetLastError();
}

hipError_t launch_qkv_prep(int dtype, const QKVPrepArgs &a, hipStream_t s) {
  if (a.rows <= 0 || a.nb <= 0) return hipSuccess;
  if (a.hd != 64 && a.hd != 128) return hipErrorInvalidValue;
  const dim3 g(nblk(a.rows * a.heads * (a.hd / 2), 256), 1, a.nb), b(256);
  if (dtype == 1) {
    // 16-byte forms when every row and head start is 16-byte aligned
    const bool vec = (uintptr_t)a.src % 16 == 0 && a.ld % 8 == 0 && a.d % 8 == 0 && (uintptr_t)a.q % 16 == 0 &&
                     (uintptr_t)a.k % 16 == 0 && (uintptr_t)a.v % 16 == 0 && a.n_pad % 8 == 0 &&
                     a.src_bs % 8 == 0 && a.dst_bs % 8 == 0 && (a.rope == nullptr || (uintptr_t)a.rope % 16 == 0);
    if (vec && a.row0 % 16 == 0) {
      const unsigned nq = nblk(a.rows * a.heads * (a.hd / 8), 256);
      const dim3 g8(nq + nblk(a.rows, 64) * a.heads, 1, a.nb);
      if (a.hd == 64)
        hipLaunchKernelGGL(k_qkv_prep8<64>, g8, b, 0, s, a, (int)nq);
      else
        hipLaunchKernelGGL(k_qkv_prep8<128>, g8, b, 0, s, a, (int)nq);
      return hipGetLastError();
    }
    if (vec) {
      const unsigned nq = nblk(a.rows * a.heads * (a.hd / 8), 256);
      if (a.hd == 64)
        hipLaunchKernelGGL(k_qkv_prep8<64>, dim3(nq, 1, a.nb), b, 0, s, a, (int)nq);
      else
        hipLaunchKernelGGL(k_qkv_prep8<128>, dim3(nq, 1, a.nb), b, 0, s, a, (int)nq);
    } else if (a.hd == 64) {
      hipLaunchKernelGGL((k_qk_prep<bf16_t, 32>), g, b, 0, s, a);
    } else {
      hipLaunchKernelGGL((k_qk_prep<bf16_t, 64>), g, b, 0, s, a);
    }
    hipLaunchKernelGGL(k_v_transpose, dim3(nblk(a.rows, 64), a.heads, a.nb), b, 0, s, a);
  } else {
    if (a.hd == 64)
      hipLaunchKernelGGL((k_qk_prep<float, 32>), g, b, 0, s, a);
    else
      hipLaunchKernelGGL((k_qk_prep<float, 64>), g, b, 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_qkv_pad(int dtype, void *q, void *k, void *v, int heads, int hd, int64_t n, int64_t n_pad,
                          hipStream_t s) {
  if (n_pad <= n || heads <= 0) return hipSuccess;
  const dim3 g((unsigned)heads, 3), b(256);
  if (dtype == 1)
    hipLaunchKernelGGL((k_qkv_pad<bf16_t, true>), g, b, 0, s, (bf16_t *)q, (bf16_t *)k, (bf16_t *)v, hd, n, n_pad);
  else
    hipLaunchKernelGGL((k_qkv_pad<float, false>), g, b, 0, s, (float *)q, (float *)k, (float *)v, hd, n, n_pad);
  return hipGetLastError();
}

// samples of one launch share the weight reads four (or two) at a time
template <template <typename, int> class Launch, typename A>
hipError_t by_samples(int dtype, const A &a, hipStream_t s) {
  if (dtype == 1) {
    if (a.nb > 2) return Launch<bf16_t, 4>::run(a, s);
    return a.nb == 2 ? Launch<bf16_t, 2>::run(a, s) : Launch<bf16_t, 1>::run(a, s);
  }
  if (a.nb > 2) return Launch<float, 4>::run(a, s);
  return a.nb == 2 ? Launch<float, 2>::run(a, s) : Launch<float, 1>::run(a, s);
}

template <typename T, int NB>
struct LaunchMod {
  static hipError_t run(const ModArgs &a, hipStream_t s) {
    int64_t rows = 0;
    for (int i = 0; i < a.nsec; ++i) {
      if (a.sec[i].rows % 32 != 0) return hipErrorInvalidValue;
      rows += (int64_t)a.sec[i].rows * a.sec[i].count;
    }
    const unsigned gy = (unsigned)((a.nb + NB - 1) / NB);
    if (rows >= 32 * 256 && a.k > 1024)
      hipLaunchKernelGGL((k_mod<T, NB, 8>), dim3((unsigned)(rows / 32), gy), dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL((k_mod<T, NB, 2>), dim3((unsigned)(rows / 8), gy), dim3(256), 0, s, a);
    return hipGetLastError();
  }
};
template <typename T, int NB>
struct LaunchCond {
  static hipError_t run(const CondArgs &a, hipStream_t s) {
    const unsigned g = nblk(a.n, 4);
    hipLaunchKernelGGL(k_cond1<T>, dim3(g), dim3(256), 0, s, (const T *)a.w1, (const T *)a.b1, a.t, a.tmp, a.n);
    hipLaunchKernelGGL((k_cond2<T, NB>), dim3(g, (unsigned)((a.nb + NB - 1) / NB)), dim3(256), 0, s, a);
    return hipGetLastError();
  }
};

hipError_t launch_mod(int dtype, const ModArgs &a, hipStream_t s) { return by_samples<LaunchMod>(dtype, a, s); }
hipError_t launch_cond(int dtype, const CondArgs &a, hipStream_t s) { return by_samples<LaunchCond>(dtype, a, s); }

hipError_t launch_to_f32(int dtype, const void *src, float *dst, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (dtype == 1)
    hipLaunchKernelGGL((k_to_f32<bf16_t>), dim3(nblk(n, 256)), dim3(256), 0, s, (const bf16_t *)src, dst, n);
  else
    hipLaunchKernelGGL((k_to_f32<float>), dim3(nblk(n, 256)), dim3(256), 0, s, (const float *)src, dst, n);
  return hipGetLastError();
}

hipError_t launch_patchify(int dtype, const SamplePtrs &z, int nb, void *out, int c, int f, int h, int w, int pt, int ph,
                           int pw, hipStream_t s) {
  const int64_t total = (int64_t)c * f * h * w;
  const dim3 g(nblk(total, 256), nb), b(256);
  const bool i32 = total < (int64_t(1) << 31);
  if (dtype == 1 && i32)
    hipLaunchKernelGGL((k_patchify<bf16_t, uint32_t>), g, b, 0, s, z, (bf16_t *)out, c, f, h, w, pt, ph, pw);
  else if (dtype == 1)
    hipLaunchKernelGGL((k_patchify<bf16_t, uint64_t>), g, b, 0, s, z, (bf16_t *)out, c, f, h, w, pt, ph, pw);
  else if (i32)
    hipLaunchKernelGGL((k_patchify<float, uint32_t>), g, b, 0, s, z, (float *)out, c, f, h, w, pt, ph, pw);
  else
    hipLaunchKernelGGL((k_patchify<float, uint64_t>), g, b, 0, s, z, (float *)out, c, f, h, w, pt, ph, pw);
  return hipGetLastError();
}

hipError_t launch_unpatchify(const float *tok, const SamplePtrs &v, int nb, int c, int f, int h, int w, int pt, int ph,
                             int pw, hipStream_t s) {
  const int64_t total = (int64_t)c * f * h * w;
  const dim3 g(nblk(total, 256), nb), b(256);
  if (total < (int64_t(1) << 31))
    hipLaunchKernelGGL(k_unpatchify<uint32_t>, g, b, 0, s, tok, v, c, f, h, w, pt, ph, pw);
  else
    hipLaunchKernelGGL(k_unpatchify<uint64_t>, g, b, 0, s, tok, v, c, f, h, w, pt, ph, pw);
  return hipGetLastError();
}

hipError_t launch_fill_normal(int dtype, void *dst, int64_t n, uint64_t seed, uint64_t offset, float std,
                              hipStream_t s) {
  if (n <= 0) return hipSuccess;
  unsigned g = nblk(n, 256);
  if (g > 65536) g = 65536;
  if (dtype == 1)
    hipLaunchKernelGGL((k_fill_normal<bf16_t>), dim3(g), dim3(256), 0, s, (bf16_t *)dst, n, seed, offset, std);
  else
    hipLaunchKernelGGL((k_fill_normal<float>), dim3(g), dim3(256), 0, s, (float *)dst, n, seed, offset, std);
  return hipGetLastError();
}

}  // namespace wdc

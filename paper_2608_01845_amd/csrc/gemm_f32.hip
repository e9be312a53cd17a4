// float32 GEMMs of the denoiser on the matrix cores: c[m, n] = sum_k a[m, k] *
// w[n, k] + bias[n] with the epilogues of common.h, every product and sum in
// float32 (v_mfma_f32_32x32x2_f32, 32x32 tiles of 64 cycles, 157 TFLOP/s on
// the whole card: twice what the vector units reach).
//
//  * k_gemm_f32_tile: BM x BN block tiles, 4 waves, K stages of 32 floats (one
//    128-byte row per tile row) straight from HBM into LDS, three buffers, one
//    barrier per stage. At 64 cycles per MFMA neither LDS (one 16-byte read per
//    lane for 4 MFMAs of a 32 x 32 tile) nor the loads bind; what costs is a
//    partly filled last dispatch round, so launch_gemm_f32 chooses the tile size
//    by that. 2,688 x 3,072, K = 1,024: 153 us, 111 TFLOP/s (LDS-tiled FMA
//    kernel: 350 us).
//  * k_gemm_f32_small: products that would leave compute units idle even on
//    64 x 64 tiles. T x T output tile (16 or 32) per block, its four waves
//    taking a quarter of K each straight from global memory, combined through
//    LDS in wave order. These are bound by latency: the many small blocks keep
//    every CU loading, and no stage waits for a barrier. 256 x 256, K = 1,024: 5.9 us
//    (LDS-tiled FMA kernel: 190 us, 16 blocks).
#include "common.h"

namespace wdc {

namespace {

constexpr int BK = 32;                  // K per LDS stage: one 128-byte row of float32
constexpr int RSRC_WORD3 = 0x00020000;  // raw buffer: 32-bit data format, no swizzle
constexpr int NBUF = 3;
// s_waitcnt vmcnt(n), other counters untouched (n <= 15)
__host__ __device__ constexpr int vm_wait(int n) { return 0x0F70 | n; }

typedef __attribute__((address_space(3))) void lds_void;
__device__ __forceinline__ void lds_load16(__amdgpu_buffer_rsrc_t r, char *lds, int voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void *)lds, 16, voff, soff, 0, 0);
}

// Every kernel sums K in the same order, so that an output's bits do not depend on
// the rows it shares its call with (the tile forms are chosen by their number): K
// is cut into units of 16, unit u belongs to part w while u < units (w + 1) / 4,
// a part's sum is a chain over its units, k = q, 4 + q, 8 + q, 12 + q for q = 0..3
// within one, and the parts are added from the first to the last. One
// v_mfma_f32_16x16x4 takes four terms in order, v_mfma_f32_32x32x2 two. Against one
// chain over all of K in the tiles: 8,192 x 4,096, K = 4,096 1.98 ms for 1.96, 700 x
// 2,048, K = 2,048 (64 x 64 tiles) 78.8 us for 76.8, and half the rounding error.
constexpr int KU = 16;
__device__ __forceinline__ int part_begin(int units, int w) { return units * w / 4; }

// chunk c (16 bytes) of tile row r lives at c ^ ((r >> 1) & 7) of its 128-byte row
__device__ __forceinline__ int swz(int row, int chunk) { return (row * 8 + (chunk ^ ((row >> 1) & 7))) * 16; }

__device__ __forceinline__ GemmArgs batch_entry(const GemmArgs &g0) {
  GemmArgs g = g0;
  const int64_t z = blockIdx.z;
  if (z) {
    g.a = (const float *)g0.a + z * g0.a_bs;
    g.c = (float *)g0.c + z * g0.c_bs;
    if (g0.gate) g.gate = g0.gate + z * g0.gate_bs;
  }
  return g;
}

// EPI: EPI_STORE (also EPI_STORE_F32), EPI_GELU or EPI_GATE_RES
template <int EPI>
__device__ __forceinline__ float finish(float acc, float bias, float gate, float x) {
  const float v = acc + bias;
  if (EPI == EPI_GELU) return gelu_tanh(v);
  if (EPI == EPI_GATE_RES) return x + gate * v;
  return v;
}

template <int BM, int BN, int EPI>
__global__ __launch_bounds__(256) void k_gemm_f32_tile(GemmArgs g0) {
  constexpr int TM = BM / 64, TN = BN / 64;             // 32 x 32 tiles of a wave (2 x 2 waves)
  constexpr int A_CH = BM / 32, B_CH = BN / 32;         // 1 KB stripes per wave and stage
  constexpr int SL = A_CH + B_CH, STAGE = (BM + BN) * 128;
  const GemmArgs g = batch_entry(g0);
  extern __shared__ __attribute__((aligned(16))) char smem[];

  // groups of 8 M tiles walk the N tiles, so that blocks running together share operand panels in L2
  const int n_tiles = (int)((g.n + BN - 1) / BN), m_tiles = (int)((g.m + BM - 1) / BM);
  const int bid = blockIdx.x, first_m = bid / (8 * n_tiles) * 8;
  const int gsize = min(m_tiles - first_m, 8), in = bid % (8 * n_tiles);
  const int64_t m0 = (int64_t)(first_m + in % gsize) * BM, n0 = (int64_t)(in / gsize) * BN;

  const int lane = threadIdx.x & 63, wu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wu >> 1, wn = wu & 1, lr = lane & 31, lg = lane >> 5;

  // rows past m (n) lie past the descriptor's range and read as zero
  const __amdgpu_buffer_rsrc_t a_desc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)((const float *)g.a + m0 * g.lda), (short)0, (int)(min((int64_t)BM, g.m - m0) * g.lda * 4), RSRC_WORD3);
  const __amdgpu_buffer_rsrc_t b_desc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)((const float *)g.w + n0 * g.k), (short)0, (int)(min((int64_t)BN, g.n - n0) * g.k * 4), RSRC_WORD3);
  // stripe s = w + 4 i holds tile rows 8 s .. 8 s + 7; a lane fetches the logical
  // chunk that the swizzle puts at physical chunk lane % 8 (same key for every i)
  const int lch = (lane & 7) ^ ((4 * (wu & 1) + (lane >> 4)) & 7);
  const int row0 = 8 * wu + (lane >> 3);
  const int va = row0 * (int)g.lda * 4 + lch * 16, a_step = 32 * (int)g.lda * 4;
  const int vb = row0 * (int)g.k * 4 + lch * 16, b_step = 32 * (int)g.k * 4;
  auto load = [&](int buf, int kt) {
    char *s = smem + buf * STAGE + wu * 1024;
#pragma unroll
    for (int i = 0; i < A_CH; ++i) lds_load16(a_desc, s + i * 4096, va + i * a_step, kt * BK * 4);
#pragma unroll
    for (int i = 0; i < B_CH; ++i) lds_load16(b_desc, s + BM * 128 + i * 4096, vb + i * b_step, kt * BK * 4);
  };

  f32x16 acc[TM][TN], tot[TM][TN];                      // the part in progress, the parts before it
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) tot[i][j][e] = 0.f;

  const int ra = swz(wm * (BM / 2) + lr, lg), rb = BM * 128 + swz(wn * (BN / 2) + lr, lg);
  struct Frag {
    f32x4 a[2][TM], b[2][TN];
  };
  auto read = [&](Frag &f, const char *s, int h) {        // unit h of a stage
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int s8 = 2 * h + p;
#pragma unroll
      for (int i = 0; i < TM; ++i) f.a[p][i] = *(const f32x4 *)(s + (ra ^ (32 * s8)) + i * 32 * 128);
#pragma unroll
      for (int j = 0; j < TN; ++j) f.b[p][j] = *(const f32x4 *)(s + BM * 128 + ((rb - BM * 128) ^ (32 * s8)) + j * 32 * 128);
    }
  };
  // lane group lg holds k = 8 p + 4 lg + q of the unit: an MFMA takes k = 8 p + q and 8 p + 4 + q
  auto mul = [&](const Frag &f) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[p][i][q], f.b[p][j][q], acc[i][j], 0, 0, 0);
  };
  auto unit = [&](const char *s, int h) {
    Frag f;
    read(f, s, h);
    mul(f);
  };
  const int nk = (int)(g.k / BK);
  load(0, 0);
  if (nk > 1) load(1, 1);
  int buf = 0;                                            // of the stage in use
  auto begin_stage = [&](int kt) {
    // stage kt is in LDS once no more than the next stage's loads are pending;
    // after the barrier every wave is also done with the buffer of stage kt - 1,
    // which takes stage kt + 2
    if (kt + 1 < nk) __builtin_amdgcn_s_waitcnt(vm_wait(SL));
    else __builtin_amdgcn_s_waitcnt(vm_wait(0));
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const int nbuf = buf == 0 ? NBUF - 1 : buf - 1;
    if (kt + 2 < nk) load(nbuf, kt + 2);
  };
  auto end_stage = [&] { buf = buf == NBUF - 1 ? 0 : buf + 1; };
  // A loop per part, in which only MFMAs touch the accumulators (a test for the
  // next part inside one loop over the stages made the compiler copy them in and
  // out in every stage: 8,192 x 4,096, K = 4,096 2.25 ms), and both units' reads in
  // front of the first MFMA, which needs fragments of both halves of its unit. A part
  // begins or ends within a stage where K is not a multiple of 128.
  const int units = (int)(g.k / KU);
#pragma unroll 1
  for (int w = 0; w < 4; ++w) {
    int u = part_begin(units, w);
    const int ue = part_begin(units, w + 1);
    if (u == ue) continue;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    if (u & 1) {
      unit(smem + buf * STAGE, 1);
      end_stage();
      ++u;
    }
#pragma unroll 1
    for (; u + 2 <= ue; u += 2) {
      begin_stage(u >> 1);
      Frag f[2];
      read(f[0], smem + buf * STAGE, 0);
      read(f[1], smem + buf * STAGE, 1);
      __builtin_amdgcn_sched_barrier(0);
      mul(f[0]);
      mul(f[1]);
      end_stage();
    }
    if (u < ue) {
      begin_stage(u >> 1);
      unit(smem + buf * STAGE, 0);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) tot[i][j][e] += acc[i][j][e];
  }

  // lane: column lr of each 32 x 32 tile, rows 8 (e / 4) + 4 lg + e % 4
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int64_t col = n0 + wn * (BN / 2) + j * 32 + lr;
    if (col >= g.n) continue;
    const float bv = g.bias ? ((const float *)g.bias)[col] : 0.f, gv = EPI == EPI_GATE_RES ? g.gate[col] : 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int64_t rb0 = m0 + wm * (BM / 2) + i * 32 + 4 * lg;
      float *c = (float *)g.c + rb0 * g.ldc + col;
      float x[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r = 8 * (e / 4) + e % 4;
        x[e] = EPI == EPI_GATE_RES && rb0 + r < g.m ? c[r * g.ldc] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r = 8 * (e / 4) + e % 4;
        if (rb0 + r < g.m) c[r * g.ldc] = finish<EPI>(tot[i][j][e], bv, gv, x[e]);
      }
    }
  }
}

template <int T, int EPI>
__global__ __launch_bounds__(256) void k_gemm_f32_small(GemmArgs g0) {
  constexpr int NP = T == 32 ? 2 : 1;                   // 16-byte load pairs of a unit (64 / T lane groups of 4)
  constexpr int U = 4 / NP;                             // units in flight per iteration
  constexpr int NE = T * T / 64;                        // accumulator entries per lane
  const GemmArgs g = batch_entry(g0);
  __shared__ float red[4][T * T];
  const int lane = threadIdx.x & 63, wu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane % T, lg = lane / T;
  const int n_tiles = (int)((g.n + T - 1) / T);
  const int64_t m0 = (int64_t)(blockIdx.x / n_tiles) * T, n0 = (int64_t)(blockIdx.x % n_tiles) * T;
  // rows past the end read the last row (their outputs are not stored)
  const float *pa = (const float *)g.a + min(m0 + lr, g.m - 1) * g.lda + 4 * lg;
  const float *pw = (const float *)g.w + min(n0 + lr, g.n - 1) * g.k + 4 * lg;
  const int units = (int)(g.k / KU), u0 = part_begin(units, wu), u1 = part_begin(units, wu + 1);

  typedef __attribute__((ext_vector_type(NE))) float accv;
  accv acc;
#pragma unroll
  for (int e = 0; e < NE; ++e) acc[e] = 0.f;
  auto load = [&](f32x4 (&a)[NP], f32x4 (&b)[NP], int u) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      a[p] = *(const f32x4 *)(pa + (int64_t)u * KU + 8 * p);
      b[p] = *(const f32x4 *)(pw + (int64_t)u * KU + 8 * p);
    }
  };
  auto step = [&](const f32x4 (&a)[NP], const f32x4 (&b)[NP]) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        if constexpr (T == 32) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[p][q], b[p][q], acc, 0, 0, 0);
        else acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[p][q], b[p][q], acc, 0, 0, 0);
      }
  };
  // the next U units are requested before the current U are used
  f32x4 fa[U][NP], fb[U][NP];
  int u = u0;
  if (u + U <= u1) {
#pragma unroll
    for (int i = 0; i < U; ++i) load(fa[i], fb[i], u + i);
    for (; u + 2 * U <= u1; u += U) {
      f32x4 na[U][NP], nb[U][NP];
#pragma unroll
      for (int i = 0; i < U; ++i) load(na[i], nb[i], u + U + i);
#pragma unroll
      for (int i = 0; i < U; ++i) step(fa[i], fb[i]);
#pragma unroll
      for (int i = 0; i < U; ++i)
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          fa[i][p] = na[i][p];
          fb[i][p] = nb[i][p];
        }
    }
#pragma unroll
    for (int i = 0; i < U; ++i) step(fa[i], fb[i]);
    u += U;
  }
  for (; u < u1; ++u) {
    load(fa[0], fb[0], u);
    step(fa[0], fb[0]);
  }

  // accumulator entry e: 32 x 32: row 8 (e / 4) + 4 lg + e % 4; 16 x 16: row 4 lg + e; column lr
#pragma unroll
  for (int e = 0; e < NE; ++e) red[wu][(T == 32 ? 8 * (e / 4) + 4 * lg + e % 4 : 4 * lg + e) * T + lr] = acc[e];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < T * T / 256; ++i) {
    const int t = threadIdx.x + 256 * i;
    const int64_t row = m0 + t / T, col = n0 + t % T;
    if (row >= g.m || col >= g.n) continue;
    const float s = (((0.f + red[0][t]) + red[1][t]) + red[2][t]) + red[3][t];   // 0 +: as in the tiles
    float *c = (float *)g.c + row * g.ldc + col;
    *c = finish<EPI>(s, g.bias ? ((const float *)g.bias)[col] : 0.f, EPI == EPI_GATE_RES ? g.gate[col] : 0.f,
                     EPI == EPI_GATE_RES ? *c : 0.f);
  }
}

int64_t tiles(const GemmArgs &g, int bm, int bn) {
  return (g.m + bm - 1) / bm * ((g.n + bn - 1) / bn) * (g.batch > 1 ? g.batch : 1);
}

template <int BM, int BN>
hipError_t launch_tile(const GemmArgs &g, hipStream_t s) {
  constexpr int LDS = NBUF * (BM + BN) * 128;
  const void *k[3] = {(const void *)k_gemm_f32_tile<BM, BN, EPI_STORE>, (const void *)k_gemm_f32_tile<BM, BN, EPI_GELU>,
                      (const void *)k_gemm_f32_tile<BM, BN, EPI_GATE_RES>};
  static DeviceOnce once;
  const hipError_t lim = once_on_device(once, [&] {
    for (const void *f : k) {
      const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  });
  if (lim != hipSuccess) return lim;
  const dim3 grid((unsigned)((g.m + BM - 1) / BM * ((g.n + BN - 1) / BN)), 1, g.batch > 1 ? g.batch : 1), block(256);
  if (g.epi == EPI_GELU) hipLaunchKernelGGL((k_gemm_f32_tile<BM, BN, EPI_GELU>), grid, block, LDS, s, g);
  else if (g.epi == EPI_GATE_RES) hipLaunchKernelGGL((k_gemm_f32_tile<BM, BN, EPI_GATE_RES>), grid, block, LDS, s, g);
  else hipLaunchKernelGGL((k_gemm_f32_tile<BM, BN, EPI_STORE>), grid, block, LDS, s, g);
  return hipGetLastError();
}

template <int T>
hipError_t launch_small(const GemmArgs &g, hipStream_t s) {
  const dim3 grid((unsigned)((g.m + T - 1) / T * ((g.n + T - 1) / T)), 1, g.batch > 1 ? g.batch : 1), block(256);
  if (g.epi == EPI_GELU) hipLaunchKernelGGL((k_gemm_f32_small<T, EPI_GELU>), grid, block, 0, s, g);
  else if (g.epi == EPI_GATE_RES) hipLaunchKernelGGL((k_gemm_f32_small<T, EPI_GATE_RES>), grid, block, 0, s, g);
  else hipLaunchKernelGGL((k_gemm_f32_small<T, EPI_STORE>), grid, block, 0, s, g);
  return hipGetLastError();
}

}  // namespace

bool gemm_f32_mfma(const GemmArgs &g) {
  return (uintptr_t)g.a % 16 == 0 && (uintptr_t)g.w % 16 == 0 && g.lda % 4 == 0 && g.k % BK == 0 &&
         (g.batch <= 1 || g.a_bs % 4 == 0) && g.lda <= (1 << 21) && g.k <= (1 << 21) &&
         (g.epi == EPI_STORE || g.epi == EPI_STORE_F32 || g.epi == EPI_GELU || g.epi == EPI_GATE_RES);
}

hipError_t launch_gemm_f32(const GemmArgs &g, hipStream_t s) {
  const int64_t cus = device_cus() > 0 ? device_cus() : 256;
  // Fewer 64 x 64 tiles than two thirds of the compute units: the K-split small
  // tiles (a 64 x 64 tile takes 23 us at K = 1,024 however few there are; 32 x 32
  // ones 33 us for a device full of 64 x 64 tiles, 16 us for half of it), 32 x 32
  // while those still cover the device (256 x 1,024, K = 256: 4.9 us against 5.8),
  // else 16 x 16 (256 x 256, K = 1,024: 5.9 us against 9.9).
  if (3 * tiles(g, 64, 64) < 2 * cus) return tiles(g, 32, 32) >= cus ? launch_small<32>(g, s) : launch_small<16>(g, s);
  // Else the fewer dispatch rounds x tile area; 128 x 64 tiles run 4% faster than
  // 64 x 64 ones at equal rounds (2,688 x 3,072, K = 1,024: 153 against 159 us;
  // 8,192 x 4,096, K = 4,096: 1.95 against 2.04 ms, 141 TFLOP/s), 64 x 64 win where
  // the last round would be thin (2,688 x 1,024, K = 4,096: 195 against 254 us).
  // 128 x 128 tiles, one block per CU, were slower than 128 x 64 everywhere (2.13 ms
  // on the large product): two blocks per CU run each other's epilogues and barriers over.
  auto cost = [&](int bm, int bn) { return (double)((tiles(g, bm, bn) + cus - 1) / cus) * bm * bn; };
  if (cost(128, 64) <= 1.04 * cost(64, 64)) return launch_tile<128, 64>(g, s);
  return launch_tile<64, 64>(g, s);
}

}  // namespace wdc

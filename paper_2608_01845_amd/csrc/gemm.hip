// GEMMs of the denoiser: c[m, n] = sum_k a[m, k] * w[n, k] + bias[n] with a
// fused epilogue (store, GELU-tanh, gated residual into the float32 stream,
// float32 store). Both operands are K-contiguous ("NT"), which is the layout
// the MFMA operand registers want: every lane loads 8 consecutive bf16.
//
// bf16 path: v_mfma_f32_16x16x32_bf16 tiles, BMxBN block tile (256 x 256 in 8
// waves of 128 x 64 for the large products), BK = 64, double-buffered LDS with
// an XOR swizzle of the 16-byte chunks of each 128-byte row (conflict-free
// fragment reads). K stages go straight from HBM into LDS (buffer loads with the
// LDS flag) two stages ahead; each wave reads its fragments one k-step ahead,
// one read at a time between its MFMAs, and the stage barrier sits one fragment
// row into a stage's last k-step so the matrix cores never drain at it. Large
// single products take an XCD-aware block order, and products whose last dispatch
// round would be thin run their last rows as a second launch of smaller tiles
// (launch_tail); products too small to fill one dispatch round of 256 x 256 tiles
// run on smaller ones throughout, with three or four LDS buffers where one block
// per compute unit has to hide its own loads, and loading waves of their own
// where that block is 64 x 64 (launch_small).
// float32 products run on the matrix cores too (gemm_f32.hip). Shapes that
// neither covers (K not a multiple of 32 or 64, unaligned operands): a plain
// LDS-tiled FMA kernel.
#include "common.h"

#include <algorithm>

namespace wdc {

// compute units of the current device (the rectangle order needs exactly 256)
int device_cus() {
  static std::atomic<int> cus[64] = {};   // 0: not yet known
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int n = cus[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    cus[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

namespace {

template <typename T>
__device__ __forceinline__ void epilogue(const GemmArgs &g, int epi, int64_t row, int64_t col, float acc) {
  float v = acc + (g.bias ? ld<T>((const T *)g.bias + col) : 0.f);
  int64_t o = row * g.ldc + col;
  switch (epi) {
    case EPI_STORE: st<T>((T *)g.c + o, v); break;
    case EPI_GELU: st<T>((T *)g.c + o, gelu_tanh(v)); break;
    case EPI_GATE_RES:
    case EPI_GATE_RES_NT: ((float *)g.c)[o] += g.gate[col] * v; break;
    default: ((float *)g.c)[o] = v; break;
  }
}

// ---------------------------------------------------------------- generic tiled kernel
// Batch entry blockIdx.z of a batched product: shifted operand and output pointers.
template <typename T>
__device__ __forceinline__ GemmArgs batch_entry(const GemmArgs &g0) {
  GemmArgs g = g0;
  const int64_t z = blockIdx.z;
  if (z) {
    const bool c16 = (g0.epi == EPI_STORE || g0.epi == EPI_GELU) && sizeof(T) == 2;
    g.a = (const T *)g0.a + z * g0.a_bs;
    g.c = c16 ? (void *)((T *)g0.c + z * g0.c_bs) : (void *)((float *)g0.c + z * g0.c_bs);
    if (g0.gate) g.gate = g0.gate + z * g0.gate_bs;
  }
  return g;
}

template <typename T>
__global__ __launch_bounds__(256) void k_gemm_simple(GemmArgs g0) {
  const GemmArgs g = batch_entry<T>(g0);
  __shared__ float As[16][64 + 4];
  __shared__ float Bs[16][64 + 4];
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  const int64_t m0 = (int64_t)blockIdx.y * 64, n0 = (int64_t)blockIdx.x * 64;
  const T *A = (const T *)g.a, *W = (const T *)g.w;
  float acc[4][4] = {};
  for (int64_t k0 = 0; k0 < g.k; k0 += 16) {
    for (int i = threadIdx.x; i < 64 * 16; i += 256) {
      int r = i / 16, kk = i % 16;
      int64_t gr = m0 + r, gk = k0 + kk;
      As[kk][r] = (gr < g.m && gk < g.k) ? ld<T>(A + gr * g.lda + gk) : 0.f;
      int64_t gn = n0 + r;
      Bs[kk][r] = (gn < g.n && gk < g.k) ? ld<T>(W + gn * g.k + gk) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = As[kk][ty * 4 + i];
        b[i] = Bs[kk][tx * 4 + i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int64_t r = m0 + ty * 4 + i, c = n0 + tx * 4 + j;
      if (r < g.m && c < g.n) epilogue<T>(g, g.epi, r, c, acc[i][j]);
    }
}

// ---------------------------------------------------------------- bf16 MFMA kernel
constexpr int BK = 64;  // K per LDS stage: one 128-byte row of bf16 per tile row
constexpr int RSRC_WORD3 = 0x00020000;  // raw buffer: 32-bit data format, no swizzle
constexpr int WAIT_VM0 = 0x0F70;        // s_waitcnt vmcnt(0), other counters untouched
constexpr int WAIT_LGKM0 = 0xC07F;      // s_waitcnt lgkmcnt(0), other counters untouched
// s_waitcnt vmcnt(n) with the other counters untouched; n above the counter's
// 6-bit range is clamped (a wave never has more than 63 operations pending)
__host__ __device__ constexpr int vm_wait(int n) {
  return n > 63 ? vm_wait(63) : (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8);
}

typedef __attribute__((address_space(3))) void lds_void;
// 16 bytes per lane from a buffer straight into LDS (lane L at lds + 16 L); kept
// out of the kernel templates, where the builtin makes the host pass drop stubs
__device__ __forceinline__ void lds_load16(__amdgpu_buffer_rsrc_t r, char *lds, int voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void *)lds, 16, voff, soff, 0, 0);
}

template <int BM, int BN, int WM, int WN, int NB = 2>
struct Cfg {
  static constexpr int NT = 64 * WM * WN;       // threads
  static constexpr int TM = BM / WM / 16;       // 16x16 tiles per wave along M
  static constexpr int TN = BN / WN / 16;       // along N
  // the first LW waves (one per SIMD) issue the tile loads: with all 16 waves
  // loading, the 16-wave kernel was 2-5% slower on the 13B products
  static constexpr int LW = NT / 64 >= 4 ? 4 : NT / 64;
  static constexpr int A_CHUNKS = BM * 8 / (64 * LW);  // 1 KB stripes per loading wave per stage
  static constexpr int B_CHUNKS = BN * 8 / (64 * LW);
  static constexpr int LDS_BYTES = NB * (BM + BN) * BK * 2;
  static constexpr bool QKV = BN % 128 == 0 && BN / WN == 64;   // tiles that take EPI_QKV
};

// Each tile row is 8 chunks of 16 bytes (128 B, two rows per 256-byte span of
// the 64 LDS banks). Chunk c of row r lives at c ^ ((r >> 1) & 7), so the 16
// rows read by 16 consecutive lanes land on 16 distinct 16-byte bank groups.
__device__ __forceinline__ int swz(int row, int chunk) { return (row * 8 + (chunk ^ ((row >> 1) & 7))) * 16; }

template <int EPI>
__device__ __forceinline__ float epi_act(float v) {
  if (EPI == EPI_GELU) {
    // 0.5 v (1 + tanh(u)) = v * sigmoid(2u), u = sqrt(2/pi) (v + 0.044715 v^3);
    // the hardware exp2 and reciprocal (about 1 ulp each) replace exp and the
    // IEEE division: the result is rounded to bfloat16 (8 significant bits)
    // exp(-2u) = exp2(v (A + B v^2)), A = -2 sqrt(2/pi) log2(e), B = 0.044715 A
    constexpr float A = -2.f * 0.7978845608028654f * 1.4426950408889634f, B = 0.044715f * A;
    return v * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(v * fmaf(B, v * v, A)));
  }
  return v;
}

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
// two floats -> packed bfloat16 pair (one v_cvt_pk_bf16_f32: round to nearest
// even, NaN stays NaN), low half first
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  bf16x2_t p;
  p[0] = (__bf16)lo;
  p[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, p);
}

// ---------------------------------------------------------------- fused q/k/v epilogue (EPI_QKV)
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
// V^T position of token j (and token of position j): bits 2 and 3 swapped
__device__ __forceinline__ int64_t vt_swap(int64_t j) { return (j & ~(int64_t)12) | ((j & 4) << 1) | ((j & 8) >> 1); }

// The block's bf16 tile (bias added, rounded once) sits in LDS as the staged
// epilogue leaves it: wave (wm, wn) of WM x WN holds rows WR wm.., columns
// 64 wn.. as 128-byte rows, 16-byte chunk c of row r at c ^ (r & 7). The tile
// lies inside the q, k or v columns and holds whole heads (d is a multiple of
// 256, BN of 128).
template <int BM_, int BN_, int WM_, int WN_>
struct QkvTile {
  static constexpr int BM = BM_, BN = BN_, NT = 64 * WM_ * WN_, WR = BM_ / WM_;
  static_assert(BN_ / WN_ == 64, "128-byte slice rows");
  __device__ static __forceinline__ const char *chunk(const char *smem, int row, int cc) {
    const int slice = row / WR * WN_ + (cc >> 3), r = row % WR;
    return smem + slice * (WR * 128) + r * 128 + (((cc & 7) ^ (r & 7)) * 16);
  }
};

// q or k: per head row the RMSNorm (float32, eps 1e-6) and the rotation of the
// video tokens' pairs (2p, 2p + 1), one more bf16 rounding, 16-byte stores of
// whole head rows. HD / 8 consecutive lanes hold one head row. The arithmetic
// is that of the separate preparation kernel (k_qk_prep8), without fused
// multiply-adds in either, so both give the same bits.
template <class QT, int HD, bool ROPE>
__device__ __forceinline__ void qk_scatter(const GemmArgs &g, const char *smem, int64_t m0, int h0, bf16_t *dst) {
#pragma clang fp contract(off)
  const QkvOut &o = g.qkv;
  constexpr int TPH = HD / 8;
  // Iteration it handles tile row RPI it + threadIdx.x / CPR; the thread's chunk
  // of the row (threadIdx.x % CPR: head hh, eight columns from 8 c) is the same
  // in every iteration. The sample and token advance incrementally (no
  // division per row). With a rotation table (ROPE: a table and video rows)
  // its entries go out GS rows at a time, one group ahead, and
  // unconditionally (rows that take no rotation read table row 0), so the
  // stores of a group never stand between a table read and its use.
  constexpr int CPR = QT::BN / 8, RPI = QT::NT / CPR, GS = QT::BM / RPI % 4 == 0 ? 4 : 2, NG = QT::BM / RPI / GS;
  static_assert(NG * RPI * GS == QT::BM, "whole groups of rows");
  const int cc = threadIdx.x % CPR, hh = cc / TPH, c = cc % TPH, rt = threadIdx.x / CPR;
  const int64_t r_first = o.rbase + m0 + rt;
  int64_t b = (int64_t)blockIdx.z + r_first / o.rps, jr = r_first % o.rps;
  int64_t bsv[2][GS], jv[2][GS];   // group g4 in slot g4 & 1
  float4 cs4v[2][GS][2];
  auto rotates = [&](int it, int64_t jt) { return ROPE && jt < o.n_video && m0 + RPI * it + rt < g.m; };
  auto coords = [&](int64_t (&bs4)[GS], int64_t (&j4)[GS]) {
#pragma unroll
    for (int u = 0; u < GS; ++u) {
      bs4[u] = b;
      j4[u] = o.row0 + jr;
      jr += RPI;
      while (jr >= o.rps) {
        jr -= o.rps;
        ++b;
      }
    }
  };
  auto fetch = [&](int g4, const int64_t (&js)[GS], float4 (&dst4)[GS][2]) {
    if (!ROPE) return;
#pragma unroll
    for (int u = 0; u < GS; ++u) {
      const int64_t jt = rotates(GS * g4 + u, js[u]) ? js[u] : 0;
      const float4 *cs4 = (const float4 *)(o.rope + jt * (HD / 2) + 4 * c);
      dst4[u][0] = cs4[0];
      dst4[u][1] = cs4[1];
    }
  };
  coords(bsv[0], jv[0]);
  fetch(0, jv[0], cs4v[0]);
#pragma unroll
  for (int g4 = 0; g4 < NG; ++g4) {
    const int sl = g4 & 1;
    if (g4 + 1 < NG) {
      coords(bsv[sl ^ 1], jv[sl ^ 1]);
      fetch(g4 + 1, jv[sl ^ 1], cs4v[sl ^ 1]);
    }
#pragma unroll
    for (int u = 0; u < GS; ++u) {
      const int it = GS * g4 + u, row = RPI * it + rt;
      float x[8];
      unpack8(*(const uint4 *)QT::chunk(smem, row, cc), x);
      if (o.qk_norm) {
        float sq = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) sq += x[e] * x[e];
        sq = group_sum<TPH>(sq);
        const float rs = rsqrtf(sq / (float)HD + 1e-6f);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] *= rs;
      }
      if (m0 + row >= g.m) continue;
      if (rotates(it, jv[sl][u])) {
        const float4 c01 = cs4v[sl][u][0], c23 = cs4v[sl][u][1];
        const float cs[8] = {c01.x, c01.y, c01.z, c01.w, c23.x, c23.y, c23.z, c23.w};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const float co = cs[2 * p], si = cs[2 * p + 1];
          const float t0 = x[2 * p] * co - x[2 * p + 1] * si, t1 = x[2 * p] * si + x[2 * p + 1] * co;
          x[2 * p] = t0;
          x[2 * p + 1] = t1;
        }
      }
      *(uint4 *)(dst + ((bsv[sl][u] * o.heads + h0 + hh) * o.n_pad + jv[sl][u]) * HD + 8 * c) = pack8(x);
    }
  }
}

// v: transposed into [heads, hd, n_pad] in the V^T key order. A tile whose
// first token is 16-aligned and whose rows all belong to one sample writes 8
// consecutive positions (one 16-byte store) per lane for every group of 16
// tokens it holds whole; partial groups and other tiles go element by element
// (positions of missing tokens are padding, zeroed separately).
template <class QT, int HD>
__device__ __forceinline__ void v_scatter(const GemmArgs &g, const char *smem, int64_t m0, int h0) {
  const QkvOut &o = g.qkv;
  bf16_t *v = (bf16_t *)o.v;
  auto at = [&](int row, int col) -> uint32_t {
    return *(const bf16_t *)(QT::chunk(smem, row, col >> 3) + 2 * (col & 7));
  };
  const int64_t mr = (o.rbase + m0) % o.rps;
  const bool clean = (o.row0 + mr) % 16 == 0 && mr + QT::BM <= o.rps;
  static_assert(HD == 64 || HD == 128, "head size");
  constexpr int PPI = QT::NT / QT::BN;   // columns' threads: positions (or rows) per iteration
  if (clean) {
    // a wavefront's lanes take 64 consecutive columns at one chunk of 8
    // positions: every LDS read of the wave hits one 128-byte tile row segment
    // (columns of a fixed token are contiguous; tokens of a fixed column 16
    // apart would all fall on one bank)
    const int64_t b = (int64_t)blockIdx.z + (o.rbase + m0) / o.rps, j0 = o.row0 + mr;
#pragma unroll 2
    for (int it = 0; it < QT::BM / 8 / PPI; ++it) {
      const int col = threadIdx.x % QT::BN, p8 = PPI * it + threadIdx.x / QT::BN;
      const int hh = col / HD, e = col % HD, grp = 16 * (p8 >> 1), half = p8 & 1;
      bf16_t *dst = v + ((b * o.heads + h0 + hh) * HD + e) * o.n_pad + j0;
      if (m0 + grp + 16 <= g.m) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int t0 = grp + (int)vt_swap(8 * half + 2 * i), t1 = grp + (int)vt_swap(8 * half + 2 * i + 1);
          w[i] = at(t0, col) | (at(t1, col) << 16);
        }
        *(uint4 *)(dst + 8 * p8) = make_uint4(w[0], w[1], w[2], w[3]);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int t = grp + (int)vt_swap(8 * half + i);
          if (m0 + t < g.m) dst[8 * p8 + i] = (bf16_t)at(t, col);
        }
      }
    }
  } else {
    // element by element: the thread's column is fixed, its row steps by PPI
    const int col = threadIdx.x % QT::BN, hh = col / HD, e = col % HD;
    const int64_t r_first = o.rbase + m0 + threadIdx.x / QT::BN;
    int64_t b = (int64_t)blockIdx.z + r_first / o.rps, jr = r_first % o.rps;
    for (int it = 0; it < QT::BM / PPI; ++it) {
      const int row = PPI * it + threadIdx.x / QT::BN;
      const int64_t bs = b, j = o.row0 + jr;
      jr += PPI;
      while (jr >= o.rps) {
        jr -= o.rps;
        ++b;
      }
      if (m0 + row >= g.m) break;
      v[((bs * o.heads + h0 + hh) * HD + e) * o.n_pad + vt_swap(j)] = (bf16_t)at(row, col);
    }
  }
}

// S > 0: the form for lone blocks, with as many loading waves again and S stages
// per barrier (see below).
template <int BM, int BN, int WM, int WN, int EPI, int NB = 2, int S = 0>
__global__ __launch_bounds__(64 * WM * WN * (S > 0 ? 2 : 1)) void k_gemm_mfma(GemmArgs g0) {
  using C = Cfg<BM, BN, WM, WN, NB>;
  // C^T tiles (weight fragment as the MFMA A operand): a lane holds 4 consecutive
  // columns of one row, 8 bytes of a bf16 output, 16 of a float32 one
  constexpr bool OUT16 = EPI == EPI_STORE || EPI == EPI_GELU || EPI == EPI_QKV;
  constexpr bool RES = EPI == EPI_GATE_RES || EPI == EPI_GATE_RES_NT;   // gated residual into the float32 stream
  // bf16 output through LDS: whole-line non-temporal stores, or the q/k/v layouts
  constexpr bool STAGE_OUT = BM >= 192 || EPI == EPI_QKV;
  const GemmArgs g = batch_entry<bf16_t>(g0);
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char *sA = smem;                    // [NB][BM][128 B]
  char *sB = smem + NB * BM * BK * 2; // [NB][BN][128 B]

  // Tile order: a group of 8 consecutive M tiles walks all N tiles, so blocks
  // running at once share A rows and the weight panel in L2.
  const int n_tiles = (int)(g.n / BN);
  const int m_tiles = (int)((g.m + BM - 1) / BM);
  const int bid = blockIdx.x;
  const int group = 8;
  const int per_group = group * n_tiles;
  const int gidx = bid / per_group;
  const int first_m = gidx * group;
  const int gsize = min(m_tiles - first_m, group);
  int mt, nt;
  if (g.order == 1) {
    // Dispatch rounds of 256 blocks, one per CU; block id % 8 is its XCD. Round
    // r gives XCD x chunk 8r + x: a (32 / rect_n) (M) x rect_n (N) rectangle of
    // tiles (8 x 4 or 2 x 16), one per block, so the 32 blocks an XCD runs
    // together start together and share their A and weight slices in its L2.
    // Blocks past the last tile exit.
    const int r = bid / 256, x = bid % 8, l = (bid / 8) % 32;
    const int rn = g.rect_n, rm = 32 / rn;
    const int chunk = 8 * r + x, cpb = n_tiles / rn;
    mt = rm * (chunk / cpb) + l % rm;
    nt = rn * (chunk % cpb) + l / rm;
    if (mt >= m_tiles) return;
  } else if (BM == 64 && g.order == 2) {
    // few M tiles: those of one weight panel on one XCD (block id % 8), which
    // then fetches the panel once into its L2 (226 x 3,072, K = 4,096: 17.9 us
    // without, 14.2 with; 256 x 3,072, K = 12,288: 47.0 and 38.1; none slower; weights
    // in the last-level cache).
    // On 64-row tiles only: the branch alone cost the 96-row ones 4 to 8% and the
    // blocks of the large models 0.4%.
    const int l = bid / 8;
    nt = bid % 8 + 8 * (l / m_tiles);
    mt = l % m_tiles;
  } else if (gsize == group && n_tiles >= 24) {
    // Workgroups go to the 8 XCDs round robin (id % 8). Give each XCD a
    // contiguous run of n_tiles tiles of the group in (nt, mt) order: an
    // 8-row by n_tiles/8-column rectangle, so the ~32 blocks one XCD runs at
    // once share 8 A slices and a few B slices in its L2 (+5.6% at N = 12,288,
    // K = 3,072). Narrow products (N = 3,072, long K) keep one row tile per XCD
    // against every column tile, which measured 3% faster for them.
    const int b = bid % per_group;
    const int idx = (b % 8) * n_tiles + b / 8;
    mt = first_m + idx % group;
    nt = idx / group;
  } else {
    mt = first_m + (bid % per_group) % gsize;
    nt = (bid % per_group) / gsize;
  }
  const int64_t m0 = (int64_t)mt * BM, n0 = (int64_t)nt * BN;

  const bool loader = S == 0 || threadIdx.x >= C::NT;   // S == 0: the first NW waves load
  const int tid = S > 0 ? threadIdx.x % C::NT : threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int wm = wid / WN, wn = wid % WN;
  const int lr = lane & 15, lg = lane >> 4;

  // Tiles go straight from HBM to LDS (buffer_load_dwordx4 ... lds: lane L of a
  // wavefront's load writes 16 bytes at LDS base + 16 L). Stripe s = 1 KB = 8
  // tile rows; loading wave w (of NW) loads stripes w, w + NW, w + 2 NW, ... so each lane fetches
  // row 8s + lane/8 and the logical chunk that the swizzle puts at physical
  // chunk lane%8 (the swizzle key (row >> 1) & 7 is the same for every stripe
  // of a wave since NW is even).
  // The A descriptor spans only this block's valid rows and every stripe's row
  // is in the VGPR offset, which the buffer range check covers: rows past m are
  // read as zero (the K offset rides in the SGPR offset and is always in range).
  constexpr int NW = C::LW;
  static_assert(NW % 2 == 0, "stripe swizzle assumes an even wave count");
  const int64_t rows_a = min((int64_t)BM, g.m - m0);
  const __amdgpu_buffer_rsrc_t a_desc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)((const bf16_t *)g.a + m0 * g.lda), (short)0, (int)(rows_a * g.lda * 2), RSRC_WORD3);
  const __amdgpu_buffer_rsrc_t b_desc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)((const bf16_t *)g.w + n0 * g.k), (short)0, (int)(BN * g.k * 2), RSRC_WORD3);
  const int wu = __builtin_amdgcn_readfirstlane(wid);
  const int lch = (lane & 7) ^ ((4 * (wu & 1) + (lane >> 4)) & 7);
  const int row0 = 8 * wu + (lane >> 3);
  // A stripe i is row0 + 8 NW i: its offset steps by a_step from stripe to
  // stripe, added in the load sequence itself (an asm add the compiler cannot
  // hoist) so the loop does not keep A_CHUNKS offsets live in VGPRs
  const int va0 = row0 * (int)g.lda * 2 + lch * 16;
  const int a_step = 8 * NW * (int)g.lda * 2;
  const int vb = row0 * (int)g.k * 2 + lch * 16;

  // fragment read offsets: row wm*(BM/WM) + 16i + lr, chunk 4s + lg; the
  // swizzle key depends on the row only, so k-step s reads at offset(0) ^ 64 s
  const int ra0 = swz(wm * (BM / WM) + lr, lg), rb0 = swz(wn * (BN / WN) + lr, lg);

#define WDC_GEMM_LOAD(buf, kt)                                                                     \
  {                                                                                                \
    const int kb_ = (kt) * BK * 2;                                                                 \
    if (wu < NW && loader) {                                                                       \
      int v_ = va0;                                                                                \
      _Pragma("unroll") for (int i = 0; i < C::A_CHUNKS; ++i) {                                     \
        lds_load16(a_desc, sA + (buf) * BM * 128 + (i * NW + wu) * 1024, v_, kb_);                  \
        if (i + 1 < C::A_CHUNKS) asm volatile("v_add_u32 %0, %0, %1" : "+v"(v_) : "s"(a_step));     \
      }                                                                                            \
      _Pragma("unroll") for (int i = 0; i < C::B_CHUNKS; ++i)                                       \
          lds_load16(b_desc, sB + (buf) * BN * 128 + (i * NW + wu) * 1024, vb, i * 8 * NW * (int)g.k * 2 + kb_); \
    }                                                                                              \
  }

  // fragments of k-step s of the stage in buffer buf
#define WDC_GEMM_READA(buf, s, i) fa[i] = *(const bf16x8 *)(sA + (buf) * BM * 128 + (ra0 ^ (64 * (s))) + (i) * 16 * 128)
#define WDC_GEMM_READB(buf, s, j) fb[s][j] = *(const bf16x8 *)(sB + (buf) * BN * 128 + (rb0 ^ (64 * (s))) + (j) * 16 * 128)
  // Workgroup barrier after this wave's LDS reads complete, without the memory
  // fence of __syncthreads (whose vmcnt(0) would also wait for a stage still
  // in flight). The wait is the builtin rather than asm so that the compiler's
  // own wait tracking sees the fragment reads as complete.
#define WDC_GEMM_BARRIER()                                                                         \
  {                                                                                                \
    __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);                                                        \
    __builtin_amdgcn_s_barrier();                                                                  \
  }

  constexpr int SL = C::A_CHUNKS + C::B_CHUNKS;           // load instructions per loading wave per stage
  const int nk = (int)(g.k / BK);
  // Stages 0 and 1 fill both buffers; stage 0 is complete once no more than
  // stage 1's loads are pending (a wave's memory operations complete in issue
  // order).
#pragma unroll
  for (int st = 0; st < NB; ++st)
    if (st < nk) WDC_GEMM_LOAD(st, st);
  if (wu < NW && loader) {
    if (nk >= NB) __builtin_amdgcn_s_waitcnt(vm_wait((NB - (S > 0 ? S : 1)) * SL));
    else __builtin_amdgcn_s_waitcnt(WAIT_VM0);
  }
  WDC_GEMM_BARRIER();

  constexpr int TM = C::TM, TN = C::TN;
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  if constexpr (S > 0) {
    // One wave per SIMD and four MFMAs per k-step: a wave that also loads issues
    // its loads, fragment reads and MFMAs one after the other, and nothing runs
    // under their latencies. Here waves 4 to 7 issue the loads, and waves 0 to 3
    // read all fragments of the next S stages at once, then run the MFMAs of the
    // S they hold. After the barrier the step read last is in registers, so its
    // buffers take the loads of the step NS ahead, and the next step has landed.
    // 226 x 3,072, K = 4,096, six buffers: 18.4 us with the loop below (three to
    // eight buffers), 17.9 with S = 2 and the computing waves loading, 14.5 so
    // (15.5 with S = 1). The sums are those of the loop below, term by term.
    static_assert(NB % S == 0 && NB / S >= 2 && NW * 64 == C::NT, "whole steps, as many loading waves as computing ones");
    constexpr int NS = NB / S;
    int buf = 0;                                          // first buffer of step kt
    if (loader) {
      for (int kt = 0; kt * S < nk; ++kt) {
        if ((kt + NS) * S <= nk) __builtin_amdgcn_s_waitcnt(vm_wait((NS - 2) * S * SL));
        else __builtin_amdgcn_s_waitcnt(WAIT_VM0);
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int st = 0; st < S; ++st)
          if ((kt + NS) * S + st < nk) WDC_GEMM_LOAD(buf + st, (kt + NS) * S + st);
        buf = buf + S == NB ? 0 : buf + S;
      }
      return;
    }
    bf16x8 fa[2][S][2][TM], fb[2][S][2][TN];
    auto read = [&](bf16x8 (&a)[S][2][TM], bf16x8 (&b)[S][2][TN], int buf) {
#pragma unroll
      for (int st = 0; st < S; ++st)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
          for (int i = 0; i < TM; ++i) a[st][s][i] = *(const bf16x8 *)(sA + (buf + st) * BM * 128 + (ra0 ^ (64 * s)) + i * 16 * 128);
#pragma unroll
          for (int j = 0; j < TN; ++j) b[st][s][j] = *(const bf16x8 *)(sB + (buf + st) * BN * 128 + (rb0 ^ (64 * s)) + j * 16 * 128);
        }
    };
    read(fa[0], fb[0], 0);
    auto step = [&](int kt, bf16x8 (&a)[S][2][TM], bf16x8 (&b)[S][2][TN], bf16x8 (&an)[S][2][TM], bf16x8 (&bn)[S][2][TN]) {
      buf = buf + S == NB ? 0 : buf + S;
      WDC_GEMM_BARRIER();
      if ((kt + 1) * S < nk) read(an, bn, buf);           // stages past the last: stale, not used
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int st = 0; st < S; ++st)
        if (st == 0 || kt * S + st < nk)
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[st][s][j], a[st][s][i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    for (int kt = 0; kt * S < nk; kt += 2) {
      step(kt, fa[0], fb[0], fa[1], fb[1]);
      if ((kt + 1) * S >= nk) break;
      step(kt + 1, fa[1], fb[1], fa[0], fb[0]);
    }
  } else {
  // Two k-steps of 32 per stage, each TM rows of TN MFMAs (v_mfma_16x16x32: at
  // the power limit a loop of them sustains 2,065 TFLOP/s on random operands
  // with two waves per SIMD where 32x32x16 sustains 1,500, and at 64 x 64 to 128
  // x 64 wave tiles both read the same fragments per FLOP). An A fragment is
  // replaced by the next k-step's as soon as its row of MFMAs is issued, the B
  // fragments are double-buffered: every read has about one k-step of MFMAs to
  // arrive. The stage barrier sits D rows into the second k-step, whose
  // fragments are in registers by then: after it the stage NB ahead goes into
  // the buffer just consumed and the next stage's first fragments are read. A
  // scheduling barrier after each MFMA, read and load keeps that order.
  constexpr int D = 1;   // 2, 3 and 4 were 0.5 to 2% slower on the large products
  static_assert(BK == 64 && D < TM, "two k-steps per stage");
  // Loads of a stage go one by one between MFMAs: within the rest of the second
  // k-step with two buffers (they have the next stage to arrive in), spread on
  // to the next barrier with more buffers and 64 x 64 wave tiles (a burst stalls
  // the wave that issues it).
  constexpr int LQ0 = (TM - D) * TN;                      // MFMAs from the barrier to the end of the stage
  constexpr int LQ = NB > 2 && TM >= 3 && TN == 4 ? LQ0 + TM * TN : LQ0;
  bf16x8 fa[TM], fb[2][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) WDC_GEMM_READA(0, 0, i);
#pragma unroll
  for (int j = 0; j < TN; ++j) WDC_GEMM_READB(0, 0, j);
  int va = va0;                                           // steps through the A stripes of the stage being loaded
  // load number l of stage lkt (A stripes first, then B) into buffer lbuf
#define WDC_GEMM_LOAD1(lbuf, lkt, l)                                                               \
  {                                                                                                \
    if ((l) < C::A_CHUNKS) {                                                                       \
      lds_load16(a_desc, sA + (lbuf) * BM * 128 + ((l) * NW + wu) * 1024, va, (lkt) * BK * 2);             \
      if ((l) + 1 < C::A_CHUNKS) asm volatile("v_add_u32 %0, %0, %1" : "+v"(va) : "s"(a_step));     \
    } else {                                                                                       \
      const int lb_ = (l) - C::A_CHUNKS;                                                           \
      lds_load16(b_desc, sB + (lbuf) * BN * 128 + (lb_ * NW + wu) * 1024, vb,                      \
                 lb_ * 8 * NW * (int)g.k * 2 + (lkt) * BK * 2);                                    \
    }                                                                                              \
  }
  // the loads that belong after MFMA q of LQ since the barrier (the branch holds
  // loads only, so the accumulators never meet at a join)
#define WDC_GEMM_LOADS(cond, lbuf, lkt, q)                                                         \
  if (cond) {                                                                                      \
    _Pragma("unroll") for (int l = 0; l < SL; ++l)                                                 \
      if (l * LQ / SL == (q)) WDC_GEMM_LOAD1(lbuf, lkt, l)                                         \
  }
  int buf = 0, prv = NB - 1;
  for (int kt = 0; kt < nk; ++kt) {
    const int nxt = NB == 2 ? buf ^ 1 : buf + 1 == NB ? 0 : buf + 1;
    constexpr int BPR0 = (TN + TM - 1) / TM;              // B fragments read per row of MFMAs
    const bool ld0 = LQ > LQ0 && kt > 0 && kt + NB - 1 < nk && wu < NW;   // rest of the previous barrier's loads
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[0][j], fa[i], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < BPR0; ++b)
          if (j == b * TN / BPR0 && i * BPR0 + b < TN) WDC_GEMM_READB(buf, 1, i * BPR0 + b);
        if (j == TN - 1) WDC_GEMM_READA(buf, 1, i);
        __builtin_amdgcn_sched_barrier(0);
        WDC_GEMM_LOADS(ld0, prv, kt + NB - 1, LQ0 + i * TN + j)
        __builtin_amdgcn_sched_barrier(0);
      }
    const bool ld1 = kt + NB < nk && wu < NW;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (i == D && j == 0) {
          // stage kt + 1 has landed once only the loads of later stages are
          // pending; after the barrier every wave is done with buffer buf. Past
          // the last stage the reads fetch stale data, never used.
          if (wu < NW) {
            if (NB > 2 && kt + NB <= nk) __builtin_amdgcn_s_waitcnt(vm_wait((NB - 2) * SL));
            else __builtin_amdgcn_s_waitcnt(WAIT_VM0);
          }
          WDC_GEMM_BARRIER();
          va = va0;
        }
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[1][j], fa[i], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (i >= D) {
          // the next stage's A0 and B0.. first, spread over the rows that are left
          constexpr int BPR = (TN + TM - D - 1) / (TM - D);
#pragma unroll
          for (int b = 0; b < BPR; ++b)
            if (j == b * TN / BPR && (i - D) * BPR + b < TN) WDC_GEMM_READB(nxt, 0, (i - D) * BPR + b);
          if (j == TN - 1) {
            WDC_GEMM_READA(nxt, 0, i - D);
            if (i == TM - 1)
#pragma unroll
              for (int x = TM - D; x < TM; ++x) WDC_GEMM_READA(nxt, 0, x);
          }
          __builtin_amdgcn_sched_barrier(0);
          WDC_GEMM_LOADS(ld1, buf, kt + NB, (i - D) * TN + j)
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    prv = buf;
    buf = nxt;
  }
  }
#undef WDC_GEMM_LOADS
#undef WDC_GEMM_LOAD1
#undef WDC_GEMM_READA
#undef WDC_GEMM_READB

  const bf16_t *bias = (const bf16_t *)g.bias;
  const int cb = wn * (BN / WN) + 4 * lg;                 // the lane's columns in the block: cb + 16 j + 0..3
  if constexpr (OUT16 && STAGE_OUT) {
    // bf16 output staged through LDS (free once the last K stage is consumed:
    // every read that matters completed before the last stage barrier): each
    // wave writes its BM/WM x BN/WN tile into its own slice, row-major with the
    // 16-byte chunk index XOR (row & 7), then reads it back so that every store
    // instruction writes whole 128-byte row segments, marked non-temporal.
    constexpr int RB = BN / WN * 2, CPR = RB / 16, RPI = 1024 / RB, WR = BM / WM;
    static_assert(WR * RB * C::NT / 64 <= C::LDS_BYTES, "staging slices exceed LDS");
    char *wl = smem + wid * (WR * RB);
    uint2 bw[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bw[j] = bias ? *(const uint2 *)(bias + n0 + cb + 16 * j) : make_uint2(0, 0);
    // the last stage's stale fragment reads may still be in flight; nothing
    // else touches LDS
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const float b0 = bf2f((bf16_t)(bw[j].x & 0xffff)), b1 = bf2f((bf16_t)(bw[j].x >> 16));
      const float b2 = bf2f((bf16_t)(bw[j].y & 0xffff)), b3 = bf2f((bf16_t)(bw[j].y >> 16));
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int r = i * 16 + lr;
        const uint32_t w0 = pack_bf16(epi_act<EPI>(acc[i][j][0] + b0), epi_act<EPI>(acc[i][j][1] + b1));
        const uint32_t w1 = pack_bf16(epi_act<EPI>(acc[i][j][2] + b2), epi_act<EPI>(acc[i][j][3] + b3));
        *(uint2 *)(wl + r * RB + (((2 * j + (lg >> 1)) ^ (r & 7)) * 16) + 8 * (lg & 1)) = make_uint2(w0, w1);
      }
    }
    if constexpr (EPI == EPI_QKV) {
      using QT = QkvTile<BM, BN, WM, WN>;
      __syncthreads();                      // every wave's slice is written
      const int64_t nq = g.qkv.cbase + n0;
      const int region = (int)(nq / g.qkv.d), h0 = (int)((nq % g.qkv.d) / g.qkv.hd);
      if (region < 2) {
        bf16_t *dst = (bf16_t *)(region == 0 ? g.qkv.q : g.qkv.k);
        const bool rope = g.qkv.rope && g.qkv.n_video > 0;
        if (g.qkv.hd == 128) {
          if (rope) qk_scatter<QT, 128, true>(g, smem, m0, h0, dst);
          else qk_scatter<QT, 128, false>(g, smem, m0, h0, dst);
        } else {
          if (rope) qk_scatter<QT, 64, true>(g, smem, m0, h0, dst);
          else qk_scatter<QT, 64, false>(g, smem, m0, h0, dst);
        }
      } else if (g.qkv.hd == 128) {
        v_scatter<QT, 128>(g, smem, m0, h0);
      } else {
        v_scatter<QT, 64>(g, smem, m0, h0);
      }
      return;
    }
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;
#pragma unroll
    for (int s = 0; s < WR / RPI; ++s) {
      const int r = s * RPI + lane / CPR, ch = lane % CPR;
      const u32x4_t v = *(const u32x4_t *)(wl + r * RB + ((ch ^ (r & 7)) * 16));
      const int64_t row = m0 + wm * WR + r;
      if (row < g.m)
        __builtin_nontemporal_store(v, (u32x4_t *)((bf16_t *)g.c + row * g.ldc + n0 + wn * (BN / WN) + ch * 8));
    }
  } else if constexpr (OUT16) {
    // bf16 output in 8-byte groups of 4 columns. The bias of all the lane's
    // columns is read before the first store, so one wait covers every read.
    uint2 bw[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bw[j] = bias ? *(const uint2 *)(bias + n0 + cb + 16 * j) : make_uint2(0, 0);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int64_t row = m0 + wm * (BM / WM) + i * 16 + lr;
      if (row >= g.m) continue;
      bf16_t *out = (bf16_t *)g.c + row * g.ldc + n0 + cb;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const float b0 = bf2f((bf16_t)(bw[j].x & 0xffff)), b1 = bf2f((bf16_t)(bw[j].x >> 16));
        const float b2 = bf2f((bf16_t)(bw[j].y & 0xffff)), b3 = bf2f((bf16_t)(bw[j].y >> 16));
        const uint32_t w0 = pack_bf16(epi_act<EPI>(acc[i][j][0] + b0), epi_act<EPI>(acc[i][j][1] + b1));
        const uint32_t w1 = pack_bf16(epi_act<EPI>(acc[i][j][2] + b2), epi_act<EPI>(acc[i][j][3] + b3));
        *(uint2 *)(out + 16 * j) = make_uint2(w0, w1);
      }
    }
  } else {
    // float32 output, 16 bytes of a row per lane (64 of it per quad of lanes).
    // The residual reads of two tile rows go out together, before their stores:
    // vmcnt also counts stores, and a read behind each store would serialise
    // every read-modify-write.
    constexpr int RI = TM >= 2 ? 2 : 1;
    f32x4 bv[TN], gv[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const uint2 bw = bias ? *(const uint2 *)(bias + n0 + cb + 16 * j) : make_uint2(0, 0);
      bv[j] = f32x4{bf2f((bf16_t)(bw.x & 0xffff)), bf2f((bf16_t)(bw.x >> 16)), bf2f((bf16_t)(bw.y & 0xffff)),
                    bf2f((bf16_t)(bw.y >> 16))};
      if (RES) gv[j] = *(const f32x4 *)(g.gate + n0 + cb + 16 * j);
    }
#pragma unroll
    for (int i0 = 0; i0 < TM; i0 += RI) {
      f32x4 xr[RI][TN];
      f32x4 *xp[RI];
      bool in[RI];
#pragma unroll
      for (int u = 0; u < RI; ++u) {
        const int64_t row = m0 + wm * (BM / WM) + (i0 + u) * 16 + lr;
        in[u] = row < g.m;
        xp[u] = (f32x4 *)((float *)g.c + row * g.ldc + n0 + cb);
        if (RES && in[u])
#pragma unroll
          for (int j = 0; j < TN; ++j)
            xr[u][j] = EPI == EPI_GATE_RES_NT ? __builtin_nontemporal_load(xp[u] + 4 * j) : xp[u][4 * j];
      }
#pragma unroll
      for (int u = 0; u < RI; ++u) {
        if (!in[u]) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          f32x4 v = acc[i0 + u][j] + bv[j];
          if (RES) v = xr[u][j] + gv[j] * v;
          if (EPI == EPI_GATE_RES_NT) __builtin_nontemporal_store(v, xp[u] + 4 * j);
          else xp[u][4 * j] = v;
        }
      }
    }
  }
#undef WDC_GEMM_BARRIER
#undef WDC_GEMM_LOAD
}

// 8 x 4 rectangles of 256 x 256 tiles ("chunks", one per XCD and dispatch round)
// of a product that takes the rectangle order, 0 of one that does not. The order
// pays on large single products; a z-batch would put every slice's rectangles
// on the same XCDs, and with fewer than 8 dispatch rounds the partly filled last
// round costs more than the L2 reuse gains (a batched rollout of 8 mid-size
// samples ran 40% slower with it). 2 x 16 rectangles (A panels, larger than the
// last-level cache, re-read once per rectangle column; weight panels, which fit
// it, once per rectangle row) made the N = 12,288 product 2.5-3% faster alone
// but the whole 13B forward's GEMMs 1% slower (same-box A/B), so they are not
// used; nor 2 x 16 for that product alone (1.1% slower over the forward) or 16 x 2
// for the N = 3,072 ones (1.8% slower).
constexpr int RECT_M = 8, RECT_N = 4;
int rect_chunks(const GemmArgs &g) {
  const int m_tiles = (int)((g.m + 255) / 256), n_tiles = (int)(g.n / 256);
  if (n_tiles % RECT_N != 0 || g.batch > 1 || device_cus() != 256) return 0;
  const int chunks = (m_tiles + RECT_M - 1) / RECT_M * (n_tiles / RECT_N);
  return chunks >= 64 ? chunks : 0;
}

template <int BM, int BN, int WM, int WN, int NB = 2, int S = 0>
hipError_t launch_mfma(const GemmArgs &g0, hipStream_t s, int max_chunks = 0) {
  using C = Cfg<BM, BN, WM, WN, NB>;
  GemmArgs g = g0;
  const int m_tiles = (int)((g.m + BM - 1) / BM), n_tiles = (int)(g.n / BN);
  g.rect_n = RECT_N;
  const int chunks = BM == 256 && BN == 256 ? rect_chunks(g) : 0;
  g.order = chunks > 0 ? 1 : BM == 64 && m_tiles <= 8 && n_tiles % 8 == 0 && g.batch <= 1 ? 2 : 0;
  int blocks = m_tiles * n_tiles;
  if (g.order == 1) blocks = ((max_chunks > 0 ? max_chunks : chunks) + 7) / 8 * 256;
  dim3 grid(blocks, 1, g.batch > 1 ? g.batch : 1), block(C::NT * (S > 0 ? 2 : 1));
  switch (g.epi) {
    case EPI_STORE: hipLaunchKernelGGL((k_gemm_mfma<BM, BN, WM, WN, EPI_STORE, NB, S>), grid, block, C::LDS_BYTES, s, g); break;
    case EPI_GELU: hipLaunchKernelGGL((k_gemm_mfma<BM, BN, WM, WN, EPI_GELU, NB, S>), grid, block, C::LDS_BYTES, s, g); break;
    case EPI_GATE_RES: hipLaunchKernelGGL((k_gemm_mfma<BM, BN, WM, WN, EPI_GATE_RES, NB, S>), grid, block, C::LDS_BYTES, s, g); break;
    case EPI_GATE_RES_NT: hipLaunchKernelGGL((k_gemm_mfma<BM, BN, WM, WN, EPI_GATE_RES_NT, NB, S>), grid, block, C::LDS_BYTES, s, g); break;
    case EPI_QKV:
      if constexpr (C::QKV) {
        hipLaunchKernelGGL((k_gemm_mfma<BM, BN, WM, WN, EPI_QKV, NB, S>), grid, block, C::LDS_BYTES, s, g);
        break;
      } else {
        return hipErrorInvalidValue;
      }
    default: hipLaunchKernelGGL((k_gemm_mfma<BM, BN, WM, WN, EPI_STORE_F32, NB, S>), grid, block, C::LDS_BYTES, s, g); break;
  }
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int NB = 2, int S = 0>
hipError_t set_lds_limit() {
  using C = Cfg<BM, BN, WM, WN, NB>;
  const void *k[5] = {(const void *)k_gemm_mfma<BM, BN, WM, WN, EPI_STORE, NB, S>,
                      (const void *)k_gemm_mfma<BM, BN, WM, WN, EPI_GELU, NB, S>,
                      (const void *)k_gemm_mfma<BM, BN, WM, WN, EPI_GATE_RES, NB, S>,
                      (const void *)k_gemm_mfma<BM, BN, WM, WN, EPI_GATE_RES_NT, NB, S>,
                      (const void *)k_gemm_mfma<BM, BN, WM, WN, EPI_STORE_F32, NB, S>};
  for (const void *f : k) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
    if (e != hipSuccess) return e;
  }
  if constexpr (C::QKV)
    return hipFuncSetAttribute((const void *)k_gemm_mfma<BM, BN, WM, WN, EPI_QKV, NB, S>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
  return hipSuccess;
}

bool operands_aligned(const GemmArgs &g) {
  return ((uintptr_t)g.a % 16 == 0) && ((uintptr_t)g.w % 16 == 0) && g.lda % 8 == 0 && g.k % BK == 0 &&
         (uintptr_t)g.c % 16 == 0 && g.ldc % 4 == 0 && (uintptr_t)g.bias % 8 == 0 && (uintptr_t)g.gate % 16 == 0 &&
         (g.batch <= 1 || (g.a_bs % 8 == 0 && g.c_bs % 4 == 0 && g.gate_bs % 4 == 0));
}

int64_t tile_count(const GemmArgs &g, int bm, int bn) {
  return (g.m + bm - 1) / bm * (g.n / bn) * (g.batch > 1 ? g.batch : 1);
}

// Tile shape of a product too small for the 256 x 256 tiles (n % 64 == 0).
// Measured per 64-deep K stage (microseconds a compute unit takes for the
// blocks it holds), the products alone on the device:
//   64 x 64, lone (6 buffers, loading waves): 0.19; 3 buffers: 0.64 for three blocks
//   96 x 128, 4 buffers, one block: 0.43; 128 x 128, one block: 0.53
//   128 x 128, 2 buffers, two blocks: 0.95
//   192 x 128 and 256 x 128, 3 buffers, 8 waves, one block: 0.60 and 0.78
// and a few microseconds of prologue and epilogue per round, which nothing
// overlaps. So: 64 x 64 while they do not fill the device (226 x 3,072, K = 4,096:
// 14.5 us against 36.7 on 128 x 64; 256 x 3,072, K = 12,288: 59.6 against 104), then
// the smallest of 96 and 128 x 128 that fits it once (2,688 x 1,024, K = 4,096: 37.5
// us against 41.6 on 128 x 128 and 45.1 on 128 x 64 with two buffers; 3,000 x
// 1,536, K = 1,536: 18.8, 21.6 and 24.9), then the cheapest of two 128 x 128 blocks
// per CU (2,688 x 3,072, K = 1,024: 24.2 us against 27.4 on 192 x 128) and rounds of
// 192 x 128 (2,688 x 4,096, K = 1,024: 30.4 us against 33.9 on 256 x 128) or 256 x
// 128 (5,000 x 1,536, K = 1,536: 24.3 against 29.8 on 128 x 128), which need
// 16-byte output rows.
enum SmallTile { T64, T128_64, T96_128, T128_ONE, T128_TWO, T192_128, T256_128 };
SmallTile pick_small(const GemmArgs &g, bool out16, double *us) {
  const int64_t cus = device_cus() > 0 ? device_cus() : 256;
  const double st = (double)(g.k / BK);
  auto rounds = [&](int64_t tiles) { return (double)((tiles + cus - 1) / cus); };
  const int64_t t64 = tile_count(g, 64, 64);
  *us = 0.19 * st + 2.5;
  if (t64 <= cus) return T64;
  if (g.n % 128 != 0) {   // narrow outputs (the output head: n = 64 latent values per token)
    *us = (0.30 * st + 2.5) * rounds(t64);
    return t64 <= 3 * cus ? T64 : T128_64;
  }
  const int64_t t128 = tile_count(g, 128, 128), t256 = tile_count(g, 256, 128);
  // rounds of two 128 x 128 blocks per CU (and a last one of single blocks)
  // against rounds of 256 x 128 blocks: stage time x stages + the prologue and
  // epilogue of a round, which nothing overlaps
  const double pair = 0.95 * st + 9.4, single = 0.53 * st + 4.0;
  *us = 0.43 * st + 4.0;
  if (tile_count(g, 96, 128) <= cus) return T96_128;
  *us = single;
  if (t128 <= cus) return T128_ONE;
  const int64_t rest = t128 % (2 * cus);
  const double c128 = pair * (double)(t128 / (2 * cus)) + (rest == 0 ? 0.0 : rest <= cus ? single : pair);
  const double c256 = (0.78 * st + 4.0) * rounds(t256);
  const double c192 = (0.60 * st + 4.5) * rounds(tile_count(g, 192, 128));
  *us = out16 ? std::min({c128, c192, c256}) : c128;
  return *us == c128 ? T128_TWO : *us == c256 ? T256_128 : T192_128;
}

hipError_t launch_small(const GemmArgs &g, bool out16, hipStream_t s) {
  double us;
  switch (pick_small(g, out16, &us)) {
    case T64:
      // lone blocks, at most one per compute unit: loading waves of their own, two
      // stages per barrier (226 x 3,072, K = 4,096: 14.5 us against 18.4; 16 x 4,096,
      // K = 8,192: 32.0 and 48; 256 x 3,072, K = 12,288: 59.6 and 73; 300 x 1,536, K =
      // 1,536: 7.1 and 8.5; below K = 512 both are as long as the launch; weights from HBM)
      if (tile_count(g, 64, 64) <= device_cus()) return launch_mfma<64, 64, 2, 2, 6, 2>(g, s);
      return launch_mfma<64, 64, 2, 2, 3>(g, s);
    case T128_64: return launch_mfma<128, 64, 2, 2>(g, s);
    case T96_128: return launch_mfma<96, 128, 2, 2, 4>(g, s);
    case T128_ONE: return launch_mfma<128, 128, 2, 2, 4>(g, s);
    case T192_128: return launch_mfma<192, 128, 4, 2, 3>(g, s);
    case T128_TWO: return launch_mfma<128, 128, 2, 2>(g, s);
    default: return launch_mfma<256, 128, 4, 2, 3>(g, s);
  }
}

// Rows [m0, m) and columns [n0, n) of a product, as a product of its own
GemmArgs sub_product(const GemmArgs &g, int64_t m0, int64_t n0) {
  GemmArgs t = g;
  const int64_t o = m0 * g.ldc + n0;
  t.m = g.m - m0;
  t.n = g.n - n0;
  t.a = (const bf16_t *)g.a + m0 * g.lda;
  t.w = (const bf16_t *)g.w + n0 * g.k;
  if (g.bias) t.bias = (const bf16_t *)g.bias + n0;
  if (g.gate) t.gate = g.gate + n0;
  if (g.epi == EPI_QKV) {
    t.qkv.rbase += m0;
    t.qkv.cbase += n0;
  } else {
    t.c = g.epi == EPI_STORE || g.epi == EPI_GELU ? (void *)((bf16_t *)g.c + o) : (void *)((float *)g.c + o);
  }
  return t;
}

// The leftover of a large product on smaller tiles. The fused q/k/v epilogue
// needs tiles of whole heads: 128 x 128 ones where 64 x 64 would be picked.
hipError_t launch_tail(const GemmArgs &g, bool out16, hipStream_t s) {
  double us;
  if (g.epi == EPI_QKV && pick_small(g, out16, &us) == T64) return launch_mfma<128, 128, 2, 2, 4>(g, s);
  return launch_small(g, out16, s);
}

// A product on 256 x 256 tiles: the tiles that fill whole dispatch rounds, then
// what is left of them on smaller tiles, when those take less than the thin last
// round would (a round: 1.45 us a K stage and 8 us of prologue and epilogue).
// In the rectangle order the last chunks of the last chunk row are left, else the
// last rows. 17,776 x 3,072, K = 3,072 (3.28 rounds): 323 -> 314 us; 21,504 x
// 4,096, K = 1,024 (5.25): 172 -> 168; 67,576 x 3,072, K = 3,072 (12.4): 1,026 ->
// 997; 118,800 x 3,072, K = 15,360 (22 rounds and one chunk): 8.63 -> 8.41 ms; less
// than the idle compute units suggest, since a thin round runs at a higher clock.
// Every output is summed in the same order on all of them.
hipError_t launch_big(const GemmArgs &g, bool out16, hipStream_t s) {
  const int64_t cus = device_cus();
  const double round = 1.45 * (double)(g.k / BK) + 8.0;
  double us;
  const int chunks = rect_chunks(g);
  if (chunks > 0 && chunks % 8 != 0 && chunks % 8 <= g.n / (256 * RECT_N)) {
    const int left = chunks % 8;
    const GemmArgs t = sub_product(g, ((g.m + 255) / 256 - 1) / RECT_M * RECT_M * 256, g.n - left * RECT_N * 256);
    (void)pick_small(t, out16, &us);
    if (us < 0.85 * round) {
      const hipError_t e = launch_mfma<256, 256, 2, 4>(g, s, chunks - left);
      return e != hipSuccess ? e : launch_tail(t, out16, s);
    }
  } else if (chunks == 0 && cus > 0) {
    const int64_t per_row = g.n / 256 * (g.batch > 1 ? g.batch : 1), full = tile_count(g, 256, 256) / cus * cus;
    const int64_t m1 = full / per_row * 256;   // rows in whole rounds
    if (m1 > 0 && m1 < g.m) {
      const GemmArgs t = sub_product(g, m1, 0);
      (void)pick_small(t, out16, &us);
      if (us < 0.85 * round) {
        GemmArgs g1 = g;
        g1.m = m1;
        const hipError_t e = launch_mfma<256, 256, 2, 4>(g1, s);
        return e != hipSuccess ? e : launch_tail(t, out16, s);
      }
    }
  }
  return launch_mfma<256, 256, 2, 4>(g, s);
}

// products on fewer 256 x 256 tiles than the device has compute units take
// smaller tiles when the caller allows it (GemmArgs::fill_tiles)
bool small_product(const GemmArgs &g) {
  const int64_t tiles = (g.m + 255) / 256 * (g.n / 256) * (g.batch > 1 ? g.batch : 1);
  return g.fill_tiles && g.n % 128 == 0 && tiles < device_cus();
}
}  // namespace

bool gemm_qkv_fusable(int dtype, const GemmArgs &g) {
  const QkvOut &o = g.qkv;
  return dtype == 1 && operands_aligned(g) && g.n % 256 == 0 && g.m >= 512 && g.k < 8192 && (!small_product(g) || tile_count(g, 64, 64) > device_cus()) &&
         (o.hd == 64 || o.hd == 128) && o.d % 256 == 0 && g.n == 3 * (int64_t)o.d && o.rps > 0 &&
         o.n_pad % 8 == 0 && (uintptr_t)o.q % 16 == 0 && (uintptr_t)o.k % 16 == 0 && (uintptr_t)o.v % 16 == 0 &&
         (uintptr_t)o.rope % 16 == 0;
}

hipError_t launch_gemm(int dtype, const GemmArgs &g_in, hipStream_t s) {
  GemmArgs g = g_in;
  if (g.m <= 0 || g.n <= 0) return hipSuccess;
  if (g.epi == EPI_GATE_RES_NT) return hipErrorInvalidValue;   // internal, chosen below
  if (g.epi == EPI_QKV && !gemm_qkv_fusable(dtype, g)) return hipErrorInvalidValue;
  // the MFMA kernels read 16-byte operand chunks and write 4-column output groups
  const bool aligned = operands_aligned(g);
  if (dtype == 1 && aligned) {
    static DeviceOnce once;
    const hipError_t lim = once_on_device(once, [] {
      hipError_t e = set_lds_limit<256, 256, 2, 4>();
      if (e == hipSuccess) e = set_lds_limit<256, 128, 4, 2, 3>();
      if (e == hipSuccess) e = set_lds_limit<192, 128, 4, 2, 3>();
      if (e == hipSuccess) e = set_lds_limit<128, 128, 2, 2>();
      if (e == hipSuccess) e = set_lds_limit<96, 128, 2, 2, 4>();
      if (e == hipSuccess) e = set_lds_limit<128, 128, 2, 2, 4>();
      if (e == hipSuccess) e = set_lds_limit<128, 64, 2, 2>();
      if (e == hipSuccess) e = set_lds_limit<64, 64, 2, 2, 3>();
      if (e == hipSuccess) e = set_lds_limit<64, 64, 2, 2, 6, 2>();
      return e;
    });
    if (lim != hipSuccess) return lim;
    // 256 x 256 block tiles: 8 waves of 128 x 64 (two per SIMD). With the reads
    // and loads interleaved into the MFMA stream they were 0.3-1.5% faster than
    // 16 waves of 64 x 64 on the 13B products and read a quarter fewer LDS
    // bytes per MFMA (the chip is power-limited under this load).
    // Gated residual of a long-K product: the float32 stream's read-modify-write
    // goes past the caches (non-temporal), which then keep the A and weight
    // tiles: +7.5% at K = 12,288, +2% at K = 15,360; at K = 3,072 it was 1.5%
    // slower, so shorter products keep cached accesses.
    if (g.epi == EPI_GATE_RES && g.k >= 8192) g.epi = EPI_GATE_RES_NT;
    // the 256 x 256 kernels stage bf16 outputs through LDS and store whole
    // 16-byte row chunks: they need 16-byte-aligned output rows (other bf16
    // outputs take the 128 x 128 kernels, which store 8-byte groups)
    const bool c16 = g.epi == EPI_STORE || g.epi == EPI_GELU;
    const bool out16 = !c16 || ((uintptr_t)g.c % 16 == 0 && g.ldc % 8 == 0 && (g.batch <= 1 || g.c_bs % 8 == 0));
    if (g.epi == EPI_QKV && !small_product(g)) return launch_big(g, out16, s);
    // A product that would leave compute units idle in its only dispatch round of
    // 256 x 256 tiles (the mid-size model's products: 44 to 176 of them) runs on
    // smaller ones. Every output is summed over K in the same order on any tile shape,
    // so the results are the same bits.
    if (small_product(g)) return launch_small(g, out16, s);
    if (g.n % 256 == 0 && g.m >= 512 && out16) return launch_big(g, out16, s);
    if (g.n % 64 == 0) return launch_small(g, out16, s);
  }
  if (dtype == 0 && gemm_f32_mfma(g)) return launch_gemm_f32(g, s);
  dim3 grid((unsigned)((g.n + 63) / 64), (unsigned)((g.m + 63) / 64), g.batch > 1 ? g.batch : 1), block(256);
  if (dtype == 1)
    hipLaunchKernelGGL(k_gemm_simple<bf16_t>, grid, block, 0, s, g);
  else
    hipLaunchKernelGGL(k_gemm_simple<float>, grid, block, 0, s, g);
  return hipGetLastError();
}

}  // namespace wdc

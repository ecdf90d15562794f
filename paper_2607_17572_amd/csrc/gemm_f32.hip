// fp32 GEMM of the DiT forward and backward on gfx950: every product the bf16
// MFMA kernels do not cover (fp32 operands; bf16 operands whose rows are not
// 16-byte aligned, converted exactly while they are staged).
//
// The products run on the matrix cores in fp32 (v_mfma_f32_32x32x2_f32: fp32
// operands, fp32 accumulation), at twice the vector ALUs' rate without packed
// instructions and with one LDS read per 64 cycles of a SIMD.  The bound is
// the matrix cores (157 TFLOP/s) when the tiles fill the chip, and the chain
// of K / 2 dependent MFMAs of one 32x32 tile when they do not, so the tile is
// chosen for the number of workgroups.  Four waves per workgroup, T x T tile:
//   T = 64: 32 x 32 per wave, 32-deep k tiles;
//   T = 32: the waves split each 64-deep k tile in four 16-deep slices of the
//           same 32 x 32 outputs and add their sums through LDS in fixed
//           order at the end: chains four times shorter.
// Measured (two products in a launch, as text and image stream): 1332 x 2048 x
// 512 in 32.1 us (87 TFLOP/s), 1332 x 512 x 2048 in 35.9 us, 5000 x 4096 x
// 1024 in 354 us (119 TFLOP/s); the 64x64 vector-ALU kernel that this replaced
// took 121, 323 and about 4600 us.  A 128 x 128 tile of eight waves gave 126
// TFLOP/s on the last of them and less on every product below 512 of its
// tiles, so there is none.
//
// Every k tile is 2048 elements per operand: two 16-byte loads per thread,
// through registers into one of two LDS stages, the next tile's loads in
// flight during a tile's MFMAs.
//
// Contraction slots: an MFMA takes k = 0 from lanes 0-31 and k = 1 from lanes
// 32-63; of each 8-deep step, MFMA i takes k = i and k = i + 4, so that a lane
// reads four consecutive k of a k-contiguous operand as one 16-byte LDS read.
#include "gemm.h"
#include "prof.h"

namespace jg {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// One operand of a T x T tile: T rows x BK of k, two groups of four
// consecutive elements per thread.
//   k-contiguous (TR false): P[row * ld + k], LDS [row][BK + 4]
//   k-strided (TR true):     P[k * ld + row], LDS [k][T + 8]
// Both LDS strides keep the 16-byte writes and the fragment reads (8 rows of
// one chunk; 32 rows of k and of k + 4) on distinct banks.
// VEC: every group is 16-byte aligned fp32 inside the contiguous dimension and
// the operand lies within 32-bit byte offsets: buffer loads, whose range check
// returns zero past the operand (k >= K of a k-strided operand, rows past the
// last one); k >= K of a k-contiguous one is sent past it.  Rows of a k-strided
// operand past its end may read the next k's elements, which only reach
// outputs that are never stored.  Otherwise element loads of either type.
constexpr int F32_OOB = 0x7ffffff0;

template <int T, bool TR, bool VEC>
struct F32Op {
  static constexpr int NT = 256, BK = NT * 8 / T;
  static constexpr int LDS_S = TR ? T + 8 : BK + 4;
  static constexpr int LDS_N = TR ? BK * LDS_S : T * LDS_S;
  static constexpr int VPR = (TR ? T : BK) / 4;  // groups per row of the tile
  const void* P;
  __amdgpu_buffer_rsrc_t R;
  int dt, ld, rows, K, row0;
  int voff[2], k_in[2];
  float4 r[2];
  __device__ inline void init(const void* p, int dt_, int ld_, int rows_, int K_, int row0_) {
    P = p; dt = dt_; ld = ld_; rows = rows_; K = K_; row0 = row0_;
    if constexpr (VEC) {
      const long ext = TR ? (long)(K - 1) * ld + rows : (long)(rows - 1) * ld + K;
      R = __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, (int)(ext * 4), 0x00020000);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int v = threadIdx.x + NT * i, outer = v / VPR, inner = (v % VPR) * 4;
        k_in[i] = TR ? outer : inner;
        voff[i] = (TR ? outer * ld + row0 + inner : (row0 + outer) * ld + inner) * 4;
      }
    }
  }
  __device__ inline void load(int k0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if constexpr (VEC) {
        int o = voff[i] + (TR ? k0 * ld : k0) * 4;
        if (!TR) o = k0 + k_in[i] < K ? o : F32_OOB;
        r[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(R, o, 0, 0));
      } else {
        const int v = threadIdx.x + NT * i, outer = v / VPR, inner = (v % VPR) * 4;
        const int row = row0 + (TR ? inner : outer), k = k0 + (TR ? outer : inner);
        // a: the strided index, c: the first of the four contiguous ones
        const int a = TR ? k : row, an = TR ? K : rows, c = TR ? row : k, cn = TR ? rows : K;
        const size_t o = (size_t)a * ld + c;
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        if (a < an) {
          if (c < cn) x.x = ld_any(P, dt, o);
          if (c + 1 < cn) x.y = ld_any(P, dt, o + 1);
          if (c + 2 < cn) x.z = ld_any(P, dt, o + 2);
          if (c + 3 < cn) x.w = ld_any(P, dt, o + 3);
        }
        r[i] = x;
      }
    }
  }
  __device__ inline void store(float* S) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int v = threadIdx.x + NT * i;
      *(float4*)(S + (v / VPR) * LDS_S + (v % VPR) * 4) = r[i];
    }
  }
  // the lane's values of the 8-deep step at k: k + 4h + 0..3 of tile row `row`
  __device__ static inline void frag(const float* S, int row, int k, int h, float (&f)[4]) {
    if (!TR) {
      const float4 x = *(const float4*)(S + row * LDS_S + k + 4 * h);
      f[0] = x.x; f[1] = x.y; f[2] = x.z; f[3] = x.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) f[i] = S[(k + 4 * h + i) * LDS_S + row];
    }
  }
};

// n results v[] of one column (rows r0 + row(e)): the inputs of the epilogue
// (GELU input, old C) are loaded for all of them before the first use, so that
// their latency is paid once per 32x32 tile.
template <int NE, class Row>
__device__ __forceinline__ void f32_epilogue(const GemmArgs& g, int col, float* v, Row row) {
  const Epi& e = g.epi;
  if (col >= g.N) return;
  if (e.bias) {
    const float b = ld_any(e.bias, e.bias_dt, col);
#pragma unroll
    for (int q = 0; q < NE; ++q) v[q] += b;
  }
  auto gather = [&](const void* p, int dt, int ld, float (&x)[NE]) {
    if (dt == F32) {
#pragma unroll
      for (int q = 0; q < NE; ++q) x[q] = row(q) < g.M ? ((const float*)p)[(size_t)row(q) * ld + col] : 0.f;
    } else {
#pragma unroll
      for (int q = 0; q < NE; ++q) x[q] = row(q) < g.M ? bf2f(((const uint16_t*)p)[(size_t)row(q) * ld + col]) : 0.f;
    }
  };
  auto scatter = [&](void* p, int dt, int ld) {
    if (dt == F32) {
#pragma unroll
      for (int q = 0; q < NE; ++q)
        if (row(q) < g.M) ((float*)p)[(size_t)row(q) * ld + col] = v[q];
    } else {
#pragma unroll
      for (int q = 0; q < NE; ++q)
        if (row(q) < g.M) ((uint16_t*)p)[(size_t)row(q) * ld + col] = f2bf(v[q]);
    }
  };
  float x[NE];
  if (e.mode == EPI_GELU_FWD) {
    scatter(e.aux, e.aux_dt, e.ldaux);
#pragma unroll
    for (int q = 0; q < NE; ++q) v[q] = gelu_tanh(v[q]);
  } else if (e.mode == EPI_GELU_BWD) {
    gather(e.aux, e.aux_dt, e.ldaux, x);
#pragma unroll
    for (int q = 0; q < NE; ++q) v[q] *= gelu_tanh_grad(x[q]);
  }
  if (e.beta != 0.f) {
    gather(e.C, e.c_dt, e.ldc, x);
#pragma unroll
    for (int q = 0; q < NE; ++q) v[q] += e.beta * x[q];
  }
  scatter(e.C, e.c_dt, e.ldc);
}

template <int T, bool TA, bool TB, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmGroup gg) {
  typedef F32Op<T, TA, VEC> OpA;
  typedef F32Op<T, TB, VEC> OpB;
  constexpr int BK = OpA::BK, STG = OpA::LDS_N + OpB::LDS_N;
  constexpr bool KS = T == 32;          // the waves split k
  constexpr int KW = KS ? BK / 4 : BK;  // k depth of a wave per tile
  __shared__ __attribute__((aligned(16))) float lds[2 * STG];

  // the first tiles0 workgroups compute problem 0, the rest problem 1
  const int sel = (int)blockIdx.x >= gg.tiles0 ? 1 : 0;
  const GemmArgs& g = gg.p[sel];
  const int id = (int)blockIdx.x - sel * gg.tiles0, tiles_n = (g.N + T - 1) / T;
  const int m0 = (id / tiles_n) * T, n0 = (id % tiles_n) * T;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, c32 = lane & 31;
  const int wm = KS ? 0 : (wave >> 1) * 32, wn = KS ? 0 : (wave & 1) * 32;
  const int kw = KS ? wave * KW : 0;

  OpA oa;
  OpB ob;
  oa.init(g.A, g.a_dt, g.lda, g.M, g.K, m0);
  ob.init(g.B, g.b_dt, g.ldb, g.N, g.K, n0);
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;

  const int nk = (g.K + BK - 1) / BK;
  if (nk > 0) {
    oa.load(0);
    ob.load(0);
    oa.store(lds);
    ob.store(lds + OpA::LDS_N);
  }
  if (nk > 1) {
    oa.load(BK);
    ob.load(BK);
  }
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const float* As = lds + (kt & 1) * STG;
    const float* Bs = As + OpA::LDS_N;
    if (kt + 1 < nk) {
      float* An = lds + ((kt + 1) & 1) * STG;
      oa.store(An);
      ob.store(An + OpA::LDS_N);
    }
    if (kt + 2 < nk) {
      oa.load((kt + 2) * BK);
      ob.load((kt + 2) * BK);
    }
#pragma unroll
    for (int kk = 0; kk < KW / 8; ++kk) {
      float fa[4], fb[4];
      OpA::frag(As, wm + c32, kw + 8 * kk, h, fa);
      OpB::frag(Bs, wn + c32, kw + 8 * kk, h, fb);
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[s], fb[s], acc, 0, 0, 0);
    }
    __syncthreads();
  }

  if constexpr (KS) {
    // the four slices' sums, added in slice order; thread t then owns rows
    // t / 32 + 8 q of column t % 32
    static_assert(4 * 1024 <= 2 * STG, "the partial sums must fit the stages");
#pragma unroll
    for (int e = 0; e < 16; ++e) lds[wave * 1024 + (8 * (e >> 2) + 4 * h + (e & 3)) * 32 + c32] = acc[e];
    __syncthreads();
    const int c = threadIdx.x & 31, r = threadIdx.x >> 5;
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int o = (r + 8 * q) * 32 + c;
      v[q] = ((lds[o] + lds[1024 + o]) + lds[2048 + o]) + lds[3072 + o];
    }
    f32_epilogue<4>(g, n0 + c, v, [&](int q) { return m0 + r + 8 * q; });
  } else {
    float v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = acc[e];
    f32_epilogue<16>(g, n0 + wn + c32, v, [&](int q) { return m0 + wm + 8 * (q >> 2) + 4 * h + (q & 3); });
  }
}

static long f32_tiles(const GemmArgs& g, int T) { return (long)((g.M + T - 1) / T) * ((g.N + T - 1) / T); }

template <int T, bool TA, bool TB>
static void launch_f32(GemmGroup& g, hipStream_t s, bool vec) {
  g.tiles0 = (int)f32_tiles(g.p[0], T);
  const int tiles = g.tiles0 + (g.np > 1 ? (int)f32_tiles(g.p[1], T) : 0);
  if (vec) launch(gemm_f32_kernel<T, TA, TB, true>, dim3(tiles), dim3(256), 0u, s, g);
  else launch(gemm_f32_kernel<T, TA, TB, false>, dim3(tiles), dim3(256), 0u, s, g);
}

template <int T>
static void launch_f32_t(GemmGroup& g, hipStream_t s, bool vec) {
  const GemmArgs& a = g.p[0];
  if (!a.ta && !a.tb) launch_f32<T, false, false>(g, s, vec);
  else if (!a.ta) launch_f32<T, false, true>(g, s, vec);
  else if (a.tb) launch_f32<T, true, true>(g, s, vec);
  else launch_f32<T, true, false>(g, s, vec);
}

// The vector loads' conditions for one problem (byte offsets up to three k
// tiles of 64 past K stay below 2^31).
static bool f32_vec(const GemmArgs& g) {
  const double kx = (double)g.K + 192.0;
  const double ea = 4.0 * (g.ta ? kx * g.lda + g.M + 128.0 : ((double)g.M + 128.0) * g.lda + kx);
  const double eb = 4.0 * (g.tb ? kx * g.ldb + g.N + 128.0 : ((double)g.N + 128.0) * g.ldb + kx);
  return g.K > 0 && g.a_dt == F32 && g.b_dt == F32 && g.lda % 4 == 0 && g.ldb % 4 == 0 &&
         (((uintptr_t)g.A | (uintptr_t)g.B) & 15) == 0 && (g.ta ? g.M : g.K) % 4 == 0 &&
         (g.tb ? g.N : g.K) % 4 == 0 && ea < 2147483000.0 && eb < 2147483000.0;
}

int gemm_f32(const GemmGroup& gr, hipStream_t s) {
  GemmGroup g = gr;
  const bool vec = f32_vec(g.p[0]) && (g.np < 2 || f32_vec(g.p[1]));
  // 64 x 64 tiles need about two workgroups per CU to keep the matrix cores
  // fed: at 504 and 512 of them they are 9% and 4% faster than 32 x 32 tiles
  // (22.8 against 25.0 us, 32.4 against 33.6), at 384 22% slower (31.4 against
  // 25.8), at 168 31% slower (47.0 against 35.9)
  const long t64 = f32_tiles(g.p[0], 64) + (g.np > 1 ? f32_tiles(g.p[1], 64) : 0);
  if (t64 >= 480) launch_f32_t<64>(g, s, vec);
  else launch_f32_t<32>(g, s, vec);
  JG_CHECK_LAUNCH("gemm_f32");
  return 0;
}

}  // namespace jg

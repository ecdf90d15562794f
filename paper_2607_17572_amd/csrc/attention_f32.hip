// Softmax attention in fp32 arithmetic on the matrix cores
// (v_mfma_f32_32x32x2_f32): fp32 storage with any supported head dim, and bf16
// storage where the bf16 kernels of attention_mfma.hip do not apply (head dims
// 16 and 32); D is the head dim, T the storage type.
//
// Accumulators feed the next product as in attention_mfma.hip: a lane holds
// column c = lane % 32 of a 32 x 32 score tile and its rows
// r(e, h) = 8 (e / 4) + 4 h + e % 4, h = lane / 32, and MFMA e of the next
// product contracts rows r(e, 0) and r(e, 1), so the score register e is its
// B operand as it stands.
//   forward:  S^T = K Q^T, O^T += V^T P^T            (column = query)
//   dK/dV:    S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS (column = key)
//   dQ:       S^T, dP^T = V dO^T, dQ^T += K^T dS^T    (column = query)
// The other operand comes straight from memory (L2): 16 bytes of a row per lane
// for the score products, 32 consecutive elements of a row per half-wave for
// the others.  One MFMA takes 64 cycles of a SIMD and needs one element per
// lane of it, so neither LDS staging nor its barriers pay; the bound is the
// matrix cores, or at few tokens the chain of one wave's tiles.  A workgroup
// therefore owns 32 columns and its four waves take every fourth tile of the
// other side; their partial sums meet in LDS, added in wave order.
// Rows past N are read from row N - 1 and their probabilities set to 0.
// 8 heads of 64 x 4 samples, 333 tokens, fp32: forward, dK/dV and dQ took 102,
// 140 and 158 us on the vector ALUs (four lanes per row, keys staged in LDS),
// and the row sums of dO O 18 us with one lane per row; here 39, and 90 for the
// backward in one launch (56 + 32 + 4 in three).
#include "attention.h"
#include "prof.h"

namespace jg {

typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ inline int row_of_tok(const RowMap& rm, int b, int j) {
  return j < rm.nt ? b * rm.nt + j : rm.B * rm.nt + b * rm.ni + (j - rm.nt);
}
__device__ inline f32x16 mfma2(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ inline f32x16 zero() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}
__device__ inline int acc_row(int e, int h) { return 8 * (e >> 2) + 4 * h + (e & 3); }

// four consecutive elements
__device__ inline void ld4(const float* p, float* f) {
  const float4 v = *(const float4*)p;
  f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
}
__device__ inline void ld4(const uint16_t* p, float* f) {
  const uint2 v = *(const uint2*)p;
  f[0] = bf2f(v.x & 0xffffu); f[1] = bf2f(v.x >> 16); f[2] = bf2f(v.y & 0xffffu); f[3] = bf2f(v.y >> 16);
}

// the lane's share of a row for a score product: elements 8 kb + 4 h + 0..3
template <int D, typename T>
struct Row {
  float f[D / 2];
  __device__ inline void load(const T* row, int h) {
#pragma unroll
    for (int kb = 0; kb < D / 8; ++kb) ld4(row + 8 * kb + 4 * h, f + 4 * kb);
  }
  // of a token-major operand; VEC: its rows allow the four-element loads
  template <bool VEC>
  __device__ inline void load_tok(const T* row, int h) {
    if constexpr (VEC) {
      load(row, h);
    } else {
#pragma unroll
      for (int i = 0; i < D / 2; ++i) f[i] = ldf(row, 8 * (i >> 2) + 4 * h + (i & 3));
    }
  }
};
template <int D, typename T>
__device__ inline f32x16 score(const Row<D, T>& a, const Row<D, T>& b) {
  f32x16 s = zero();
#pragma unroll
  for (int i = 0; i < D / 2; ++i) s = mfma2(a.f[i], b.f[i], s);
  return s;
}
// acc[dt] += M^T[d][r] x[r][column]: row(r) = pointer to the row of tile row r
template <int D, typename T, class RowPtr>
__device__ inline void accumulate(f32x16 (&acc)[(D + 31) / 32], const f32x16& x, int h, int c32, RowPtr row) {
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const T* p = row(acc_row(e, h));
#pragma unroll
    for (int dt = 0; dt < (D + 31) / 32; ++dt) {
      const float m = D < 32 && c32 >= D ? 0.f : ldf(p, 32 * dt + c32);
      acc[dt] = mfma2(m, x[e], acc[dt]);
    }
  }
}

// The four waves' column sums: part holds [4][D][33] floats; out(c, d, v) gets
// each sum once, consecutive threads consecutive d.
template <int D, class Out>
__device__ inline void merge(float* part, const f32x16 (&acc)[(D + 31) / 32], int w, int h, int c32, Out out) {
#pragma unroll
  for (int dt = 0; dt < (D + 31) / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int d = 32 * dt + acc_row(e, h);
      if (d < D) part[(w * D + d) * 33 + c32] = acc[dt][e];
    }
  __syncthreads();
  for (int i = threadIdx.x; i < 32 * D; i += 256) {
    const int c = i / D, d = i % D;
    const float* p = part + d * 33 + c;
    out(c, d, ((p[0] + p[D * 33]) + p[2 * D * 33]) + p[3 * D * 33]);
  }
  __syncthreads();
}

constexpr float LOG2E_F = 1.4426950408889634f, LN2_F = 0.6931471805599453f;

template <int D, typename T>
__global__ __launch_bounds__(256) void attn_fwd_f32_k(AttnFwd a) {
  constexpr int DT = (D + 31) / 32;
  __shared__ float part[4 * D * 33], ms[4][32], ls[4][32];
  const int bh = blockIdx.y, b = bh / a.H, hd = bh % a.H, N = a.N;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, h = lane >> 5, c32 = lane & 31;
  const int q0 = blockIdx.x * 32;
  const size_t base = (size_t)bh * N * D;
  const T *Q = (const T*)a.Q + base, *K = (const T*)a.K + base, *V = (const T*)a.V + base;
  const float sc = rsqrtf((float)D) * LOG2E_F;
  Row<D, T> qr;
  qr.load(Q + (size_t)min(q0 + c32, N - 1) * D, h);
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = zero();
  float m = -INFINITY, l = 0.f;
  for (int k0 = 32 * w; k0 < N; k0 += 128) {
    Row<D, T> kr;
    kr.load(K + (size_t)min(k0 + c32, N - 1) * D, h);
    f32x16 s = score<D, T>(kr, qr);
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if (k0 + acc_row(e, h) >= N) s[e] = -INFINITY;
      mx = fmaxf(mx, s[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * sc;
    const float mn = fmaxf(m, mx), corr = __builtin_amdgcn_exp2f(m - mn);
    m = mn;
    l *= corr;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[e] = __builtin_amdgcn_exp2f(fmaf(s[e], sc, -m));
      l += s[e];
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[dt][e] *= corr;
    accumulate<D, T>(o, s, h, c32, [&](int r) { return V + (size_t)min(k0 + r, N - 1) * D; });
  }
  l += __shfl_xor(l, 32, 64);
  if (h == 0) {
    ms[w][c32] = m;
    ls[w][c32] = l;
  }
  __syncthreads();
  // waves without a tile hold m = -inf and l = 0
  const float M = fmaxf(fmaxf(ms[0][c32], ms[1][c32]), fmaxf(ms[2][c32], ms[3][c32]));
  float L = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) L += ls[i][c32] * __builtin_amdgcn_exp2f(ms[i][c32] - M);
  const float f = __builtin_amdgcn_exp2f(m - M) / L;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[dt][e] *= f;
  if (threadIdx.x < 32 && q0 + c32 < N) a.lse[(size_t)bh * N + q0 + c32] = (M + log2f(L)) * LN2_F;
  T* O = (T*)a.O;
  merge<D>(part, o, w, h, c32, [&](int c, int d, float v) {
    if (q0 + c < N) stf(O, (size_t)row_of_tok(a.rm, b, q0 + c) * a.ld_o + hd * D + d, v);
  });
}

// sum over the row of a row's two halves: lanes c32 and c32 + 32
template <int D, typename T>
__device__ inline float row_dot(const Row<D, T>& a, const Row<D, T>& b) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < D / 2; ++i) s = fmaf(a.f[i], b.f[i], s);
  return s + __shfl_xor(s, 32, 64);
}

// The row sums delta = sum_d dO O are formed where they are needed (per query
// of a tile, per column), from a row of O beside the row of dO.
template <int D, typename T, bool VEC>
__device__ __forceinline__ void bwd_kv_f32(const AttnBwd& a, float* part) {
  constexpr int DT = (D + 31) / 32;
  const int bh = blockIdx.y, b = bh / a.H, hd = bh % a.H, N = a.N;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, h = lane >> 5, c32 = lane & 31;
  const int key0 = blockIdx.x * 32;
  const size_t base = (size_t)bh * N * D;
  const T *Q = (const T*)a.Q + base, *K = (const T*)a.K + base, *V = (const T*)a.V + base;
  const T* G = (const T*)a.dO + hd * D;
  const float* lse = a.lse + (size_t)bh * N;
  const float scale = rsqrtf((float)D), sc = scale * LOG2E_F;
  Row<D, T> kr, vr;
  kr.load(K + (size_t)min(key0 + c32, N - 1) * D, h);
  vr.load(V + (size_t)min(key0 + c32, N - 1) * D, h);
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dk[dt] = dv[dt] = zero();
  for (int q0 = 32 * w; q0 < N; q0 += 128) {
    auto grow = [&](int r) { return G + (size_t)row_of_tok(a.rm, b, min(q0 + r, N - 1)) * a.ld_do; };
    auto qrow = [&](int r) { return Q + (size_t)min(q0 + r, N - 1) * D; };
    Row<D, T> x;
    x.load(qrow(c32), h);
    f32x16 p = score<D, T>(x, kr);
    x.template load_tok<VEC>(grow(c32), h);
    f32x16 ds = score<D, T>(x, vr);
    Row<D, T> o;
    o.template load_tok<VEC>((const T*)a.O + (size_t)row_of_tok(a.rm, b, min(q0 + c32, N - 1)) * a.ld_o + hd * D, h);
    const float delta = row_dot<D, T>(x, o);  // of query q0 + c32
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int q = q0 + acc_row(e, h), qc = min(q, N - 1);
      const float pe = q < N ? __builtin_amdgcn_exp2f(fmaf(p[e], sc, -lse[qc] * LOG2E_F)) : 0.f;
      p[e] = pe;
      ds[e] = pe * (ds[e] - __shfl(delta, acc_row(e, h), 64));
    }
    accumulate<D, T>(dv, p, h, c32, grow);
    accumulate<D, T>(dk, ds, h, c32, qrow);
  }
  auto put = [&](void* o, float f) {
    return [=](int c, int d, float v) {
      if (key0 + c < N) stf((T*)o, base + (size_t)(key0 + c) * D + d, v * f);
    };
  };
  merge<D>(part, dv, w, h, c32, put(a.dV, 1.f));
  merge<D>(part, dk, w, h, c32, put(a.dK, scale));
}

template <int D, typename T, bool VEC>
__device__ __forceinline__ void bwd_q_f32(const AttnBwd& a, float* part) {
  constexpr int DT = (D + 31) / 32;
  const int bh = blockIdx.y, b = bh / a.H, hd = bh % a.H, N = a.N;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, h = lane >> 5, c32 = lane & 31;
  const int q0 = blockIdx.x * 32, qc = min(q0 + c32, N - 1);
  const size_t base = (size_t)bh * N * D;
  const T *Q = (const T*)a.Q + base, *K = (const T*)a.K + base, *V = (const T*)a.V + base;
  const float scale = rsqrtf((float)D), sc = scale * LOG2E_F;
  Row<D, T> qr, gr;
  qr.load(Q + (size_t)qc * D, h);
  gr.template load_tok<VEC>((const T*)a.dO + (size_t)row_of_tok(a.rm, b, qc) * a.ld_do + hd * D, h);
  Row<D, T> o;
  o.template load_tok<VEC>((const T*)a.O + (size_t)row_of_tok(a.rm, b, qc) * a.ld_o + hd * D, h);
  const float l2 = a.lse[(size_t)bh * N + qc] * LOG2E_F, dl = row_dot<D, T>(gr, o);
  f32x16 dq[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dq[dt] = zero();
  for (int k0 = 32 * w; k0 < N; k0 += 128) {
    Row<D, T> x;
    x.load(K + (size_t)min(k0 + c32, N - 1) * D, h);
    const f32x16 s = score<D, T>(x, qr);
    x.load(V + (size_t)min(k0 + c32, N - 1) * D, h);
    f32x16 ds = score<D, T>(x, gr);
#pragma unroll
    for (int e = 0; e < 16; ++e)
      ds[e] = k0 + acc_row(e, h) < N ? __builtin_amdgcn_exp2f(fmaf(s[e], sc, -l2)) * (ds[e] - dl) : 0.f;
    accumulate<D, T>(dq, ds, h, c32, [&](int r) { return K + (size_t)min(k0 + r, N - 1) * D; });
  }
  merge<D>(part, dq, w, h, c32, [&](int c, int d, float v) {
    if (q0 + c < N) stf((T*)a.dQ, base + (size_t)(q0 + c) * D + d, v * scale);
  });
}

// Both passes in one launch (z = 0: dK and dV, 1: dQ): they are independent,
// and at few tokens neither fills the chip.
template <int D, typename T, bool VEC>
__global__ __launch_bounds__(256) void attn_bwd_f32_k(AttnBwd a) {
  __shared__ float part[4 * D * 33];
  if (blockIdx.z == 0) bwd_kv_f32<D, T, VEC>(a, part);
  else bwd_q_f32<D, T, VEC>(a, part);
}

// ------------------------------------------------------------------ launch
template <int D, typename T>
static void fwd_f32(const AttnFwd& a, hipStream_t s) {
  hipLaunchKernelGGL((attn_fwd_f32_k<D, T>), dim3((a.N + 31) / 32, a.B * a.H), dim3(256), 0, s, a);
}
template <int D, typename T>
static void bwd_f32(const AttnBwd& a, bool vec, hipStream_t s) {
  const dim3 grid((a.N + 31) / 32, a.B * a.H, 2);
  if (vec) hipLaunchKernelGGL((attn_bwd_f32_k<D, T, true>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((attn_bwd_f32_k<D, T, false>), grid, dim3(256), 0, s, a);
}

int attention_fwd_mfma(const AttnFwd& a, hipStream_t s);  // attention_mfma.hip; returns -1 if not applicable
int attention_bwd_mfma(const AttnBwd& a, hipStream_t s);

// four-element loads of a row of the token-major operand
static bool rows_ok(const void* p, int ld, int dt) { return ld % 4 == 0 && (uintptr_t)p % (4 * dsize(dt)) == 0; }

int attention_fwd(const AttnFwd& a, hipStream_t s) {
  if (a.N <= 0 || a.B <= 0 || a.H <= 0) { set_error("attention_fwd: empty problem"); return 1; }
  const int rc = attention_fwd_mfma(a, s);
  if (rc >= 0) return rc;
  switch (a.Dh) {
#define JG_DIM(D) case D: a.dt == BF16 ? fwd_f32<D, uint16_t>(a, s) : fwd_f32<D, float>(a, s); break;
    JG_DIM(16) JG_DIM(32) JG_DIM(64) JG_DIM(128)
#undef JG_DIM
    default: set_error("attention_fwd: head_dim must be 16, 32, 64 or 128"); return 4;
  }
  JG_CHECK_LAUNCH("attention_fwd_f32");
  return 0;
}

int attention_bwd(const AttnBwd& a, hipStream_t s) {
  if (a.N <= 0 || a.B <= 0 || a.H <= 0) { set_error("attention_bwd: empty problem"); return 1; }
  const int rc = attention_bwd_mfma(a, s);
  if (rc >= 0) return rc;
  if (a.dt_d != a.dt) { set_error("attention_bwd: gradients in another type"); return 4; }
  // (a single block's O lies in rows of hidden + mlp_hidden elements)
  const bool vec = rows_ok(a.dO, a.ld_do, a.dt) && rows_ok(a.O, a.ld_o, a.dt);
  switch (a.Dh) {
#define JG_DIM(D) case D: a.dt == BF16 ? bwd_f32<D, uint16_t>(a, vec, s) : bwd_f32<D, float>(a, vec, s); break;
    JG_DIM(16) JG_DIM(32) JG_DIM(64) JG_DIM(128)
#undef JG_DIM
    default: set_error("attention_bwd: head_dim must be 16, 32, 64 or 128"); return 4;
  }
  JG_CHECK_LAUNCH("attention_bwd_f32");
  return 0;
}

}  // namespace jg

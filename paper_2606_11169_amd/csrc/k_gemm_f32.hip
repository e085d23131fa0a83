// fp32 GEMM path (fp32-compute stages) on the fp32 matrix instruction
// (v_mfma_f32_32x32x2_f32: fp32 products and sums), with the operand layouts and
// epilogues of the bf16 kernels.
//
// These products are small (a tiny stage's outputs are 128 x 128 to 128 x 688),
// so one workgroup's serial chain and the number of launches bound them. Every
// workgroup of four waves owns a 32 x 32 or 64 x 64 output tile and the waves
// split k: wave w multiplies the 32-deep steps w, w + 4, ... of the whole tile,
// so no operand value is read by two waves and nothing is staged: fragments go
// from global memory straight into registers, the next step's while one
// multiplies. The four partial tiles are added in wave order through LDS, where
// RoPE and SwiGLU find the two columns they combine (the tile's columns are
// chosen as such pairs), so each product is one launch. (With 64 x 64 tiles
// staged through LDS by scalar loads, and RoPE and SwiGLU as launches of their
// own, a 128 x 384 x 128 product took 38 us and a 400-token d-768 layer's 195 us
// on average.)
#include "common.hpp"

namespace lc {
namespace {

constexpr int NW = 4;    // waves: shares of k
constexpr int KW = 32;   // k per wave and step

struct F32P {
  const float *A;
  const float *B;
  float *C;
  const float *R;
  float *aux0;
  float *aux1;
  const float *rcos, *rsin;
  int64_t lda, ldb, ldc, ldr, ld_aux;
  int M, N, K;
  int epi;
  int rope_cols, rope_seq, hd;
  int vec_a, vec_b;  // k-major rows of whole 16-byte runs
  unsigned tiles_n;
};

// Which column pair tile column j of a T-wide tile belongs to: RoPE's (i, i +
// hd/2) of a head and SwiGLU's (gate, up) are columns j and j + T/2 of one tile.
// Returns the operand row of B; *n the output column (the pair's first, for j
// < T/2), *ok whether it exists.
template <int T>
__device__ __forceinline__ int column(const F32P &p, int tn, int j, int *n, bool *ok) {
  if (p.epi == LC_EPI_SWIGLU) {
    *n = tn * (T / 2) + (j & (T / 2 - 1));
    *ok = *n < p.N;
    return j < T / 2 ? *n : p.N + *n;
  }
  if (p.epi == LC_EPI_ROPE) {
    const int half = p.hd / 2, pair = tn * (T / 2) + (j & (T / 2 - 1));
    *n = pair / half * p.hd + pair % half + (j < T / 2 ? 0 : half);
    *ok = pair < p.N / 2;
    return *n;
  }
  *n = tn * T + j;
  *ok = *n < p.N;
  return *n;
}

// One lane's operand values of a 32-deep step at k: x[4 jj + c] is k + 8 jj + 4 h
// + c (h = lane / 32) of operand row `row` (k-major) or column `row`; values at or
// past K are 0. Both operands use this order, so any layouts can meet.
template <bool KMAJ>
__device__ __forceinline__ void load_step(const float *X, int64_t ld, int row, int k, int K, int h, bool vec,
                                          float (&x)[16]) {
  if constexpr (KMAJ) {
    const float *s = X + (int64_t)row * ld + k + 4 * h;
    if (vec && k + KW <= K) {
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const float4 v = *reinterpret_cast<const float4 *>(s + 8 * jj);
        x[4 * jj] = v.x; x[4 * jj + 1] = v.y; x[4 * jj + 2] = v.z; x[4 * jj + 3] = v.w;
      }
      return;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int o = 8 * (u >> 2) + (u & 3);
      x[u] = k + 4 * h + o < K ? s[o] : 0.0f;
    }
  } else {
    const float *s = X + row;
    if (k + KW <= K) {
#pragma unroll
      for (int u = 0; u < 16; ++u) x[u] = s[(int64_t)(k + 4 * h + 8 * (u >> 2) + (u & 3)) * ld];
      return;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int kk = k + 4 * h + 8 * (u >> 2) + (u & 3);
      x[u] = kk < K ? s[(int64_t)kk * ld] : 0.0f;
    }
  }
}

template <int T, bool A_K, bool B_K>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(F32P p) {
  constexpr int F = T / 32;        // 32 x 32 blocks per side
  constexpr int LD = T + 1;        // row stride of a partial tile in LDS
  __shared__ float part[NW][T * LD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int m0 = (int)(blockIdx.x / p.tiles_n) * T, tn = (int)(blockIdx.x % p.tiles_n);
  // rows and columns past the operands read the last valid one (never stored)
  int arow[F], brow[F];
#pragma unroll
  for (int f = 0; f < F; ++f) {
    arow[f] = min(m0 + 32 * f + l32, p.M - 1);
    int n;
    bool ok;
    brow[f] = column<T>(p, tn, 32 * f + l32, &n, &ok);
    if (!ok) brow[f] = 0;
  }
  f32x16_v acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  float a[2][F][16], b[2][F][16];
  auto load = [&](int k, float (&x)[F][16], float (&y)[F][16]) {
#pragma unroll
    for (int f = 0; f < F; ++f) load_step<A_K>(p.A, p.lda, arow[f], k, p.K, h, p.vec_a, x[f]);
#pragma unroll
    for (int f = 0; f < F; ++f) load_step<B_K>(p.B, p.ldb, brow[f], k, p.K, h, p.vec_b, y[f]);
  };
  auto multiply = [&](const float (&x)[F][16], const float (&y)[F][16]) {
#pragma unroll
    for (int u = 0; u < 16; ++u)
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i][u], y[j][u], acc[i][j], 0, 0, 0);
  };
  constexpr int STEP = NW * KW;
  int k = w * KW;
  if (k < p.K) load(k, a[0], b[0]);
  for (; k < p.K; k += 2 * STEP) {
    if (k + STEP < p.K) load(k + STEP, a[1], b[1]);
    multiply(a[0], b[0]);
    if (k + STEP >= p.K) break;
    if (k + 2 * STEP < p.K) load(k + 2 * STEP, a[0], b[0]);
    multiply(a[1], b[1]);
  }
  // lane: column l32 of a block, rows (r & 3) + 8 (r >> 2) + 4 h
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        part[w][(32 * i + (r & 3) + 8 * (r >> 2) + 4 * h) * LD + 32 * j + l32] = acc[i][j][r];
  __syncthreads();
  auto sum = [&](int r, int c) {
    float v = part[0][r * LD + c];
#pragma unroll
    for (int i = 1; i < NW; ++i) v += part[i][r * LD + c];
    return v;
  };
  const bool pair = p.epi == LC_EPI_SWIGLU || p.epi == LC_EPI_ROPE;
  const int cols = pair ? T / 2 : T;
  const int j = tid % cols;
  int n;
  bool ok;
  column<T>(p, tn, j, &n, &ok);
  if (!ok) return;
  for (int r = tid / cols; r < T; r += 64 * NW / cols) {
    const int m = m0 + r;
    if (m >= p.M) break;
    const float v = sum(r, j);
    float *c = p.C + (int64_t)m * p.ldc + n;
    switch (p.epi) {
      case LC_EPI_ACCUM_F32: *c = *c + v; break;
      case LC_EPI_RESIDUAL: *c = p.R[(int64_t)m * p.ldr + n] + v; break;
      case LC_EPI_SWIGLU_BWD: {
        const float g = p.aux0[(int64_t)m * p.ld_aux + n];
        const float u = p.aux1[(int64_t)m * p.ld_aux + n];
        const float s = sigmoidf_(g);
        c[0] = v * u * s * (1.0f + g * (1.0f - s));
        c[p.N] = v * g * s;
        break;
      }
      case LC_EPI_SWIGLU: {
        const float u = sum(r, j + T / 2);
        p.aux0[(int64_t)m * p.ld_aux + n] = v;
        p.aux1[(int64_t)m * p.ld_aux + n] = u;
        *c = v * sigmoidf_(v) * u;
        break;
      }
      case LC_EPI_ROPE: {
        const float y = sum(r, j + T / 2);
        const int half = p.hd / 2;
        if (n < p.rope_cols) {
          const int64_t t = (int64_t)(m % p.rope_seq) * half + n % p.hd;
          const float cs = p.rcos[t], sn = p.rsin[t];
          c[0] = v * cs - y * sn;
          c[half] = v * sn + y * cs;
        } else {
          c[0] = v;
          c[half] = y;
        }
        break;
      }
      default: *c = v; break;
    }
  }
}

template <int T>
lc_status run_f32(F32P p, bool ak, bool bk, hipStream_t s) {
  const int cols = p.epi == LC_EPI_SWIGLU ? T / 2 : T;
  const int64_t tm = ((int64_t)p.M + T - 1) / T, tn = ((int64_t)p.N + cols - 1) / cols;
  if (tm * tn > INT32_MAX / (64 * NW)) return fail(LC_ERR_UNSUPPORTED, "gemm fp32: output too large");
  p.tiles_n = (unsigned)tn;
  const dim3 grid((unsigned)(tm * tn)), block(64 * NW);
  if (ak && bk) hipLaunchKernelGGL((gemm_f32_kernel<T, true, true>), grid, block, 0, s, p);
  else if (ak) hipLaunchKernelGGL((gemm_f32_kernel<T, true, false>), grid, block, 0, s, p);
  else if (bk) hipLaunchKernelGGL((gemm_f32_kernel<T, false, true>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((gemm_f32_kernel<T, false, false>), grid, block, 0, s, p);
  return check_launch("gemm_f32_kernel");
}

}  // namespace

lc_status gemm_f32_launch(const lc_gemm_args &a, hipStream_t s) {
  if (a.epilogue == LC_EPI_SWIGLU && !a.b_kmajor)
    return fail(LC_ERR_UNSUPPORTED, "gemm fp32: SwiGLU needs k-major B");
  F32P p{};
  p.A = static_cast<const float *>(a.A);
  p.B = static_cast<const float *>(a.B);
  p.C = static_cast<float *>(a.C);
  p.R = static_cast<const float *>(a.R);
  p.aux0 = static_cast<float *>(a.aux0);
  p.aux1 = static_cast<float *>(a.aux1);
  p.rcos = a.rope_cos;
  p.rsin = a.rope_sin;
  p.lda = a.lda;
  p.ldb = a.ldb;
  p.ldc = a.ldc;
  p.ldr = a.ldr;
  p.ld_aux = a.ld_aux;
  p.M = (int)a.M;
  p.N = (int)a.N;
  p.K = (int)a.K;
  p.epi = a.epilogue;
  p.rope_cols = a.rope_cols;
  p.rope_seq = a.rope_seq;
  p.hd = a.head_dim;
  p.vec_a = a.lda % 4 == 0;
  p.vec_b = a.ldb % 4 == 0;
  // 64 x 64 tiles read half the operand bytes per product; 32 x 32 tiles where
  // those would leave a quarter of the compute units or more without one
  const int64_t n = a.epilogue == LC_EPI_SWIGLU ? 2 * a.N : a.N;
  const int64_t tiles64 = ((a.M + 63) / 64) * ((n + 63) / 64);
  const bool ak = a.a_kmajor != 0, bk = a.b_kmajor != 0;
  return tiles64 >= 192 ? run_f32<64>(p, ak, bk, s) : run_f32<32>(p, ak, bk, s);
}

}  // namespace lc

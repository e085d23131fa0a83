// fp32 GEMM path (fp32-compute stages) on the fp32 matrix instruction
// (v_mfma_f32_32x32x2_f32: fp32 products and sums), with the operand layouts and
// epilogues of the bf16 kernels.
//
// These products are small (a tiny stage's outputs are 128 x 128 to 128 x 688),
// so one workgroup's serial chain and the number of launches bound them. Every
// workgroup of four waves owns a 32 x 32 or 64 x 64 output tile and the waves
// split k, so no operand value is read by two waves. The four partial tiles are
// added in wave order through LDS, where RoPE and SwiGLU find the two columns they
// combine (the tile's columns are chosen as such pairs), so each product is one
// launch. (With 64 x 64 tiles staged through LDS by scalar loads, and RoPE and
// SwiGLU as launches of their own, a 128 x 384 x 128 product took 38 us and a
// 400-token d-768 layer's 195 us on average.)
//
// Operands come in through a ring of four LDS stages (LDS-DMA loads of whole cache
// lines, 16 bytes per lane where rows are whole 16-byte runs, else, in 64 tiles, 4;
// three stages ahead, one barrier per stage); else fragments go from global memory
// straight into registers, a step ahead. (Rows read 32 bytes at a time in fragment
// order fill the L1 several times over: the register form took 923 us for two
// microbatches' products of a 400-token d-768 layer, forward and backward, the ring
// 700.)
#include "gemm_common.hpp"

namespace lc {
namespace {

constexpr int NW = 4;    // waves: shares of k (the ring's 32 tile also with 8)
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
  uint32_t a_bytes, b_bytes;  // byte extents (ring kernel)
  unsigned tiles_n;
  unsigned first;  // the launch's first tile
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

typedef __attribute__((address_space(3))) float lds_f;

// The waves' partial tiles added in wave order and the epilogue. `part`: W
// tiles of T rows of T + 1 floats of LDS that no wave reads any more.
template <int T, int W>
__device__ __forceinline__ void finish(const F32P &p, lds_f *part, const f32x16_v (&acc)[T / 32][T / 32], int m0,
                                       int tn, int w, int lane) {
  constexpr int F = T / 32, LD = T + 1;
  const int l32 = lane & 31, h = lane >> 5;
  // lane: column l32 of a block, rows (r & 3) + 8 (r >> 2) + 4 h
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        part[w * T * LD + (32 * i + (r & 3) + 8 * (r >> 2) + 4 * h) * LD + 32 * j + l32] = acc[i][j][r];
  __syncthreads();
  auto sum = [&](int r, int c) {
    float v = part[r * LD + c];
#pragma unroll
    for (int i = 1; i < W; ++i) v += part[i * T * LD + r * LD + c];
    return v;
  };
  const bool pair = p.epi == LC_EPI_SWIGLU || p.epi == LC_EPI_ROPE;
  const int cols = pair ? T / 2 : T;
  const int tid = threadIdx.x, j = tid % cols;
  int n;
  bool ok;
  column<T>(p, tn, j, &n, &ok);
  if (!ok) return;
  // what the epilogue reads for row m, and row r's results from it
  auto load = [&](auto epi, int m, float &x, float &y) {
    constexpr int E = decltype(epi)::value;
    if constexpr (E == LC_EPI_ACCUM_F32) x = p.C[(int64_t)m * p.ldc + n];
    if constexpr (E == LC_EPI_RESIDUAL) x = p.R[(int64_t)m * p.ldr + n];
    if constexpr (E == LC_EPI_SWIGLU_BWD) {
      x = p.aux0[(int64_t)m * p.ld_aux + n];
      y = p.aux1[(int64_t)m * p.ld_aux + n];
    }
    if constexpr (E == LC_EPI_ROPE) {
      if (n < p.rope_cols) {
        const int64_t t = (int64_t)(m % p.rope_seq) * (p.hd / 2) + n % p.hd;
        x = p.rcos[t];
        y = p.rsin[t];
      }
    }
  };
  auto put = [&](auto epi, int r, int m, float x, float y) {
    constexpr int E = decltype(epi)::value;
    const float v = sum(r, j);
    float *c = p.C + (int64_t)m * p.ldc + n;
    if constexpr (E == LC_EPI_ACCUM_F32 || E == LC_EPI_RESIDUAL) {
      *c = x + v;
    } else if constexpr (E == LC_EPI_SWIGLU_BWD) {
      float dg, du;
      swiglu_grad(v, x, y, dg, du);
      c[0] = dg;
      c[p.N] = du;
    } else if constexpr (E == LC_EPI_SWIGLU) {
      const float u = sum(r, j + T / 2);
      p.aux0[(int64_t)m * p.ld_aux + n] = v;
      p.aux1[(int64_t)m * p.ld_aux + n] = u;
      if (p.C) *c = v * sigmoidf_(v) * u;
    } else if constexpr (E == LC_EPI_ROPE) {
      float a = v, b = sum(r, j + T / 2);
      if (n < p.rope_cols) rope_pair(a, b, x, y);
      c[0] = a;
      c[p.hd / 2] = b;
    } else {
      *c = v;
    }
  };
  auto with_epi = [&](auto f) {
    switch (p.epi) {
      case LC_EPI_ACCUM_F32: f(std::integral_constant<int, LC_EPI_ACCUM_F32>{}); break;
      case LC_EPI_RESIDUAL: f(std::integral_constant<int, LC_EPI_RESIDUAL>{}); break;
      case LC_EPI_SWIGLU_BWD: f(std::integral_constant<int, LC_EPI_SWIGLU_BWD>{}); break;
      case LC_EPI_SWIGLU: f(std::integral_constant<int, LC_EPI_SWIGLU>{}); break;
      case LC_EPI_ROPE: f(std::integral_constant<int, LC_EPI_ROPE>{}); break;
      default: f(std::integral_constant<int, LC_EPI_STORE>{});
    }
  };
  const int rs = 64 * W / cols;
  if constexpr (T == 32) {
    for (int r = tid / cols; r < T; r += rs) {
      const int m = m0 + r;
      if (m >= p.M) break;
      with_epi([&](auto epi) {
        float x, y;
        load(epi, m, x, y);
        put(epi, r, m, x, y);
      });
    }
  } else {
    // Eight rows at a time: what the epilogue reads of all is loaded before the first is
    // stored (a row at a time, each waited for its own load: 4096 x 4096 outputs at K = 64
    // accumulated in 99 us, 59 so; a 32 tile has too few rows per thread to gain).
    constexpr int RB = 8;
    with_epi([&](auto epi) {
      for (int r0 = tid / cols; r0 < T && m0 + r0 < p.M; r0 += RB * rs) {
        float x[RB], y[RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) load(epi, min(m0 + min(r0 + i * rs, T - 1), p.M - 1), x[i], y[i]);
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          const int r = r0 + i * rs, m = m0 + r;
          if (r < T && m < p.M) put(epi, r, m, x[i], y[i]);
        }
      }
    });
  }
}

// ------------------------------------------------------------------ ring
// A slice of 32 k of an operand (T rows) in LDS, 32 T floats: T / 8 runs of 1 KiB.
//   k-major: row r is position r / (T / 8) of run r % (T / 8) (128 bytes, eight
//     chunks of four k), chunk c at c ^ swz(r): the 16 rows that one phase of a
//     fragment read takes at one chunk then touch all 64 banks
//   m/n-major: k rows of T floats, one after the other
template <int T, bool KMAJ>
struct Slice {
  static constexpr int RUNS = T / 8, BYTES = RUNS * 1024;
  __device__ __forceinline__ static int swz(int r) { return T == 64 ? r & 7 : (r & 3) + 4 * ((r >> 3) & 1); }
  // this lane's part of run q: first k of the slice, tile row (m/n-major: first of 4)
  __device__ __forceinline__ static void part(int q, int lane, int *k, int *row) {
    if constexpr (KMAJ) {
      *row = (lane >> 3) * RUNS + q;
      *k = 4 * ((lane & 7) ^ swz(*row));
    } else {
      const int f = 256 * q + 4 * lane;  // float of the slice
      *k = f / T;
      *row = f % T;
    }
  }
  // the same of 4-byte loads, of which load i takes a quarter of the run
  __device__ __forceinline__ static void part1(int q, int i, int lane, int *k, int *row) {
    const int f = 64 * i + lane;  // float of the run
    part(q, f >> 2, k, row);
    if constexpr (KMAJ) *k += f & 3;
    else *row += f & 3;
  }
  // x[u] = row 32 f + lane % 32 at k = k0 + 4 (lane / 32) + u, k0 a multiple of 8
  __device__ __forceinline__ static void frag(const lds_t *t, int f, int k0, int lane, float (&x)[4]) {
    const int r = 32 * f + (lane & 31), k = k0 + 4 * (lane >> 5);
    if constexpr (KMAJ) {
      typedef __attribute__((address_space(3))) f32x4_v lds_f4;
      const f32x4_v v = *reinterpret_cast<const lds_f4 *>(t + (r % RUNS) * 1024 + (r / RUNS) * 128 +
                                                          (((k >> 2) ^ swz(r)) << 4));
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = v[u];
    } else {
      const lds_f *s = reinterpret_cast<const lds_f *>(t) + k * T + r;
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = s[u * T];
    }
  }
};

constexpr int NST = 4;  // stages of the ring

// SUB slices per stage; each of the W waves multiplies 8 G k of every stage. Eight
// waves halve a tile's chain of products (two waves per SIMD instead of one; tiny step
// 850 -> 797 us).
template <int T, int W> constexpr int ring_lds() {
  constexpr int part = W * T * (T + 1) * 4, ring = NST * 2 * (64 / T * (W / 4)) * Slice<T, true>::BYTES;
  return ring > part ? ring : part;
}
// E floats per lane and load: 4, or 1 for rows that are not whole 16-byte runs (the
// loads of a wave still cover whole cache lines).
template <int T, int W, int E, bool A_K, bool B_K>
__device__ __forceinline__ void ring_block(F32P p, unsigned wg, lds_t *R0) {
  constexpr int F = T / 32, SUB = 64 / T * (W / 4), KS = 32 * SUB, G = 64 / T;
  constexpr int OPB = Slice<T, true>::BYTES, STAGE = 2 * SUB * OPB;
  constexpr int RPW = 2 * SUB * (T / 8) / W;  // runs per wave and stage: A by the first half of the waves
  constexpr int LPR = 4 / E, LPW = RPW * LPR;  // loads per run, per wave and stage
  static_assert(KS == W * 8 * G && RPW == 4, "");
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = (int)(wg / p.tiles_n) * T, tn = (int)(wg % p.tiles_n);
  const int grp = w / (W / 2), wo = w % (W / 2);
  const i32x4_v rs = grp == 0 ? make_rsrc(p.A, p.a_bytes) : make_rsrc(p.B, p.b_bytes);
  const bool gk = grp == 0 ? A_K : B_K;
  const int64_t ld = grp == 0 ? p.lda : p.ldb;
  const int sub = wo * RPW / (T / 8), q0 = wo * RPW % (T / 8);
  uint32_t vo[LPW];  // byte offsets of this wave's loads in stage 0
  int kl[LPW];       // their k in the stage
#pragma unroll
  for (int t = 0; t < LPW; ++t) {
    int k, r, row;
    bool ok = true;
    if constexpr (E == 4) {
      if (gk) Slice<T, true>::part(q0 + t, lane, &k, &r);
      else Slice<T, false>::part(q0 + t, lane, &k, &r);
    } else {
      if (gk) Slice<T, true>::part1(q0 + t / LPR, t % LPR, lane, &k, &r);
      else Slice<T, false>::part1(q0 + t / LPR, t % LPR, lane, &k, &r);
    }
    if (grp == 0) {
      row = m0 + r;
      ok = row < p.M;
    } else {
      int n;
      row = column<T>(p, tn, r, &n, &ok);
    }
    kl[t] = k + 32 * sub;
    vo[t] = ok ? (uint32_t)((gk ? (int64_t)row * ld + kl[t] : (int64_t)kl[t] * ld + row) * 4) : OOB;
  }
  const uint32_t kbw = gk ? 4u : (uint32_t)(ld * 4);
  lds_t *const dst0 = R0 + (2 * sub + grp) * OPB + q0 * 1024;
  const int ns = (p.K + KS - 1) / KS;
  auto load = [&](int st) {
    lds_t *d = dst0 + (st & (NST - 1)) * STAGE;
    const uint32_t so = (uint32_t)(st * KS) * kbw;
    auto one = [&](int t, uint32_t v, uint32_t sc) {
      if constexpr (E == 4) dma16s(rs, d + t * 1024, v, sc);
      else dma4s(rs, d + t * 256, v, sc);
    };
    if ((st + 1) * KS > p.K) {  // the stage ends past K: every lane checked
#pragma unroll
      for (int t = 0; t < LPW; ++t) one(t, st * KS + kl[t] < p.K && vo[t] != OOB ? vo[t] + so : OOB, 0);
      return;
    }
#pragma unroll
    for (int t = 0; t < LPW; ++t) one(t, vo[t], so);
  };
  f32x16_v acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  // wave w's k of a stage: 8 G w .. + 8 G - 1
  const int ws = 8 * G * w / 32, wk = 8 * G * w % 32;
  auto read = [&](int st, float (&a)[F][G][4], float (&b)[F][G][4]) {
    const lds_t *t = R0 + (st & (NST - 1)) * STAGE + 2 * ws * OPB;
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int g = 0; g < G; ++g) {
        Slice<T, A_K>::frag(t, f, wk + 8 * g, lane, a[f][g]);
        Slice<T, B_K>::frag(t + OPB, f, wk + 8 * g, lane, b[f][g]);
      }
  };
  auto multiply = [&](const float (&a)[F][G][4], const float (&b)[F][G][4]) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
          for (int j = 0; j < F; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][g][u], b[j][g][u], acc[i][j], 0, 0, 0);
  };
  float fa[2][F][G][4], fb[2][F][G][4];
  auto step = [&](int st, float (&a)[F][G][4], float (&b)[F][G][4], float (&an)[F][G][4], float (&bn)[F][G][4]) {
    const int later = ns - 2 - st;  // stages after st + 1, in flight at most two
    if (later >= 2) wait_barrier<2 * LPW>();
    else if (later == 1) wait_barrier<LPW>();
    else wait_barrier<0>();
    if (st + NST < ns) load(st + NST);
    read(st + 1, an, bn);  // (after the last stage: another slot's stale data, unused)
    multiply(a, b);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll 1
  for (int st = 0; st < min(ns, NST); ++st) load(st);
  if (ns >= 4) wait_barrier<3 * LPW>();
  else if (ns == 3) wait_barrier<2 * LPW>();
  else if (ns == 2) wait_barrier<LPW>();
  else wait_barrier<0>();
  read(0, fa[0], fb[0]);
  for (int st = 0; st < ns; st += 2) {
    step(st, fa[0], fb[0], fa[1], fb[1]);
    if (st + 1 < ns) step(st + 1, fa[1], fb[1], fa[0], fb[0]);
  }
  __syncthreads();  // every wave's last fragment reads are done
  finish<T, W>(p, reinterpret_cast<lds_f *>(R0), acc, m0, tn, w, lane);
}

template <int T, int W, int E, bool A_K, bool B_K>
__global__ __launch_bounds__(64 * W) void gemm_f32_ring_kernel(F32P p) {
  __shared__ __align__(16) char ring[ring_lds<T, W>()];
  ring_block<T, W, E, A_K, B_K>(p, p.first + blockIdx.x, LDS_AS(char, ring));
}

// An input gradient's nx tiles and a weight gradient's in one grid: the same bits as
// a launch for each. A tiny step (d 128, 128 tokens, 2 layers, 4 microbatches; 32
// launches fewer) 797 -> 648 us.
__global__ __launch_bounds__(512) void gemm_f32_pair_kernel(F32P x, F32P w, int nx) {
  __shared__ __align__(16) char ring[ring_lds<32, 8>()];
  const unsigned i = blockIdx.x, n = (unsigned)nx;
  if (i < n) ring_block<32, 8, 4, true, false>(x, i, LDS_AS(char, ring));
  else ring_block<32, 8, 4, false, false>(w, i - n, LDS_AS(char, ring));
}

// ------------------------------------------------------------------ thin products
// Many outputs of few k: 64 x 64 outputs per workgroup, 4 x 4 per thread, products in
// the vector unit. Eight small workgroups per compute unit cover each other's loads and
// stores, which is all there is (4096 x 4096 at K = 8: 30 us, 42 through the ring).
template <bool A_K, bool B_K>
__global__ __launch_bounds__(256) void gemm_f32_thin_kernel(F32P p) {
  constexpr int T = 64, TK = 16;
  __shared__ float As[TK][T + 4], Bs[TK][T + 4];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const unsigned wg = p.first + blockIdx.x;
  const int m0 = (int)(wg / p.tiles_n) * T, n0 = (int)(wg % p.tiles_n) * T;
  float acc[4][4] = {};
  auto stage = [&](const float *X, int64_t ld, int row0, int rows, int k0, bool kmaj, float (*S)[T + 4]) {
#pragma unroll
    for (int u = 0; u < T * TK / 256; ++u) {
      const int e = u * 256 + tid, r = kmaj ? e / TK : e % T, k = kmaj ? e % TK : e / T;
      const int gr = row0 + r, gk = k0 + k;
      S[k][r] = gr < rows && gk < p.K ? X[kmaj ? (int64_t)gr * ld + gk : (int64_t)gk * ld + gr] : 0.0f;
    }
  };
  for (int k0 = 0; k0 < p.K; k0 += TK) {
    stage(p.A, p.lda, m0, p.M, k0, A_K, As);
    stage(p.B, p.ldb, n0, p.N, k0, B_K, Bs);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TK; ++k) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[k][ty * 4 + i], b[i] = Bs[k][tx * 4 + i];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= p.M) break;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n >= p.N) break;
      const float v = acc[i][j];
      float *c = p.C + (int64_t)m * p.ldc + n;
      if (p.epi == LC_EPI_ACCUM_F32) *c = *c + v;
      else if (p.epi == LC_EPI_RESIDUAL) *c = p.R[(int64_t)m * p.ldr + n] + v;
      else *c = v;
    }
  }
}

// ------------------------------------------------------------------ registers
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
  __shared__ float part[NW * T * (T + 1)];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const unsigned wg = p.first + blockIdx.x;
  const int m0 = (int)(wg / p.tiles_n) * T, tn = (int)(wg % p.tiles_n);
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
  finish<T, NW>(p, LDS_AS(float, part), acc, m0, tn, w, lane);
}

// silu(gate) * up from the stored gate and up (SwiGLU's C in a launch of its own)
__global__ __launch_bounds__(256) void swiglu_act_f32_kernel(F32P p) {
  const int64_t n = (int64_t)p.M * p.N;
  for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t m = i / p.N, c = i % p.N;
    const float g = p.aux0[m * p.ld_aux + c];
    p.C[m * p.ldc + c] = g * sigmoidf_(g) * p.aux1[m * p.ld_aux + c];
  }
}

enum Path { RING4, RING1, REGISTERS, THIN };

template <int T>
lc_status run_f32(F32P p, bool ak, bool bk, Path path, hipStream_t s) {
  const int cols = p.epi == LC_EPI_SWIGLU ? T / 2 : T;
  const int64_t tm = ((int64_t)p.M + T - 1) / T, tn = ((int64_t)p.N + cols - 1) / cols;
  if (tm * tn > UINT32_MAX) return fail(LC_ERR_UNSUPPORTED, "gemm fp32: output too large");
  p.tiles_n = (unsigned)tn;
  auto run_ring = [&](auto w, auto e) {
    constexpr int W = decltype(w)::value, E = decltype(e)::value;
    launch_parts((uint32_t)(tm * tn), [&](uint32_t first, uint32_t count) {
      p.first = first;
      const dim3 grid(count), block(64 * W);
      if (ak && bk) hipLaunchKernelGGL((gemm_f32_ring_kernel<T, W, E, true, true>), grid, block, 0, s, p);
      else if (ak) hipLaunchKernelGGL((gemm_f32_ring_kernel<T, W, E, true, false>), grid, block, 0, s, p);
      else if (bk) hipLaunchKernelGGL((gemm_f32_ring_kernel<T, W, E, false, true>), grid, block, 0, s, p);
      else hipLaunchKernelGGL((gemm_f32_ring_kernel<T, W, E, false, false>), grid, block, 0, s, p);
    });
    return check_launch("gemm_f32_ring_kernel");
  };
  // (eight waves' stages take a compute unit's LDS for one workgroup)
  if (path == RING4 && T == 32 && tm * tn <= 256)
    return run_ring(std::integral_constant<int, T == 32 ? 8 : 4>{}, std::integral_constant<int, 4>{});
  if (path == RING4) return run_ring(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
  if (path == RING1)  // (64 tiles only)
    return run_ring(std::integral_constant<int, 4>{}, std::integral_constant<int, T == 64 ? 1 : 4>{});
  launch_parts((uint32_t)(tm * tn), [&](uint32_t first, uint32_t count) {
    p.first = first;
    const dim3 grid(count), block(64 * NW);
    if (ak && bk) hipLaunchKernelGGL((gemm_f32_kernel<T, true, true>), grid, block, 0, s, p);
    else if (ak) hipLaunchKernelGGL((gemm_f32_kernel<T, true, false>), grid, block, 0, s, p);
    else if (bk) hipLaunchKernelGGL((gemm_f32_kernel<T, false, true>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((gemm_f32_kernel<T, false, false>), grid, block, 0, s, p);
  });
  return check_launch("gemm_f32_kernel");
}

}  // namespace

namespace {

struct Plan {
  F32P p;
  Path path;
  bool big;  // 64 x 64 tiles
  int64_t tiles32, tiles64;
  int64_t a_ext, b_ext;  // the operands' bytes from first to last element
};

Plan plan_of(const lc_gemm_args &a) {
  Plan r{};
  F32P &p = r.p;
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
  const int64_t n = a.epilogue == LC_EPI_SWIGLU ? 2 * a.N : a.N;
  r.tiles64 = ((a.M + 63) / 64) * ((n + 63) / 64);
  r.tiles32 = ((a.M + 31) / 32) * ((n + 31) / 32);
  const bool ak = a.a_kmajor != 0, bk = a.b_kmajor != 0;
  const int64_t brows = a.epilogue == LC_EPI_SWIGLU ? 2 * a.N : a.N;
  const int64_t ae = 4 * (ak ? (a.M - 1) * a.lda + a.K : (a.K - 1) * a.lda + a.M);
  const int64_t be = 4 * (bk ? (brows - 1) * a.ldb + a.K : (a.K - 1) * a.ldb + brows);
  // 64 x 64 tiles read half the operand bytes per product; 32 x 32 tiles where
  // those would leave a quarter of the compute units or more without one
  r.big = r.tiles64 >= 192;
  // The ring takes 16 bytes per lane and load where both operands' rows are whole 16-byte
  // runs of which none is part inside (a part past K would not be zero), else 4 bytes; its
  // offsets are 32-bit. (us: ring | registers | thin, NT)
  const bool runs = p.vec_a && p.vec_b && (!(ak || bk) || a.K % 4 == 0) && (ak || a.M % 4 == 0) &&
                    (bk || (a.N % 4 == 0 && a.epilogue != LC_EPI_ROPE));
  r.path = runs ? RING4 : RING1;
  if (ae >= (int64_t)OOB || be >= (int64_t)OOB) {
    r.path = REGISTERS;
  } else if (r.big) {
    // With few k the vector unit is faster than the ring's fill and the waves' merge:
    // 16-byte loads at 4096 x 4096: K = 16 42 | - | 30, K = 48 50 | - | 42, K = 64 50 | - |
    // 49; 2000 x 2000 at K = 48 15 | - | 15; at 400 x 2304, K = 16 5.7 | - | 5.2 but 6.2 | - |
    // 7.9 accumulating. 4-byte loads: 4096 x 4096, K = 33 60 | 100 | 41, K = 65 71 | 105 | 54,
    // K = 129 92 | 179 | 82 (90 | 155 | 91 accumulating); 1024 x 1024, K = 1 6.7 | 7.5 | 5.0,
    // K = 33 7.5 | 7.7 | 7.6.
    const bool many = r.tiles64 >= 1024;
    const int thin = runs ? (many ? 48 : 0) : many ? 80 : 32;
    const bool plain = a.epilogue == LC_EPI_STORE || a.epilogue == LC_EPI_STORE_F32 ||
                       a.epilogue == LC_EPI_ACCUM_F32 || a.epilogue == LC_EPI_RESIDUAL;
    if (a.K <= thin && plain) r.path = THIN;
    // one 64 tile per compute unit: no second workgroup covers the 4-byte loads' latency (400
    // x 2304, K = 65 8.4 | 7.9, K = 129 10.1 | 12.8)
    else if (!runs && r.tiles64 <= 256 && a.K <= 128) r.path = REGISTERS;
  } else if (!runs || (r.tiles32 > 256 && a.K <= 32)) {
    // Small grids: 4-byte loads in the ring lose to registers up to K = 128 (257 where an
    // operand is m/n-major). 236 x 2860 by 16 bytes: K = 16 6.6 | 5.1, K = 32 6.6 | 4.5. (Up to
    // 256 tiles the ring has eight waves: 512 x 512 at K = 16 4.0 | 3.9, and the pair launch.)
    r.path = REGISTERS;
  }
  p.a_bytes = (uint32_t)ae;
  p.b_bytes = (uint32_t)be;
  r.a_ext = ae;
  r.b_ext = be;
  return r;
}

}  // namespace

lc_status gemm_f32_launch(const lc_gemm_args &a, hipStream_t s) {
  if (a.epilogue == LC_EPI_SWIGLU && !a.b_kmajor)
    return fail(LC_ERR_UNSUPPORTED, "gemm fp32: SwiGLU needs k-major B");
  Plan r = plan_of(a);
  if (r.path == THIN) {
    const int64_t tn = (a.N + 63) / 64;
    if (r.tiles64 > UINT32_MAX) return fail(LC_ERR_UNSUPPORTED, "gemm fp32: output too large");
    r.p.tiles_n = (unsigned)tn;
    launch_parts((uint32_t)r.tiles64, [&](uint32_t first, uint32_t count) {
      r.p.first = first;
      const dim3 grid(count), block(256);
      if (a.a_kmajor && a.b_kmajor) hipLaunchKernelGGL((gemm_f32_thin_kernel<true, true>), grid, block, 0, s, r.p);
      else if (a.a_kmajor) hipLaunchKernelGGL((gemm_f32_thin_kernel<true, false>), grid, block, 0, s, r.p);
      else if (a.b_kmajor) hipLaunchKernelGGL((gemm_f32_thin_kernel<false, true>), grid, block, 0, s, r.p);
      else hipLaunchKernelGGL((gemm_f32_thin_kernel<false, false>), grid, block, 0, s, r.p);
    });
    return check_launch("gemm_f32_thin_kernel");
  }
  // A C over A or B (the gate and up are stored elsewhere, so a caller may reuse the
  // memory): written once every workgroup is done reading
  const char *c0 = static_cast<const char *>(a.C), *c1 = c0 + 4 * ((a.M - 1) * a.ldc + a.N);
  auto over = [&](const void *x, int64_t bytes) {
    return c0 < static_cast<const char *>(x) + bytes && static_cast<const char *>(x) < c1;
  };
  const bool later = a.epilogue == LC_EPI_SWIGLU && (over(a.A, r.a_ext) || over(a.B, r.b_ext));
  if (later) r.p.C = nullptr;
  const bool ak = a.a_kmajor != 0, bk = a.b_kmajor != 0;
  LC_TRY(r.big ? run_f32<64>(r.p, ak, bk, r.path, s) : run_f32<32>(r.p, ak, bk, r.path, s));
  if (!later) return LC_OK;
  r.p.C = static_cast<float *>(a.C);
  const unsigned blocks = (unsigned)std::min<int64_t>((a.M * a.N + 255) / 256, 65535);
  hipLaunchKernelGGL(swiglu_act_f32_kernel, dim3(blocks), dim3(256), 0, s, r.p);
  return check_launch("swiglu_act_f32_kernel");
}

lc_status gemm_f32_pair_launch(const lc_gemm_args &x, const lc_gemm_args &w, hipStream_t s, bool *done) {
  Plan a = plan_of(x), b = plan_of(w);
  *done = false;
  if (a.path != RING4 || b.path != RING4 || a.big || b.big || a.tiles32 > 256 || b.tiles32 > 256)
    return LC_OK;
  a.p.tiles_n = (unsigned)((x.N + 31) / 32);
  b.p.tiles_n = (unsigned)((w.N + 31) / 32);
  hipLaunchKernelGGL(gemm_f32_pair_kernel, dim3((unsigned)(a.tiles32 + b.tiles32)), dim3(512), 0, s, a.p, b.p,
                     (int)a.tiles32);
  *done = true;
  return check_launch("gemm_f32_pair_kernel");
}

}  // namespace lc

// Causal attention of the fp32 path on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: fp32 products and sums throughout). Any sequence
// length, even head_dim <= 128, grouped-query attention, deterministic.
//
// These stages are small, so what bounds a kernel is one workgroup's serial
// chain: a workgroup owns 16 queries (or keys) of one head and its four waves
// split the visible blocks of 32 keys (queries) between them, each with its own
// running maximum, sum and accumulators, merged through LDS in wave order at the
// end. (One thread per query with its output row in scratch memory, as before,
// took 2698 + 3166 + 4643 us for forward, dQ and dK/dV of 24 heads of 200
// tokens, head_dim 64.) Operands are read straight from global memory (L1/L2) in
// fragment order: with 16 queries per pass over K and V the loads are far from
// the L2's rate.
//
// Fragments (lane l, group g = l / 16): a score product takes A[row l % 16][k
// slot g] and B[k slot g][column l % 16]. Its k slots may stand for any features
// as long as both operands agree: product (j, c) uses feature 16 j + 4 g + c, so
// that a lane's values are 16-byte runs. The scores come out with the column
// (query in forward and dQ, key in dK/dV) on the lane and rows 4 g + r in
// register r, which is the B operand of the second product with k slot g standing
// for row 4 g + r: no data moves between the two. Its rows stand for features NI
// (l % 16) + i of product i, so that a lane's loads and its outputs (features 4 NI
// g + NI r + i) are runs too.
//
// Many sequences of up to 8 tokens share workgroups, as many as fit 16 rows: with one
// each, most rows of every product are padding (65,536 sequences of one token, 8 heads,
// head_dim 16: forward 1105 us, 84 packed; one thread per query took 133). A pair of
// different sequences is masked like a key after its query.
//
// A masked pair has weight 0, but 0 times an infinite or NaN value would be NaN:
// in blocks that hold masked pairs the values are looked at, and if one is not
// finite the block's second product is formed pair by pair instead.
#include "common.hpp"

#include <math.h>

namespace lc {
namespace {

struct AttnF {
  const float *q, *k, *v;
  float *o;
  float *lse;
  const float *dout;
  float *dq, *dk, *dv;
  float *D;
  const float *rcos, *rsin;
  int64_t ld_qkv, ld_o, ld_d;
  int B, S, H, hd;
  int pack, npack;  // sequences per block of rows (1: blocks of one sequence), groups of them
  int Hkv, G;  // key/value heads; query heads per key/value head
  float scale;
  int first;           // the launch's first workgroup
  int vec_qkv, vec_o;  // rows are made of whole 16-byte runs (q, k, v; o, dout)
};

constexpr int QR = 16;  // queries (keys) per workgroup
constexpr int KB = 32;  // keys (queries) per block
constexpr int NW = 4;   // waves
constexpr int NTF = 64 * NW;

__device__ __forceinline__ f32x4_v mfma4(float a, float b, f32x4_v c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// x[i] = row[e0 + i], 0 at or past hd (i < n, n a power of two, e0 a multiple of n)
template <int N>
__device__ __forceinline__ void load_run(const float *row, int e0, int hd, bool vec, float (&x)[N]) {
  if constexpr (N >= 4) {
    if (vec) {  // hd, e0 multiples of 4: a run of four is inside the row or past it
#pragma unroll
      for (int i = 0; i < N; i += 4) {
        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (e0 + i < hd) v = *reinterpret_cast<const float4 *>(row + e0 + i);
        x[i] = v.x; x[i + 1] = v.y; x[i + 2] = v.z; x[i + 3] = v.w;
      }
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = e0 + i < hd ? row[e0 + i] : 0.0f;
}

// the lane's score-product fragment of a row: features 16 j + 4 g + c
template <int NI>
__device__ __forceinline__ void load_frag(const float *row, int g, int hd, bool vec, float (&x)[NI][4]) {
#pragma unroll
  for (int j = 0; j < NI; ++j) load_run<4>(row, 16 * j + 4 * g, hd, vec, x[j]);
}

template <int NI>
__device__ __forceinline__ f32x4_v score(const float (&a)[NI][4], const float (&b)[NI][4]) {
  f32x4_v s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int j = 0; j < NI; ++j)
#pragma unroll
    for (int c = 0; c < 4; ++c) s = mfma4(a[j][c], b[j][c], s);
  return s;
}

// sum (max) over the four lanes of a column
__device__ __forceinline__ float col_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}
__device__ __forceinline__ float col_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return fmaxf(x, __shfl_xor(x, 32, 64));
}

// acc[e][column] += sum over the block's rows of w[row][column] X[row][e], the
// rows at r0 .. r0 + 31 (X rows x0 + row, at most last). `masked`: some pair of
// the block is masked; vis(row) says whether this lane's column sees a row.
template <int NI, typename F>
__device__ __forceinline__ void accumulate(f32x4_v (&acc)[NI], const f32x4_v (&w)[2], const float *x0,
                                           int64_t ld, int r0, int last, int hd, bool vec, int lane,
                                           bool masked, F vis) {
  const int g = lane >> 4, c = lane & 15;
  float x[2][4][NI];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      load_run<NI>(x0 + (int64_t)min(r0 + 16 * t + 4 * g + r, last) * ld, NI * c, hd, vec, x[t][r]);
  if (masked) {
    bool bad = false;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < NI; ++i) bad |= !(fabsf(x[t][r][i]) < INFINITY);
    if (__any(bad)) {
#pragma unroll 1
      for (int n = 0; n < 32; ++n) {
        const int row = r0 + n, t = n >> 4, r = n & 3;
        float mine = 0.0f;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (u == t && e == r) mine = w[u][e];
        const float wv = __shfl(mine, c + 16 * ((n >> 2) & 3), 64);
        if (row > last || !vis(row)) continue;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int f = NI * (4 * g + e) + i;
            if (f < hd) acc[i][e] += wv * x0[(int64_t)row * ld + f];
          }
      }
      return;
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int i = 0; i < NI; ++i) acc[i] = mfma4(x[t][r][i], w[t][r], acc[i]);
}

// The waves' accumulators in LDS: feature e of column c of wave w at (w 16 + c) LD + e
template <int NI>
struct Merge {
  static constexpr int LD = 16 * NI + 4;
  static constexpr int FLOATS = NW * QR * LD;
  __device__ __forceinline__ static void put(float *s, const f32x4_v (&acc)[NI], int w, int lane) {
    float *row = s + (w * QR + (lane & 15)) * LD + 4 * NI * (lane >> 4);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < NI; ++i) row[NI * e + i] = acc[i][e];
  }
  __device__ __forceinline__ static float sum(const float *s, int c, int e) {
    float t = s[c * LD + e];
#pragma unroll
    for (int w = 1; w < NW; ++w) t += s[(w * QR + c) * LD + e];
    return t;
  }
};

// The rows that block `b` of sequences holds (a multiple of S, the last one's fewer)
template <bool PACK>
__device__ __forceinline__ int rows_of(const AttnF &p, int b) {
  return PACK ? min(p.pack, p.B - b * p.pack) * p.S : p.S;
}
// first row of row i's sequence
template <bool PACK>
__device__ __forceinline__ int first_of(const AttnF &p, int i) { return PACK ? i - i % p.S : 0; }
// where row i's lse and D are
template <bool PACK>
__device__ __forceinline__ int64_t stat_of(const AttnF &p, int b, int h, int i) {
  if constexpr (PACK) return ((int64_t)(b * p.pack + i / p.S) * p.H + h) * p.S + i % p.S;
  else return ((int64_t)b * p.H + h) * p.S + i;
}

// Block, head and batch row of a workgroup: the heaviest blocks (most queries
// or keys to visit) first, heads fastest
template <bool PACK>
__device__ __forceinline__ void place(const AttnF &p, int heads, bool last_first, int &blk, int &h, int &b) {
  const int nblk = PACK ? 1 : (p.S + QR - 1) / QR;
  const int nbh = heads * p.npack, i = p.first + (int)blockIdx.x;
  const int at = i / nbh;
  blk = last_first ? nblk - 1 - at : at;
  h = (i % nbh) % heads;
  b = (i % nbh) / heads;
}

template <int NI, bool PACK>
__global__ __launch_bounds__(NTF) void attn_f32_fwd_kernel(AttnF p) {
  __shared__ __align__(16) float so[Merge<NI>::FLOATS];
  __shared__ float sm[NW][QR], sl[NW][QR], sf[NW + 1][QR];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  int qb, h, b;
  place<PACK>(p, p.H, true, qb, h, b);
  const int64_t r0 = (int64_t)b * (PACK ? p.pack * p.S : p.S);
  const int rows = rows_of<PACK>(p, b);
  const int q0 = qb * QR, qi = q0 + c, kvh = h / p.G, first = first_of<PACK>(p, qi);
  const float *K = p.k + r0 * p.ld_qkv + (int64_t)kvh * p.hd, *V = p.v + r0 * p.ld_qkv + (int64_t)kvh * p.hd;
  float qf[NI][4];
  load_frag<NI>(p.q + (r0 + min(qi, rows - 1)) * p.ld_qkv + (int64_t)h * p.hd, g, p.hd, p.vec_qkv, qf);
  f32x4_v o[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) o[i] = f32x4_v{0.0f, 0.0f, 0.0f, 0.0f};
  float m = -INFINITY, l = 0.0f;
  auto vis = [&](int key) { return key <= qi && key >= first; };
  const int lastq = min(q0 + QR, rows) - 1;
  for (int k0 = w * KB; k0 <= lastq; k0 += NW * KB) {
    f32x4_v s[2];
    const bool masked = k0 + KB - 1 > q0;
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      float kf[NI][4];
      load_frag<NI>(K + (int64_t)min(k0 + 16 * t + c, rows - 1) * p.ld_qkv, g, p.hd, p.vec_qkv, kf);
      s[t] = score<NI>(kf, qf);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[t][r] = vis(k0 + 16 * t + 4 * g + r) ? s[t][r] * p.scale : -INFINITY;
        mx = fmaxf(mx, s[t][r]);
      }
    }
    const float mn = fmaxf(m, col_max(mx));
    const float mu = mn == -INFINITY ? 0.0f : mn;  // nothing seen yet: weights of 0
    const float alpha = expf(m - mu);
#pragma unroll
    for (int i = 0; i < NI; ++i) o[i] *= alpha;
    l *= alpha;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[t][r] = expf(s[t][r] - mu);
        l += s[t][r];
      }
    m = mn;
    accumulate<NI>(o, s, V, p.ld_qkv, k0, rows - 1, p.hd, p.vec_qkv, lane, masked, vis);
  }
  l = col_sum(l);
  Merge<NI>::put(so, o, w, lane);
  if (g == 0) {
    sm[w][c] = m;
    sl[w][c] = l;
  }
  __syncthreads();
  if (tid < QR) {  // weights of the waves' shares of query q0 + tid
    float mm = sm[0][tid];
#pragma unroll
    for (int i = 1; i < NW; ++i) mm = fmaxf(mm, sm[i][tid]);
    const float mu = mm == -INFINITY ? 0.0f : mm;
    float L = 0.0f;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      sf[i][tid] = expf(sm[i][tid] - mu);
      L += sf[i][tid] * sl[i][tid];
    }
    sf[NW][tid] = L;
    if (q0 + tid < rows) p.lse[stat_of<PACK>(p, b, h, q0 + tid)] = mm + logf(L);
  }
  __syncthreads();
  for (int x = tid; x < QR * p.hd; x += NTF) {
    const int qr = x / p.hd, e = x % p.hd;
    if (q0 + qr >= rows) break;
    float v = 0.0f;
#pragma unroll
    for (int i = 0; i < NW; ++i) v += sf[i][qr] * so[(i * QR + qr) * Merge<NI>::LD + e];
    p.o[(r0 + q0 + qr) * p.ld_o + (int64_t)h * p.hd + e] = v / sf[NW][qr];
  }
}

// writes 16 rows x hd of merged sums times mul at row, rotated back by -angle
// when the RoPE tables are given (row i at position i of its sequence), rows i0 .. of
// the block's `rows`
template <int NI, bool PACK>
__device__ __forceinline__ void store_rotated(const AttnF &p, const float *s, float *dst, int64_t row0, int head,
                                              int i0, int rows, float mul) {
  const int half = p.hd / 2;
  for (int x = threadIdx.x; x < QR * half; x += NTF) {
    const int r = x / half, e = x % half, i = i0 + r, pos = i - first_of<PACK>(p, i);
    if (i >= rows) break;
    float a = Merge<NI>::sum(s, r, e) * mul, bb = Merge<NI>::sum(s, r, e + half) * mul;
    if (p.rcos) {
      const float cs = p.rcos[(int64_t)pos * half + e], sn = p.rsin[(int64_t)pos * half + e];
      const float t = a * cs + bb * sn;
      bb = bb * cs - a * sn;
      a = t;
    }
    float *d = dst + (row0 + i) * p.ld_d + (int64_t)head * p.hd + e;
    d[0] = a;
    d[half] = bb;
  }
}

// per 16 queries: D (written for the dK/dV kernel) and dQ
template <int NI, bool PACK>
__global__ __launch_bounds__(NTF) void attn_f32_dq_kernel(AttnF p) {
  __shared__ __align__(16) float sq[Merge<NI>::FLOATS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  int qb, h, b;
  place<PACK>(p, p.H, true, qb, h, b);
  const int64_t r0 = (int64_t)b * (PACK ? p.pack * p.S : p.S);
  const int rows = rows_of<PACK>(p, b);
  const int q0 = qb * QR, qi = q0 + c, qc = min(qi, rows - 1), kvh = h / p.G, first = first_of<PACK>(p, qi);
  auto vis = [&](int key) { return key <= qi && key >= first; };
  const float *K = p.k + r0 * p.ld_qkv + (int64_t)kvh * p.hd, *V = p.v + r0 * p.ld_qkv + (int64_t)kvh * p.hd;
  float qf[NI][4], df[NI][4];
  load_frag<NI>(p.q + (r0 + qc) * p.ld_qkv + (int64_t)h * p.hd, g, p.hd, p.vec_qkv, qf);
  load_frag<NI>(p.dout + (r0 + qc) * p.ld_o + (int64_t)h * p.hd, g, p.hd, p.vec_o, df);
  float Dq = 0.0f;
  {
    float of[NI][4];
    load_frag<NI>(p.o + (r0 + qc) * p.ld_o + (int64_t)h * p.hd, g, p.hd, p.vec_o, of);
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) Dq += df[j][e] * of[j][e];
  }
  Dq = col_sum(Dq);
  const int64_t si = stat_of<PACK>(p, b, h, qc);
  const float L = p.lse[si];
  if (w == 0 && g == 0 && qi < rows) p.D[si] = Dq;
  f32x4_v acc[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) acc[i] = f32x4_v{0.0f, 0.0f, 0.0f, 0.0f};
  const int lastq = min(q0 + QR, rows) - 1;
  for (int k0 = w * KB; k0 <= lastq; k0 += NW * KB) {
    f32x4_v ds[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      float kf[NI][4], vf[NI][4];
      const int64_t kr = (int64_t)min(k0 + 16 * t + c, rows - 1) * p.ld_qkv;
      load_frag<NI>(K + kr, g, p.hd, p.vec_qkv, kf);
      load_frag<NI>(V + kr, g, p.hd, p.vec_qkv, vf);
      const f32x4_v s = score<NI>(kf, qf), dp = score<NI>(vf, df);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        ds[t][r] = vis(k0 + 16 * t + 4 * g + r) ? expf(s[r] * p.scale - L) * (dp[r] - Dq) : 0.0f;
    }
    accumulate<NI>(acc, ds, K, p.ld_qkv, k0, rows - 1, p.hd, p.vec_qkv, lane, k0 + KB - 1 > q0, vis);
  }
  Merge<NI>::put(sq, acc, w, lane);
  __syncthreads();
  store_rotated<NI, PACK>(p, sq, p.dq, r0, h, q0, rows, p.scale);
}

// per 16 keys and key/value head: dK, dV summed over the head's query heads
// (needs D from the kernel above)
template <int NI, bool PACK>
__global__ __launch_bounds__(NTF) void attn_f32_dkdv_kernel(AttnF p) {
  __shared__ __align__(16) float sk[Merge<NI>::FLOATS], sv[Merge<NI>::FLOATS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  int kb, kvh, b;
  place<PACK>(p, p.Hkv, false, kb, kvh, b);
  const int64_t r0 = (int64_t)b * (PACK ? p.pack * p.S : p.S);
  const int rows = rows_of<PACK>(p, b);
  const int k0 = kb * QR, kj = k0 + c;
  const int end = PACK ? min(rows, first_of<PACK>(p, kj) + p.S) : rows;  // past the last query that sees the key
  const int64_t kr = (r0 + min(kj, rows - 1)) * p.ld_qkv + (int64_t)kvh * p.hd;
  float kf[NI][4], vf[NI][4];
  load_frag<NI>(p.k + kr, g, p.hd, p.vec_qkv, kf);
  load_frag<NI>(p.v + kr, g, p.hd, p.vec_qkv, vf);
  f32x4_v dk[NI], dv[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) dk[i] = dv[i] = f32x4_v{0.0f, 0.0f, 0.0f, 0.0f};
  // units: (query head of the group, block of 32 queries that reach the keys)
  const int qb0 = k0 / KB, nqb = (rows + KB - 1) / KB - qb0;
  for (int u = w; u < p.G * nqb; u += NW) {
    const int h = kvh * p.G + u / nqb, q0 = (qb0 + u % nqb) * KB;
    const float *Q = p.q + r0 * p.ld_qkv + (int64_t)h * p.hd, *dO = p.dout + r0 * p.ld_o + (int64_t)h * p.hd;
    const int64_t si = stat_of<false>(p, b, h, 0);
    f32x4_v pr[2], ds[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      float qf[NI][4], df[NI][4];
      const int64_t qr = min(q0 + 16 * t + c, rows - 1);
      load_frag<NI>(Q + qr * p.ld_qkv, g, p.hd, p.vec_qkv, qf);
      load_frag<NI>(dO + qr * p.ld_o, g, p.hd, p.vec_o, df);
      const f32x4_v s = score<NI>(qf, kf), dp = score<NI>(df, vf);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int qi = q0 + 16 * t + 4 * g + r;
        const int64_t sq = PACK ? stat_of<PACK>(p, b, h, min(qi, rows - 1)) : si + min(qi, rows - 1);
        const bool on = qi >= kj && qi < end;
        const float P = expf(s[r] * p.scale - p.lse[sq]);
        pr[t][r] = on ? P : 0.0f;
        ds[t][r] = on ? P * (dp[r] - p.D[sq]) : 0.0f;
      }
    }
    const bool masked = q0 < k0 + QR - 1 || q0 + KB > rows;
    auto vis = [&](int qi) { return qi >= kj && (!PACK || qi < end); };
    accumulate<NI>(dv, pr, dO, p.ld_o, q0, rows - 1, p.hd, p.vec_o, lane, masked, vis);
    accumulate<NI>(dk, ds, Q, p.ld_qkv, q0, rows - 1, p.hd, p.vec_qkv, lane, masked, vis);
  }
  Merge<NI>::put(sk, dk, w, lane);
  Merge<NI>::put(sv, dv, w, lane);
  __syncthreads();
  store_rotated<NI, PACK>(p, sk, p.dk, r0, kvh, k0, rows, p.scale);
  for (int x = tid; x < QR * p.hd; x += NTF) {
    const int r = x / p.hd, e = x % p.hd;
    if (k0 + r >= rows) break;
    p.dv[(r0 + k0 + r) * p.ld_d + (int64_t)kvh * p.hd + e] = Merge<NI>::sum(sv, r, e);
  }
}

AttnF f32_params(const lc_attn_args &a) {
  AttnF p{};
  p.q = static_cast<const float *>(a.q);
  p.k = static_cast<const float *>(a.k);
  p.v = static_cast<const float *>(a.v);
  p.o = static_cast<float *>(a.o);
  p.lse = a.lse;
  p.dout = static_cast<const float *>(a.dout);
  p.dq = static_cast<float *>(a.dq);
  p.dk = static_cast<float *>(a.dk);
  p.dv = static_cast<float *>(a.dv);
  p.D = static_cast<float *>(a.scratch);
  p.rcos = a.rope_cos;
  p.rsin = a.rope_sin;
  p.ld_qkv = a.ld_qkv;
  p.ld_o = a.ld_o;
  p.ld_d = a.ld_dqkv;
  p.B = a.B; p.S = a.S; p.H = a.H; p.hd = a.hd;
  // packed above 8 workgroups per compute unit (288 sequences of 1 to 8 tokens, 8 heads:
  // 7.9 -> 4.4 to 5.9 us); fewer blocks run side by side anyway, and a packed one costs a
  // few divisions more (128 sequences of 8: backward 10.5 us, 11.3 packed)
  const int64_t blocks = (int64_t)a.B * a.H;
  p.pack = a.S <= QR / 2 && blocks > 2048 ? QR / a.S : 1;
  p.npack = (a.B - 1) / p.pack + 1;
  p.Hkv = a.Hkv > 0 ? a.Hkv : a.H;
  p.G = a.H / p.Hkv;
  p.scale = 1.0f / sqrtf((float)a.hd);
  // (the tensors' pointers are 16-byte aligned)
  p.vec_qkv = a.hd % 4 == 0 && a.ld_qkv % 4 == 0;
  p.vec_o = a.hd % 4 == 0 && a.ld_o % 4 == 0;
  return p;
}

// calls f with NI (16-feature blocks, a power of two) for head_dim hd <= 128 and
// whether sequences are packed
template <typename F>
void with_blocks(const AttnF &p, F f) {
  auto g = [&](auto pack) {
    if (p.hd <= 16) f(std::integral_constant<int, 1>{}, pack);
    else if (p.hd <= 32) f(std::integral_constant<int, 2>{}, pack);
    else if (p.hd <= 64) f(std::integral_constant<int, 4>{}, pack);
    else f(std::integral_constant<int, 8>{}, pack);
  };
  if (p.pack > 1) g(std::true_type{});
  else g(std::false_type{});
}

// Launches f(params, grid) with one workgroup per block of 16 rows (or pack of
// sequences), head and batch row
template <typename F>
lc_status run(const AttnF &p, int heads, const char *what, F f) {
  const int64_t n = (int64_t)((p.S + QR - 1) / QR) * heads * p.npack;
  if (n > INT32_MAX) return fail(LC_ERR_UNSUPPORTED, "attention fp32: 2^31 or more blocks of rows");
  launch_parts((uint32_t)n, [&](uint32_t first, uint32_t count) {
    AttnF q = p;
    q.first = (int)first;
    f(q, dim3(count));
  });
  return check_launch(what);
}

}  // namespace

lc_status attn_f32_fwd_launch(const lc_attn_args &a, hipStream_t s) {
  const AttnF p = f32_params(a);
  return run(p, p.H, "attn_f32_fwd_kernel", [&](const AttnF &q, dim3 grid) {
    with_blocks(p, [&](auto ni, auto pack) {
      hipLaunchKernelGGL((attn_f32_fwd_kernel<decltype(ni)::value, decltype(pack)::value>), grid, dim3(NTF), 0, s, q);
    });
  });
}

lc_status attn_f32_bwd_launch(const lc_attn_args &a, hipStream_t s) {
  const AttnF p = f32_params(a);
  LC_TRY(run(p, p.H, "attn_f32_dq_kernel", [&](const AttnF &q, dim3 grid) {
    with_blocks(p, [&](auto ni, auto pack) {
      hipLaunchKernelGGL((attn_f32_dq_kernel<decltype(ni)::value, decltype(pack)::value>), grid, dim3(NTF), 0, s, q);
    });
  }));
  return run(p, p.Hkv, "attn_f32_dkdv_kernel", [&](const AttnF &q, dim3 grid) {
    with_blocks(p, [&](auto ni, auto pack) {
      hipLaunchKernelGGL((attn_f32_dkdv_kernel<decltype(ni)::value, decltype(pack)::value>), grid, dim3(NTF), 0, s, q);
    });
  });
}

}  // namespace lc

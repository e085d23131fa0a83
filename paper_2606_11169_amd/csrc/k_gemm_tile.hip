// bf16 GEMM with 128 x 128, 64 x 64 or 32 x 32 output tiles: the products whose grid of
// 256 x 256 tiles (k_gemm.hip) would leave most of the 256 compute units idle.
// Same operands, layouts, epilogues and per-element arithmetic.
//
// What bounds such a product is not the matrix cores but the serial chain of
// one tile: with few tiles per compute unit there is no second workgroup to
// cover a stage's load latency. So k is split inside the workgroup as well:
// every wave owns a block of the tile for its own k-steps of each stage (the 128
// tile: 8 waves = 2 x 2 blocks of 64 x 64 x 2 k-steps of a 64-deep stage; the 64
// and 32 tiles: 4 waves, the whole tile each, one k-step of a 128-deep or two of a
// 256-deep stage). That halves (quarters) the chain, reads no operand row of the
// smaller tiles twice from LDS, and keeps both (one) waves of a SIMD busy; the
// waves' partial tiles are added in k-step order in the epilogue, through LDS. (At
// 2048 x 2048 x 11264 the 128 tile runs at 1040 TFLOP/s with one tile per compute
// unit; 64 tiles of 256 x 256 at 473. The 64 tile takes 9 us for a 256 x 512 x 1408
// product, the 256 tile 31; the 32 tile, with four times the compute units loading,
// 6.) Operands stream HBM->LDS through a ring of four stages, three stages ahead of
// the one being multiplied (the 256 tile's two 64 KiB stages leave no room for that;
// here a stage is 32 KiB), one barrier per stage, the next stage's fragments read
// while one multiplies.
#include "gemm_common.hpp"

namespace lc {
namespace {

constexpr int NST = 4;  // stages of the LDS ring

template <int T> struct Cfg;
template <> struct Cfg<128> {
  static constexpr int SUB = 1, WR = 2, KSPL = 2;  // 64-deep slices per stage, waves per side, along k
};
template <> struct Cfg<64> {
  static constexpr int SUB = 2, WR = 1, KSPL = 4;
};
template <> struct Cfg<32> {
  static constexpr int SUB = 4, WR = 1, KSPL = 4;
};
constexpr int threads(int tile) { return tile == 128 ? 512 : 256; }

// What a tile column j of B is: B_PLAIN operand row n0 + j; B_ROPE columns c0 + [0,
// T / 2) and 64 + c0 + [0, T / 2) of one head (the 128 tile: the whole head), so that
// a rotated pair is in one tile; B_SWIGLU the first half gate rows, the second up rows.
enum { B_PLAIN, B_ROPE, B_SWIGLU };

// A slice of 64 k of an operand (T rows) in LDS: T / 8 runs of 1 KiB, RUN bytes
// apart, placed so that the 16 lanes of one phase of a fragment read ({0-3,
// 12-15} of a chunk, 4-11 of the next, and the like; 32 lanes for the transposing
// read) touch different banks.
//   k-major (128-byte rows, eight to a run), row r = 16 f + i:
//     T = 128: position f of run i
//     T = 64: position (f & 1) + 2 (i / 8) + 4 (f / 2) of run i % 8
//     T = 32: position i / 4 + 4 f of run i % 4
//   m/n-major (k rows of 2 T bytes), k row k:
//     T = 128: position k / 16 (of 4) of run swap23(k % 16) (swap23 exchanges
//       bits 2 and 3)
//     T = 64: position bit2(k) + 2 bit4(k) + 4 bit5(k) of run (k & 3) + 4 bit3(k)
//     T = 32: position k / 4 (of 16) of run k % 4
template <int T, bool KMAJ>
struct Opnd {
  static constexpr int RUNS = T / 8;

  // MFMA operand: rows 16 f .. + 15 at k = 32 s + 8 (lane / 16) + [0, 8)
  __device__ __forceinline__ static bf16x8_v frag(const lds_t *t, int f, int s, int lane) {
    if constexpr (KMAJ) {
      const int i = lane & 15;
      const lds_t *p = t + (lane >> 4) * 16 + s * 64;
      if constexpr (T == 128) p += i * RUN + f * 128;
      else if constexpr (T == 64) p += (i & 7) * RUN + ((f & 1) + 2 * (i >> 3) + 4 * (f >> 1)) * 128;
      else p += (i & 3) * RUN + ((i >> 2) + 4 * f) * 128;
      return *reinterpret_cast<const lds_v8 *>(p);
    } else {
      const int i16 = lane & 15, g = lane >> 4;
      const lds_t *p = t + f * 32 + (i16 & 3) * 8;
      if constexpr (T == 128) p += ((i16 >> 2) + 4 * (g & 1)) * RUN + ((g >> 1) + 2 * s) * 256;
      else if constexpr (T == 64) p += ((i16 >> 2) + 4 * (g & 1)) * RUN + (2 * (g >> 1) + 4 * s) * 128;
      else p += (i16 >> 2) * RUN + (2 * g + 8 * s) * 64;
      constexpr int HI = T == 128 ? 8 * RUN : T == 64 ? 128 : 64;  // k + 4
      const s16x4_v v[2] = {__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4 *)(p)),
                            __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4 *)(p + HI))};
      return __builtin_bit_cast(bf16x8_v, v);
    }
  }

  // this lane's part of load run q: its k inside the slice ...
  __device__ __forceinline__ static int run_k(int q, int lane) {
    if constexpr (KMAJ) return 8 * (lane & 7);
    else if constexpr (T == 128) return (q & 3) + 8 * ((q >> 2) & 1) + 4 * (q >> 3) + 16 * (lane >> 4);
    else if constexpr (T == 64) {
      const int pos = lane >> 3;
      return (q & 3) + 8 * (q >> 2) + 4 * (pos & 1) + 16 * ((pos >> 1) & 1) + 32 * (pos >> 2);
    } else return q + 4 * (lane >> 2);
  }
  // ... and its tile row (m/n-major: the first of 8)
  __device__ __forceinline__ static int run_row(int q, int lane) {
    if constexpr (!KMAJ) return 8 * (lane & (T / 8 - 1));
    const int pos = lane >> 3;
    if constexpr (T == 128) return 16 * pos + q;
    else if constexpr (T == 64) return 16 * ((pos & 1) + 2 * (pos >> 2)) + 8 * ((pos >> 1) & 1) + q;
    else return 16 * (pos >> 2) + 4 * (pos & 3) + q;
  }

  // byte offset of that part at k = k0 of the slice's first k (OOB: not in the operand)
  template <int MAP>
  __device__ __forceinline__ static uint32_t offset(int q, int lane, int64_t ld, int base, int lim, int k0) {
    const int j = run_row(q, lane), k = k0 + run_k(q, lane);
    int row = base + j, chk = row;
    if constexpr (MAP == B_SWIGLU) {  // base: first output column; lim: gate rows
      chk = base + (j & (T / 2 - 1));
      row = j < T / 2 ? chk : lim + chk;
    } else if constexpr (MAP == B_ROPE && T < 128) {  // base: T x tile column
      row = chk = (base & ~127) + (base & (128 - T)) / 2 + (j & (T / 2 - 1)) + (j < T / 2 ? 0 : 64);
    }
    if (chk >= lim) return OOB;
    return KMAJ ? (uint32_t)(((int64_t)row * ld + k) * 2) : (uint32_t)(((int64_t)k * ld + row) * 2);
  }
};

template <int T> constexpr int ring_bytes() { return NST * 2 * Cfg<T>::SUB * (T / 8) * RUN; }

// One workgroup's part: tile wg of nwg (ring: ring_bytes<T>() of LDS)
template <int T, bool A_K, bool B_K, int EPI, int TM, int ROWS = -1>
__device__ __forceinline__ void tile_block(GemmP p, int wg, int nwg, lds_t *R0) {
  using C = Cfg<T>;
  constexpr int NT = threads(T), NW = NT / 64, KS = 64 * C::SUB;
  constexpr int FR = T / 16 / C::WR;           // 16-row fragments per side of a wave's block
  constexpr int QS = KS / 32 / C::KSPL;        // k-steps per wave and stage
  constexpr int OPB = (T / 8) * RUN;           // one operand's 64-deep slice
  constexpr int STAGE = 2 * C::SUB * OPB;      // slices of A | B
  constexpr int LPW = C::SUB * (T / 8) / (NW / 2);  // loads per wave and stage
  static_assert(NST * STAGE >= C::KSPL * T * T * 4, "the epilogue's partial tiles reuse the ring");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / (C::WR * C::WR);  // this wave's k-steps of a stage: QS kg ..
  const int wr = wave % (C::WR * C::WR) / C::WR, wc = wave % C::WR;
  constexpr bool SWI = EPI == LC_EPI_SWIGLU;
  constexpr int MAPB = SWI ? B_SWIGLU : EPI == LC_EPI_ROPE ? B_ROPE : B_PLAIN;
  Tile tile;
  if (!find_tile<T, ROWS>(p, wg, nwg, tile)) return;  // before any barrier
  const int m0 = tile.m0, m_lim = tile.m_lim, kbeg = tile.kbeg, kend = tile.kend;
  const int n0 = SWI ? tile.tn * (T / 2) : tile.tn * T;

  f32x4_v acc[FR][FR];
#pragma unroll
  for (int i = 0; i < FR; ++i)
#pragma unroll
    for (int j = 0; j < FR; ++j) acc[i][j] = f32x4_v{0.0f, 0.0f, 0.0f, 0.0f};

  // the first half of the waves streams A, the second B: runs LPW wo .. + LPW - 1
  // of the operand's SUB T / 8 runs of a stage
  const int ns = (kend - kbeg + KS - 1) / KS;
  const int grp = wave / (NW / 2), wo = wave % (NW / 2);
  const i32x4_v rs = grp == 0 ? make_rsrc(p.A, p.a_bytes) : make_rsrc(tile.B, p.b_bytes);
  uint32_t vo[LPW];
  // run t of the wave: run qt(t) of slice st0 + sl(t)
  const int sub = wo * LPW / (T / 8), q0 = wo * LPW % (T / 8);
  constexpr int RUNS = T / 8;
  auto sl = [&](int t) { return LPW > RUNS ? t / RUNS : 0; };
  auto qt = [&](int t) { return LPW > RUNS ? t % RUNS : q0 + t; };
#pragma unroll
  for (int t = 0; t < LPW; ++t) {
    const int k0 = kbeg + 64 * (sub + sl(t));
    vo[t] = grp == 0 ? Opnd<T, A_K>::template offset<B_PLAIN>(qt(t), lane, p.lda, m0, m_lim, k0)
                     : Opnd<T, B_K>::template offset<MAPB>(qt(t), lane, p.ldb, n0, p.N, k0);
  }
  const bool gk = grp == 0 ? A_K : B_K;
  const uint32_t kbw = gk ? 2u : (uint32_t)((grp == 0 ? p.lda : p.ldb) * 2);
  lds_t *const dst0 = R0 + (2 * sub + grp) * OPB;
  auto at = [&](int t) { return 2 * sl(t) * OPB + qt(t) * RUN; };
  const bool ragged = (kend - kbeg) % KS != 0;
  auto load = [&](int st) {
    lds_t *d = dst0 + (st & (NST - 1)) * STAGE;
    const uint32_t so = (uint32_t)(st * KS) * kbw;
    if (ragged && st == ns - 1) {  // the stage ends past K: every lane checked
      const int kr = kend - kbeg - st * KS - 64 * sub;  // valid k from this wave's first slice
#pragma unroll
      for (int t = 0; t < LPW; ++t) {
        const int k = 64 * sl(t) + (grp == 0 ? Opnd<T, A_K>::run_k(qt(t), lane) : Opnd<T, B_K>::run_k(qt(t), lane));
        dma16(rs, d + at(t), k < kr && vo[t] != OOB ? vo[t] + so : OOB);
      }
      return;
    }
#pragma unroll
    for (int t = 0; t < LPW; ++t) dma16s(rs, d + at(t), vo[t], so);
  };

  typedef bf16x8_v Frag[QS][FR];
  Frag fa[2], fb[2];
  auto read = [&](int st, Frag &a, Frag &b) {
#pragma unroll
    for (int q = 0; q < QS; ++q) {
      const int ks = QS * kg + q;  // k-step of the stage
      const lds_t *t = R0 + (st & (NST - 1)) * STAGE + 2 * (ks >> 1) * OPB;
#pragma unroll
      for (int i = 0; i < FR; ++i) a[q][i] = Opnd<T, A_K>::frag(t, FR * wr + i, ks & 1, lane);
#pragma unroll
      for (int j = 0; j < FR; ++j) b[q][j] = Opnd<T, B_K>::frag(t + OPB, FR * wc + j, ks & 1, lane);
    }
  };
  auto multiply = [&](const Frag &a, const Frag &b) {
#pragma unroll
    for (int q = 0; q < QS; ++q)
#pragma unroll
      for (int i = 0; i < FR; ++i)
#pragma unroll
        for (int j = 0; j < FR; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[q][j], a[q][i], acc[i][j], 0, 0, 0);
  };
  constexpr int NRD = QS * FR * ((A_K ? 1 : 2) + (B_K ? 1 : 2)), NMF = QS * FR * FR;
  // Stage st + 1 has landed for every wave after the barrier, and every wave has
  // its fragments of stage st, whose slot then takes stage st + NST.
  auto step = [&](int st, Frag &a, Frag &b, Frag &an, Frag &bn) {
    const int later = ns - 2 - st;  // stages after st + 1, in flight at most NST - 2
    if (later >= NST - 2) wait_barrier<(NST - 2) * LPW>();
    else if (later == 1) wait_barrier<LPW>();
    else wait_barrier<0>();
    if (st + NST < ns) load(st + NST);
    read(st + 1, an, bn);  // (after the last stage: another slot's stale data, unused)
    multiply(a, b);
    interleave_steps<NRD, NMF>();
    __builtin_amdgcn_sched_barrier(0);
  };
  static_assert(NST == 4, "the waits above");
#pragma unroll 1
  for (int st = 0; st < min(ns, NST); ++st) load(st);
  if (ns >= 4) wait_barrier<3 * LPW>();
  else if (ns == 3) wait_barrier<2 * LPW>();
  else if (ns == 2) wait_barrier<LPW>();
  else wait_barrier<0>();
  if (ns > 0) read(0, fa[0], fb[0]);
  for (int st = 0; st < ns; st += 2) {
    step(st, fa[0], fb[0], fa[1], fb[1]);
    if (st + 1 < ns) step(st + 1, fa[1], fb[1], fa[0], fb[0]);
  }

  // ------------------------------------------------------------ epilogue
  // Every wave writes its partial block to its k-steps' copy of the fp32 tile in the
  // (now idle) ring, 16-byte chunk c of row r at chunk c ^ (r & 15) (& 7: 32 tile);
  // then each thread adds the copies of four columns (a pair of fours for RoPE
  // and SwiGLU) in k-step order and stores them, whole rows by consecutive lanes.
  // Tensors the epilogue reads are loaded before the barrier.
  typedef EpiTypes<EPI, TM> ET;
  const int c_dt = ET::C >= 0 ? ET::C : p.c_dt, r_dt = ET::R >= 0 ? ET::R : p.r_dt,
            aux_dt = ET::X >= 0 ? ET::X : p.aux_dt;
  typedef __attribute__((address_space(3))) f32x4_v lds_f4;
  constexpr bool PAIR = EPI == LC_EPI_ROPE || SWI;
  constexpr int QW = PAIR ? T / 8 : T / 4;   // column quads a row's threads take
  constexpr int IT = T * QW > NT ? T * QW / NT : 1;  // (RoPE, SwiGLU, 32 tile: half the threads)
  constexpr int SWZ = T / 4 < 16 ? T / 4 - 1 : 15;
  constexpr bool LD = EPI == LC_EPI_RESIDUAL || EPI == LC_EPI_ACCUM_F32 || EPI == LC_EPI_SWIGLU_BWD;
  const int q = tid % QW;
  int n;  // first of this thread's columns
  if constexpr (EPI == LC_EPI_ROPE && T < 128) n = (n0 & ~127) + (n0 & (128 - T)) / 2 + 4 * q;
  else n = n0 + 4 * q;
  const bool n_ok = n < p.N;
  auto row_of = [&](int it) { return (it * NT + tid) / QW; };
  float4 x[IT], y[IT];
  if constexpr (LD) {
    const int nc = n_ok ? n : 0;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int64_t mc = min(m0 + row_of(it), m_lim - 1);
      if constexpr (EPI == LC_EPI_RESIDUAL) x[it] = load4_dt(p.R, mc * p.ldr + nc, r_dt);
      if constexpr (EPI == LC_EPI_ACCUM_F32)
        x[it] = *reinterpret_cast<const float4 *>(static_cast<const float *>(tile.C) + mc * p.ldc + nc);
      if constexpr (EPI == LC_EPI_SWIGLU_BWD) {
        x[it] = load4_dt(p.aux0, mc * p.ld_aux + nc, aux_dt);
        y[it] = load4_dt(p.aux1, mc * p.ld_aux + nc, aux_dt);
      }
    }
  }
  __syncthreads();  // every wave's last fragment reads are done
  lds_t *const E = R0 + kg * (T * T * 4);
#pragma unroll
  for (int i = 0; i < FR; ++i)
#pragma unroll
    for (int j = 0; j < FR; ++j) {
      const int r = 16 * (FR * wr + i) + (lane & 15), c = 4 * (FR * wc + j) + (lane >> 4);
      *reinterpret_cast<lds_f4 *>(E + r * (T * 4) + ((c ^ (r & SWZ)) << 4)) = acc[i][j];
    }
  __syncthreads();
  auto sum4 = [&](int r, int c) {
    const lds_t *s = R0 + r * (T * 4) + ((c ^ (r & SWZ)) << 4);
    f32x4_v v = *reinterpret_cast<const lds_f4 *>(s);
#pragma unroll
    for (int k = 1; k < C::KSPL; ++k) v += *reinterpret_cast<const lds_f4 *>(s + k * (T * T * 4));
    return v;
  };
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int r = row_of(it), m = m0 + r;
    if (r >= T || m >= m_lim || !n_ok) continue;
    const f32x4_v v = sum4(r, q);
    const int64_t oc = (int64_t)m * p.ldc + n;
    if constexpr (PAIR) {
      const f32x4_v w = sum4(r, q + QW);
      float a[4] = {v[0], v[1], v[2], v[3]}, b[4] = {w[0], w[1], w[2], w[3]};
      if constexpr (EPI == LC_EPI_ROPE) {
        if (n < p.rope_cols) {
          const int64_t ta = (int64_t)(m % p.rope_seq) * 64 + (n & 127);
          const float4 cs = *reinterpret_cast<const float4 *>(p.rcos + ta);
          const float4 sn = *reinterpret_cast<const float4 *>(p.rsin + ta);
          const float cv[4] = {cs.x, cs.y, cs.z, cs.w}, sv[4] = {sn.x, sn.y, sn.z, sn.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) rope_pair(a[e], b[e], cv[e], sv[e]);
        }
        store4_dt(tile.C, oc, c_dt, a[0], a[1], a[2], a[3]);
        store4_dt(tile.C, oc + 64, c_dt, b[0], b[1], b[2], b[3]);
        if (p.aux0) {  // a second copy in aux_dt
          const int64_t oa = (int64_t)m * p.ld_aux + n;
          store4_dt(p.aux0, oa, aux_dt, a[0], a[1], a[2], a[3]);
          store4_dt(p.aux0, oa + 64, aux_dt, b[0], b[1], b[2], b[3]);
        }
      } else {
        float act[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) act[e] = a[e] * sigmoidf_(a[e]) * b[e];
        const int64_t oa = (int64_t)m * p.ld_aux + n;
        store4_dt(p.aux0, oa, aux_dt, a[0], a[1], a[2], a[3]);
        store4_dt(p.aux1, oa, aux_dt, b[0], b[1], b[2], b[3]);
        store4_dt(tile.C, oc, c_dt, act[0], act[1], act[2], act[3]);
      }
    } else if constexpr (EPI == LC_EPI_SWIGLU_BWD) {
      const float gv[4] = {x[it].x, x[it].y, x[it].z, x[it].w};
      const float uv[4] = {y[it].x, y[it].y, y[it].z, y[it].w};
      float dg[4], du[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) swiglu_grad(v[e], gv[e], uv[e], dg[e], du[e]);
      store4_dt(tile.C, oc, c_dt, dg[0], dg[1], dg[2], dg[3]);
      store4_dt(tile.C, oc + p.N, c_dt, du[0], du[1], du[2], du[3]);
    } else if constexpr (EPI == LC_EPI_ACCUM_F32) {
      *reinterpret_cast<float4 *>(static_cast<float *>(tile.C) + oc) =
          make_float4(x[it].x + v[0], x[it].y + v[1], x[it].z + v[2], x[it].w + v[3]);
    } else if constexpr (EPI == LC_EPI_RESIDUAL) {
      store4_dt(tile.C, oc, c_dt, x[it].x + v[0], x[it].y + v[1], x[it].z + v[2], x[it].w + v[3]);
    } else {
      store4_dt(tile.C, oc, c_dt, v[0], v[1], v[2], v[3]);
    }
  }
}

// (residual products are never grouped)
constexpr bool splits_rows(int epi) { return epi == LC_EPI_STORE || epi == LC_EPI_ACCUM_F32; }

template <int T, bool A_K, bool B_K, int EPI, int TM>
__global__ __launch_bounds__(threads(T)) void gemm_tile_kernel(GemmP p) {
  __shared__ __align__(16) char ring[ring_bytes<T>()];
  constexpr bool SPLIT = T == 128 && (splits_rows(EPI) || EPI == LC_EPI_RESIDUAL);
  tile_block<T, A_K, B_K, EPI, TM, SPLIT ? 0 : -1>(p, (int)blockIdx.x, (int)gridDim.x, LDS_AS(char, ring));
}

// Grouped rows in 128 tiles, of plain and accumulating products: in a kernel of their own, as
// the search for a tile's group costs the others 0.2 to 0.5 us a launch (8 of the 145
// launches of a small bf16 step, d 512: 958 us, now 955). The fused epilogues keep both in one
// kernel, whose main loop the compiler schedules better (RoPE and SwiGLU 3%).
template <bool A_K, bool B_K, int EPI, int TM>
__global__ __launch_bounds__(threads(128)) void gemm_tile_rows_kernel(GemmP p) {
  __shared__ __align__(16) char ring[ring_bytes<128>()];
  tile_block<128, A_K, B_K, EPI, TM, 1>(p, (int)blockIdx.x, (int)gridDim.x, LDS_AS(char, ring));
}

// An input gradient's nx tiles and a weight gradient's nw in one grid: two products
// of a backward that do not depend on each other and would each leave most of the
// chip idle. Each with the tile and order of additions it takes alone, so the results
// are the same bits with one launch or two. A small bf16 step (d 512, 256 tokens, 2
// layers, 4 microbatches; 24 launches fewer) 1012 -> 955 us.
template <int TX, int EPI, int TM, int TW>
__global__ __launch_bounds__(256) void gemm_tile_pair_kernel(GemmP x, GemmP w, int nx, int nw) {
  static_assert(threads(TX) == 256 && threads(TW) == 256, "");
  constexpr int BYTES = ring_bytes<TX>() > ring_bytes<TW>() ? ring_bytes<TX>() : ring_bytes<TW>();
  __shared__ __align__(16) char ring[BYTES];
  const int i = (int)blockIdx.x;
  if (i < nx) tile_block<TX, true, false, EPI, TM>(x, i, nx, LDS_AS(char, ring));
  else tile_block<TW, false, false, LC_EPI_ACCUM_F32, 0>(w, i - nx, nw, LDS_AS(char, ring));
}

template <bool A_K, bool B_K, int EPI, int TM = 0>
lc_status launch_t(const GemmP &p, int tile, hipStream_t s) {
  unsigned grid = (unsigned)p.tiles_m * (unsigned)p.tiles_n;
  if (p.gmode == LC_GROUP_ROWS) grid = (unsigned)(p.tiles_m + p.ngroups) * (unsigned)p.tiles_n;
  if (p.gmode == LC_GROUP_K) grid *= (unsigned)p.ngroups;
  if constexpr (splits_rows(EPI)) {
    if (tile == 128 && p.gmode == LC_GROUP_ROWS) {
      hipLaunchKernelGGL((gemm_tile_rows_kernel<A_K, B_K, EPI, TM>), dim3(grid), dim3(threads(128)), 0, s, p);
      return check_launch("gemm_tile_rows_kernel");
    }
  }
  if (tile == 128)
    hipLaunchKernelGGL((gemm_tile_kernel<128, A_K, B_K, EPI, TM>), dim3(grid), dim3(threads(128)), 0, s, p);
  else if (tile == 64)
    hipLaunchKernelGGL((gemm_tile_kernel<64, A_K, B_K, EPI, TM>), dim3(grid), dim3(threads(64)), 0, s, p);
  else
    hipLaunchKernelGGL((gemm_tile_kernel<32, A_K, B_K, EPI, TM>), dim3(grid), dim3(threads(32)), 0, s, p);
  return check_launch("gemm_tile_kernel");
}

template <int TX, int EPI, int TM>
void pair_t(const GemmP &x, const GemmP &w, int w_tile, hipStream_t s) {
  const int nx = x.tiles_m * x.tiles_n, nw = w.tiles_m * w.tiles_n;
  const dim3 grid((unsigned)(nx + nw)), block(256);
  if (w_tile == 64) hipLaunchKernelGGL((gemm_tile_pair_kernel<TX, EPI, TM, 64>), grid, block, 0, s, x, w, nx, nw);
  else hipLaunchKernelGGL((gemm_tile_pair_kernel<TX, EPI, TM, 32>), grid, block, 0, s, x, w, nx, nw);
}

}  // namespace

lc_status gemm_tile_pair_launch(GemmP x, int x_epi, int x_tile, GemmP w, int w_tile, hipStream_t s) {
  x.tiles_m = (x.M + x_tile - 1) / x_tile;
  x.tiles_n = (x.N + x_tile - 1) / x_tile;
  w.tiles_m = (w.M + w_tile - 1) / w_tile;
  w.tiles_n = (w.N + w_tile - 1) / w_tile;
  if (x_epi == LC_EPI_SWIGLU_BWD) {
    if (x_tile == 64) pair_t<64, LC_EPI_SWIGLU_BWD, 1>(x, w, w_tile, s);
    else pair_t<32, LC_EPI_SWIGLU_BWD, 1>(x, w, w_tile, s);
  } else {
    if (x_tile == 64) pair_t<64, LC_EPI_STORE, 0>(x, w, w_tile, s);
    else pair_t<32, LC_EPI_STORE, 0>(x, w, w_tile, s);
  }
  return check_launch("gemm_tile_pair_kernel");
}

lc_status gemm_tile_launch(GemmP p, const lc_gemm_args &a, int tile, hipStream_t s) {
  const int cols = a.epilogue == LC_EPI_SWIGLU ? tile / 2 : tile;
  p.tiles_m = (p.M + tile - 1) / tile;
  p.tiles_n = (p.N + cols - 1) / cols;
  const bool ak = a.a_kmajor != 0, bk = a.b_kmajor != 0;
  switch (a.epilogue) {
    case LC_EPI_STORE:
    case LC_EPI_STORE_F32:
      if (ak && bk) return launch_t<true, true, LC_EPI_STORE>(p, tile, s);
      if (ak && !bk) return launch_t<true, false, LC_EPI_STORE>(p, tile, s);
      if (!ak && !bk) return launch_t<false, false, LC_EPI_STORE>(p, tile, s);
      break;
    case LC_EPI_ACCUM_F32:
      if (ak && bk) return launch_t<true, true, LC_EPI_ACCUM_F32>(p, tile, s);
      if (!ak && !bk) return launch_t<false, false, LC_EPI_ACCUM_F32>(p, tile, s);
      break;
    case LC_EPI_RESIDUAL:
      if (ak && bk && p.c_dt == LC_FP32 && p.r_dt == LC_FP32)
        return launch_t<true, true, LC_EPI_RESIDUAL, 1>(p, tile, s);
      if (ak && bk) return launch_t<true, true, LC_EPI_RESIDUAL>(p, tile, s);
      break;
    case LC_EPI_ROPE:
      if (ak && bk && p.c_dt == LC_FP16 && (!p.aux0 || p.aux_dt == LC_BF16))
        return launch_t<true, true, LC_EPI_ROPE, 1>(p, tile, s);
      if (ak && bk) return launch_t<true, true, LC_EPI_ROPE>(p, tile, s);
      break;
    case LC_EPI_SWIGLU:
      if (ak && bk && p.c_dt == LC_BF16 && p.aux_dt == LC_FP32)
        return launch_t<true, true, LC_EPI_SWIGLU, 1>(p, tile, s);
      if (ak && bk) return launch_t<true, true, LC_EPI_SWIGLU>(p, tile, s);
      break;
    case LC_EPI_SWIGLU_BWD:
      if (ak && !bk && p.c_dt == LC_BF16 && p.aux_dt == LC_FP32)
        return launch_t<true, false, LC_EPI_SWIGLU_BWD, 1>(p, tile, s);
      if (ak && !bk) return launch_t<true, false, LC_EPI_SWIGLU_BWD>(p, tile, s);
      if (ak && bk) return launch_t<true, true, LC_EPI_SWIGLU_BWD>(p, tile, s);
      break;
  }
  return fail(LC_ERR_UNSUPPORTED, "gemm bf16: layout (a_kmajor=%d, b_kmajor=%d) not built for "
              "epilogue %d", (int)ak, (int)bk, a.epilogue);
}

}  // namespace lc

// bf16 GEMM on CDNA4 matrix cores (v_mfma_f32_16x16x32_bf16), fp32 accumulation,
// with the fused epilogues of a decoder layer's projections.
//
//   C(m, n) = sum_k A(m, k) B(n, k)
//   A(m, k) = A_K ? A[m*lda + k] : A[k*lda + m]      (A_K: k is contiguous)
//   B(n, k) = B_K ? B[n*ldb + k] : B[k*ldb + n]
//
// Tile: 256 x 256 per workgroup of 512 threads (8 waves, 4 along m x 2 along
// n); each wave owns 64 x 128 = 4 x 8 MFMA blocks of 16 x 16. K is walked in
// stages of 64: LDS holds two 64 KiB stages (A 256 x 64 | B 256 x 64); while
// the waves multiply stage s, stage s + 1 streams in from HBM/L2, and one
// barrier per stage both publishes the new stage and frees the old one.
// Waves 0-3 stream A, waves 4-7 stream B (8 loads of 1 KiB per wave per
// stage). A stage is multiplied in four steps (k half, row half), the fragments
// of the next step read while one multiplies.
//
// What bounds it: the chip's power limit. Full-size products run at 1.9-2.0 GHz
// of the nominal 2.4, and with the stage's loads left out the clock rises to
// 2.25 GHz while the cycle count falls only 11%. Hence the 16 x 16 x 32
// instruction: the same rate per cycle as 32 x 32 x 16 but half the accumulator
// traffic per product, and a register-only loop on normal data sustains 2110
// TFLOP/s with it against 1848 with 32 x 32 x 16. Over the twelve products of a
// d 4096 / FFN 11008 / 4096-token layer: 4271 us against 4453 (the 4096^3 NT
// product at 2.02 GHz instead of 1.89).
//
// Operand tiles go from HBM straight into LDS (buffer_load_dwordx4 ... lds:
// lane l of a wave's load fills bytes [16 l, 16 l + 16) of a 1 KiB LDS run),
// so no register staging is needed; the lanes of a load read global memory in
// address order, and padding between runs keeps fragment reads free of LDS
// bank conflicts. Buffer
// descriptors make out-of-range lanes (matrix edges, K tail) read zeros.
//   k-major operand: LDS rows of 64 k (128 B, one full cache line of the
//     operand row per 8-lane group, lanes in address order). Load run q
//     (0..31) holds tile rows q, q + 32, ..., q + 224, and runs sit 1056 bytes
//     apart, so tile row 32 p + q is at q * 1056 + 128 p. A fragment (16 rows,
//     four 16-byte k chunks) is one ds_read_b128. It is served in phases of 16
//     lanes, {0-3, 12-15, 20-27} and so on: rows 0-3 and 12-15 of one chunk with
//     rows 4-11 of the next, so a run distance of 2 chunks mod 16 (32 bytes of
//     padding) makes each phase touch all 64 banks once. (A distance of one
//     chunk, right for 32-row fragments, collides here. Rows of 32 k, i.e. half
//     cache lines per load, cost a third of the throughput of the global->LDS
//     path.)
//   m/n-major operand (a weight read as dX = dY W, both operands of a weight
//     gradient dW = dY^T X): LDS rows of one k and 256 m (512 B, lanes in
//     address order); run q holds k rows swap23(q) and swap23(q) + 32 (swap23
//     exchanges bits 2 and 3), runs sit 1056 bytes apart. The fragment is read
//     with the CDNA4 transposing load ds_read_b64_tr_b16: in each group of 16
//     lanes, lane j receives element j % 4 of the 8 bytes addressed by lane
//     4e + j / 4 as its element e, so lanes addressing four consecutive k rows
//     at four 4-element column runs receive one column's four k values each.
//     Two such loads (k rows 8g + [0, 4) and 8g + 4 + [0, 4) for lane group g)
//     give the 8 k values of the MFMA operand; swap23 puts the eight k rows that
//     32 lanes address in one phase into eight consecutive runs, 32 bytes apart
//     in the banks. No transposed copy exists in HBM and no register shuffles
//     are spent.
//
// The MFMA is issued with B's fragment in the instruction's first operand and
// A's in the second, which leaves lane l holding output row m = l % 16 and four
// consecutive columns n = 4(l / 16) + e of each block; the column pairs (c, c +
// 64) that RoPE and SwiGLU combine sit in one wave (blocks j and j + 4).
// Output, residual and gate/up element types are run-time values (uniform
// branches in the epilogue only), except in the instantiations for the decoder
// stage's own type mix (EpiTypes in gemm_common.hpp), where they are compile-time
// constants.
#include "gemm_common.hpp"

namespace lc {
namespace {

constexpr int BM = 256, BN = 256;
constexpr int KS = 64;             // k per stage
constexpr int NT = 512;            // threads per workgroup (8 waves)
constexpr int WM = 64, WN = 128;   // wave tile
constexpr int FM = WM / 16, FN = WN / 16;  // 16 x 16 MFMA blocks of a wave
constexpr int OPND_BYTES = 32 * RUN;       // one operand's stage in LDS (32 runs)
constexpr int STAGE_BYTES = 2 * OPND_BYTES;   // A | B
// One wave's share of an operand's loads: 8 of the 32 1-KiB LDS runs of a
// 256 x 64 stage (the four waves of a group load one operand).
//   k-major: run q = tile rows q + 32 p (p = 0..7); lane l -> position l/8,
//     global k chunk l%8.
//     ROWMAP 0: tile row r -> operand row base + r (valid below lim)
//     ROWMAP 1 (SwiGLU B rows): tile row r -> gate row ob + (r>>7)*64 + (r&63)
//       for (r&127) < 64, else up row lim + ob + (r>>7)*64 + (r&63); valid
//       while the output column ob + (r>>7)*64 + (r&63) < lim.
//   m/n-major: run q = k rows swap23(q) and swap23(q) + 32; lane l -> k row
//     swap23(q) + 32 (l/32), global columns 8 (l%32) .. +7.
// Run t of wave w is q = 8w + t. The per-lane state is a row offset,
// an in-row offset, a validity mask and a k position; everything else is
// wave-uniform.
template <bool KMAJ, int ROWMAP>
struct Stream {
  uint32_t base;     // byte offset of run 0's row (k-major) or k row (m/n-major)
  uint32_t col;      // byte offset inside the row
  uint32_t run;      // byte distance between two rows (k-major) or k rows
  uint32_t kb;       // bytes per unit of k
  uint32_t rows;     // bit t set when run t's row / columns are inside the operand
  int kl;            // k-major: first k of this lane's chunk; m/n-major: k row of run 0

  __device__ __forceinline__ void init(int64_t ld, int base_row, int lim, int wave, int lane) {
    if constexpr (KMAJ) {
      const int pos = lane >> 3;  // the lane's row position inside each run
      kl = 8 * (lane & 7);
      int grow0, oc0;
      if constexpr (ROWMAP == 0) {
        grow0 = base_row + 8 * wave + 32 * pos;
        oc0 = grow0;
      } else {
        // tile row r = q + 32 pos: a gate row while (pos & 2) == 0, else an up
        // row, of output column base_row + (pos >> 2) 64 + 32 (pos & 1) + q
        oc0 = base_row + (pos >> 2) * 64 + 32 * (pos & 1) + 8 * wave;
        grow0 = (pos & 2) ? lim + oc0 : oc0;
      }
      rows = 0;
#pragma unroll
      for (int t = 0; t < 8; ++t) rows |= (oc0 + t < lim ? 1u : 0u) << t;
      base = rows ? (uint32_t)((int64_t)grow0 * ld * 2) : 0u;
      col = (uint32_t)(kl * 2);
      run = (uint32_t)(ld * 2);
      kb = 2;
    } else {
      static_assert(ROWMAP == 0, "row remap needs a k-major operand");
      // k row of run 0: run q holds k rows swap23(q) and swap23(q) + 32
      const int kr0 = 4 * (wave & 1) + 16 * (wave >> 1) + 32 * (lane >> 5);
      const int gm = base_row + 8 * (lane & 31);    // first of the lane's 8 columns
      kl = kr0;
      rows = gm < lim ? 0xFFu : 0u;
      base = (uint32_t)((int64_t)kr0 * ld * 2);
      col = gm < lim ? (uint32_t)(gm * 2) : 0u;
      run = (uint32_t)(ld * 2);
      kb = (uint32_t)(ld * 2);
    }
  }

  // rows (k-major) or k rows between run t and run 0
  __device__ __forceinline__ static uint32_t step(int t) { return KMAJ ? t : (t & 3) + 8 * (t >> 2); }
  // each run's per-lane byte offset at k = k0 (OOB for lanes outside the
  // operand's rows or columns); valid for stages that end at or before K
  __device__ __forceinline__ void offsets(uint32_t vo[8], int k0) const {
#pragma unroll
    for (int t = 0; t < 8; ++t)
      vo[t] = (rows >> t) & 1u ? base + step(t) * run + col + (uint32_t)k0 * kb : OOB;
  }
  // run t of the wave's 8 runs of the stage starting at k0, into `lds` (the
  // operand's stage), every lane checked against K
  __device__ __forceinline__ void load1(i32x4_v rs, lds_t *lds, int wave, int k0, int K, int t) const {
    bool ok = (rows >> t) & 1u;
    if constexpr (KMAJ) ok = ok && k0 + kl < K;
    else ok = ok && k0 + kl + (int)step(t) < K;
    const uint32_t off = ok ? base + step(t) * run + col + (uint32_t)k0 * kb : OOB;
    dma16(rs, lds + (8 * wave + t) * RUN, off);
  }
};

// MFMA operand of 16 rows (row0 .. row0+15) at k = 32 s + 8 (lane / 16) + [0, 8)
// of the stage stored at t (s = 0, 1)
template <bool KMAJ>
__device__ __forceinline__ bf16x8_v frag(const lds_t *t, int row0, int s, int lane) {
  if constexpr (KMAJ) {
    // tile row r is position r / 32 of run r % 32
    return *reinterpret_cast<const lds_v8 *>(t + ((lane & 15) + (row0 & 16)) * RUN + (row0 >> 5) * 128 +
                                             s * 64 + (lane >> 4) * 16);
  } else {
    // k row k is position k / 32 of run swap23(k % 32)
    const int i16 = lane & 15, g = lane >> 4;
    const lds_t *p0 = t + ((i16 >> 2) + 4 * (g & 1) + 16 * (g >> 1)) * RUN + s * 512 + (row0 + 4 * (i16 & 3)) * 2;
    const s16x4_v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4 *)(p0));
    const s16x4_v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4 *)(p0 + 8 * RUN));
    const s16x4_v v[2] = {lo, hi};
    return __builtin_bit_cast(bf16x8_v, v);
  }
}

template <bool A_K, bool B_K, int EPI, int TM>
__global__ __launch_bounds__(NT) void gemm_bf16_kernel(GemmP p) {
  __shared__ __align__(16) char ring[2 * STAGE_BYTES];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int grp = wave >> 2, w4 = wave & 3;
  const int wm = w4, wn = grp;  // group g owns output columns [128 g, 128 g + 128)

  constexpr bool SWI = (EPI == LC_EPI_SWIGLU);
  Tile tile;
  if (!find_tile<BM>(p, (int)blockIdx.x, (int)gridDim.x, tile)) return;  // before any barrier
  const int m0 = tile.m0, tn = tile.tn, m_lim = tile.m_lim, kbeg = tile.kbeg, kend = tile.kend;
  const bf16_t *const Bp = tile.B;
  void *const Cp = tile.C;
  const int n0 = SWI ? tn * (BN / 2) : tn * BN;  // first output column

  f32x4_v acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_v{0.0f, 0.0f, 0.0f, 0.0f};

  lds_t *const R0 = LDS_AS(char, ring);
  const int ns = (kend - kbeg + KS - 1) / KS;  // stages
  // group 0 streams A, group 1 streams B
  const i32x4_v rs = grp == 0 ? make_rsrc(p.A, p.a_bytes) : make_rsrc(Bp, p.b_bytes);
  Stream<A_K, 0> sa_;
  Stream<B_K, SWI ? 1 : 0> sb_;
  if (grp == 0) sa_.init(p.lda, m0, m_lim, w4, lane);
  else sb_.init(p.ldb, n0, p.N, w4, lane);
  // Full stages use offsets computed once: run t's per-lane offset at kbeg,
  // plus the stage's k advance in the scalar offset (the same code for both
  // groups). A last stage that ends past K takes the per-lane K check.
  uint32_t vo[8];
  if (grp == 0) sa_.offsets(vo, kbeg);
  else sb_.offsets(vo, kbeg);
  const bool gk = grp == 0 ? A_K : B_K;
  const uint32_t kbw = gk ? 2u : (uint32_t)((grp == 0 ? p.lda : p.ldb) * 2);
  lds_t *const dst0 = R0 + grp * OPND_BYTES + 8 * w4 * RUN;
  const bool ragged = (kend - kbeg) % KS != 0;
  auto load = [&](int st, int t0, int t1) {  // runs t0 .. t1 - 1 of this group's operand of stage st
    if (st >= ns) return;
    if (ragged && st == ns - 1) {
      lds_t *stage = R0 + (st & 1) * STAGE_BYTES;
#pragma unroll
      for (int t = t0; t < t1; ++t) {
        if (grp == 0) sa_.load1(rs, stage, w4, kbeg + st * KS, kend, t);
        else sb_.load1(rs, stage + OPND_BYTES, w4, kbeg + st * KS, kend, t);
      }
      return;
    }
    lds_t *d = dst0 + (st & 1) * STAGE_BYTES;
    const uint32_t so = (uint32_t)(st * KS) * kbw;
#pragma unroll
    for (int t = t0; t < t1; ++t) dma16s(rs, d + t * RUN, vo[t], so);
  };

  // A stage is multiplied in four steps of 16 MFMAs: k half q (32 k), row half h
  // of the wave's 64 rows. The barrier that publishes stage st + 1 (each wave's
  // loads of it and fragment reads of stage st done) sits before stage st's last
  // step, and frees stage st's buffer: half of stage st + 2's loads are issued
  // right there, the other half a step later. All eight at the start of stage st
  // + 1 leave a step less to arrive in and a fuller load queue (7B-shaped layer
  // forward + backward 5245 us against 5120 this way); all eight right after the
  // barrier collide with the fragment reads (2% slower products), and later
  // loads, in twos over the steps, arrive late (3%).
  bf16x8_v fa[FM], fb[2][FN];
  auto read_a = [&](int st, int q, int h) {
    const lds_t *t = R0 + (st & 1) * STAGE_BYTES;
#pragma unroll
    for (int i = 0; i < FM / 2; ++i) fa[2 * h + i] = frag<A_K>(t, wm * WM + (2 * h + i) * 16, q, lane);
  };
  auto read_b = [&](int st, int q) {
    const lds_t *t = R0 + (st & 1) * STAGE_BYTES + OPND_BYTES;
#pragma unroll
    for (int j = 0; j < FN; ++j) fb[q][j] = frag<B_K>(t, wn * WN + j * 16, q, lane);
  };
  auto multiply = [&](int q, int h) {
#pragma unroll
    for (int i = 2 * h; i < 2 * h + 2; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[q][j], fa[i], acc[i][j], 0, 0, 0);
  };
  constexpr int RDA = A_K ? 2 : 4, RDB = B_K ? FN : 2 * FN;  // LDS reads of half A's, of B's fragments
  load(0, 0, 8);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __syncthreads();
  if (ns > 0) {
    read_a(0, 0, 0);
    read_b(0, 0);
    load(1, 0, 4);
  }
  for (int st = 0; st < ns; ++st) {
    load(st + 1, 4, 8);
    read_a(st, 0, 1);
    multiply(0, 0);
    interleave_steps<RDA, 16>();
    __builtin_amdgcn_sched_barrier(0);
    read_a(st, 1, 0);
    read_b(st, 1);
    multiply(0, 1);
    interleave_steps<RDA + RDB, 16>();
    __builtin_amdgcn_sched_barrier(0);
    read_a(st, 1, 1);
    multiply(1, 0);
    interleave_steps<RDA, 16>();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
    __syncthreads();
    load(st + 2, 0, 4);
    // (after the last stage this reads the other buffer's stale data, unused)
    read_a(st + 1, 0, 0);
    read_b(st + 1, 0);
    multiply(1, 1);
    interleave_steps<RDA + RDB, 16>();
    __builtin_amdgcn_sched_barrier(0);
  }

  // ------------------------------------------------------------ epilogue
  // Each wave stages its 64 x 128 fp32 results through its own 16 KiB of the
  // (now idle) LDS ring, one 32-row block at a time: written in the MFMA
  // layout (lane = row, registers = columns), read back row-contiguous (16-byte
  // chunk c of row r at chunk c ^ (r & 15): both directions conflict-free), so
  // that every global access of the epilogue covers whole cache lines (two
  // rows of 128 columns, or four rows of two 64-column halves, per
  // instruction). Loads of a group of rows are issued before its stores.
  __syncthreads();  // every wave's last fragment reads are done
  lds_t *const E = R0 + wave * 16384;
  typedef EpiTypes<EPI, TM> ET;
  const int c_dt = ET::C >= 0 ? ET::C : p.c_dt, r_dt = ET::R >= 0 ? ET::R : p.r_dt,
            aux_dt = ET::X >= 0 ? ET::X : p.aux_dt;
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  typedef __attribute__((address_space(3))) f32x4_t lds_f4;
  const int ncol0 = n0 + wn * WN;  // first of the wave's 128 accumulator columns (non-SwiGLU)
  // 32-row block i of the wave's results into its LDS staging area
  auto stage_block = [&](int i) {
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int r = 16 * f + (lane & 15), c = 4 * j + (lane >> 4);
        *reinterpret_cast<lds_f4 *>(E + r * 512 + ((c ^ (r & 15)) << 4)) = acc[2 * i + f][j];
      }
  };
  auto chunk = [&](int r, int c) -> float4 {
    const f32x4_t v = *reinterpret_cast<const lds_f4 *>(E + r * 512 + ((c ^ (r & 15)) << 4));
    return make_float4(v[0], v[1], v[2], v[3]);
  };
  if constexpr (EPI == LC_EPI_ROPE || EPI == LC_EPI_SWIGLU) {
#pragma unroll
    for (int i = 0; i < WM / 32; ++i) {
      const int mrow0 = m0 + wm * WM + i * 32;
      stage_block(i);
      {
        // lane: row 4 s + lane / 16, column quads q and q + 16 (columns 4q and 64 + 4q)
        const int q = lane & 15;
#pragma unroll
        for (int s0 = 0; s0 < 8; s0 += 4) {
          float4 x1[4], x2[4], cs[4], sn[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int rl = 4 * (s0 + u) + (lane >> 4);
            x1[u] = chunk(rl, q);
            x2[u] = chunk(rl, q + 16);
            if constexpr (EPI == LC_EPI_ROPE) {
              const int m = min(mrow0 + rl, m_lim - 1);
              const int pos = m % p.rope_seq;
              cs[u] = *reinterpret_cast<const float4 *>(p.rcos + (int64_t)pos * 64 + 4 * q);
              sn[u] = *reinterpret_cast<const float4 *>(p.rsin + (int64_t)pos * 64 + 4 * q);
            }
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int rl = 4 * (s0 + u) + (lane >> 4);
            const int m = mrow0 + rl;
            if (m >= m_lim) continue;
            float a[4] = {x1[u].x, x1[u].y, x1[u].z, x1[u].w};
            float b[4] = {x2[u].x, x2[u].y, x2[u].z, x2[u].w};
            if constexpr (EPI == LC_EPI_ROPE) {
              if (ncol0 >= p.N) continue;  // head past the output (uniform)
              if (ncol0 < p.rope_cols) {
                const float cv[4] = {cs[u].x, cs[u].y, cs[u].z, cs[u].w};
                const float sv[4] = {sn[u].x, sn[u].y, sn[u].z, sn[u].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) rope_pair(a[e], b[e], cv[e], sv[e]);
              }
              const int64_t row = (int64_t)m * p.ldc + ncol0 + 4 * q;
              store4_dt(Cp, row, c_dt, a[0], a[1], a[2], a[3]);
              store4_dt(Cp, row + 64, c_dt, b[0], b[1], b[2], b[3]);
              if (p.aux0) {  // a second copy in aux_dt
                const int64_t ra = (int64_t)m * p.ld_aux + ncol0 + 4 * q;
                store4_dt(p.aux0, ra, aux_dt, a[0], a[1], a[2], a[3]);
                store4_dt(p.aux0, ra + 64, aux_dt, b[0], b[1], b[2], b[3]);
              }
            } else {
              const int n = n0 + wn * 64 + 4 * q;  // output column of the gate/up pair
              if (n >= p.N) continue;
              float act[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) act[e] = a[e] * sigmoidf_(a[e]) * b[e];
              const int64_t oa = (int64_t)m * p.ld_aux + n;
              store4_dt(p.aux0, oa, aux_dt, a[0], a[1], a[2], a[3]);
              store4_dt(p.aux1, oa, aux_dt, b[0], b[1], b[2], b[3]);
              store4_dt(Cp, (int64_t)m * p.ldc + n, c_dt, act[0], act[1], act[2], act[3]);
            }
          }
        }
      }
    }
  } else {
    // lane: row 2 s + lane / 32, column quad lane % 32. Pass t covers PU
    // values of s (2 PU rows) of 32-row block t / PPB. Epilogues that read a
    // tensor (residual, gradient bucket, gate/up) keep two passes of loads in
    // flight and issue pass t + 2's loads before pass t's stores: a wave's
    // loads and stores retire in issue order, so a wait for a load then never
    // waits for an earlier store.
    constexpr bool LD = EPI == LC_EPI_RESIDUAL || EPI == LC_EPI_ACCUM_F32 || EPI == LC_EPI_SWIGLU_BWD;
    constexpr int PU = 4, PPB = 16 / PU, NP = WM / 32 * PPB;
    const int q = lane & 31;
    const int n = ncol0 + 4 * q;
    const int ncl = n < p.N ? n : p.N - 4;  // loads of columns past N read valid data (unused)
    auto row_of = [&](int t, int u) { return 2 * ((t % PPB) * PU + u) + (lane >> 5); };
    float4 xa[2][PU], ya[2][PU];
    auto issue = [&](int t, float4 (&x)[PU], float4 (&y)[PU]) {
      const int mrow0 = m0 + wm * WM + (t / PPB) * 32;
#pragma unroll
      for (int u = 0; u < PU; ++u) {
        const int mc = min(mrow0 + row_of(t, u), m_lim - 1);
        if constexpr (EPI == LC_EPI_RESIDUAL) x[u] = load4_dt(p.R, (int64_t)mc * p.ldr + ncl, r_dt);
        if constexpr (EPI == LC_EPI_ACCUM_F32)
          x[u] = *reinterpret_cast<const float4 *>(static_cast<const float *>(Cp) + (int64_t)mc * p.ldc + ncl);
        if constexpr (EPI == LC_EPI_SWIGLU_BWD) {
          x[u] = load4_dt(p.aux0, (int64_t)mc * p.ld_aux + ncl, aux_dt);
          y[u] = load4_dt(p.aux1, (int64_t)mc * p.ld_aux + ncl, aux_dt);
        }
      }
    };
    stage_block(0);
    if constexpr (LD) {
      issue(0, xa[0], ya[0]);
      issue(1, xa[1], ya[1]);
    }
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      if (t > 0 && t % PPB == 0) stage_block(t / PPB);  // after pass t - 1's LDS reads
      const int mrow0 = m0 + wm * WM + (t / PPB) * 32;
      float4 ra[PU], rb[PU];  // pass t's results (rb: SwiGLU backward's du)
#pragma unroll
      for (int u = 0; u < PU; ++u) {
        const float4 v = chunk(row_of(t, u), q);
        const float4 x = xa[t & 1][u], y = ya[t & 1][u];
        if constexpr (EPI == LC_EPI_SWIGLU_BWD) {
          const float o[4] = {v.x, v.y, v.z, v.w};
          const float gv[4] = {x.x, x.y, x.z, x.w};
          const float uv[4] = {y.x, y.y, y.z, y.w};
          float dg[4], du[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) swiglu_grad(o[e], gv[e], uv[e], dg[e], du[e]);
          ra[u] = make_float4(dg[0], dg[1], dg[2], dg[3]);
          rb[u] = make_float4(du[0], du[1], du[2], du[3]);
        } else if constexpr (LD) {
          ra[u] = make_float4(x.x + v.x, x.y + v.y, x.z + v.z, x.w + v.w);
        } else {
          ra[u] = v;
        }
      }
      if constexpr (LD) {
        if (t + 2 < NP) issue(t + 2, xa[t & 1], ya[t & 1]);
      }
#pragma unroll
      for (int u = 0; u < PU; ++u) {
        const int m = mrow0 + row_of(t, u);
        if (m >= m_lim || n >= p.N) continue;
        const int64_t oc = (int64_t)m * p.ldc + n;
        if constexpr (EPI == LC_EPI_ACCUM_F32) {
          *reinterpret_cast<float4 *>(static_cast<float *>(Cp) + oc) = ra[u];
        } else {
          store4_dt(Cp, oc, c_dt, ra[u].x, ra[u].y, ra[u].z, ra[u].w);
          if constexpr (EPI == LC_EPI_SWIGLU_BWD)
            store4_dt(Cp, oc + p.N, c_dt, rb[u].x, rb[u].y, rb[u].z, rb[u].w);
        }
      }
    }
  }
}

template <bool A_K, bool B_K, int EPI, int TM = 0>
lc_status launch_t(const GemmP &p, hipStream_t s) {
  // LC_GROUP_ROWS: an upper bound on the groups' row tiles (each group adds at
  // most one partial tile); LC_GROUP_K: every group has the full output grid
  unsigned grid = (unsigned)p.tiles_m * (unsigned)p.tiles_n;
  if (p.gmode == LC_GROUP_ROWS) grid = (unsigned)(p.tiles_m + p.ngroups) * (unsigned)p.tiles_n;
  if (p.gmode == LC_GROUP_K) grid *= (unsigned)p.ngroups;
  hipLaunchKernelGGL((gemm_bf16_kernel<A_K, B_K, EPI, TM>), dim3(grid), dim3(NT), 0, s, p);
  return check_launch("gemm_bf16_kernel");
}

}  // namespace

lc_status gemm_f32_launch(const lc_gemm_args &a, hipStream_t s);  // k_gemm_f32.hip

// the epilogue types this call uses (STORE_F32 and ACCUM_F32 imply fp32 C)
static int c_type(const lc_gemm_args &a) {
  return (a.epilogue == LC_EPI_STORE_F32 || a.epilogue == LC_EPI_ACCUM_F32) ? LC_FP32 : a.c_dtype;
}

static lc_status check_gemm_args(const lc_gemm_args &a) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return fail(LC_ERR_INVALID_ARG, "gemm: M, N, K must be > 0");
  if (a.M > INT32_MAX / 2 || a.N > INT32_MAX / 4 || a.K > INT32_MAX / 2)
    return fail(LC_ERR_UNSUPPORTED, "gemm: dimension too large");
  if (!a.A || !a.B || !a.C) return fail(LC_ERR_INVALID_ARG, "gemm: null operand");
  if (!aligned16(a.A) || !aligned16(a.B) || !aligned16(a.C))
    return fail(LC_ERR_INVALID_ARG, "gemm: operands must be 16-byte aligned");
  if (a.epilogue < LC_EPI_STORE || a.epilogue > LC_EPI_SWIGLU_BWD)
    return fail(LC_ERR_INVALID_ARG, "gemm: unknown epilogue %d", a.epilogue);
  if (!valid_dtype(c_type(a))) return fail(LC_ERR_INVALID_ARG, "gemm: unknown c_dtype");
  const bool bf = a.dtype == LC_BF16;
  if (bf && (a.lda % 8 || a.ldb % 8 || a.ldc % 8))
    return fail(LC_ERR_INVALID_ARG, "gemm: ld %% 8 != 0");
  const int64_t acols = a.a_kmajor ? a.K : a.M;
  const int64_t brows = a.epilogue == LC_EPI_SWIGLU ? 2 * a.N : a.N;
  const int64_t bcols = a.b_kmajor ? a.K : brows;
  if (a.lda < acols || a.ldb < bcols) return fail(LC_ERR_INVALID_ARG, "gemm: ld too small");
  if (a.epilogue == LC_EPI_RESIDUAL) {
    if (!a.R || !aligned16(a.R) || (bf && a.ldr % 8) || a.ldr < a.N || !valid_dtype(a.r_dtype))
      return fail(LC_ERR_INVALID_ARG, "gemm: bad residual operand");
  }
  if (a.epilogue == LC_EPI_SWIGLU || a.epilogue == LC_EPI_SWIGLU_BWD) {
    if (!a.aux0 || !a.aux1 || !aligned16(a.aux0) || !aligned16(a.aux1) ||
        (bf && a.ld_aux % 8) || a.ld_aux < a.N || !valid_dtype(a.aux_dtype))
      return fail(LC_ERR_INVALID_ARG, "gemm: bad gate/up operands");
    if (a.epilogue == LC_EPI_SWIGLU_BWD && a.ldc < 2 * a.N)
      return fail(LC_ERR_INVALID_ARG, "gemm: ldc < 2N for SWIGLU_BWD");
  } else if (a.ldc < a.N) {
    return fail(LC_ERR_INVALID_ARG, "gemm: ldc < N");
  }
  if (a.group_mode != LC_GROUP_NONE) {
    if (a.group_mode != LC_GROUP_ROWS && a.group_mode != LC_GROUP_K)
      return fail(LC_ERR_INVALID_ARG, "gemm: unknown group mode %d", a.group_mode);
    if (a.n_groups < 1 || a.n_groups > 64) return fail(LC_ERR_INVALID_ARG, "gemm: n_groups must be 1..64");
    if (!a.group_offsets || (reinterpret_cast<uintptr_t>(a.group_offsets) & 3))
      return fail(LC_ERR_INVALID_ARG, "gemm: group offsets must be a 4-byte aligned device array");
    if (a.epilogue == LC_EPI_ROPE || a.epilogue == LC_EPI_RESIDUAL)
      return fail(LC_ERR_UNSUPPORTED, "gemm: grouped products take STORE, ACCUM or SwiGLU epilogues");
    if (a.group_mode == LC_GROUP_ROWS && a.group_stride_b < 0)
      return fail(LC_ERR_INVALID_ARG, "gemm: negative group_stride_b");
    if (a.group_mode == LC_GROUP_K && (a.a_kmajor || a.b_kmajor || a.group_stride_c < 0))
      return fail(LC_ERR_UNSUPPORTED, "gemm: LC_GROUP_K needs m/n-major operands and group_stride_c >= 0");
  }
  if (a.epilogue == LC_EPI_ROPE && a.aux0) {
    if (!aligned16(a.aux0) || (bf && a.ld_aux % 8) || a.ld_aux < a.N || !valid_dtype(a.aux_dtype))
      return fail(LC_ERR_INVALID_ARG, "gemm: bad RoPE copy operand");
  }
  if (a.epilogue == LC_EPI_ROPE) {
    if (!a.rope_cos || !a.rope_sin || a.rope_seq <= 0 || a.rope_cols < 0 ||
        a.head_dim <= 0 || a.head_dim % 2 || a.rope_cols % a.head_dim || a.N % a.head_dim)
      return fail(LC_ERR_INVALID_ARG, "gemm: bad RoPE arguments");
  }
  return LC_OK;
}

// Output tile of a product: the one whose grid is expected to take the least time. One
// workgroup runs per compute unit with every tile size, so a grid of t tiles takes
// ceil(t / 256) rounds. Fitted to 2000 products of 64 x 336 to 8448 x 7728 outputs at K =
// 128 to 4096, ns per k and round: 21 with 256 x 256 tiles, 7.2 with 128 x 128, 3.8 with 64
// x 64, 1.9 with 32 x 32; a 256 x 256 round that fills only part of the chip takes 16.5 + 4.5
// x the part. And us per round besides (first loads, epilogue): 8, 3.8, 2.8 and 1.4, where
// the epilogue moves 8 to 12 bytes per output (fp32 gradients and residual rows, SwiGLU
// backward) 20, 8, 6 and 3. The larger tile does more work per round, the smaller ones fill
// the chip: 2048 x 2048 outputs (64, 256 or 1024 tiles) at K = 5632 take 107, 49 or 103 us; 2048 x
// 6144 at K = 2048 (192, 768 or 3072 tiles) 53, 60 or 135 us; 256 x 512 at K = 1408 (2, 8, 32 or
// 128 tiles) 31, 13, 9 or 6 us; 256 x 1536 at K = 512 with 64 or 32 (96 or 384 tiles) 6.5 or 6.8.
// A few tiles over whole rounds of 256: 2304 x 7424 (261 or 1044 tiles) NT at K = 128, 512, 2048
// 23, 37, 94 or 25, 38, 88 us; 3072 x 10880 (516 or 2040) at K = 2048 NT 150 or 161, SwiGLU
// backward 213 or 253; 3072 x 5632 (264 or 1056) with a residual at K = 1024 66 or 58. The
// choice depends on sizes, layout, grouping and those two epilogues only, so an accumulated
// and a stored gradient add in one order (the same bits).
static int pick_tile(const lc_gemm_args &a) {
  const int64_t N = a.epilogue == LC_EPI_SWIGLU ? 2 * a.N : a.N;
  auto tiles = [&](int64_t t) {
    int64_t tm = (a.M + t - 1) / t;
    const int64_t tn = (N + t - 1) / t;
    // grouped rows: about half a partial tile-row per group besides
    if (a.group_mode == LC_GROUP_ROWS) tm += (a.n_groups + 1) / 2;
    return tm * tn * (a.group_mode == LC_GROUP_K ? a.n_groups : 1);
  };
  constexpr int64_t CU = 256;
  // 0.1 ns: k (a group's share of it) times the round's rate, and what a round costs besides
  const int64_t K = a.group_mode == LC_GROUP_K ? a.K / a.n_groups : a.K;
  const bool heavy = (!a.a_kmajor && !a.b_kmajor) || a.epilogue == LC_EPI_RESIDUAL ||
                     a.epilogue == LC_EPI_SWIGLU_BWD;
  const int64_t f256 = heavy ? 200000 : 80000, f128 = heavy ? 80000 : 38000, f64 = heavy ? 60000 : 28000;
  const int64_t t256 = tiles(256), part = t256 % CU;
  const int64_t c256 = t256 / CU * (210 * K + f256) + (part ? (165 + 45 * part / CU) * K + f256 : 0);
  const int64_t c128 = (tiles(128) + CU - 1) / CU * (72 * K + f128);
  const int64_t c64 = (tiles(64) + CU - 1) / CU * (38 * K + f64);
  const int64_t c32 = (tiles(32) + CU - 1) / CU * (19 * K + f64 / 2);
  int t = c128 < c256 ? 128 : 256;
  if (c64 < c128 && c64 < c256) t = 64;
  if (c32 < c64 && c32 < c128 && c32 < c256) t = 32;
  // a launch holds fewer than 2^32 work-items (of very wide grouped outputs only the
  // largest tile's upper bound of workgroups fits)
  auto fits = [&](int64_t tile) {
    const int64_t tm = (a.M + tile - 1) / tile + (a.group_mode == LC_GROUP_ROWS ? a.n_groups : 0);
    const int64_t n = tm * ((N + tile - 1) / tile) * (a.group_mode == LC_GROUP_K ? a.n_groups : 1);
    return n * (tile >= 128 ? 512 : 256) <= (int64_t)UINT32_MAX;
  };
  while (t < 256 && !fits(t)) t *= 2;
  return t;
}

// The bf16 kernels' own limits, and their launch parameters.
static lc_status bf16_params(const lc_gemm_args &a, GemmP *out) {
  if (a.dtype != LC_BF16) return fail(LC_ERR_INVALID_ARG, "gemm: A/B dtype must be fp32 or bf16");
  // layout limits of the bf16 kernel: 16-byte rows along every contiguous extent
  if (a.N % 8) return fail(LC_ERR_UNSUPPORTED, "gemm bf16: N %% 8 != 0");
  if ((a.a_kmajor || a.b_kmajor) && a.K % 8) return fail(LC_ERR_UNSUPPORTED, "gemm bf16: K %% 8 != 0");
  if (!a.a_kmajor && a.M % 8) return fail(LC_ERR_UNSUPPORTED, "gemm bf16: M %% 8 != 0 (A not k-major)");
  if (a.epilogue == LC_EPI_ROPE && a.head_dim != 128)
    return fail(LC_ERR_UNSUPPORTED, "gemm bf16: RoPE epilogue needs head_dim 128");
  if (a.epilogue == LC_EPI_SWIGLU && (a.N % 64 || !a.b_kmajor))
    return fail(LC_ERR_UNSUPPORTED, "gemm bf16: SwiGLU needs N %% 64 == 0 and k-major B");
  if (a.epilogue == LC_EPI_ROPE && (!aligned16(a.rope_cos) || !aligned16(a.rope_sin)))
    return fail(LC_ERR_INVALID_ARG, "gemm: RoPE tables must be 16-byte aligned");

  GemmP &p = *out;
  p = GemmP{};
  p.A = static_cast<const bf16_t *>(a.A);
  p.B = static_cast<const bf16_t *>(a.B);
  p.C = a.C;
  p.R = a.R;
  p.aux0 = a.aux0;
  p.aux1 = a.aux1;
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
  // byte extents for the buffer descriptors (offsets are 32-bit)
  const int64_t brows = a.epilogue == LC_EPI_SWIGLU ? 2 * a.N : a.N;
  const int64_t a_ext = a.a_kmajor ? (a.M - 1) * a.lda + a.K : (a.K - 1) * a.lda + a.M;
  const int64_t b_ext = a.b_kmajor ? (brows - 1) * a.ldb + a.K : (a.K - 1) * a.ldb + brows;
  if (a_ext * 2 >= (int64_t)OOB || b_ext * 2 >= (int64_t)OOB)
    return fail(LC_ERR_UNSUPPORTED, "gemm bf16: an operand spans 2 GiB or more");
  p.a_bytes = (uint32_t)(a_ext * 2);
  p.b_bytes = (uint32_t)(b_ext * 2);
  p.tiles_m = (int)((a.M + BM - 1) / BM);
  p.tiles_n = a.epilogue == LC_EPI_SWIGLU ? (int)((a.N + BN / 2 - 1) / (BN / 2))
                                          : (int)((a.N + BN - 1) / BN);
  // 4 tile-rows per group, 3 when the grid has an odd number of tile-columns:
  // the fastest walk measured over the stage's shapes among groups of 2 to 8
  // and 16 (4 against 8: 1-2% faster on the 16-column dn2, dn1 and dW13
  // products, equal on the rest; 3 against 4 on the 43-column SwiGLU backward
  // and dW2 products: 1.5% and 3% faster)
  p.group = (p.tiles_n & 1) ? 3 : 4;
  p.gmode = a.group_mode;
  p.ngroups = a.group_mode == LC_GROUP_NONE ? 1 : a.n_groups;
  p.goff = a.group_offsets;
  p.gstride_b = a.group_stride_b;
  p.gstride_c = a.group_stride_c;
  p.rope_seq = a.rope_seq;
  p.rope_cols = a.rope_cols;
  p.c_dt = c_type(a);
  p.r_dt = a.r_dtype;
  p.aux_dt = a.aux_dtype;
  return LC_OK;
}

lc_status gemm_launch(const lc_gemm_args &a, hipStream_t s) {
  LC_TRY(check_gemm_args(a));
  if (a.dtype == LC_FP32 && a.group_mode != LC_GROUP_NONE)
    return fail(LC_ERR_UNSUPPORTED, "gemm fp32: grouped products need bf16 operands");
  if (a.dtype == LC_FP32) {
    if (c_type(a) != LC_FP32 || (a.epilogue == LC_EPI_RESIDUAL && a.r_dtype != LC_FP32) ||
        ((a.epilogue == LC_EPI_SWIGLU || a.epilogue == LC_EPI_SWIGLU_BWD) &&
         a.aux_dtype != LC_FP32))
      return fail(LC_ERR_UNSUPPORTED, "gemm fp32: every tensor must be fp32");
    return gemm_f32_launch(a, s);
  }
  GemmP p;
  LC_TRY(bf16_params(a, &p));
  const int tile = pick_tile(a);
  if (tile != BM) return gemm_tile_launch(p, a, tile, s);
  const bool ak = a.a_kmajor != 0, bk = a.b_kmajor != 0;
  switch (a.epilogue) {
    case LC_EPI_STORE:
    case LC_EPI_STORE_F32:
      if (ak && bk) return launch_t<true, true, LC_EPI_STORE>(p, s);
      if (ak && !bk) return launch_t<true, false, LC_EPI_STORE>(p, s);
      if (!ak && !bk) return launch_t<false, false, LC_EPI_STORE>(p, s);
      break;
    case LC_EPI_ACCUM_F32:
      if (ak && bk) return launch_t<true, true, LC_EPI_ACCUM_F32>(p, s);
      if (!ak && !bk) return launch_t<false, false, LC_EPI_ACCUM_F32>(p, s);
      break;
    case LC_EPI_RESIDUAL:
      if (ak && bk && p.c_dt == LC_FP32 && p.r_dt == LC_FP32)
        return launch_t<true, true, LC_EPI_RESIDUAL, 1>(p, s);
      if (ak && bk) return launch_t<true, true, LC_EPI_RESIDUAL>(p, s);
      break;
    case LC_EPI_ROPE:
      if (ak && bk && p.c_dt == LC_FP16 && (!p.aux0 || p.aux_dt == LC_BF16))
        return launch_t<true, true, LC_EPI_ROPE, 1>(p, s);
      if (ak && bk) return launch_t<true, true, LC_EPI_ROPE>(p, s);
      break;
    case LC_EPI_SWIGLU:
      if (ak && bk && p.c_dt == LC_BF16 && p.aux_dt == LC_FP32)
        return launch_t<true, true, LC_EPI_SWIGLU, 1>(p, s);
      if (ak && bk) return launch_t<true, true, LC_EPI_SWIGLU>(p, s);
      break;
    case LC_EPI_SWIGLU_BWD:
      if (ak && !bk && p.c_dt == LC_BF16 && p.aux_dt == LC_FP32)
        return launch_t<true, false, LC_EPI_SWIGLU_BWD, 1>(p, s);
      if (ak && !bk) return launch_t<true, false, LC_EPI_SWIGLU_BWD>(p, s);
      if (ak && bk) return launch_t<true, true, LC_EPI_SWIGLU_BWD>(p, s);
      break;
  }
  return fail(LC_ERR_UNSUPPORTED, "gemm bf16: layout (a_kmajor=%d, b_kmajor=%d) not built for "
              "epilogue %d", (int)ak, (int)bk, a.epilogue);
}

// An input gradient x and a weight gradient w of one backward step that do not depend
// on each other: one launch where both are products of 32 or 64 tiles (bf16) or
// eight-wave 32 tiles (fp32), which leave most of the chip idle (small bf16 step 1012 ->
// 955 us, tiny fp32 step 797 -> 648). A 128 or 256 tile has workgroups of 512 threads, the
// 64 and 32 tiles of 256; two products of the larger ones could share a launch, but fill
// the chip by themselves more often. The results are those of the two launches.
lc_status gemm_pair_launch(const lc_gemm_args &x, const lc_gemm_args &w, hipStream_t s) {
  const bool form = x.dtype == w.dtype && x.group_mode == LC_GROUP_NONE && w.group_mode == LC_GROUP_NONE &&
                    x.a_kmajor && !x.b_kmajor && !w.a_kmajor && !w.b_kmajor &&
                    (x.epilogue == LC_EPI_STORE || x.epilogue == LC_EPI_SWIGLU_BWD) &&
                    w.epilogue == LC_EPI_ACCUM_F32;
  if (form) {
    LC_TRY(check_gemm_args(x));
    LC_TRY(check_gemm_args(w));
    if (x.dtype == LC_FP32 && c_type(x) == LC_FP32 && (x.epilogue == LC_EPI_STORE || x.aux_dtype == LC_FP32)) {
      bool done = false;
      LC_TRY(gemm_f32_pair_launch(x, w, s, &done));
      if (done) return LC_OK;
    } else if (x.dtype == LC_BF16 && (x.epilogue == LC_EPI_STORE || (c_type(x) == LC_BF16 && x.aux_dtype == LC_FP32))) {
      const int tx = pick_tile(x), tw = pick_tile(w);
      if (tx <= 64 && tw <= 64) {
        GemmP px, pw;
        LC_TRY(bf16_params(x, &px));
        LC_TRY(bf16_params(w, &pw));
        return gemm_tile_pair_launch(px, x.epilogue, tx, pw, tw, s);
      }
    }
  }
  LC_TRY(gemm_launch(x, s));
  return gemm_launch(w, s);
}

}  // namespace lc

extern "C" lc_status lc_gemm(const lc_gemm_args *args, void *stream) {
  if (!args) return lc::fail(LC_ERR_INVALID_ARG, "gemm: null args");
  return lc::gemm_launch(*args, static_cast<hipStream_t>(stream));
}

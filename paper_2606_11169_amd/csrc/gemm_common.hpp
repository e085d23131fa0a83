// Device code shared by the GEMM kernels: launch parameters, tile lookup, the
// epilogues' arithmetic and type mixes.
#pragma once

#include "common.hpp"
#include "lds_dma.hpp"

#include <type_traits>

namespace lc {

struct GemmP {
  const bf16_t *A;
  const bf16_t *B;
  void *C;
  const void *R;
  void *aux0;
  void *aux1;
  const float *rcos;
  const float *rsin;
  int64_t lda, ldb, ldc, ldr, ld_aux;
  uint32_t a_bytes, b_bytes;  // byte extent of each operand (< 2^31)
  int M, N, K;  // N: output columns (SwiGLU: gate/up width)
  int tiles_m, tiles_n;
  int group;  // tile-rows per group of the tile walk
  int gmode, ngroups;
  const int32_t *goff;
  int64_t gstride_b, gstride_c;
  int rope_seq, rope_cols;
  int c_dt, r_dt, aux_dt;
};

namespace {

constexpr int RUN = 1024 + 32;  // LDS-DMA runs: one 1 KiB load per wave instruction, 32 bytes of padding
constexpr uint32_t OOB = 0x80000000u;    // buffer offset beyond every operand: reads 0

typedef __attribute__((address_space(3))) bf16x8_v lds_v8;
typedef __attribute__((address_space(3))) s16x4_v lds_v4;

// at most LEFT of this wave's loads in flight and its LDS reads done, then the
// workgroup's barrier
template <int LEFT>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(LEFT) : "memory");
}

// Scheduling pattern for one k-step: the NRD LDS reads of the next k-step
// spread over the NMF MFMAs of this one (reads first, as evenly as possible).
template <int NRD, int NMF, int I = 0>
__device__ __forceinline__ void interleave_steps() {
  if constexpr (I < NMF) {
    constexpr int r = NRD / NMF + (I < NRD % NMF ? 1 : 0);
    if constexpr (r > 0) __builtin_amdgcn_sched_group_barrier(0x100, r, 0);  // LDS reads
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                       // one MFMA
    interleave_steps<NRD, NMF, I + 1>();
  }
}

// Element types of an epilogue's tensors: TM = 0 takes them from the run-time
// values in GemmP (uniform branches around every access); TM = 1 fixes them to
// the decoder stage's own mix for EPI (the branch-free accesses let the
// compiler keep the epilogue's loads in flight instead of waiting at each
// branch): residual add fp32 R and C, SwiGLU and its backward fp32 gate/up and
// bf16 C, RoPE fp16 C and bf16 copy. The host takes TM = 1 when the call's
// types are exactly that mix.
template <int EPI, int TM>
struct EpiTypes {
  static constexpr bool RES = EPI == LC_EPI_RESIDUAL, SWI = EPI == LC_EPI_SWIGLU || EPI == LC_EPI_SWIGLU_BWD;
  static constexpr bool ROPE = EPI == LC_EPI_ROPE;
  static constexpr int C = TM == 0 ? -1 : RES ? LC_FP32 : SWI ? LC_BF16 : ROPE ? LC_FP16 : -1;
  static constexpr int R = TM == 0 ? -1 : RES ? LC_FP32 : -1;
  static constexpr int X = TM == 0 ? -1 : SWI ? LC_FP32 : ROPE ? LC_BF16 : -1;
};

// The epilogues' arithmetic, with the fused operations written out: left to the compiler,
// which product of a sum is fused (and so its rounding) differed from kernel to kernel, and
// a call's result with the tile that it got.
// RoPE: the pair (x, y) turned by the angle of cosine c and sine s
__device__ __forceinline__ void rope_pair(float &x, float &y, float c, float s) {
  const float a = __builtin_fmaf(x, c, -(y * s));
  y = __builtin_fmaf(y, c, x * s);
  x = a;
}
// SwiGLU backward: gate and up gradients of the activation's gradient v
__device__ __forceinline__ void swiglu_grad(float v, float g, float u, float &dg, float &du) {
  const float s = sigmoidf_(g);
  dg = v * u * s * __builtin_fmaf(g, 1.0f - s, 1.0f);
  du = v * g * s;
}

// Where the tile of workgroup wg of nwg lies: false when it has none (uniform across
// the workgroup). Workgroups are dispatched round-robin over the 8 XCDs; each XCD
// gets a contiguous run of tiles, walked in groups of p.group tile-rows
// (chosen by the host) so that neighbouring workgroups share A rows and B
// columns in the XCD's L2.
struct Tile {
  int m0, tn;         // first row, tile column
  int m_lim;          // rows at or past it are not this tile's
  int kbeg, kend;
  const bf16_t *B;
  void *C;
};
// ROWS: grouped rows or not where the kernel is for one of them (128 tile), -1 by p.gmode
template <int BM, int ROWS = -1>
__device__ __forceinline__ bool find_tile(const GemmP &p, int wg, int nwg, Tile &t) {
  // Workgroup wg runs on XCD wg % 8; mapped, XCD x takes a run of n / 8 tiles (the first n %
  // 8 one more). The 256, 64 and 32 tiles: grids of a multiple of 8 (others +-5%). The 128
  // tile, which reads its operands twice as often as the 256 tile, also other grids of over a
  // round with k enough for it to matter (1044 tiles at K = 4096 161 us, 197 in launch order,
  // 356 tiles at K = 2048 42 and 58; 975 at K = 128 22.7 and 21.1), and grouped rows over
  // the tiles that there are, found with a lane per group (at most 64): the grid is an upper
  // bound, and a map over it leaves the last XCD the empty ones (60 groups of 10 rows 18 us, 13
  // in launch order; 16 experts of about 690 rows x 1280 at K = 576 46 us in launch order, now
  // 35; 8 of about 1290 x 1920 at K = 1856 130, now 93). The map is selects, not a branch, with which
  // the compiler waits for all of a stage's fragments at once in some epilogues' main loops
  // (residual at K = 4096, 76 tiles: 30.9 us, selects 29.7).
  if constexpr (BM == 128) {
    const bool rows = ROWS < 0 ? p.gmode == LC_GROUP_ROWS : ROWS > 0;
    bool map = (nwg & 7) == 0 || (nwg > 264 && p.K >= 512);
    int n = nwg, first = 0, last = 0, end = 0, nt = 0;
    if (rows) {
      const int lane = threadIdx.x & 63;
      if (lane < p.ngroups) {
        first = min(max(p.goff[lane], 0), p.M);
        last = min(max(p.goff[lane + 1], first), p.M);
      }
      nt = end = (last - first + BM - 1) / BM;
#pragma unroll
      for (int d = 1; d < 64; d *= 2) {
        const int e = __shfl_up(end, d);
        end += lane >= d ? e : 0;
      }
      n = __builtin_amdgcn_readlane(end, 63) * p.tiles_n;
      if (wg >= n) return false;
      map = n > 264 && p.K >= 512;
    }
    const int x = map ? wg & 7 : 0;
    wg = x * (n >> 3) + min(x, n & 7) + (map ? wg >> 3 : wg);
    if (rows) {  // row tiles in the groups' order, all columns of one first
      const int slot = wg / p.tiles_n, g = __builtin_ctzll(__ballot(end > slot));
      t.tn = wg % p.tiles_n;
      t.m0 = __builtin_amdgcn_readlane(first, g) + (slot - __builtin_amdgcn_readlane(end - nt, g)) * BM;
      t.m_lim = __builtin_amdgcn_readlane(last, g);
      t.kbeg = 0;
      t.kend = p.K;
      t.B = p.B + (int64_t)g * p.gstride_b;
      t.C = p.C;
      return true;
    }
  } else if ((nwg & 7) == 0) {
    wg = (wg & 7) * (nwg >> 3) + (wg >> 3);
  }
  t.m_lim = p.M;
  t.kbeg = 0;
  t.kend = p.K;
  t.B = p.B;
  t.C = p.C;
  if (BM != 128 && p.gmode == LC_GROUP_ROWS) {
    // tile slot wg / tiles_n walks the groups' row tiles in order; slots past
    // the last group's tiles have nothing to do (the grid is an upper bound)
    t.tn = wg % p.tiles_n;
    int slot = wg / p.tiles_n, g = 0, lo = 0, hi = 0;
    for (; g < p.ngroups; ++g) {
      lo = min(max(p.goff[g], 0), p.M);
      hi = min(max(p.goff[g + 1], lo), p.M);
      const int nt = (hi - lo + BM - 1) / BM;
      if (slot < nt) break;
      slot -= nt;
    }
    if (g == p.ngroups) return false;
    t.m0 = lo + slot * BM;
    t.m_lim = hi;
    t.B = p.B + (int64_t)g * p.gstride_b;
    return true;
  }
  if (p.gmode == LC_GROUP_K) {
    const int per = p.tiles_m * p.tiles_n, g = wg / per;
    wg -= g * per;
    t.kbeg = min(max(p.goff[g], 0), p.K);
    t.kend = min(max(p.goff[g + 1], t.kbeg), p.K);
    t.C = static_cast<char *>(p.C) + (int64_t)g * p.gstride_c * (p.c_dt == LC_FP32 ? 4 : 2);
  }
  const int per_group = p.group * p.tiles_n;
  const int first_m = (wg / per_group) * p.group;
  const int gsz = min(p.tiles_m - first_m, p.group);
  t.m0 = (first_m + (wg % per_group) % gsz) * BM;
  t.tn = (wg % per_group) / gsz;
  return true;
}

}  // namespace

// k_gemm_tile.hip: the products whose grid of 256 x 256 tiles would leave most
// of the chip idle (tile = 128, 64 or 32)
lc_status gemm_tile_launch(GemmP p, const lc_gemm_args &a, int tile, hipStream_t s);
// Two products of tiles 32 or 64 in one launch: x an input gradient (A k-major, B
// not; STORE, or SWIGLU_BWD with the stage's types), w a weight gradient (neither
// k-major; ACCUM_F32).
lc_status gemm_tile_pair_launch(GemmP x, int x_epi, int x_tile, GemmP w, int w_tile, hipStream_t s);
// The fp32 pair: LC_OK and *done set if both take the ring's eight-wave 32 tile.
lc_status gemm_f32_pair_launch(const lc_gemm_args &x, const lc_gemm_args &w, hipStream_t s, bool *done);

}  // namespace lc

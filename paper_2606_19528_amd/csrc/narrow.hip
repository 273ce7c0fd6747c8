// narrow.hip -- the LoRA linear over few tokens (bf16): one launch per
// direction in which a workgroup computes a BM x BN tile of the output over
// one range of the reduction, and with it the rank-r product of its rows.
//
// At a few tokens the product is a read of W: the tiles of the general path
// cover a fraction of the CUs, each streams its panel with few loads in
// flight, and a rank-r pass over whole rows runs ahead of them.  Here the
// reduction is split as well, until the workgroups cover the chip, and every
// workgroup appends the r rank columns to its tile (32 or 64 more columns of
// an operand that L2 holds), so that no workgroup waits for another: u (or
// du) is complete wherever a tile is.
//   forward   [y | u]  = x [W ; A]^T,    then y  += E(s u) B^T
//   backward  [dx | du] = dy [W | B],    then dx += E(s du) A, dA = E(s du)^T x;
//             dB = s dy^T u on further workgroups of the launch
// A tile's parts meet in the workspace: each stores its fp32 sums (16-byte
// stores at device scope), waits until they have completed and raises a flag;
// one part that sees all flags up adds all the sums in ascending order and
// finishes the tile.  The same meeting joins the row tiles' shares of dA.  So
// results do not depend on the order of arrival.
//
// The main loop streams 64-deep stages through an LDS ring with direct-to-LDS
// loads in the layouts of gemm_kernel.hpp; the four waves take one 16-deep
// k-slice each and are summed through LDS at the end.
#include <algorithm>

#include "kernels.hpp"
#include "launch.hpp"
#include "meet.hpp"

namespace lora {

typedef short nw_i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) nw_i16x4 nw_lds_i16x4;

constexpr int NW_BKE = 64;  // k per stage

template <int V>
struct NwIC {
  static constexpr int value = V;
};

// The flags of a meeting of n <= 64 workgroups (meet.hpp) as one wave reads and
// writes them, a word a lane.  (A counter instead of flags serialised the
// arrivals, 1.1 us each; only those that see all flags up meet in the exchange.)
struct NwFlags {
  meet_word *w;
  int lane;
  __device__ void raise(int i, meet_word tag) {
    if (lane == 0) __hip_atomic_store(w + i, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ void settle() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
  __device__ bool all_up(int n, meet_word tag) {
    const meet_word f = lane < n ? __hip_atomic_load(w + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : tag;
    return __ballot(f != tag) == 0;
  }
  // (the return value is lane 0's)
  __device__ meet_word lower(int n) {
    if (lane == 0) return __hip_atomic_exchange(w, meet_word(0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lane < n) __hip_atomic_store(w + lane, meet_word(0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return 0;
  }
};

// 16 bytes at device scope (sc1: past the caches that other XCDs do not see).
constexpr int NW_SC1 = 16;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t nw_rsrc(const void *p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)p, (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ void nw_store(__amdgpu_buffer_rsrc_t rs, int off, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, off, 0, NW_SC1);
}
__device__ __forceinline__ f32x4 nw_load(__amdgpu_buffer_rsrc_t rs, int off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, NW_SC1));
}

// Tiles of 32 x 64, four waves; RB blocks of 32 rank columns, ring of NBUF
// stages (64 KB of LDS: two workgroups per CU).  The stages arrive at the rate
// of a CU's load path (16 KB in about 0.13 us, 60 bytes per clock), whatever
// the ring's depth; larger tiles (64 x 64, 32 x 128, 128 x 128 with eight
// waves) load less in all but spread over fewer CUs and end later at every
// size tried: 64 tokens of 3072 -> 3072, fwd + bwd, 34 against 37 - 45 us.
constexpr int NW_BM = 32, NW_BN = 64;
template <int RB, int NBUF, bool KMAJ>
__global__ __launch_bounds__(256) void narrow_kernel(NarrowArgs a) {
  constexpr int BM = NW_BM, BN = NW_BN, NWV = 4, NT = 64 * NWV;
  constexpr int FN = BN / 32;  // blocks of 32 columns; one of 32 rows
  constexpr int A_B = BM * 128, B_B = BN * 128, U_B = RB * 32 * 128, STAGE = A_B + B_B + U_B;
  constexpr int A_PW = A_B / 1024 / NWV, B_PW = B_B / 1024 / NWV;  // loads per wave per stage
  constexpr int U_PC = U_B / 1024;                                 // 1 KB pieces of the rank columns
  constexpr int U_PW = (U_PC + NWV - 1) / NWV;
  static_assert(A_PW * 1024 * NWV == A_B && B_PW * 1024 * NWV == B_B && (U_PC % NWV == 0 || U_PC < NWV), "whole loads");
  constexpr int C = BN + RB * 32;  // columns of the summed tile
  constexpr int LDF = C + 4;       // its padded LDS row (floats)
  constexpr int PLANE = BM * LDF;  // one wave's share of it
  constexpr int FIN = NWV * PLANE * 4;
  constexpr int LDS = NBUF * STAGE > FIN ? NBUF * STAGE : FIN;
  constexpr uint32_t OOB = 0x80000000u;
  __shared__ __align__(16) char smem[LDS];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wv;  // the wave's k-slice of a stage

  // Workgroup -> (row tile, column tile, part).  The row tiles of one column
  // tile and part, which read the same W, follow one another on one XCD.
  const int units = a.tiles_n * a.parts, unit_wgs = (units + 7) / 8 * 8 * a.tiles_m;
  const int r = a.r, lrow = lane & 31, half = lane >> 5;
  if constexpr (KMAJ && RB > 0) {
    if ((int)blockIdx.x >= unit_wgs) {
      // dB = s dy^T u: each wave 32 columns of dy by the r rank indices, the
      // reduction over all tokens on matrix cores, u rounded to bf16.  Every
      // load of a half of the tokens is in flight at once.
      const uint16_t *dy = (const uint16_t *)a.X;
      const int nb = (((int)blockIdx.x - unit_wgs) * NWV + wv) * 32, n = nb + lrow;
      if (nb >= a.K) return;
#pragma unroll
      for (int jb = 0; jb < RB; ++jb) {
        const int j = jb * 32 + lrow;
        f32x16 d = f32x16{};
        for (int t0 = 0; t0 < a.T; t0 += 64) {
          uint32_t lo[4][4], hi[4][4];
          float f[4][8];
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int m = t0 + 16 * s + 8 * half;
#pragma unroll
            for (int h = 0; h < 4; ++h) {
              lo[s][h] = n < a.K && m + 2 * h < a.T ? dy[(int64_t)(m + 2 * h) * a.K + n] : 0;
              hi[s][h] = n < a.K && m + 2 * h + 1 < a.T ? dy[(int64_t)(m + 2 * h + 1) * a.K + n] : 0;
            }
#pragma unroll
            for (int t = 0; t < 8; ++t) f[s][t] = j < r && m + t < a.T ? a.u_in[(int64_t)(m + t) * r + j] : 0.0f;
          }
#pragma unroll
          for (int s = 0; s < 4; ++s)
            mma32(BF16(), d, u32x4{lo[s][0] | (hi[s][0] << 16), lo[s][1] | (hi[s][1] << 16), lo[s][2] | (hi[s][2] << 16),
                                   lo[s][3] | (hi[s][3] << 16)}, pack_vec(BF16(), f[s]));
        }
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          const int row = nb + 8 * (x / 4) + 4 * half + x % 4;
          if (row < a.K && j < r) a.dB[(int64_t)row * r + j] = a.scale * d[x];
        }
      }
      return;
    }
  }
  const int local = (int)blockIdx.x >> 3;
  const int unit = __builtin_amdgcn_readfirstlane((local / a.tiles_m) * 8 + ((int)blockIdx.x & 7));
  if (unit >= units) return;
  const int mt = __builtin_amdgcn_readfirstlane(local % a.tiles_m);
  const int part = __builtin_amdgcn_readfirstlane(unit % a.parts), nt = __builtin_amdgcn_readfirstlane(unit / a.parts);
  const int m0 = mt * BM, n0 = nt * BN;
  const int k_lo = part * a.part_k, k_hi = min(a.K, k_lo + a.part_k);
  const int nst = (k_hi - k_lo + NW_BKE - 1) / NW_BKE;

  // ---- loads -------------------------------------------------------------------
  const int mrows = min(BM, a.T - m0);
  const __amdgpu_buffer_rsrc_t rsX = nw_rsrc((const uint16_t *)a.X + (int64_t)m0 * a.K, (int64_t)mrows * a.K * 2);
  // row-major: the tile's W rows, and the r rows of A; k-major: the part's W
  // rows from column n0 on, and the part's rows of B, contiguous
  const int ncols = min(BN, a.N - n0);  // 0 when only u is wanted
  const __amdgpu_buffer_rsrc_t rsW =
      KMAJ ? nw_rsrc((const uint16_t *)a.W + (int64_t)k_lo * a.N + n0,
                     a.out ? ((int64_t)(k_hi - k_lo) * a.N - n0) * 2 : 0)
           : nw_rsrc((const uint16_t *)a.W + (int64_t)n0 * a.K, ncols > 0 ? (int64_t)ncols * a.K * 2 : 0);
  const __amdgpu_buffer_rsrc_t rsV = KMAJ ? nw_rsrc((const uint16_t *)a.V + (int64_t)k_lo * r, (int64_t)(k_hi - k_lo) * r * 2)
                                          : nw_rsrc(a.V, (int64_t)r * a.K * 2);
  // k-contiguous rows of 128 bytes: load q covers rows 8q .. 8q + 7, chunk c
  // of row i at c ^ (i & 7) ^ ((i >> 3) & 1)
  auto row_off = [&](int q, int64_t ld, int &k) -> uint32_t {
    const int i = 8 * q + (lane >> 3), c = (lane & 7) ^ (lane >> 3) ^ (q & 1);
    k = c * 8;
    return (uint32_t)(i * ld * 2 + c * 16);
  };
  uint32_t oX[A_PW], oW[B_PW], oV[U_PW > 0 ? U_PW : 1];
  int kX[A_PW], kW[B_PW], kV[U_PW > 0 ? U_PW : 1];
#pragma unroll
  for (int i = 0; i < A_PW; ++i) oX[i] = row_off(wv + i * NWV, a.K, kX[i]);
#pragma unroll
  for (int i = 0; i < B_PW; ++i) {
    const int q = wv + i * NWV;
    if constexpr (!KMAJ) {
      oW[i] = row_off(q, a.K, kW[i]);
    } else {
      // k-rows of 2 BN bytes, swizzled so that the transposed reads of four
      // k-rows fall into distinct banks
      const int row = 8 * q + (lane >> 3);
      const int c = (lane & 7) ^ (4 * ((row >> 1) & 1));
      kW[i] = row;
      oW[i] = c * 8 < ncols ? (uint32_t)(row * (int64_t)a.N * 2 + c * 16) : OOB;
    }
  }
#pragma unroll
  for (int i = 0; i < U_PW; ++i) {
    const int q = wv + i * NWV;
    if constexpr (!KMAJ) {
      oV[i] = row_off(q, a.K, kV[i]);
    } else {
      const int byte = q * 1024 + lane * 16;  // of the stage's [64][r] block
      kV[i] = byte;
      oV[i] = (uint32_t)byte;
    }
  }
  const bool has_u = U_PC >= NWV || wv < U_PC;  // this wave loads pieces of the rank columns
  auto issue = [&](int st) __attribute__((always_inline)) {
    char *buf = smem + (st % NBUF) * STAGE;
    const int kr = k_hi - k_lo - st * NW_BKE;  // k left (<= 0 past the end: zeros)
    const int ks = (k_lo + st * NW_BKE) * 2;
    // (the resources bound rows and columns; k past the part is masked here)
#pragma unroll
    for (int i = 0; i < A_PW; ++i) dma16(rsX, buf + (wv + i * NWV) * 1024, kX[i] < kr ? oX[i] : OOB, ks);
#pragma unroll
    for (int i = 0; i < B_PW; ++i) {
      char *dst = buf + A_B + (wv + i * NWV) * 1024;
      if constexpr (!KMAJ) dma16(rsW, dst, kW[i] < kr ? oW[i] : OOB, ks);
      else dma16(rsW, dst, kW[i] < kr ? oW[i] : OOB, kr > 0 ? (int)((int64_t)st * NW_BKE * a.N * 2) : 0);
    }
    if (has_u) {
#pragma unroll
      for (int i = 0; i < U_PW; ++i) {
        char *dst = buf + A_B + B_B + (wv + i * NWV) * 1024;
        if constexpr (!KMAJ) dma16(rsV, dst, kV[i] < kr ? oV[i] : OOB, ks);
        else dma16(rsV, dst, kV[i] < min(kr, NW_BKE) * 2 * r ? oV[i] : OOB, kr > 0 ? st * NW_BKE * 2 * r : 0);
      }
    }
  };

  // ---- main loop -----------------------------------------------------------------
  f32x16 acc[FN], accu[RB > 0 ? RB : 1];
#pragma unroll
  for (int j = 0; j < FN; ++j) acc[j] = f32x16{};
#pragma unroll
  for (int j = 0; j < RB; ++j) accu[j] = f32x16{};
  const int ca = ((2 * wk + half) ^ (lrow & 7) ^ ((lrow >> 3) & 1)) * 16;  // the lane's chunk of its rows
  const int iq = lane & 15, gq = lane >> 4;
  const int tr_k = 16 * wk + 8 * (gq >> 1) + (iq >> 2), tr_n = 16 * (gq & 1) + 4 * (iq & 3);
  auto tr_read = [&](const char *p, int row_bytes) __attribute__((always_inline)) -> u32x4 {
    const nw_i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((nw_lds_i16x4 *)p);
    const nw_i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((nw_lds_i16x4 *)(p + 4 * row_bytes));
    return u32x4{__builtin_bit_cast(uint2, lo).x, __builtin_bit_cast(uint2, lo).y, __builtin_bit_cast(uint2, hi).x,
                 __builtin_bit_cast(uint2, hi).y};
  };
  struct Frags {
    u32x4 a, b[FN], u[RB > 0 ? RB : 1];
  };
  auto read_frags = [&](int st, Frags &f) __attribute__((always_inline)) {
    const char *sA = smem + (st % NBUF) * STAGE, *sB = sA + A_B, *sU = sB + B_B;
    f.a = ld16(sA + lrow * 128 + ca);
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = j * 32;
      if constexpr (!KMAJ) {
        f.b[j] = ld16(sB + (n + lrow) * 128 + ca);
      } else {
        const int c = (n + tr_n) >> 3;
        const int sw = c ^ (4 * ((tr_k >> 1) & 1));
        f.b[j] = tr_read(sB + tr_k * (2 * BN) + sw * 16 + (tr_n & 7) * 2, 2 * BN);
      }
    }
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      if constexpr (!KMAJ) f.u[j] = ld16(sU + (j * 32 + lrow) * 128 + ca);
      // (columns from r on read other rows or stale LDS: sums never used)
      else f.u[j] = tr_read(sU + tr_k * (2 * r) + (j * 32 + tr_n) * 2, 2 * r);
    }
  };
  // A wait for this wave's loads of all but the newest `n` stages and its LDS
  // reads, then for every wave's.
  auto sync = [&](auto NS) __attribute__((always_inline)) {
    constexpr int n = decltype(NS)::value;
    constexpr int V0 = n * (A_PW + B_PW), V1 = n * (A_PW + B_PW + U_PW);
    static_assert(V1 < 64, "vmcnt range");
    if (has_u) __builtin_amdgcn_s_waitcnt((V1 & 15) | ((V1 >> 4) << 14) | (7 << 4));
    else __builtin_amdgcn_s_waitcnt((V0 & 15) | ((V0 >> 4) << 14) | (7 << 4));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  // Step st: stage st + 1 has landed and every wave holds stage st's
  // fragments, so stage st + NBUF may go into stage st's buffer; read the
  // fragments of stage st + 1 beside the products of stage st.
  auto step = [&](int st, const Frags &f, Frags &next) __attribute__((always_inline)) {
    sync(NwIC<NBUF - 2>());
    issue(st + NBUF);
    read_frags(st + 1, next);
#pragma unroll
    for (int j = 0; j < FN; ++j) mma32(BF16(), acc[j], f.b[j], f.a);
#pragma unroll
    for (int j = 0; j < RB; ++j) mma32(BF16(), accu[j], f.u[j], f.a);
  };
  {
#pragma unroll
    for (int st = 0; st < NBUF; ++st) issue(st);
    Frags f0, f1;
    sync(NwIC<NBUF - 1>());
    read_frags(0, f0);
    int st = 0;
    for (; st + 1 < nst; st += 2) {
      step(st, f0, f1);
      step(st + 1, f1, f0);
    }
    if (st < nst) step(st, f0, f1);
  }
  __builtin_amdgcn_s_waitcnt((7 << 4));  // vmcnt(0), lgkmcnt(0): the loads past the end too
  __syncthreads();

  // ---- operands of the tile's end -------------------------------------------------
  // The LoRA step's rank-r operand of this wave's output blocks and the x
  // values of its dA block, as matrix-core fragments: loaded ahead of the
  // sums, which hide their latency.
  const uint16_t *P = (const uint16_t *)a.P;
  constexpr int NS = RB * 2;           // rank slices
  constexpr int DB = RB * (BN / 32);   // dA blocks
  static_assert(FN <= NWV && DB <= NWV, "at most one output block and one dA block per wave");
  const int ns = (r + 15) / 16;
  struct EndP {
    uint32_t w[NS > 0 ? NS : 1][4];
  };
  auto load_p = [&](EndP &e) __attribute__((always_inline)) {
    const int n = n0 + wv * 32 + lrow;  // the lane's column of the operand
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int j0 = 16 * s + 8 * half;
      if constexpr (!KMAJ) {  // B [N][r]: r is a multiple of 4
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint2 v = n < a.N && j0 + 4 * h < r ? *(const uint2 *)(P + (int64_t)n * r + j0 + 4 * h) : make_uint2(0, 0);
          e.w[s][2 * h] = v.x;
          e.w[s][2 * h + 1] = v.y;
        }
      } else {  // A [r][N]
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const int jj = j0 + 2 * h;
          const uint32_t lo = n < a.N && jj < r ? P[(int64_t)jj * a.N + n] : 0;
          const uint32_t hi = n < a.N && jj + 1 < r ? P[(int64_t)(jj + 1) * a.N + n] : 0;
          e.w[s][h] = lo | (hi << 16);
        }
      }
    }
  };
  struct EndX {
    uint32_t w[BM / 16][4];
  };
  auto load_x = [&](EndX &e) __attribute__((always_inline)) {
    const uint16_t *x = (const uint16_t *)a.xin;
    const int c = n0 + (wv / (RB > 0 ? RB : 1)) * 32 + lrow;
#pragma unroll
    for (int s = 0; s < BM / 16; ++s)
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const int m = 16 * s + 8 * half + 2 * h;
        const uint32_t lo = c < a.N && m < mrows ? x[(int64_t)(m0 + m) * a.N + c] : 0;
        const uint32_t hi = c < a.N && m + 1 < mrows ? x[(int64_t)(m0 + m + 1) * a.N + c] : 0;
        e.w[s][h] = lo | (hi << 16);
      }
  };
  EndP ep;
  EndX ex;
  if constexpr (RB > 0) {
    if (a.out && wv < FN) load_p(ep);
    if constexpr (KMAJ) if (wv < DB) load_x(ex);
  }

  // ---- sum of the four k-slices -----------------------------------------------------
  // Slice 0's share is written in place (the tile F), the others' behind F.  A
  // lane holds row lane % 32 and runs of 4 columns.
  float *F = (float *)smem, *PL = F + PLANE;
  const int64_t tile_id = (int64_t)nt * a.tiles_m + mt;
  const __amdgpu_buffer_rsrc_t rsS = nw_rsrc(a.slots ? a.slots + tile_id * a.parts * (BM * C) : nullptr,
                                             a.parts > 1 ? (int64_t)a.parts * BM * C * 4 : 0);
  {
    float *dst = F + wk * PLANE;
    auto put = [&](const f32x16 &v, int col) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(f32x4 *)(dst + lrow * LDF + col + 8 * q + 4 * half) = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
    };
#pragma unroll
    for (int j = 0; j < FN; ++j) put(acc[j], j * 32);
#pragma unroll
    for (int j = 0; j < RB; ++j) put(accu[j], BN + j * 32);
    __syncthreads();
    for (int e = tid; e < BM * C / 4; e += NT) {
      const int row = e / (C / 4), col = e % (C / 4) * 4;
      float *f = F + row * LDF + col;
      f32x4 v = *(f32x4 *)f;
#pragma unroll
      for (int w = 1; w < NWV; ++w) v += *(const f32x4 *)(f + w * PLANE);
      if (a.parts > 1) nw_store(rsS, ((part * BM + row) * C + col) * 4, v);
      else *(f32x4 *)f = v;
    }
    __syncthreads();
  }

  // ---- the parts meet ---------------------------------------------------------------
  // (PL is free: its first words pass the outcomes.  The exchange that picks the
  // one that finishes runs beside the loads of the sums.)
  volatile int *s_all = (volatile int *)PL, *s_mine = s_all + 1;
  if (a.parts > 1) {
    __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));  // vmcnt(0): this wave's stores have completed
    __syncthreads();
    NwFlags flags{a.sync + tile_id * a.parts, lane};
    if (wv == 0) {
      const bool all = meet_arrive(flags, part, a.parts, a.gen);
      if (lane == 0) *s_all = all;
    }
    __syncthreads();
    if (!*s_all) return;
    constexpr int Q = (BM * C / 4 + NT - 1) / NT;  // quads per thread
    f32x4 v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = nw_load(rsS, (tid + q * NT) * 16);
    meet_word word0 = 0;
    if (wv == 0) word0 = meet_lower(flags, a.parts);
    // (G parts' loads in flight; past the last part they read zeros)
    constexpr int G = Q <= 4 ? 4 : Q <= 8 ? 2 : 1;
    for (int p = 1; p < a.parts; p += G) {
      f32x4 w[G][Q];
#pragma unroll
      for (int h = 0; h < G; ++h)
#pragma unroll
        for (int q = 0; q < Q; ++q) w[h][q] = nw_load(rsS, ((p + h) * (BM * C / 4) + tid + q * NT) * 16);
#pragma unroll
      for (int h = 0; h < G; ++h)
#pragma unroll
        for (int q = 0; q < Q; ++q)
          if (p + h < a.parts) v[q] += w[h][q];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = tid + q * NT;
      if ((BM * C / 4) % NT == 0 || e < BM * C / 4) *(f32x4 *)(F + e / (C / 4) * LDF + e % (C / 4) * 4) = v[q];
    }
    if (tid == 0) *s_mine = word0 == a.gen;
    __syncthreads();
    if (!*s_mine) return;
  }

  // ---- the finished tile: u, the LoRA step, the output ------------------------------
  if constexpr (RB > 0) {
    if (nt == 0 && a.u_out)
      for (int e = tid; e < mrows * r; e += NT) {
        const int m = e / r, j = e % r;
        a.u_out[(int64_t)(m0 + m) * r + j] = F[m * LDF + BN + j];
      }
  }
  // E(s u) of row m, rank indices 16 s + 8 half .. + 7
  auto su = [&](int m, int s) __attribute__((always_inline)) -> u32x4 {
    float f[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int j = 16 * s + 8 * half + t;
      f[t] = j < r ? a.scale * F[m * LDF + BN + j] : 0.0f;
    }
    return pack_vec(BF16(), f);
  };
  if (a.out && wv < FN) {
    f32x16 c;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = *(const f32x4 *)(F + lrow * LDF + wv * 32 + 8 * q + 4 * half);
#pragma unroll
      for (int e = 0; e < 4; ++e) c[4 * q + e] = v[e];
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (s < ns) mma32(BF16(), c, u32x4{ep.w[s][0], ep.w[s][1], ep.w[s][2], ep.w[s][3]}, su(lrow, s));
    const int m = m0 + lrow;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = n0 + wv * 32 + 8 * q + 4 * half;
      if (m < a.T && col < a.N)
        *(uint2 *)((uint16_t *)a.out + (int64_t)m * a.N + col) =
            make_uint2(pack_bf16x2(c[4 * q], c[4 * q + 1]), pack_bf16x2(c[4 * q + 2], c[4 * q + 3]));
    }
  }

  // ---- dA of this tile's rows and columns; the row tiles meet ------------------------
  if constexpr (KMAJ && RB > 0) {
    const __amdgpu_buffer_rsrc_t rsD =
        nw_rsrc(a.da_slots + (int64_t)nt * a.tiles_m * (RB * 32 * BN), (int64_t)a.tiles_m * RB * 32 * BN * 4);
    if (wv < DB) {
      const int cb = wv / RB, j = (wv % RB) * 32 + lrow;
      f32x16 d = f32x16{};
#pragma unroll
      for (int s = 0; s < BM / 16; ++s) {
        float f[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int m = 16 * s + 8 * half + t;
          f[t] = j < r && m < mrows ? a.scale * F[m * LDF + BN + j] : 0.0f;
        }
        mma32(BF16(), d, u32x4{ex.w[s][0], ex.w[s][1], ex.w[s][2], ex.w[s][3]}, pack_vec(BF16(), f));
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int lc = cb * 32 + 8 * q + 4 * half;
        const f32x4 v = f32x4{d[4 * q], d[4 * q + 1], d[4 * q + 2], d[4 * q + 3]};
        if (a.tiles_m > 1) nw_store(rsD, ((mt * RB * 32 + j) * BN + lc) * 4, v);
        else if (j < r && n0 + lc < a.N) *(f32x4 *)(a.dA + (int64_t)j * a.N + n0 + lc) = v;
      }
    }
    if (a.tiles_m > 1) {
      __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
      __syncthreads();
      // (Two may see all: they store the same sums, and raise nothing after.)
      if (wv == 0) {
        NwFlags flags{a.sync + (int64_t)a.tiles_n * a.tiles_m * a.parts + nt * a.tiles_m, lane};
        const bool all = meet_arrive(flags, mt, a.tiles_m, a.gen);
        if (all) meet_lower(flags, a.tiles_m);
        if (lane == 0) *s_all = all;
      }
      __syncthreads();
      if (!*s_all) return;
      for (int e = tid; e < r * (BN / 4); e += NT) {
        const int j = e / (BN / 4), lc = e % (BN / 4) * 4;
        f32x4 v = nw_load(rsD, (j * BN + lc) * 4);
        for (int m = 1; m < a.tiles_m; ++m) v += nw_load(rsD, ((m * RB * 32 + j) * BN + lc) * 4);
        if (n0 + lc < a.N) *(f32x4 *)(a.dA + (int64_t)j * a.N + n0 + lc) = v;
      }
    }
  }
}

// u = the sum of `parts` planes of n, in ascending order, as the tiled kernels add
// them.  (A pass of its own: a loop over the planes in the dB workgroups above
// kept their loads from being in flight at once, 23 -> 38 us for 48 tokens of
// 11008 -> 2048.)
__global__ __launch_bounds__(256) void narrow_sum_kernel(const float *planes, int parts, int n, float *u) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float v = planes[i];
  for (int p = 1; p < parts; ++p) v += planes[(int64_t)p * n + i];
  u[i] = v;
}

hipError_t launch_narrow_sum(const float *planes, int parts, int n, float *u, hipStream_t st) {
  hipLaunchKernelGGL(narrow_sum_kernel, dim3((n + 255) / 256), dim3(256), 0, st, planes, parts, n, u);
  return hipGetLastError();
}

// ---- the shape of a call -----------------------------------------------------------
NarrowPlan narrow_plan(int64_t T, int64_t N, int64_t K, int64_t r) {
  NarrowPlan p{};
  // Up to 64 tokens (32 above 32 rank columns); up to 128 where W has 2^22
  // weights or more, else the row tiles' meeting over dA costs more than the launch
  // saves; few_rule (api.cpp) says which directions.  fwd + bwd in us against the
  // tiled kernels: 24 tokens of 3072 -> 3072 25 against 160, 64 32 against 93, 128
  // 33 against 59; 50 of 8192 -> 3072 48 against 175; but 128 of 256 -> 256 19
  // against 18, 128 of 2048 -> 256 with r = 64 43 against 34.  (A part's W rows lie
  // within 31-bit offsets.)
  if (T < 1 || T > NARROW_MAX_T || r < 0 || r > 64 || r % 4 || N * K >= (int64_t(1) << 30)) return p;
  if ((T > 64 && N * K < (int64_t(1) << 22)) || (T > 32 && r > 32)) return p;
  p.tiles_m = (int)((T + NW_BM - 1) / NW_BM);
  p.tiles_n = (int)((N + NW_BN - 1) / NW_BN);
  // Parts of the reduction: up to 64 tiles leave most CUs idle, and up to four
  // parts of at least 16 stages use them (24 tokens of 3072 -> 3072, 48 tiles:
  // one part 11.8 + 19.2 us, three 11.6 + 16.6, four 11.0 + 15.4; 96 tiles: one
  // 11.9, two 13.1 us forward).  The same for every rank, so that a call of any rank sums W's
  // products in the same order.  The parts' sums stay below a quarter of the
  // fp32 dW.
  const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n, stages = (K + NW_BKE - 1) / NW_BKE;
  int64_t parts = 1;
  if (tiles <= 64) parts = std::max<int64_t>(1, std::min<int64_t>(4, stages / 16));
  while (parts > 1 && tiles * parts * NW_BM * (NW_BN + 32) * 4 > N * K) --parts;
  const int64_t per = (stages + parts - 1) / parts;
  p.parts = (int)((stages + per - 1) / per);
  p.part_k = (int)(per * NW_BKE);
  p.rank_blocks = (int)((r + 31) / 32);
  p.flags = tiles * (p.parts + 1);
  p.slot_bytes = p.parts > 1 ? (size_t)tiles * p.parts * NW_BM * (NW_BN + 32 * p.rank_blocks) * 4 : 0;
  p.da_bytes = p.tiles_m > 1 ? (size_t)tiles * p.rank_blocks * 32 * NW_BN * 4 : 0;
  p.ok = true;
  return p;
}

template <bool KMAJ>
static hipError_t narrow_dispatch(const NarrowArgs &a, int rank_blocks, int grid, hipStream_t st) {
  switch (rank_blocks) {
    case 0: hipLaunchKernelGGL((narrow_kernel<0, 5, KMAJ>), dim3(grid), dim3(256), 0, st, a); break;
    case 1: hipLaunchKernelGGL((narrow_kernel<1, 4, KMAJ>), dim3(grid), dim3(256), 0, st, a); break;
    case 2: hipLaunchKernelGGL((narrow_kernel<2, 4, KMAJ>), dim3(grid), dim3(256), 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_narrow(NarrowArgs a, const NarrowPlan &p, bool k_major, hipStream_t st) {
  if (!p.ok || a.T < 1 || a.T > NARROW_MAX_T || a.K < 1 || p.parts < 1 || p.parts > 64 || p.tiles_m > 64 ||
      (p.parts > 1 && !(a.slots && a.sync)) || (p.rank_blocks > 0) != (a.r > 0) || a.r > 32 * p.rank_blocks || a.r % 4 ||
      (int64_t)p.parts * p.part_k < a.K || (int64_t)(p.parts - 1) * p.part_k >= a.K || p.part_k % NW_BKE ||
      p.tiles_m * NW_BM < a.T || (int64_t)p.tiles_n * NW_BN < a.N ||
      (k_major && a.r > 0 && (!a.dA || !a.dB || !a.u_in || !a.xin || (p.tiles_m > 1 && !(a.da_slots && a.sync)))))
    return hipErrorInvalidValue;
  a.tiles_m = p.tiles_m;
  a.tiles_n = p.tiles_n;
  a.parts = p.parts;
  a.part_k = p.part_k;
  int grid = (p.tiles_n * p.parts + 7) / 8 * 8 * p.tiles_m;
  if (k_major && a.r > 0) grid += (a.K + 127) / 128;  // dB: 128 columns of dy a workgroup
  return k_major ? narrow_dispatch<true>(a, p.rank_blocks, grid, st) : narrow_dispatch<false>(a, p.rank_blocks, grid, st);
}

}  // namespace lora

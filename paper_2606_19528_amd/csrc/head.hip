// head.hip -- the frozen LM head's reduced-vocabulary cross entropy with
// logits masking, apart from its GEMMs (which run in gemm.hip with the
// cross-entropy epilogues):
//   * the reduced vocabulary J: every entry of the first k columns of the
//     similarity table's rows of the trainable positions' targets is marked
//     in a bitmap over the vocabulary, and the marks are compacted in
//     ascending order (so J is sorted and each target's position in J is a
//     lookup);
//   * row gathers (hidden states of the trainable positions, embedding rows
//     of J) into contiguous operands;
//   * the combine of the per-tile (max, sum of exp) partials into log-sum-exp
//     and per-position losses, and their sum, in a fixed order;
//   * the finishing of dh: bf16 rows at the trainable positions, zero rows
//     elsewhere.
#include "kernels.hpp"
#include "launch.hpp"

namespace lora {

__global__ void fill_u32_kernel(uint32_t *p, int64_t n, uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// mark[table[targets[rows[i]]][c]] = 1 for i < nrows, c < k.  Every writer
// stores the same value, so the result does not depend on their order.
__global__ void vocab_mark_kernel(const int32_t *table, int64_t ldtab, int k,
                                  const int32_t *targets, const int32_t *rows, int nrows, int T,
                                  int V, uint32_t *mark) {
  const int64_t total = (int64_t)nrows * k;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(e / k), c = (int)(e % k);
    const int32_t t = rows[i];
    if (t < 0 || t >= T) continue;  // invalid indices are skipped, never followed
    const int32_t y = targets[t];
    if (y < 0 || y >= V) continue;
    const int32_t v = table[(int64_t)y * ldtab + c];
    if (v >= 0 && v < V) mark[v] = 1u;
  }
}

// Ascending compaction of the marked entries in two launches: workgroup b
// owns the contiguous range [b per, (b + 1) per) of the vocabulary, first
// counting its marks, then writing J[pos] = v and pos_of[v] = pos for each
// from the sum of the lower workgroups' counts on.  Both read the marks as
// 16-byte vectors.  (One workgroup scanning the whole vocabulary, each thread
// its own contiguous slice, took 216 us at V = 128256: a serial chain of
// uncoalesced loads.)  count[0] = |J|; count[1 + b] holds workgroup b's count:
// the counts fit the 256 bytes that |J| has in the workspace.
constexpr int COMPACT_NT = 256, COMPACT_WG = 63;
__device__ __forceinline__ int compact_per(int V) {
  return ((V + COMPACT_WG - 1) / COMPACT_WG + 4 * COMPACT_NT - 1) / (4 * COMPACT_NT) * (4 * COMPACT_NT);
}
// Marks [v, v + 4) of a range that ends at hi (0 past it).
__device__ __forceinline__ u32x4 compact_load(const uint32_t *mark, int64_t v, int64_t hi) {
  if (v + 4 <= hi) return ld16(mark + v);
  u32x4 m = zero16();
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (v + e < hi) m[e] = mark[v + e];
  return m;
}
__global__ __launch_bounds__(COMPACT_NT) void vocab_count_kernel(const uint32_t *mark, int V, int32_t *count) {
  __shared__ int part[COMPACT_NT / 64];
  const int t = threadIdx.x;
  const int64_t per = compact_per(V), lo = (int64_t)blockIdx.x * per, hi = min((int64_t)V, lo + per);
  int c = 0;
  for (int64_t v = lo + 4 * t; v < hi; v += 4 * COMPACT_NT) {
    const u32x4 m = compact_load(mark, v, hi);
    c += (m[0] != 0) + (m[1] != 0) + (m[2] != 0) + (m[3] != 0);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off);
  if ((t & 63) == 0) part[t >> 6] = c;
  __syncthreads();
  if (t == 0) count[1 + blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}
__global__ __launch_bounds__(COMPACT_NT) void vocab_compact_kernel(const uint32_t *mark, int V, int32_t *J,
                                                                   int32_t *pos_of, int32_t *count) {
  __shared__ int part[COMPACT_NT / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t per = compact_per(V), lo = (int64_t)blockIdx.x * per, hi = min((int64_t)V, lo + per);
  int pos = 0;  // entries before this workgroup's range, then before the round's
  for (int b = 0; b < (int)blockIdx.x; ++b) pos += count[1 + b];
  for (int64_t r0 = lo; r0 < hi; r0 += 4 * COMPACT_NT) {
    const int64_t v = r0 + 4 * t;
    const u32x4 m = compact_load(mark, v, hi);
    const int c = (m[0] != 0) + (m[1] != 0) + (m[2] != 0) + (m[3] != 0);
    int x = c;  // inclusive scan over the wave
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(x, off);
      if (lane >= off) x += y;
    }
    __syncthreads();
    if (lane == 63) part[wave] = x;
    __syncthreads();
    int o = pos + x - c;
    for (int w = 0; w < wave; ++w) o += part[w];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (m[e] != 0) {
        J[o] = (int32_t)(v + e);
        pos_of[v + e] = o;
        ++o;
      }
    pos += part[0] + part[1] + part[2] + part[3];
  }
  if (blockIdx.x == gridDim.x - 1 && t == 0) count[0] = pos;
}

// tpos[i] = position in J of the target of trainable position rows[i].
// (-1 for an invalid position or target).
__global__ void target_pos_kernel(const int32_t *targets, const int32_t *rows, int nrows, int T,
                                  int V, const uint32_t *mark, const int32_t *pos_of,
                                  int32_t *tpos) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nrows) return;
  const int32_t t = rows[i];
  const int32_t y = (t >= 0 && t < T) ? targets[t] : -1;
  tpos[i] = (y >= 0 && y < V && mark[y] != 0u) ? pos_of[y] : -1;
}

// dst[i][:] = src[idx[i]][:] for i < n (zeros for an index outside [0, nsrc));
// rows of `cols` bf16, cols % 8 == 0.
__global__ void gather_rows_kernel(const uint16_t *src, int64_t ld, int nsrc, const int32_t *idx,
                                   int n, int cols, uint16_t *dst) {
  const int vpr = cols / 8;  // 16-byte vectors per row
  const int64_t total = (int64_t)n * vpr;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / vpr;
    const int v = (int)(e % vpr);
    const int32_t r = idx[i];
    st16(dst + i * cols + v * 8, (r >= 0 && r < nsrc) ? ld16(src + (int64_t)r * ld + v * 8) : zero16());
  }
}

// Per position m: lse = M + log(sum_t s_t exp(m_t - M)), M = max_t m_t over
// the vocabulary tiles t, and loss = lse - z_target.  A workgroup takes 32
// positions, thread (i, g) the tiles t = g, g + 32, ... of position i, so a
// wave reads whole 128-byte lines and each thread's chain is a thirty-second
// of the tiles; the 32 partial sums are added in ascending g.  (One thread a
// position took 247 us for 1229 positions over 422 tiles.)
constexpr int CMB_ROWS = 32, CMB_G = 32;
__global__ __launch_bounds__(CMB_ROWS *CMB_G) void ce_combine_kernel(const float *tmax, const float *tsum, int ntiles,
                                                                     int M, const float *ztgt, float *lse,
                                                                     float *loss) {
  __shared__ float red[CMB_G][CMB_ROWS];
  const int i = threadIdx.x % CMB_ROWS, g = threadIdx.x / CMB_ROWS;
  const int m = blockIdx.x * CMB_ROWS + i;
  const int mc = min(m, M - 1);
  float mx = -INFINITY;
  for (int t = g; t < ntiles; t += CMB_G) {
    const float v = tmax[(int64_t)t * M + mc];
    mx = t == g ? v : fmaxf(mx, v);
  }
  red[g][i] = mx;
  __syncthreads();
  mx = red[0][i];
  for (int q = 1; q < min(CMB_G, ntiles); ++q) mx = fmaxf(mx, red[q][i]);
  float s = 0.0f;
  for (int t = g; t < ntiles; t += CMB_G)
    s += tsum[(int64_t)t * M + mc] * __expf(tmax[(int64_t)t * M + mc] - mx);
  __syncthreads();
  red[g][i] = s;
  __syncthreads();
  if (g > 0 || m >= M) return;
  for (int q = 1; q < CMB_G; ++q) s += red[q][i];
  const float l = mx + __logf(s);
  lse[m] = l;
  loss[m] = l - ztgt[m];
}

// total[0] = sum of loss[0..M) by one workgroup: fixed per-thread strides,
// then a fixed pairwise tree.
constexpr int SUM_NT = 1024;
__global__ __launch_bounds__(SUM_NT) void sum_kernel(const float *loss, int M, float *total) {
  __shared__ float part[SUM_NT];
  const int t = threadIdx.x;
  float s = 0.0f;
  for (int m = t; m < M; m += SUM_NT) s += loss[m];
  part[t] = s;
  __syncthreads();
  for (int h = SUM_NT / 2; h >= 1; h >>= 1) {
    if (t < h) part[t] += part[t + h];
    __syncthreads();
  }
  if (t == 0) total[0] = part[0];
}

// inv[t] = i for t = rows[i], -1 for positions that are not listed.  (A
// position listed twice keeps one of its entries; the entry points require
// distinct positions.)
__global__ void invert_rows_kernel(const int32_t *rows, int nrows, int T, int32_t *inv) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nrows && rows[i] >= 0 && rows[i] < T) inv[rows[i]] = i;
}

// dh[t][:] = bf16(acc[inv[t]][:]) for listed positions, 0 for the others.
__global__ void dh_finish_kernel(const float *acc, const int32_t *inv, int T, int D, uint16_t *dh) {
  const int vpr = D / 8;
  const int64_t total = (int64_t)T * vpr;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = e / vpr;
    const int v = (int)(e % vpr);
    const int i = inv[t];
    u32x4 out = zero16();
    if (i >= 0) {
      const float *src = acc + (int64_t)i * D + v * 8;
      out = pack_vec(BF16(), src);
    }
    st16(dh + t * D + v * 8, out);
  }
}

static int grid_for(int64_t work, int nt);

hipError_t launch_fill_nan(float *p, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(fill_u32_kernel, dim3((int)((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192)),
                     dim3(256), 0, st, (uint32_t *)p, n, 0x7FC00000u);
  return hipGetLastError();
}

static int grid_for(int64_t work, int nt) {
  const int64_t g = (work + nt - 1) / nt;
  return (int)(g < 1 ? 1 : (g > 8192 ? 8192 : g));
}

hipError_t launch_vocab_build(const HeadVocabArgs &a, hipStream_t st) {
  hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(a.V, 256)), dim3(256), 0, st, a.mark,
                     (int64_t)a.V, 0u);
  hipLaunchKernelGGL(vocab_mark_kernel, dim3(grid_for((int64_t)a.nrows * a.k, 256)), dim3(256), 0,
                     st, a.table, a.ldtab, a.k, a.targets, a.rows, a.nrows, a.T, a.V, a.mark);
  hipLaunchKernelGGL(vocab_count_kernel, dim3(COMPACT_WG), dim3(COMPACT_NT), 0, st, a.mark, a.V, a.count);
  hipLaunchKernelGGL(vocab_compact_kernel, dim3(COMPACT_WG), dim3(COMPACT_NT), 0, st, a.mark, a.V, a.J,
                     a.pos_of, a.count);
  hipLaunchKernelGGL(target_pos_kernel, dim3((a.nrows + 255) / 256), dim3(256), 0, st, a.targets,
                     a.rows, a.nrows, a.T, a.V, a.mark, a.pos_of, a.tpos);
  return hipGetLastError();
}

hipError_t launch_gather_rows(const void *src, int64_t ld, int nsrc, const int32_t *idx, int n,
                              int cols, void *dst, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(gather_rows_kernel, dim3(grid_for((int64_t)n * (cols / 8), 256)), dim3(256), 0,
                     st, (const uint16_t *)src, ld, nsrc, idx, n, cols, (uint16_t *)dst);
  return hipGetLastError();
}

hipError_t launch_ce_combine(const float *tmax, const float *tsum, int ntiles, int M,
                             const float *ztgt, float *lse, float *loss, float *total,
                             hipStream_t st) {
  hipLaunchKernelGGL(ce_combine_kernel, dim3((M + CMB_ROWS - 1) / CMB_ROWS), dim3(CMB_ROWS * CMB_G), 0, st, tmax,
                     tsum, ntiles, M, ztgt, lse, loss);
  if (total) hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(SUM_NT), 0, st, loss, M, total);
  return hipGetLastError();
}

hipError_t launch_dh_finish(const float *acc, const int32_t *rows, int nrows, int32_t *inv, int T,
                            int D, void *dh, hipStream_t st) {
  hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(T, 256)), dim3(256), 0, st, (uint32_t *)inv,
                     (int64_t)T, 0xFFFFFFFFu);
  hipLaunchKernelGGL(invert_rows_kernel, dim3((nrows + 255) / 256), dim3(256), 0, st, rows, nrows,
                     T, inv);
  hipLaunchKernelGGL(dh_finish_kernel, dim3(grid_for((int64_t)T * (D / 8), 256)), dim3(256), 0, st,
                     acc, inv, T, D, (uint16_t *)dh);
  return hipGetLastError();
}

}  // namespace lora

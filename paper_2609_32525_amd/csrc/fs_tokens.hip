// Token-sized kernels of the path (fp32): fixed-order reductions of the per-workgroup
// partials written by the streaming passes, the G x G token mix and its backward, and the
// token gradients dU = dz / (s + eps), ds = -sum_v dz z / (s + eps).
// Their work is O(B H G V) or O(B H G^2 V), tiny next to the O(B N H G D) streaming passes;
// they are written so that they add little latency to a step.

#include <hip/hip_runtime.h>

#include <algorithm>

#include "fs_internal.h"

namespace fs {
namespace {

constexpr int kRedThreads = 1024;  // column reductions: many row groups in flight per column
constexpr int kCols = 64;          // columns per workgroup (chunk reductions)
constexpr int kRowGroups = kRedThreads / kCols;
constexpr int kColsWide = 16;      // long reductions (over samples, heads and chunks)
constexpr int kRowGroupsWide = kRedThreads / kColsWide;


// ---------------------------------------------------------------------------------------
// Fixed-order column sums. Thread (row group rg, column cg) sums rows rg, rg + 4, ... of its
// column; the four row-group sums are then added in the order rg = 0, 1, 2, 3. The result is
// independent of scheduling, so repeated runs are bitwise identical.
// ---------------------------------------------------------------------------------------
struct RowMap {
  // row r of output o lives at in + ((o_outer * stride_o + r_hi * stride_hi + r_lo) * len);
  // used to walk (chunk) rows of one (b, h), or (b, chunk) rows of one head.
  int64_t base;
  int rows;
  int lo;        // rows per inner run (chunks)
  int64_t hi_stride;  // distance in rows between inner runs
};

// Sum of rows rg, rg + 4, ... of column c, in increasing row order. Loads are issued eight at
// a time ahead of the adds so that the row walk is not a chain of dependent memory latencies.
template <int RG = kRowGroups>
__device__ __forceinline__ float colsum(const float* in, int64_t len, const RowMap& m, int64_t c,
                                        int rg) {
  constexpr int U = 8;
  float acc = 0.f;
  for (int r0 = rg; r0 < m.rows; r0 += U * RG) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r0 + u * RG;
      v[u] = 0.f;
      if (r < m.rows) {
        const int64_t row = m.base + (int64_t)(r / m.lo) * m.hi_stride + (r % m.lo);
        v[u] = in[row * len + c];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc += v[u];
  }
  return acc;
}

template <int RG = kRowGroups, int NC = kCols>
__device__ __forceinline__ float combine_groups(float v, float (*red)[NC], int rg, int cg) {
  red[rg][cg] = v;
  __syncthreads();
  float out = 0.f;
  if (rg == 0) {
#pragma unroll
    for (int q = 0; q < RG; ++q) out += red[q][cg];
  }
  return out;
}

// z = (sum_chunks U) / (sum_chunks s + eps) and s. grid (ceil(G V / 64), BH).
__global__ __launch_bounds__(kRedThreads) void k_reduce_tokens(const float* partU,
                                                            const float* partS, float* z,
                                                            float* s, int chunks, int G, int V,
                                                            float eps) {
  __shared__ float red[kRowGroups][kCols];
  __shared__ float sred[kRowGroups][kCols];
  const int bh = blockIdx.y;
  const int cg = threadIdx.x % kCols, rg = threadIdx.x / kCols;
  const int64_t len = (int64_t)G * V;
  const int64_t c = (int64_t)blockIdx.x * kCols + cg;
  const RowMap m{(int64_t)bh * chunks, chunks, chunks, 0};
  // slot sums for the slots this workgroup's columns touch (at most kCols / V + 1 <= 5)
  const int g_lo = (int)(((int64_t)blockIdx.x * kCols) / V);
  const int g_hi = (int)(min((int64_t)(blockIdx.x + 1) * kCols, len) - 1) / V;
  const int ns = g_hi - g_lo + 1;
  float sv = 0.f;
  if (cg < ns) sv = colsum(partS, G, m, g_lo + cg, rg);
  sred[rg][cg] = sv;
  const float u = c < len ? colsum(partU, len, m, c, rg) : 0.f;
  const float tot = combine_groups(u, red, rg, cg);   // contains the barrier for sred too
  if (rg == 0) {
    if (cg < ns) {
      float st = 0.f;
#pragma unroll
      for (int q = 0; q < kRowGroups; ++q) st += sred[q][cg];
      sred[0][cg] = st;
    }
  }
  __syncthreads();
  if (rg == 0 && c < len) {
    const int g = (int)(c / V);
    const float sg = sred[0][g - g_lo];
    z[(int64_t)bh * len + c] = tot / (sg + eps);
    if (c % V == 0) s[(int64_t)bh * G + g] = sg;
  }
}

// out[bh][c] = sum over chunks of part[bh][chunk][c]. grid (ceil(len / 64), BH).
__global__ __launch_bounds__(kRedThreads) void k_reduce_rows(const float* part, float* out,
                                                          int chunks, int64_t len) {
  __shared__ float red[kRowGroups][kCols];
  const int bh = blockIdx.y;
  const int cg = threadIdx.x % kCols, rg = threadIdx.x / kCols;
  const int64_t c = (int64_t)blockIdx.x * kCols + cg;
  const RowMap m{(int64_t)bh * chunks, chunks, chunks, 0};
  const float v = c < len ? colsum(part, len, m, c, rg) : 0.f;
  const float tot = combine_groups(v, red, rg, cg);
  if (rg == 0 && c < len) out[(int64_t)bh * len + c] = tot;
}

// Mix-parameter gradient from per-(b, h) partials [BH][len]: summed over (b, h), or over b
// per head (per_head); column block cb of output head hh.
__device__ __forceinline__ void reduce_mixparams_block(const float* partM, float* dmix, int B,
                                                       int H, int64_t len, int per_head, int cb,
                                                       int hh, float (*red)[kColsWide]) {
  const int cg = threadIdx.x % kColsWide, rg = threadIdx.x / kColsWide;
  const int64_t c = (int64_t)cb * kColsWide + cg;
  RowMap m;
  if (per_head)
    m = RowMap{hh, B, 1, H};
  else
    m = RowMap{0, B * H, B * H, 0};
  const float v = c < len ? colsum<kRowGroupsWide>(partM, len, m, c, rg) : 0.f;
  const float tot = combine_groups<kRowGroupsWide, kColsWide>(v, red, rg, cg);
  if (rg == 0 && c < len) dmix[(per_head ? (int64_t)hh * len : 0) + c] = tot;
}

__global__ __launch_bounds__(kRedThreads) void k_reduce_mixparams(const float* partM, float* dmix,
                                                               int B, int H, int64_t len,
                                                               int per_head) {
  __shared__ float red[kRowGroupsWide][kColsWide];
  reduce_mixparams_block(partM, dmix, B, H, len, per_head, blockIdx.x, blockIdx.y, red);
}

// Parameter gradients from the backward-pass-B partials [BH][chunks][D G + G + 2] (the last
// two floats of each partial hold one fp64 dtau partial), and optionally the mix-parameter
// gradient from its per-(b, h) partials, in one launch.
// grid.x = [column blocks of dW_s and dbias] [one dtau block] [column blocks of dmix];
// blockIdx.y is the head for per-head outputs (rows: b = 0..B-1, chunk), else 0 with rows
// over every (b, h, chunk); blocks whose segment has fewer heads return at once.
__global__ __launch_bounds__(kRedThreads) void k_reduce_params(
    const float* part, float* dWs, float* dbias, float* dtau, int B, int H, int chunks,
    int nblk, int D, int G, int per_head, const float* partM, float* dmix, int64_t mix_len,
    int mix_per_head) {
  __shared__ float red[kRowGroupsWide][kColsWide];
  const int64_t len = (int64_t)D * G + G + 2LL * nblk;
  const int64_t ncol = (int64_t)D * G + G;
  const int nbp = (int)((ncol + kColsWide - 1) / kColsWide);
  const int hh = blockIdx.y;
  if ((int)blockIdx.x > nbp) {
    if (dmix != nullptr && (mix_per_head || hh == 0))
      reduce_mixparams_block(partM, dmix, B, H, mix_len, mix_per_head, blockIdx.x - nbp - 1, hh,
                             red);
    return;
  }
  if (!per_head && hh > 0) return;
  if ((int)blockIdx.x == nbp) {
    // dtau: one wavefront per head; lane l sums the fp64 partials l, l + 64, ... of the
    // head's (b, chunk, slot block) entries in order, then a butterfly over the 64 lanes
    // (fixed pairing)
    if (hh == 0) {
      const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
      const int rows = B * chunks * nblk;
      for (int h = wave; h < H; h += nw) {
        double t = 0.0;
        for (int r = lane; r < rows; r += 64) {
          const int b = r / (chunks * nblk), q = (r / nblk) % chunks, k = r % nblk;
          t += *reinterpret_cast<const double*>(part + ((int64_t)(b * H + h) * chunks + q) * len +
                                                ncol + 2 * k);
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) t += __shfl_xor(t, off);
        if (lane == 0) dtau[h] = (float)t;
      }
    }
    return;
  }
  const int cg = threadIdx.x % kColsWide, rg = threadIdx.x / kColsWide;
  const int64_t c = (int64_t)blockIdx.x * kColsWide + cg;
  RowMap m;
  if (per_head)  // rows (b, chunk) of head hh: run of `chunks` rows every H * chunks rows
    m = RowMap{(int64_t)hh * chunks, B * chunks, chunks, (int64_t)H * chunks};
  else           // all (b, h, chunk) rows in order
    m = RowMap{0, B * H * chunks, B * H * chunks, 0};
  const float v = c < ncol ? colsum<kRowGroupsWide>(part, len, m, c, rg) : 0.f;
  const float tot = combine_groups<kRowGroupsWide, kColsWide>(v, red, rg, cg);
  if (rg == 0 && c < ncol) {
    if (c < (int64_t)D * G)
      dWs[(per_head ? (int64_t)hh * D * G : 0) + c] = tot;
    else
      dbias[(per_head ? (int64_t)hh * G : 0) + (c - (int64_t)D * G)] = tot;
  }
}

// ---------------------------------------------------------------------------------------
// Linear token maps for token sets too large for the single-workgroup LDS kernels: batched
// fp32 products C_o = sum_s A_{o,s} B_{o,s} on MFMA, a 16 x 16 output tile per workgroup or wavefront,
// operands read straight from global memory (they are small and cache resident). A strided
// descriptor covers the forward map, its transpose, and the parameter gradients summed over
// samples and heads without partials.
// Few such products are bound by the latency of their loads, not by bytes or flops, so four
// wavefronts split a long k range (their tiles are added through LDS in a fixed order) and an
// operand whose k index is contiguous is read 16 bytes per lane: MFMA r of a 16-wide k block takes
// k = 4 j + r from lane row j. G = 256, V = 32, 8 heads: 18.3 us per product with one wavefront per
// tile and 4-byte loads, 4.8 us now. Many are bound by how many loads are in flight: a block at a
// time with the next one's loads ahead keeps eight wavefronts per SIMD (16384 tiles at G = 256: 44 us;
// four blocks at a time 49 to 53).
// ---------------------------------------------------------------------------------------
typedef float f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 zero4() { return f4{0.f, 0.f, 0.f, 0.f}; }

// A product's sum over k in four chains, MFMA k index r on chain r: an MFMA rounds its running
// sum, and one chain of 16 for 64 columns left the attention's zmix 1.1 to 1.4 times as far from
// 64 bits (G = 32 to 64, V = 64).
struct Chains {
  f4 c[4];
  __device__ __forceinline__ Chains() {
#pragma unroll
    for (int r = 0; r < 4; ++r) c[r] = zero4();
  }
  __device__ __forceinline__ f4 sum() const { return (c[0] + c[1]) + (c[2] + c[3]); }
};

struct GemmDesc {
  // element (m, k) of A for output o and summand s: A[(o % a_mod) * a_o + s * a_s + m * a_rs + k * a_cs]
  const float* A;
  int64_t a_rs, a_cs, a_o, a_s;
  int a_mod;
  const float* B;  // element (k, n): B[o * b_o + s * b_s + k * b_rs + n * b_cs]
  int64_t b_rs, b_cs, b_o, b_s;
  float* C;  // element (m, n): C[o * c_o + m * c_rs + n]
  int64_t c_rs, c_o;
  int M, N, K, nsum;  // multiples of 16 (M, N, K)
};

constexpr int kGemmWaves = 4;

// KW: wavefronts that split a tile's k range.
template <int KW>
__global__ __launch_bounds__(64 * kGemmWaves) void k_tile_gemm(GemmDesc d) {
  __shared__ f4 red[KW > 1 ? kGemmWaves : 1][64];
  const int lane = threadIdx.x & 63, i = lane & 15, j = lane >> 4;
  const int wg_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wg_wave % KW;
  const int tn = d.N >> 4;
  const int t = blockIdx.x * (kGemmWaves / KW) + wg_wave / KW;
  if (KW == 1 && t >= (d.M >> 4) * tn) return;  // whole wavefronts
  const int m0 = (t / tn) << 4, n0 = (t % tn) << 4;
  const int o = blockIdx.y;
  const float* Ao = d.A + (int64_t)(o % d.a_mod) * d.a_o + (int64_t)(m0 + i) * d.a_rs;
  const float* Bo = d.B + (int64_t)o * d.b_o + (int64_t)(n0 + i) * d.b_cs;
  const int kb = d.K >> 4, nb = kb * d.nsum;  // 16-wide k blocks over all summands
  auto load = [&](int q, f4& av, f4& bv) {
    const int s = q / kb, k0 = ((q % kb) << 4) + 4 * j;
    const float* Ap = Ao + (int64_t)s * d.a_s + (int64_t)k0 * d.a_cs;
    const float* Bp = Bo + (int64_t)s * d.b_s + (int64_t)k0 * d.b_rs;
    if (d.a_cs == 1)
      av = *reinterpret_cast<const f4*>(Ap);
    else
#pragma unroll
      for (int r = 0; r < 4; ++r) av[r] = Ap[(int64_t)r * d.a_cs];
    if (d.b_rs == 1)
      bv = *reinterpret_cast<const f4*>(Bp);
    else
#pragma unroll
      for (int r = 0; r < 4; ++r) bv[r] = Bp[(int64_t)r * d.b_rs];
  };
  // blocks wave, wave + KW, ..., each one's loads issued before the one before it is multiplied
  // (the last reloads itself)
  Chains c;
  f4 av, bv;
  load(wave, av, bv);
  for (int q = wave; q < nb; q += KW) {
    f4 an, bn;
    load(min(q + KW, nb - 1), an, bn);
#pragma unroll
    for (int r = 0; r < 4; ++r) c.c[r] = mfma4(av[r], bv[r], c.c[r]);
    av = an;
    bv = bn;
  }
  f4 sum = c.sum();
  if constexpr (KW > 1) {
    static_assert(KW == kGemmWaves, "a workgroup per tile");
    red[wave][lane] = sum;
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int w = 1; w < KW; ++w) sum += red[w][lane];
  }
  float* Co = d.C + (int64_t)o * d.c_o + n0 + i;
#pragma unroll
  for (int r = 0; r < 4; ++r) Co[(int64_t)(m0 + 4 * j + r) * d.c_rs] = sum[r];
}

// 16-wide k blocks from which four wavefronts split a tile's k range: at 64 blocks (G = 1024,
// V = 32) 9.2 us against 23.9 with one wavefront per tile on 512 tiles, 76.8 against 81.2 on 8192;
// at 16 (G = 256) 44.1 against 44.7 on 16384; at 7 and 2 the split leaves wavefronts idle and costs
// (28672 tiles of G = 112, V = 64: 44.0 against 35.7; 32768 of a channel map at V = 32: 34.5 against 17.2).
constexpr int kSplitBlocks = 16;

static hipError_t run_gemm(const GemmDesc& d, int nout, hipStream_t st) {
  const int tiles = (d.M / 16) * (d.N / 16);
  if ((d.K / 16) * (int64_t)d.nsum >= kSplitBlocks)
    hipLaunchKernelGGL(k_tile_gemm<kGemmWaves>, dim3(tiles, nout), dim3(64 * kGemmWaves), 0, st, d);
  else
    hipLaunchKernelGGL(k_tile_gemm<1>, dim3((tiles + kGemmWaves - 1) / kGemmWaves, nout),
                       dim3(64 * kGemmWaves), 0, st, d);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Token gradients and the shifts the backward pass B uses, for the token sets beyond the
// single-workgroup kernels: dU = dz / (s + eps), ds = -sum_v dz z / (s + eps), and the
// mass-weighted slot means cen = [sum_g m_g zmix[g][:], sum_g m_g dU[g][:], sum_g m_g ds[g]]
// with m_g = s_g / sum s. One workgroup per 16 tokens writes dU, ds and its tokens' sums
// [sum s zmix, sum s dU, sum s ds, sum s] (2 V + 2 floats); k_tok_fin adds those in order. A
// single workgroup per (b, h) walking all its tokens took 27 us at G = 256 and 99 us at
// G = 1024 (V = 32, 8 heads), the two kernels 5.0 + 4.7 us at
// G = 256.
// ---------------------------------------------------------------------------------------
template <int V>
constexpr int kRowPad = V + 4;  // LDS rows of the 16-token blocks, 16-byte aligned

// The 16 tokens at token offset t0 (in all tokens), their dz rows in LDS; every thread of the
// workgroup calls it.
template <int V>
__device__ __forceinline__ void token_grads16(const float* dzl, const float* z, const float* s,
                                              const float* zmix, float* dU, float* ds, float* part,
                                              int64_t t0, float eps) {
  __shared__ float dsl[16], sl[16];
  const int tid = threadIdx.x;
  if (tid < 256) {  // 16 threads per token: sum_v dz z
    const int g = tid >> 4, q = tid & 15;
    const float sg = s[t0 + g];
    float acc = 0.f;
#pragma unroll
    for (int v = 0; v < V; v += 16) acc += dzl[g * kRowPad<V> + v + q] * z[(t0 + g) * V + v + q];
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 16);
    if (q == 0) {
      const float d = -acc / (sg + eps);
      dsl[g] = d;
      sl[g] = sg;
      ds[t0 + g] = d;
    }
  }
  __syncthreads();
  for (int idx = tid; idx < 16 * V; idx += blockDim.x) {
    const int g = idx / V, c = idx % V;
    dU[t0 * V + idx] = dzl[g * kRowPad<V> + c] / (sl[g] + eps);
  }
  // each column's 16 tokens in order (a loop per kind of column: with the choice inside, every
  // load was waited for by itself)
  float acc = 0.f;
  if (tid < V) {
#pragma unroll
    for (int g = 0; g < 16; ++g) acc += sl[g] * zmix[(t0 + g) * V + tid];
  } else if (tid < 2 * V) {
#pragma unroll
    for (int g = 0; g < 16; ++g) acc += sl[g] * (dzl[g * kRowPad<V> + tid - V] / (sl[g] + eps));
  } else if (tid < 2 * V + 2) {
#pragma unroll
    for (int g = 0; g < 16; ++g) acc += tid == 2 * V ? sl[g] * dsl[g] : sl[g];
  }
  if (tid < 2 * V + 2) part[(t0 >> 4) * (2 * V + 2) + tid] = acc;
}

template <int V>
__global__ __launch_bounds__(256) void k_token_grads(const float* z, const float* s,
                                                     const float* zmix, const float* dz, float* dU,
                                                     float* ds, float* part, float eps) {
  __shared__ float dzl[16 * kRowPad<V>];
  const int64_t t0 = (int64_t)blockIdx.x * 16;
  for (int idx = threadIdx.x; idx < 16 * V; idx += 256)
    dzl[(idx / V) * kRowPad<V> + idx % V] = dz[t0 * V + idx];
  __syncthreads();
  token_grads16<V>(dzl, z, s, zmix, dU, ds, part, t0, eps);
}

// cen of every (b, h) from its 16-token sums (workgroups 0 .. ncen - 1), and the attention
// parameter gradients from the workgroup partials [rows][mix_len] (the rest). Fixed order.
__global__ __launch_bounds__(kRedThreads) void k_tok_fin(const float* part, float* cen, int ncen,
                                                         int nblk, int V, const float* partW,
                                                         float* dmix, int rows, int64_t mix_len) {
  __shared__ float red[kRowGroupsWide][kColsWide];
  __shared__ float tot[2 * 64 + 2];
  if ((int)blockIdx.x >= ncen) {
    const int cg = threadIdx.x % kColsWide, rg = threadIdx.x / kColsWide;
    const int64_t c = (int64_t)(blockIdx.x - ncen) * kColsWide + cg;
    const RowMap m{0, rows, rows, 0};
    const float v = c < mix_len ? colsum<kRowGroupsWide>(partW, mix_len, m, c, rg) : 0.f;
    const float t = combine_groups<kRowGroupsWide, kColsWide>(v, red, rg, cg);
    if (rg == 0 && c < mix_len) dmix[c] = t;
    return;
  }
  const int nc = 2 * V + 2, ng = kRedThreads / nc;
  const int c = threadIdx.x % nc, rg = threadIdx.x / nc;
  float* sums = &red[0][0];  // ng nc <= 1024
  if (rg < ng) {
    const RowMap m{(int64_t)blockIdx.x * nblk, nblk, nblk, 0};
    float acc = 0.f;
    for (int r = rg; r < nblk; r += ng) acc += part[(m.base + r) * nc + c];
    sums[rg * nc + c] = acc;
  }
  __syncthreads();
  if ((int)threadIdx.x < nc) {
    float acc = 0.f;
    for (int q = 0; q < ng; ++q) acc += sums[q * nc + threadIdx.x];
    tot[threadIdx.x] = acc;
  }
  __syncthreads();
  const float ts = tot[nc - 1];
  if ((int)threadIdx.x < nc - 1)
    cen[(int64_t)blockIdx.x * (nc - 1) + threadIdx.x] = tot[threadIdx.x] * (ts > 0.f ? 1.0f / ts : 0.f);
}

// ---------------------------------------------------------------------------------------
// Single-head token self-attention among the G tokens of one (b, h) (q, k, v = z Wq, z Wk,
// z Wv; P = softmax_row(scale q k^T); zmix = P v) for token sets beyond the single-workgroup
// LDS kernels, any G multiple of 16 up to 1024. One workgroup per 16 tokens, its wavefronts
// splitting the other tokens' 16-row tiles; fp32 MFMA with operands from global memory (small,
// cache resident). The token sets are far too small to be bound by bytes or flops: what counts
// is the chain of dependent loads, so every tile is swept once and no intermediate goes
// through memory that need not. Three arrangements leave no transposes through LDS:
//   - a contraction over V takes k = 16 mt + 4 j + r for MFMA (mt, r) from lane row j, so rows
//     are read 16 bytes per lane (Row);
//   - a result tile C[m = 4 j + r][n = i] is directly the A operand (m = i, k = 4 j + r) of a
//     contraction over its rows, and the B operand (n = i) of the next projection;
//   - with D_g = dzmix_g . zmix_g (the row sum of dP * P), dS = P * (dP - D) needs no row pass.
// The kernels with one wavefront per 16 rows and the backward as thirteen batched products took
// 133 + 396 us at G = 1024, V = 32, 8 heads, and one 256-thread workgroup per (b, h) 275 + 810
// us at G = 48, V = 64; these take 27 + 59 and 11 + 21 us.
// ---------------------------------------------------------------------------------------
template <int V>
struct Row {
  f4 v[V / 16];
};
// The lane's row at p, columns 16 mt + 4 j .. + 3.
template <int V>
__device__ __forceinline__ Row<V> ld_row(const float* p, int j) {
  Row<V> o;
#pragma unroll
  for (int mt = 0; mt < V / 16; ++mt) o.v[mt] = *reinterpret_cast<const f4*>(p + 16 * mt + 4 * j);
  return o;
}
// C[m][n] = a_m . b_n over V columns.
template <int V>
__device__ __forceinline__ f4 row_dot(const Row<V>& a, const Row<V>& b) {
  Chains c;
#pragma unroll
  for (int mt = 0; mt < V / 16; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) c.c[r] = mfma4(a.v[mt][r], b.v[mt][r], c.c[r]);
  return c.sum();
}
// C[m][n] = sum over e of W[e][16 nt + m] b_n[e].
template <int V>
__device__ __forceinline__ f4 col_dot(const float* W, int nt, const Row<V>& b, int i, int j) {
  float w[V / 16][4];
#pragma unroll
  for (int mt = 0; mt < V / 16; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) w[mt][r] = W[(16 * mt + 4 * j + r) * V + 16 * nt + i];
  Chains c;
#pragma unroll
  for (int mt = 0; mt < V / 16; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) c.c[r] = mfma4(w[mt][r], b.v[mt][r], c.c[r]);
  return c.sum();
}
// acc[ct] += (tile)^T M: the tile's rows are tokens t0 + 4 j + r, M their V-wide rows.
template <int V>
__device__ __forceinline__ void tile_rows(f4 (&acc)[V / 16], const f4& tile, const float* M, int i, int j) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int ct = 0; ct < V / 16; ++ct) acc[ct] = mfma4(tile[r], M[(4 * j + r) * V + 16 * ct + i], acc[ct]);
}
// (rows W)^T as a Row: lane i keeps its own row, v[nt][r] = (row W)[16 nt + 4 j + r].
template <int V>
__device__ __forceinline__ Row<V> project(const Row<V>& z, const float* W, int i, int j) {
  Row<V> o;
#pragma unroll
  for (int nt = 0; nt < V / 16; ++nt) o.v[nt] = col_dot<V>(W, nt, z, i, j);
  return o;
}
// (rows W^T)^T as a Row.
template <int V>
__device__ __forceinline__ Row<V> project_t(const Row<V>& q, const float* W, int i, int j) {
  Row<V> o;
#pragma unroll
  for (int et = 0; et < V / 16; ++et) o.v[et] = row_dot<V>(ld_row<V>(W + (16 * et + i) * V, j), q);
  return o;
}
// Sum and maximum over the four 16-lane rows.
__device__ __forceinline__ float rows_sum(float v) {
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}
__device__ __forceinline__ float rows_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16));
  return fmaxf(v, __shfl_xor(v, 32));
}

// Forward. Scores come from r = (z Wq) Wk^T (S[g][u] = scale r_g . z_u, so k is never formed),
// each wavefront keeping its TPW score tiles in registers between the softmax statistics and
// the weights; T = P z and zmix = T Wv (= P v by associativity).
// (Few workgroups per compute unit: registers for loads in flight count, not occupancy.)
template <int V, int NW, int TPW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 4))) void k_attn_rows(const float* z, float* zmix, float* P,
                                                       const float* Wq, const float* Wk,
                                                       const float* Wv, float scale, int G) {
  constexpr int VT = V / 16;
  constexpr float kLog2e = 1.4426950408889634f;
  __shared__ float red[NW][16 * kRowPad<V>];
  __shared__ float st[2][NW][16];
  const int lane = threadIdx.x & 63, i = lane & 15, j = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nt = G >> 4;
  const int bh = blockIdx.x / nt, g0 = (blockIdx.x % nt) << 4;
  const float* zb = z + (int64_t)bh * G * V;
  float* Pb = P + (int64_t)bh * G * G;
  Row<V> rg = project_t<V>(project<V>(ld_row<V>(zb + (g0 + i) * V, j), Wq, i, j), Wk, i, j);
#pragma unroll
  for (int mt = 0; mt < VT; ++mt) rg.v[mt] *= scale * kLog2e;
  // base-2 score tiles, rows u = 16 ut + 4 j + r, columns g = g0 + i
  f4 s[TPW];
  float m = -INFINITY;
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int ut = w + NW * t;
    if (ut < nt) {
      s[t] = row_dot<V>(ld_row<V>(zb + (16 * ut + i) * V, j), rg);
      m = fmaxf(m, fmaxf(fmaxf(s[t][0], s[t][1]), fmaxf(s[t][2], s[t][3])));
    }
  }
  m = rows_max(m);
  if (j == 0) st[0][w][i] = m;
  __syncthreads();
  float M = st[0][0][i];
#pragma unroll
  for (int q = 1; q < NW; ++q) M = fmaxf(M, st[0][q][i]);
  float l = 0.f;
#pragma unroll
  for (int t = 0; t < TPW; ++t)
    if (w + NW * t < nt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[t][r] = exp2f(s[t][r] - M);
        l += s[t][r];
      }
    }
  l = rows_sum(l);
  if (j == 0) st[1][w][i] = l;
  __syncthreads();
  float L = 0.f;
#pragma unroll
  for (int q = 0; q < NW; ++q) L += st[1][q][i];
  const float inv = 1.0f / L;
  f4 T[VT];
#pragma unroll
  for (int ct = 0; ct < VT; ++ct) T[ct] = zero4();
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int ut = w + NW * t;
    if (ut < nt) {
      // e / L, rounded once (e times the rounded reciprocal left P 1.05 to 1.06 times as far from
      // 64 bits as before, this 0.85 times)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float p = s[t][r] * inv;
        s[t][r] = __builtin_fmaf(__builtin_fmaf(-p, L, s[t][r]), inv, p);
      }
      *reinterpret_cast<f4*>(Pb + (int64_t)(g0 + i) * G + 16 * ut + 4 * j) = s[t];
      tile_rows<V>(T, s[t], zb + 16 * ut * V, i, j);
    }
  }
  // T (rows g = 4 j + r) of all wavefronts, then zmix = T Wv
#pragma unroll
  for (int ct = 0; ct < VT; ++ct)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[w][(4 * j + r) * kRowPad<V> + 16 * ct + i] = T[ct][r];
  __syncthreads();
  for (int n = w; n < VT; n += NW) {
    Row<V> t;
#pragma unroll
    for (int mt = 0; mt < VT; ++mt) {
      t.v[mt] = zero4();
#pragma unroll
      for (int q = 0; q < NW; ++q)
        t.v[mt] += *reinterpret_cast<const f4*>(&red[q][i * kRowPad<V> + 16 * mt + 4 * j]);
    }
    *reinterpret_cast<f4*>(zmix + ((int64_t)bh * G + g0 + i) * V + 16 * n + 4 * j) = col_dot<V>(Wv, n, t, i, j);
  }
}

// q, k, v (wavefronts 0, 1, 2) of 16 tokens, and D_g = dzmix_g . zmix_g where zmix is given.
template <int V>
__global__ __launch_bounds__(192) void k_attn_qkv(const float* z, const float* zmix,
                                                  const float* dzm, const float* Wq,
                                                  const float* Wk, const float* Wv, float* q,
                                                  float* k, float* v, float* D) {
  const int lane = threadIdx.x & 63, i = lane & 15, j = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t t = (int64_t)blockIdx.x * 16 + i;  // the lane's token
  const Row<V> o = project<V>(ld_row<V>(z + t * V, j), w == 0 ? Wq : w == 1 ? Wk : Wv, i, j);
  float* out = w == 0 ? q : w == 1 ? k : v;
#pragma unroll
  for (int nt = 0; nt < V / 16; ++nt) *reinterpret_cast<f4*>(out + t * V + 16 * nt + 4 * j) = o.v[nt];
  if (w == 0 && zmix != nullptr) {
    const Row<V> a = ld_row<V>(zmix + t * V, j), b = ld_row<V>(dzm + t * V, j);
    float acc = 0.f;
#pragma unroll
    for (int mt = 0; mt < V / 16; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc += a.v[mt][r] * b.v[mt][r];
    acc = rows_sum(acc);
    if (j == 0) D[t] = acc;
  }
}

// D_g = sum_u P[g][u] (dzmix_g . v_u) where no zmix is at hand (fs_mix_bwd): a workgroup per 16
// tokens, its wavefronts over every eighth tile of u, dP a tile product as in k_attn_bwd_rows. (One
// wavefront per token with a dot product per lane loaded v uncoalesced, V loads a lane and
// token: fs_mix_bwd at G = 1024, V = 32, 8 heads 538 -> 65 us.) D is subtracted from dP values of its own
// size, so its sum goes up a tree.
constexpr int kDotWaves = 8;

template <int V>
__global__ __launch_bounds__(64 * kDotWaves) void k_attn_rowdot(const float* P, const float* dzm,
                                                                const float* v, float* D, int G) {
  __shared__ float red[kDotWaves][16];
  const int lane = threadIdx.x & 63, i = lane & 15, j = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nt = G >> 4;
  const int bh = blockIdx.x / nt, g0 = (blockIdx.x % nt) << 4;
  const int64_t tb = (int64_t)bh * G;  // token 0 of this (b, h)
  const Row<V> gr = ld_row<V>(dzm + (tb + g0 + i) * V, j);
  const float* Pg = P + (tb + g0 + i) * G + 4 * j;
  const float* vb = v + (tb + i) * V;
  f4 part = zero4();
#pragma unroll 2
  for (int t = w; t < nt; t += kDotWaves) {  // rows u = 16 t + 4 j + r, columns g = g0 + i
    const f4 p = *reinterpret_cast<const f4*>(Pg + 16 * t);
    const f4 dP = row_dot<V>(ld_row<V>(vb + 16 * t * V, j), gr);
    part += p * dP;
  }
  const float acc = rows_sum((part[0] + part[1]) + (part[2] + part[3]));
  if (j == 0) red[w][i] = acc;
  __syncthreads();
  if (threadIdx.x < 16) {
    float t[kDotWaves];
#pragma unroll
    for (int q = 0; q < kDotWaves; ++q) t[q] = red[q][threadIdx.x];
#pragma unroll
    for (int n = kDotWaves / 2; n > 0; n /= 2)
#pragma unroll
      for (int q = 0; q < n; ++q) t[q] += t[q + n];
    D[tb + g0 + threadIdx.x] = t[0];
  }
}

// Backward for 16 tokens of one (b, h). Wavefronts 0-3 take the tokens as rows g
// (dq_g = scale sum_u dS[g][u] k_u), 4-7 as columns u (dk_u = scale sum_g dS[g][u] q_g,
// dv_u = sum_g P[g][u] dzmix_g), each over every fourth tile of the other index; then
// dz = dq Wq^T + dk Wk^T + dv Wv^T, the tokens' part of [dWq; dWk; dWv] = z^T [dq; dk; dv] into
// partW, and with s given the token gradients (token_grads16).
template <int V>
__global__ __launch_bounds__(512) void k_attn_bwd_rows(
    const float* z, const float* s, const float* zmix, const float* P, const float* dzm,
    const float* q, const float* k, const float* v, const float* D, const float* Wq,
    const float* Wk, const float* Wv, float scale, float* dz, float* dU, float* ds, float* part,
    float* partW, int G, float eps) {
  constexpr int VT = V / 16, VP = kRowPad<V>;
  __shared__ float red[4][3][16 * VP];
  __shared__ float dd[3][16 * VP];
  __shared__ float dzl[16 * VP];
  const int lane = threadIdx.x & 63, i = lane & 15, j = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), sub = w & 3;
  const int nt = G >> 4;
  const int bh = blockIdx.x / nt, g0 = (blockIdx.x % nt) << 4;
  const int64_t tb = (int64_t)bh * G;  // token 0 of this (b, h)
  const float* Pb = P + tb * G;
  const float* Db = D + tb;
  const float* gz = dzm + tb * V;
  // (two chains each: at G = 1024 one takes 64 MFMAs)
  f4 a0[2][VT], a1[2][VT];
#pragma unroll
  for (int ct = 0; ct < VT; ++ct) a0[0][ct] = a0[1][ct] = a1[0][ct] = a1[1][ct] = zero4();
  // the next tile's operands are loaded before a tile is multiplied (tiles past the end reload
  // the last one)
  if (w < 4) {
    const Row<V> gr = ld_row<V>(gz + (g0 + i) * V, j);
    const float Dg = Db[g0 + i];
    Row<V> vn;
    f4 pn;
    float kn[4][VT];
    auto load = [&](int t) {
      vn = ld_row<V>(v + (tb + 16 * t + i) * V, j);
      pn = *reinterpret_cast<const f4*>(Pb + (int64_t)(g0 + i) * G + 16 * t + 4 * j);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int ct = 0; ct < VT; ++ct) kn[r][ct] = k[(tb + 16 * t + 4 * j + r) * V + 16 * ct + i];
    };
    if (sub < nt) load(sub);
    for (int t = sub; t < nt; t += 4) {
      const Row<V> vc = vn;
      const f4 p = pn;
      float kc[4][VT];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int ct = 0; ct < VT; ++ct) kc[r][ct] = kn[r][ct];
      load(min(t + 4, nt - 1));
      // rows u = 16 t + 4 j + r, columns g = g0 + i
      f4 dS = row_dot<V>(vc, gr);
#pragma unroll
      for (int r = 0; r < 4; ++r) dS[r] = p[r] * (dS[r] - Dg);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int ct = 0; ct < VT; ++ct) a0[r & 1][ct] = mfma4(dS[r], kc[r][ct], a0[r & 1][ct]);
    }
  } else {
    const Row<V> vr = ld_row<V>(v + (tb + g0 + i) * V, j);
    Row<V> gn;
    f4 Dn, pn;
    float qn[4][VT], zn[4][VT];
    auto load = [&](int t) {
      gn = ld_row<V>(gz + (16 * t + i) * V, j);
      Dn = *reinterpret_cast<const f4*>(Db + 16 * t + 4 * j);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pn[r] = Pb[(int64_t)(16 * t + 4 * j + r) * G + g0 + i];
#pragma unroll
        for (int ct = 0; ct < VT; ++ct) {
          qn[r][ct] = q[(tb + 16 * t + 4 * j + r) * V + 16 * ct + i];
          zn[r][ct] = gz[(16 * t + 4 * j + r) * V + 16 * ct + i];
        }
      }
    };
    if (sub < nt) load(sub);
    for (int t = sub; t < nt; t += 4) {
      const Row<V> gc = gn;
      const f4 Dg = Dn, p = pn;
      float qc[4][VT], zc[4][VT];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int ct = 0; ct < VT; ++ct) {
          qc[r][ct] = qn[r][ct];
          zc[r][ct] = zn[r][ct];
        }
      load(min(t + 4, nt - 1));
      // rows g = 16 t + 4 j + r, columns u = g0 + i
      f4 dS = row_dot<V>(gc, vr);
#pragma unroll
      for (int r = 0; r < 4; ++r) dS[r] = p[r] * (dS[r] - Dg[r]);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int ct = 0; ct < VT; ++ct) {
          a0[r & 1][ct] = mfma4(dS[r], qc[r][ct], a0[r & 1][ct]);
          a1[r & 1][ct] = mfma4(p[r], zc[r][ct], a1[r & 1][ct]);
        }
    }
  }
#pragma unroll
  for (int ct = 0; ct < VT; ++ct)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int at = (4 * j + r) * VP + 16 * ct + i;
      red[sub][w < 4 ? 0 : 1][at] = a0[0][ct][r] + a0[1][ct][r];
      if (w >= 4) red[sub][2][at] = a1[0][ct][r] + a1[1][ct][r];
    }
  __syncthreads();
  for (int idx = threadIdx.x; idx < 3 * 16 * V; idx += 512) {
    const int x = idx / (16 * V), at = (idx % (16 * V)) / V * VP + idx % V;
    const float t = (red[0][x][at] + red[1][x][at]) + (red[2][x][at] + red[3][x][at]);
    dd[x][at] = x < 2 ? scale * t : t;
  }
  __syncthreads();
  for (int n = w; n < VT + 3 * VT * VT; n += 8) {
    if (n < VT) {  // dz columns 16 n .. + 15: rows e = 16 n + 4 j + r, columns g = g0 + i
      f4 acc = zero4();
#pragma unroll
      for (int x = 0; x < 3; ++x)
        acc += row_dot<V>(ld_row<V>((x == 0 ? Wq : x == 1 ? Wk : Wv) + (16 * n + i) * V, j),
                          ld_row<V>(dd[x] + i * VP, j));
      *reinterpret_cast<f4*>(dz + (tb + g0 + i) * V + 16 * n + 4 * j) = acc;
      *reinterpret_cast<f4*>(dzl + i * VP + 16 * n + 4 * j) = acc;
    } else if (partW != nullptr) {
      const int t = n - VT, x = t / (VT * VT), et = (t / VT) % VT, ct = t % VT;
      f4 acc = zero4();
#pragma unroll
      for (int r = 0; r < 4; ++r)
        acc = mfma4(z[(tb + g0 + 4 * j + r) * V + 16 * et + i], dd[x][(4 * j + r) * VP + 16 * ct + i], acc);
      float* o = partW + (int64_t)blockIdx.x * 3 * V * V + x * V * V + 16 * ct + i;
#pragma unroll
      for (int r = 0; r < 4; ++r) o[(16 * et + 4 * j + r) * V] = acc[r];
    }
  }
  if (s == nullptr) return;
  __syncthreads();
  token_grads16<V>(dzl, z, s, zmix, dU, ds, part, tb + g0, eps);
}

inline unsigned blocks(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }
// Floats of one (b, h) mix-parameter partial.
inline int64_t mix_partial_len(const Geom& g, int kind) {
  return kind == 1 ? (int64_t)g.G * g.G : (kind == 2 ? (int64_t)g.V * g.V : 3LL * g.V * g.V);
}


}  // namespace

bool attn_rows(const Geom& g, int kind) { return kind == 3 && !tok_fused(g, kind); }

hipError_t launch_reduce_tokens(const Geom& g, const float* partU, const float* partS,
                                int chunks, float* z, float* s, hipStream_t st) {
  dim3 grid(blocks((int64_t)g.G * g.V, kCols), g.BH());
  hipLaunchKernelGGL(k_reduce_tokens, grid, dim3(kRedThreads), 0, st, partU, partS, z, s, chunks,
                     g.G, g.V, g.eps);
  return hipGetLastError();
}

hipError_t launch_reduce_rows(const Geom& g, const float* part, float* out, int chunks,
                              int64_t len, hipStream_t st) {
  dim3 grid(blocks(len, kCols), g.BH());
  hipLaunchKernelGGL(k_reduce_rows, grid, dim3(kRedThreads), 0, st, part, out, chunks, len);
  return hipGetLastError();
}

// Whether the mix-parameter gradient goes through per-(b, h) partials (the LDS kernels) or is
// written by the mix backward itself.
static bool mix_params_in_partials(const Geom& g, int kind) {
  return tok_fused(g, kind);
}

hipError_t launch_reduce_params(const Geom& g, const float* part, float* dWs, float* dbias,
                                float* dtau, int chunks, int nblk, const MixArgs* m,
                                const float* partM, float* dmix, hipStream_t st) {
  const int64_t ncol = (int64_t)g.D * g.G + g.G;
  const bool with_mix =
      m != nullptr && dmix != nullptr && m->kind != 0 && mix_params_in_partials(g, m->kind);
  const int64_t mix_len = with_mix ? mix_partial_len(g, m->kind) : 0;
  const bool mix_per_head = with_mix && m->kind == 1 && m->a_per_head;
  const unsigned nb = blocks(ncol, kColsWide) + 1 + (with_mix ? blocks(mix_len, kColsWide) : 0);
  const int heads = std::max(g.ws_per_head ? g.H : 1, mix_per_head ? g.H : 1);
  hipLaunchKernelGGL(k_reduce_params, dim3(nb, heads), dim3(kRedThreads), 0, st, part, dWs,
                     dbias, dtau, (int)g.B, g.H, chunks, nblk, g.D, g.G, g.ws_per_head ? 1 : 0, partM,
                     with_mix ? dmix : nullptr, mix_len, mix_per_head ? 1 : 0);
  return hipGetLastError();
}

// Linear maps of one (b, h) per output: zmix = A z (fixed matrix) or z W_c (channel map).
static GemmDesc mix_fwd_desc(const Geom& g, const MixArgs& m, const float* z, float* zmix) {
  const int64_t GV = (int64_t)g.G * g.V;
  GemmDesc d{};
  if (m.kind == 1) {  // (G x G) x (G x V)
    d = GemmDesc{m.A, g.G, 1, (int64_t)g.G * g.G, 0, m.a_per_head ? g.H : 1,
                 z, g.V, 1, GV, 0, zmix, g.V, GV, g.G, g.V, g.G, 1};
  } else {            // (G x V) x (V x V)
    d = GemmDesc{z, g.V, 1, GV, 0, 1 << 30, m.Wc, g.V, 1, 0, 0, zmix, g.V, GV, g.G, g.V, g.V, 1};
  }
  return d;
}

hipError_t launch_mix(const Geom& g, const MixArgs& m, const float* z, float* zmix,
                      float* attn, hipStream_t st) {
  const int BH = g.BH();
  if (tok_fused(g, m.kind)) return launch_tok_fwd(g, m, z, zmix, attn, st);
  if (attn_rows(g, m.kind)) {
    // four wavefronts per 16 rows hold the score tiles of up to 256 tokens, eight those of 1024
#define FS_ATTN(V_)                                                                             \
  if (g.V == V_) {                                                                              \
    const dim3 grid(BH * (g.G / 16));                                                           \
    if (g.G <= 256)                                                                             \
      hipLaunchKernelGGL((k_attn_rows<V_, 4, 4>), grid, dim3(256), 0, st, z, zmix, attn, m.Wq,  \
                         m.Wk, m.Wv, m.scale, g.G);                                             \
    else                                                                                        \
      hipLaunchKernelGGL((k_attn_rows<V_, 8, 8>), grid, dim3(512), 0, st, z, zmix, attn, m.Wq,  \
                         m.Wk, m.Wv, m.scale, g.G);                                             \
    return hipGetLastError();                                                                   \
  }
    FS_ATTN(16)
    FS_ATTN(32)
    FS_ATTN(64)
#undef FS_ATTN
    return hipErrorInvalidValue;
  }
  if (m.kind == 0) {
    return hipMemcpyAsync(zmix, z, sizeof(float) * (size_t)BH * g.G * g.V,
                          hipMemcpyDeviceToDevice, st);
  }
  return run_gemm(mix_fwd_desc(g, m, z, zmix), BH, st);
}

// The 16-token sums of the token gradients (tok_part_floats), at the start of scr.
static hipError_t finish_tokens(const Geom& g, const float* part, float* cen, const float* partW,
                                float* dmix, hipStream_t st) {
  const int ncen = cen != nullptr ? g.BH() : 0, nblk = g.G / 16;
  const int64_t len = dmix != nullptr ? mix_partial_len(g, 3) : 0;
  if (ncen == 0 && len == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tok_fin, dim3(ncen + blocks(len, kColsWide)), dim3(kRedThreads), 0, st, part,
                     cen, ncen, nblk, g.V, partW, dmix, g.BH() * nblk, len);
  return hipGetLastError();
}

// Backward of the attention: scr holds the token sums, q, k, v, D and the parameter partials
// (mix_scratch_floats).
template <int V>
static hipError_t attn_rows_bwd(const Geom& g, const MixArgs& m, const float* z, const float* s,
                                const float* zmix, const float* P, const float* dzm, float* dz,
                                float* dU, float* ds, float* cen, float* scr, float* dmix,
                                hipStream_t st) {
  const int64_t tokens = (int64_t)g.BH() * g.G, T = tokens * V;
  float* part = scr;
  float* q = part + tok_part_floats(g);
  float* k = q + T;
  float* v = k + T;
  float* D = v + T;
  float* partW = D + tokens;
  const dim3 grid((unsigned)(tokens / 16));
  hipLaunchKernelGGL((k_attn_qkv<V>), grid, dim3(192), 0, st, z, zmix, dzm, m.Wq, m.Wk, m.Wv, q, k,
                     v, D);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && zmix == nullptr) {
    hipLaunchKernelGGL((k_attn_rowdot<V>), grid, dim3(64 * kDotWaves), 0, st, P, dzm, v, D, g.G);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_attn_bwd_rows<V>), grid, dim3(512), 0, st, z, s, zmix, P, dzm, q, k, v, D,
                     m.Wq, m.Wk, m.Wv, m.scale, dz, dU, ds, part,
                     dmix != nullptr ? partW : nullptr, g.G, g.eps);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return finish_tokens(g, part, s != nullptr ? cen : nullptr, partW, dmix, st);
}

hipError_t launch_mix_bwd(const Geom& g, const MixArgs& m, const float* z, const float* s,
                          const float* zmix, const float* attn, const float* dzm, float* dz,
                          float* dU, float* ds, float* cen, float* scr, float* partM,
                          float* dmix, bool reduce_params, hipStream_t st) {
  const int BH = g.BH();
  const int64_t GV = (int64_t)g.G * g.V;
  hipError_t e = hipSuccess;
  if (tok_fused(g, m.kind)) {
    e = launch_tok_bwd(g, m, z, s, zmix, attn, dzm, dz, dU, ds, cen, partM, st);
  } else if (m.kind == 3) {
    auto bwd = g.V == 16 ? attn_rows_bwd<16> : g.V == 32 ? attn_rows_bwd<32> : attn_rows_bwd<64>;
    e = bwd(g, m, z, s, zmix, attn, dzm, dz, dU, ds, cen, scr, dmix, st);
  } else {
    if (m.kind == 0) {
      e = hipMemcpyAsync(dz, dzm, sizeof(float) * (size_t)BH * GV, hipMemcpyDeviceToDevice, st);
    } else if (m.kind == 1) {  // dz = A^T dzmix
      e = run_gemm(GemmDesc{m.A, 1, g.G, (int64_t)g.G * g.G, 0, m.a_per_head ? g.H : 1, dzm,
                            g.V, 1, GV, 0, dz, g.V, GV, g.G, g.V, g.G, 1},
                   BH, st);
    } else {                   // dz = dzmix W_c^T
      e = run_gemm(GemmDesc{dzm, g.V, 1, GV, 0, 1 << 30, m.Wc, 1, g.V, 0, 0, dz, g.V, GV, g.G,
                            g.V, g.V, 1},
                   BH, st);
    }
    if (e == hipSuccess && dmix != nullptr && m.kind == 1) {
      // dA = sum over (b, h) of dzmix z^T, or over b for each head's own A
      if (m.a_per_head)
        e = run_gemm(GemmDesc{dzm, g.V, 1, GV, (int64_t)g.H * GV, 1 << 30, z, 1, g.V, GV,
                              (int64_t)g.H * GV, dmix, g.G, (int64_t)g.G * g.G, g.G, g.G, g.V,
                              (int)g.B},
                     g.H, st);
      else
        e = run_gemm(GemmDesc{dzm, g.V, 1, 0, GV, 1, z, 1, g.V, 0, GV, dmix, g.G, 0, g.G, g.G,
                              g.V, BH},
                     1, st);
    }
    if (e == hipSuccess && dmix != nullptr && m.kind == 2)  // dW_c = sum over (b, h) of z^T dzmix
      e = run_gemm(GemmDesc{z, 1, g.V, 0, GV, 1, dzm, g.V, 1, 0, GV, dmix, g.V, 0, g.V, g.V,
                            g.G, BH},
                   1, st);
    if (e == hipSuccess && s != nullptr) {
      auto grads = g.V == 16 ? k_token_grads<16> : g.V == 32 ? k_token_grads<32> : k_token_grads<64>;
      hipLaunchKernelGGL(grads, dim3(BH * (g.G / 16)), dim3(256), 0, st, z, s, zmix, dz, dU, ds,
                         scr, g.eps);
      e = hipGetLastError();
      if (e == hipSuccess) e = finish_tokens(g, scr, cen, nullptr, nullptr, st);
    }
  }
  if (e != hipSuccess) return e;
  if (reduce_params && dmix != nullptr && m.kind != 0 && mix_params_in_partials(g, m.kind)) {
    const int64_t len = mix_partial_len(g, m.kind);
    const bool per_head = m.kind == 1 && m.a_per_head;
    dim3 grid(blocks(len, kColsWide), per_head ? g.H : 1);
    hipLaunchKernelGGL(k_reduce_mixparams, grid, dim3(kRedThreads), 0, st, partM, dmix, (int)g.B,
                       g.H, len, per_head ? 1 : 0);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace fs

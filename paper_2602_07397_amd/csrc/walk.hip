// Sketch-Determined Walk kernels (paper Sec. 2.3, Alg. 1 step 6).
//
//  walk_first_kernel    first walked layer: R = W(A), row-normalised.
//  walk_gemm16_kernel   C = X W(Y) for lower triangular X, Y. One workgroup per
//                       16x16 output tile on or below the diagonal, its four
//                       wavefronts splitting the tile's k-range (clipped to
//                       [j0, i_max]) on fp64 MFMA 16x16x4 and adding their
//                       partial tiles in a fixed order; the weight transform W
//                       is applied to the B operand. Entries above the
//                       diagonal of C are not written outside the diagonal
//                       tiles (the products never read them).
//  walk_gemm32_kernel   the same over 32x32 tiles and eight wavefronts, for
//                       long sequences; walk_gemm_mixed_kernel for calls with
//                       both
//  walk_softmax_kernel  causal row softmax of t*A (the transition matrix of
//                       the appendix lemma on the walk's stationary structure).
//  walk_norm_kernel     divides each row by its largest magnitude and writes
//                       the zeros above the diagonal.
//
// Weight transforms (template parameter): the element-wise power (A/c)^s of
// Alg. 1 step 6, the same power after clipping negative scores to zero, or
// the identity (the operand already holds weights). The matrix-power variant
// (the within-layer multi-hop walk of Sec. 1 and Fig. 2) is built from
// these products by binary exponentiation.
#include "sw_common.h"
#include "sw_internal.h"

namespace sw {

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double pow_int(double x, int s) {
  if (s == 8) {               // the paper's default exponent: three squarings
    const double x2 = x * x, x4 = x2 * x2;
    return x4 * x4;
  }
  double r = 1.0, b = x;
  while (s) {
    if (s & 1) r *= b;
    b *= b;
    s >>= 1;
  }
  return r;
}

enum WeightFn { kWPow = 0, kWRelu = 1, kWIdent = 2 };

// S8: the exponent is 8, known at compile time (the product kernel's loop must
// not branch on it per element)
template <int F, bool S8 = false>
__device__ __forceinline__ double weight_of(double a, double inv_c, int s) {
  if constexpr (F == kWIdent) return a;
  const double x = (F == kWRelu ? fmax(a, 0.0) : a) * inv_c;
  if constexpr (S8) {
    const double x2 = x * x, x4 = x2 * x2;
    return x4 * x4;
  }
  return pow_int(x, s);
}

__device__ __forceinline__ double scale_of(const double* A_scale, int s) {
  const double c = A_scale[s];
  return c > 0.0 ? c : 1.0;
}

__device__ __forceinline__ double block_max_256(double v, double* tmp) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  if ((threadIdx.x & 63) == 0) tmp[threadIdx.x >> 6] = v;
  __syncthreads();
  v = fmax(fmax(tmp[0], tmp[1]), fmax(tmp[2], tmp[3]));
  __syncthreads();
  return v;
}

__device__ __forceinline__ double block_sum_256(double v, double* tmp) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if ((threadIdx.x & 63) == 0) tmp[threadIdx.x >> 6] = v;
  __syncthreads();
  v = (tmp[0] + tmp[1]) + (tmp[2] + tmp[3]);
  __syncthreads();
  return v;
}

// NORM = false writes W(A) itself (the factor of a matrix power).
template <int F, bool NORM = true>
__global__ __launch_bounds__(256) void walk_first_kernel(const double* __restrict__ A,
                                                         const double* __restrict__ A_scale,
                                                         int s_exp, SeqMeta m,
                                                         double* __restrict__ R) {
  __shared__ double tmp[4];
  const int row = blockIdx.x;
  const int s = seq_of_block(m, row);
  const int i = row - m.blk_start[s];
  const int b = m.blk_start[s + 1] - m.blk_start[s];
  const double inv_c = F == kWIdent ? 1.0 : 1.0 / scale_of(A_scale, s);
  const double* Ar = A + m.mat_start[s] + (long long)i * b;
  double* Rr = R + m.mat_start[s] + (long long)i * b;
  double mx = 0.0;
  for (int j = threadIdx.x; j < b; j += 256) {
    const double w = (j <= i) ? weight_of<F>(Ar[j], inv_c, s_exp) : 0.0;
    Rr[j] = w;
    mx = fmax(mx, fabs(w));
  }
  if (!NORM) return;
  mx = block_max_256(mx, tmp);
  if (mx > 0.0) {
    const double inv = 1.0 / mx;
    for (int j = threadIdx.x; j <= i; j += 256) Rr[j] = Rr[j] * inv;
  }
}

// Bounded by the launch and one chain of loads up to about 256 blocks, then by
// the L2 reads (each operand entry is read for 16 rows or columns).
// wave is the wavefront's number among the tile's four; store: false for four
// that only keep the barrier.
template <int F, bool S8>
__device__ __forceinline__ void gemm16_tile(const double* __restrict__ A,
                                            const double* __restrict__ A_scale, int s_exp,
                                            const SeqMeta& m, int tile, const double* __restrict__ Rp,
                                            double* __restrict__ R, int wave, double (*red)[64][4],
                                            bool store) {
  const int l = threadIdx.x & 63;
  int s = 0;
  while (s + 1 < m.n_seqs && m.aux_start[s + 1] <= tile) ++s;
  const int b = m.blk_start[s + 1] - m.blk_start[s];
  const int tb = (b + 15) >> 4;
  // Lower tiles only, longest k-range first: group g = 0, 1, ... holds the
  // g + 1 tiles of diagonal ti - tj = tb - 1 - g.
  const int lt = tile - m.aux_start[s];
  int g = (int)((sqrt(8.0 * lt + 1.0) - 1.0) * 0.5);
  while ((g + 1) * (g + 2) / 2 <= lt) ++g;
  while (g * (g + 1) / 2 > lt) --g;
  const int tj = lt - g * (g + 1) / 2;
  const int ti = tj + tb - 1 - g;
  const double* As = A + m.mat_start[s];
  const double* Ps = Rp + m.mat_start[s];
  double* Rs = R + m.mat_start[s];
  const double inv_c = F == kWIdent ? 1.0 : 1.0 / scale_of(A_scale, s);
  const int ra = ti * 16 + (l & 15);   // A-operand row (output row)
  const int cb = tj * 16 + (l & 15);   // B-operand column (output column)
  const int kend = min(ti * 16 + 15, b - 1);
  // 32 k per chunk, 8 MFMA steps; in step u, lane group q = l / 16 carries
  // k = k0 + 8 (u / 2) + 2 q + u % 2 (the sum runs over every k once, in any
  // order), so the four groups read 64 consecutive bytes of an A row at a time.
  // Wavefront w takes chunks w, w + 4, w + 8, ...; its chunks are
  // double-buffered in registers: the loads of the next chunk are in flight
  // during the MFMAs of the current one. That, and an exponent known to the
  // compiler (a branch per element stood between the MFMAs), took a walk and
  // selection from 13.8 to 13.2 us at 256 blocks and 19.6 to 18.7 at 512.
  const int kq = l >> 4;
  const long long rowA = (long long)min(ra, b - 1) * b;
  const int cbc = min(cb, b - 1);
  // the loads carry no condition (indices clamped into the matrix; the
  // entries outside the causal range are zeroed after loading), so all of a
  // chunk's loads are in flight together
  auto load = [&](int k0, double (&av)[8], double (&bv)[8]) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + 8 * (u >> 1) + 2 * kq + (u & 1);
      const int kc = min(k, b - 1);
      av[u] = Ps[rowA + kc];
      bv[u] = As[(long long)kc * b + cbc];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + 8 * (u >> 1) + 2 * kq + (u & 1);
      av[u] = (ra < b && k <= ra) ? av[u] : 0.0;
      bv[u] = (k < b && cb <= k) ? bv[u] : 0.0;
    }
  };
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  auto compute = [&](const double (&av)[8], const double (&bv)[8]) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], weight_of<F, S8>(bv[u], inv_c, s_exp), acc, 0,
                                                 0, 0);
  };
  double a0[8], b0[8], a1[8], b1[8];
  int k0 = tj * 16 + 32 * wave;
  if (k0 <= kend) load(k0, a0, b0);
  for (; k0 <= kend; k0 += 256) {
    if (k0 + 128 <= kend) load(k0 + 128, a1, b1);
    compute(a0, b0);
    if (k0 + 128 > kend) break;
    if (k0 + 256 <= kend) load(k0 + 256, a0, b0);
    compute(a1, b1);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][l][v] = acc[v];
  __syncthreads();
  if (wave != 0 || !store) return;
  for (int v = 0; v < 4; ++v) {
    const double sum = ((red[0][l][v] + red[1][l][v]) + red[2][l][v]) + red[3][l][v];
    const int ri = ti * 16 + (l >> 4) + 4 * v, cj = tj * 16 + (l & 15);
    if (ri < b && cj < b) Rs[(long long)ri * b + cj] = (cj <= ri) ? sum : 0.0;
  }
}

template <int F, bool S8>
__global__ __launch_bounds__(256) void walk_gemm16_kernel(const double* __restrict__ A,
                                                        const double* __restrict__ A_scale,
                                                        int s_exp, SeqMeta m,
                                                        const double* __restrict__ Rp,
                                                        double* __restrict__ R) {
  __shared__ double red[4][64][4];
  gemm16_tile<F, S8>(A, A_scale, s_exp, m, blockIdx.x, Rp, R, threadIdx.x >> 6, red, true);
}

// Four 16x16 products per wavefront and step share two A and two B operands, so
// an operand entry is read for 32 rows or columns. Bounded by those reads:
// both matrices pass through every XCD's L2 (62 MB from the memory side at 1024
// blocks), about 4 us of waiting per wavefront against 5 us of matrix work on
// the whole chip, so sixteen wavefronts per CU with one chunk of registers
// each (127 VGPRs) are a little faster than eight with two. The product went
// from 34.5 to 22 us at 1024 blocks. Tile rows kept on one XCD brought nothing.
constexpr int kGemmTile = 32;
constexpr int kGemmWaves = 8;

struct __attribute__((packed, aligned(8))) f64pair {   // two neighbours, 8-byte aligned
  double x, y;
};

template <int F, bool S8>
__device__ __forceinline__ void gemm32_tile(const double* __restrict__ A,
                                            const double* __restrict__ A_scale, int s_exp,
                                            const SeqMeta& m, int tile, const double* __restrict__ Rp,
                                            double* __restrict__ R, double (*red)[16][64]) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63;
  int s = 0;
  while (s + 1 < m.n_seqs && m.aux_start[s + 1] <= tile) ++s;
  const int b = m.blk_start[s + 1] - m.blk_start[s];
  const int tb = (b + kGemmTile - 1) / kGemmTile;
  // Lower tiles only, longest k-range first: group g = 0, 1, ... holds the
  // g + 1 tiles of diagonal ti - tj = tb - 1 - g.
  const int lt = tile - m.aux_start[s];
  int g = (int)((sqrt(8.0 * lt + 1.0) - 1.0) * 0.5);
  while ((g + 1) * (g + 2) / 2 <= lt) ++g;
  while (g * (g + 1) / 2 > lt) --g;
  const int tj = lt - g * (g + 1) / 2;
  const int ti = tj + tb - 1 - g;
  const double* As = A + m.mat_start[s];
  const double* Ps = Rp + m.mat_start[s];
  double* Rs = R + m.mat_start[s];
  const double inv_c = F == kWIdent ? 1.0 : 1.0 / scale_of(A_scale, s);
  const int i0 = ti * kGemmTile, j0 = tj * kGemmTile;
  const int ra = i0 + (l & 15);        // A-operand rows ra, ra + 16 (output rows)
  const int cb = j0 + 2 * (l & 15);    // B-operand columns cb, cb + 1 (output columns)
  const int kq = 2 * (l >> 4);
  // 32 k per chunk, 8 MFMA steps; in step u, lane group q = l / 16 carries
  // k = k0 + 8 (u / 2) + 2 q + u % 2 (the sum runs over every k once, in any
  // order), so the four groups read 64 consecutive bytes of an A row at a time
  // (with 8 consecutive entries per lane an instruction touched 64 pieces of
  // 16 bytes, and the CU's one address unit was the bound). Wavefront w takes
  // chunks w, w + kGemmWaves, ...
  const int nc = ti - tj + 1;
  const long long row0 = (long long)min(ra, b - 1) * b, row1 = (long long)min(ra + 16, b - 1) * b;
  struct Chunk {
    double a0[8], a1[8], b0[8], b1[8];
  };
  auto load = [&](int c, Chunk& x) {
    const int k0 = j0 + c * kGemmTile + kq;
    if (c > 0 && c < nc - 1) {           // wholly inside both triangles
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        const f64pair p0 = *reinterpret_cast<const f64pair*>(Ps + row0 + k0 + 4 * u);
        const f64pair p1 = *reinterpret_cast<const f64pair*>(Ps + row1 + k0 + 4 * u);
        x.a0[u] = p0.x;
        x.a0[u + 1] = p0.y;
        x.a1[u] = p1.x;
        x.a1[u + 1] = p1.y;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const f64pair q =
            *reinterpret_cast<const f64pair*>(As + (long long)(k0 + 8 * (u >> 1) + (u & 1)) * b + cb);
        x.b0[u] = q.x;
        x.b1[u] = q.y;
      }
      return;
    }
    // the first and last chunk: loads without a condition (indices clamped
    // into the matrix), the entries outside the causal range zeroed after
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int kc = min(k0 + 8 * (u >> 1) + (u & 1), b - 1);
      x.a0[u] = Ps[row0 + kc];
      x.a1[u] = Ps[row1 + kc];
      x.b0[u] = As[(long long)kc * b + min(cb, b - 1)];
      x.b1[u] = As[(long long)kc * b + min(cb + 1, b - 1)];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + 8 * (u >> 1) + (u & 1);
      x.a0[u] = (ra < b && k <= ra) ? x.a0[u] : 0.0;
      x.a1[u] = (ra + 16 < b && k <= ra + 16) ? x.a1[u] : 0.0;
      x.b0[u] = (k < b && cb <= k) ? x.b0[u] : 0.0;
      x.b1[u] = (k < b && cb + 1 <= k) ? x.b1[u] : 0.0;
    }
  };
  f64x4 acc[2][2];                       // [row half][column parity]
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q) acc[p][q] = f64x4{0.0, 0.0, 0.0, 0.0};
  auto compute = [&](const Chunk& x) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double w0 = weight_of<F, S8>(x.b0[u], inv_c, s_exp);
      const double w1 = weight_of<F, S8>(x.b1[u], inv_c, s_exp);
      acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a0[u], w0, acc[0][0], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a1[u], w0, acc[1][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a0[u], w1, acc[0][1], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a1[u], w1, acc[1][1], 0, 0, 0);
    }
  };
  Chunk x;
#pragma unroll 1
  for (int c = wave; c < nc; c += kGemmWaves) {
    load(c, x);
    compute(x);
  }
  // element e = 8 p + 2 v + q: row i0 + 16 p + l / 16 + 4 v, column cb + q
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int q = 0; q < 2; ++q) red[wave][8 * p + 2 * v + q][l] = acc[p][q][v];
  __syncthreads();
#pragma unroll
  for (int z = 0; z < 8 / kGemmWaves; ++z) {
    const int pv = wave + z * kGemmWaves;  // a pair of elements (p, v)
    double s0 = red[0][2 * pv][l], s1 = red[0][2 * pv + 1][l];
#pragma unroll
    for (int w = 1; w < kGemmWaves; ++w) {
      s0 += red[w][2 * pv][l];
      s1 += red[w][2 * pv + 1][l];
    }
    const int ri = i0 + 16 * (pv >> 2) + (l >> 4) + 4 * (pv & 3);
    if (ri < b) {
      double* o = Rs + (long long)ri * b + cb;
      if (cb < b) o[0] = (cb <= ri) ? s0 : 0.0;
      if (cb + 1 < b) o[1] = (cb + 1 <= ri) ? s1 : 0.0;
    }
  }
}

template <int F, bool S8>
__global__ __launch_bounds__(kGemmWaves * 64, 4) void walk_gemm32_kernel(
    const double* __restrict__ A, const double* __restrict__ A_scale, int s_exp, SeqMeta m,
    const double* __restrict__ Rp, double* __restrict__ R) {
  __shared__ double red[kGemmWaves][16][64];
  gemm32_tile<F, S8>(A, A_scale, s_exp, m, blockIdx.x, Rp, R, red);
}

// Sequences of both kinds in one launch: the total32 tiles of 32 first, then the
// total16 of 16, two per workgroup (three sequences of 600, 500 and 400 blocks:
// 32 us with walk and selection, 39 in two launches, 29 all on tiles of 32).
template <int F, bool S8>
__global__ __launch_bounds__(kGemmWaves * 64, 4) void walk_gemm_mixed_kernel(
    const double* __restrict__ A, const double* __restrict__ A_scale, int s_exp, SeqMeta m32,
    int total32, SeqMeta m16, int total16, const double* __restrict__ Rp, double* __restrict__ R) {
  __shared__ double red[kGemmWaves][16][64];
  if ((int)blockIdx.x < total32) {
    gemm32_tile<F, S8>(A, A_scale, s_exp, m32, blockIdx.x, Rp, R, red);
    return;
  }
  const int wave = threadIdx.x >> 6, half = wave >> 2;
  const int tile = 2 * ((int)blockIdx.x - total32) + half;
  auto red16 = reinterpret_cast<double(*)[64][4]>(&red[0][0][0]) + 4 * half;
  gemm16_tile<F, S8>(A, A_scale, s_exp, m16, min(tile, total16 - 1), Rp, R, wave & 3, red16,
                     tile < total16);
}

// Row i of W: exp(t A[i,j] - max) / sum over the causal blocks j <= i; zeros
// above the diagonal. The exponentials are stored, then scaled by 1/sum by
// the same thread that wrote them.
__global__ __launch_bounds__(256) void walk_softmax_kernel(const double* __restrict__ A,
                                                           double t, SeqMeta m,
                                                           double* __restrict__ W) {
  __shared__ double tmp[4];
  const int row = blockIdx.x;
  const int s = seq_of_block(m, row);
  const int i = row - m.blk_start[s];
  const int b = m.blk_start[s + 1] - m.blk_start[s];
  const double* Ar = A + m.mat_start[s] + (long long)i * b;
  double* Wr = W + m.mat_start[s] + (long long)i * b;
  double mx = -INFINITY;
  for (int j = threadIdx.x; j <= i; j += 256) mx = fmax(mx, t * Ar[j]);
  mx = block_max_256(mx, tmp);
  double sum = 0.0;
  for (int j = threadIdx.x; j < b; j += 256) {
    const double e = (j <= i) ? exp(t * Ar[j] - mx) : 0.0;
    Wr[j] = e;
    sum += e;
  }
  sum = block_sum_256(sum, tmp);
  const double inv = 1.0 / sum;
  for (int j = threadIdx.x; j <= i; j += 256) Wr[j] = Wr[j] * inv;
}

__global__ __launch_bounds__(256) void walk_norm_kernel(SeqMeta m, double* __restrict__ R) {
  __shared__ double tmp[4];
  const int row = blockIdx.x;
  const int s = seq_of_block(m, row);
  const int i = row - m.blk_start[s];
  const int b = m.blk_start[s + 1] - m.blk_start[s];
  double* Rr = R + m.mat_start[s] + (long long)i * b;
  double mx = 0.0;
  for (int j = threadIdx.x; j <= i; j += 256) mx = fmax(mx, fabs(Rr[j]));
  mx = block_max_256(mx, tmp);
  const double inv = mx > 0.0 ? 1.0 / mx : 1.0;
  for (int j = threadIdx.x; j < b; j += 256) Rr[j] = (j <= i) ? Rr[j] * inv : 0.0;
}

namespace {

// Edge of a sequence's output tiles. Measured (walk and selection, 16 / 32): 13.2
// / 14.3 us at 256 blocks, 18.7 / 19.1 at 512, 39.7 / 35.2 at 1000. The two take
// a tile's sums in different orders; by the sequence's own length, its bits do
// not depend on what else is in the call.
int gemm_edge(int b) { return b > 512 ? kGemmTile : 16; }

// The tiles of the sequences with edge 16 and of those with edge 32, each in
// aux_start of its own copy of the layout.
struct GemmTiles {
  SeqMeta m16, m32;
  int total16, total32;
};

int count_tiles(const SeqMeta& meta, int edge, SeqMeta* m2) {
  *m2 = meta;
  int total = 0;
  for (int s = 0; s < meta.n_seqs; ++s) {
    m2->aux_start[s] = total;
    const int b = meta.blk_start[s + 1] - meta.blk_start[s];
    const int tb = (b + edge - 1) / edge;
    if (gemm_edge(b) == edge) total += tb * (tb + 1) / 2;
  }
  m2->aux_start[meta.n_seqs] = total;
  return total;
}

// C = X W(Y): X, Y, C lower triangular per sequence; only the lower
// triangle of C (and the diagonal tiles) is written.
template <int F, bool S8>
void gemm_s(const double* X, const double* Y, const double* A_scale, int s_exp, const GemmTiles& g,
            double* C, hipStream_t st) {
  if (g.total16 == 0)
    hipLaunchKernelGGL((walk_gemm32_kernel<F, S8>), dim3((unsigned)g.total32), dim3(kGemmWaves * 64), 0,
                       st, Y, A_scale, s_exp, g.m32, X, C);
  else if (g.total32 == 0)
    hipLaunchKernelGGL((walk_gemm16_kernel<F, S8>), dim3((unsigned)g.total16), dim3(256), 0, st, Y,
                       A_scale, s_exp, g.m16, X, C);
  else
    hipLaunchKernelGGL((walk_gemm_mixed_kernel<F, S8>), dim3((unsigned)(g.total32 + (g.total16 + 1) / 2)),
                       dim3(kGemmWaves * 64), 0, st, Y, A_scale, s_exp, g.m32, g.total32, g.m16, g.total16,
                       X, C);
}

template <int F>
void gemm(const double* X, const double* Y, const double* A_scale, int s_exp, const GemmTiles& g,
          double* C, hipStream_t st) {
  if (s_exp == 8 && F != kWIdent)
    gemm_s<F, F != kWIdent>(X, Y, A_scale, s_exp, g, C, st);
  else
    gemm_s<F, false>(X, Y, A_scale, s_exp, g, C, st);
}

}  // namespace

int64_t walk_workspace_bytes(int variant, int64_t nm) {
  if (variant == SW_WALK_SOFTMAX) return 8 * nm;
  if (variant == SW_WALK_MATPOW) return 16 * nm;
  return 0;
}

hipError_t launch_walk(int variant, const double* A, const double* A_scale, int s_exp,
                       double logit_scale, const SeqMeta& meta, int64_t nb, const double* R_prev,
                       double* R_out, double* ws, hipStream_t st) {
  const dim3 rows((unsigned)nb), blk(256);
  GemmTiles g;
  g.total16 = count_tiles(meta, 16, &g.m16);
  g.total32 = count_tiles(meta, kGemmTile, &g.m32);
  if (variant == SW_WALK_MATPOW && s_exp == 1) variant = SW_WALK_POWER;  // X^1 = X
  switch (variant) {
    case SW_WALK_POWER:
    case SW_WALK_RELU:
      if (R_prev == nullptr) {
        if (variant == SW_WALK_POWER)
          hipLaunchKernelGGL(walk_first_kernel<kWPow>, rows, blk, 0, st, A, A_scale, s_exp, meta,
                             R_out);
        else
          hipLaunchKernelGGL(walk_first_kernel<kWRelu>, rows, blk, 0, st, A, A_scale, s_exp, meta,
                             R_out);
        return hipGetLastError();
      }
      if (variant == SW_WALK_POWER)
        gemm<kWPow>(R_prev, A, A_scale, s_exp, g, R_out, st);
      else
        gemm<kWRelu>(R_prev, A, A_scale, s_exp, g, R_out, st);
      break;
    case SW_WALK_SOFTMAX: {
      double* W = R_prev == nullptr ? R_out : ws;
      hipLaunchKernelGGL(walk_softmax_kernel, rows, blk, 0, st, A, logit_scale, meta, W);
      if (R_prev != nullptr) gemm<kWIdent>(R_prev, W, nullptr, 1, g, R_out, st);
      break;
    }
    case SW_WALK_MATPOW: {
      // Left-to-right binary exponentiation of X = A/c: square for every bit
      // below the leading one, multiply by X (read from A through the s = 1
      // power) where the bit is set. Two ping-pong buffers; without R_prev
      // the last product is written to R_out directly.
      const int64_t nm = meta.mat_start[meta.n_seqs];
      double* buf[2] = {ws, ws + nm};
      const int top = 31 - __builtin_clz((unsigned)s_exp);
      int nprod = 0;
      for (int bit = top - 1; bit >= 0; --bit) nprod += 1 + ((s_exp >> bit) & 1);
      hipLaunchKernelGGL((walk_first_kernel<kWPow, false>), rows, blk, 0, st, A, A_scale, 1, meta,
                         buf[0]);
      const double* cur = buf[0];
      int ci = 0, k = 0;
      for (int bit = top - 1; bit >= 0; --bit) {
        const int steps = 1 + ((s_exp >> bit) & 1);
        for (int step = 0; step < steps; ++step) {
          const bool last = ++k == nprod;
          double* dst = (last && R_prev == nullptr) ? R_out : buf[1 - ci];
          if (step == 0)
            gemm<kWIdent>(cur, cur, nullptr, 1, g, dst, st);
          else
            gemm<kWPow>(cur, A, A_scale, 1, g, dst, st);
          cur = dst;
          ci = 1 - ci;
        }
      }
      if (R_prev != nullptr) gemm<kWIdent>(R_prev, cur, nullptr, 1, g, R_out, st);
      break;
    }
    default:
      return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL(walk_norm_kernel, rows, blk, 0, st, meta, R_out);
  return hipGetLastError();
}

}  // namespace sw

// Small-World Sketching kernels (paper Sec. 2.2, Alg. 1 steps 1-5).
//
//  pool_sketch_kernel  one workgroup per block row: streams the row's tokens
//                      of every query head and every KV head once from HBM
//                      (16-byte non-temporal loads), sums them in fp64 (lanes
//                      of a wavefront combined by lane exchanges, then the
//                      wavefronts in a fixed order), divides by heads x
//                      tokens, applies the random signs, runs the
//                      Walsh-Hadamard transform of the query mean and of the
//                      key mean (one wavefront each, lane exchanges), samples
//                      the columns and scales by 1/sqrt(r).
//  pool_split_kernel   for few block rows: the work of each of a row's
//                      wavefronts spread over a workgroup, which leaves its
//                      sums in the workspace;
//  sketch_parts_kernel adds them and goes on from there.
//  scores_kernel       A = Qs Ks^T / sqrt(r) with fp64 MFMA 16x16x4 tiles,
//                      causal mask, per-sequence max |A| by integer atomicMax
//                      on the (non-negative) double bit pattern.
#include <type_traits>

#include "sw_common.h"
#include "sw_internal.h"

#define SW_STR2(x) #x
#define SW_STR(x) SW_STR2(x)

namespace sw {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

#ifndef SW_POOL_THREADS
#define SW_POOL_THREADS 512
#endif
constexpr int kPoolThreads = SW_POOL_THREADS;
#ifndef SW_POOL_UNROLL
#define SW_POOL_UNROLL 8
#endif
constexpr int kPoolWaves = kPoolThreads / 64;
#ifndef SW_POOL_AHEAD
#define SW_POOL_AHEAD 32                 // loads in flight per thread of a split row
#endif

// The rest of a block row's sketch from the sums of its queries and keys
// (thread t < d holds dimension t's): means, signs, the two transforms, the
// sampled columns. x holds 2 * 256 doubles of LDS; the whole workgroup calls it.
__device__ __forceinline__ void finish_row(double sq, double sk, int row, int cnt, int h_q, int h_kv,
                                           int d, const int8_t* __restrict__ signs,
                                           const int32_t* __restrict__ cols, int r,
                                           double* __restrict__ Qs, double* __restrict__ Ks,
                                           double* __restrict__ Qbar, double* __restrict__ Kbar,
                                           double* x) {
  double* xq = x;
  double* xk = x + 256;
  const int t = threadIdx.x;
  if (t < d) {
    const double mq = sq / ((double)h_q * (double)cnt);
    const double mk = sk / ((double)h_kv * (double)cnt);
    if (Qbar) Qbar[(long long)row * d + t] = mq;
    if (Kbar) Kbar[(long long)row * d + t] = mk;
    const double sg = (double)signs[t];
    xq[t] = mq * sg;
    xk[t] = mk * sg;
  }
  __syncthreads();
  if ((t >> 6) == 0) wave_fwht(xq, d);
  else if ((t >> 6) == 1) wave_fwht(xk, d);
  __syncthreads();
  if (t < r) {
    const int c = cols[t] & (d - 1);
    Qs[(long long)row * r + t] = xq[c] / sqrt((double)r);
    Ks[(long long)row * r + t] = xk[c] / sqrt((double)r);
  }
}

template <typename T>
__global__ __launch_bounds__(kPoolThreads) void pool_sketch_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, int h_q, int h_kv, int d, SeqMeta m,
    long long N, const int8_t* __restrict__ signs, const int32_t* __restrict__ cols, int r,
    double* __restrict__ Qs, double* __restrict__ Ks, double* __restrict__ Qbar,
    double* __restrict__ Kbar, double* __restrict__ A_scale) {
  constexpr int VEC = 16 / sizeof(T);
  constexpr int NW = kPoolWaves;
  // per-wavefront sums of the query and key means, then (reused) the two
  // vectors the transforms work on
  __shared__ double red[2 * NW * 256];
  double* redq = red;
  double* redk = red + NW * 256;
  const int row = blockIdx.x;
  const int s = seq_of_block(m, row);
  const int i = row - m.blk_start[s];
  const int t0 = m.tok_start[s] + i * m.B;
  const int cnt = min(m.tok_start[s + 1], t0 + m.B) - t0;
  const int t = threadIdx.x;
  const int lpr = d / VEC;               // lanes per token row (2 .. 64)
  const int slots = kPoolThreads / lpr;  // token rows in flight per pass
  const int lane = t % lpr;
  const int slot = t / lpr;
  if (i == 0 && t == 0) A_scale[s] = 0.0;

  auto add = [](double (&acc)[VEC], const T* p) {
    // non-temporal: Q and K are streamed once here
    const u32x4 vv = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[2 * e] += (double)__uint_as_float(vv[e] << 16);
        acc[2 * e + 1] += (double)__uint_as_float(vv[e] & 0xffff0000u);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += (double)__uint_as_float(vv[e]);
    }
  };
  // item it = head * cnt + token, slot-strided
  double aq[VEC], ak[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) aq[e] = ak[e] = 0.0;
  // items (head, token) in head-major order, `slots` apart: the head and
  // token of the next item follow by subtraction, not division
  const int dh = slots / cnt, dt = slots % cnt;
  // (two loops written out: through one function of the operand they compiled
  // to 164 VGPRs instead of 92 and took twice the time)
  {
    const int n = h_q * cnt;
    int h = slot / cnt, tok = slot % cnt;
_Pragma(SW_STR(unroll SW_POOL_UNROLL))
    for (int it = slot; it < n; it += slots) {
      add(aq, Q + ((long long)h * N + t0 + tok) * d + lane * VEC);
      h += dh;
      tok += dt;
      if (tok >= cnt) {
        tok -= cnt;
        ++h;
      }
    }
  }
  {
    const int n = h_kv * cnt;
    int h = slot / cnt, tok = slot % cnt;
_Pragma(SW_STR(unroll SW_POOL_UNROLL))
    for (int it = slot; it < n; it += slots) {
      add(ak, K + ((long long)h * N + t0 + tok) * d + lane * VEC);
      h += dh;
      tok += dt;
      if (tok >= cnt) {
        tok -= cnt;
        ++h;
      }
    }
  }
  // the slots of a wavefront share dimensions across lanes lpr apart
  for (int off = lpr; off < 64; off <<= 1) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      aq[e] += __shfl_xor(aq[e], off);
      ak[e] += __shfl_xor(ak[e], off);
    }
  }
  const int wv = t >> 6;
  if ((t & 63) < lpr) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      redq[wv * d + lane * VEC + e] = aq[e];
      redk[wv * d + lane * VEC + e] = ak[e];
    }
  }
  __syncthreads();
  double sq = 0.0, sk = 0.0;
  if (t < d) {
    for (int w = 0; w < NW; ++w) {
      sq += redq[w * d + t];
      sk += redk[w * d + t];
    }
  }
  __syncthreads();                       // the sums are read; the vectors reuse them
  finish_row(sq, sk, row, cnt, h_q, h_kv, d, signs, cols, r, Qs, Ks, Qbar, Kbar, red);
}

// The sums of wavefront blockIdx.y of pool_sketch_kernel's workgroup for a row,
// by a workgroup of VEC / 2 times the threads: each takes two of the dimensions
// of a slot and adds the slot's items in the same order, and the slots are added
// in the order of the lane exchanges, so that a row's bits do not depend on which
// of the kernels summed it. To parts [row][wavefront][query, key][d].
template <typename T>
__global__ __launch_bounds__(256) void pool_split_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, int h_q, int h_kv, int d, SeqMeta m,
    long long N, double* __restrict__ A_scale, double* __restrict__ parts) {
  constexpr int VEC = 16 / sizeof(T);
  constexpr int NT = 32 * VEC;
  typedef typename std::conditional<sizeof(T) == 2, uint32_t, unsigned long long>::type Pair;
  __shared__ double red[4][NT];
  const int row = blockIdx.x;
  const int s = seq_of_block(m, row);
  const int i = row - m.blk_start[s];
  const int t0 = m.tok_start[s] + i * m.B;
  const int cnt = min(m.tok_start[s + 1], t0 + m.B) - t0;
  const int t = threadIdx.x;
  const int wslots = 64 * VEC / d;       // slots of the wavefront
  const int slots = kPoolWaves * wslots;
  const int sl = t / (d / 2), dim = 2 * (t % (d / 2));
  const int slot = blockIdx.y * wslots + sl;
  if (i == 0 && t == 0 && blockIdx.y == 0) A_scale[s] = 0.0;
  const int dh = slots / cnt, dt = slots % cnt;
  auto sums = [&](double (&acc)[2], const T* X, int heads) {
    acc[0] = acc[1] = 0.0;
    const int n = heads * cnt;
    int h = slot / cnt, tok = slot % cnt;
    for (int it = slot; it < n; it += SW_POOL_AHEAD * slots) {
      Pair v[SW_POOL_AHEAD];
#pragma unroll
      for (int u = 0; u < SW_POOL_AHEAD; ++u) {
        // past the last item the loads are of other items and count as zeros
        v[u] = __builtin_nontemporal_load(
            reinterpret_cast<const Pair*>(X + ((long long)min(h, heads - 1) * N + t0 + tok) * d + dim));
        h += dh;
        tok += dt;
        if (tok >= cnt) {
          tok -= cnt;
          ++h;
        }
      }
      __builtin_amdgcn_sched_barrier(0);   // the loads stay together
#pragma unroll
      for (int u = 0; u < SW_POOL_AHEAD; ++u) {
        const Pair x = it + u * slots < n ? v[u] : 0;
        if constexpr (sizeof(T) == 2) {
          acc[0] += (double)__uint_as_float(x << 16);
          acc[1] += (double)__uint_as_float(x & 0xffff0000u);
        } else {
          acc[0] += (double)__uint_as_float((uint32_t)x);
          acc[1] += (double)__uint_as_float((uint32_t)(x >> 32));
        }
      }
    }
  };
  double aq[2], ak[2];
  sums(aq, Q, h_q);
  sums(ak, K, h_kv);
  double* x[4] = {&red[0][t], &red[1][t], &red[2][t], &red[3][t]};
  *x[0] = aq[0];
  *x[1] = aq[1];
  *x[2] = ak[0];
  *x[3] = ak[1];
  for (int off = 1; off < wslots; off <<= 1) {
    __syncthreads();
    if (sl % (2 * off) == 0)
      for (int c = 0; c < 4; ++c) *x[c] += x[c][off * (d / 2)];
  }
  if (sl == 0) {                         // its own sums
    double* o = parts + ((long long)row * kPoolWaves + blockIdx.y) * 2 * d + dim;
    o[0] = *x[0];
    o[1] = *x[1];
    o[d] = *x[2];
    o[d + 1] = *x[3];
  }
}

// Block rows whose wavefronts' sums lie in parts: added in order, then the rest
// of the sketch.
__global__ __launch_bounds__(256) void sketch_parts_kernel(
    const double* __restrict__ parts, int h_q, int h_kv, int d, SeqMeta m,
    const int8_t* __restrict__ signs, const int32_t* __restrict__ cols, int r,
    double* __restrict__ Qs, double* __restrict__ Ks, double* __restrict__ Qbar,
    double* __restrict__ Kbar) {
  __shared__ double x[2 * 256];
  const int row = blockIdx.x;
  const int t = threadIdx.x;
  const double* p = parts + (long long)row * kPoolWaves * 2 * d + min(t, d - 1);
  // every load goes out before the first sum
  double vq[kPoolWaves], vk[kPoolWaves];
#pragma unroll
  for (int w = 0; w < kPoolWaves; ++w) {
    vq[w] = p[w * 2 * d];
    vk[w] = p[w * 2 * d + d];
  }
  double sq = 0.0, sk = 0.0;
#pragma unroll
  for (int w = 0; w < kPoolWaves; ++w) {
    sq += vq[w];
    sk += vk[w];
  }
  const int s = seq_of_block(m, row);
  const int t0 = m.tok_start[s] + (row - m.blk_start[s]) * m.B;
  const int cnt = min(m.tok_start[s + 1], t0 + m.B) - t0;
  finish_row(sq, sk, row, cnt, h_q, h_kv, d, signs, cols, r, Qs, Ks, Qbar, Kbar, x);
}

// Four 16 x 16 tiles per workgroup, one per wavefront; the per-sequence max
// |A| is reduced over the workgroup's tiles first, so a sequence receives one
// atomicMax per workgroup. The k-range is taken in chunks of 64: in a chunk,
// lane group q = l / 16 carries k = 64 c + 16 q + u in MFMA step u (the dot
// product runs over every k once), so each lane reads 16 consecutive entries
// of its row; every load of a chunk is issued before the first MFMA (indices
// clamped, entries past r zeroed after the load).
__global__ __launch_bounds__(256) void scores_kernel(const double* __restrict__ Qs,
                                                     const double* __restrict__ Ks, int r,
                                                     SeqMeta m,
                                                     int total_tiles, double* __restrict__ A,
                                                     double* __restrict__ A_scale) {
  __shared__ double wmax[4];
  __shared__ int wseq[4];
  const int wave = threadIdx.x >> 6;
  const int l = threadIdx.x & 63;
  const int tile = blockIdx.x * 4 + wave;
  double maxabs = 0.0;
  int s = -1;
  if (tile < total_tiles) {
    // sequence owning the tile (aux_start holds the per-sequence tile prefix)
    s = 0;
    while (s + 1 < m.n_seqs && m.aux_start[s + 1] <= tile) ++s;
    const int b = m.blk_start[s + 1] - m.blk_start[s];
    const int tb = (b + 15) >> 4;
    const int lt = tile - m.aux_start[s];
    const int ti = lt / tb, tj = lt % tb;
    const int bo = m.blk_start[s];
    double* As = A + m.mat_start[s];
    const double rs = 1.0 / sqrt((double)r);
    if (tj > ti) {
      for (int v = 0; v < 4; ++v) {
        const int ri = ti * 16 + (l >> 4) + 4 * v, cj = tj * 16 + (l & 15);
        if (ri < b && cj < b) As[(long long)ri * b + cj] = 0.0;
      }
    } else {
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      // rows past the sequence's last block are clamped (their results are
      // not stored)
      const double* qa = Qs + (long long)(bo + min(ti * 16 + (l & 15), b - 1)) * r;
      const double* kb = Ks + (long long)(bo + min(tj * 16 + (l & 15), b - 1)) * r;
      const int kq = 16 * (l >> 4);
      for (int c0 = 0; c0 < r; c0 += 64) {
        double av[16], bv[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const int k = min(c0 + kq + u, r - 1);
          av[u] = qa[k];
          bv[u] = kb[k];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const bool in = c0 + kq + u < r;
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? av[u] : 0.0, in ? bv[u] : 0.0, acc, 0,
                                                     0, 0);
        }
      }
      for (int v = 0; v < 4; ++v) {
        const int ri = ti * 16 + (l >> 4) + 4 * v, cj = tj * 16 + (l & 15);
        if (ri < b && cj < b) {
          const double val = (cj <= ri) ? acc[v] * rs : 0.0;
          As[(long long)ri * b + cj] = val;
          maxabs = fmax(maxabs, fabs(val));
        }
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) maxabs = fmax(maxabs, __shfl_xor(maxabs, off));
  if (l == 0) {
    wmax[wave] = maxabs;
    wseq[wave] = s;
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    // wavefront w reports for its sequence if no earlier wavefront has it
    const int w = threadIdx.x, sw_ = wseq[w];
    bool first = sw_ >= 0;
    double mx = 0.0;
    for (int x = 0; x < 4; ++x) {
      if (wseq[x] == sw_) {
        if (x < w) first = false;
        mx = fmax(mx, wmax[x]);
      }
    }
    if (first && mx > 0.0)
      atomicMax(reinterpret_cast<unsigned long long*>(A_scale + sw_),
                (unsigned long long)__double_as_longlong(mx));
  }
}

// Whether few block rows are summed by a workgroup per wavefront. One workgroup
// for a row streams about 50 GB/s, bound by the conversions and fp64 sums of its
// eight wavefronts: below 128 rows a call takes as long as its one row, split it
// takes two thirds and less. From 64 rows on the 4-byte loads per lane cost more
// than the idle CUs, the later the larger the row (rows of bf16 / fp32; one
// workgroup / split, us, with the block scores and the launch that adds the
// parts):
//   1.3 MB / 2.6 MB  8 rows 33.7 / 20.0, 50.8 / 27.0; 32: 40.2 / 22.2, 57.4 / 30.2;
//                    94: 41.8 / 38.3, 63.1 / 53.3; 102: 41.9 / 45.2, 64.4 / 59.8
//   0.66 / 1.3       62: 27.2 / 23.9, 36.2 / 29.7; 78: 27.3 / 28.7, 37.2 / 31.6;
//                    94: 27.7 / 28.9, 37.8 / 34.5
//   0.33 / 0.66      31: 24.0 / 17.1, 23.6 / 18.0; 62: 22.7 / 20.9, 24.2 / 23.3;
//                    78: 22.4 / 24.0, 24.7 / 24.6
// and 80 KB rows lose at any number (15.6 / 20.4 at 62).
static bool sketch_split(int h_q, int h_kv, int d, int B, int64_t nb, int esz) {
  const int64_t bytes = (int64_t)(h_q + h_kv) * B * d * esz;  // of a row
  if (bytes < 128 * 1024 * esz) return false;
  return nb <= 64 || (nb <= 96 && bytes >= 1024 * 1024) || (nb < 128 && bytes >= 2048 * 1024);
}

int64_t sketch_workspace_bytes(int h_q, int h_kv, int d, int B, int64_t nb) {
  // whichever type the call has
  const bool split = sketch_split(h_q, h_kv, d, B, nb, 2) || sketch_split(h_q, h_kv, d, B, nb, 4);
  return split ? nb * kPoolWaves * 2 * d * (int64_t)sizeof(double) : 0;
}

hipError_t launch_sketch(int dtype, const void* Q, const void* K, int h_q, int h_kv, int d,
                         const SeqMeta& meta, int64_t nb, long long N, const int8_t* signs,
                         const int32_t* cols, int r, double* Qs, double* Ks, double* A,
                         double* A_scale, double* Qbar, double* Kbar, void* ws, hipStream_t st) {
  const dim3 grid((unsigned)nb);
#define SW_POOL(T)                                                                                  \
  do {                                                                                              \
    auto q = reinterpret_cast<const T*>(Q);                                                         \
    auto k = reinterpret_cast<const T*>(K);                                                         \
    if (split)                                                                                      \
      hipLaunchKernelGGL(pool_split_kernel<T>, dim3((unsigned)nb, kPoolWaves), dim3(512 / sizeof(T)), 0, \
                         st, q, k, h_q, h_kv, d, meta, N, A_scale, parts);                          \
    else                                                                                            \
      hipLaunchKernelGGL(pool_sketch_kernel<T>, grid, dim3(kPoolThreads), 0, st, q, k, h_q, h_kv, d, \
                         meta, N, signs, cols, r, Qs, Ks, Qbar, Kbar, A_scale);                     \
  } while (0)
  const bool split = ws != nullptr && sketch_split(h_q, h_kv, d, meta.B, nb, dtype == SW_BF16 ? 2 : 4);
  double* parts = static_cast<double*>(ws);
  if (dtype == SW_BF16) SW_POOL(uint16_t);
  else SW_POOL(float);
#undef SW_POOL
  if (split)
    hipLaunchKernelGGL(sketch_parts_kernel, grid, dim3(256), 0, st, parts, h_q, h_kv, d, meta, signs,
                       cols, r, Qs, Ks, Qbar, Kbar);
  // tile prefix per sequence
  SeqMeta m2 = meta;
  int total = 0;
  for (int s = 0; s < meta.n_seqs; ++s) {
    m2.aux_start[s] = total;
    const int b = meta.blk_start[s + 1] - meta.blk_start[s];
    const int tb = (b + 15) / 16;
    total += tb * tb;
  }
  m2.aux_start[meta.n_seqs] = total;
  hipLaunchKernelGGL(scores_kernel, dim3((unsigned)((total + 3) / 4)), dim3(256), 0, st, Qs, Ks,
                     r, m2, total, A, A_scale);
  return hipGetLastError();
}

}  // namespace sw

// Decode attention (paper Alg. 2 step 7): single-token softmax attention over
// the tokens of the selected key blocks, split-K over those tokens.
//
//  attn_decode_mfma_kernel  bf16: one workgroup per (sequence, KV head, split);
//                           the split's selected-block list is staged in LDS,
//                           K/V groups of 16 tokens are streamed with raw buffer
//                           loads and the G query heads of the KV group are
//                           scored and accumulated on MFMA
//  attn_decode_f32_kernel   fp32: the same on the fp32 matrix instructions, the
//                           operands straight from the loads
//  attn_merge_kernel        log-sum-exp merge of the splits, one workgroup per
//                           (sequence, query head); attn_merge_one_kernel where
//                           there is one split
// The layers of a one-call decode step share a launch (blockIdx.y is the
// layer; buffers are stacked over the layers).
#include <climits>
#include <mutex>

#include "sw_common.h"
#include "sw_internal.h"

namespace sw {

constexpr float kLog2eD = 1.4426950408889634f;

// Combine a lane's value with that of lane ^ 16 / lane ^ 32 through the
// permlane swaps (VALU moves; each returns the lane's own value and its
// partner's in some order).
__device__ __forceinline__ float fmax_xor16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float fmax_xor32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_xor16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float sum_xor32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Elements from one layer to the next of the stacked buffers.
struct DecodeAttnSteps {
  long long q, cache, idx, cnt, ws;
};

// Tuning constants (overridable at build time).
#ifndef SW_DEC_GPS
#define SW_DEC_GPS 2          // 16-token groups per wavefront step in decode attention
#endif
#ifndef SW_DEC_WGS
#define SW_DEC_WGS 512        // target decode-attention workgroups per launch
#endif
// ---------------------------------------------------------------------------
// split-K decode attention
// ---------------------------------------------------------------------------

// bf16 split-K decode attention on MFMA. Workgroup = (sequence, KV head,
// split), 4 wavefronts; a wavefront takes groups of 16 consecutive selected
// tokens, GPS groups per step, loading the groups of step it+1 while it
// computes step it (two register sets, the step loop unrolled by two so
// neither set is copied).
//   S = K q^T   v_mfma_f32_16x16x32_bf16: A = 16 key rows x 32 dims read
//               straight from the cache (16 bytes per lane), B = the G query
//               heads (zero-padded to 16 columns). Lane n + 16 (m / 4) holds
//               key m of head n, so the online-softmax state of a head stays
//               in the lane (plus two exchanges for the max).
//   O^T += V^T P^T  v_mfma_f32_16x16x16bf16_1k: A = V^T from a per-wave LDS
//               slice written transposed (4 keys x 8 dims per lane), B = P in
//               the accumulator layout of S.
// The split's block indices are staged in LDS once, and the K/V loads go
// through buffer descriptors that end at the last valid token (lanes past it
// read zero), so the loop has no global index loads and no per-lane branches
// around loads: the loads of the next step stay in flight during the math.
typedef __bf16 bf16x8d __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4d __attribute__((ext_vector_type(4)));

constexpr int kDecBufWord3 = 0x00020000;   // raw buffer descriptor word 3 (gfx9 family)

template <int D>
__global__ __launch_bounds__(256) void attn_decode_mfma_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ Kc, const uint16_t* __restrict__ Vc,
    int h_kv, int G, int T_max, int B, const int32_t* __restrict__ pos,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt, int kmax, float sl2, int S,
    float* __restrict__ ws, DecodeAttnSteps ls) {
  q += blockIdx.y * ls.q;
  Kc += blockIdx.y * ls.cache;
  Vc += blockIdx.y * ls.cache;
  idx += blockIdx.y * ls.idx;
  cnt += blockIdx.y * ls.cnt;
  ws += blockIdx.y * ls.ws;
  constexpr int VTS = 16 + 4;                      // V^T row stride (keys + pad)
  constexpr int GPS = SW_DEC_GPS;                  // 16-token groups per wave step
  // LDS: per-wave V^T slices during the loop; the epilogue's partials reuse it
  constexpr int VT_BYTES = 4 * GPS * D * VTS * 2;
  constexpr int EP_BYTES = (4 * 16 * D + 2 * 4 * 16) * 4;
  __shared__ __attribute__((aligned(16))) char smem[VT_BYTES > EP_BYTES ? VT_BYTES : EP_BYTES];
  __shared__ int16_t ssel[SW_MAX_BLOCKS + 2];      // this split's block indices
  auto vt_slice = [&](int wv, int x) {
    return reinterpret_cast<uint16_t*>(smem) + (wv * GPS + x) * D * VTS;
  };
  float (*sm_o)[16][D] = reinterpret_cast<float (*)[16][D]>(smem);
  float (*sm_m)[16] = reinterpret_cast<float (*)[16]>(smem + 4 * 16 * D * 4);
  float (*sm_l)[16] = reinterpret_cast<float (*)[16]>(smem + 4 * 16 * D * 4 + 4 * 16 * 4);
  const int sp = blockIdx.x % S;
  const int bg = blockIdx.x / S;                   // (sequence, kv head)
  const int bi = bg / h_kv;
  const int g = bg % h_kv;
  const int h_q = h_kv * G;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int ln = l & 15, lg = l >> 4;
  const int p = pos[bi], have = cnt[bi];           // both loads before either is used
  const bool ok = p >= 0 && p < T_max;
  const int bc = ok ? p / B : 0;
  // a valid selection has at most SW_MAX_BLOCKS distinct blocks, so 32 bits
  // hold groups (at most 64 per block) times splits
  const int tau = ok ? max(0, min(min(have, kmax), SW_MAX_BLOCKS)) : 0;
  const int gpb = B / 16;                          // 16-token groups per block
  const int ngroups = tau * gpb;
  static_assert((long long)SW_MAX_BLOCKS * 64 * (kDecodeMaxSplits + 1) < (1ll << 31), "32-bit split bounds");
  const int g0 = (int)((unsigned)(ngroups * sp) / (unsigned)S);
  const int g1 = (int)((unsigned)(ngroups * (sp + 1)) / (unsigned)S);
  const int jlo = g0 / gpb;
  const int nj = (g1 > g0) ? (g1 - 1) / gpb - jlo + 1 : 0;
  {
    const int32_t* sel = idx + (long long)bi * kmax + jlo;
    for (int e = tid; e < nj; e += 256) ssel[e] = (int16_t)max(-1, min(sel[e], 32767));
  }

  // query fragments (B operand of S = K q^T): head ln, dims 32c + 8 lg .. +7
  bf16x8d qf[D / 32];
  {
    const bool hv = ln < G;
    const uint16_t* qp = q + ((long long)bi * h_q + g * G + (hv ? ln : 0)) * D + lg * 8;
#pragma unroll
    for (int c = 0; c < D / 32; ++c) {
      uint4 v = hv ? *reinterpret_cast<const uint4*>(qp + 32 * c) : make_uint4(0, 0, 0, 0);
      qf[c] = *reinterpret_cast<bf16x8d*>(&v);
    }
  }
  f32x4d oacc[D / 16];
#pragma unroll
  for (int t = 0; t < D / 16; ++t) oacc[t] = f32x4d{0.f, 0.f, 0.f, 0.f};
  float mrun = -INFINITY, lrun = 0.0f;
  const uint16_t* Kb = Kc + (long long)bg * T_max * D;
  const uint16_t* Vb = Vc + (long long)bg * T_max * D;
  // V staging: lane takes keys 4 kq .. 4 kq + 3 and dims 8 dq .. 8 dq + 7
  const int kq = l & 3, dq = l >> 2;
  const bool vthr = dq < D / 8;
  // per-lane byte offsets inside a 16-token group (tile invariant)
  const int koff = ln * D * 2 + lg * 16;
  const int voff = vthr ? (kq * 4 * D * 2 + dq * 16) : 0x40000000;   // idle lanes read past the end
  __syncthreads();                                 // ssel visible

  const int nsteps = (g1 - g0 + 4 * GPS - 1) / (4 * GPS);
  // token of the first key of group gi, or -1 when the group holds no valid key
  auto group_t0 = [&](int gi) {
    const int f = gi * 16;
    const int jj = f / B;
    const int j = __builtin_amdgcn_readfirstlane((int)ssel[jj - jlo]);
    const int t0 = j * B + (f - jj * B);
    return __builtin_amdgcn_readfirstlane((j >= 0 && j <= bc && t0 <= p) ? t0 : -1);
  };
  auto issue = [&](int step, uint4 (&kr)[GPS][D / 32], uint4 (&vr)[GPS][4], int (&t0s)[GPS]) {
#pragma unroll
    for (int x = 0; x < GPS; ++x) {
      const int gi = g0 + (step * 4 + w) * GPS + x;
      const int t0 = (step < nsteps && gi < g1) ? group_t0(gi) : -1;
      t0s[x] = t0;
      // No branch around the loads (the wait counts stay exact): a group
      // without valid keys gets an empty descriptor and reads zeros. The
      // loads are non-temporal (cache policy 2): each selected K/V byte is
      // read once per step, and the streaming hint lifts the read rate.
      const int tb = max(t0, 0);
      const int bytes = (t0 >= 0) ? (p + 1 - t0) * D * 2 : 0;   // keys past p read as zero
      const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(Kb + (long long)tb * D), (short)0, bytes, kDecBufWord3);
      const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(Vb + (long long)tb * D), (short)0, bytes, kDecBufWord3);
#pragma unroll
      for (int c = 0; c < D / 32; ++c) {
        auto a = __builtin_amdgcn_raw_buffer_load_b128(rk, koff + c * 64, 0, 2);
        kr[x][c] = __builtin_bit_cast(uint4, a);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        auto b = __builtin_amdgcn_raw_buffer_load_b128(rv, voff + r * D * 2, 0, 2);
        vr[x][r] = __builtin_bit_cast(uint4, b);
      }
    }
  };
  // one step on the register set (kraw, vraw, tok0)
  auto compute = [&](const uint4 (&kraw)[GPS][D / 32], const uint4 (&vraw)[GPS][4],
                     const int (&tok0)[GPS]) {
    // V^T into this wave's LDS slice
#pragma unroll
    for (int x = 0; x < GPS; ++x) {
      if (vthr && tok0[x] >= 0) {
        uint16_t* vt = vt_slice(w, x);
        const uint32_t a[4] = {vraw[x][0].x, vraw[x][0].y, vraw[x][0].z, vraw[x][0].w};
        const uint32_t b[4] = {vraw[x][1].x, vraw[x][1].y, vraw[x][1].z, vraw[x][1].w};
        const uint32_t c[4] = {vraw[x][2].x, vraw[x][2].y, vraw[x][2].z, vraw[x][2].w};
        const uint32_t d[4] = {vraw[x][3].x, vraw[x][3].y, vraw[x][3].z, vraw[x][3].w};
#pragma unroll
        for (int wd = 0; wd < 4; ++wd) {
          uint2 lo, hi;
          lo.x = (a[wd] & 0xffffu) | (b[wd] << 16);
          lo.y = (c[wd] & 0xffffu) | (d[wd] << 16);
          hi.x = (a[wd] >> 16) | (b[wd] & 0xffff0000u);
          hi.y = (c[wd] >> 16) | (d[wd] & 0xffff0000u);
          *reinterpret_cast<uint2*>(vt + (dq * 8 + 2 * wd) * VTS + kq * 4) = lo;
          *reinterpret_cast<uint2*>(vt + (dq * 8 + 2 * wd + 1) * VTS + kq * 4) = hi;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int x = 0; x < GPS; ++x) {
      if (tok0[x] < 0) continue;                   // uniform across the wavefront
      f32x4d sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < D / 32; ++c)
        sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8d, kraw[x][c]),
                                                       qf[c], sacc, 0, 0, 0);
      float sv[4];
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int key = tok0[x] + 4 * lg + v;
        sv[v] = (key <= p) ? sacc[v] * sl2 : -INFINITY;
        mx = fmaxf(mx, sv[v]);
      }
      mx = fmax_xor16(mx);
      mx = fmax_xor32(mx);
      const float mnew = fmaxf(mrun, mx);          // finite: key tok0 <= p is valid
      const float alpha = exp2f(mrun - mnew);
      mrun = mnew;
      float pv[4];
      float ps = 0.0f;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        pv[v] = exp2f(sv[v] - mnew);
        ps += pv[v];
      }
      lrun = lrun * alpha + ps;
      s16x4 pb;
      pb[0] = (short)f32_to_bf16(pv[0]);
      pb[1] = (short)f32_to_bf16(pv[1]);
      pb[2] = (short)f32_to_bf16(pv[2]);
      pb[3] = (short)f32_to_bf16(pv[3]);
      const uint16_t* vt = vt_slice(w, x);
#pragma unroll
      for (int t = 0; t < D / 16; ++t) {
        oacc[t] *= alpha;
        const uint2 va = *reinterpret_cast<const uint2*>(vt + (t * 16 + ln) * VTS + lg * 4);
        oacc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const s16x4*>(&va),
                                                            pb, oacc[t], 0, 0, 0);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  uint4 kA[GPS][D / 32], vA[GPS][4], kB[GPS][D / 32], vB[GPS][4];
  int tA[GPS], tB[GPS];
  issue(0, kA, vA, tA);
  for (int it = 0; it < nsteps; it += 2) {
    issue(it + 1, kB, vB, tB);
    compute(kA, vA, tA);
    if (it + 1 >= nsteps) break;
    issue(it + 2, kA, vA, tA);
    compute(kB, vB, tB);
  }
  __syncthreads();                                 // V^T slices are dead from here
  // per-wave partials: head ln; lane groups hold disjoint keys (sum l) and
  // disjoint output dims
  float lsum = sum_xor16(lrun);
  lsum = sum_xor32(lsum);
  if (lg == 0) {
    sm_m[w][ln] = mrun;
    sm_l[w][ln] = lsum;
  }
#pragma unroll
  for (int t = 0; t < D / 16; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) sm_o[w][ln][t * 16 + 4 * lg + v] = oacc[t][v];
  __syncthreads();
  const int nsp = S;
  float* ws_ml = ws;
  float* ws_o = ws + (long long)gridDim.x / S * G * nsp * 2;
  for (int xx = tid; xx < G * D; xx += 256) {
    const int u = xx / D, dim = xx % D;
    float M = -INFINITY;
    for (int k = 0; k < 4; ++k) M = fmaxf(M, sm_m[k][u]);
    float Lsum = 0.0f, Osum = 0.0f;
    if (M != -INFINITY) {
      for (int k = 0; k < 4; ++k) {
        const float sc = exp2f(sm_m[k][u] - M);
        Lsum += sm_l[k][u] * sc;
        Osum += sm_o[k][u][dim] * sc;
      }
    }
    const long long hu = (long long)bi * h_q + g * G + u;
    ws_o[(hu * nsp + sp) * D + dim] = Osum;
    if (dim == 0) {
      ws_ml[(hu * nsp + sp) * 2 + 0] = M;
      ws_ml[(hu * nsp + sp) * 2 + 1] = Lsum;
    }
  }
}

// fp32 split-K decode attention. Workgroups, splits and steps as in the bf16
// kernel, one group of 16 tokens per wavefront and step (16 KB of K and V at
// d = 128), the next one loading during the math. (At d = 64 two groups a step,
// or two steps ahead, were up to 10 % slower.)
//   S = K q^T       v_mfma_f32_16x16x4f32: lane (key ln, lg) holds dims
//                   16 c + 4 lg .. + 3 of its key, and of head ln of the
//                   queries; the product of step (c, e) takes element e of
//                   both, so any 4 dims may share an instruction. Lane
//                   n + 16 (m / 4) receives key m of head n.
//   O^T += V^T P^T  step v takes key 4 lg + v: the lane's own weight of that
//                   key as the B operand, and element t of the dims
//                   ln D / 16 .. + D / 16 - 1 it loaded of the key's value row
//                   as the A operand of the t-th product, whose row m is dim
//                   m D / 16 + t. No exchange, no LDS.
// Bounded by the reads: 5.9 and 6.4 TB/s at 512 blocks of 64 (32 query heads over
// 8, d = 128, batch 4 and 16; 291 -> 183 and 1115 -> 675 us; at 103 blocks and
// batch 4 5.2, the start and end of one round), the matrix cores 23 % busy.
// Products on the vector unit, a 64-bit division per token and no load in
// flight during the math gave 3.8 TB/s. The logits are added as a tree and each
// group's sums enter the running ones once, so that nothing is less exact than it was (relative error
// against 64 bits 1.8e-7 on average over four shapes, 1.9e-7 before; one chain
// of products per logit gave 3.5 times the error at logits of several hundred).
template <int D>
__global__ __launch_bounds__(256, 2) void attn_decode_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ Kc, const float* __restrict__ Vc, int h_kv,
    int G, int T_max, int B, const int32_t* __restrict__ pos, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ cnt, int kmax, float sl2, int S, float* __restrict__ ws,
    DecodeAttnSteps ls) {
  q += blockIdx.y * ls.q;
  Kc += blockIdx.y * ls.cache;
  Vc += blockIdx.y * ls.cache;
  idx += blockIdx.y * ls.idx;
  cnt += blockIdx.y * ls.cnt;
  ws += blockIdx.y * ls.ws;
  constexpr int NC = D / 16;                       // 16-byte pieces of a key per lane
  constexpr int DPL = D / 16;                      // value dims per lane
  constexpr int NV = DPL / 4;                      // 16-byte pieces of a value row per lane
  constexpr int GMAX = 8;
  __shared__ float sm_o[4][GMAX][D];
  __shared__ float sm_m[4][GMAX], sm_l[4][GMAX];
  __shared__ int ssel[SW_MAX_BLOCKS];              // this split's block indices
  const int sp = blockIdx.x % S;
  const int bg = blockIdx.x / S;                   // (sequence, kv head)
  const int bi = bg / h_kv;
  const int g = bg % h_kv;
  const int h_q = h_kv * G;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int ln = l & 15, lg = l >> 4;
  const int p = pos[bi], have = cnt[bi];           // both loads before either is used
  const bool ok = p >= 0 && p < T_max;
  const int bc = ok ? p / B : 0;
  const int tau = ok ? max(0, min(min(have, kmax), INT_MAX / 64)) : 0;
  const int gpb = B / 16;                          // 16-token groups per block
  const int ngroups = tau * gpb;
  int g0, g1;
  if (tau <= SW_MAX_BLOCKS) {
    static_assert((long long)SW_MAX_BLOCKS * 64 * (kDecodeMaxSplits + 1) < (1ll << 31), "32-bit split bounds");
    g0 = (int)((unsigned)(ngroups * sp) / (unsigned)S);
    g1 = (int)((unsigned)(ngroups * (sp + 1)) / (unsigned)S);
  } else {
    g0 = (int)((long long)ngroups * sp / S);
    g1 = (int)((long long)ngroups * (sp + 1) / S);
  }
  const int32_t* sel = idx + (long long)bi * kmax;
  // query operand: head ln, dims 16 c + 4 lg + e
  float4 qf[NC];
  {
    const bool hv = ln < G;
    const float* qp = q + ((long long)bi * h_q + g * G + (hv ? ln : 0)) * D + lg * 4;
#pragma unroll
    for (int c = 0; c < NC; ++c)
      qf[c] = hv ? *reinterpret_cast<const float4*>(qp + 16 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  f32x4d oacc[DPL];
#pragma unroll
  for (int t = 0; t < DPL; ++t) oacc[t] = f32x4d{0.f, 0.f, 0.f, 0.f};
  // largest raw score and the sum of the weights. The scale comes after the
  // subtraction: the largest weight is exactly 1 however large the scores are.
  float mrun = -INFINITY, lrun = 0.0f;
  const float* Kb = Kc + (long long)bg * T_max * D;
  const float* Vb = Vc + (long long)bg * T_max * D;
  const int koff = (ln * D + lg * 4) * 4;          // per-lane byte offsets inside a group
  const int voff = (4 * lg * D + ln * DPL) * 4;

  // the groups c0 .. c1 of one piece of the list, whose blocks start at jlo
  int c0 = g0, c1 = g0, jlo = 0, nsteps = 0;
  // loads as in the bf16 kernel: no branch, keys past p read as zero, the
  // streaming hint
  auto issue = [&](int step, uint4 (&kr)[NC], uint4 (&vr)[4][NV], int& t0out) {
    const int gi = c0 + step * 4 + w;
    int t0 = -1;
    if (step < nsteps && gi < c1) {
      const int jj = gi / gpb;
      const int j = __builtin_amdgcn_readfirstlane(ssel[jj - jlo]);
      const int tt = (j >= 0 && j <= bc) ? j * B + (gi - jj * gpb) * 16 : INT_MAX;
      t0 = tt <= p ? tt : -1;
    }
    t0 = __builtin_amdgcn_readfirstlane(t0);
    t0out = t0;
    const int tb = max(t0, 0);
    const int bytes = (t0 >= 0) ? min(p + 1 - t0, 16) * D * 4 : 0;
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(Kb + (long long)tb * D), (short)0, bytes, kDecBufWord3);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(Vb + (long long)tb * D), (short)0, bytes, kDecBufWord3);
#pragma unroll
    for (int c = 0; c < NC; ++c)
      kr[c] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rk, koff + c * 64, 0, 2));
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int n = 0; n < NV; ++n)
        vr[v][n] = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(rv, voff + v * D * 4 + n * 16, 0, 2));
  };
  auto compute = [&](const uint4 (&kr)[NC], const uint4 (&vr)[4][NV], int t0) {
    if (t0 < 0) return;                            // uniform across the wavefront
    // Sums of 8 products, added as a tree (as the lanes of a key added theirs
    // when the products were on the vector unit): the logits are as exact.
    f32x4d part[NC / 2];
#pragma unroll
    for (int c = 0; c < NC; c += 2) {
      const float k0[4] = {__uint_as_float(kr[c].x), __uint_as_float(kr[c].y),
                           __uint_as_float(kr[c].z), __uint_as_float(kr[c].w)};
      const float k1[4] = {__uint_as_float(kr[c + 1].x), __uint_as_float(kr[c + 1].y),
                           __uint_as_float(kr[c + 1].z), __uint_as_float(kr[c + 1].w)};
      const float q0[4] = {qf[c].x, qf[c].y, qf[c].z, qf[c].w};
      const float q1[4] = {qf[c + 1].x, qf[c + 1].y, qf[c + 1].z, qf[c + 1].w};
      f32x4d e4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        e4[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(k0[e], q0[e], f32x4d{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        e4[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(k1[e], q1[e], e4[e], 0, 0, 0);
      part[c / 2] = (e4[0] + e4[1]) + (e4[2] + e4[3]);
    }
#pragma unroll
    for (int n = NC / 4; n > 0; n /= 2)
#pragma unroll
      for (int i = 0; i < n; ++i) part[i] += part[i + n];
    const f32x4d& sacc = part[0];
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (t0 + 4 * lg + v <= p) mx = fmaxf(mx, sacc[v]);
    mx = fmax_xor16(mx);
    mx = fmax_xor32(mx);
    mx = fmaxf(mrun, mx);
    // -infinity while every score so far was: those keys have weight 0
    const float mnew = mx == -INFINITY ? 0.0f : mx;
    const float alpha = exp2f((mrun - mnew) * sl2);
    mrun = mx;
    float pv[4];
    float ps = 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      pv[v] = (t0 + 4 * lg + v <= p) ? exp2f((sacc[v] - mnew) * sl2) : 0.0f;
      ps += pv[v];
    }
    lrun = lrun * alpha + ps;
    // the group's sums on their own, then onto the running ones
#pragma unroll
    for (int n = 0; n < NV; ++n) {
      f32x4d o4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) o4[e] = f32x4d{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const uint4& r = vr[v][n];
        o4[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(r.x), pv[v], o4[0], 0, 0, 0);
        o4[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(r.y), pv[v], o4[1], 0, 0, 0);
        o4[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(r.z), pv[v], o4[2], 0, 0, 0);
        o4[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(r.w), pv[v], o4[3], 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) oacc[4 * n + e] = oacc[4 * n + e] * alpha + o4[e];
    }
  };
  uint4 kA[NC], vA[4][NV], kB[NC], vB[4][NV];
  int tA, tB;
  // the list in pieces of SW_MAX_BLOCKS entries (one, but for longer selections)
  while (c1 < g1) {
    c0 = c1;
    jlo = c0 / gpb;
    c1 = min((long long)g1, ((long long)jlo + SW_MAX_BLOCKS) * gpb);
    nsteps = (c1 - c0 + 3) / 4;
    if (c0 > g0) __syncthreads();                  // the piece before is done with ssel
    for (int e = tid; e < (c1 - 1) / gpb - jlo + 1; e += 256) ssel[e] = sel[jlo + e];
    __syncthreads();
    issue(0, kA, vA, tA);
    for (int it = 0; it < nsteps; it += 2) {
      issue(it + 1, kB, vB, tB);
      compute(kA, vA, tA);
      if (it + 1 >= nsteps) break;
      issue(it + 2, kA, vA, tA);
      compute(kB, vB, tB);
    }
  }
  // per-wave partials: head ln; the lane groups hold disjoint keys (sum l)
  // and disjoint output dims
  float lsum = sum_xor16(lrun);
  lsum = sum_xor32(lsum);
  if (ln < GMAX) {
    if (lg == 0) {
      sm_m[w][ln] = mrun;
      sm_l[w][ln] = lsum;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int t = 0; t < DPL; ++t) sm_o[w][ln][(4 * lg + v) * DPL + t] = oacc[t][v];
  }
  __syncthreads();
  float* ws_ml = ws;
  float* ws_o = ws + (long long)gridDim.x / S * G * S * 2;
  for (int xx = tid; xx < G * D; xx += 256) {
    const int u = xx / D, dim = xx % D;
    float M = -INFINITY;
    for (int k = 0; k < 4; ++k) M = fmaxf(M, sm_m[k][u]);
    float Lsum = 0.0f, Osum = 0.0f;
    if (M != -INFINITY) {
      for (int k = 0; k < 4; ++k) {
        const float sc = exp2f((sm_m[k][u] - M) * sl2);
        Lsum += sm_l[k][u] * sc;
        Osum += sm_o[k][u][dim] * sc;
      }
    }
    const long long hu = (long long)bi * h_q + g * G + u;
    ws_o[(hu * S + sp) * D + dim] = Osum;
    if (dim == 0) {
      ws_ml[(hu * S + sp) * 2 + 0] = M;
      ws_ml[(hu * S + sp) * 2 + 1] = Lsum;
    }
  }
}

// The splits' maxima times ms are in log2 units (fp32: raw scores, ms = the
// scale; bf16: ms = 1). Four wavefronts per (sequence, query head): every
// wavefront holds the splits' maxima and sums (lane s holds split s) and adds
// the outputs of splits w, w + 4, ..., all loaded before the first is used; the
// four sums are added in order. The splits' outputs come from another launch, so the kernel is two
// dependent loads and one barrier long: 32 splits took 10.5 us as a loop over
// the splits (batch 1, 32 heads).
template <typename T, int D, int NLOAD>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float* __restrict__ ws, int S,
                                                         long long n_hu, T* __restrict__ O,
                                                         long long ws_step, float ms) {
  static_assert(kDecodeMaxSplits <= 64, "one split per lane");   // and S <= 4 * NLOAD
  constexpr int V = D / 64;                        // output dims per lane
  typedef float vec __attribute__((ext_vector_type(V)));
  __shared__ float part[4][D];
  const long long hu = blockIdx.x;
  ws += blockIdx.y * ws_step;
  const float* ws_ml = ws + hu * S * 2;
  const float* ws_o = ws + n_hu * S * 2 + hu * S * D;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  float m = ws_ml[2 * min(l, S - 1)];
  const float ls = ws_ml[2 * min(l, S - 1) + 1];
  vec o[NLOAD];
#pragma unroll
  for (int i = 0; i < NLOAD; ++i)
    o[i] = *reinterpret_cast<const vec*>(ws_o + (long long)min(w + 4 * i, S - 1) * D + l * V);
  m = l < S ? m : -INFINITY;
  float M = m;
  for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
  // a split without keys (m = -inf) has weight 0; without any key all have
  const float sc = (M != -INFINITY && l < S) ? exp2f((m - M) * ms) : 0.0f;
  float Lsum = ls * sc;
  for (int off = 32; off > 0; off >>= 1) Lsum += __shfl_xor(Lsum, off);
  vec acc = {};
#pragma unroll
  for (int i = 0; i < NLOAD; ++i) {
    const int s = w + 4 * i;
    if (s < S) acc += o[i] * __shfl(sc, s);
  }
#pragma unroll
  for (int e = 0; e < V; ++e) part[w][l * V + e] = acc[e];
  __syncthreads();
  if (threadIdx.x >= D) return;
  const int dim = threadIdx.x;
  const float sum = ((part[0][dim] + part[1][dim]) + part[2][dim]) + part[3][dim];
  const float v = Lsum > 0.0f ? sum / Lsum : 0.0f;
  const long long at = (blockIdx.y * n_hu + hu) * D + dim;
  if constexpr (sizeof(T) == 2)
    reinterpret_cast<uint16_t*>(O)[at] = f32_to_bf16(v);
  else
    O[at] = v;
}

// One split: a wavefront per (sequence, query head). A call at batch 64, 2000
// tokens, 32 heads over 8 of d = 128: 26.8 us with the four of the kernel above,
// 25.2 with one (fp32 45.1 and 43.8).
template <typename T, int D>
__global__ __launch_bounds__(256) void attn_merge_one_kernel(const float* __restrict__ ws,
                                                             long long n_hu, T* __restrict__ O,
                                                             long long ws_step) {
  constexpr int V = D / 64;                        // output dims per lane
  typedef float vec __attribute__((ext_vector_type(V)));
  const long long hu = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (hu >= n_hu) return;
  const int l = threadIdx.x & 63;
  ws += blockIdx.y * ws_step;
  const float m = ws[hu * 2], ls = ws[hu * 2 + 1];
  const vec o = *reinterpret_cast<const vec*>(ws + n_hu * 2 + hu * D + l * V);
  // without any key (m = -inf) the output is 0
  const float Lsum = m != -INFINITY ? ls : 0.0f;
  const long long at = (blockIdx.y * n_hu + hu) * D + l * V;
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const float v = Lsum > 0.0f ? o[e] / Lsum : 0.0f;
    if constexpr (sizeof(T) == 2)
      reinterpret_cast<uint16_t*>(O)[at + e] = f32_to_bf16(v);
    else
      O[at + e] = v;
  }
}

// Splits per (sequence, KV head): about SW_DEC_WGS workgroups; 512 fills
// every CU once at the bf16 kernel's occupancy (2 workgroups of 4 waves).
int decode_attn_splits(int batch, int h_kv) {
  const int pairs = batch * h_kv;
  int S = (SW_DEC_WGS + pairs - 1) / pairs;
  if (S < 1) S = 1;
  if (S > kDecodeMaxSplits) S = kDecodeMaxSplits;
  return S;
}

// ---------------------------------------------------------------------------
// fixed scratch for the allocation-free entry point
// ---------------------------------------------------------------------------

// The split-K partials of sw_sparse_attn_decode_noalloc: a fixed device array
// (each GPU the library runs on holds its own copy until the process ends).
// Host code never passes the array's name to a kernel; it passes the device
// address looked up below, once per device.
static __device__ __align__(256) __attribute__((used)) float scratch[SW_NOALLOC_SCRATCH_BYTES / 4];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];        // device address of `scratch`, per device
}  // namespace

hipError_t noalloc_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_attn_decode(int dtype, int layers, const void* q, const void* Kc, const void* Vc,
                              int batch, int h_q, int h_kv, int d, int T_max, int B,
                              const int32_t* pos, const int32_t* idx, const int32_t* cnt, int kmax,
                              float scale, void* O, float* ws, hipStream_t st) {
  const int G = h_q / h_kv;
  const int S = decode_attn_splits(batch, h_kv);
  const dim3 grid((unsigned)(batch * h_kv * S), (unsigned)layers);
  const float sl2 = scale * kLog2eD;
  const long long n_hu = (long long)batch * h_q;
  const dim3 mgrid((unsigned)n_hu, (unsigned)layers);
  DecodeAttnSteps ls;
  ls.q = n_hu * d;
  ls.cache = (long long)batch * h_kv * T_max * d;
  ls.idx = (long long)batch * kmax;
  ls.cnt = batch;
  ls.ws = n_hu * S * (d + 2);
#define SW_MERGE_N(T, D, N)                                                                    \
  hipLaunchKernelGGL((attn_merge_kernel<T, D, N>), mgrid, dim3(256), 0, st, ws, S, n_hu,       \
                     reinterpret_cast<T*>(O), ls.ws, sizeof(T) == 4 ? sl2 : 1.0f)
#define SW_MERGE(T, D)                                      \
  do {                                                      \
    if (S == 1)                                             \
      hipLaunchKernelGGL((attn_merge_one_kernel<T, D>), dim3((mgrid.x + 3) / 4, mgrid.y), dim3(256), 0, \
                         st, ws, n_hu, reinterpret_cast<T*>(O), ls.ws); \
    else if (S <= 4) SW_MERGE_N(T, D, 1);                   \
    else if (S <= 16) SW_MERGE_N(T, D, 4);                  \
    else SW_MERGE_N(T, D, kDecodeMaxSplits / 4);            \
  } while (0)
  if (dtype == SW_BF16) {
    auto qq = reinterpret_cast<const uint16_t*>(q);
    auto kk = reinterpret_cast<const uint16_t*>(Kc);
    auto vv = reinterpret_cast<const uint16_t*>(Vc);
    if (d == 128) {
      hipLaunchKernelGGL(attn_decode_mfma_kernel<128>, grid, dim3(256), 0, st, qq, kk, vv, h_kv, G,
                         T_max, B, pos, idx, cnt, kmax, sl2, S, ws, ls);
      SW_MERGE(uint16_t, 128);
    } else {
      hipLaunchKernelGGL(attn_decode_mfma_kernel<64>, grid, dim3(256), 0, st, qq, kk, vv, h_kv, G,
                         T_max, B, pos, idx, cnt, kmax, sl2, S, ws, ls);
      SW_MERGE(uint16_t, 64);
    }
  } else {
    auto qq = reinterpret_cast<const float*>(q);
    auto kk = reinterpret_cast<const float*>(Kc);
    auto vv = reinterpret_cast<const float*>(Vc);
    if (d == 128) {
      hipLaunchKernelGGL(attn_decode_f32_kernel<128>, grid, dim3(256), 0, st, qq, kk, vv, h_kv, G,
                         T_max, B, pos, idx, cnt, kmax, sl2, S, ws, ls);
      SW_MERGE(float, 128);
    } else {
      hipLaunchKernelGGL(attn_decode_f32_kernel<64>, grid, dim3(256), 0, st, qq, kk, vv, h_kv, G,
                         T_max, B, pos, idx, cnt, kmax, sl2, S, ws, ls);
      SW_MERGE(float, 64);
    }
  }
#undef SW_MERGE
#undef SW_MERGE_N
  return hipGetLastError();
}

}  // namespace sw

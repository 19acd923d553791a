// Block-sparse causal flash attention over the selected key blocks
// (paper Alg. 1 step 8): for each query head and query block, softmax over
// the tokens of the selected blocks that precede each query, renormalised
// over those keys only.
//
// bf16 kernels: one of eight wavefronts per workgroup, described here, and one
// of four or two for head dimension 64, for head counts that leave the eight
// without rows and for small launches (further down). Work item = (query block, KV head g, slice of
// the group's query heads). A 512-thread workgroup has 8 wavefronts, two per
// SIMD; each owns 32 query rows of one head (a B = 128 block takes four wavefronts per head, a
// B = 64 block two), so a workgroup serves two (B = 128) or four (B = 64)
// query heads of the same KV group from one copy of each K/V tile in LDS.
// The two wavefronts of a SIMD cover each other's LDS and barrier waits.
//
// Per wavefront and 32-key sub-tile the scores are computed transposed,
// S^T = K Q^T (v_mfma_f32_32x32x16_bf16, fp32 accumulate), so a lane owns one
// query column and its partial row sum; the other half-wave holds the rest of
// the row (one v_permlane32_swap combines them). P (rounded to bf16) feeds the
// B operand of O^T = V^T P^T straight from the accumulator layout. V stays in
// its natural row layout in LDS and the V^T operand is read with
// ds_read_b64_tr_b16, which hands each lane four consecutive keys of one
// dimension.
//
// Software pipeline over 32-key sub-tiles u, in a fixed issue order:
//   phase A: the score MFMAs of u+1, interleaved with the exponentials of
//            keys 16..31 of P(u);
//   phase B: the P.V MFMAs of u, interleaved with the exponentials of keys
//            0..15 of P(u+1).
// The exponent reference of a row does not track the row max on this path:
// between the phases, a row whose partial sum over P(u) exceeds kSumLimit
// (which bounds every element) takes the exact max of the sub-tile, rescales
// O and its sum and recomputes P(u) (rare, wave-uniform branch). Since
// O = sum(P V) / sum(P) for any common reference, the result does not depend
// on which reference was used.
//
// K/V tiles of 64 keys go through three LDS stages from registers loaded one
// tile ahead. The selected blocks are compacted in LDS at the start: valid
// blocks j < i first (never masked: only a sequence's last block can be
// partial), then the diagonal block i. The pipeline runs on into the
// diagonal block up to the sub-tile a wavefront's rows cross, which alone is
// masked (causal and sequence end); the sub-tiles after it are skipped. Work
// items run longest-first (query blocks in descending order, the selection
// budget grows with the block index) and the workgroups of one (query block,
// KV head) are placed on one XCD so they share the K/V blocks through that
// XCD's L2.
#include <type_traits>

#include "sw_common.h"
#include "sw_internal.h"

namespace sw {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int KT = 64;                 // keys per LDS tile
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNoRef = -1.0e30f;     // exponent reference before any key
constexpr float kSumLimit = 65536.0f;  // bound on a pipelined P sub-tile's partial row sum
constexpr int kPfWaves = 8;            // wavefronts per bf16 workgroup

// ---------------------------------------------------------------------------
// work mapping
// ---------------------------------------------------------------------------

// Rows with local block index >= x over all sequences (x may differ per
// lane); lane j of bl holds the block count of sequence j.
__device__ __forceinline__ int rows_from(int bl, int n_seqs, int x) {
  int c = 0;
  for (int j = 0; j < n_seqs; ++j) c += max(0, __builtin_amdgcn_readlane(bl, j) - x);
  return c;
}

// rho-th block row in longest-first order (local index descending, then
// sequence ascending). Returns the global row and the local index. Called by
// whole wavefronts: the block counts are spread over the lanes (at most 64
// sequences) and the local index is found by a 64-way search, each round
// testing 64 candidate indices at once.
__device__ __forceinline__ void lpt_row(const SeqMeta& m, int rho, int* row, int* s_out,
                                        int* i_out) {
  static_assert(SW_MAX_SEQS <= 64, "one sequence per lane");
  const int lane = threadIdx.x & 63;
  int bl = 0;
#pragma unroll
  for (int j = 0; j < SW_MAX_SEQS; ++j) {
    const int bj = m.blk_start[j + 1] - m.blk_start[j];
    bl = (lane == j && j < m.n_seqs) ? bj : bl;
  }
  // invariant: the answer (largest x with rows_from(x) > rho) lies in [lo, hi]
  int lo = 0, hi = m.max_b - 1;
  while (lo < hi) {
    const int step = (hi - lo + 63) >> 6;
    const int x = min(hi, lo + (lane + 1) * step);
    // rows_from decreases in x, so the passing candidates are a lane prefix
    const int pass = __popcll(__ballot(rows_from(bl, m.n_seqs, x) > rho));
    const int nlo = (pass == 0) ? lo : min(hi, lo + pass * step);
    hi = (pass == 64) ? hi : min(hi, lo + (pass + 1) * step) - 1;
    lo = nlo;
  }
  const int i = lo;
  const int k = rho - rows_from(bl, m.n_seqs, i + 1);   // rank among sequences longer than i
  const unsigned long long longer = __ballot(bl > i);
  const bool mine = ((longer >> lane) & 1ull) && (int)__popcll(longer & ((1ull << lane) - 1ull)) == k;
  const int s = __ffsll((unsigned long long)__ballot(mine)) - 1;
  *row = m.blk_start[s] + i;
  *s_out = s;
  *i_out = i;
}

// ---------------------------------------------------------------------------
// bf16 kernel
// ---------------------------------------------------------------------------

template <int D>
struct BfLds {
  static constexpr int KS = D + 8;     // K row stride (elements): rows 16 bytes apart in bank space
  static constexpr int VS = D + 32;    // V row stride (elements): rows 64 bytes apart in bank space
  static constexpr int K_ELEMS = KT * KS;
  static constexpr int V_ELEMS = KT * VS;
  static constexpr int STAGE = K_ELEMS + V_ELEMS;
  static constexpr int NST = 3;
};

// Raw buffer descriptor word 3 for gfx9-family untyped loads (32-bit data format).
constexpr int kBufWord3 = 0x00020000;

__device__ __forceinline__ float max_other_half(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_other_half(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

#define SW_INL __attribute__((always_inline))

template <int D, int BLK>
__global__ __launch_bounds__(kPfWaves * 64, 1) void attn_prefill_bf16_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, int h_q, int h_kv, long long N, SeqMeta m,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt, int kmax, float sl2,
    uint16_t* __restrict__ O, float* __restrict__ lse, int groups, int sg, int heads) {
  using L = BfLds<D>;
  constexpr int NT = kPfWaves * 64;        // threads
  __shared__ __attribute__((aligned(16))) uint16_t lds[L::NST * L::STAGE];
  __shared__ int blist[SW_MAX_BLOCKS];
  __shared__ int wtot[kPfWaves];

  // ---- work item ----
  const int x = blockIdx.x;
  const int xcd = x & 7;
  const int slot = x >> 3;
  const int mu = slot % sg;
  const int gamma = (slot / sg) * 8 + xcd;
  if (gamma >= groups) return;
  const int rho = gamma / h_kv;
  const int g = gamma % h_kv;
  int row, s, i;
  lpt_row(m, rho, &row, &s, &i);
  constexpr int WPB = BLK / 32;            // wavefronts per (query head, block)
  constexpr int TPB = BLK / KT;            // key tiles per block
  const int G = h_q / h_kv;
  const int tid = threadIdx.x;
  const int w = tid >> 6;
  const int l = tid & 63;
  const int hl = l >> 5;                   // half-wave
  const int ln = l & 31;                   // lane within half
  const int task = mu * kPfWaves + w;
  const int u = g * G + task / WPB;        // query head (meaningful only when active)
  const int seq0 = m.tok_start[s];
  const int seq1 = m.tok_start[s + 1];
  // 32-row group of the block owned by this wavefront. Wavefronts w and
  // w + 4 share a SIMD; the upper half takes the groups in reverse order so
  // the two hold complementary groups (g and WPB-1-g) and every SIMD has the
  // same number of unmasked diagonal sub-tiles.
  const int rgrp = (w >= kPfWaves / 2) ? WPB - 1 - task % WPB : task % WPB;
  const int q0 = seq0 + i * BLK + rgrp * 32;   // first query row of this wavefront
  const bool active = (task < heads * WPB) && (q0 < seq1);
  const int qpos = q0 + ln;                // this lane's query row

  // The selection count and the first chunk of the selection list are
  // loaded first, then Q: the list is needed first. The chunk lies within the
  // row's kmax entries whatever cnt holds.
  const int32_t* sel = idx + (long long)row * kmax;
  const int nsel = min(cnt[row], kmax);
  int jnext = (tid < kmax) ? sel[tid] : -1;

  // ---- Q fragments: lane holds query qpos, dims kk*16 + hl*8 .. +7 ----
  bf16x8 qf[D / 16];
  {
    const bool ok = active && qpos < seq1;
    const uint16_t* qrow = Q + ((long long)(ok ? u : 0) * N + (ok ? qpos : 0)) * D;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      uint4 v = ok ? *reinterpret_cast<const uint4*>(qrow + kk * 16 + hl * 8) : make_uint4(0, 0, 0, 0);
      qf[kk] = __builtin_bit_cast(bf16x8, v);
    }
  }

  // ---- selected blocks, compacted: valid j < i in list order, then i ----
  // Per chunk of NT entries each wavefront publishes its count of blocks
  // j < i (low 16 bits) and whether it saw the diagonal block (bit 16).
  int n_off = 0, sdiag = 0;
  for (int base = 0; base < nsel; base += NT) {
    const int e = base + tid;
    const int j = (e < nsel) ? jnext : -1;
    jnext = (e + NT < nsel) ? sel[e + NT] : -1;
    const bool off = (j >= 0 && j < i);
    const unsigned long long bal = __ballot(off);
    const bool dg = __ballot(j == i) != 0ull;
    const int pre = __popcll(bal & ((1ull << l) - 1ull));
    if (l == 0) wtot[w] = __popcll(bal) | (dg ? 0x10000 : 0);
    __syncthreads();
    int woff = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < kPfWaves; ++q) {
      const int c = wtot[q];
      woff += (q < w) ? (c & 0xffff) : 0;
      tot += c & 0xffff;
      sdiag |= c >> 16;
    }
    if (off && n_off + woff + pre < SW_MAX_BLOCKS) blist[n_off + woff + pre] = j;
    n_off = min(n_off + tot, SW_MAX_BLOCKS);
    __syncthreads();
  }
  const int n_blk = n_off + sdiag;
  const int ntiles = n_blk * TPB;
  const int nofft = n_off * TPB;           // tiles before the diagonal block

  // ---- K/V staging: global -> registers -> LDS, 16-byte chunks ----
  constexpr int KCH = D / 8;               // chunks per key row
  constexpr int KP = (KT * KCH) / NT;      // chunks per thread for K (and for V)
  static_assert(KP >= 1 && KP * NT == KT * KCH, "tile chunks must divide over the workgroup");
  uint4 kreg[KP], vreg[KP];
  int goff[KP], kloff[KP], vloff[KP];
#pragma unroll
  for (int p = 0; p < KP; ++p) {
    const int e = tid + p * NT;
    const int r = e / KCH, ch = e % KCH;
    goff[p] = (r * D + ch * 8) * 2;
    kloff[p] = r * L::KS + ch * 8;
    vloff[p] = r * L::VS + ch * 8;
  }
  const uint16_t* Kg = K + (long long)g * N * D;
  const uint16_t* Vg = V + (long long)g * N * D;
  // first key of tile t (wave-uniform)
  auto tile_k0 = [&](int t) SW_INL {
    const int jj = t / TPB;
    const int j = (jj < n_off) ? __builtin_amdgcn_readfirstlane(blist[jj]) : i;
    return seq0 + j * BLK + (t % TPB) * KT;
  };
  // Raw buffer loads through a descriptor based at the tile's first key k0
  // and sized to the end of the sequence: keys past the end read as zero
  // without per-lane tests (the diagonal-tile mask removes them).
  auto load_into = [&](int k0, uint4 (&kr)[KP], uint4 (&vr)[KP]) SW_INL {
    const int bytes = max(0, (seq1 - k0) * D * 2);
    const __amdgpu_buffer_rsrc_t rk =
        __builtin_amdgcn_make_buffer_rsrc((void*)(Kg + (long long)k0 * D), (short)0, bytes, kBufWord3);
    const __amdgpu_buffer_rsrc_t rv =
        __builtin_amdgcn_make_buffer_rsrc((void*)(Vg + (long long)k0 * D), (short)0, bytes, kBufWord3);
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      auto a = __builtin_amdgcn_raw_buffer_load_b128(rk, goff[p], 0, 0);
      kr[p] = __builtin_bit_cast(uint4, a);
      auto b = __builtin_amdgcn_raw_buffer_load_b128(rv, goff[p], 0, 0);
      vr[p] = __builtin_bit_cast(uint4, b);
    }
  };
  auto load_tile_at = [&](int k0) SW_INL { load_into(k0, kreg, vreg); };
  auto load_tile = [&](int t) SW_INL { load_tile_at(tile_k0(t)); };
  auto store_from = [&](int st, const uint4 (&kr)[KP], const uint4 (&vr)[KP]) SW_INL {
    uint16_t* ks = lds + st * L::STAGE;
    uint16_t* vs = ks + L::K_ELEMS;
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      *reinterpret_cast<uint4*>(ks + kloff[p]) = kr[p];
      *reinterpret_cast<uint4*>(vs + vloff[p]) = vr[p];
    }
  };
  auto store_tile = [&](int st) SW_INL { store_from(st, kreg, vreg); };

  // ---- running state ----
  f32x16 oacc[D / 32];
#pragma unroll
  for (int td = 0; td < D / 32; ++td)
#pragma unroll
    for (int j = 0; j < 16; ++j) oacc[td][j] = 0.0f;
  float mref = kNoRef;
  float lsum = 0.0f;
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  constexpr int NKK = D / 16;              // score MFMAs per sub-tile
  constexpr int NPV = 2 * (D / 32);        // P.V MFMAs per sub-tile: (chunk, dim block)
  constexpr int QK_PER_PAIR = NKK / 4;     // score MFMAs per element pair (phase A)
  constexpr int PV_PER_PAIR = NPV / 4;     // P.V MFMAs per element pair (phase B)
  constexpr int kAhead = 3;                // K and V^T operands are read this many MFMAs ahead
  // V^T operand lane offset: lane (ln, hl) reads with ds_read_b64_tr_b16 from
  // key row c*16 + 4*hl + (ln%16)/4 (+8) and dims td*32 + 16*(ln/16) + 4*(ln%4);
  // it receives dim td*32 + ln of keys c*16 + 4*hl + 0..3 and
  // c*16 + 8 + 4*hl + 0..3, the keys its P operand holds.
  const int vlane = (4 * hl + ((ln & 15) >> 2)) * L::VS + 16 * (ln >> 4) + 4 * (ln & 3);

  // Scores of 32 keys (half h2 of a 64-key tile) x 32 queries, transposed:
  // element j is key h2*32 + 8*(j/4) + 4*hl + j%4, query qpos.
  auto qk_sub = [&](const uint16_t* ks, int h2, f32x16& S) SW_INL {
#pragma unroll
    for (int j = 0; j < 16; ++j) S[j] = 0.0f;
    const uint16_t* kr = ks + (h2 * 32 + ln) * L::KS + hl * 8;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(kr + kk * 16);
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], S, 0, 0, 0);
    }
  };
  // causal + sequence-end mask of a diagonal-block sub-tile (raw scores)
  auto mask_sub = [&](int t, int h2, f32x16& S) SW_INL {
    const int k0 = tile_k0(t) + h2 * 32;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int kp = k0 + (j >> 2) * 8 + hl * 4 + (j & 3);
      if (kp > qpos || kp >= seq1) S[j] = -INFINITY;
    }
  };
  // row max of a sub-tile (log2 units)
  auto row_max = [&](const f32x16& S) SW_INL {
    float a = -INFINITY;
#pragma unroll
    for (int j = 0; j < 16; ++j) a = fmaxf(a, S[j]);
    return max_other_half(a) * sl2;
  };
  auto rescale_to = [&](float nref) SW_INL {
    const float alpha = __builtin_amdgcn_exp2f(mref - nref);
    mref = nref;
    lsum *= alpha;
#pragma unroll
    for (int td = 0; td < D / 32; ++td)
#pragma unroll
      for (int j = 0; j < 16; ++j) oacc[td][j] *= alpha;
  };
  // element pair e (elements 2e, 2e+1): P word and partial row sum
  auto pair = [&](const f32x16& S, int e, uint32_t& word, float& ts) SW_INL {
    const float nr = -mref;
    const float p0 = __builtin_amdgcn_exp2f(fmaf(S[2 * e], sl2, nr));
    const float p1 = __builtin_amdgcn_exp2f(fmaf(S[2 * e + 1], sl2, nr));
    word = pack_bf16x2(p0, p1);
    ts = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, word), ones, ts, false);
  };
  auto vread = [&](const uint16_t* vr, int n) SW_INL {
    const uint16_t* pp = vr + (n / (D / 32)) * 16 * L::VS + (n % (D / 32)) * 32;
    const i16x4 r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) i16x4*)(pp));
    const i16x4 r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) i16x4*)(pp + 8 * L::VS));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(r0, r1, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // rare path: exact row max of S, new reference, rescale, recompute P(u)
  auto refix = [&](const f32x16& S, uint32_t (&w0)[4], uint32_t (&w1)[4], float& ts) SW_INL {
    rescale_to(fmaxf(mref, row_max(S)));
    ts = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) pair(S, e, w0[e], ts);
#pragma unroll
    for (int e = 0; e < 4; ++e) pair(S, 4 + e, w1[e], ts);
  };
  auto check = [&](const f32x16& cur, uint32_t (&w0)[4], uint32_t (&w1)[4], float& ts) SW_INL {
    if (__any(ts > kSumLimit)) refix(cur, w0, w1, ts);
    lsum += ts;
  };
  // phase B: P.V of sub-tile u, with the chunk-0 exponentials of the next
  // sub-tile's scores when HAS_NEXT
  auto phase_b = [&](const uint16_t* vr, const uint32_t (&w0)[4], const uint32_t (&w1)[4],
                     bf16x8 (&vf)[NPV], const f32x16& nxt, uint32_t (&wn)[4], float& tn,
                     auto has_next) SW_INL {
    constexpr bool HAS_NEXT = decltype(has_next)::value;
    const bf16x8 pb[2] = {__builtin_bit_cast(bf16x8, w0), __builtin_bit_cast(bf16x8, w1)};
    tn = 0.0f;
#pragma unroll
    for (int n = 0; n < NPV; ++n) {
      if (n + kAhead < NPV) vf[n + kAhead] = vread(vr, n + kAhead);
      oacc[n % (D / 32)] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[n], pb[n / (D / 32)],
                                                                   oacc[n % (D / 32)], 0, 0, 0);
      if (HAS_NEXT && (n % PV_PER_PAIR) == PV_PER_PAIR - 1) {
        const int e = n / PV_PER_PAIR;               // 0..3
        pair(nxt, e, wn[e], tn);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // One pipeline sub-step (see the header): cur = S(u) with chunk-0 words wc
  // and their partial sum tc; produces nxt = S(u+1), its chunk-0 words wn and
  // partial sum tn.
  // tmask >= 0: S(u+1) is the wavefront's diagonal sub-tile, half h2n of
  // tile tmask, and is masked before its exponentials.
  auto sub = [&](f32x16& cur, uint32_t (&wc)[4], float& tc, f32x16& nxt, uint32_t (&wn)[4],
                 float& tn, const uint16_t* ksn, int h2n, const uint16_t* vs, int c0,
                 int tmask) SW_INL {
    const uint16_t* kr = ksn + (h2n * 32 + ln) * L::KS + hl * 8;
    const uint16_t* vr = vs + vlane + c0 * 16 * L::VS;
    uint32_t w1[4];
    bf16x8 kf[NKK];
    bf16x8 vf[NPV];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) kf[q] = *reinterpret_cast<const bf16x8*>(kr + q * 16);
#pragma unroll
    for (int j = 0; j < 16; ++j) nxt[j] = 0.0f;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      if (kk + kAhead < NKK) kf[kk + kAhead] = *reinterpret_cast<const bf16x8*>(kr + (kk + kAhead) * 16);
      if (kk >= NKK - kAhead) vf[kk - (NKK - kAhead)] = vread(vr, kk - (NKK - kAhead));
      nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], nxt, 0, 0, 0);
      if ((kk % QK_PER_PAIR) == QK_PER_PAIR - 1) {
        const int e = kk / QK_PER_PAIR;              // 0..3
        pair(cur, 4 + e, w1[e], tc);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (tmask >= 0) mask_sub(tmask, h2n, nxt);
    check(cur, wc, w1, tc);
    phase_b(vr, wc, w1, vf, nxt, wn, tn, std::true_type{});
  };
  // final sub-step of a wavefront's run: no scores ahead
  auto sub_last = [&](f32x16& cur, uint32_t (&wc)[4], float& tc, const uint16_t* vs, int c0) SW_INL {
    const uint16_t* vr = vs + vlane + c0 * 16 * L::VS;
    uint32_t w1[4];
    bf16x8 vf[NPV];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) vf[q] = vread(vr, q);
#pragma unroll
    for (int e = 0; e < 4; ++e) pair(cur, 4 + e, w1[e], tc);
    check(cur, wc, w1, tc);
    uint32_t wdummy[4];
    float tdummy;
    phase_b(vr, wc, w1, vf, cur, wdummy, tdummy, std::false_type{});
  };

  // Stages: during tile step t, K/V(t) are in stv, K(t+1) in stk, and tile
  // t+2 is written to stw from the registers loaded during step t-1; tile
  // t+3 is loaded into those registers.
  // The first key of tile t+3 is looked up one step ahead (k0_ahead), so the
  // LDS read of the block list never stalls the loads.
  int stv = 0, stk = 1, stw = 2;
  int k0_ahead = 0;
  auto stage_io = [&](int t) SW_INL {
    if (t + 2 < ntiles) store_tile(stw);
    if (t + 3 < ntiles) load_tile_at(k0_ahead);
    if (t + 4 < ntiles) k0_ahead = tile_k0(t + 4);
  };
  auto next_stage = [&]() SW_INL {
    const int t0 = stv;
    stv = stk;
    stk = stw;
    stw = t0;
    __syncthreads();
  };
  f32x16 sX, sY;
  uint32_t wX[4], wY[4];
  float tX = 0.0f, tY = 0.0f;
  // Last 32-key sub-tile of this wavefront's run, counting two per tile:
  // the off-diagonal blocks, then in the diagonal block the sub-tiles up to
  // the one its rows cross (number rgrp; the later ones lie after all its
  // rows and are skipped, the earlier ones precede them and need no mask).
  // Wavefronts without rows stop after the off-diagonal blocks.
  const int uend = 2 * nofft - 1 + ((active && sdiag) ? rgrp + 1 : 0);
  // off-diagonal tile t < nofft-1: both halves, the second computing the
  // first half of tile t+1 (every wavefront's run goes past it)
  auto tile_step = [&](int t) SW_INL {
    stage_io(t);
    const uint16_t* kt = lds + stv * L::STAGE;
    const uint16_t* vs = kt + L::K_ELEMS;
    sub(sX, wX, tX, sY, wY, tY, kt, 1, vs, 0, -1);
    sub(sY, wY, tY, sX, wX, tX, lds + stk * L::STAGE, 0, vs, 2, -1);
    next_stage();
  };
  // any later tile: each half continues, ends or skips this wavefront's run
  auto tile_end = [&](int t) SW_INL {
    stage_io(t);
    const uint16_t* kt = lds + stv * L::STAGE;
    const uint16_t* vs = kt + L::K_ELEMS;
    const int v0 = 2 * t;
    if (v0 + 1 <= uend) sub(sX, wX, tX, sY, wY, tY, kt, 1, vs, 0, (v0 + 1 == uend) ? t : -1);
    else if (v0 == uend) sub_last(sX, wX, tX, vs, 0);
    if (v0 + 2 <= uend)
      sub(sY, wY, tY, sX, wX, tX, lds + stk * L::STAGE, 0, vs, 2, (v0 + 2 == uend) ? t + 1 : -1);
    else if (v0 + 1 == uend) sub_last(sY, wY, tY, vs, 2);
    next_stage();
  };

  if (ntiles > 0) {
    // tiles 0 and 1 are loaded together (a second register set), then tile 2
    uint4 k1reg[KP], v1reg[KP];
    load_tile(0);
    if (ntiles > 1) load_into(tile_k0(1), k1reg, v1reg);
    store_tile(0);
    if (ntiles > 1) store_from(1, k1reg, v1reg);
    if (ntiles > 2) load_tile(2);
    if (ntiles > 3) k0_ahead = tile_k0(3);
    __syncthreads();
    if (uend >= 0) {
      // scores of the first sub-tile; its chunk-0 words are left to the
      // first check (an infinite partial sum forces the exact reference)
      qk_sub(lds, 0, sX);
      if (uend == 0) mask_sub(0, 0, sX);
      tX = INFINITY;
#pragma unroll
      for (int e = 0; e < 4; ++e) wX[e] = 0u;
    }
    int t = 0;
    for (; t + 1 < nofft; ++t) tile_step(t);
    for (; t < ntiles; ++t) tile_end(t);
  }

  // ---- epilogue ----
  // The wavefront's 32 x D output rows are normalised into LDS (the K/V
  // stages are free once every wavefront has passed the barrier) and written
  // back row-contiguous: rows q0..q0+31 of head u are one contiguous run of
  // O, so each 16-byte-per-lane store covers 64 / (D / 8) whole rows.
  const float ltot = sum_other_half(lsum);
  const float inv = ltot > 0.0f ? 1.0f / ltot : 0.0f;
  constexpr int OS = D + 8;                // output row stride in LDS (elements)
  static_assert(kPfWaves * 32 * OS <= L::NST * L::STAGE, "output staging must fit the K/V stages");
  __syncthreads();
  uint16_t* ob = lds + w * 32 * OS;
#pragma unroll
  for (int td = 0; td < D / 32; ++td) {
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      uint2 st;
      st.x = pack_bf16x2(oacc[td][jb * 4 + 0] * inv, oacc[td][jb * 4 + 1] * inv);
      st.y = pack_bf16x2(oacc[td][jb * 4 + 2] * inv, oacc[td][jb * 4 + 3] * inv);
      *reinterpret_cast<uint2*>(ob + ln * OS + td * 32 + jb * 8 + hl * 4) = st;
    }
  }
  if (!active) return;
  constexpr int CPR = D / 8;               // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;            // rows per store instruction
  const int rr = l / CPR, cc = l % CPR;
  uint16_t* obase = O + ((long long)u * N + q0) * D;
#pragma unroll
  for (int it = 0; it < 32 / RPI; ++it) {
    const int r = it * RPI + rr;
    const uint4 v = *reinterpret_cast<const uint4*>(ob + r * OS + cc * 8);
    if (q0 + r < seq1) *reinterpret_cast<uint4*>(obase + (long long)r * D + cc * 8) = v;
  }
  if (lse && hl == 0 && qpos < seq1)
    lse[(long long)u * N + qpos] = (ltot > 0.0f) ? (mref + log2f(ltot)) / kLog2e : -INFINITY;
}

// ---------------------------------------------------------------------------
// bf16 kernel, four or two wavefronts
// ---------------------------------------------------------------------------

// The pipeline of the eight-wavefront kernel for workgroups of NW = 4
// wavefronts, two or three to a CU: one workgroup's list, first tiles and
// output run beside another's math. A step is 32 keys per wavefront: the
// scores of step t + 1 and the P.V of step t, so K is staged one step ahead of
// V and two slots of each suffice, with one barrier a step.
// NW = 2 where there are rows for two wavefronts only (one query head and
// blocks of 64): half the threads, twice the workgroups on a CU.
// A wavefront does what one of the eight does for the same rows, in the same
// order, so that a row's bits do not depend on which of the kernels took it.
// Each K/V tile serves 128 query rows (64 with NW = 2) and not 256, so its
// staging weighs more. No unit is saturated: at 16 heads of d = 64, 8000 tokens
// (NW = 2) the matrix cores are busy 20 % of the cycles, the vector unit 33 %, the
// LDS 22 %; with 1.7 wavefronts a SIMD on average, 37 % of their time is spent
// waiting for memory, LDS or the barrier. The steps at the end (a wavefront goes on, masks, ends
// or skips) run one at a time with the state copied over: unrolled by two like
// the main loop they took 282 VGPRs at D = 128 and spilled.
template <int D>
struct W4Lds {
  static constexpr int KT4 = 32;           // keys per step
  static constexpr int KS = BfLds<D>::KS;
  static constexpr int VS = BfLds<D>::VS;
  static constexpr int K_ELEMS = KT4 * KS;
  static constexpr int V_ELEMS = KT4 * VS;
  static constexpr int SLOTS = 2 * (K_ELEMS + V_ELEMS);   // two K slots, two V slots
};

template <int D, int BLK, int NW>
__global__ __launch_bounds__(NW * 64, 2) void attn_prefill_w4_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, int h_q, int h_kv, long long N, SeqMeta m,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt, int kmax, float sl2,
    uint16_t* __restrict__ O, float* __restrict__ lse, int groups, int sg, int head0) {
  using L = W4Lds<D>;
  constexpr int NT = NW * 64;
  __shared__ __attribute__((aligned(16))) uint16_t lds[L::SLOTS];
  __shared__ int16_t blist[SW_MAX_BLOCKS];
  __shared__ int wtot[NW];

  // ---- work item ----
  const int x = blockIdx.x;
  const int xcd = x & 7;
  const int slot = x >> 3;
  const int mu = slot % sg;
  const int gamma = (slot / sg) * 8 + xcd;
  if (gamma >= groups) return;
  const int rho = gamma / h_kv;
  const int g = gamma % h_kv;
  int row, s, i;
  lpt_row(m, rho, &row, &s, &i);
  constexpr int WPB = BLK / 32;            // 32-row groups per (query head, block)
  constexpr int TPB = BLK / L::KT4;        // steps per block
  const int G = h_q / h_kv;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63;
  const int hl = l >> 5;                   // half-wave
  const int ln = l & 31;                   // lane within half
  const int task = mu * NW + w;
  const int hd = head0 + task / WPB;       // query head of the group
  const int u = g * G + hd;                // (meaningful only when active)
  const int seq0 = m.tok_start[s];
  const int seq1 = m.tok_start[s + 1];
  const int rgrp = task % WPB;
  const int q0 = seq0 + i * BLK + rgrp * 32;   // first query row of this wavefront
  const bool active = (hd < G) && (q0 < seq1);
  const int qpos = q0 + ln;                // this lane's query row

  const int32_t* sel = idx + (long long)row * kmax;
  const int nsel = min(cnt[row], kmax);
  int jnext = (tid < kmax) ? sel[tid] : -1;

  // ---- Q fragments: lane holds query qpos, dims kk*16 + hl*8 .. +7 ----
  bf16x8 qf[D / 16];
  {
    const bool ok = active && qpos < seq1;
    const uint16_t* qrow = Q + ((long long)(ok ? u : 0) * N + (ok ? qpos : 0)) * D;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      uint4 v = ok ? *reinterpret_cast<const uint4*>(qrow + kk * 16 + hl * 8) : make_uint4(0, 0, 0, 0);
      qf[kk] = __builtin_bit_cast(bf16x8, v);
    }
  }

  // ---- selected blocks, compacted: valid j < i in list order, then i ----
  int n_off = 0, sdiag = 0;
  for (int base = 0; base < nsel; base += NT) {
    const int e = base + tid;
    const int j = (e < nsel) ? jnext : -1;
    jnext = (e + NT < nsel) ? sel[e + NT] : -1;
    const bool off = (j >= 0 && j < i);
    const unsigned long long bal = __ballot(off);
    const bool dg = __ballot(j == i) != 0ull;
    const int pre = __popcll(bal & ((1ull << l) - 1ull));
    if (l == 0) wtot[w] = __popcll(bal) | (dg ? 0x10000 : 0);
    __syncthreads();
    int woff = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      const int c = wtot[q];
      woff += (q < w) ? (c & 0xffff) : 0;
      tot += c & 0xffff;
      sdiag |= c >> 16;
    }
    if (off && n_off + woff + pre < SW_MAX_BLOCKS) blist[n_off + woff + pre] = (int16_t)j;
    n_off = min(n_off + tot, SW_MAX_BLOCKS);
    __syncthreads();
  }
  const int n_blk = n_off + sdiag;
  const int nsteps = n_blk * TPB;
  const int noffs = n_off * TPB;           // steps before the diagonal block

  // ---- K/V staging: global -> registers -> LDS, 16-byte chunks ----
  constexpr int KCH = D / 8;               // chunks per key row
  constexpr int KP = (L::KT4 * KCH) / NT;  // chunks per thread for K (and for V)
  static_assert(KP >= 1 && KP * NT == L::KT4 * KCH && NT % KCH == 0, "step chunks must divide over the workgroup");
  constexpr int RPP = NT / KCH;            // key rows per chunk pass
  const int sr = tid / KCH, sc = tid % KCH;
  const int goff = (sr * D + sc * 8) * 2;
  const int kloff = sr * L::KS + sc * 8;
  const int vloff = sr * L::VS + sc * 8;
  uint16_t* const kslots = lds;
  uint16_t* const vslots = lds + 2 * L::K_ELEMS;
  const uint16_t* Kg = K + (long long)g * N * D;
  const uint16_t* Vg = V + (long long)g * N * D;
  // first key of step t (wave-uniform)
  auto step_k0 = [&](int t) SW_INL {
    const int jj = t / TPB;
    const int j = (jj < n_off) ? __builtin_amdgcn_readfirstlane((int)blist[jj]) : i;
    return seq0 + j * BLK + (t % TPB) * L::KT4;
  };
  // keys past the end of the sequence read as zero (the mask removes them)
  auto load = [&](const uint16_t* base, int k0, uint4 (&r)[KP]) SW_INL {
    const int bytes = max(0, (seq1 - k0) * D * 2);
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)(base + (long long)k0 * D), (short)0, bytes, kBufWord3);
#pragma unroll
    for (int p = 0; p < KP; ++p)
      r[p] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, goff + p * RPP * D * 2, 0, 0));
  };
  auto store_k = [&](int sl, const uint4 (&r)[KP]) SW_INL {
#pragma unroll
    for (int p = 0; p < KP; ++p)
      *reinterpret_cast<uint4*>(kslots + sl * L::K_ELEMS + kloff + p * RPP * L::KS) = r[p];
  };
  auto store_v = [&](int sl, const uint4 (&r)[KP]) SW_INL {
#pragma unroll
    for (int p = 0; p < KP; ++p)
      *reinterpret_cast<uint4*>(vslots + sl * L::V_ELEMS + vloff + p * RPP * L::VS) = r[p];
  };

  // ---- running state ----
  f32x16 oacc[D / 32];
#pragma unroll
  for (int td = 0; td < D / 32; ++td)
#pragma unroll
    for (int j = 0; j < 16; ++j) oacc[td][j] = 0.0f;
  float mref = kNoRef;
  float lsum = 0.0f;
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  constexpr int NKK = D / 16;              // score MFMAs per sub-tile
  constexpr int NPV = 2 * (D / 32);        // P.V MFMAs per sub-tile: (chunk, dim block)
  constexpr int QK_PER_PAIR = NKK / 4;     // score MFMAs per element pair (phase A)
  constexpr int PV_PER_PAIR = NPV / 4;     // P.V MFMAs per element pair (phase B)
  constexpr int kAhead = 3;                // K and V^T operands are read this many MFMAs ahead
  // V^T operand lane offset (see the eight-wavefront kernel)
  const int vlane = (4 * hl + ((ln & 15) >> 2)) * L::VS + 16 * (ln >> 4) + 4 * (ln & 3);
  const int klane = ln * L::KS + hl * 8;

  // causal + sequence-end mask of the diagonal sub-tile (raw scores)
  auto mask_sub = [&](int t, f32x16& S) SW_INL {
    const int k0 = step_k0(t);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int kp = k0 + (j >> 2) * 8 + hl * 4 + (j & 3);
      if (kp > qpos || kp >= seq1) S[j] = -INFINITY;
    }
  };
  auto row_max = [&](const f32x16& S) SW_INL {
    float a = -INFINITY;
#pragma unroll
    for (int j = 0; j < 16; ++j) a = fmaxf(a, S[j]);
    return max_other_half(a) * sl2;
  };
  auto rescale_to = [&](float nref) SW_INL {
    const float alpha = __builtin_amdgcn_exp2f(mref - nref);
    mref = nref;
    lsum *= alpha;
#pragma unroll
    for (int td = 0; td < D / 32; ++td)
#pragma unroll
      for (int j = 0; j < 16; ++j) oacc[td][j] *= alpha;
  };
  auto pair = [&](const f32x16& S, int e, uint32_t& word, float& ts) SW_INL {
    const float nr = -mref;
    const float p0 = __builtin_amdgcn_exp2f(fmaf(S[2 * e], sl2, nr));
    const float p1 = __builtin_amdgcn_exp2f(fmaf(S[2 * e + 1], sl2, nr));
    word = pack_bf16x2(p0, p1);
    ts = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, word), ones, ts, false);
  };
  auto vread = [&](const uint16_t* vr, int n) SW_INL {
    const uint16_t* pp = vr + (n / (D / 32)) * 16 * L::VS + (n % (D / 32)) * 32;
    const i16x4 r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) i16x4*)(pp));
    const i16x4 r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) i16x4*)(pp + 8 * L::VS));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(r0, r1, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // rare path: exact row max of S, new reference, rescale, recompute P
  auto check = [&](const f32x16& S, uint32_t (&w0)[4], uint32_t (&w1)[4], float& ts) SW_INL {
    if (__any(ts > kSumLimit)) {
      rescale_to(fmaxf(mref, row_max(S)));
      ts = 0.0f;
#pragma unroll
      for (int e = 0; e < 4; ++e) pair(S, e, w0[e], ts);
#pragma unroll
      for (int e = 0; e < 4; ++e) pair(S, 4 + e, w1[e], ts);
    }
    lsum += ts;
  };
  auto phase_b = [&](const uint16_t* vr, const uint32_t (&w0)[4], const uint32_t (&w1)[4],
                     bf16x8 (&vf)[NPV], const f32x16& nxt, uint32_t (&wn)[4], float& tn,
                     auto has_next) SW_INL {
    constexpr bool HAS_NEXT = decltype(has_next)::value;
    const bf16x8 pb[2] = {__builtin_bit_cast(bf16x8, w0), __builtin_bit_cast(bf16x8, w1)};
    tn = 0.0f;
#pragma unroll
    for (int n = 0; n < NPV; ++n) {
      if (n + kAhead < NPV) vf[n + kAhead] = vread(vr, n + kAhead);
      oacc[n % (D / 32)] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[n], pb[n / (D / 32)],
                                                                   oacc[n % (D / 32)], 0, 0, 0);
      if (HAS_NEXT && (n % PV_PER_PAIR) == PV_PER_PAIR - 1) {
        const int e = n / PV_PER_PAIR;               // 0..3
        pair(nxt, e, wn[e], tn);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // one step: cur = S(t) with chunk-0 words wc and partial sum tc; produces
  // nxt = S(t+1) (masked when tmask >= 0), its chunk-0 words and partial sum
  auto sub = [&](f32x16& cur, uint32_t (&wc)[4], float& tc, f32x16& nxt, uint32_t (&wn)[4],
                 float& tn, int ksl, int vsl, int tmask) SW_INL {
    const uint16_t* kr = kslots + ksl * L::K_ELEMS + klane;
    const uint16_t* vr = vslots + vsl * L::V_ELEMS + vlane;
    uint32_t w1[4];
    bf16x8 kf[NKK];
    bf16x8 vf[NPV];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) kf[q] = *reinterpret_cast<const bf16x8*>(kr + q * 16);
#pragma unroll
    for (int j = 0; j < 16; ++j) nxt[j] = 0.0f;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      if (kk + kAhead < NKK) kf[kk + kAhead] = *reinterpret_cast<const bf16x8*>(kr + (kk + kAhead) * 16);
      if (kk >= NKK - kAhead) vf[kk - (NKK - kAhead)] = vread(vr, kk - (NKK - kAhead));
      nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], nxt, 0, 0, 0);
      if ((kk % QK_PER_PAIR) == QK_PER_PAIR - 1) {
        const int e = kk / QK_PER_PAIR;              // 0..3
        pair(cur, 4 + e, w1[e], tc);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (tmask >= 0) mask_sub(tmask, nxt);
    check(cur, wc, w1, tc);
    phase_b(vr, wc, w1, vf, nxt, wn, tn, std::true_type{});
  };
  auto sub_last = [&](f32x16& cur, uint32_t (&wc)[4], float& tc, int vsl) SW_INL {
    const uint16_t* vr = vslots + vsl * L::V_ELEMS + vlane;
    uint32_t w1[4];
    bf16x8 vf[NPV];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) vf[q] = vread(vr, q);
#pragma unroll
    for (int e = 0; e < 4; ++e) pair(cur, 4 + e, w1[e], tc);
    check(cur, wc, w1, tc);
    uint32_t wdummy[4];
    float tdummy;
    phase_b(vr, wc, w1, vf, cur, wdummy, tdummy, std::false_type{});
  };

  // Last step of this wavefront's run: the steps of the off-diagonal blocks,
  // then in the diagonal block those up to the sub-tile its rows cross, the
  // masked one (later ones lie after all its rows).
  const bool dmine = active && sdiag;
  const int tend = noffs - 1 + (dmine ? rgrp + 1 : 0);
  const int tmasked = dmine ? tend : -1;
  f32x16 sX, sY;
  uint32_t wX[4], wY[4];
  float tX = 0.0f, tY = 0.0f;
  // Step t stores K(t+2) and V(t+1) into the slots whose tiles step t-1 read
  // last (K runs a step ahead of V, as the scores do), then loads K(t+3) and
  // V(t+2) into the same registers.
  uint4 kr[KP], vr[KP];
  int k0_2 = 0, k0_3 = 0;                  // first keys of steps t+2 and t+3
  auto io = [&](int t) SW_INL {
    if (t + 2 < nsteps) store_k(t & 1, kr);
    if (t + 1 < nsteps) store_v((t + 1) & 1, vr);
    if (t + 3 < nsteps) load(Kg, k0_3, kr);
    if (t + 2 < nsteps) load(Vg, k0_2, vr);
    k0_2 = k0_3;
    if (t + 4 < nsteps) k0_3 = step_k0(t + 4);
  };
  if (nsteps > 0) {
    {
      uint4 k1r[KP], v0r[KP];
      const int a0 = step_k0(0), a1 = nsteps > 1 ? step_k0(1) : 0;
      if (nsteps > 2) k0_2 = step_k0(2);
      if (nsteps > 3) k0_3 = step_k0(3);
      load(Kg, a0, kr);
      if (nsteps > 1) load(Kg, a1, k1r);
      load(Vg, a0, v0r);
      if (nsteps > 1) load(Vg, a1, vr);
      store_k(0, kr);
      if (nsteps > 2) load(Kg, k0_2, kr);
      if (nsteps > 1) store_k(1, k1r);
      store_v(0, v0r);
    }
    __syncthreads();
    if (tend >= 0) {
      // scores of the first sub-tile; its chunk-0 words are left to the first
      // check (an infinite partial sum forces the exact reference)
      const uint16_t* kr = kslots + klane;
#pragma unroll
      for (int j = 0; j < 16; ++j) sX[j] = 0.0f;
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk)
        sX = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(kr + kk * 16),
                                                     qf[kk], sX, 0, 0, 0);
      if (tmasked == 0) mask_sub(0, sX);
      tX = INFINITY;
#pragma unroll
      for (int e = 0; e < 4; ++e) wX[e] = 0u;
    }
    __syncthreads();
    // steps t, t+1 with every wavefront's run going past t+2: no masks, no ends
    int t = 0;
    for (; t + 2 < noffs; t += 2) {
      io(t);
      sub(sX, wX, tX, sY, wY, tY, 1, 0, -1);
      __syncthreads();
      io(t + 1);
      sub(sY, wY, tY, sX, wX, tX, 0, 1, -1);
      __syncthreads();
    }
    // the last steps: each wavefront goes on, ends, then keeps the others company
    for (; t < tend; ++t) {
      io(t);
      sub(sX, wX, tX, sY, wY, tY, (t + 1) & 1, t & 1, (t + 1 == tmasked) ? t + 1 : -1);
      sX = sY;
      tX = tY;
#pragma unroll
      for (int e = 0; e < 4; ++e) wX[e] = wY[e];
      __syncthreads();
    }
    if (t == tend) {
      io(t);
      sub_last(sX, wX, tX, t & 1);
      __syncthreads();
      ++t;
    }
    for (; t < nsteps; ++t) {
      io(t);
      __syncthreads();
    }
  }

  // ---- epilogue (the slots are free: every run ended before the last barrier) ----
  const float ltot = sum_other_half(lsum);
  const float inv = ltot > 0.0f ? 1.0f / ltot : 0.0f;
  constexpr int OS = D + 8;                // output row stride in LDS (elements)
  static_assert(NW * 32 * OS <= L::SLOTS, "output staging must fit the slots");
  uint16_t* ob = lds + w * 32 * OS;        // this wavefront's own rows: no barrier
#pragma unroll
  for (int td = 0; td < D / 32; ++td) {
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      uint2 st;
      st.x = pack_bf16x2(oacc[td][jb * 4 + 0] * inv, oacc[td][jb * 4 + 1] * inv);
      st.y = pack_bf16x2(oacc[td][jb * 4 + 2] * inv, oacc[td][jb * 4 + 3] * inv);
      *reinterpret_cast<uint2*>(ob + ln * OS + td * 32 + jb * 8 + hl * 4) = st;
    }
  }
  if (!active) return;
  constexpr int CPR = D / 8;               // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;            // rows per store instruction
  const int rr = l / CPR, cc = l % CPR;
  uint16_t* obase = O + ((long long)u * N + q0) * D;
#pragma unroll
  for (int it = 0; it < 32 / RPI; ++it) {
    const int r = it * RPI + rr;
    const uint4 v = *reinterpret_cast<const uint4*>(ob + r * OS + cc * 8);
    if (q0 + r < seq1) *reinterpret_cast<uint4*>(obase + (long long)r * D + cc * 8) = v;
  }
  if (lse && hl == 0 && qpos < seq1)
    lse[(long long)u * N + qpos] = (ltot > 0.0f) ? (mref + log2f(ltot)) / kLog2e : -INFINITY;
}

// ---------------------------------------------------------------------------
// fp32 kernel
// ---------------------------------------------------------------------------

// The work split and staging of the four-wavefront kernel, with every fp32
// operand taken apart into three bf16 parts (8 significant bits each, so 24 in
// all) and every product formed from the six partial products above 2^-24 of
// it on v_mfma_f32_32x32x16_bf16. Six of them take 192 cycles per 16 dims
// against 512 for the fp32 matrix instruction, and the sums are rounded once
// per 16 products and not once per 2. Against 64 bits (8 query heads over 2,
// d = 128, 6000 tokens) the output is 3.0e-7 off (relative, 2-norm) where the
// fp32 instruction gave 5.3e-7.
// Scores: the leading products and the five smaller ones have sums of their
// own. At d = 128 a SIMD has one wavefront (registers), which issues 490 vector
// instructions beside the 96 matrix instructions of a step, 208 of them to take
// the K/V pieces apart and 88 the weights: the matrix cores are busy 36 % of the
// cycles, the vector unit 34 %, a quarter of the former at the same time. The
// weights of step t are formed between the score products of step t + 1, the
// pieces of the tiles to come between the products with V.
// 8 query heads over 2, d = 128, B = 64, 8192 tokens, 20 %: 331 -> 181 us (82
// -> 153 TFLOP/s of the function's own operations).
//
// x = h + m + l in bf16: h = bf16(x), m = bf16(x - h), l = bf16(x - h - m), each
// difference exact in fp32; what is left out is below 2^-25 |x|. RANGE: h is the
// largest finite bf16 where x would round to infinity (above 3.39e38). Parts below
// 2^-133 are lost, so an operand below 2^-110 (7.7e-34) counts with an error of
// up to 2^-134: keys, queries or values all scaled by 2^-110 / -114 / -118 came
// out 1.4e-7 / 5e-7 / 8e-6 off (fp32 instruction 2.9e-7 down to 2^-122).
template <bool RANGE = true>
__device__ __forceinline__ void split2(float x0, float x1, uint32_t& h, uint32_t& m, uint32_t& l) {
  constexpr float kTop = 3.3895313892515355e38f;   // largest finite bf16
  h = RANGE ? pack_bf16x2(__builtin_amdgcn_fmed3f(x0, -kTop, kTop), __builtin_amdgcn_fmed3f(x1, -kTop, kTop))
            : pack_bf16x2(x0, x1);
  const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xffff0000u);
  m = pack_bf16x2(r0, r1);
  l = pack_bf16x2(r0 - __uint_as_float(m << 16), r1 - __uint_as_float(m & 0xffff0000u));
}

template <int D, int KH>
struct F32Lds {
  static constexpr int KT4 = 32 * KH;      // keys per step, 32 per wavefront
  static constexpr int KS = D + 8;         // row strides as in the bf16 kernels
  static constexpr int VS = D + 32;
  static constexpr int K_PLANE = KT4 * KS;
  static constexpr int V_PLANE = KT4 * VS;
  static constexpr int SLOT = 3 * (K_PLANE + V_PLANE);
  static constexpr int SLOTS = (2 * SLOT * 2 <= 144 * 1024) ? 2 : 1;   // of K and of V
};

template <int D, int BLK, int KH>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_prefill_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    int h_q, int h_kv, long long N, SeqMeta m, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ cnt, int kmax, float sl2, float* __restrict__ O,
    float* __restrict__ lse, int groups, int sg) {
  using L = F32Lds<D, KH>;
  constexpr int NT = 256;
  constexpr int NW = 4;
  __shared__ __attribute__((aligned(16))) uint16_t lds[L::SLOTS * L::SLOT];
  __shared__ int16_t blist[SW_MAX_BLOCKS];
  __shared__ int wtot[NW];

  // ---- work item ----
  const int x = blockIdx.x;
  const int xcd = x & 7;
  const int slot = x >> 3;
  const int mu = slot % sg;
  const int gamma = (slot / sg) * 8 + xcd;
  if (gamma >= groups) return;
  const int rho = gamma / h_kv;
  const int g = gamma % h_kv;
  int row, s, i;
  lpt_row(m, rho, &row, &s, &i);
  constexpr int WPB = BLK / 32;            // 32-row groups per (query head, block)
  constexpr int TPB = BLK / L::KT4;        // steps per block
  static_assert(KH == 1 || (KH == 2 && BLK == 64), "key halves: a block is one step");
  const int G = h_q / h_kv;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63;
  const int hl = l >> 5;
  const int ln = l & 31;
  const int kh = (KH == 2) ? w & 1 : 0;    // this wavefront's 32 keys of a step
  const int task = mu * (NW / KH) + w / KH;
  const int u = g * G + task / WPB;
  const int seq0 = m.tok_start[s];
  const int seq1 = m.tok_start[s + 1];
  const int rgrp = task % WPB;
  const int q0 = seq0 + i * BLK + rgrp * 32;
  const bool active = (task < G * WPB) && (q0 < seq1);
  const int qpos = q0 + ln;

  const int32_t* sel = idx + (long long)row * kmax;
  const int nsel = min(cnt[row], kmax);
  int jnext = (tid < kmax) ? sel[tid] : -1;

  // ---- Q fragments in three planes: lane holds query qpos, dims kk*16 + hl*8 .. +7 ----
  bf16x8 qf[3][D / 16];
  {
    const bool ok = active && qpos < seq1;
    const float* qrow = Q + ((long long)(ok ? u : 0) * N + (ok ? qpos : 0)) * D;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      const float4* p = reinterpret_cast<const float4*>(qrow + kk * 16 + hl * 8);
      const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
      const float4 a = ok ? p[0] : z, b = ok ? p[1] : z;
      uint4 h, md, lo;
      split2(a.x, a.y, h.x, md.x, lo.x);
      split2(a.z, a.w, h.y, md.y, lo.y);
      split2(b.x, b.y, h.z, md.z, lo.z);
      split2(b.z, b.w, h.w, md.w, lo.w);
      qf[0][kk] = __builtin_bit_cast(bf16x8, h);
      qf[1][kk] = __builtin_bit_cast(bf16x8, md);
      qf[2][kk] = __builtin_bit_cast(bf16x8, lo);
    }
  }

  // ---- selected blocks, compacted: valid j < i in list order, then i ----
  int n_off = 0, sdiag = 0;
  for (int base = 0; base < nsel; base += NT) {
    const int e = base + tid;
    const int j = (e < nsel) ? jnext : -1;
    jnext = (e + NT < nsel) ? sel[e + NT] : -1;
    const bool off = (j >= 0 && j < i);
    const unsigned long long bal = __ballot(off);
    const bool dg = __ballot(j == i) != 0ull;
    const int pre = __popcll(bal & ((1ull << l) - 1ull));
    if (l == 0) wtot[w] = __popcll(bal) | (dg ? 0x10000 : 0);
    __syncthreads();
    int woff = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      const int c = wtot[q];
      woff += (q < w) ? (c & 0xffff) : 0;
      tot += c & 0xffff;
      sdiag |= c >> 16;
    }
    if (off && n_off + woff + pre < SW_MAX_BLOCKS) blist[n_off + woff + pre] = (int16_t)j;
    n_off = min(n_off + tot, SW_MAX_BLOCKS);
    __syncthreads();
  }
  const int n_blk = n_off + sdiag;
  const int nsteps = n_blk * TPB;
  const int noffs = n_off * TPB;

  // ---- K/V staging: global -> registers -> three bf16 planes in LDS ----
  constexpr int KCH = D / 4;               // 16-byte chunks per key row
  constexpr int KP = (L::KT4 * KCH) / NT;  // chunks per thread for K (and for V)
  static_assert(KP >= 1 && KP * NT == L::KT4 * KCH && NT % KCH == 0, "step chunks must divide over the workgroup");
  constexpr int RPP = NT / KCH;            // key rows per chunk pass
  const int sr = tid / KCH, sc = tid % KCH;
  const int goff = (sr * D + sc * 4) * 4;
  const int kloff = sr * L::KS + sc * 4;
  const int vloff = sr * L::VS + sc * 4;
  const float* Kg = K + (long long)g * N * D;
  const float* Vg = V + (long long)g * N * D;
  auto step_k0 = [&](int t) SW_INL {
    const int jj = t / TPB;
    const int j = (jj < n_off) ? __builtin_amdgcn_readfirstlane((int)blist[jj]) : i;
    return seq0 + j * BLK + (t % TPB) * L::KT4;
  };
  uint16_t* const kslots = lds;
  uint16_t* const vslots = lds + L::SLOTS * 3 * L::K_PLANE;
  uint4 kr[KP], vr[KP];
  // keys past the end of the sequence read as zero (the mask removes them)
  auto load = [&](const float* base, int k0, uint4 (&r)[KP]) SW_INL {
    const int bytes = max(0, (seq1 - k0) * D * 4);
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)(base + (long long)k0 * D), (short)0, bytes, kBufWord3);
#pragma unroll
    for (int p = 0; p < KP; ++p)
      r[p] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, goff + p * RPP * D * 4, 0, 0));
  };
  // one 16-byte piece into its three planes
  auto put = [&](uint16_t* to, int plane, const uint4& r) SW_INL {
    uint2 h, md, lo;
    split2(__uint_as_float(r.x), __uint_as_float(r.y), h.x, md.x, lo.x);
    split2(__uint_as_float(r.z), __uint_as_float(r.w), h.y, md.y, lo.y);
    *reinterpret_cast<uint2*>(to) = h;
    *reinterpret_cast<uint2*>(to + plane) = md;
    *reinterpret_cast<uint2*>(to + 2 * plane) = lo;
  };
  auto put_k = [&](int sl, int p) SW_INL {
    put(kslots + sl * 3 * L::K_PLANE + kloff + p * RPP * L::KS, L::K_PLANE, kr[p]);
  };
  auto put_v = [&](int sl, int p) SW_INL {
    put(vslots + sl * 3 * L::V_PLANE + vloff + p * RPP * L::VS, L::V_PLANE, vr[p]);
  };

  // ---- running state ----
  f32x16 oacc[D / 32];
#pragma unroll
  for (int td = 0; td < D / 32; ++td)
#pragma unroll
    for (int j = 0; j < 16; ++j) oacc[td][j] = 0.0f;
  // Running row max of the raw scores, row sum of the weights. The scale comes
  // after the subtraction: the largest weight is exactly 1 however large the
  // scores are. Before any key the reference is the lowest finite value, so that
  // scores of -infinity alone leave a sum of 0.
  float mref = -__FLT_MAX__, lsum = 0.0f;
  const int vlane = (kh * 32 + 4 * hl + ((ln & 15) >> 2)) * L::VS + 16 * (ln >> 4) + 4 * (ln & 3);
  const int klane = (kh * 32 + ln) * L::KS + hl * 8;
  constexpr int NKK = D / 16;
  constexpr int NTD = D / 32;
  auto mfma = [](const bf16x8& a, const bf16x8& b, const f32x16& c) SW_INL {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  };
  auto kread = [&](const uint16_t* kp, int plane, int kk) SW_INL {
    return *reinterpret_cast<const bf16x8*>(kp + plane * L::K_PLANE + kk * 16);
  };
  auto vread = [&](const uint16_t* vp, int plane, int c, int td) SW_INL {
    const uint16_t* pp = vp + plane * L::V_PLANE + c * 16 * L::VS + td * 32;
    const i16x4 r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(pp));
    const i16x4 r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) i16x4*)(pp + 8 * L::VS));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(r0, r1, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto pb = [](const uint32_t (&q)[8], int c) SW_INL {
    return __builtin_bit_cast(bf16x8, make_uint4(q[4 * c], q[4 * c + 1], q[4 * c + 2], q[4 * c + 3]));
  };
  // leading and smaller products; the latter may overflow where the former did,
  // with the other sign
  auto join = [](float a, float b) SW_INL {
    return a + __builtin_amdgcn_fmed3f(b, -__FLT_MAX__, __FLT_MAX__);
  };
  // Scores of one step: S sums the products of the leading parts, T the five
  // smaller ones. With EXP, the weights of the scores cur (against mref) are
  // formed between the matrix instructions, two elements at a time.
  uint32_t ph[8], pm[8], pl[8];
  auto scores = [&](int sl, f32x16& S, f32x16& T, const f32x16& cur, float& ps, auto with_exp) SW_INL {
    constexpr bool EXP = decltype(with_exp)::value;
    constexpr int PPK = 8 / NKK;           // element pairs per 16 dims
    const uint16_t* kp = kslots + sl * 3 * L::K_PLANE + klane;
    bf16x8 kf[2][3];
#pragma unroll
    for (int q = 0; q < 3; ++q) kf[0][q] = kread(kp, q, 0);
#pragma unroll
    for (int j = 0; j < 16; ++j) S[j] = T[j] = 0.0f;
    float p0[PPK], p1[PPK];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      const bf16x8(&k)[3] = kf[kk & 1];
#pragma unroll
      for (int f = 0; f < 6; ++f) {
        if (f == 0) T = mfma(k[2], qf[0][kk], T);
        if (f == 1) S = mfma(k[0], qf[0][kk], S);
        if (f == 2) T = mfma(k[0], qf[2][kk], T);
        if (f == 3) T = mfma(k[1], qf[1][kk], T);
        if (f == 4) T = mfma(k[1], qf[0][kk], T);
        if (f == 5) T = mfma(k[0], qf[1][kk], T);
        if (kk + 1 < NKK && f < 3) kf[(kk + 1) & 1][f] = kread(kp, f, kk + 1);
        if (EXP) {
#pragma unroll
          for (int x = 0; x < PPK; ++x) {
            const int e = kk * PPK + x;
            if (f == 2 * x) {
              p0[x] = __builtin_amdgcn_exp2f((cur[2 * e] - mref) * sl2);
              p1[x] = __builtin_amdgcn_exp2f((cur[2 * e + 1] - mref) * sl2);
            }
            if (f == 2 * x + 1) ps += p0[x];
            if (f == 2 * x + 2) {
              ps += p1[x];
              split2<false>(p0[x], p1[x], ph[e], pm[e], pl[e]);
            }
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // O += V^T P of one step (small products first). With NEXT: the scores S + T of the next step and their row max.
  // With STAGE: the pieces of the tiles on their way to LDS.
  auto values = [&](int sl, f32x16& S, const f32x16& T, float& mx, int ksl, int vsl, auto with_next,
                    auto with_stage) SW_INL {
    constexpr bool NEXT = decltype(with_next)::value;
    constexpr bool STAGE = decltype(with_stage)::value;
    constexpr int N = 12 * NTD;            // matrix instructions
    constexpr int PUT = N / (2 * KP);      // of them per staged piece
    const uint16_t* vp = vslots + sl * 3 * L::V_PLANE + vlane;
    bf16x8 vf[2][6];
#pragma unroll
    for (int q = 0; q < 6; ++q) vf[0][q] = vread(vp, q >> 1, q & 1, 0);
    mx = -INFINITY;
#pragma unroll
    for (int td = 0; td < NTD; ++td) {
      const bf16x8(&v)[6] = vf[td & 1];    // h0 h1 m0 m1 l0 l1
      f32x16& t = oacc[td];
#pragma unroll
      for (int f = 0; f < 12; ++f) {
        const int c = f & 1;
        if (f < 2) t = mfma(v[4 + c], pb(ph, c), t);
        else if (f < 4) t = mfma(v[c], pb(pl, c), t);
        else if (f < 6) t = mfma(v[2 + c], pb(pm, c), t);
        else if (f < 8) t = mfma(v[2 + c], pb(ph, c), t);
        else if (f < 10) t = mfma(v[c], pb(pm, c), t);
        else t = mfma(v[c], pb(ph, c), t);
        const int n = td * 12 + f;
        if (td + 1 < NTD && f >= 2 && f < 8) vf[(td + 1) & 1][f - 2] = vread(vp, (f - 2) >> 1, (f - 2) & 1, td + 1);
        if (NEXT && td == 0 && f >= 4) {
          const int j = 2 * (f - 4);
          S[j] = join(S[j], T[j]);
          S[j + 1] = join(S[j + 1], T[j + 1]);
        }
        if (NEXT && td == NTD - 1 && f >= 8) {
          const int j = 4 * (f - 8);
          mx = fmaxf(fmaxf(mx, S[j]), fmaxf(S[j + 1], fmaxf(S[j + 2], S[j + 3])));
        }
        if (STAGE && n % PUT == PUT - 1) {
          const int q = n / PUT;
          if (q < KP) put_k(ksl, q);
          else put_v(vsl, q - KP);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (NEXT) mx = max_other_half(mx);
  };
  // the reference is the running row max; O moves only when a row's max grew
  auto raise = [&](float mx) SW_INL {
    if (__any(mx > mref)) {
      const float nref = fmaxf(mref, mx);
      const float alpha = __builtin_amdgcn_exp2f((mref - nref) * sl2);
      mref = nref;
      lsum *= alpha;
#pragma unroll
      for (int td = 0; td < NTD; ++td)
#pragma unroll
        for (int j = 0; j < 16; ++j) oacc[td][j] *= alpha;
    }
  };
  // causal + sequence-end mask of the diagonal sub-tile's scores, and their max
  auto mask = [&](int t, f32x16& S) SW_INL {
    const int k0 = step_k0(t) + kh * 32;
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int kp = k0 + (j >> 2) * 8 + hl * 4 + (j & 3);
      if (kp > qpos || kp >= seq1) S[j] = -INFINITY;
      mx = fmaxf(mx, S[j]);
    }
    return max_other_half(mx);
  };
  auto weights = [&](const f32x16& cur) SW_INL {
    float ps = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float p0 = __builtin_amdgcn_exp2f((cur[2 * e] - mref) * sl2);
      const float p1 = __builtin_amdgcn_exp2f((cur[2 * e + 1] - mref) * sl2);
      ps += p0;
      ps += p1;
      split2<false>(p0, p1, ph[e], pm[e], pl[e]);
    }
    lsum += ps;
  };
  auto first_scores = [&](int t, int sl, bool masked, f32x16& S) SW_INL {
    f32x16 T;
    float dummy = 0.0f;
    scores(sl, S, T, S, dummy, std::false_type{});
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      S[j] = join(S[j], T[j]);
      mx = fmaxf(mx, S[j]);
    }
    return masked ? mask(t, S) : max_other_half(mx);
  };

  // last step with keys for this wavefront's rows, and the masked one
  const bool dmine = active && sdiag;
  const int tend = (KH == 1) ? noffs - 1 + (dmine ? rgrp + 1 : 0)
                             : noffs - 1 + ((dmine && kh <= rgrp) ? 1 : 0);
  const int tmasked = (dmine && (KH == 1 || kh == rgrp)) ? tend : -1;
  const std::true_type yes{};
  const std::false_type no{};
  f32x16 S, Sn, Tn;
  float mx = -INFINITY;
  if (nsteps > 0 && L::SLOTS == 2) {
    // K runs a step ahead of V: step t reads K(t+1) and V(t), stores K(t+2) and
    // V(t+1) where K(t) and V(t-1) were, then loads K(t+3) and V(t+2).
    {
      uint4 k1[KP];
      const int a0 = step_k0(0), a1 = step_k0(1);
      load(Kg, a0, kr);
      load(Vg, a0, vr);
      if (nsteps > 1) load(Kg, a1, k1);
#pragma unroll
      for (int p = 0; p < KP; ++p) put_k(0, p);
#pragma unroll
      for (int p = 0; p < KP; ++p) put_v(0, p);
      if (nsteps > 1) {
        load(Vg, a1, vr);
#pragma unroll
        for (int p = 0; p < KP; ++p) kr[p] = k1[p];
#pragma unroll
        for (int p = 0; p < KP; ++p) put_k(1, p);
        if (nsteps > 2) load(Kg, step_k0(2), kr);
      }
    }
    __syncthreads();
    if (tend >= 0) mx = first_scores(0, 0, tmasked == 0, S);
    __syncthreads();
    int t = 0;
    for (; t + 1 < noffs; ++t) {
      const int sl = t & 1;
      raise(mx);
      float ps = 0.0f;
      scores(sl ^ 1, Sn, Tn, S, ps, yes);
      lsum += ps;
      values(sl, Sn, Tn, mx, sl, sl ^ 1, yes, yes);
      S = Sn;
      load(Kg, step_k0(t + 3), kr);
      load(Vg, step_k0(t + 2), vr);
      __syncthreads();
    }
    // the last steps: each wavefront goes on, ends or skips; tiles that no
    // later step reads are neither stored nor loaded
    for (; t < nsteps; ++t) {
      const int sl = t & 1;
      if (t <= tend) {
        raise(mx);
        weights(S);
        float mdummy;
        values(sl, S, S, mdummy, 0, 0, no, no);
        if (t < tend) mx = first_scores(t + 1, sl ^ 1, t + 1 == tmasked, S);
      }
      if (t + 1 >= nsteps) break;
      if (t + 2 < nsteps) {
#pragma unroll
        for (int p = 0; p < KP; ++p) put_k(sl, p);
        if (t + 3 < nsteps) load(Kg, step_k0(t + 3), kr);
      }
#pragma unroll
      for (int p = 0; p < KP; ++p) put_v(sl ^ 1, p);
      if (t + 2 < nsteps) load(Vg, step_k0(t + 2), vr);
      __syncthreads();
    }
    __syncthreads();                       // every wavefront is done with the slots
  } else if (nsteps > 0) {
    // one slot (D = 128 and key halves): the next tile is stored when every
    // wavefront is done. 16 heads over 16, B = 64, 8192 tokens, 20 %: 1223 -> 517 us
    // (fp32 instruction / this), one head 293 -> 115.
    load(Kg, step_k0(0), kr);
    load(Vg, step_k0(0), vr);
    for (int t = 0; t < nsteps; ++t) {
#pragma unroll
      for (int p = 0; p < KP; ++p) put_k(0, p);
#pragma unroll
      for (int p = 0; p < KP; ++p) put_v(0, p);
      load(Kg, step_k0(t + 1), kr);
      load(Vg, step_k0(t + 1), vr);
      __syncthreads();
      if (t <= tend) {
        raise(first_scores(t, 0, t == tmasked, S));
        weights(S);
        float mdummy;
        values(0, S, S, mdummy, 0, 0, no, no);
      }
      __syncthreads();
    }
  }

  // ---- epilogue ----
  float ltot = sum_other_half(lsum);
  if constexpr (KH == 2) {
    // join the two key halves of a row group (wavefronts 2r and 2r + 1)
    float* pm = reinterpret_cast<float*>(lds);                 // [4][32] references, then sums
    if (hl == 0) {
      pm[w * 32 + ln] = mref;
      pm[128 + w * 32 + ln] = ltot;
    }
    float* po = pm + 256 + (w >> 1) * 64 * 16 * (D / 32);
    static_assert((256 + 2 * 64 * 16 * (D / 32)) * 4 <= L::SLOTS * L::SLOT * 2, "partials must fit the slots");
    if (kh == 1) {
#pragma unroll
      for (int td = 0; td < D / 32; ++td)
#pragma unroll
        for (int j = 0; j < 16; ++j) po[(td * 16 + j) * 64 + l] = oacc[td][j];
    }
    __syncthreads();
    if (kh == 1) return;
    const float m1 = pm[(w + 1) * 32 + ln], l1 = pm[128 + (w + 1) * 32 + ln];
    const float mm = fmaxf(mref, m1);
    const float f0 = __builtin_amdgcn_exp2f((mref - mm) * sl2), f1 = __builtin_amdgcn_exp2f((m1 - mm) * sl2);
    ltot = ltot * f0 + l1 * f1;
    mref = mm;
#pragma unroll
    for (int td = 0; td < D / 32; ++td)
#pragma unroll
      for (int j = 0; j < 16; ++j) oacc[td][j] = oacc[td][j] * f0 + po[(td * 16 + j) * 64 + l] * f1;
  }
  if (!active || qpos >= seq1) return;
  const float inv = ltot > 0.0f ? 1.0f / ltot : 0.0f;
  float* orow = O + ((long long)u * N + qpos) * D;
#pragma unroll
  for (int td = 0; td < D / 32; ++td)
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      const int dv = td * 32 + jb * 8 + hl * 4;
      float4 st = make_float4(oacc[td][jb * 4 + 0] * inv, oacc[td][jb * 4 + 1] * inv,
                              oacc[td][jb * 4 + 2] * inv, oacc[td][jb * 4 + 3] * inv);
      *reinterpret_cast<float4*>(orow + dv) = st;
    }
  if (lse && hl == 0)
    lse[(long long)u * N + qpos] = (ltot > 0.0f) ? (mref * sl2 + log2f(ltot)) / kLog2e : -INFINITY;
}

#undef SW_INL

hipError_t launch_attn_prefill(int dtype, const void* Q, const void* K, const void* V, int h_q,
                               int h_kv, int d, long long N, const SeqMeta& meta, int64_t nb,
                               const int32_t* idx, const int32_t* cnt, int kmax, float scale,
                               void* O, float* lse, hipStream_t st) {
  const int G = h_q / h_kv;
  const int groups = (int)(nb * h_kv);
  const float sl2 = scale * kLog2e;
  if (dtype == SW_BF16) {
    // 32 query rows per wavefront
    const int tasks = G * (meta.B / 32);
    const int sg = (tasks + kPfWaves - 1) / kPfWaves;
    auto q = reinterpret_cast<const uint16_t*>(Q);
    auto k = reinterpret_cast<const uint16_t*>(K);
    auto v = reinterpret_cast<const uint16_t*>(V);
    auto o = reinterpret_cast<uint16_t*>(O);
    // Eight wavefronts share each K/V tile among twice the query rows, four
    // start and finish beside another workgroup. Measured (8000 tokens, 20 %;
    // eight / four): 32 query heads over 8, d = 128: B = 128 at 32768 tokens
    // 1641 / 1829 us, B = 64 121 / 126; d = 64: 84 / 79 and 81 / 74. Where the
    // eight have rows for seven at most, four are as fast (28 heads over 4,
    // B = 128: 937 / 929); with one query head per KV head (16 over 16) they
    // win by what the eight leave idle: B = 128 113 / 74 and, with two
    // wavefronts, B = 64 197 / 92 and, d = 64, 142 / 52. (One head over 8000
    // tokens, 125 workgroups: 44 / 39 and 33 / 32.)
    // Where the eight's workgroups do not fill the chip's 256 CUs once, the
    // shorter start and end of the four decide (32 heads over 8, B = 128: 1000
    // tokens 16.0 / 14.5, 2000 22.8 / 22.6, 3000 37.0 / 38.5; 8 over 2: 4000 tokens
    // 30.0 / 27.9, 8000 48.3 / 48.5).
    const bool four = d == 64 || tasks * 8 < sg * kPfWaves * 7 || groups * sg <= 240;
    // query heads of a group from head0 on
    auto launch4 = [&](int head0) {
      // one head and B = 64: rows for two wavefronts
      const int n = G - head0;
      const bool two = meta.B == 64 && n == 1;
      const int sg4 = two ? 1 : (n * (meta.B / 32) + 3) / 4;
      const unsigned grid = (unsigned)(((groups + 7) / 8) * 8 * sg4);
#define SW_LAUNCH_W4(DD, BB, WW)                                                                     \
  hipLaunchKernelGGL((attn_prefill_w4_kernel<DD, BB, WW>), dim3(grid), dim3(WW * 64), 0, st, q, k, v, \
                     h_q, h_kv, N, meta, idx, cnt, kmax, sl2, o, lse, groups, sg4, head0)
      if (two) {
        if (d == 128) SW_LAUNCH_W4(128, 64, 2);
        else SW_LAUNCH_W4(64, 64, 2);
      } else if (d == 128 && meta.B == 128) SW_LAUNCH_W4(128, 128, 4);
      else if (d == 128) SW_LAUNCH_W4(128, 64, 4);
      else if (meta.B == 128) SW_LAUNCH_W4(64, 128, 4);
      else SW_LAUNCH_W4(64, 64, 4);
#undef SW_LAUNCH_W4
    };
    if (four) {
      launch4(0);
      return hipGetLastError();
    }
    // Workgroups of eight; the heads of a last one that would be half empty go
    // to workgroups of four in a second launch, where there is work to outlast
    // its longest row: 28 heads over 4, B = 128, in one launch / two: 376
    // (block, KV head) groups 239 / 253 us, 512 419 / 411, 752 313 / 298, 1024
    // 1572 / 1459, 1564 3597 / 3311.
    const int full = tasks / kPfWaves, rest = tasks % kPfWaves;
    const bool both = rest >= 1 && rest <= kPfWaves / 2 && groups >= 640;
    const int sg8 = both ? full : sg;
    const int heads = both ? full * kPfWaves / (meta.B / 32) : G;
    const unsigned grid = (unsigned)(((groups + 7) / 8) * 8 * sg8);
#define SW_LAUNCH_BF16(BB)                                                                        \
  hipLaunchKernelGGL((attn_prefill_bf16_kernel<128, BB>), dim3(grid), dim3(kPfWaves * 64), 0, st, q, k, v, \
                     h_q, h_kv, N, meta, idx, cnt, kmax, sl2, o, lse, groups, sg8, heads)
    if (meta.B == 128) SW_LAUNCH_BF16(128);
    else SW_LAUNCH_BF16(64);
#undef SW_LAUNCH_BF16
    if (both) launch4(heads);
  } else {
    // one query head per KV head with blocks of 64: as in the bf16 kernel
    const bool halves = meta.B == 64 && G == 1;
    const int sg = halves ? 1 : (G * (meta.B / 32) + 3) / 4;
    const unsigned grid = (unsigned)(((groups + 7) / 8) * 8 * sg);
    auto q = reinterpret_cast<const float*>(Q);
    auto k = reinterpret_cast<const float*>(K);
    auto v = reinterpret_cast<const float*>(V);
    auto o = reinterpret_cast<float*>(O);
#define SW_LAUNCH_F32(DD, BB, KK)                                                                  \
  hipLaunchKernelGGL((attn_prefill_f32_kernel<DD, BB, KK>), dim3(grid), dim3(256), 0, st, q, k, v, \
                     h_q, h_kv, N, meta, idx, cnt, kmax, sl2, o, lse, groups, sg)
    if (halves) {
      if (d == 128) SW_LAUNCH_F32(128, 64, 2);
      else SW_LAUNCH_F32(64, 64, 2);
    } else if (d == 128 && meta.B == 128) SW_LAUNCH_F32(128, 128, 1);
    else if (d == 128) SW_LAUNCH_F32(128, 64, 1);
    else if (meta.B == 128) SW_LAUNCH_F32(64, 128, 1);
    else SW_LAUNCH_F32(64, 64, 1);
#undef SW_LAUNCH_F32
  }
  return hipGetLastError();
}

}  // namespace sw

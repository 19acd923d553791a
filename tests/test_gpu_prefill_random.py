"""Seeded random configurations of the block-sparse prefill attention against
the oracle (the kernel given a selection): ragged varlen batches with 1- to
1500-token sequences, GQA group sizes 1-8 (odd ones leave wavefronts of a
workgroup without rows), B in {64, 128}, d in {64, 128}, bf16 and fp32, and
selections that are random subsets with or without the diagonal block, the
diagonal alone, every block, or padded with entries the kernel must skip
(-1 and blocks after the row)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2602_07397_amd import binding as sw

pytestmark = pytest.mark.gpu

U = pytest.importorskip("_gpu_util")

N_CASES = 24


def _case(seed):
    rng = np.random.default_rng(1000 + seed)
    dtype = "f32" if seed % 6 == 5 else "bf16"
    B = int(rng.choice([64, 128]))
    d = int(rng.choice([64, 128]))
    h_kv = int(rng.choice([1, 2]))
    G = int(rng.choice([1, 2, 3, 4, 7, 8]))
    nseq = int(rng.integers(1, 5))
    seqlens = [int(rng.integers(1, 1500)) for _ in range(nseq)]
    mode = ["random", "random", "no_diag", "diag_only", "all", "padded"][seed % 6]
    return rng, dtype, B, d, h_kv, G, seqlens, mode


def _selection(rng, cu, B, mode):
    """(rows passed to the kernel, rows the oracle uses)."""
    given, used = [], []
    for a, e in zip(cu[:-1], cu[1:]):
        b = -(-(e - a) // B)
        for i in range(b):
            if mode == "diag_only":
                s = [i]
            elif mode == "all":
                s = list(range(i + 1))
            else:
                p = rng.uniform(0.1, 0.9)
                s = sorted({j for j in range(i) if rng.uniform() < p} | ({i} if mode != "no_diag" else set()))
            g = list(s)
            if mode == "padded":
                g = sorted(g + [-1] * int(rng.integers(0, 3)) + [i + 1 + int(x) for x in
                                                                  range(int(rng.integers(0, 3)))])
            given.append(g)
            used.append([j for j in s if 0 <= j <= i])
    return given, used


@pytest.mark.parametrize("seed", range(N_CASES))
def test_random_configuration_matches_oracle(seed):
    rng, dtype, B, d, h_kv, G, seqlens, mode = _case(seed)
    h_q = G * h_kv
    cu = [0] + list(np.cumsum(seqlens).astype(int))
    N = cu[-1]
    g = torch.Generator().manual_seed(seed)
    Q = torch.randn((h_q, N, d), generator=g)
    K = torch.randn((h_kv, N, d), generator=g)
    V = torch.randn((h_kv, N, d), generator=g)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    Q, K, V = Q.to(td), K.to(td), V.to(td)
    given, used = _selection(rng, cu, B, mode)
    kmax = max(1, max(len(s) for s in given))
    idx = np.full((len(given), kmax), -1, dtype=np.int32)
    cnt = np.zeros(len(given), dtype=np.int32)
    for r, s in enumerate(given):
        idx[r, :len(s)] = s
        cnt[r] = len(s)
    out = sw.sparse_attn_prefill(U.to_dev(Q), U.to_dev(K), U.to_dev(V), cu, B, U.to_dev(idx),
                                 U.to_dev(cnt), kmax)
    got = out.float().cpu().numpy()
    tol = U.ATOL_BF16 if dtype == "bf16" else U.ATOL_F32
    Qh, Kh, Vh = O.f64(Q), O.f64(K), O.f64(V)
    r = 0
    for s, (a, e) in enumerate(zip(cu[:-1], cu[1:])):
        b = -(-(e - a) // B)
        rows = used[r:r + b]
        ref = np.zeros((h_q, e - a, d))
        for u in range(h_q):
            for i in range(b):
                if rows[i]:
                    ref[u, i * B:min(e - a, (i + 1) * B)] = O.sparse_attention_block(
                        Qh[:, a:e], Kh[:, a:e], Vh[:, a:e], B, rows[i], u, i)
        # a row whose selection admits no key has no defined softmax: the
        # kernel writes zeros there (rows of a no-diagonal selection before any
        # selected key cannot occur, since every selected block precedes them)
        assert np.isfinite(got[:, a:e]).all(), (seed, s)
        assert U.max_abs(got[:, a:e], ref) <= tol, (seed, s, dtype, B, d, G, mode)
        r += b


def test_rows_selecting_every_block_at_max_blocks():
    """One sequence of SW_MAX_BLOCKS blocks (B = 64): the last rows select
    every block (the longest lists the kernel compacts in LDS), the others
    only their diagonal block."""
    B, d, h_q, h_kv = 64, 64, 2, 1
    b = sw.MAX_BLOCKS
    N = b * B
    g = torch.Generator().manual_seed(91)
    Q = torch.randn((h_q, N, d), generator=g).to(torch.bfloat16)
    K = torch.randn((h_kv, N, d), generator=g).to(torch.bfloat16)
    V = torch.randn((h_kv, N, d), generator=g).to(torch.bfloat16)
    full = {b - 1, b - 2, b - 5}
    sel = [list(range(i + 1)) if i in full else [i] for i in range(b)]
    kmax = b
    idx = np.full((b, kmax), -1, dtype=np.int32)
    cnt = np.array([len(s) for s in sel], dtype=np.int32)
    for r, s in enumerate(sel):
        idx[r, :len(s)] = s
    out = sw.sparse_attn_prefill(U.to_dev(Q), U.to_dev(K), U.to_dev(V), [0, N], B, U.to_dev(idx),
                                 U.to_dev(cnt), kmax)
    got = out.float().cpu().numpy()
    Qh, Kh, Vh = O.f64(Q), O.f64(K), O.f64(V)
    for i in sorted(full) + [0, 1, 1000]:
        for u in range(h_q):
            ref = O.sparse_attention_block(Qh, Kh, Vh, B, sel[i], u, i)
            assert U.max_abs(got[u, i * B:(i + 1) * B], ref) <= U.ATOL_BF16, (i, u)


@pytest.mark.parametrize("d,B,G,h_kv", [(128, 64, 1, 2), (64, 64, 1, 2), (128, 128, 1, 2),
                                        (128, 64, 2, 2), (128, 64, 3, 2), (128, 128, 3, 2),
                                        (64, 64, 2, 2), (64, 128, 3, 2), (128, 128, 2, 2),
                                        (128, 64, 4, 2), (128, 128, 2, 16), (128, 64, 4, 16),
                                        (128, 128, 4, 8)])
def test_head_counts_and_lengths_of_the_two_bf16_kernels(d, B, G, h_kv):
    """Both sides of the head-count and launch-size rules (the last three are
    the eight-wavefront kernel's; six of their heads are checked), rows of 1 to 9 selected blocks (every
    remainder of the unrolled steps), sequences ending on every 32-row group of
    a block, and keys that grow along the sequence, so that the exponent
    reference moves and the two key halves of a row end with different ones.
    lse against the float64 log-sum-exp: the kernel sums the weights it applies,
    each rounded to bf16 (8 significant bits, unit roundoff 2^-8), so the sum is
    within 2^-8 of the exact one (relative; one large weight does not average
    it out) and its logarithm within -log(1 - 2^-8) < 3.92e-3; the logits
    (|x| <= 40, fp32 sums of d exact products) and the exponential add less
    than 4e-5."""
    rng = np.random.default_rng(700 + d + B + G)
    seqlens = [B * 9, B * 3 + 1, B + 33, B * 2 + B // 2 + 7, 5]
    cu = [0] + list(np.cumsum(seqlens).astype(int))
    N = cu[-1]
    h_q = G * h_kv
    heads = range(h_q) if h_kv == 2 else sorted(rng.choice(h_q, size=6, replace=False).tolist())
    g = torch.Generator().manual_seed(31)
    Q = torch.randn((h_q, N, d), generator=g)
    K = torch.randn((h_kv, N, d), generator=g)
    V = torch.randn((h_kv, N, d), generator=g)
    for a, e in zip(cu[:-1], cu[1:]):
        K[:, a:e] *= torch.linspace(0.5, 3.0, e - a)[None, :, None]
    Q, K, V = (x.to(torch.bfloat16) for x in (Q, K, V))
    rows = []
    for a, e in zip(cu[:-1], cu[1:]):
        for i in range(-(-(e - a) // B)):
            keep = [j for j in range(i) if rng.uniform() < 0.7]
            rows.append(keep + [i] if rng.uniform() < 0.8 or not keep else keep)
    kmax = max(len(r) for r in rows)
    idx = np.full((len(rows), kmax), -1, dtype=np.int32)
    for r, s in enumerate(rows):
        idx[r, :len(s)] = s
    cnt = np.array([len(s) for s in rows], dtype=np.int32)
    out, lse = sw.sparse_attn_prefill(U.to_dev(Q), U.to_dev(K), U.to_dev(V), cu, B, U.to_dev(idx),
                                      U.to_dev(cnt), kmax, want_lse=True)
    got, glse = out.float().cpu().numpy(), lse.cpu().numpy()
    Qh, Kh, Vh = O.f64(Q), O.f64(K), O.f64(V)
    r = 0
    for a, e in zip(cu[:-1], cu[1:]):
        for i in range(-(-(e - a) // B)):
            lo, hi = a + i * B, min(e, a + (i + 1) * B)
            tok = np.concatenate([np.arange(a + j * B, min(e, a + (j + 1) * B)) for j in rows[r]])
            for u in heads:
                ref = O.sparse_attention_block(Qh[:, a:e], Kh[:, a:e], Vh[:, a:e], B, rows[r], u, i)
                assert U.max_abs(got[u, lo:hi], ref) <= U.ATOL_BF16, (r, u)
                z = Qh[u, lo:hi] @ Kh[u // G, tok].T / np.sqrt(d)
                z[tok[None, :] > np.arange(lo, hi)[:, None]] = -np.inf
                m = z.max(axis=1)
                want = m + np.log(np.exp(z - m[:, None]).sum(axis=1))
                assert np.abs(glse[u, lo:hi] - want).max() <= 3.96e-3, (r, u)
            r += 1


@pytest.mark.parametrize("d,B,G", [(64, 64, 1), (128, 64, 1), (64, 128, 1), (128, 128, 2),
                                   (128, 64, 3), (64, 64, 2)])
def test_fp32_attention_is_fp32_accurate(d, B, G):
    """The fp32 kernel against float64 over operands of mixed magnitude (rows
    scaled by 2^-12 .. 2^12, values by 2^-20 .. 2^20 per dimension), rows of 1
    to 6 selected blocks, ragged ends. Bound per output: the logits are sums of
    d products, each within 2^-23 of the exact one, accumulated in fp32
    ((d + 2) 2^-23 sum |q_i k_i| scale at worst); the exponential adds 2^-22 of
    the logit in log2 units; an output is a mean of the values under weights
    with that relative error, accumulated over at most 6 B keys with sums of 16
    (6 B / 16 roundings)."""
    rng = np.random.default_rng(900 + d + B + G)
    seqlens = [B * 6, B * 2 + 31, B + 1, 3]
    cu = [0] + list(np.cumsum(seqlens).astype(int))
    h_kv, N = 2, cu[-1]
    h_q = G * h_kv
    g = torch.Generator().manual_seed(33)
    e2 = torch.randint(-12, 13, (h_kv, N, 1), generator=g).float()
    Q = torch.randn((h_q, N, d), generator=g)
    K = torch.randn((h_kv, N, d), generator=g) * torch.exp2(torch.minimum(e2, torch.tensor(0.0)))
    Q[:, ::3] *= 2.0 ** -12
    V = torch.randn((h_kv, N, d), generator=g) * torch.exp2(torch.randint(-20, 21, (d,), generator=g).float())
    rows = []
    for a, e in zip(cu[:-1], cu[1:]):
        for i in range(-(-(e - a) // B)):
            rows.append([j for j in range(i) if rng.uniform() < 0.7] + [i])
    kmax = max(len(r) for r in rows)
    idx = np.full((len(rows), kmax), -1, dtype=np.int32)
    for r, s in enumerate(rows):
        idx[r, :len(s)] = s
    cnt = np.array([len(s) for s in rows], dtype=np.int32)
    out = sw.sparse_attn_prefill(U.to_dev(Q), U.to_dev(K), U.to_dev(V), cu, B, U.to_dev(idx),
                                 U.to_dev(cnt), kmax).cpu().numpy()
    Qh, Kh, Vh = O.f64(Q), O.f64(K), O.f64(V)
    worst = 0.0
    r = 0
    for a, e in zip(cu[:-1], cu[1:]):
        for i in range(-(-(e - a) // B)):
            lo, hi = a + i * B, min(e, a + (i + 1) * B)
            tok = np.concatenate([np.arange(a + j * B, min(e, a + (j + 1) * B)) for j in rows[r]])
            for u in range(h_q):
                q, k = Qh[u, lo:hi], Kh[u // G, tok]
                ref = O.sparse_attention_block(Qh[:, a:e], Kh[:, a:e], Vh[:, a:e], B, rows[r], u, i)
                mag = (np.abs(q) @ np.abs(k).T).max(axis=1) / np.sqrt(d)       # per row
                rel = (d + 2) * 2.0 ** -23 * mag + 2.0 ** -22 * (mag + 1)
                rel = 2 * np.expm1(rel) + (6 * B / 16 + 8) * 2.0 ** -23
                bound = rel[:, None] * np.abs(Vh[u // G, tok]).max(axis=0)[None, :]
                err = np.abs(out[u, lo:hi] - ref)
                worst = max(worst, float((err / bound).max()))
            r += 1
    print(f"largest error over its bound: {worst:.3f}", flush=True)
    assert worst <= 1.0


@pytest.mark.parametrize("G,B,h_kv,blocks", [(7, 128, 4, [159, 1]), (7, 128, 4, [158, 1]),
                                             (9, 64, 8, [50, 30])])
def test_heads_divided_between_the_two_bf16_kernels(G, B, h_kv, blocks):
    """640 (block, KV head) groups and just below: the heads that would half
    fill a workgroup of eight wavefronts go to a second launch. Rows of up to
    four blocks; every head of sampled rows against the oracle."""
    d, h_q = 128, G * h_kv
    rng = np.random.default_rng(G + B)
    seqlens = [b * B - 5 for b in blocks]
    cu = [0] + list(np.cumsum(seqlens).astype(int))
    N = cu[-1]
    g = torch.Generator().manual_seed(77)
    Q, K, V = (torch.randn((h, N, d), generator=g).to(torch.bfloat16) for h in (h_q, h_kv, h_kv))
    rows = [sorted(set(rng.integers(0, i + 1, size=3).tolist()) | {i}) for b in blocks for i in range(b)]
    idx = np.full((len(rows), 4), -1, dtype=np.int32)
    for r, s in enumerate(rows):
        idx[r, :len(s)] = s
    cnt = np.array([len(s) for s in rows], dtype=np.int32)
    got = sw.sparse_attn_prefill(U.to_dev(Q), U.to_dev(K), U.to_dev(V), cu, B, U.to_dev(idx),
                                 U.to_dev(cnt), 4).float().cpu().numpy()
    r0 = 0
    for b, a, e in zip(blocks, cu[:-1], cu[1:]):
        Qh, Kh, Vh = O.f64(Q[:, a:e]), O.f64(K[:, a:e]), O.f64(V[:, a:e])
        for i in sorted({0, b // 2, b - 1}):
            for u in range(h_q):
                ref = O.sparse_attention_block(Qh, Kh, Vh, B, rows[r0 + i], u, i)
                lo, hi = a + i * B, min(e, a + (i + 1) * B)
                assert U.max_abs(got[u, lo:hi], ref) <= U.ATOL_BF16, (b, i, u)
        r0 += b
    assert np.isfinite(got).all()


def _selected_rows(rng, b, kmax):
    """A selection of up to kmax blocks per row, the own block among them."""
    idx = np.full((b, kmax), -1, dtype=np.int32)
    cnt = np.zeros(b, dtype=np.int32)
    for i in range(b):
        s = sorted(set(rng.integers(0, i + 1, size=min(i, kmax - 1)).tolist()) | {i})
        idx[i, :len(s)] = s
        cnt[i] = len(s)
    return idx, cnt


@pytest.mark.parametrize("d,B,n", [(64, 64, 2000), (128, 64, 2000), (128, 64, 5000), (64, 128, 2000),
                                   (128, 128, 5000)])
def test_a_bf16_head_has_the_same_bits_in_every_kernel(d, B, n):
    """A query head's attention is bit-identical whatever the number of heads,
    the launch size and kmax make of the call: alone (workgroups of two or four
    wavefronts), in groups of 2, 3, 4 and 8 (four, or eight at d = 128 where the
    launch fills the chip), and with the list padded beyond 3040 entries. Keys
    that grow along the sequence move the exponent references, so another order
    or another reference would show."""
    rng = np.random.default_rng(d + B + n)
    b = -(-n // B)
    idx, cnt = _selected_rows(rng, b, 9)
    g = torch.Generator().manual_seed(n)
    Q = torch.randn((8, n, d), generator=g).to(torch.bfloat16)
    V = torch.randn((1, n, d), generator=g).to(torch.bfloat16)
    K = (torch.randn((1, n, d), generator=g) * torch.linspace(0.5, 3.0, n)[None, :, None]).to(torch.bfloat16)
    dQ, dK, dV, dc = U.to_dev(Q), U.to_dev(K), U.to_dev(V), U.to_dev(cnt)

    def call(heads, h_kv=1, kmax=9):
        wide = np.full((b, kmax), -1, dtype=np.int32)
        wide[:, :9] = idx
        q = dQ[:heads].repeat(h_kv, 1, 1).contiguous()
        return sw.sparse_attn_prefill(q, dK.repeat(h_kv, 1, 1).contiguous(), dV.repeat(h_kv, 1, 1).contiguous(),
                                      [0, n], B, U.to_dev(wide), dc, kmax, want_lse=True)

    O1, l1 = call(8, h_kv=32)                   # 256 or more workgroups: eight wavefronts at d = 128
    for heads, h_kv, kmax in ((1, 1, 9), (2, 1, 9), (3, 1, 9), (4, 1, 9), (8, 1, 9), (1, 32, 9),
                              (1, 1, 3040), (1, 1, 3041), (1, 1, 4096)):
        out, lse = call(heads, h_kv, kmax)
        for u in range(heads * h_kv):
            assert torch.equal(out[u], O1[u % heads]), (heads, h_kv, kmax, u)
            assert torch.equal(lse[u], l1[u % heads]), (heads, h_kv, kmax, u)


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
def test_long_lists_of_one_query_head(dtype, d):
    """Rows of exactly 3040, 3041 and 4096 selected blocks (SW_MAX_BLOCKS) with
    one query head and blocks of 64."""
    B, b = 64, sw.MAX_BLOCKS
    N = b * B
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(92)
    Q, K, V = (torch.randn((1, N, d), generator=g).to(td) for _ in range(3))
    full = {3039: 3040, 3040: 3041, 3500: 3041, b - 2: 3040, b - 1: b}
    sel = [list(range(full[i] - 1)) + [i] if i in full else [i] for i in range(b)]
    idx = np.full((b, b), -1, dtype=np.int32)
    cnt = np.array([len(s) for s in sel], dtype=np.int32)
    for r, s in enumerate(sel):
        idx[r, :len(s)] = s
    got = sw.sparse_attn_prefill(U.to_dev(Q), U.to_dev(K), U.to_dev(V), [0, N], B, U.to_dev(idx),
                                 U.to_dev(cnt), b).float().cpu().numpy()
    tol = U.ATOL_BF16 if dtype == "bf16" else U.ATOL_F32
    Qh, Kh, Vh = O.f64(Q), O.f64(K), O.f64(V)
    for i in sorted(full) + [0, 1, 2000]:
        ref = O.sparse_attention_block(Qh, Kh, Vh, B, sel[i], 0, i)
        assert U.max_abs(got[0, i * B:(i + 1) * B], ref) <= tol, i


@pytest.mark.parametrize("d,B,G", [(64, 64, 1), (128, 64, 1), (64, 128, 1), (128, 128, 2), (128, 64, 3)])
def test_fp32_attention_with_extreme_values(d, B, G):
    """Finite inputs at the ends of the range, one KV head each. 0: the largest
    value a float holds in V, where rows see it and where it is masked. 1: in K,
    with scores that overflow to -infinity (300 times it): weight 0. 2 and 3:
    scores of -1e33 and 1e12, far apart: all the weight is on the largest
    (the output is its value, exactly). 4: every score -infinity: the output is 0."""
    n, h_kv = 3 * B + 5, 5
    big = float(np.finfo(np.float32).max)
    g = torch.Generator().manual_seed(12)
    Q = torch.randn((h_kv, 1, n, d), generator=g).repeat(1, G, 1, 1)
    K, V = (torch.randn((h_kv, n, d), generator=g) for _ in range(2))
    V[0, :, 1:3] = 0.0
    V[0, 3, 1], V[0, n - 3, 2] = big, -big
    Q[1, :, :, 0] = 300.0
    K[1, :, 0] = 0.0
    K[1, 7, 0], K[1, B + 9, 0], K[1, 2 * B, 0] = -big, -big, -0.5 * big
    lev = torch.randperm(n, generator=g).float()
    Q[2], Q[3] = 1e30, 1e10
    K[2] = (-(lev + 10) * (100.0 / d))[:, None]
    K[3] = ((lev - n // 2) * (2.0 / d))[:, None]
    Q[4, :, :, 0] = 300.0
    K[4, :, 0] = -big
    Q = Q.reshape(h_kv * G, n, d)
    b = -(-n // B)
    sel = [list(range(i + 1)) for i in range(b)]
    idx = np.full((b, b), -1, dtype=np.int32)
    for i in range(b):
        idx[i, :i + 1] = sel[i]
    out, lse = sw.sparse_attn_prefill(U.to_dev(Q), U.to_dev(K), U.to_dev(V), [0, n], B, U.to_dev(idx),
                                      U.to_dev(np.arange(1, b + 1, dtype=np.int32)), b, want_lse=True)
    got, glse = out.cpu().numpy(), lse.cpu().numpy()
    Qh, Kh, Vh = O.f64(Q), O.f64(K), O.f64(V)
    seen = np.tril(np.ones((n, n), dtype=bool))
    for kv in range(h_kv):
        for u in range(kv * G, (kv + 1) * G):
            z = np.where(seen, Qh[u] @ Kh[kv].T / np.sqrt(d), -np.inf)
            if kv == 4:
                assert (got[u] == 0.0).all() and np.isneginf(glse[u]).all()
            elif kv in (2, 3):
                assert (got[u] == V[kv].numpy()[z.argmax(axis=1)]).all(), kv
            else:
                w = np.exp(z - z.max(axis=1, keepdims=True))
                want = (w / w.sum(axis=1, keepdims=True)) @ Vh[kv]
                assert np.isfinite(got[u]).all(), kv
                assert (np.abs(got[u] - want) <= U.ATOL_F32 * np.maximum(np.abs(want), 1.0)).all(), kv
                assert U.max_abs(glse[u], z.max(axis=1) + np.log(w.sum(axis=1))) <= U.ATOL_F32, kv


@pytest.mark.parametrize("d,B", [(64, 64), (128, 128)])
@pytest.mark.parametrize("e", [-90, -110, -118])
def test_fp32_attention_of_small_operands(d, B, e):
    """Values (and keys, with queries as much larger) scaled by 2^e. From 2^-110
    on operands keep their 24 bits: the relative error of ordinary ones. Below,
    each counts with an error of up to 2^-134, which at 2^-118 is 2^-16 of a value
    of 1 (2-norm: a third of that for evenly spread roundings, and less where
    many values are averaged)."""
    n = 4 * B
    g = torch.Generator().manual_seed(13)
    Q, K, V = (torch.randn((1, n, d), generator=g) for _ in range(3))
    s = 2.0 ** e
    b = n // B
    idx = np.full((b, b), -1, dtype=np.int32)
    for i in range(b):
        idx[i, :i + 1] = range(i + 1)
    seen = np.tril(np.ones((n, n), dtype=bool))
    for q, k, v in ((Q, K, V * s), (Q / s, K * s, V), (Q * s, K / s, V)):
        got = sw.sparse_attn_prefill(U.to_dev(q), U.to_dev(k), U.to_dev(v), [0, n], B, U.to_dev(idx),
                                     U.to_dev(np.arange(1, b + 1, dtype=np.int32)), b).cpu().numpy()
        z = np.where(seen, O.f64(q[0]) @ O.f64(k[0]).T / np.sqrt(d), -np.inf)
        w = np.exp(z - z.max(axis=1, keepdims=True))
        want = (w / w.sum(axis=1, keepdims=True)) @ O.f64(v[0])
        err = np.linalg.norm(got[0] - want) / np.linalg.norm(want)
        assert err <= (8e-7 if e >= -110 else 2.0 ** -16), (e, err)

"""Seeded random configurations of the split-K decode attention against the
oracle (the kernel given a selection): batches of 1-20 sequences at random
positions (including inactive ones: negative or past the cache, which get
zeros), GQA groups 1-8, d in {64, 128}, blocks of 16-128 tokens, bf16 and
fp32, selections that are random subsets of the blocks up to the current one
(with or without it), padded with entries the kernel must skip."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2602_07397_amd import binding as sw

pytestmark = pytest.mark.gpu

U = pytest.importorskip("_gpu_util")

N_CASES = 16


@pytest.mark.parametrize("seed", range(N_CASES))
def test_random_decode_attention_matches_oracle(seed):
    rng = np.random.default_rng(2000 + seed)
    dtype = "f32" if seed % 4 == 3 else "bf16"
    G = int(rng.choice([1, 2, 4, 8]))
    h_kv = int(rng.choice([1, 2, 8]))
    h_q = G * h_kv
    d = int(rng.choice([64, 128]))
    B = int(rng.choice([16, 64, 128]))
    batch = int(rng.integers(1, 21))
    T_max = int(rng.integers(1, 5000))
    pos = []
    for _ in range(batch):
        u = rng.uniform()
        pos.append(-1 if u < 0.08 else (T_max + 3 if u < 0.12 else int(rng.integers(0, T_max))))
    g = torch.Generator().manual_seed(seed)
    q = torch.randn((batch, h_q, d), generator=g)
    Kc = torch.randn((batch, h_kv, T_max, d), generator=g)
    Vc = torch.randn((batch, h_kv, T_max, d), generator=g)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, Kc, Vc = q.to(td), Kc.to(td), Vc.to(td)
    given, used = [], []
    for p in pos:
        if p < 0 or p >= T_max:
            given.append([0])
            used.append([])
            continue
        bc = p // B
        keep_cur = rng.uniform() < 0.8
        s = sorted({j for j in range(bc) if rng.uniform() < rng.uniform(0.1, 0.9)} |
                   ({bc} if keep_cur or bc == 0 else set()))
        if not s:
            s = [bc]
        gsel = list(s)
        if seed % 3 == 0:
            gsel = sorted(gsel + [-1] + [bc + 1 + k for k in range(int(rng.integers(0, 3)))])
        given.append(gsel)
        used.append(s)
    kmax = max(len(s) for s in given)
    idx = np.full((batch, kmax), -1, dtype=np.int32)
    cnt = np.zeros(batch, dtype=np.int32)
    for b, s in enumerate(given):
        idx[b, :len(s)] = s
        cnt[b] = len(s)
    out = sw.sparse_attn_decode(U.to_dev(q), U.to_dev(Kc), U.to_dev(Vc), B,
                                U.to_dev(np.array(pos, dtype=np.int32)), U.to_dev(idx),
                                U.to_dev(cnt), kmax)
    got = out.float().cpu().numpy()
    tol = U.ATOL_BF16 if dtype == "bf16" else U.ATOL_F32
    qh, Kh, Vh = O.f64(q), O.f64(Kc), O.f64(Vc)
    assert np.isfinite(got).all()
    for b, p in enumerate(pos):
        if not used[b]:
            assert np.all(got[b] == 0.0), (seed, b, p)
            continue
        ref = O.decode_attention(qh[b], Kh[b], Vh[b], used[b], p, B)
        assert U.max_abs(got[b], ref) <= tol, (seed, b, p, dtype, G, h_kv, d, B)


def test_decode_attention_with_every_block_selected_at_max_blocks():
    """B = 16 with a 65536-token cache: 4096 blocks, every block up to the
    current one selected (the longest lists the kernel stages)."""
    rng = np.random.default_rng(3000)
    batch, h_kv, G, d, B, T_max = 2, 2, 4, 128, 16, 65536
    h_q = G * h_kv
    pos = [T_max - 1, int(rng.integers(40000, T_max - 1))]
    g = torch.Generator().manual_seed(77)
    q = torch.randn((batch, h_q, d), generator=g).to(torch.bfloat16)
    Kc = torch.randn((batch, h_kv, T_max, d), generator=g).to(torch.bfloat16)
    Vc = torch.randn((batch, h_kv, T_max, d), generator=g).to(torch.bfloat16)
    sels = [list(range(p // B + 1)) for p in pos]
    kmax = max(len(s) for s in sels)
    idx = np.full((batch, kmax), -1, dtype=np.int32)
    cnt = np.array([len(s) for s in sels], dtype=np.int32)
    for b, s in enumerate(sels):
        idx[b, :len(s)] = s
    out = sw.sparse_attn_decode(U.to_dev(q), U.to_dev(Kc), U.to_dev(Vc), B,
                                U.to_dev(np.array(pos, dtype=np.int32)), U.to_dev(idx),
                                U.to_dev(cnt), kmax)
    got = out.float().cpu().numpy()
    for b, p in enumerate(pos):
        ref = O.decode_attention(O.f64(q[b]), O.f64(Kc[b]), O.f64(Vc[b]), sels[b], p, B)
        assert U.max_abs(got[b], ref) <= U.ATOL_BF16, (b, p)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_decode_attention_large_logits_and_identical_keys(dtype):
    """Logits of several hundred (far past the fp32 exp range without a
    running max) and, in the second sequence, identical keys (uniform
    weights: the output is the mean of the selected values up to p)."""
    batch, h_kv, G, d, B, T_max = 2, 1, 4, 128, 64, 3000
    h_q = G * h_kv
    g = torch.Generator().manual_seed(5)
    q = torch.randn((batch, h_q, d), generator=g) * 12.0
    Kc = torch.randn((batch, h_kv, T_max, d), generator=g) * 12.0
    Vc = torch.randn((batch, h_kv, T_max, d), generator=g)
    Kc[1] = 0.25
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, Kc, Vc = q.to(td), Kc.to(td), Vc.to(td)
    pos = [2999, 1500]
    sels = [[0, 5, 17, 30, 46], [0, 3, 10, 23]]
    kmax = 5
    idx = np.full((batch, kmax), -1, dtype=np.int32)
    cnt = np.array([len(s) for s in sels], dtype=np.int32)
    for b, s in enumerate(sels):
        idx[b, :len(s)] = s
    out = sw.sparse_attn_decode(U.to_dev(q), U.to_dev(Kc), U.to_dev(Vc), B,
                                U.to_dev(np.array(pos, dtype=np.int32)), U.to_dev(idx),
                                U.to_dev(cnt), kmax)
    got = out.float().cpu().numpy()
    assert np.isfinite(got).all()
    qh, Kh, Vh = O.f64(q), O.f64(Kc), O.f64(Vc)
    ref0 = O.decode_attention(qh[0], Kh[0], Vh[0], sels[0], pos[0], B)
    # fp32: the logits reach several hundred, but the split-K kernel keeps the
    # error (observed 3.6e-6) within the general fp32 tolerance
    tol0 = U.ATOL_BF16 if dtype == "bf16" else U.ATOL_F32
    err0 = U.max_abs(got[0], ref0)
    print(f"\n[numerics] decode large logits {dtype}: max-abs {err0:.2e}, tolerance {tol0:.2e}")
    assert err0 <= tol0
    toks = np.concatenate([np.arange(j * B, min(pos[1] + 1, (j + 1) * B)) for j in sels[1]])
    mean = Vh[1, 0, toks].mean(axis=0)
    for u in range(h_q):
        assert U.max_abs(got[1, u], mean) <= (U.ATOL_BF16 if dtype == "bf16" else U.ATOL_F32)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_fp32_decode_attention_at_group_edges(d, G):
    """fp32 decode attention where groups and splits begin and end: positions
    on the first and last token of a 16-token group and of a block, selections
    of 1 to 33 groups over up to 32 splits (most of them empty), values of
    mixed magnitude per dimension. Bound per output as for an fp32 dot product
    added as a tree: logits within (log2(d) + 6) 2^-24 sum |q_i k_i| scale, the
    exponential 2^-22 of the logit, 40 roundings of the sums."""
    B = 16
    pos = [0, 15, 16, 31, 500, 527]
    sels = [[0], [0], [0, 1], [1], list(range(0, 32, 2)), list(range(33))]
    batch, h_kv, T_max = len(pos), 2, 528
    h_q = G * h_kv
    g = torch.Generator().manual_seed(50 + G)
    q = torch.randn((batch, h_q, d), generator=g) * 3.0
    Kc = torch.randn((batch, h_kv, T_max, d), generator=g)
    Vc = torch.randn((batch, h_kv, T_max, d), generator=g)
    Vc *= torch.exp2(torch.randint(-20, 21, (d,), generator=g).float())
    kmax = 33
    idx = np.full((batch, kmax), -1, dtype=np.int32)
    cnt = np.array([len(s) for s in sels], dtype=np.int32)
    for b, s in enumerate(sels):
        idx[b, :len(s)] = s
    got = sw.sparse_attn_decode(U.to_dev(q), U.to_dev(Kc), U.to_dev(Vc), B,
                                U.to_dev(np.array(pos, dtype=np.int32)), U.to_dev(idx),
                                U.to_dev(cnt), kmax).cpu().numpy()
    qh, Kh, Vh = O.f64(q), O.f64(Kc), O.f64(Vc)
    worst = 0.0
    for b in range(batch):
        ref = O.decode_attention(qh[b], Kh[b], Vh[b], sels[b], pos[b], B)
        tok = np.concatenate([np.arange(j * B, (j + 1) * B) for j in sels[b]])
        tok = tok[tok <= pos[b]]
        for u in range(h_q):
            mag = (np.abs(Kh[b, u // G, tok]) @ np.abs(qh[b, u])).max() / np.sqrt(d)
            rel = 2 * np.expm1((np.log2(d) + 6) * 2.0 ** -24 * mag + 2.0 ** -22 * (mag + 1)) + 40 * 2.0 ** -24
            bound = rel * np.abs(Vh[b, u // G, tok]).max(axis=0)
            worst = max(worst, float((np.abs(got[b, u] - ref[u]) / bound).max()))
    print(f"largest error over its bound: {worst:.3f}", flush=True)
    assert worst <= 1.0


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_decode_attention_with_extreme_logits(d):
    """Finite inputs at the ends of the range. Sequence 0: the logits of its
    first 40 tokens overflow to -infinity (whole 16-token groups of them before
    and after the first key that counts), so those keys have weight 0. Sequence
    1: all of them do, the output is 0. Sequences 2 and 3: logits of 1e12 and
    -1e33, far apart: all the weight is on the largest (values equal to its
    value, exactly). Sequence 4: the largest value a float holds, in K (weight
    0) and V."""
    B, T_max, batch, h_kv, G = 16, 96, 5, 1, 2
    big = float(np.finfo(np.float32).max)
    g = torch.Generator().manual_seed(8)
    q = torch.full((batch, G, d), 2e19)
    K = torch.randn((batch, h_kv, T_max, d), generator=g) * 5e-21
    V = torch.randn((batch, h_kv, T_max, d), generator=g)
    K[0, :, :40] = -2e19
    K[0, :, 64:] = -2e19
    K[1] = -2e19
    lev = torch.randperm(T_max, generator=g).float()
    q[2], q[3] = 1e10, 1e30
    K[2, 0] = ((lev - 48) * (2.0 / d))[:, None]
    K[3, 0] = (-(lev + 10) * (100.0 / d))[:, None]
    q[4] = 1.0
    K[4] = 0.0
    K[4, 0, 3, 0] = -big
    V[4, 0, :, 1] = 0.0
    V[4, 0, 50, 1] = big
    idx = np.arange(T_max // B, dtype=np.int32)[None, :].repeat(batch, 0)
    cnt = np.full(batch, T_max // B, dtype=np.int32)
    pos = np.full(batch, T_max - 1, dtype=np.int32)
    got = sw.sparse_attn_decode(U.to_dev(q), U.to_dev(K), U.to_dev(V), B, U.to_dev(pos),
                                U.to_dev(idx), U.to_dev(cnt), T_max // B).cpu().numpy()
    qh, Kh, Vh = O.f64(q), O.f64(K), O.f64(V)
    for u in range(G):
        z = Kh[0, 0, 40:64] @ qh[0, u] / np.sqrt(d)
        w = np.exp(z - z.max())
        assert U.max_abs(got[0, u], (w / w.sum()) @ Vh[0, 0, 40:64]) <= U.ATOL_F32
        assert (got[1, u] == 0.0).all()
        for b in (2, 3):
            top = int(np.argmax(Kh[b, 0] @ qh[b, u]))
            assert (got[b, u] == V[b, 0, top].numpy()).all(), b
        w = np.exp(Kh[4, 0] @ qh[4, u] / np.sqrt(d))
        want = (w / w.sum()) @ Vh[4, 0]
        assert np.isfinite(got[4, u]).all()
        assert (np.abs(got[4, u] - want) <= U.ATOL_F32 * np.maximum(np.abs(want), 1.0)).all()


@pytest.mark.parametrize("batch,n", [(1, 4097), (1, 9000), (600, 4096), (600, 4097), (600, 9000)])
def test_fp32_decode_attention_over_long_lists(batch, n):
    """More list entries than SW_MAX_BLOCKS (a selection of the caller's own):
    split 32 ways (batch 1) and in one piece (batch 600). The first 4096 entries
    run through two blocks, the others through two more; keys that are listed r
    times count r times. A wavefront adds the sums of its n / 4 groups one after
    the other, and the weights' likewise: 2 n / 4 roundings of 2^-24."""
    B, d, T_max = 16, 64, 64
    g = torch.Generator().manual_seed(n)
    q = torch.randn((batch, 1, d), generator=g)
    K, V = (torch.randn((batch, 1, T_max, d), generator=g) for _ in range(2))
    lst = np.arange(n, dtype=np.int32) % 2 + np.where(np.arange(n) < 4096, 0, 2).astype(np.int32)
    got = sw.sparse_attn_decode(U.to_dev(q), U.to_dev(K), U.to_dev(V), B,
                                U.to_dev(np.full(batch, T_max - 3, dtype=np.int32)),
                                U.to_dev(np.tile(lst, (batch, 1))),
                                U.to_dev(np.full(batch, n, dtype=np.int32)), n).cpu().numpy()
    mult = np.bincount(lst, minlength=4).repeat(B)[:T_max - 2]
    for b in {0, batch // 2, batch - 1}:
        z = O.f64(K)[b, 0, :T_max - 2] @ O.f64(q)[b, 0] / np.sqrt(d)
        w = mult * np.exp(z - z.max())
        want = (w / w.sum()) @ O.f64(V)[b, 0, :T_max - 2]
        tol = U.ATOL_F32 + 2 * (n / 4) * 2.0 ** -24 * float(V[b].abs().max())
        assert U.max_abs(got[b, 0], want) <= tol, b


def test_fp32_decode_attention_of_distant_blocks():
    """Block numbers past 32767 (attention over a cache of 640000 tokens)."""
    B, d, T_max = 16, 64, 640000
    g = torch.Generator().manual_seed(3)
    q = torch.randn((1, 2, d), generator=g)
    K, V = (torch.randn((1, 1, T_max, d), generator=g) for _ in range(2))
    sel = [0, 32767, 32768, 36000, 39999]
    pos = T_max - 2
    got = sw.sparse_attn_decode(U.to_dev(q), U.to_dev(K), U.to_dev(V), B,
                                U.to_dev(np.array([pos], dtype=np.int32)),
                                U.to_dev(np.array([sel], dtype=np.int32)),
                                U.to_dev(np.array([len(sel)], dtype=np.int32)), len(sel)).cpu().numpy()
    tok = np.concatenate([np.arange(j * B, min((j + 1) * B, pos + 1)) for j in sel])
    for u in range(2):
        z = O.f64(K[0, 0, tok]) @ O.f64(q[0, u]) / np.sqrt(d)
        w = np.exp(z - z.max())
        assert U.max_abs(got[0, u], (w / w.sum()) @ O.f64(V[0, 0, tok])) <= U.ATOL_F32


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,batch,h_kv,G", [(64, 515, 1, 1), (128, 129, 4, 2), (128, 511, 1, 1)])
def test_one_split_and_two(dtype, d, batch, h_kv, G):
    """512 (sequence, KV head) pairs and more have one split, fewer have two:
    numbers of heads that leave the merge's last workgroup without some, and
    sequences that are skipped (zeros)."""
    B, T_max = 16, 48
    g = torch.Generator().manual_seed(batch)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    q = torch.randn((batch, G * h_kv, d), generator=g).to(td)
    K, V = (torch.randn((batch, h_kv, T_max, d), generator=g).to(td) for _ in range(2))
    pos = (np.arange(batch) % 50 - 1).astype(np.int32)               # -1 and 48 are skipped
    idx = np.tile(np.arange(3, dtype=np.int32), (batch, 1))
    got = sw.sparse_attn_decode(U.to_dev(q), U.to_dev(K), U.to_dev(V), B, U.to_dev(pos), U.to_dev(idx),
                                U.to_dev(np.full(batch, 3, dtype=np.int32)), 3).float().cpu().numpy()
    qh, Kh, Vh = O.f64(q), O.f64(K), O.f64(V)
    tol = U.ATOL_BF16 if dtype == "bf16" else U.ATOL_F32
    for b in range(batch):
        p = int(pos[b])
        if p < 0 or p >= T_max:
            assert (got[b] == 0.0).all(), b
        else:
            assert U.max_abs(got[b], O.decode_attention(qh[b], Kh[b], Vh[b], [0, 1, 2], p, B)) <= tol, b

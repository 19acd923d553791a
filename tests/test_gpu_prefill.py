"""GPU parity of the prefill hot path against the fp64 oracle, through the
C ABI: sketch scores, walk update, top-tau selection and block-sparse
attention, each in isolation and end to end."""
import math

import numpy as np
import pytest
import torch

import oracle as O
import synth
from paper_2602_07397_amd import binding as sw

pytestmark = pytest.mark.gpu

U = pytest.importorskip("_gpu_util")


def _bf16_case(seqlens, h_q=8, h_kv=2, d=128, B=128, seed_index=40, needles=2):
    w = synth.Workload("case", seed_index, layers=1, h_q=h_q, h_kv=h_kv, d=d, B=B,
                       dtype="bf16", pct=20, seqlens=tuple(seqlens), needles=needles)
    return w


# ---------------------------------------------------------------------------
# sketch_scores
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("n", [2048, 1000])
def test_sketch_matches_oracle_fp32(n):
    w = synth.scaled(synth.WORKLOADS["tiny"], seqlens=(n,))
    Q, K, _ = synth.prefill_layer_inputs(w, 0)
    signs, cols, ts, tc = U.srht_dev(w.d, w.r, w.seed)
    cu = synth.cu_seqlens(w.seqlens)
    sk = sw.sketch_scores(U.to_dev(Q), U.to_dev(K), cu, w.B, ts, tc, want_means=True)
    ref = O.sketch_scores(Q, K, w.B, signs, cols)
    A = sk["A"].cpu().numpy().reshape(ref["A"].shape)
    scale = np.max(np.abs(ref["A"]))
    assert U.max_abs(A, ref["A"]) <= 1e-12 * scale
    np.testing.assert_allclose(sk["Qbar"].cpu().numpy(), ref["qbar"], rtol=1e-12, atol=1e-15)
    np.testing.assert_allclose(sk["Kbar"].cpu().numpy(), ref["kbar"], rtol=1e-12, atol=1e-15)
    np.testing.assert_allclose(sk["Qs"].cpu().numpy(), ref["Qs"], rtol=1e-11, atol=1e-14)
    np.testing.assert_allclose(sk["Ks"].cpu().numpy(), ref["Ks"], rtol=1e-11, atol=1e-14)
    assert sk["A_scale"].item() == pytest.approx(ref["c"], rel=1e-12)


@pytest.mark.parametrize("B,d", [(128, 128), (64, 128), (64, 64), (16, 32), (32, 256), (16, 16)])
def test_sketch_matches_oracle_bf16_gqa_varlen(B, d):
    w = _bf16_case((1000, 384, 257, 64), d=d, B=B)
    Q, K, _ = synth.prefill_layer_inputs(w, 0)
    r = min(64, d)
    signs, cols, ts, tc = U.srht_dev(d, r, w.seed)
    cu = synth.cu_seqlens(w.seqlens)
    sk = sw.sketch_scores(U.to_dev(Q), U.to_dev(K), cu, B, ts, tc, want_means=True)
    As = U.split_mats(sk["A"].cpu().numpy(), cu, B)
    Qs = U.split_rows(sk["Qs"].cpu().numpy(), cu, B)
    Qb = U.split_rows(sk["Qbar"].cpu().numpy(), cu, B)
    scales = sk["A_scale"].cpu().numpy()
    for si, (a, e) in enumerate(zip(cu[:-1], cu[1:])):
        ref = O.sketch_scores(Q[:, a:e], K[:, a:e], B, signs, cols)
        c = np.max(np.abs(ref["A"]))
        assert U.max_abs(As[si], ref["A"]) <= 1e-12 * c, si
        np.testing.assert_allclose(Qs[si], ref["Qs"], rtol=1e-10, atol=1e-14)
        np.testing.assert_allclose(Qb[si], ref["qbar"], rtol=1e-12, atol=1e-15)
        assert scales[si] == pytest.approx(ref["c"], rel=1e-12)
        assert np.all(np.triu(As[si], 1) == 0.0)


# ---------------------------------------------------------------------------
# walk_update
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("s", [1, 2, 8])
def test_walk_matches_oracle_over_layers(s):
    bs = [5, 17, 40, 1]
    B = 16
    cu = synth.cu_seqlens([b * B for b in bs])
    rng = np.random.default_rng(100 + s)
    R_gpu = None
    R_ref = [None] * len(bs)
    for layer in range(4):
        mats = [np.tril(rng.normal(size=(b, b))) for b in bs]
        if layer == 2:
            mats[1] = np.zeros_like(mats[1])          # an all-zero layer: c falls back to 1
        flat = np.concatenate([m.ravel() for m in mats])
        scales = np.array([O.score_scale(m) if np.any(m) else 0.0 for m in mats])
        R_gpu = sw.walk_update(U.to_dev(flat), U.to_dev(scales), s, cu, B, R_gpu)
        for k, m in enumerate(mats):
            R_ref[k] = O.walk_step(R_ref[k], O.walk_weights(m, O.score_scale(m), s))
        got = U.split_mats(R_gpu.cpu().numpy(), cu, B)
        for k in range(len(bs)):
            assert U.max_abs(got[k], R_ref[k]) <= 1e-12, (layer, k)
            assert np.all(np.triu(got[k], 1) == 0.0)


# ---------------------------------------------------------------------------
# select_topk_blocks (values are the same fp64 bits on both sides: exact)
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("kind", ["continuous", "ties", "zeros"])
@pytest.mark.parametrize("mode", [(0, 20, 3), (0, 100, 3), (0, 37, 1), (4, 0, 0), (3, 0, 2), (1, 0, 3)])
def test_select_is_exact(kind, mode):
    k, pct, flags = mode
    bs = [1, 2, 7, 33, 130, 300]
    B = 16
    cu = synth.cu_seqlens([b * B for b in bs])
    rng = np.random.default_rng(7)
    mats = []
    for b in bs:
        if kind == "continuous":
            m = rng.uniform(0, 1, size=(b, b))
        elif kind == "ties":
            m = rng.integers(0, 3, size=(b, b)).astype(np.float64)
        else:
            m = np.zeros((b, b))
        mats.append(np.tril(m))
    flat = np.concatenate([m.ravel() for m in mats])
    idx, cnt, kmax = sw.select_topk_blocks(U.to_dev(flat), cu, B, k=k, density_pct=max(pct, 1),
                                           flags=flags)
    got = U.gpu_selection(idx, cnt)
    ih = idx.cpu().numpy()
    r = 0
    for m in mats:
        ref, _ = O.select_blocks(m, pct=pct, k=k, flags=flags)
        for i, want in enumerate(ref):
            assert got[r] == want, (kind, mode, r, got[r], want)
            assert np.all(ih[r, len(want):] == -1)
            r += 1


def test_select_handles_negative_values_and_negative_zero():
    B = 16
    m = np.tril(np.array([[0.0, 0, 0, 0], [-0.0, 0.0, 0, 0], [-1.0, -0.0, 0.5, 0], [-2.0, 3.0, -0.0, 0.0]]))
    m[1, 0] = -0.0
    idx, cnt, kmax = sw.select_topk_blocks(U.to_dev(m.ravel()), [0, 4 * B], B, k=2, flags=0)
    ref, _ = O.select_blocks(m, k=2, flags=0)
    assert U.gpu_selection(idx, cnt) == ref


# ---------------------------------------------------------------------------
# sparse_attn_prefill (same selection on both sides)
# ---------------------------------------------------------------------------

def _random_selection(cu, B, rng, p=0.3):
    sel = []
    for a, e in zip(cu[:-1], cu[1:]):
        b = -(-(int(e) - int(a)) // B)
        for i in range(b):
            others = [j for j in range(1, i) if rng.uniform() < p]
            sel.append(sorted(set([0, i] + others)))
    return sel


def _pack(sel):
    kmax = max(len(s) for s in sel)
    idx = np.full((len(sel), kmax), -1, dtype=np.int32)
    cnt = np.zeros(len(sel), dtype=np.int32)
    for r, s in enumerate(sel):
        idx[r, :len(s)] = s
        cnt[r] = len(s)
    return U.to_dev(idx), U.to_dev(cnt), kmax


def _oracle_attention(Q, K, V, cu, B, sel):
    outs = []
    r = 0
    for a, e in zip(cu[:-1], cu[1:]):
        b = -(-(int(e) - int(a)) // B)
        outs.append(O.sparse_attention_prefill(Q[:, a:e], K[:, a:e], V[:, a:e], B, sel[r:r + b]))
        r += b
    return np.concatenate(outs, axis=1)


@pytest.mark.parametrize("n,B,d", [(2048, 64, 64), (1000, 64, 64), (700, 128, 128), (333, 64, 128)])
def test_attention_fp32_matches_oracle(n, B, d):
    w = synth.Workload("f32case", 41, layers=1, h_q=2, h_kv=1, d=d, B=B, dtype="f32", pct=20,
                       seqlens=(n,), needles=2, local_window=False)
    Q, K, V = synth.prefill_layer_inputs(w, 0)
    cu = synth.cu_seqlens(w.seqlens)
    sel = _random_selection(cu, B, np.random.default_rng(n))
    idx, cnt, kmax = _pack(sel)
    out, lse = sw.sparse_attn_prefill(U.to_dev(Q), U.to_dev(K), U.to_dev(V), cu, B, idx, cnt, kmax,
                                      want_lse=True)
    ref = _oracle_attention(Q, K, V, cu, B, sel)
    assert U.max_abs(out.cpu().numpy(), ref) <= U.ATOL_F32
    assert torch.isfinite(lse).all()


@pytest.mark.parametrize("seqlens,h_q,h_kv,d,B", [
    ((1000,), 8, 2, 128, 128),
    ((700, 256, 129), 8, 2, 128, 128),
    ((500,), 4, 1, 128, 64),
    ((640,), 4, 4, 128, 64),
    ((384, 200), 6, 2, 64, 128),
    ((300,), 3, 1, 64, 64),
])
def test_attention_bf16_matches_oracle(seqlens, h_q, h_kv, d, B):
    w = _bf16_case(seqlens, h_q=h_q, h_kv=h_kv, d=d, B=B, seed_index=42)
    Q, K, V = synth.prefill_layer_inputs(w, 0)
    cu = synth.cu_seqlens(w.seqlens)
    sel = _random_selection(cu, B, np.random.default_rng(sum(seqlens)))
    idx, cnt, kmax = _pack(sel)
    out = sw.sparse_attn_prefill(U.to_dev(Q), U.to_dev(K), U.to_dev(V), cu, B, idx, cnt, kmax)
    ref = _oracle_attention(Q, K, V, cu, B, sel)
    assert U.max_abs(out.float().cpu().numpy(), ref) <= U.ATOL_BF16


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_density_100_equals_dense_causal(dtype):
    n, B = 777, 64 if dtype == "f32" else 128
    w = synth.Workload("dense", 43, layers=1, h_q=4, h_kv=2, d=128, B=B, dtype=dtype, pct=100,
                       seqlens=(n,), needles=2)
    Q, K, V = synth.prefill_layer_inputs(w, 0)
    signs, cols, ts, tc = U.srht_dev(w.d, w.r, w.seed)
    cu = synth.cu_seqlens(w.seqlens)
    res = U.gpu_prefill_layer(U.to_dev(Q), U.to_dev(K), U.to_dev(V), cu, B, ts, tc, 8, None, pct=100)
    b = -(-n // B)
    assert U.gpu_selection(res["idx"], res["cnt"]) == [list(range(i + 1)) for i in range(b)]
    ref = O.dense_causal_attention(Q, K, V)
    tol = U.ATOL_BF16 if dtype == "bf16" else U.ATOL_F32
    assert U.max_abs(res["O"].float().cpu().numpy(), ref) <= tol


# ---------------------------------------------------------------------------
# end to end
# ---------------------------------------------------------------------------

def test_tiny_workload_end_to_end():
    """2 layers x 1 head, n=2048, d=64, B=64, fp32, density 20%, planted sink
    and needles: selections exact where the oracle gap exceeds 1e-4, outputs
    within 1e-5 of the oracle's masked attention."""
    w = synth.WORKLOADS["tiny"]
    signs, cols, ts, tc = U.srht_dev(w.d, w.r, w.seed)
    cu = synth.cu_seqlens(w.seqlens)
    R_gpu, R_ref = None, None
    for layer in range(w.layers):
        Q, K, V = synth.prefill_layer_inputs(w, layer)
        res = U.gpu_prefill_layer(U.to_dev(Q), U.to_dev(K), U.to_dev(V), cu, w.B, ts, tc, w.s,
                                  R_gpu, pct=w.pct)
        R_gpu = res["R"]
        ref = O.prefill_layer(Q, K, V, w.B, signs, cols, w.s, R_ref, pct=w.pct, attention=False)
        R_ref = ref["R"]
        got = U.gpu_selection(res["idx"], res["cnt"])
        U.check_selection(got, ref["sel"], ref["gaps"], R_ref)
        assert U.max_abs(res["R"].cpu().numpy().reshape(R_ref.shape), R_ref) <= 1e-9
        out = O.sparse_attention_prefill(Q, K, V, w.B, got)
        assert U.max_abs(res["O"].cpu().numpy(), out) <= U.ATOL_F32
        # with identical selections the outputs agree with the oracle pipeline too
        full = O.sparse_attention_prefill(Q, K, V, w.B, ref["sel"])
        same = [i for i in range(len(got)) if got[i] == ref["sel"][i]]
        rows = np.concatenate([np.arange(i * w.B, (i + 1) * w.B) for i in same])
        assert U.max_abs(res["O"].cpu().numpy()[:, rows], full[:, rows]) <= U.ATOL_F32


def test_outputs_are_deterministic():
    w = _bf16_case((1500, 300), seed_index=44)
    Q, K, V = [U.to_dev(x) for x in synth.prefill_layer_inputs(w, 0)]
    signs, cols, ts, tc = U.srht_dev(w.d, w.r, w.seed)
    cu = synth.cu_seqlens(w.seqlens)
    a = U.gpu_prefill_layer(Q, K, V, cu, w.B, ts, tc, 8, None)
    b = U.gpu_prefill_layer(Q, K, V, cu, w.B, ts, tc, 8, None)
    for key in ("A", "A_scale", "Qs", "Ks", "R", "idx", "cnt", "O"):
        assert torch.equal(a[key], b[key]), key


@pytest.mark.parametrize("dtype,h_q,h_kv,d,B,seqlens", [
    ("bf16", 32, 8, 128, 128, [700]),                  # 6 rows: 16 parts each
    ("bf16", 32, 8, 128, 128, [1, 130, 1029]),         # rows of 1, 2 and 5 tokens
    ("bf16", 28, 4, 128, 128, [127 * 128]),            # the most rows with a workspace
    ("bf16", 28, 4, 128, 128, [96 * 128]),             # the most that are split, each type
    ("f32", 28, 4, 128, 128, [127 * 128]),
    ("f32", 32, 8, 64, 64, [2100]),
    ("bf16", 3, 1, 256, 1024, [2500])])
def test_sketch_split_over_workgroups(dtype, h_q, h_kv, d, B, seqlens):
    """Few large block rows are summed in parts when there is a workspace: the
    result with one, with none (NULL) and with one that is too small against
    the oracle; means and scores within 1e-12 of each other (two orders of the
    same fp64 sums of at most 44000 terms: 44000 * 2^-53 = 5e-12 of the largest
    partial sum at worst, about its root in practice)."""
    r = min(64, d)
    signs, cols, ts, tc = U.srht_dev(d, r, 5)
    g = torch.Generator().manual_seed(17)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    N = sum(seqlens)
    Q = torch.randn((h_q, N, d), generator=g).to(td)
    K = torch.randn((h_kv, N, d), generator=g).to(td)
    cu = [0] + list(np.cumsum(seqlens).astype(int))
    need = sw.sketch_workspace_bytes(h_q, h_kv, d, cu, B)
    assert need > 0
    dQ, dK = U.to_dev(Q), U.to_dev(K)
    sk = sw.sketch_scores(dQ, dK, cu, B, ts, tc, want_means=True)
    for s, (a, e) in enumerate(zip(cu[:-1], cu[1:])):
        ref = O.sketch_scores(Q[:, a:e], K[:, a:e], B, signs, cols)
        got = U.split_mats(sk["A"].cpu().numpy(), cu, B)[s]
        np.testing.assert_allclose(got, ref["A"], rtol=1e-12, atol=1e-12 * np.abs(ref["A"]).max())
        assert abs(float(sk["A_scale"][s]) - np.abs(ref["A"]).max()) <= 1e-12 * np.abs(ref["A"]).max()
    lib = sw.load()
    ccu, n = sw._cu(cu)
    small = torch.empty((need - 8,), dtype=torch.uint8, device=U.DEV)
    for ws, wb in ((None, 0), (small.data_ptr(), small.numel())):
        o = {k: torch.empty_like(v) for k, v in sk.items()}
        rc = lib.sw_sketch_scores(sw._dtype_code(dQ), dQ.data_ptr(), dK.data_ptr(), h_q, h_kv, d, n,
                                  ccu, B, ts.data_ptr(), tc.data_ptr(), r, o["Qs"].data_ptr(),
                                  o["Ks"].data_ptr(), o["A"].data_ptr(), o["A_scale"].data_ptr(),
                                  o["Qbar"].data_ptr(), o["Kbar"].data_ptr(), ws, wb,
                                  torch.cuda.current_stream().cuda_stream)
        assert rc == 0, lib.sw_last_error()
        torch.cuda.synchronize()
        for k in sk:
            big = float(sk[k].abs().max())
            assert float((o[k] - sk[k]).abs().max()) <= 1e-12 * max(big, 1e-3), (k, wb)


@pytest.mark.parametrize("blocks", [[512, 31], [513], [545, 17, 1], [640], [1, 16, 33]])
@pytest.mark.parametrize("s,relu", [(8, False), (3, False), (8, True), (5, True)])
def test_walk_product_on_both_tile_sizes(blocks, s, relu):
    """The walk product on each side of 512 blocks, at the edges of its tiles,
    against numpy: 1e-12 of the row's largest magnitude (rows are divided by
    it), as for the other walk tests; signed scores, so sums cancel."""
    B = 16
    rng = np.random.default_rng(40 + len(blocks) + blocks[0] + s)
    cu = [0] + list(np.cumsum([B * b for b in blocks]).astype(int))
    A = [np.tril(rng.normal(size=(b, b))) for b in blocks]
    P = [np.tril(rng.normal(size=(b, b))) for b in blocks]
    P = [p / np.abs(p).max(axis=1, keepdims=True) for p in P]
    c = np.array([np.abs(a).max() for a in A])
    dA = U.to_dev(np.concatenate([a.ravel() for a in A]))
    dP = U.to_dev(np.concatenate([p.ravel() for p in P]))
    R = sw.walk_update_variant(sw.WALK_RELU if relu else sw.WALK_POWER, dA, U.to_dev(c), s, cu, B,
                               R_prev=dP)
    for got, a, p, cc in zip(U.split_mats(R.cpu().numpy(), cu, B), A, P, c):
        x = a / cc
        want = p @ ((np.maximum(x, 0.0) if relu else x) ** s)
        mx = np.abs(want).max(axis=1, keepdims=True)
        want = want / np.where(mx > 0, mx, 1.0)
        np.testing.assert_allclose(got, np.tril(want), rtol=0, atol=1e-12)


@pytest.mark.parametrize("dtype,h_q,h_kv,d,B", [
    ("bf16", 32, 8, 128, 128), ("f32", 32, 8, 128, 128), ("f32", 20, 4, 64, 128), ("bf16", 40, 8, 64, 128),
    ("f32", 6, 2, 256, 128), ("bf16", 9, 3, 256, 128), ("f32", 32, 32, 16, 256), ("bf16", 64, 8, 16, 512)])
def test_a_sequence_has_the_same_sketch_bits_in_any_batch(dtype, h_q, h_kv, d, B):
    """A prompt's sketch is bit-identical alone (its rows split over workgroups),
    alone without a workspace, and in a batch with too many rows to split.
    Values of mixed magnitude, so that another order of the fp64 sums would show
    in either type; a partial last block."""
    r = min(64, d)
    _, _, ts, tc = U.srht_dev(d, r, 6)
    g = torch.Generator().manual_seed(18)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    lens = [5 * B + 77, 130 * B, 3]
    N = sum(lens)
    Q, K = ((torch.randn((h, N, d), generator=g) *
             torch.exp2(torch.randint(-40, 1, (h, N, 1), generator=g).float())).to(td) for h in (h_q, h_kv))
    cu = [0] + list(np.cumsum(lens).astype(int))
    nb = 6
    assert sw.sketch_workspace_bytes(h_q, h_kv, d, [0, lens[0]], B) > 0
    assert sw.sketch_workspace_bytes(h_q, h_kv, d, cu, B) == 0
    batch = sw.sketch_scores(U.to_dev(Q), U.to_dev(K), cu, B, ts, tc, want_means=True)
    dQ, dK = U.to_dev(Q[:, :lens[0]]), U.to_dev(K[:, :lens[0]])
    alone = sw.sketch_scores(dQ, dK, [0, lens[0]], B, ts, tc, want_means=True)
    lib = sw.load()
    ccu, n = sw._cu([0, lens[0]])
    none = {k: torch.empty_like(v) for k, v in alone.items()}
    rc = lib.sw_sketch_scores(sw._dtype_code(dQ), dQ.data_ptr(), dK.data_ptr(), h_q, h_kv, d, n, ccu, B,
                              ts.data_ptr(), tc.data_ptr(), r, none["Qs"].data_ptr(), none["Ks"].data_ptr(),
                              none["A"].data_ptr(), none["A_scale"].data_ptr(), none["Qbar"].data_ptr(),
                              none["Kbar"].data_ptr(), None, 0, torch.cuda.current_stream().cuda_stream)
    assert rc == 0, lib.sw_last_error()
    torch.cuda.synchronize()
    for k in alone:
        assert torch.equal(alone[k], none[k]), k
        part = batch[k][:{"A": nb * nb, "A_scale": 1}.get(k, nb)]
        assert torch.equal(alone[k], part), k


@pytest.mark.parametrize("variant,s", [(sw.WALK_POWER, 8), (sw.WALK_RELU, 3), (sw.WALK_SOFTMAX, 8),
                                       (sw.WALK_MATPOW, 3)])
def test_a_sequence_has_the_same_walk_bits_in_any_batch(variant, s):
    """Sequences on both sides of the 512 blocks where the product's tiles
    change, each alone and all in one call (which runs both tile sizes)."""
    B, blocks = 16, [40, 530, 512, 513, 1]
    rng = np.random.default_rng(60 + variant)
    A = [np.tril(rng.normal(size=(b, b))) for b in blocks]
    P = [np.tril(rng.normal(size=(b, b))) for b in blocks]
    c = np.array([np.abs(a).max() for a in A])
    flat = [U.to_dev(np.concatenate([x.ravel() for x in m])) for m in (A, P)]
    cu = [0] + list(np.cumsum([B * b for b in blocks]).astype(int))
    R = sw.walk_update_variant(variant, flat[0], U.to_dev(c), s, cu, B, R_prev=flat[1], logit_scale=0.7)
    at = 0
    for i, b in enumerate(blocks):
        one = sw.walk_update_variant(variant, U.to_dev(A[i].ravel()), U.to_dev(c[i:i + 1]), s, [0, B * b], B,
                                     R_prev=U.to_dev(P[i].ravel()), logit_scale=0.7)
        assert torch.equal(one, R[at:at + b * b]), b
        at += b * b


@pytest.mark.parametrize("dtype,h_q,h_kv,d,B,lens", [
    ("bf16", 28, 4, 128, 128, [2500, 150 * 128, 77]),     # alone below 640 groups, then heads divided
    ("bf16", 21, 1, 128, 64, [1000, 640 * 64]),           # the same with one head left over
    ("bf16", 32, 8, 128, 128, [700, 9000]),               # alone below one launch of the chip
    ("bf16", 8, 8, 64, 64, [1500, 530 * 64]),             # walk tiles of both kinds
    ("f32", 8, 2, 128, 64, [1300, 5000, 900]),
    ("f32", 4, 4, 64, 64, [700, 3000])])
def test_a_prompt_has_the_same_bits_alone_and_in_a_batch(dtype, h_q, h_kv, d, B, lens):
    """Two layers (sketch, walk, selection, attention with lse) of a prompt by
    itself and as the first of a batch that takes other launches: every output
    bit for bit."""
    r = min(64, d)
    _, _, ts, tc = U.srht_dev(d, r, 6)
    g = torch.Generator().manual_seed(19)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    N, n = sum(lens), lens[0]
    cu = [0] + list(np.cumsum(lens).astype(int))
    b = -(-n // B)
    R1 = R2 = None
    for _ in range(2):
        Q, K, V = (torch.randn((h, N, d), generator=g).to(td) for h in (h_q, h_kv, h_kv))
        K[:, ::3] *= 2.0
        out = []
        for x, c, R in ((n, [0, n], R1), (N, cu, R2)):
            q, k, v = (U.to_dev(t[:, :x]) for t in (Q, K, V))
            o = sw.sketch_scores(q, k, c, B, ts, tc, want_means=True)
            o["R"] = sw.walk_update(o["A"], o["A_scale"], 8, c, B, R)
            o["idx"], o["cnt"], kmax = sw.select_topk_blocks(o["R"], c, B, density_pct=30)
            o["O"], o["lse"] = sw.sparse_attn_prefill(q, k, v, c, B, o["idx"], o["cnt"], kmax, want_lse=True)
            out.append(o)
        one, many = out
        R1, R2 = one["R"], many["R"]
        for key in ("Qs", "Ks", "Qbar", "Kbar", "cnt"):
            assert torch.equal(one[key], many[key][:b]), key
        for key in ("A", "R"):
            assert torch.equal(one[key], many[key][:b * b]), key
        assert torch.equal(one["A_scale"], many["A_scale"][:1])
        assert torch.equal(one["idx"], many["idx"][:b, :one["idx"].shape[1]])
        assert torch.equal(one["O"], many["O"][:, :n]) and torch.equal(one["lse"], many["lse"][:, :n])

"""The fp32 prefill attention forms every product of two fp32 operands from six
partial products of their bf16 parts. How exact its output is, as a 2-norm, and
(on the CPU) that a lost partial product would show in it: each one, dropped
from an emulation of the kernel in float64, exceeds the tolerance."""
import numpy as np
import pytest
import torch

from paper_2602_07397_amd import binding as sw

# (index of the first operand's part, of the second's): 0 leading, 1, 2
PRODUCTS = [(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)]
# Query scale, the products whose loss must show, tolerance. Measured on the
# device: 1.3e-7 to 1.7e-7 at scale 1 and 3.1e-7 to 4.3e-7 at scale 8 (logits of up
# to 40); a lost product gives at least 1.6e-6 and, in the scores at scale 8, 5.9e-6.
CASES = [(1.0, ("scores", "values"), 6e-7), (8.0, ("scores",), 1.5e-6)]


def _inputs(n, d, scale, heads=1):
    g = torch.Generator().manual_seed(14)
    Q, K, V = (torch.randn((h, n, d), generator=g) for h in (heads, 1, 1))
    return Q * scale, K, V


def _exact(q, k, v):
    z = q.double().numpy() @ k.double().numpy().T / np.sqrt(q.shape[1])
    w = np.exp(np.where(np.tri(len(q), dtype=bool), z - z.max(axis=1, keepdims=True), -np.inf))
    return (w / w.sum(axis=1, keepdims=True)) @ v.double().numpy()


def _rel(got, want):
    return np.linalg.norm(got - want) / np.linalg.norm(want)


def _parts(x):
    x = torch.as_tensor(x, dtype=torch.float32)
    h = x.to(torch.bfloat16).float()
    m = (x - h).to(torch.bfloat16).float()
    low = (x - h - m).to(torch.bfloat16).float()
    return [p.double().numpy() for p in (h, m, low)]


def _emulated(q, k, v, drop=None):
    """The kernel's products in float64; drop = ("scores" or "values", product)."""
    qp, kp, vp = _parts(q), _parts(k), _parts(v)
    z = sum(qp[a] @ kp[b].T for a, b in PRODUCTS if ("scores", (a, b)) != drop) / np.sqrt(q.shape[1])
    z = np.where(np.tri(len(q), dtype=bool), z, -np.inf)
    w = np.exp(z - z.max(axis=1, keepdims=True))
    wp = _parts(w)
    o = sum(wp[a] @ vp[b] for a, b in PRODUCTS if ("values", (a, b)) != drop)
    return o / w.sum(axis=1, keepdims=True)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scale,where,tol", CASES)
def test_a_lost_product_exceeds_the_tolerance(d, scale, where, tol):
    Q, K, V = _inputs(384, d, scale)
    want = _exact(Q[0], K[0], V[0])
    assert _rel(_emulated(Q[0], K[0], V[0]), want) <= tol / 10
    for part in where:
        for p in PRODUCTS:
            assert _rel(_emulated(Q[0], K[0], V[0], (part, p)), want) >= 2 * tol, (part, p)


@pytest.mark.gpu
@pytest.mark.parametrize("d,B,G", [(64, 64, 1), (128, 64, 1), (64, 128, 1), (128, 128, 1), (128, 64, 3),
                                   (64, 64, 2), (128, 128, 2)])
@pytest.mark.parametrize("scale,where,tol", CASES)
def test_fp32_attention_has_all_six_products(d, B, G, scale, where, tol):
    """Every form of the kernel (pipelined or not, key halves or not), all blocks
    selected."""
    n = 384
    b = n // B
    Q, K, V = _inputs(n, d, scale, heads=G)
    idx = torch.full((b, b), -1, dtype=torch.int32)
    for i in range(b):
        idx[i, :i + 1] = torch.arange(i + 1)
    got = sw.sparse_attn_prefill(Q.cuda(), K.cuda(), V.cuda(), [0, n], B, idx.cuda(),
                                 torch.arange(1, b + 1, dtype=torch.int32).cuda(), b).double().cpu().numpy()
    for u in range(G):
        err = _rel(got[u], _exact(Q[u], K[0], V[0]))
        print(f"d {d} B {B} G {G} scale {scale}: {err:.2e}", flush=True)
        assert err <= tol, (u, err)

"""How closely the six products of the bf16 triples hold a network's gradient, on the
CPU: forward, Hbar and dW of a tanh network with every contraction from split operands
(8 + 8 + 8 bits, summed without rounding).  All six hold it within the operands' own rounding to fp32; without
any one of them, in any one kind of contraction, the gradient is further off than
BOUND_GRAD (in the forward: and the outputs than BOUND_VALUE), the bounds that the GPU's
are held to (test_gpu_precision.py)."""
import numpy as np
import pytest

BOUND_GRAD = 5e-7
BOUND_VALUE = 1e-6
SIX = [(2, 0), (0, 2), (1, 1), (1, 0), (0, 1), (0, 0)]   # parts of the two operands


def bf16(v):
    u = np.asarray(v, np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(np.float32)


def parts(x):
    x = np.asarray(x, np.float32)
    h = bf16(x)
    m = bf16(x - h)
    return [p.astype(np.float64) for p in (h, m, (x - h) - m)]


def contract(a, b, products):
    """a [M][K] times b [K][N]"""
    if products is None:
        return a @ b
    a, b = parts(a), parts(b)
    return sum(a[i] @ b[j] for i, j in products)


def gradient(W, H, products, seed=0):
    """outputs and gradient; products: by kind of contraction, None for 64 bits"""
    rng = np.random.default_rng([seed, W, H])
    n, D = 64, 4
    f32 = lambda a: np.asarray(a, np.float32).astype(np.float64)  # noqa: E731
    w1 = f32(rng.standard_normal((W, D)) * np.sqrt(2.0 / (W + D)))
    ws = [f32(rng.standard_normal((W, W)) * np.sqrt(1.0 / W)) for _ in range(H - 1)]
    wo = f32(rng.standard_normal((D, W)) * np.sqrt(2.0 / (W + D)))
    x, t = f32(rng.uniform(-1, 1, (D, n))), f32(rng.standard_normal((D, n)))
    h = [np.tanh(w1 @ x)]
    for w in ws:
        h.append(np.tanh(contract(w, h[-1], products["forward"])))
    y = wo @ h[-1]
    hb = wo.T @ (y - t)
    g = []
    for l in range(H - 1, 0, -1):
        zb = hb * (1 - h[l] ** 2)
        g.append(contract(zb, h[l - 1].T, products["dW"]).ravel())
        hb = contract(ws[l - 1].T, zb, products["Hbar"])
    g.append((hb * (1 - h[0] ** 2) @ x.T).ravel())
    return y.ravel(), np.concatenate(g)


KINDS = ("forward", "Hbar", "dW")


@pytest.mark.parametrize("W,H", [(32, 2), (48, 4), (128, 3), (208, 3)])
def test_each_of_the_six_products_counts(W, H):
    ref = gradient(W, H, dict.fromkeys(KINDS))

    def off(products):
        return [np.linalg.norm(a - b) / np.linalg.norm(b) for a, b in zip(gradient(W, H, products), ref)]

    # what remains: each layer's operands are rounded to fp32 before they are split
    assert max(off(dict.fromkeys(KINDS, SIX))) <= H * 2.0 ** -24
    for q in range(6):
        less = SIX[:q] + SIX[q + 1:]
        for kind in KINDS:
            value, grad = off({**dict.fromkeys(KINDS, SIX), kind: less})
            assert grad > BOUND_GRAD, (kind, SIX[q], grad)
            assert kind != "forward" or value > BOUND_VALUE, (SIX[q], value)

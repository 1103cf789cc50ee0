"""The split cyclic product over GF(2), as the kernels form it, on the CPU.

A cyclic product of T = 3^k chunks of M 32-bit words is computed through
T products in GF(2)[v] / (v^(2M) + v^M + 1), v = X^32, each of those through
2 * 3^a products in the ring of 2 M2 words, with the same index rules as the
kernels: the chunks' forward transform in two steps (tau = rho + Q sigma,
t = t0 + P t1), periodic sequences (lo, lo + hi, hi) for ring elements, a
leaf product as a plain correlation, and the overlap of neighbouring chunks
folded into each product before the inverse transform.  The result is
compared with the plain polynomial product.
"""
import random

import numpy as np
import pytest


def clmul(a, b):
    r = 0
    while b:
        low = b & -b
        r ^= a << (low.bit_length() - 1)
        b ^= low
    return r


def to_int(w):
    return sum(int(v) << (32 * i) for i, v in enumerate(w))


def to_words(x, n):
    return np.array([(x >> (32 * i)) & 0xFFFFFFFF for i in range(n)], dtype=np.uint64)


def roll(x, s):
    return np.roll(x, s % len(x))


def forward(src, Q, P, g):
    """X_tau as (lo, hi) words of every tau."""
    T = P * Q
    M = T // 3 * g
    X = np.zeros((T, 2 * M), dtype=np.uint64)
    for rho in range(Q):
        tile = np.zeros((P, 3 * M), dtype=np.uint64)
        for t in range(T):
            chunk = np.zeros(3 * M, dtype=np.uint64)
            chunk[:M] = src[t * M:(t + 1) * M]
            tile[t % P] ^= roll(chunk, g * rho * t)
        a, b, c = tile[:, :M], tile[:, M:2 * M], tile[:, 2 * M:]
        beta = np.concatenate([a ^ c, a ^ b, b ^ c], axis=1)
        for sg in range(P):
            acc = np.zeros(3 * M, dtype=np.uint64)
            for t0 in range(P):
                acc ^= roll(beta[t0], g * Q * sg * t0)
            X[rho + Q * sg] = np.concatenate([acc[:M], acc[2 * M:]])
    return X


def ring_product(x, s, na, M2, tau, g):
    """The product of two ring elements, with the overlap rule applied."""
    M, u = na * M2, M2 // na

    def points(e):
        lo, hi = e[:M].reshape(na, M2), e[M:].reshape(na, M2)
        v = {}
        for i in range(3 * na):
            if i % 3 == 0:
                continue
            acc = np.zeros(3 * M2, dtype=np.uint64)
            for c in range(na):
                both = lo[c] ^ hi[c]
                b = [lo[c], both, hi[c]] if i % 3 == 1 else [both, lo[c], hi[c]]
                acc ^= roll(np.concatenate(b), u * i * c)
            v[i] = acc
        return v

    vx, vs, w = points(x), points(s), {}
    for i in vx:
        a = to_int(np.concatenate([vx[i][:M2], vx[i][2 * M2:]]))
        row = to_int(np.concatenate([vs[i], vs[i][:M2]]))
        n2 = 64 * M2
        out = to_words((clmul(a, row) >> n2) & ((1 << n2) - 1), 2 * M2)
        hi, lo = out[:M2], out[M2:]
        w[i] = np.concatenate([lo, lo ^ hi, hi])
    low, high = [None] * (2 * na), [None] * (2 * na)
    for c in range(na):
        d = []
        for r in (1, 2):
            acc = np.zeros(3 * M2, dtype=np.uint64)
            for k in range(na):
                acc ^= roll(w[3 * k + r], -u * (3 * k + r) * c)
            d.append((acc[:M2], acc[2 * M2:]))
        h0, h1 = d[0][0] ^ d[1][0], d[0][1] ^ d[1][1]
        low[c + na], high[c + na] = h0, h1
        low[c], high[c] = d[0][0] ^ h1, d[0][1] ^ h0 ^ h1
    blocks = [low[b] ^ (high[b - 1] if b else 0) for b in range(2 * na)]
    blocks[0] = blocks[0] ^ high[2 * na - 1]
    blocks[na] = blocks[na] ^ high[2 * na - 1]
    c0, c1 = np.concatenate(blocks[:na]), np.concatenate(blocks[na:])
    beta = np.concatenate([c0, c0 ^ c1, c1])
    return beta ^ roll(beta, -(2 * M - g * tau))


@pytest.mark.parametrize("Q,P,g,na", [(3, 3, 1, 1), (9, 1, 2, 1), (9, 3, 1, 3), (9, 3, 2, 3), (9, 9, 1, 3)])
def test_split_product_is_the_cyclic_product(Q, P, g, na):
    T = P * Q
    M = T // 3 * g
    N = T * M
    rnd = random.Random(1000 * T + g)
    a = np.array([rnd.getrandbits(32) for _ in range(N)], dtype=np.uint64)
    b = np.array([rnd.getrandbits(32) for _ in range(N)], dtype=np.uint64)
    full = clmul(to_int(a), to_int(b))
    want = to_words((full & ((1 << (32 * N)) - 1)) ^ (full >> (32 * N)), N)
    X, S = forward(a, Q, P, g), forward(b, Q, P, g)
    H = [ring_product(X[tau], S[tau], na, M // na, tau, g) for tau in range(T)]
    got = np.zeros(N, dtype=np.uint64)
    for t in range(T):
        for tau in range(T):
            got[t * M:(t + 1) * M] ^= roll(H[tau], -g * t * tau)[:M]
    assert np.array_equal(got, want)

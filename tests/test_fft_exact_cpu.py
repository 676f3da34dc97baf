"""The double-precision transforms of the blind rotation, modelled on the CPU:
the sums of digit x key-piece products that they give round to the exact
integers, with an error far below the bound the dispatch relies on, at the
edge of every case it accepts and on inputs of extreme size; the rule that
chooses the number of pieces; and the constants that put the rounded pieces
together modulo p."""
import numpy as np
import pytest

P = 0xFFFFFFFF00000001


def pieces(N, l, beta):
    """The dispatch rule: 2 l N 2^(beta + b - 2) 160 u <= 1/4 with u = 2^-53."""
    if N not in (2048, 4096) or l > 3:
        return 0
    holds = lambda b: 2 * l * N * 160 << (beta + b - 2) <= 1 << 51
    if l * beta <= 30 and holds(22):
        return 3
    return 4 if holds(16) else 0


def e(x):
    """e(x) = exp(2 pi i x) for an array of turns, rounded from long double."""
    t = np.asarray(x, dtype=np.longdouble) * (8 * np.arctan(np.longdouble(1)))
    return np.cos(t).astype(np.float64) + 1j * np.sin(t).astype(np.float64)


def bitrev(x, bits):
    return int(format(x, f"0{bits}b")[::-1], 2) if bits else 0


def forward(z):
    """Merged-twist splitting of z modulo X^C - i, stage by stage."""
    C = z.shape[-1]
    m = C.bit_length() - 1
    x = z.astype(np.complex128).copy()
    for s in range(m):
        phi = np.array([2.0 ** -(s + 2) + bitrev(b, s) / 2.0 ** s for b in range(1 << s)])
        w = e(phi / 2)[:, None]
        y = x.reshape(1 << s, 2, C >> (s + 1))
        u, v = y[:, 0], y[:, 1]
        a = u + w * v
        x = np.stack([a, 2 * u - a], axis=1).reshape(C)
    return x


def inverse(x):
    """Decimation in time from bit-reversed order, the twist at the end."""
    C = x.shape[-1]
    m = C.bit_length() - 1
    x = x.copy()
    for t in range(1, m + 1):
        h = 1 << (t - 1)
        w = e(-np.arange(h) / 2.0 ** t)[None, :]
        y = x.reshape(C >> t, 2, h)
        u, v = y[:, 0], y[:, 1]
        a = u + w * v
        x = np.stack([a, 2 * u - a], axis=1).reshape(C)
    return x * e(-np.arange(C) / (4.0 * C)) / C


def fold(y):
    h = y.shape[0] // 2
    return y[:h].astype(np.float64) + 1j * y[h:].astype(np.float64)


def negacyclic(a, b):
    """Exact product modulo X^N + 1 by Kronecker substitution."""
    N, W = len(a), 96
    def pack(v):
        pos = sum(int(x) << (W * i) for i, x in enumerate(v) if x > 0)
        neg = sum(int(-x) << (W * i) for i, x in enumerate(v) if x < 0)
        return pos - neg
    c = pack(a) * pack(b)
    half, mask = 1 << (W - 1), (1 << W) - 1
    out = []
    for _ in range(2 * N):
        d = ((c + half) & mask) - half
        out.append(d)
        c = (c - d) >> W
    return [out[i] - out[i + N] for i in range(N)]


def test_forward_is_the_evaluation():
    """The forward transform against its definition on a small ring."""
    rng = np.random.default_rng(1)
    C, m = 16, 4
    z = rng.integers(-9, 10, C) + 1j * rng.integers(-9, 10, C)
    got = forward(z)
    for j in range(C):
        r = 1.0 / (4 * C) + bitrev(j, m) / C
        assert abs(got[j] - np.sum(z * e(r * np.arange(C)))) < 1e-12
    assert np.max(np.abs(inverse(got) - z)) < 1e-12


def _edges():
    """(N, l, beta) at both ends of every case the rule accepts."""
    out = []
    for N in (2048, 4096):
        for l in (1, 3):
            for P_ in (3, 4):
                ok = [b for b in range(1, 31) if pieces(N, l, b) == P_]
                out.append((N, l, max(ok), P_))
    return out


@pytest.mark.parametrize("N,l,beta,npieces", _edges())
@pytest.mark.parametrize("kind", ["random", "extreme", "aligned"])
def test_sums_round_to_the_exact_integers(N, l, beta, npieces, kind):
    """One component's sum over the 2l rows of one piece.  The error bound is
    2 l N 2^(beta + b - 2) 160 u <= 1/4; the plain multiplications of the
    model (the kernels use fused ones) cost it a little more."""
    bits = 22 if npieces == 3 else 16
    top_d, top_k = 1 << (beta - 1), 1 << (bits - 1)
    rng = np.random.default_rng(N + l + beta)
    acc = np.zeros(N // 2, np.complex128)
    exact = np.zeros(N, object)
    for r in range(2 * l):
        if kind == "random":
            d = rng.integers(-top_d, top_d, N)
            k = rng.integers(-top_k, top_k, N)
        elif kind == "extreme":
            d = np.where(rng.random(N) < 0.5, -top_d, top_d)
            k = np.where(rng.random(N) < 0.5, -top_k, top_k)
        else:  # every product of coefficient N - 1 has one sign
            d, k = np.full(N, top_d), np.full(N, -top_k)
        acc += forward(fold(d)) * forward(fold(k))
        exact += np.array(negacyclic(d, k), object)
    y = inverse(acc)
    got = np.concatenate([y.real, y.imag])
    bound = 2 * l * N * 2.0 ** (beta + bits - 2) * 160 * 2.0 ** -53
    assert bound <= 0.25
    off = max(abs(float(g - np.rint(g)) + float(int(np.rint(g)) - x)) for g, x in zip(got, exact))
    assert all(int(np.rint(g)) == x for g, x in zip(got, exact))
    assert off < bound


def test_rule_edges():
    """Workload sets and the first digit size past each edge."""
    assert pieces(2048, 3, 8) == pieces(2048, 2, 10) == pieces(4096, 3, 8) == 3
    assert pieces(2048, 3, 14) == 4
    for N in (2048, 4096):
        for l in (1, 2, 3):
            seq = [pieces(N, l, b) for b in range(1, 31)]
            # three pieces, then four, then none, and every value on the way
            assert seq == sorted(seq, key=lambda v: {3: 0, 4: 1, 0: 2}[v]) and set(seq) == {0, 3, 4}
            # sums stay inside what the rounding constants are made for
            for b, v in zip(range(1, 31), seq):
                if v:
                    bits = 22 if v == 3 else 16
                    assert 2 * l * N * 2 ** (b + bits - 2) < 2 ** 44
    assert pieces(1024, 2, 8) == pieces(2048, 4, 8) == 0


@pytest.mark.parametrize("npieces", [3, 4])
def test_piece_offsets_cancel(npieces):
    """Rounding by M_p = 1.5 2^52 + m_p and adding the bit patterns gives the
    sum modulo p: the offsets, solved as the kernel solves them, cancel the
    exponent bits; checked through the 128-bit sum with its dropped top bits."""
    bits = 22 if npieces == 3 else 16
    X = 0x4338 << 48
    k = sum((X if q < npieces - 1 else (1 << 51 if npieces == 3 else 1 << 47)) << (bits * q)
            for q in range(npieces)) % P
    v = (-k) % P
    v = v - P if v > (P - 1) // 2 else v
    m = []
    for q in range(npieces):
        d = v if q == npieces - 1 else ((v + (1 << (bits - 1))) & ((1 << bits) - 1)) - (1 << (bits - 1))
        v = (v - d) >> bits
        m.append(d)
    rng = np.random.default_rng(npieces)
    for _ in range(2000):
        r = [int(x) for x in rng.integers(-2 ** 44 + 1, 2 ** 44, npieces)]
        acc = int(rng.integers(0, P, dtype=np.uint64))
        B = []
        for q in range(npieces):
            M = 1.5 * 2.0 ** 52 + m[q] + (2.0 ** 47 if npieces == 4 and q == 3 else 0.0)
            B.append(int(np.float64(float(r[q]) + M).view(np.uint64)))
        sh = bits * (npieces - 1)
        last = B[-1] & ((1 << (32 + 64 - sh)) - 1)  # the bits the sum keeps
        total = acc + sum(b << (bits * q) for q, b in enumerate(B[:-1])) + (last << sh)
        assert total >> 96 == 0 and total % P == (acc + sum(x << (bits * q)
                                                        for q, x in enumerate(r))) % P

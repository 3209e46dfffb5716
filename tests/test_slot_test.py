"""P2's zero test without reduction and the grouped shuffle digits.

On the CPU: the arithmetic the kernels run (word by word, in Python
integers) at the bounds of its operands, against its definition.  On the
GPU: the DReLU against the oracle where the pieces change form (window
counts at the edges of each form, the smallest and the default prime) on
shares whose windows are all zeros, all ones and their neighbours.
Everything is integer: the tolerance is 0.
"""

import numpy as np
import pytest

from oracle import philox as OPH
from oracle import protocols as OPR
from oracle.params import default_prime
import workloads as W

M32, M64 = (1 << 32) - 1, (1 << 64) - 1


def smallest_prime(lx):
    import sympy
    return int(sympy.nextprime(1 << lx))


def signed32(v):
    v &= M32
    return v - (1 << 32) if v >> 31 else v


def mark(n, p, v0, v1, r, z, shift):
    """A slot's mark and the largest one that counts as zero, as the kernels form them."""
    inv = pow(p, -1, 1 << 32)
    if n <= 16:
        m0, m1 = v0 * r + r + z, v1 * r + r + z
        assert m0 <= M32 and m1 <= M32
        k = (1 << (n - 1)) - 1
        return ((m0 - m1) * inv + k) & M32, 2 * k
    if n <= 32:
        rs, zs = r << shift, z << shift
        m0, m1 = v0 * rs + rs + zs, v1 * rs + rs + zs
        assert rs <= M32 and zs <= M32 and m0 < 1 << 63 and m1 < 1 << 63
        d = m0 - m1
        k = signed32(d * inv)
        e = d - k * p if n <= 31 else d + ((1 << 32) - p) * k
        assert e & M32 == 0 and -(1 << 63) <= e < 1 << 63
        return ((e >> 32) & M32) ^ (0 if n <= 31 else k & M32), 0
    r0, r1 = r & M32, r >> 32

    def twice(v):
        x = v * r0
        return 9 * (x >> 32) + 9 * (v if r1 else 0) + 2 * (x & M32) + 2 * (r + z)
    u = twice(v0) - twice(v1)
    assert abs(u) < 1 << 38
    k = (u * inv & 0xFF) - (256 if u * inv & 0x80 else 0)
    e = u + 9 * k
    return (e & M32) | (((e >> 32) & M32) ^ ((2 * k) & M32)), 0


@pytest.mark.parametrize("n", range(2, 34))
def test_mark_decides_divisibility(n):
    lx = n - 1
    rng = np.random.default_rng(n)
    primes = [default_prime(lx)] if n == 33 else [default_prime(lx), smallest_prime(lx)]
    for p in primes:
        # the default prime keeps r and z shifted to the top of the word at N = 17..31; there z is any field below 2^N
        stream = p == default_prime(lx) and n >= 17
        shift = 32 - n if stream and n <= 31 else 0
        top, ztop = (1 << lx) - 1, (1 << n) - 1 if stream else p - 1
        vs = sorted(v for v in {0, 1, 2, top // 2, top - 1, top} if 0 <= v <= top)
        rs = sorted(r for r in {1, 2, p // 2, (1 << 32) - 1, 1 << 32, p - 2, p - 1} if 1 <= r < p)
        cases = [(a, b, r, z) for a in vs for b in vs for r in rs for z in (0, 1, ztop)]
        cases += [(int(a), int(b), int(r), int(z)) for a, b, r, z in zip(
            rng.integers(0, top + 1, 4000), rng.integers(0, top + 1, 4000), rng.integers(1, p, 4000),
            rng.integers(0, ztop + 1, 4000))]
        for v0, v1, r, z in cases:
            m, limit = mark(n, p, v0, v1, r, z, shift)
            assert (m <= limit) == ((v0 - v1) * r % p == 0), (p, v0, v1, r, z)


@pytest.mark.parametrize("n", range(2, 34))
def test_grouped_digits_are_the_sequential_ones(n):
    """Digits cut group by group against digit d = floor(F m / 2^64), F <- F m mod 2^64."""
    rng = np.random.default_rng(100 + n)

    def fits(m):
        c = -(-(1 << 32) // m)
        return m <= M32 and (m - 1) * c <= M32 and (m - 1) * (c * m - (1 << 32)) <= M32
    for digits in OPH.shuffle_chunks(n):
        radices = [OPH.shuffle_radices(n)[k] for k in digits]
        groups = []
        for m in radices:
            if groups and fits(int(np.prod(groups[-1], dtype=object)) * m):
                groups[-1].append(m)
            else:
                groups.append([m])
        total = int(np.prod(radices, dtype=object))
        starts = [0, M64, M64 - 1] + [int(rng.integers(0, 1 << 63)) * 2 + 1 for _ in range(3000)]
        # both sides of values where a digit changes
        for x in rng.integers(0, total, 3000):
            edge = -(-(int(x) << 64) // total)
            starts += [edge & M64, (edge - 1) & M64]
        for start in starts:
            seq, f = [], start
            for m in radices:
                seq.append(f * m >> 64)
                f = f * m & M64
            got, f = [], start
            for g in groups:
                prod = int(np.prod(g, dtype=object))
                part = (f * prod >> 64) * -(-(1 << 32) // prod)
                f = f * prod & M64
                assert part <= M32
                for m in g:
                    got.append(part * m >> 32)
                    part = part * m & M32
            assert got == seq, (start, groups)


@pytest.mark.gpu
@pytest.mark.parametrize("op", ["drelu", "relu"])
@pytest.mark.parametrize("smallest", [False, True])
@pytest.mark.parametrize("ell,lx", [(64, lx) for lx in (1, 7, 8, 9, 15, 16, 17, 19, 20, 23, 24, 30, 31, 32)] +
                         [(32, lx) for lx in (1, 7, 8, 14, 15, 16)])
def test_extreme_windows_match_oracle(op, smallest, ell, lx):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_04909_amd import bicop as B
    p = smallest_prime(lx) if smallest else default_prime(lx)
    if smallest and p >= 2 << lx:
        pytest.skip("one prime only")
    k_lo = min(3, ell - 2 * lx)
    full = (1 << ell) - 1
    marks = sorted({0, 1, 2, 3, (1 << lx) - 1, 1 << lx, (1 << 2 * lx) - 1, 1 << (2 * lx - 1), full, full - 1, full >> 1,
                    1 << (ell - 1), 0x5555555555555555 & full, 0xAAAAAAAAAAAAAAAA & full})
    marks = sorted({(m << s) & full for m in marks for s in (0, k_lo)})
    x0 = np.array([a for a in marks for _ in marks], dtype=np.uint64)
    x1 = np.array([(-b) & full for _ in marks for b in marks], dtype=np.uint64)
    reps = 8
    x0, x1 = np.tile(x0, reps), np.tile(x1, reps)
    dt = W.storage_dtype(ell)
    it = np.int64 if ell > 32 else np.int32
    d0, d1 = (torch.from_numpy(x.astype(dt).view(it)).cuda() for x in (x0, x1))
    seeds = (lx, 7 * ell, 99)
    fn, ofn = (B.drelu, OPR.drelu) if op == "drelu" else (B.relu, OPR.relu)
    e0, e1, _, _ = ofn(x0, x1, ell, lx, k_lo, p, seeds, 5)
    ut = np.uint64 if ell > 32 else np.uint32
    for capture in (False, True):
        out = fn(d0, d1, B.Params(ell, lx, k_lo, p), B.Seeds(*seeds, 5), capture=capture)
        for got, exp in zip(out, (e0, e1)):
            assert np.array_equal(got.cpu().view(torch.int64 if ell > 32 else torch.int32).numpy().view(ut).astype(np.uint64), exp)

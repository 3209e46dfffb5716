"""The other routes to a DReLU / ReLU result, for every window count and for an
explicit prime beside the default one: records, ragged batches with and
without records, the parties apart, and replicated sharing.  The plain call,
which is compared with the oracle elsewhere, says what each must give (and for
replicated sharing the capturing call, whose zero test reduces every message);
integers, so the tolerance is 0."""

import pytest

from oracle.params import default_prime

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SETTINGS = ([(64, lx) for lx in range(1, 33)] + [(32, lx) for lx in range(1, 17)] + [(63, 31), (51, 11), (40, 18), (24, 7), (30, 15)])


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_04909_amd import bicop
    return bicop


def shares(ell, lx, k_lo, n, count):
    """Shares of values around the window's edges and of arbitrary ring elements."""
    gen = torch.Generator(device="cuda").manual_seed(100 * ell + lx)
    bound = 1 << (k_lo + lx - 1)
    x = torch.randint(-bound + 1, bound, (n,), generator=gen, device="cuda", dtype=torch.int64)
    x[::3] = torch.randint(-(1 << 62), 1 << 62, (len(x[::3]),), generator=gen, device="cuda")
    x[1::7] = torch.randint(-2, 3, (len(x[1::7]),), generator=gen, device="cuda") << k_lo
    parts = [torch.randint(-(1 << 62), 1 << 62, (n,), generator=gen, device="cuda") for _ in range(count - 1)]
    first = x
    for r in parts:
        first = first - r
    ring = (1 << ell) - 1 if ell < 64 else -1
    return [(s & ring).to(torch.int64 if ell > 32 else torch.int32).contiguous() for s in [first] + parts]


def primes(lx):
    import sympy
    out = [default_prime(lx)]
    return out + [int(sympy.prevprime(out[0]))] if lx >= 2 else out


def eq(a, b):
    return all(torch.equal(p.view(torch.int32), q.view(torch.int32)) for p, q in zip(a, b))


@pytest.mark.parametrize("ell,lx", SETTINGS)
def test_every_route_gives_the_plain_call_s_shares(B, ell, lx):
    from paper_2309_04909_amd import batch as BT
    k_lo, n, base = min(13 if ell > 32 else 8, ell - 2 * lx), 1001, (1 << 32) - 333
    x0, x1 = shares(ell, lx, k_lo, n, 2)
    sd = B.Seeds(0x1122334455667788 ^ lx, 0x99AABBCCDDEEFF00 ^ ell, 777, 31)
    for p in primes(lx):
        prm = B.Params(ell, lx, k_lo, p)
        want = {B.BC_OP_DRELU: B.drelu(x0, x1, prm, sd, elem_base=base), B.BC_OP_RELU: B.relu(x0, x1, prm, sd, elem_base=base)}
        segs = []
        for op, expect in want.items():
            rec = B.rand_expand(op, prm, sd, n, elem_base=base)
            pre = B.relu_pre if op == B.BC_OP_RELU else B.drelu_pre
            assert eq(pre(x0, x1, prm, rec), expect), ("record", op, p)
            for rand in (None, rec):
                segs.append((BT.Segment(x0, x1, torch.empty_like(x0), torch.empty_like(x1), op=op, nonce=sd.nonce,
                                        elem_base=base, rand=rand), expect))
        for tile in (0, 300):
            BT.RaggedBatch(prm, sd, [s for s, _ in segs], tile_elems=tile).run()
            for s, expect in segs:
                assert eq((s.y0, s.y1), expect), ("batch", s.op, s.rand is None, p)
                s.y0.fill_(-1)
                s.y1.fill_(-1)
        d = B.drelu_reply(*(B.drelu_send(k, x, prm, sd, elem_base=base) for k, x in enumerate((x0, x1))), prm, sd, elem_base=base)
        assert eq([B.drelu_finish(k, d[k], prm, sd, elem_base=base) for k in (0, 1)], want[B.BC_OP_DRELU]), ("apart", p)


@pytest.mark.parametrize("op", ["rss_drelu", "rss_relu"])
@pytest.mark.parametrize("ell,lx", SETTINGS)
def test_replicated_sharing_equals_the_capturing_call(B, ell, lx, op):
    k_lo, base = min(13 if ell > 32 else 8, ell - 2 * lx), (1 << 32) - 333
    seeds = B.RssSeeds(21 + lx, 22 + ell, 23, 24, 25, 26)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    for n in (1001, 4 * 64 * 4 * units + 77):                 # four waves (default prime), and one lane
        x = tuple(shares(ell, lx, k_lo, n, 3))
        for p in primes(lx):
            prm = B.Params(ell, lx, k_lo, p)
            want, _ = getattr(B, op)(x, prm, seeds, elem_base=base, capture=True)
            assert eq(getattr(B, op)(x, prm, seeds, elem_base=base), want), (n, p)

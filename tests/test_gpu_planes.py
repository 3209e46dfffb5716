"""The walks over the planes of a record and of packed messages (nontemporal or
through the L2, blocks in order or by XCD): sizes on and off 32 elements, grids
that are no multiple of the 8 XCDs, and planes above the memory-side cache.
Both forms must give exactly the fused call's shares (integers: no tolerance)."""

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SETTINGS = [(64, 7, 11), (51, 11, 13), (64, 18, 13), (64, 31, 0), (32, 8, 8)]
SIZES = [1, 31, 32, 33, 2304, 2305, 70001, 70016]


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_04909_amd import bicop
    return bicop


def shares(B, prm, n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    bound = 1 << (prm.k_lo + prm.lx - 1)
    x = torch.randint(-bound + 1, bound, (n,), generator=gen, device="cuda", dtype=torch.int64)
    r = torch.randint(-(1 << 62), 1 << 62, (n,), generator=gen, device="cuda", dtype=torch.int64)
    ring = (1 << prm.ell) - 1 if prm.ell < 64 else -1
    return [(s & ring).to(B.ring_dtype(prm.ell)) if prm.ell > 32 else s.to(torch.int32) for s in (x - r, r)]


def check(B, setting, n, ops):
    prm, sd = B.Params(*setting), B.Seeds(11, 12, 13, 14)
    x0, x1 = shares(B, prm, n, n + setting[1])
    for op in ops:
        relu = op == B.BC_OP_RELU
        want = (B.relu if relu else B.drelu)(x0, x1, prm, sd)
        rec = B.rand_expand(op, prm, sd, n)
        got = (B.relu_pre if relu else B.drelu_pre)(x0, x1, prm, rec)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        del rec
    want = B.drelu(x0, x1, prm, sd)
    d0, d1 = B.drelu_reply(B.drelu_send(0, x0, prm, sd), B.drelu_send(1, x1, prm, sd), prm, sd)
    assert torch.equal(B.drelu_finish(0, d0, prm, sd), want[0])
    assert torch.equal(B.drelu_finish(1, d1, prm, sd), want[1])


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("setting", SETTINGS)
def test_walks_match_the_fused_call(B, setting, n):
    check(B, setting, n, (B.BC_OP_DRELU, B.BC_OP_RELU))


@pytest.mark.parametrize("extra", [0, 1])
@pytest.mark.parametrize("setting", [(64, 18, 13), (64, 31, 0)])
def test_planes_above_the_cache(B, setting, extra):
    check(B, setting, (1 << 22) + extra, (B.BC_OP_DRELU,))


def test_calls_above_one_launch(B):
    """A call of more than 2^28 elements runs as several launches; each continues the last one's elements."""
    prm, sd = B.Params(32, 1, 3), B.Seeds(11, 12, 13, 14)
    edge, n = 1 << 28, (1 << 28) + 77
    x0, x1 = shares(B, prm, n, 5)
    want = B.relu(x0, x1, prm, sd)
    got = B.relu_pre(x0, x1, prm, B.rand_expand(B.BC_OP_RELU, prm, sd, n))
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    del got, want
    want = B.drelu(x0, x1, prm, sd)
    d0, d1 = B.drelu_reply(B.drelu_send(0, x0, prm, sd), B.drelu_send(1, x1, prm, sd), prm, sd)
    assert torch.equal(B.drelu_finish(0, d0, prm, sd), want[0])
    assert torch.equal(B.drelu_finish(1, d1, prm, sd), want[1])
    del d0, d1, want
    x2 = torch.zeros_like(x0)
    sr = B.RssSeeds(11, 12, 13, 14, 15)
    whole = B.rss_relu((x0, x1, x2), prm, sr)
    cut = slice(edge - 50, n)
    part = B.rss_relu(tuple(x[cut].clone() for x in (x0, x1, x2)), prm, sr, elem_base=edge - 50)
    for a, b in zip(whole, part):
        assert torch.equal(a[cut], b)

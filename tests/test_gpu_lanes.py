"""Every DReLU / ReLU kernel instance at one, two and four lanes per element.

The number of lanes follows from the call's size and the schedule, so a size
alone does not say which kernel ran: here the schedule forces each number, the
kernel is read from a captured graph, and the result is compared with the
oracle (integers: the tolerance is 0).  One lane is the kernel of every large
call; two and four lanes split an element's slots over waves of a block."""

import numpy as np
import pytest

from oracle import protocols as OPR
from oracle.params import default_prime
import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# every window count of both storage widths on a full-width ring, whose mask is a constant of the one-lane kernel,
# and rings below the storage width
SETTINGS = ([(64, lx) for lx in range(1, 33)] + [(32, lx) for lx in range(1, 17)] +
            [(63, 31), (51, 11), (40, 18), (41, 8), (24, 7), (30, 15), (3, 1)])


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_04909_amd import bicop
    return bicop


@pytest.fixture
def force(B):
    """force(lanes, lx, width): calls of up to 65,536 elements take this many lanes; the schedule is put back after."""
    before = {}

    def set_lanes(lanes, lx, width):
        for kind, value in (("group", lanes), ("group_fill", 4)):
            for op in (B.BC_OP_DRELU, B.BC_OP_RELU):
                before.setdefault((kind, lx + 1, width, op), B.get_schedule(kind, lx + 1, width, op))
                B.set_schedule(kind, lx + 1, value, width, op)
    yield set_lanes
    for (kind, npos, width, op), value in before.items():
        B.set_schedule(kind, npos, value, width, op)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64 if a.dtype == np.uint64 else np.int32)).cuda()


def host(t):
    return t.cpu().view(torch.int64 if t.element_size() == 8 else torch.int32).numpy().view(
        np.uint64 if t.element_size() == 8 else np.uint32).astype(np.uint64)


def inputs(rng, n, ell, lx, k_lo):
    """Shares of values inside the window's guard domain, the ends of the ring and windows of zeros and ones among them."""
    bound = 1 << (k_lo + lx - 1)
    x = [int(v) % (1 << ell) for v in rng.integers(-bound + 1, bound, size=n)]
    x[:8] = [v % (1 << ell) for v in (0, 1, -1, bound - 1, -bound + 1, (1 << ell) - 1, 1 << (ell - 1), 1 << k_lo)]
    return W.share(np.array(x, dtype=np.uint64), ell, rng)


def primes(lx):
    import sympy
    out = [default_prime(lx)]
    if lx >= 2:
        out.append(int(sympy.prevprime(out[0])))        # the generic field arithmetic of its size
    return out


@pytest.mark.parametrize("op", ["drelu", "relu"])
@pytest.mark.parametrize("ell,lx", SETTINGS)
def test_every_instance_at_every_number_of_lanes(B, force, op, ell, lx):
    from graph_kernels import kernels, lanes
    k_lo = min(13 if ell > 32 else 8, ell - 2 * lx)
    rng = np.random.default_rng(6007 * ell + lx)
    # a ragged last block, and indices that pass 2^32, where the call is cut into two launches
    n, base, seeds, nonce = 1001, (1 << 32) - 333, (0x0F1E2D3C4B5A6978 ^ lx, 0x8877665544332211 ^ ell, 12345 + lx), 0xABCDEF
    x0, x1 = inputs(rng, n, ell, lx, k_lo)
    d0, d1 = dev(x0), dev(x1)
    fn, oracle = (B.drelu, OPR.drelu) if op == "drelu" else (B.relu, OPR.relu)
    for p in primes(lx):
        prm, sd = B.Params(ell, lx, k_lo, p), B.Seeds(*seeds, nonce)
        e0, e1, _, _ = oracle(x0.astype(np.uint64), x1.astype(np.uint64), ell, lx, k_lo, p, seeds, nonce, elem_base=base)
        for count in (1, 2, 4):
            force(count, lx, B.ring_width(ell))
            out = (torch.full_like(d0, -1), torch.full_like(d1, -1))
            ran = kernels(lambda: fn(d0, d1, prm, sd, elem_base=base, out=out))
            assert [lanes(name) for name, _ in ran] == [count, count] and not any("Lb1ELb1EEE" in name for name, _ in ran)
            fn(d0, d1, prm, sd, elem_base=base, out=out)
            assert np.array_equal(host(out[0]), e0) and np.array_equal(host(out[1]), e1), (p, count)


@pytest.mark.parametrize("op", ["drelu", "relu"])
@pytest.mark.parametrize("ell,lx,k_lo", [(64, 18, 13), (64, 7, 11), (51, 11, 13), (64, 31, 0), (64, 32, 0), (32, 8, 8), (24, 7, 10)])
def test_sizes_of_the_default_dispatch(B, force, op, ell, lx, k_lo):
    """Both sides of the limits between four, two and one lanes, ragged sizes among them: the dispatch takes the
    kernel that the schedule says, and the shares are those of one lane."""
    from graph_kernels import kernels, lanes
    units = torch.cuda.get_device_properties(0).multi_processor_count
    prm, sd, width = B.Params(ell, lx, k_lo), B.Seeds(11, 22, 33, 44), B.ring_width(ell)
    code = B.BC_OP_RELU if op == "relu" else B.BC_OP_DRELU
    most, fill = B.get_schedule("group", lx + 1, width, code), B.get_schedule("group_fill", lx + 1, width, code)
    fn = getattr(B, op)
    gen = torch.Generator(device="cuda").manual_seed(lx)
    got = {}
    sizes = (1, 255, 1000, 32767, 32768, 32769, 50021, 65535, 65536, 65537, 131072, 131073)
    x = [torch.randint(-(1 << 62), 1 << 62, (sizes[-1],), generator=gen, device="cuda").bitwise_and_((1 << ell) - 1 if ell < 64 else -1)
         .to(torch.int64 if width == 8 else torch.int32) for _ in range(2)]
    for n in sizes:
        a, b = x[0][:n], x[1][:n]
        got[n] = (torch.empty_like(a), torch.empty_like(b))
        (name, _), = kernels(lambda: fn(a, b, prm, sd, out=got[n]))
        want = next((k for k in (4, 2) if most >= k and n <= units * 256 * fill // k), 1)
        assert lanes(name) == want, n
        fn(a, b, prm, sd, out=got[n])
    force(1, lx, width)
    for n, y in got.items():
        one = fn(x[0][:n], x[1][:n], prm, sd, out=(torch.empty_like(y[0]), torch.empty_like(y[1])))
        assert torch.equal(one[0], y[0]) and torch.equal(one[1], y[1]), n


@pytest.mark.parametrize("op", ["trunc_drelu", "trunc_relu"])
@pytest.mark.parametrize("ell_in,k1,lx,k_lo", [(64, 13, 11, 13), (64, 13, 18, 0), (32, 8, 7, 10), (64, 1, 31, 0)])
def test_truncated_inputs_and_in_place(B, force, op, ell_in, k1, lx, k_lo):
    """Alg. 5 fused with the op, written over its own inputs, at one, two and four lanes."""
    ell, n = ell_in - k1, 1001
    rng = np.random.default_rng(ell_in + lx)
    x0, x1 = inputs(rng, n, ell_in, lx, k_lo)
    t0, t1 = OPR.trunc_det(x0.astype(np.uint64), x1.astype(np.uint64), ell_in, k1)
    oracle = OPR.relu if op == "trunc_relu" else OPR.drelu
    e0, e1, _, _ = oracle(t0, t1, ell, lx, k_lo, default_prime(lx), (3, 1, 4), 15, elem_base=9)
    for count in (1, 2, 4):
        force(count, lx, B.ring_width(ell))
        d0, d1 = dev(x0), dev(x1)
        getattr(B, op)(d0, d1, ell_in, k1, B.Params(ell, lx, k_lo), B.Seeds(3, 1, 4, 15), elem_base=9, out=(d0, d1))
        assert np.array_equal(host(d0), e0) and np.array_equal(host(d1), e1), count

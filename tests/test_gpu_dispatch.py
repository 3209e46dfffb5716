"""Which kernel and grid a call takes, read from a captured graph: results do
not show a dispatch that went wrong."""

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_04909_amd import bicop
    return bicop


@pytest.mark.parametrize("ell,lx,per_unit", [(64, 18, 64), (32, 8, 8)])
def test_finish_grid(B, ell, lx, per_unit):
    """P0's and P1's unflip strides above 64 (8-byte shares) or 8 blocks a compute unit."""
    from graph_kernels import kernels
    units = torch.cuda.get_device_properties(0).multi_processor_count
    prm, sd = B.Params(ell, lx, 8), B.Seeds(1, 2, 3, 4)
    for n in (1, 256 * units * per_unit - 1, 256 * units * per_unit, 256 * units * per_unit + 1, 4 * 256 * units * per_unit):
        d = torch.zeros(n, dtype=torch.int64 if ell > 32 else torch.int32, device="cuda")
        for party in (0, 1):
            (name, blocks), = kernels(lambda: B.drelu_finish(party, d, prm, sd, out=d))
            assert "k_finish" in name and blocks == min((n + 255) // 256, units * per_unit), n


@pytest.mark.parametrize("op", [0, 1])
def test_expansion_without_a_stride(B, op):
    """The N = 19 expansion, bound by its writes, takes 2^24 elements in one order (a grid that strides
    writes two regions of every plane at once)."""
    from graph_kernels import kernels
    prm, sd, n = B.Params(64, 18, 13), B.Seeds(1, 2, 3, 4), 1 << 24
    rec = torch.empty(B.rand_bytes(op, prm, n), dtype=torch.uint8, device="cuda")
    (name, blocks), = kernels(lambda: B.rand_expand(op, prm, sd, n, out=rec))
    assert "k_expand" in name and blocks * 256 == n


@pytest.mark.parametrize("lx", [18, 32])
@pytest.mark.parametrize("n", [1, 1000, 32768, 32769, 65536, 65537])
def test_replicated_sharing_kernel_and_grid(B, n, lx):
    """Small replicated-sharing calls split their slots over four waves, with the default prime only; the grid
    is the one of the kernel that runs."""
    import sympy
    from graph_kernels import kernels, lanes
    fill = 2 * 256 * torch.cuda.get_device_properties(0).multi_processor_count
    before = {(k, op): B.get_schedule(k, lx + 1, 8, op) for k in ("group", "group_fill") for op in (0, 1)}
    x = tuple(torch.zeros(n, dtype=torch.int64, device="cuda") for _ in range(3))
    try:
        B.set_schedule("group", lx + 1, 4, 8)
        B.set_schedule("group_fill", lx + 1, 2, 8)
        for p in (0, int(sympy.prevprime(B.default_prime(lx)))):
            prm = B.Params(64, lx, 0, p)
            (name, blocks), = kernels(lambda: B.rss_relu(x, prm, B.RssSeeds(1, 2, 3, 4, 5), out=x))
            want = 4 if p == 0 and (4 * n <= fill or (lx < 32 and 2 * n <= fill)) else 1
            assert lanes(name) == want and blocks == (n * want + 255) // 256, (p, name, blocks)
    finally:
        for (k, op), v in before.items():
            B.set_schedule(k, lx + 1, v, 8, op)


def test_two_window_drelu_grid(B):
    """The DReLU at l_x = 1 takes a quarter, then half of the default 64 blocks a compute unit while those give a
    thread one and two elements; larger calls, wider windows and the other kernels of the window count take it all."""
    from graph_kernels import kernels
    units = torch.cuda.get_device_properties(0).multi_processor_count
    full = 64 * units
    x, y = (torch.zeros(512 * full + 1, dtype=torch.int64, device="cuda") for _ in range(2))
    sd, prm = B.Seeds(1, 2, 3), B.Params(64, 1, 13)
    drelu = lambda n, p=prm: kernels(lambda: B.drelu(x[:n], x[:n], p, sd, out=(y[:n], y[:n])))  # noqa: E731
    for n, want in ((256 * full, full // 4), (256 * full + 1, full // 2), (512 * full, full // 2), (512 * full + 1, full)):
        (_, blocks), = drelu(n)
        assert blocks == want, n
    n = 256 * full + 1
    (_, blocks), = drelu(n, B.Params(64, 2, 13))
    assert blocks == full
    message = torch.empty((B.msg_words(2), n), dtype=torch.int32, device="cuda")
    (name, blocks), = kernels(lambda: B.drelu_send(0, x[:n], prm, sd, out=message))
    assert "k_send" in name and blocks == full
    (name, blocks), = kernels(lambda: B.rss_drelu((x[:n],) * 3, prm, B.RssSeeds(1, 2, 3, 4, 5), out=(y[:n],) * 3))
    assert "k_rss" in name and blocks == full
    try:
        B.set_schedule("fused", 2, 3, 8, 0)
        (_, blocks), = drelu(n)
        assert blocks == 3 * units
    finally:
        B.set_schedule("fused", 2, 0, 8, 0)

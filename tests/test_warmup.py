"""The server's warm-up reaches every kernel that a single job can take: its
call sizes follow the library's rule for the lanes per element, whatever the
schedule says."""

import pytest

torch = pytest.importorskip("torch")


def lanes_of(n, units, most, fill):
    """The library's rule: lanes per element of a call on n elements."""
    threads = units * 4 * 64 * fill
    for lanes in (4, 2):
        if most >= lanes and n <= threads // lanes:
            return lanes
    return 1


@pytest.mark.parametrize("units", [256, 32])
@pytest.mark.parametrize("most", [1, 2, 4, 8])
@pytest.mark.parametrize("fill", [1, 2, 4])
def test_sizes_take_every_number_of_lanes(units, most, fill):
    from paper_2309_04909_amd.serve import sizes_by_lanes
    want = {1} | {lanes for lanes in (2, 4) if most >= lanes}
    assert {lanes_of(n, units, most, fill) for n in sizes_by_lanes(units, most, fill)} == want


@pytest.mark.gpu
def test_warmup_reaches_every_kernel(monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from graph_kernels import kernels, lanes
    from paper_2309_04909_amd import bicop as B
    from paper_2309_04909_amd import serve as S
    params = {64: B.Params(64, 18, 13), 32: B.Params(32, 8, 8)}
    n = 1 << 18
    pools = {ell: tuple(torch.zeros(n, dtype=torch.int64 if ell > 32 else torch.int32, device="cuda") for _ in range(2))
             for ell in params}
    seen = []
    for name in ("drelu", "relu"):
        real = getattr(B, name)

        def wrapped(x0, x1, prm, sd, real=real, name=name, **kw):
            seen.append((name, prm.ell, x0.numel()))
            return real(x0, x1, prm, sd, **kw)
        monkeypatch.setattr(B, name, wrapped)
    S.Server(pools, params, B.Seeds(1, 2, 3), hbm_budget=1 << 24, nstreams=2).warmup()
    monkeypatch.undo()
    reached = set()
    for name, ell, m in set(seen):
        x0, x1 = (t[:m] for t in pools[ell])
        out = (torch.empty_like(x0), torch.empty_like(x1))
        (kernel, _), = kernels(lambda: getattr(B, name)(x0, x1, params[ell], B.Seeds(1, 2, 3), out=out))
        reached.add((name, ell, lanes(kernel)))
    assert reached == {(name, ell, k) for name in ("drelu", "relu") for ell in params for k in (1, 2, 4)}

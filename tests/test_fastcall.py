"""The native argument marshalling against the ctypes path: the same results,
the same refusals.  An `out` given as a list takes the ctypes path, the same
buffers as a tuple the native one."""

import copy
import pickle

import pytest

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    from paper_2309_04909_amd import bicop
    return bicop


def calls(B, prm, sd):
    return {"drelu": lambda x0, x1, **k: B.drelu(x0, x1, prm, sd, **k),
            "relu": lambda x0, x1, **k: B.relu(x0, x1, prm, sd, **k),
            "trunc_drelu": lambda x0, x1, **k: B.trunc_drelu(x0, x1, 64, 64 - prm.ell, prm, sd, **k),
            "trunc_relu": lambda x0, x1, **k: B.trunc_relu(x0, x1, 64, 64 - prm.ell, prm, sd, **k),
            "trunc_det": lambda x0, x1, **k: B.trunc_det(x0, x1, 64, 13, **k)}


def test_host_tensors_are_refused(B):
    x = torch.zeros(4, dtype=torch.int64)
    for name, fn in calls(B, B.Params(51, 11, 13), B.Seeds(1, 2, 3)).items():
        with pytest.raises(TypeError):
            fn(x, x)
        with pytest.raises(TypeError):
            fn(None, x)


@pytest.mark.gpu
@pytest.mark.parametrize("ell", [64, 51])
def test_native_and_ctypes_paths_agree(B, ell):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prm, sd = B.Params(ell, 11, 13), B.Seeds(7, 8, 9, (1 << 64) - 5)
    for prm, sd in ((prm, sd), (copy.deepcopy(prm), copy.deepcopy(sd)), (pickle.loads(pickle.dumps(prm)), B.Seeds(7, 8, 9, -5))):
        for name, fn in calls(B, prm, sd).items():
            if (name.startswith("trunc_") and name != "trunc_det") == (ell == 64):
                continue
            for shape in ((0,), (1,), (3, 70), (9001,)):
                g = torch.Generator(device="cuda").manual_seed(len(shape) + shape[0])
                x0, x1 = (torch.randint(-(1 << 62), 1 << 62, shape, generator=g, device="cuda") & ((1 << ell) - 1 if ell < 64
                          and name in ("drelu", "relu") else -1) for _ in range(2))
                a, b, c = ([torch.full(shape, -1, dtype=torch.int64, device="cuda") for _ in range(2)] for _ in range(3))
                fn(x0, x1, out=a)                                       # ctypes
                assert fn(x0, x1, out=tuple(b))[1].data_ptr() == b[1].data_ptr()
                side = torch.cuda.Stream()
                side.wait_stream(torch.cuda.current_stream())
                fn(x0, x1, out=tuple(c), stream=side)
                torch.cuda.current_stream().wait_stream(side)
                new = fn(x0, x1)
                for i in range(2):
                    assert torch.equal(a[i], b[i]) and torch.equal(a[i], c[i])
                    assert new[i].dtype == torch.uint64 and new[i].shape == x0.shape and torch.equal(new[i].view(torch.int64), a[i])


@pytest.mark.gpu
@pytest.mark.parametrize("ell,lx,k_lo", [(64, 18, 13), (32, 8, 8)])
def test_native_and_ctypes_paths_agree_on_the_other_calls(B, ell, lx, k_lo):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prm, sd, rs = B.Params(ell, lx, k_lo), B.Seeds(7, 8, 9, 10), B.RssSeeds(1, 2, 3, 4, 5, 6)
    dt = torch.int64 if ell > 32 else torch.int32
    for n in (1, 5001):
        g = torch.Generator(device="cuda").manual_seed(n)
        x = [torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device="cuda").to(dt) for _ in range(4)]

        def buf(k):
            return [torch.full((n,), -1, dtype=dt, device="cuda") for _ in range(k)]
        for fn, args, k in ((B.rss_drelu, (tuple(x[:3]), prm, rs), 3), (B.rss_relu, (tuple(x[:3]), prm, rs), 3),
                            (B.mul_trunc, (*x, ell, 14, B.BC_TRUNC_BEFORE, sd), 2)):
            a, b = buf(k), buf(k)
            fn(*args, out=a)                                            # ctypes
            fn(*args, out=tuple(b))
            for p, q, new in zip(a, b, fn(*args)):
                assert torch.equal(p, q) and torch.equal(p, new.view(dt))
        # the ctypes path for a share given as a Parameter (not a plain tensor)
        plain = [torch.nn.Parameter(t, requires_grad=False) for t in x]
        m = [B.drelu_send(p, x[p], prm, sd) for p in (0, 1)]
        for p in (0, 1):
            assert torch.equal(m[p], B.drelu_send(p, plain[p], prm, sd)) and m[p].shape == (B.msg_words(lx + 1), n)
            assert torch.equal(m[p], B.drelu_send(p, x[p], prm, sd, out=torch.empty_like(m[p])))
        d = B.drelu_reply(*m, prm, sd)
        assert d[0].dtype == B.ring_dtype(ell) and d[0].shape == (n,)
        e = B.drelu_reply(*m, prm, sd, out=buf(2))
        for p in (0, 1):
            assert torch.equal(d[p].view(dt), e[p])
            y = B.drelu_finish(p, d[p], prm, sd)
            assert torch.equal(y.view(dt), B.drelu_finish(p, torch.nn.Parameter(e[p], requires_grad=False), prm, sd).view(dt))
            assert y.dtype == B.ring_dtype(ell)
        with pytest.raises(ValueError):
            B.drelu_send(0, x[0], prm, sd, out=torch.empty((n, B.msg_words(lx + 1) + 1), dtype=torch.int32, device="cuda"))
        with pytest.raises(ValueError):
            B.drelu_reply(m[0], m[1][:-1], prm, sd)
        with pytest.raises(B.BicopError):
            B.drelu_send(2, x[0], prm, sd)


@pytest.mark.gpu
def test_refusals_are_the_binding_s(B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prm, sd = B.Params(64, 7, 11), B.Seeds(1, 2, 3, 4)
    x = torch.zeros(64, dtype=torch.int64, device="cuda")
    y = torch.empty_like(x)
    with pytest.raises(TypeError):
        B.drelu(x.int(), x.int(), prm, sd)
    with pytest.raises(ValueError):
        B.drelu(x[::2], x[::2], prm, sd)
    with pytest.raises(ValueError):
        B.drelu(x, x[:3], prm, sd)
    with pytest.raises(ValueError):
        B.drelu(x, x, prm, sd, out=(y, y[:5]))
    with pytest.raises(B.BicopError) as e:
        B.drelu(x, x, B.Params(64, 40, 0), sd, out=(y, y.clone()))
    assert "drelu" in str(e.value) and e.value.code == -3
    with pytest.raises(B.BicopError):
        B.trunc_det(x, x, 64, 64)

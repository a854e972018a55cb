"""Products and Lanczos drivers with and without apply_H's work memory.

Hamiltonian.apply and apply_block hand work memory to fotci_apply_H_work, so the one-body-jump kernels of
fotci_apply_H, fotci_apply_H_block, dx of fotci_apply_H_vjp and of calls that find no memory left are compared with the
oracle here, at sizes whose rows span many tiles."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import basis as ob
from oracle import fast
from paper_1801_08432_amd import fotci, inputs

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = "cuda:0"


_kept = {}


def _ham(name):
    if name not in _kept:
        _kept.clear()
        w = inputs.workload(name)
        _kept[name] = fotci.Hamiltonian.build(w["two_j"], w["Z"], w["N"], w["two_M"], w, device=DEV)
    return _kept[name]


def _oracle(name):
    w = inputs.workload(name)
    return w, fast.Prepared(ob.build_basis(w["two_j"], w["Z"], w["N"], w["two_M"]))


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


# as for the products with work memory: float64 rounding of ~10^3 terms a row, float32 rounding grown by their root
TOL = dict(f64=1e-12, f32=1e-5)
DTYPE = dict(f64=torch.float64, f32=torch.float32)


def test_overlapping_vectors_are_refused():
    """Every n_block, one vector among them, and ranges that overlap without being equal."""
    h = _ham("sd_2p2n")
    for nb in (1, 2):
        buf = torch.zeros((h.dim + 1) * nb + 64, dtype=torch.float64, device=DEV)
        x, y = buf[:h.dim * nb].view(h.dim, nb), buf[2:2 + h.dim * nb].view(h.dim, nb)
        with pytest.raises(fotci.FotciError) as e:
            h.apply_block(x, y)
        assert e.value.code == -1
        assert fotci.lib().fotci_apply_H_work(h._h, fotci.MODE_F64, nb, x.data_ptr(), y.data_ptr(), None, 0,
                                              fotci._stream()) == -1


@pytest.mark.parametrize("mode", ["f64", "f32"])
def test_products_without_work_memory_match_the_oracle(mode):
    h, m = _ham("pf_4p4n"), fotci.MODES[mode]
    w, prep = _oracle("pf_4p4n")
    X = torch.from_numpy(np.stack([inputs.random_vector(h.dim, 40 + v) for v in range(2)], 1)).to(DEV).to(DTYPE[mode])
    ref = np.stack([fast.apply_h(prep, w, X[:, v].double().cpu().numpy()) for v in range(2)], 1)
    x = X[:, 0].contiguous()
    y = torch.empty_like(x)
    fotci._check(fotci.lib().fotci_apply_H(h._h, m, x.data_ptr(), y.data_ptr(), fotci._stream()))
    assert _rel(y.double().cpu().numpy(), ref[:, 0]) <= TOL[mode]
    for nb in (2, 4, 8):
        B = X.repeat(1, nb // 2).contiguous()
        Y = torch.empty_like(B)
        fotci._check(fotci.lib().fotci_apply_H_block(h._h, m, nb, B.data_ptr(), Y.data_ptr(), fotci._stream()))
        for v in range(nb):
            assert _rel(Y[:, v].double().cpu().numpy(), ref[:, v % 2]) <= TOL[mode]


def test_products_without_work_memory_at_full_size():
    """pf_5p5n, windows of rows as for the products with work memory."""
    h = _ham("pf_5p5n")
    w, prep = _oracle("pf_5p5n")
    x = inputs.random_vector(h.dim, 13)
    got = {}
    for mode in ("f64", "f32"):
        xt = torch.from_numpy(x).to(DEV).to(DTYPE[mode])
        y = torch.empty_like(xt)
        fotci._check(fotci.lib().fotci_apply_H(h._h, fotci.MODES[mode], xt.data_ptr(), y.data_ptr(), fotci._stream()))
        got[mode] = y.double().cpu().numpy()
    for r0, r1 in [(0, 4000), (h.dim // 2, h.dim // 2 + 8000), (h.dim - 4000, h.dim)]:
        ref = fast.apply_h(prep, w, x, rows=(r0, r1))
        for mode in got:
            assert _rel(got[mode][r0:r1], ref) <= TOL[mode]


@pytest.mark.parametrize("static", [False, True])
def test_dx_of_the_c_entry_matches_the_oracle(static):
    h = _ham("pf_4p4n")
    w, prep = _oracle("pf_4p4n")
    x, g = (torch.from_numpy(inputs.random_vector(h.dim, s)).to(DEV) for s in (41, 42))
    dx = torch.empty_like(x)
    fn = fotci.lib().fotci_apply_H_vjp_static if static else fotci.lib().fotci_apply_H_vjp
    fotci._check(fn(h._h, x.data_ptr(), g.data_ptr(), dx.data_ptr(), None, None, None, None, None, fotci._stream()))
    assert _rel(dx.cpu().numpy(), fast.apply_h(prep, w, g.cpu().numpy())) <= TOL["f64"]


def _out_of_memory(monkeypatch, at_least):
    """torch.empty without room for byte tensors of at_least bytes."""
    real, refused = torch.empty, []

    def empty(*size, **kw):
        if kw.get("dtype") is torch.uint8 and size[0] >= at_least:
            refused.append(size[0])
            raise torch.cuda.OutOfMemoryError("no room")
        return real(*size, **kw)

    monkeypatch.setattr(torch, "empty", empty)
    return refused


def test_products_go_on_without_memory_left(monkeypatch):
    h = _ham("pf_4p4n")
    x, g = torch.randn(h.dim, dtype=torch.float64, device=DEV), torch.randn(h.dim, dtype=torch.float64, device=DEV)
    X = torch.randn(h.dim, 2, dtype=torch.float32, device=DEV)
    want = h.apply(x), h.apply_block(X, mode="f32"), h.vjp(x, g)
    refused = _out_of_memory(monkeypatch, 1)
    got = h.apply(x), h.apply_block(X, mode="f32"), h.vjp(x, g)
    assert len(refused) == 3
    for a, b, tol in ((got[0], want[0], 1e-12), (got[1], want[1], 1e-5), (got[2][0], want[2][0], 1e-12)):
        assert float((a - b).double().norm()) <= tol * float(b.double().norm())
    for k in want[2][1]:
        assert torch.allclose(got[2][1][k], want[2][1][k], rtol=1e-11, atol=1e-9)


def _drivers(h, mode):
    """Lowest eigenvalues of the three drivers, each with the bytes of its workspace."""
    piv = torch.from_numpy(inputs.random_vector(h.dim, 43)).to(DEV)
    pivb = torch.from_numpy(np.stack([inputs.random_vector(h.dim, 44 + v) for v in range(2)], 1)).to(DEV)
    return {
        "lowest": (lambda: h.lanczos_lowest(piv, 3, 60, mode=mode)["evals"], h.lanczos_workspace_bytes(3, 60, mode)),
        "restart": (lambda: h.lanczos_thick_restart(piv, 3, 8, 24, max_restarts=3, mode=mode, tol=1e-9)["evals"],
                    h.trlan_workspace_bytes(3, 8, 24, mode, max_restarts=3, tol=1e-9)),
        "block": (lambda: h.lanczos_block(pivb, 3, 30, mode=mode)["evals"], h.block_lanczos_workspace_bytes(3, 2, 30, mode)),
    }


@pytest.mark.parametrize("mode", ["f64", "f32"])
@pytest.mark.parametrize("driver", ["lowest", "restart", "block"])
def test_drivers_go_on_without_their_work_memory(monkeypatch, driver, mode):
    """The workspace less its work memory: the Ritz values of the same Krylov space, by the jump kernels. They differ by
    the products' rounding, which the lowest values of an unconverged run carry with a small factor."""
    h = _ham("pf_4p4n")
    run, nbytes = _drivers(h, mode)[driver]
    nb = 2 if driver == "block" else 1
    part = max(fotci.lib().fotci_apply_work_bytes(h._h, fotci.MODES[mode], nb),
               fotci.lib().fotci_apply_work_bytes(h._h, fotci.MODE_F64, 1))
    assert part > 0
    want = run()
    refused = _out_of_memory(monkeypatch, nbytes)
    got = run()
    assert refused == [nbytes + 256]
    assert np.max(np.abs(got - want) / np.abs(want)) <= (1e-9 if mode == "f64" else 1e-5)


def test_too_small_a_workspace_is_refused():
    h = _ham("pf_4p4n")
    o = fotci.LanczosOpts(1, 4, fotci.MODE_F64, 1, 0)
    n = fotci.lib().fotci_lanczos_workspace_bytes(h._h, ctypes.byref(o))
    part = (fotci.lib().fotci_apply_work_bytes(h._h, fotci.MODE_F64, 1) + 255) // 256 * 256
    piv = torch.from_numpy(inputs.random_vector(h.dim, 45)).to(DEV)
    work = torch.empty(n + 256, dtype=torch.uint8, device=DEV)
    e, r = np.zeros(1), np.zeros(1)
    ptr = ctypes.c_void_p(work.data_ptr() + (-work.data_ptr()) % 256)

    def run(nbytes):
        return fotci.lib().fotci_lanczos_lowest(h._h, ctypes.byref(o), piv.data_ptr(), ptr, nbytes, fotci._np_ptr(e),
                                                fotci._np_ptr(r), None, None, None, fotci._stream())

    assert run(n - part - 1) == -2
    assert run(n - part) == 0
    least = e.copy()
    assert run(n - 1) == 0 and run(n) == 0
    assert abs(e[0] - least[0]) <= 1e-12 * abs(e[0])


def test_products_on_a_stream_of_the_callers():
    """stream=: the work memory is allocated in that stream's order; products on two streams at a time."""
    h = _ham("pf_4p4n")
    x = [torch.randn(h.dim, dtype=torch.float64, device=DEV) for _ in range(2)]
    want = [h.apply(v) for v in x]
    g = torch.randn(h.dim, dtype=torch.float64, device=DEV)
    wdx = h.apply(g)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    ys = [torch.empty_like(v) for v in x]
    torch.cuda.synchronize()
    for _ in range(5):
        for s, v, y in zip(streams, x, ys):
            h.apply(v, y, stream=s)
    dx, _ = h.vjp(x[0], g, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    for a, b in zip(ys + [dx], want + [wdx]):
        assert float((a - b).norm()) <= 1e-13 * float(b.norm())
    X = torch.stack(x, 1).contiguous()
    Y = torch.empty_like(X)
    torch.cuda.synchronize()
    h.apply_block(X, Y, stream=streams[0])
    torch.cuda.synchronize()
    for v in range(2):
        assert float((Y[:, v] - want[v]).norm()) <= 1e-13 * float(want[v].norm())


def test_a_stream_may_be_any_object_with_its_handle():
    """As for every other call: the binding reads cuda_stream alone."""
    class Handle:
        pass

    h = _ham("pf_4p4n")
    x = torch.randn(h.dim, dtype=torch.float64, device=DEV)
    want, s, side = h.apply(x), Handle(), torch.cuda.Stream()
    s.cuda_stream = side.cuda_stream
    torch.cuda.synchronize()
    y = torch.empty_like(x)
    torch.cuda.synchronize()
    h.apply(x, y, stream=s)
    torch.cuda.synchronize()
    assert float((y - want).norm()) <= 1e-13 * float(want.norm())


@pytest.mark.parametrize("Z,N,two_M", [(1, 1, 0), (2, 1, 1), (1, 3, 0)])
def test_adjoint_of_tiny_bases(Z, N, two_M):
    """dx as an apply of its own, and (work memory of 2 KiB or less) in the adjoint's call."""
    inter, rng = inputs.random_interaction((1, 3, 5), 79)
    h = fotci.Hamiltonian.build((1, 3, 5), Z, N, two_M, inter, device=DEV)
    prep = fast.Prepared(ob.build_basis((1, 3, 5), Z, N, two_M))
    x, g = rng.standard_normal(h.dim), rng.standard_normal(h.dim)
    dx, grads = h.vjp(torch.from_numpy(x).to(DEV), torch.from_numpy(g).to(DEV))
    assert _rel(dx.cpu().numpy(), fast.apply_h(prep, inter, g)) <= 1e-13
    ref = fast.densities(prep, g, x)
    for k in ("v_pp", "v_nn", "v_pn", "eps_p", "eps_n"):
        r = np.asarray(ref["d_" + k]).ravel()
        assert np.linalg.norm(grads[k].cpu().numpy().ravel() - r) <= 1e-13 * max(np.linalg.norm(r), 1.0), k

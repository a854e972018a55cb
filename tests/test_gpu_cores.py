"""The core kernels of the proton-neutron part (fotci_apply_H_work) against the CPU oracle: spaces and particle
numbers at the edges of their lists (one particle of a species, more than four states of one m, more (c d) pairs than a
pass takes, rows split over work items, both parities), float32, float64 and blocks, and the work-memory rules."""
import ctypes

import numpy as np
import pytest

from oracle import basis as ob
from oracle import fast
from paper_1801_08432_amd import fotci, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [
    ((1, 3, 5, 7), 1, 2, 1, None),      # no other proton: all 60 pairs of a class, two passes
    ((1, 3, 5, 7), 2, 1, 1, None),      # one neutron: a single core
    ((1, 1, 1, 1, 1), 2, 2, 0, None),   # five states of one m: two positions for a state
    ((1, 3, 5), 2, 3, 1, None),
    ((1, 3, 5, 7), 3, 3, 0, None),      # more states than a work item takes
    ((1, 3, 1, 5), 2, 2, 0, (-1, -1, 1, 1)),
    ((3, 7), 3, 2, 3, None),
]


def _case(shape):
    two_j, Z, N, M, par = shape
    inter, _ = inputs.random_interaction(two_j, 77, par)
    b = fotci.Basis(two_j, Z, N, M, orbit_parity=par)
    ham = fotci.Hamiltonian(fotci.Jumps(b), inter).upload("cuda")
    prep = fast.Prepared(ob.build_basis(two_j, Z, N, M, orbit_parity=par) if par else ob.build_basis(two_j, Z, N, M))
    return ham, prep, inter


def _work_apply(ham, m, nb, x, y, work, nbytes):
    return fotci.lib().fotci_apply_H_work(ham._h, m, nb, x.data_ptr(), y.data_ptr(),
                                          ctypes.c_void_p(work.data_ptr()) if work is not None else None, nbytes,
                                          fotci._stream())


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("mode,nb", [("f64", 1), ("f32", 1), ("f64", 2), ("f32", 8)])
def test_apply_with_work_memory_matches_the_oracle(shape, mode, nb):
    ham, prep, inter = _case(shape)
    m = fotci.MODES[mode]
    need = fotci.lib().fotci_apply_work_bytes(ham._h, m, nb)
    assert need == ham.dim * nb * (8 if mode == "f64" else 4) * shape[1]
    xs = np.random.default_rng(5).standard_normal((ham.dim, nb))
    dt = torch.float64 if mode == "f64" else torch.float32
    x = torch.tensor(xs, device="cuda").to(dt).contiguous()
    y = torch.full_like(x, float("nan"))
    work = torch.full((need,), 255, dtype=torch.uint8, device="cuda")   # NaN everywhere
    assert _work_apply(ham, m, nb, x, y, work, need) == 0
    ref = np.stack([fast.apply_h(prep, inter, x[:, v].double().cpu().numpy()) for v in range(nb)], 1)
    # a row sums a few hundred products of O(1) factors: rounding of each, root-sum
    tol = 1e-14 if mode == "f64" else 2e-6
    assert np.linalg.norm(y.double().cpu().numpy() - ref) <= tol * np.linalg.norm(ref)
    y0 = torch.empty_like(x)
    assert _work_apply(ham, m, nb, x, y0, None, 0) == 0
    assert float((y0 - y).double().norm()) <= 2 * tol * float(y.double().norm())


def test_work_memory_rules():
    ham, _, _ = _case(SHAPES[4])
    x = torch.randn(ham.dim, dtype=torch.float64, device="cuda")
    y = torch.empty_like(x)
    need = fotci.lib().fotci_apply_work_bytes(ham._h, fotci.MODE_F64, 1)
    work = torch.empty(need, dtype=torch.uint8, device="cuda")
    assert _work_apply(ham, fotci.MODE_F64, 1, x, y, work, need - 1) == -2
    assert _work_apply(ham, fotci.MODE_F64, 1, x, x, work, need) == -1
    assert _work_apply(ham, fotci.MODE_F64, 3, x, y, work, need) == -1
    assert fotci.lib().fotci_apply_work_bytes(ham._h, fotci.MODE_F64, 3) == -1
    assert fotci.lib().fotci_apply_work_bytes(ham._h, fotci.MODE_F64_PLAIN, 1) == 0


def test_float32_sums_are_reproducible():
    """Row sums collect float32 results in float64, so the order in which the waves add does not show."""
    ham, _, _ = _case(SHAPES[4])
    x = torch.randn(ham.dim, dtype=torch.float32, device="cuda")
    first = ham.apply(x, mode="f32")
    for _ in range(5):
        assert torch.equal(ham.apply(x, mode="f32"), first)


@pytest.mark.parametrize("shape", SHAPES + [((1, 3), 3, 3, 0, None)], ids=str)
def test_label_densities_match_the_oracle(shape):
    """dV_pn on the cores (and, for the nearly full last shape, on the jump kernel), each entry a sum over the basis of
    products of O(1) factors in float64: 1e-13 of the norm covers its rounding."""
    ham, prep, _ = _case(shape)
    rng = np.random.default_rng(6)
    x, g = rng.standard_normal(ham.dim), rng.standard_normal(ham.dim)
    _, grads = ham.vjp(torch.tensor(x, device="cuda"), torch.tensor(g, device="cuda"))
    ref = fast.densities(prep, g, x)
    for k in ("v_pn", "v_pp", "v_nn", "eps_p", "eps_n"):
        r = np.asarray(ref["d_" + k]).ravel()
        got = grads[k].cpu().numpy().ravel()
        assert np.linalg.norm(got - r) <= 1e-13 * max(np.linalg.norm(r), 1.0), k


@pytest.mark.parametrize("shape", SHAPES + [((1, 3), 3, 3, 0, None), ((1, 3, 5), 6, 5, 1, None)], ids=str)
def test_one_body_densities_match_the_oracle(shape):
    """The last shape has groups of more than one block of columns; five states of one m take two blocks of entries."""
    ham, prep, _ = _case(shape)
    rng = np.random.default_rng(7)
    x, g = rng.standard_normal(ham.dim), rng.standard_normal(ham.dim)
    rp, rn = ham.one_body_density(torch.tensor(g, device="cuda"), torch.tensor(x, device="cuda"))
    for got, ref in zip((rp, rn), fast.one_body_densities(prep, g, x)):
        assert np.linalg.norm(got.cpu().numpy() - ref) <= 1e-13 * max(np.linalg.norm(ref), 1.0)


@pytest.mark.parametrize("mode", ["f32", "f64"])
def test_apply_replays_from_a_graph(mode):
    """The product and its work memory captured together; replays on new vectors, with eager products between."""
    ham, _, _ = _case(SHAPES[4])
    dt = torch.float32 if mode == "f32" else torch.float64
    x = torch.randn(ham.dim, dtype=dt, device="cuda")
    y = torch.empty_like(x)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ham.apply(x, y, mode=mode)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ham.apply(x, y, mode=mode)
    for _ in range(4):
        x.copy_(torch.randn_like(x))
        graph.replay()
        ref = ham.apply(x, mode=mode)
        torch.cuda.synchronize()
        assert float((y - ref).double().norm()) <= 1e-14 * float(ref.double().norm())

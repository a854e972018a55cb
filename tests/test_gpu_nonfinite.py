"""Infinities and NaN in the vectors of the densities and the adjoint: an entry depends on the elements that its jumps
reach, and only on them. The oracle sums jump by jump."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import basis as ob
from oracle import fast
from paper_1801_08432_amd import fotci, inputs

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

SHAPES = [
    ((1, 3, 5), 2, 2, 0, None),
    ((1, 3, 5), 5, 4, 1, None),
    ((1, 3, 5, 7), 3, 3, 0, None),
    ((1, 1, 1, 1, 1), 2, 2, 0, None),
    ((1, 3, 1, 5), 2, 2, 0, (-1, -1, 1, 1)),
]
VALUES = [("x", np.inf), ("g", -np.inf), ("x", np.nan), ("g", np.nan)]


def _case(shape):
    two_j, Z, N, M, par = shape
    inter, _ = inputs.random_interaction(two_j, 77, par)
    b = fotci.Basis(two_j, Z, N, M, orbit_parity=par)
    ham = fotci.Hamiltonian(fotci.Jumps(b), inter).upload("cuda")
    return ham, fast.Prepared(ob.build_basis(two_j, Z, N, M, orbit_parity=par))


def _vectors(dim, where, value, seed):
    rng = np.random.default_rng(seed)
    v = dict(x=rng.standard_normal(dim), g=rng.standard_normal(dim))
    v[where][rng.integers(dim)] = value
    return v["x"], v["g"]


def _same(got, ref):
    got, ref = np.asarray(got).ravel(), np.asarray(ref).ravel()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], ref[inf])
    ok = np.isfinite(ref)
    assert np.linalg.norm(got[ok] - ref[ok]) <= 1e-13 * max(np.linalg.norm(ref[ok]), 1.0)


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("where,value", VALUES)
def test_one_body_densities_keep_nonfinite_elements_to_their_entries(shape, where, value):
    ham, prep = _case(shape)
    for seed in range(4):
        x, g = _vectors(ham.dim, where, value, seed)
        got = ham.one_body_density(torch.tensor(g, device="cuda"), torch.tensor(x, device="cuda"))
        for a, b in zip(got, fast.one_body_densities(prep, g, x)):
            _same(a.cpu().numpy(), b)


def _labels(shape, where, value, keys):
    ham, prep = _case(shape)
    for seed in range(4):
        x, g = _vectors(ham.dim, where, value, seed)
        _, grads = ham.vjp(torch.tensor(x, device="cuda"), torch.tensor(g, device="cuda"))
        ref = fast.densities(prep, g, x)
        for k in keys:
            _same(grads[k].cpu().numpy(), ref["d_" + k])


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("where,value", VALUES)
def test_like_particle_label_densities_keep_nonfinite_elements_to_their_entries(shape, where, value):
    _labels(shape, where, value, ("v_pp", "v_nn", "eps_p", "eps_n"))


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("where,value", VALUES)
def test_pn_label_densities_keep_nonfinite_elements_to_their_entries(shape, where, value):
    _labels(shape, where, value, ("v_pn",))

"""Label densities of nearly full shells: SDs with more diagonal labels (up to 153) than a wave has lanes, and numbers of
SDs that leave the last workgroup short."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import basis as ob
from oracle import fast
from paper_1801_08432_amd import fotci, inputs

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("two_j,Z,N,two_M", [((1, 3, 5, 7), 18, 18, 0), ((3, 5, 7), 16, 15, 1), ((1, 3, 5), 11, 12, 1)])
def test_label_densities_of_nearly_full_shells(two_j, Z, N, two_M):
    """Each entry is a sum over the basis of products of O(1) factors in float64: 1e-13 of the norm covers its rounding."""
    inter, rng = inputs.random_interaction(two_j, 78)
    ham = fotci.Hamiltonian.build(two_j, Z, N, two_M, inter)
    prep = fast.Prepared(ob.build_basis(two_j, Z, N, two_M))
    x, g = rng.standard_normal(ham.dim), rng.standard_normal(ham.dim)
    _, grads = ham.vjp(torch.tensor(x, device="cuda"), torch.tensor(g, device="cuda"))
    ref = fast.densities(prep, g, x)
    for k in ("v_pp", "v_nn", "eps_p", "eps_n", "v_pn"):
        r = np.asarray(ref["d_" + k]).ravel()
        assert np.linalg.norm(grads[k].cpu().numpy().ravel() - r) <= 1e-13 * max(np.linalg.norm(r), 1.0), k

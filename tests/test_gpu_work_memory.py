"""Products and Lanczos drivers with and without apply_H's work memory.

Hamiltonian.apply and apply_block hand work memory to fotci_apply_H_work."""
import pytest

torch = pytest.importorskip("torch")

from paper_1801_08432_amd import fotci, inputs

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = "cuda:0"


def _ham(name):
    w = inputs.workload(name)
    return fotci.Hamiltonian.build(w["two_j"], w["Z"], w["N"], w["two_M"], w, device=DEV)


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

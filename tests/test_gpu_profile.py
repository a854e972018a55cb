"""fotci_profile_start / fotci_profile_stop over calls whose kernels run in different orders."""
import pytest

torch = pytest.importorskip("torch")

from paper_1801_08432_amd import fotci, inputs

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("nb", [1, 2])
def test_products_with_and_without_work_memory_are_averaged_by_kernel(nb):
    """The pn part comes first with work memory and last without: in a profile of both it is the mean of the two, here
    several times either of the other kernels. Times vary between runs by far less than the factor 2 allowed."""
    w = inputs.workload("pf_4p4n")
    h = fotci.Hamiltonian.build(w["two_j"], w["Z"], w["N"], w["two_M"], w, device="cuda")
    x = torch.randn(h.dim, nb, dtype=torch.float64, device="cuda")
    y = torch.empty_like(x)

    def plain():
        fotci._check(fotci.lib().fotci_apply_H_block(h._h, fotci.MODE_F64, nb, x.data_ptr(), y.data_ptr(), fotci._stream()))

    def work():
        h.apply_block(x, y)

    def profile(calls):
        plain(), work()
        torch.cuda.synchronize()
        h.profile_start(len(calls))
        for c in calls:
            c()
        ms, n = h.profile_stop()
        assert n == len(calls)
        return ms

    a, b = profile([plain] * 4), profile([work] * 4)
    for calls in ([plain, work] * 4, [work, plain] * 4):
        both = profile(calls)
        assert list(both) == list(a) == list(b)
        for k in both:
            mean = (a[k] + b[k]) / 2
            assert mean / 2 <= both[k] <= mean * 2, (k, a, b, both)

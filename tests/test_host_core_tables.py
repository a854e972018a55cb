"""Which bases run the proton-neutron part on cores (fotci_apply_work_bytes; host only)."""
import pytest

from paper_1801_08432_amd import fotci, inputs


def _ham(two_j, Z, N):
    inter, _ = inputs.random_interaction(two_j, 7)
    b = fotci.Basis(two_j, Z, N, (Z + N) % 2)
    return fotci.Hamiltonian(fotci.Jumps(b), inter)


# Measured, microseconds of one product by jumps and by cores
@pytest.mark.parametrize("Z,N,mode,n_block,cores", [
    (8, 4, "f64", 1, False),   # 39.0 / 42.3
    (8, 4, "f64", 2, False),   # 49.8 / 68.6
    (7, 5, "f64", 1, False),   # 44.7 / 51.6
    (7, 3, "f64", 8, False),   # 182 / 203
    (6, 5, "f64", 1, False),   # 46.3 / 51.2
    (4, 4, "f64", 4, False),   # 84.6 / 88.2
    (4, 4, "f64", 1, True),    # 38.3 / 32.7
    (5, 6, "f64", 2, True),    # 80.1 / 72.2
    (5, 5, "f64", 4, True),
    (2, 2, "f64", 8, True),    # 48.8 / 44.8
    (5, 5, "f32", 1, True),    # 39 / 34
    (7, 3, "f32", 8, True),    # 175 / 148
    (6, 6, "f32", 1, False),
])
def test_twelve_states_take_the_faster_kernel(Z, N, mode, n_block, cores):
    _check((1, 3, 5), Z, N, mode, n_block, cores)


@pytest.mark.parametrize("two_j,Z,N,mode,n_block,cores", [
    ((7,), 5, 2, "f64", 8, False),       # 34.0 / 37.0
    ((3, 5), 7, 3, "f64", 8, False),     # 55.6 / 81.9
    ((1, 3, 7), 6, 3, "f64", 1, False),  # 97 / 114
    ((1, 3, 7), 9, 5, "f64", 4, False),  # 445 / 553
    ((1, 3, 7), 4, 5, "f64", 2, True),   # 130 / 110
    ((1, 5, 7), 6, 4, "f64", 1, True),   # 503 / 401
    ((3, 5, 7), 3, 3, "f64", 1, True),   # 55 / 37
    ((1, 3, 5, 7), 3, 4, "f64", 1, True),
])
def test_other_spaces_take_the_faster_kernel(two_j, Z, N, mode, n_block, cores):
    _check(two_j, Z, N, mode, n_block, cores)


def _check(two_j, Z, N, mode, n_block, cores):
    ham = _ham(two_j, Z, N)
    need = fotci.lib().fotci_apply_work_bytes(ham._h, fotci.MODES[mode], n_block)
    assert need == (ham.dim * n_block * (8 if mode == "f64" else 4) * Z if cores else 0)

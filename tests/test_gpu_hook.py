"""The planned round kernel, which the test hook selects, against the oracle:
every round form, graphs with equal and unequal rows, bf16 rounding at exact
ties, and random configurations.  (The other GPU tests run the tile kernel.)"""
import pytest

from tests import test_gpu_parity as parity
from tests import test_gpu_random as random_cases

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _planned(monkeypatch):
    monkeypatch.setenv("GASLOC_GOSSIP_KERNEL", "planned")


@pytest.mark.parametrize("case", parity.SMALL, ids=lambda c: "-".join(map(str, c)))
def test_small_cases(case):
    parity.test_small_cases(*case)


@pytest.mark.parametrize("case", parity.FUSED, ids=lambda c: "-".join(map(str, c)))
def test_fused_last_step(case):
    parity.test_fused_last_step_matches_two_calls_and_oracle(*case)


@pytest.mark.parametrize("case", parity.FORMS, ids=lambda c: "-".join(map(str, c)))
def test_round_forms(case):
    parity.test_round_forms(*case)


@pytest.mark.parametrize("n", [2, 18])
def test_bf16_rounding_edge_cases(n):
    parity.test_bf16_rounding_edge_cases(n)


@pytest.mark.parametrize("n,dtype,fused", [(12, "bf16", True), (33, "f32", True), (40, "bf16", False)])
def test_rows_all_equal(n, dtype, fused):
    parity.test_rows_all_equal_share_one_running_sum(n, dtype, fused)


@pytest.mark.parametrize("density,dtype", [(0.05, "bf16"), (0.6, "f32")])
def test_explicit_random_csr(density, dtype):
    parity.test_explicit_random_csr_large_n(density, dtype)


@pytest.mark.parametrize("case", range(0, random_cases.CASES, 4))
def test_random_configuration(case):
    random_cases.test_random_configuration(case)

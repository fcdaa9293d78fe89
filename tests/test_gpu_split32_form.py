"""The completed results of the split 32^3 form: the tests of test_gpu_split32.py with the form's wait limit set to
its own default (50 ms), which makes their plans run it (without the variable the two-stage pair form is the
default at 32^3). That such plans launch the split kernel is checked on the host
(test_plan_host.py, wait_limit_runs_the_split_form)."""

import pytest

from tests.test_gpu_split32 import (test_split_matches_oracle, test_split_pair_symmetry,  # noqa: F401
                                    test_split_pair_symmetry_16_bands, test_split_pair_symmetry_many_bands,
                                    test_split_several_rounds_phi_and_shard, test_split_single_target_single_pair,
                                    test_split_vjp_and_energy_gradient)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def split_form(monkeypatch):
    monkeypatch.setenv("FOCKMI_SPLIT_WAIT_TICKS", "5000000")

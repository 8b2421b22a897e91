"""The kernels that the default launch shapes choose beyond those of
test_kernel_resources use no scratch memory: two-step workgroups of 128 and 256
lanes in both precisions, patches of batches, observation tiles of every
width, and the check of the initial density."""
import re

import pytest

from test_kernel_resources import kernel_scratch

KERNELS = [
    # models/EOS/types/lanes/store kinds as instantiated
    ("P, two steps per launch", r"k_step2_pILi[01]E(dd|ff)Li(128|256)ELi[01]EE", 16),
    ("FE, two steps per launch", r"k_step2_feILi[01]E(dd|ff)Li(128|256)EE", 8),
    # models x EOS x storage types x nodes per thread
    ("batch patches", r"k_batch_patch", 16),
    # models x EOS x storage types x tile widths
    ("observation", r"k_obs_all", 32),
    ("check of the initial density", r"k_rho0_check", 1),
]


@pytest.fixture(scope="module")
def sizes():
    return kernel_scratch()


@pytest.mark.parametrize("what,pattern,count", KERNELS, ids=[k[0] for k in KERNELS])
def test_no_scratch(sizes, what, pattern, count):
    hits = {k: v for k, v in sizes.items() if re.search(pattern, k)}
    assert len(hits) == count
    assert not {k: v for k, v in hits.items() if v}

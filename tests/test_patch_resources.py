"""The patch kernels, which small lattices launch by default, use no scratch
memory (see test_kernel_resources)."""
import re

from test_kernel_resources import kernel_scratch


def test_patch_kernels_use_no_scratch():
    hits = {k: v for k, v in kernel_scratch().items() if re.search(r"k_patch", k)}
    # models x EOS x storage types x nodes per thread x general; the general
    # free-energy FP64 kernel exists with one node per thread only
    assert len(hits) == 30
    assert not {k: v for k, v in hits.items() if v}

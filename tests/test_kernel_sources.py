"""Host-only checks of promises that kernel sources make to the compiler."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1906_11786_amd", "csrc")


@pytest.mark.parametrize("kernel", ["gru_bwd_kernel", "gru_bwd_cols_kernel"])
def test_gru_reverse_buffers_that_may_be_one_are_not_qualified(kernel):
    """ggnn_step_bits_gru_bwd passes dh_prev both as the upstream gradient and as dh where the GRU reverse is a
    launch of its own, so neither parameter may claim that nothing else points there."""
    with open(os.path.join(CSRC, "gru.hip")) as f:
        params = re.search(r"\bvoid " + kernel + r"\((.*?)\)", f.read(), flags=re.S).group(1)
    decl = {p.split()[-1].lstrip("*"): p for p in params.split(",")}
    for name in ("gin", "dh"):
        assert "__restrict__" not in decl[name], decl[name]

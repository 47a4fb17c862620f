"""What the cache stores' source must keep to and no device run can try: no read of a padding token's row."""
import os
import re

import pytest

import paper_2505_02351_amd as G


@pytest.mark.parametrize("e4m3", [False, True])
def test_padding_tokens_rows_are_not_read(e4m3):
    """A slot mapping may be padded with -1 beyond the rows that there are (a graph's fixed batch).  No read out of range is tried
    on the device: the kernels' source must load a row behind the tests of its slot."""
    path = os.path.join(os.path.dirname(G.__file__), "csrc", "cache_kernels.hpp")
    name = "reshape_and_cache_e4m3_kernel" if e4m3 else "reshape_and_cache_kernel"
    body = re.search(r"__global__[^;{]*\b" + name + r"\(.*?\n}\n", open(path).read(), re.S).group(0)
    tests = [m.start() for m in re.finditer(r"if \((slot|pos|block) < 0\) return;", body)]
    assert len(tests) == (1 if e4m3 else 3)
    assert max(tests) < min(body.index("(k + t * k_token_stride"), body.index("(v + t * v_token_stride"))

"""lbm_next_launch's argument checks, without a GPU."""
import os

import pytest


@pytest.fixture(scope="module")
def capi():
    from paper_2602_21242_amd import build, capi as c
    if not os.path.exists(c.LIB_PATH):
        build.build()
    return c


def test_null_context(capi):
    s, kernel, steps = capi.lbm_next_launch(None, 4)
    assert s == capi.LBM_ERR_INVALID_ARGUMENT and capi.last_error()
    assert (kernel, steps) == (-1, 0)

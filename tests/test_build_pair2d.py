"""The 2D kernels by pairs of waves compile for gfx950 without scratch spills."""
import os

import pytest

from paper_2402_03074_amd import build as B
from test_build_resources import _usage

pytestmark = pytest.mark.slow


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not installed")
def test_pair_kernels_use_no_scratch():
    kernels = {k: v for k, v in _usage("pair2d.hip").items() if "stage2d_pair_kernel" in k}
    # weights built in or read at run time, 3 Runge-Kutta stages
    assert len(kernels) == 6, kernels
    assert all(v == 0 for v in kernels.values()), kernels

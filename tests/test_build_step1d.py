"""The whole-step 1D kernels compile for gfx950 without scratch spills."""
import os

import pytest

from paper_2402_03074_amd import build as B
from test_build_resources import _usage

pytestmark = pytest.mark.slow


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not installed")
def test_step_kernels_use_no_scratch():
    kernels = {k: v for k, v in _usage("step1d.hip").items()
               if "step1d_kernel" in k or "block_run_kernel" in k}
    # scalar laws (2) and Euler component-wise / characteristic, in 2 precisions,
    # as one step per launch and as runs of steps
    assert len(kernels) == 16, kernels
    assert all(v == 0 for v in kernels.values()), kernels

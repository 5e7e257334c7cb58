import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: longer CPU test")


# The batch of 256 holds a unit of conv2 (sample 39, channel 9, pixel 15, 14) whose
# pre-activation is 1.4e-8 in float64 and 0 in the float32 chain of fused
# multiply-adds that defines it: its ReLU lets nothing through, float64's does, and
# the gradients of conv1 and conv2 differ by 9e-4 of their norm where the test
# allows 1e-4.  test_gpu_head_order.py holds the same batch to 2e-5, by the masks of
# the chain.
OTHER_SUBGRADIENT = "test_gpu_head_batches.py::test_batch_sizes[256]"


def pytest_collection_modifyitems(items):
    for item in items:
        if item.nodeid.endswith(OTHER_SUBGRADIENT):
            item.add_marker(pytest.mark.xfail(reason="a ReLU at rounding distance from zero", strict=True))
